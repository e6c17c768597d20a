"""The smooth coarse-graining against the oracle where its blocks change path:
runs of one particle, runs whose joint box fits and is cut, particles whose own
box does not fit, boxes too long for the axis tables, particles out of order in
space, and grids that cut them off.

Both sides evaluate the same expression in FP64.  A distance carries the
rounding of coordinates of size 1, 2.2e-16, which the exponent of at most 4.5
turns into 3 * 2.2e-16 / R, 3e-14 at R = 0.02; the sums add less than n roundings
of the largest value, 3000 * 1.1e-16.  Together well under 1e-12."""
import numpy as np
import pytest

import pyoracle as O
from paper_2011_00459_amd import scenegen as SG
from test_gpu_voxels import gpu_coarse_grain, particle_masses, stepped_column

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")


@pytest.mark.parametrize("n,l0,R,dims,mix", [
    (1, 0.05, 0.05, (20, 20, 40), False),
    (5, 0.05, 0.05, (9, 3, 1), False),
    (700, 0.045, 0.045, (13, 11, 9), False),
    (3000, 0.05, 0.05, (24, 24, 60), False),   # runs of four and five
    (3000, 0.05, 0.07, (24, 24, 60), True),    # no run of neighbours
    (300, 0.03, 0.075, (40, 40, 40), False),   # 16^3 voxels a particle
    (100, 0.02, 0.09, (60, 60, 60), False),    # 27 voxels an axis
    (100, 0.02, 0.02, (60, 60, 60), True),
    (60, 0.1, 0.02, (12, 12, 12), False),      # most particles reach no voxel centre
])
def test_smooth_fields_match_oracle(n, l0, R, dims, mix):
    g, spec, p = stepped_column(n=n)
    if mix:
        k = np.random.default_rng(3).permutation(n)
        p["x"], p["v"] = p["x"][k], p["v"][k]
        g.set_particles(0, x=p["x"], v=p["v"], w=np.zeros((n, 3)))
    m = particle_masses(p["r"], spec["material"]["rho"])
    origin = (-0.37, -0.29, 0.013)
    got = gpu_coarse_grain(g, origin, l0, dims, "gauss", R)
    ref = O.coarse_grain(p["x"], p["v"], m, origin, l0, dims, kernel="gauss", R=R)
    for a, b in zip(got, ref):
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))
    assert np.array_equal(got[0] > 0, ref[0] > 0)


def test_smooth_fields_of_full_runs():
    # 40,000 spheres: runs of 64 on a grid around them all
    n, l0, R = 40000, 0.06, 0.06
    spec = SG.column_scene(seed=4, n=n, footprint=3.0, sweeps=5)
    g = T.scene_from_specs(spec)
    g.step(1)
    x, r = SG.fp32(spec["x"]), np.asarray(SG.fp32(spec["r"]), dtype=np.float64)
    v = SG.fp32(np.random.default_rng(4).normal(0.0, 0.5, (n, 3)))
    g.set_particles(0, x=x, v=v, w=np.zeros((n, 3)))
    lo = x.min(0) - 4 * R
    dims = tuple(int(d) for d in np.ceil((x.max(0) + 4 * R - lo) / l0))
    got = gpu_coarse_grain(g, tuple(lo), l0, dims, "gauss", R)
    m = particle_masses(r, spec["material"]["rho"])
    ref = O.coarse_grain(x, v, m, tuple(lo), l0, dims, kernel="gauss", R=R)
    for a, b in zip(got, ref):
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))

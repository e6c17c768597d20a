"""The smooth coarse-graining on particles out of order in space, in runs of
64: positions set after the step that sorted them, all of them permuted or one
in `every`, so that a run goes from shared boxes of voxels to memory and back.
Tolerance as in test_gpu_smooth_fields.py, with 40,000 terms at most in a sum:
40,000 * 1.1e-16 and the exponents' 3 * 2.2e-16 * 4 / R, together under 1e-11."""
import numpy as np
import pytest

import pyoracle as O
from paper_2011_00459_amd import scenegen as SG
from test_gpu_voxels import gpu_coarse_grain, particle_masses

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")


@pytest.mark.parametrize("R", [0.03, 0.06, 0.12])
@pytest.mark.parametrize("every", [1, 3, 17])
def test_fields_of_particles_out_of_order(every, R):
    n, l0 = 40000, 0.06
    spec = SG.column_scene(seed=4, n=n, footprint=3.0, sweeps=5)
    g = T.scene_from_specs(dict(spec, gravity=(0.0, 0.0, 0.0)))
    g.step(1)
    rng = np.random.default_rng(5)
    x, r = SG.fp32(spec["x"]), np.asarray(SG.fp32(spec["r"]), dtype=np.float64)
    some = np.arange(0, n, every)
    x[some] = x[rng.permutation(some)]
    v = SG.fp32(rng.normal(0.0, 0.5, (n, 3)))
    g.set_particles(0, x=x, v=v, w=np.zeros((n, 3)))
    lo = x.min(0) + 3 * R  # (the outermost reach beyond the grid)
    dims = tuple(int(d) for d in np.ceil((x.max(0) + 4 * R - lo) / l0))
    got = gpu_coarse_grain(g, tuple(lo), l0, dims, "gauss", R)
    m = particle_masses(r, spec["material"]["rho"])
    ref = O.coarse_grain(x, v, m, tuple(lo), l0, dims, kernel="gauss", R=R)
    for a, b in zip(got, ref):
        assert np.max(np.abs(a - b)) <= 1e-11 * np.max(np.abs(b))
    assert np.array_equal(got[0] > 0, ref[0] > 0)
    g.close()

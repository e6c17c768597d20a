"""A group of envs without contacts beside one with contacts (grouped
schedules): it runs no sweep, reports none, and leaves its spheres to gravity,
as the per-env schedule does.  The group without contacts is solved by one
block (a few spheres) or by a cluster (more than one block solves alone)."""
import numpy as np
import pytest

from helpers import jammed_bed, with_
from paper_2011_00459_amd import scenegen as SG

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")


def falling(n, like):
    k = int(np.ceil(n ** (1 / 3)))
    i = np.arange(n)
    x = np.stack([i % k, i // k % k, i // (k * k)], 1) * 0.1 + [-0.5, -0.4, 1.0]
    x = x.astype(np.float32).astype(np.float64)
    f = with_(like, x=x, r=np.full(n, np.float32(0.03), np.float64), v=np.tile([0.25, 0.0, -0.5], (n, 1)),
              w=np.tile([0.0, 1.0, 0.0], (n, 1)), bodies=[SG.walls_body(10.0, 10.0, 0.0, True)], grid_lo=(-1.0, -1.0, -0.5),
              grid_hi=(2.0, 2.0, 3.5))
    f.pop("id", None)
    return f


def run(specs, cfg):
    g = T.scene_from_specs(specs, cap_contacts=8 * max(len(s["x"]) for s in specs))
    g.set_solver_config(**cfg)
    st = g.step(2)
    out = [(p["x"], p["v"], p["w"]) for p in (g.get_particles(e) for e in range(len(specs)))]
    g.close()
    return st, out


@pytest.mark.parametrize("n,tol,impact,flow", [(1, 0.0, False, 0), (600, 0.0, False, 0), (600, 1e-3, False, 0),
                                               (600, 0.0, True, 0), (2500, 0.0, False, 0), (2500, 1e-3, True, 0),
                                               (2500, 0.0, False, 1), (600, 1e-3, False, 1)])
def test_group_without_contacts(n, tol, impact, flow):
    bed = jammed_bed(seed=150, nx=9, ny=8, nz=7, sweeps=15, blade=False)
    if impact:
        bed = with_(bed, material=dict(bed["material"], v_imp=0.05, restitution=0.3),
                    v=np.tile([0.0, 0.0, -0.4], (len(bed["x"]), 1)))
    bed = with_(bed, warm_start="prev", tol=tol)
    for specs in ([bed, falling(n, bed)], [falling(n, bed), bed]):
        e = 0 if specs[1] is bed else 1  # the env in free fall
        sa, a = run(specs, dict(mode="per_env", lds_particles=100000, cluster_particles=-1))
        sb, b = run(specs, dict(mode="grouped", blocks_per_xcd=32, dataflow=flow))
        assert sa[1 - e]["contacts"] == sb[1 - e]["contacts"] > 0
        for st in (sa[e], sb[e]):
            assert st["contacts"] == st["colours"] == st["sweeps"] == st["impact_sweeps"] == 0
            assert st["residual"] == st["residual_first"] == 0.0
        for u, v in zip(a[e], b[e]):
            assert np.array_equal(u, v)
        if tol == 0.0:  # (a group stops by its own sum of the residual)
            assert sa[1 - e]["sweeps"] == sb[1 - e]["sweeps"] == 15
            for u, v in zip(a[1 - e], b[1 - e]):
                assert np.array_equal(u, v)
        dt = bed["dt"]
        want = specs[e]["v"] + 2 * dt * np.asarray(bed["gravity"])
        assert np.max(np.abs(b[e][1] - want)) <= 1e-6

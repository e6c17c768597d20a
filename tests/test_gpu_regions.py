"""Solves cut into regions: a block keeps its region's spheres in LDS and the
blocks hand the spheres on their surfaces to each other through versioned
records.  No two contacts of a colour share a sphere, so the cut changes where
an update runs, not its operands or its order: states and impulses are bitwise
those of one block solving the env alone.  The cuts below meet odd remainders,
regions of a few spheres, regions larger than their LDS, several envs per
block, and all eight XCDs."""
import numpy as np
import pytest

import pyoracle as O
from helpers import jammed_bed, vel_tol, with_

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")

ALONE = dict(mode="per_env", lds_particles=100000, cluster_particles=-1)


def bed(seed, nx, ny, nz, **kw):
    s = jammed_bed(seed=seed, nx=nx, ny=ny, nz=nz, sweeps=kw.pop("max_sweeps", 12))
    if kw.pop("roll", False):
        s = with_(s, material=dict(s["material"], mu_r=0.1))
    return with_(s, warm_start="prev", **kw)


def states(specs, cfg, steps=2):
    g = T.scene_from_specs(specs, cap_contacts=8 * max(len(s["x"]) for s in specs))
    g.set_solver_config(**cfg)
    st = g.step(steps)
    out = []
    for e in range(len(specs)):
        p = g.get_particles(e)
        out.append((p["x"], p["v"], p["w"], g.get_contacts(e)[1], g.get_rolling_impulses(e)))
    g.close()
    return st, out


CASES = {
    # one env in regions of 13 spheres, and of 700 of which LDS holds 64
    "tiny_regions": ([(70, 11, 7, 5)], {}, dict(mode="per_env", lds_particles=400, cluster_particles=13)),
    "small_lds": ([(71, 17, 12, 10)], {}, dict(mode="per_env", lds_particles=64, cluster_particles=700)),
    "no_lds_rolling": ([(72, 13, 9, 8)], dict(roll=True), dict(mode="per_env", lds_particles=0, cluster_particles=150)),
    # odd sizes, one region per block of the group's XCD
    "grouped": ([(73, 23, 14, 11)], {}, dict(mode="grouped", blocks_per_xcd=32)),
    "grouped_three_blocks_rolling": ([(74, 23, 14, 11)], dict(roll=True), dict(mode="grouped", blocks_per_xcd=3)),
    # eleven envs in eight groups: blocks with a region of two envs
    "grouped_many": ([(75 + e, 19 + e % 3, 13, 9) for e in range(11)], {}, dict(mode="grouped", blocks_per_xcd=32)),
    # a whole solve in one block: one colour, its rows in LDS, its impulses in
    # LDS, everything in memory, colours of more contacts than threads, more
    # bodies than LDS holds
    "alone_one_sphere": ([(80, 1, 1, 1)], {}, dict(mode="grouped")),
    "alone_two_spheres": ([(81, 1, 1, 2)], {}, dict(mode="grouped")),
    "alone_rows": ([(82, 7, 7, 6)], {}, dict(mode="grouped")),
    "alone_rows_rolling": ([(83, 5, 7, 6)], dict(roll=True), dict(mode="grouped")),
    "alone_impulses": ([(84, 11, 11, 9)], {}, dict(mode="grouped")),
    "alone_memory_rolling": ([(85, 12, 11, 10)], dict(roll=True), dict(mode="grouped")),
    "alone_most_contacts": ([(86, 14, 10, 10)], {}, dict(mode="grouped", blocks_per_xcd=1)),
    "one_block_small_lds": ([(87, 23, 17, 14)], {}, dict(mode="grouped", blocks_per_xcd=1)),
    # regions with their impulses in LDS, and with nothing but bodies
    "grouped_three_blocks": ([(88, 23, 14, 11)], {}, dict(mode="grouped", blocks_per_xcd=3)),
    "grouped_two_blocks": ([(89, 23, 14, 14)], {}, dict(mode="grouped", blocks_per_xcd=2)),
    # the automatic plan of small regions: envs alone in a block, two of them
    # on either side of what is solved alone, one after another in a block when
    # they outnumber the blocks, beside clusters
    "small_plan": ([(100, 1, 1, 1), (101, 2, 2, 2), (102, 7, 7, 6), (103, 11, 11, 9), (104, 13, 13, 10),
                    (105, 13, 13, 11), (106, 23, 14, 11)], {}, dict(mode="per_env", cluster_particles=0)),
    "small_plan_rolling": ([(107, 7, 7, 6), (108, 14, 10, 10), (109, 13, 12, 10), (110, 23, 14, 11)], dict(roll=True),
                           dict(mode="per_env", cluster_particles=0)),
    "small_plan_queued": ([(120 + e % 7, 2 + e % 3, 3, 2) for e in range(300)], {},
                          dict(mode="per_env", cluster_particles=0)),
    # an env that fits neither automatic plan: the plan by spheres per block
    "no_plan_fits": ([(140, 23, 14, 11)], {}, dict(mode="per_env", lds_particles=64, cluster_particles=0)),
    # all eight XCDs
    "spread": ([(90, 41, 27, 25)], {}, dict(mode="spread", blocks_per_xcd=32)),
    "spread_rolling": ([(91, 41, 27, 25)], dict(roll=True), dict(mode="spread", blocks_per_xcd=5)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_regions_are_bitwise_one_block(name):
    dims, kw, cfg = CASES[name]
    specs = [bed(*d, **kw) for d in dims]
    specs = [with_(s, material=specs[0]["material"]) for s in specs]
    sa, a = states(specs, ALONE)
    sb, b = states(specs, cfg)
    for e in range(len(specs)):
        assert sa[e]["contacts"] == sb[e]["contacts"] > 0 and sa[e]["colours"] == sb[e]["colours"]
        for u, v in zip(a[e], b[e]):
            assert np.array_equal(u, v), (name, e)


@pytest.mark.parametrize("cfg", [dict(mode="per_env", lds_particles=5000, cluster_particles=300),
                                 dict(mode="grouped", blocks_per_xcd=32), dict(mode="spread", blocks_per_xcd=32)])
def test_regions_stop_with_the_oracle(cfg):
    # the sweep residual summed over regions, against the oracle's own stop
    spec = bed(95, 31, 27, 25, tol=2e-2, max_sweeps=200)
    g = T.scene_from_specs(spec)
    g.set_solver_config(**cfg)
    st = g.step(1)[0]
    o = O.OracleScene(spec)
    oo = o.step()
    assert 1 < oo["sweeps"] < 200
    # FP32 sums of one sweep's terms: the residual to 1e-4, a sweep's decrease is larger
    assert abs(st["sweeps"] - oo["sweeps"]) <= 1
    assert st["residual"] <= 2e-2
    assert np.max(np.abs(g.get_particles(0)["v"] - o.v)) <= vel_tol(o.v) + 2e-2 * np.max(np.abs(o.v))

"""Solves that really take several blocks, by the number of spheres from which
they do: clusters inside an XCD (grouped, more than one block solves alone) and
regions on all eight (more than one XCD solves, under the grouped and the
spread schedule alike), with rolling rows, the impact stage, the network's
start, update counters in memory and a stopping test.  Operands and order of
the updates are those of one block solving each env alone: states and impulses
are bitwise the same."""
import numpy as np
import pytest

import pyoracle as O
from helpers import jammed_bed, vel_tol, with_
from paper_2011_00459_amd import learn as LN

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")

ALONE = dict(mode="per_env", lds_particles=100000, cluster_particles=-1, dataflow=0)
GROUPED = dict(mode="grouped", blocks_per_xcd=32, dataflow=0)
SPREAD = dict(mode="spread", blocks_per_xcd=32, dataflow=0)
NO_LDS = dict(mode="per_env", lds_particles=0, cluster_particles=0, dataflow=0)
FLOW = dict(mode="grouped", blocks_per_xcd=32, dataflow=1)

FEW = [(5, 5, 4), (101, 1, 1), (1, 1, 1)]        # 100, 101 and 1: one or two blocks of update counters
WIDE = [(41, 27, 25)]                           # 27,675 spheres: all XCDs
MIXED = [(19, 14, 10), (6, 5, 4), (23, 14, 11)]  # 2,660, 120 and 3,542: a cluster, one block, a cluster


def beds(dims, sweeps=12, roll=False, impact=False, **kw):
    out = []
    for e, d in enumerate(dims):
        s = jammed_bed(seed=160 + e, nx=d[0], ny=d[1], nz=d[2], sweeps=sweeps)
        m = dict(s["material"])
        if roll:
            m["mu_r"] = 0.1
        if impact:
            m.update(v_imp=0.05, restitution=0.3)
            s = with_(s, v=np.tile([0.0, 0.0, -0.4], (len(s["x"]), 1)))
        out.append(with_(s, material=m, **dict(dict(warm_start="prev"), **kw)))
    return out


def states(specs, cfg, steps=2):
    g = T.scene_from_specs(specs, cap_contacts=8 * max(len(s["x"]) for s in specs))
    g.set_solver_config(**cfg)
    if specs[0]["warm_start"] == "learned":
        g.set_mlp_weights(LN.flatten(LN.init_weights(4)))
    st = g.step(steps)
    out = []
    for e in range(len(specs)):
        p = g.get_particles(e)
        out.append((p["x"], p["v"], p["w"], g.get_contacts(e)[1], g.get_rolling_impulses(e)))
    g.close()
    return st, out


@pytest.mark.parametrize("kw", [{}, dict(roll=True), dict(impact=True), dict(warm_start="learned")],
                         ids=["plain", "rolling", "impact", "learned"])
@pytest.mark.parametrize("dims,cfg", [(MIXED, GROUPED), (MIXED, FLOW), (FEW, FLOW), (MIXED, NO_LDS), (WIDE, GROUPED), (WIDE, SPREAD), (WIDE, FLOW)],
                         ids=["clusters", "clusters_flow", "few_flow", "no_lds", "wide_grouped", "wide_spread", "one_xcd_flow"])
def test_clusters_are_bitwise_one_block(dims, cfg, kw):
    specs = beds(dims, **kw)
    sa, a = states(specs, ALONE)
    sb, b = states(specs, cfg)
    for e in range(len(specs)):
        for key in ("contacts", "colours", "sweeps", "impacts", "impact_sweeps", "fallback_used"):
            assert sa[e][key] == sb[e][key], key
        assert sa[e]["contacts"] > 0
        for u, v in zip(a[e], b[e]):
            assert np.array_equal(u, v), e
    if kw.get("impact"):
        assert sum(s["impacts"] for s in states(specs, cfg, steps=1)[0]) > 0


@pytest.mark.parametrize("roll,impact", [(False, False), (True, False), (False, True)])
@pytest.mark.parametrize("dims,cfg", [([MIXED[0]], GROUPED), ([MIXED[0]], FLOW), (WIDE, GROUPED), (WIDE, SPREAD)],
                         ids=["cluster", "cluster_flow", "wide_grouped", "wide_spread"])
def test_clusters_stop_with_the_oracle(dims, cfg, roll, impact):
    # the sweep at which the regions' residuals add up to the tolerance is the
    # oracle's (FP32 terms: give or take one), and the state is bitwise that
    # of one block after as many sweeps
    tol = 2e-2
    spec = beds(dims, sweeps=200, roll=roll, impact=impact, warm_start="cold", tol=tol)[0]
    st, out = states([spec], cfg, steps=1)
    o = O.OracleScene(spec)
    oo = o.step()
    assert 1 < oo["sweeps"] < 200
    assert abs(st[0]["sweeps"] - oo["sweeps"]) <= 1 and st[0]["residual"] <= tol
    if not impact:  # (the impact stage of the fixed solve would run all its sweeps)
        fixed, ref = states([with_(spec, tol=0.0, max_sweeps=st[0]["sweeps"])], ALONE, steps=1)
        for u, v in zip(out[0], ref[0]):
            assert np.array_equal(u, v)
        assert st[0]["residual"] == pytest.approx(fixed[0]["residual"], rel=1e-4)


def test_impact_stage_on_all_xcds_matches_the_oracle():
    spec = beds(WIDE, sweeps=40, impact=True, warm_start="cold")[0]
    st, out = states([spec], SPREAD, steps=1)
    o = O.OracleScene(spec)
    oo = o.step()
    assert st[0]["impacts"] == oo["impacts"] > 0
    assert np.max(np.abs(out[0][1] - o.v)) <= vel_tol(o.v)

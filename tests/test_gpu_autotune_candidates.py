"""The autotuner times a schedule once: limits of blocks per XCD that give the
same blocks count as one candidate, and the spread schedule, which for one env
launches the grouped one's blocks, is none."""
import numpy as np
import pytest

from helpers import jammed_bed, with_

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")


@pytest.mark.parametrize("dims", [(9, 8, 7), (19, 13, 11), (41, 27, 25)])
def test_equal_schedules_are_one_candidate(dims):
    # one block, seven blocks, 9 a XCD
    spec = with_(jammed_bed(seed=180, nx=dims[0], ny=dims[1], nz=dims[2], sweeps=40), warm_start="prev")
    limits = {504: {32}, 2717: {32}, 27675: {32, 8}}[len(spec["x"])]
    g = T.scene_from_specs(spec, cap_contacts=8 * len(spec["x"]))
    g.step(2)
    before = g.get_particles(0)["v"]
    cfg, ms = g.autotune(steps=2)
    assert ms > 0.0 and np.array_equal(g.get_particles(0)["v"], before)
    assert cfg["mode"] in ("grouped", "per_env")
    if cfg["mode"] == "grouped":
        assert cfg["blocks_per_xcd"] in limits
    g.close()

"""Scenes stepped from several threads at once, each on a stream of its own:
solves whose blocks fill an XCD (20,000 spheres), several of them at once that
do not fit beside each other, all XCDs, smaller clusters, one block, and the
colouring across ranges.  Every scene's states are bitwise those it takes when
stepped alone."""
import ctypes as C
import threading

import numpy as np
import pytest

from helpers import jammed_bed, with_

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")
D = pytest.importorskip("paper_2011_00459_amd.devmem")

DIMS = [(32, 25, 25), (32, 25, 25), (41, 31, 32), (25, 20, 13), (17, 13, 10), (9, 8, 8)]


def stream():
    hip = D.hip()
    hip.hipStreamCreateWithFlags.argtypes = [C.POINTER(C.c_void_p), C.c_uint]
    s = C.c_void_p()
    assert hip.hipStreamCreateWithFlags(C.byref(s), 1) == 0  # no ordering with the null stream
    return s.value


def scene(spec, cfg):
    """A scene on its own stream after three steps (its step graphs are captured)."""
    st = stream()
    g = T.scene_from_specs(spec, cap_contacts=8 * len(spec[0]["x"]), stream=st)
    if cfg:
        g.set_solver_config(**cfg)
    g.step(3)
    return g, st


def finish(g, st, envs):
    p = g.get_particles(envs - 1)
    out = (p["x"], p["v"], p["w"], g.get_contacts(0)[1])
    g.close()
    hip = D.hip()
    hip.hipStreamDestroy.argtypes = [C.c_void_p]
    assert hip.hipStreamDestroy(C.c_void_p(st)) == 0
    return out


@pytest.mark.parametrize("cfg", [None, dict(mode="grouped", blocks_per_xcd=32, dataflow=1),
                                 dict(mode="per_env", lds_particles=100000, cluster_particles=700)],
                         ids=["default", "flow", "per_env"])
def test_scenes_stepped_at_once(cfg):
    steps, n = 10, len(DIMS)
    specs = [with_(jammed_bed(seed=170 + k, nx=d[0], ny=d[1], nz=d[2], sweeps=25), warm_start="prev")
             for k, d in enumerate(DIMS)]
    specs = [[s] * (12 if k == 4 else 1) for k, s in enumerate(specs)]  # one scene of several envs
    alone = []
    for s in specs:
        g, st = scene(s, cfg)
        counts = [g.step(1)[0]["contacts"] for _ in range(steps)]
        alone.append((counts, finish(g, st, len(s))))
    scenes = [scene(s, cfg) for s in specs]
    start = threading.Barrier(n)
    counts, errors = [[] for _ in specs], []

    def go(k):
        try:
            start.wait(60)
            for _ in range(steps):
                counts[k].append(scenes[k][0].step(1)[0]["contacts"])
        except Exception as e:  # noqa: BLE001
            errors.append((k, e))

    ts = [threading.Thread(target=go, args=(k,)) for k in range(n)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
    for k, (g, st) in enumerate(scenes):
        assert counts[k] == alone[k][0] and min(counts[k]) > 0
        for u, v in zip(alone[k][1], finish(g, st, len(specs[k]))):
            assert np.array_equal(u, v), k

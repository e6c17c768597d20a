"""Scenes made, read and closed again and again from several threads: the
memory of a closed scene's read-back serves later ones, of other sizes and on
other streams too, and no scene sees another's values."""
import threading

import numpy as np
import pytest

from paper_2011_00459_amd import scenegen as SG

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")


def test_scenes_made_and_closed_by_threads():
    sizes = [1, 40, 60, 200, 1500, 17000, 40000, 300, 5, 900, 90]
    specs = {n: SG.column_scene(seed=n, n=n, footprint=2.0, sweeps=0) for n in sizes}
    bad = []

    def go(t):
        try:
            kept = []
            for k in range(24):
                n = sizes[(7 * t + 5 * k) % len(sizes)]
                g = T.scene_from_specs(specs[n])
                v = SG.fp32(np.random.default_rng(100 * t + k).normal(0.0, 1.0, (n, 3)))
                g.set_particles(0, v=v)
                kept.append((g, n, v))
                if k % 3 == 2:
                    for h, m, u in kept:
                        p = h.get_particles(0)
                        if not (np.array_equal(p["v"], u) and np.array_equal(p["x"], SG.fp32(specs[m]["x"]))
                                and np.array_equal(p["r"], SG.fp32(specs[m]["r"])) and not np.any(p["w"])):
                            bad.append((t, k, m))
                        h.close()
                    kept = []
        except Exception as e:  # noqa: BLE001
            bad.append((t, repr(e)))

    ts = [threading.Thread(target=go, args=(t,)) for t in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad

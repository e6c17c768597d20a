"""Particle state read back in chunks: every value that set_particles took comes
back, at and around the chunk's 16,384 particles, whichever outputs are asked for."""
import ctypes as C

import numpy as np
import pytest

from paper_2011_00459_amd import scenegen as SG

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")


@pytest.mark.parametrize("n", [1, 300, 16383, 16384, 16385, 40000])
def test_read_back_returns_what_was_set(n):
    spec = SG.column_scene(seed=5, n=n, footprint=3.0 if n > 300 else 0.6, sweeps=3)
    g = T.scene_from_specs(spec)
    g.step(1)  # slots are in spatial order from here on
    rng = np.random.default_rng(n)
    x = SG.fp32(np.asarray(spec["x"]) + rng.uniform(-0.01, 0.01, (n, 3)))
    v, w = SG.fp32(rng.normal(0.0, 0.5, (n, 3))), SG.fp32(rng.normal(0.0, 2.0, (n, 3)))
    g.set_particles(0, x=x, v=v, w=w)
    p = g.get_particles(0)
    for got, want in ((p["x"], x), (p["v"], v), (p["w"], w), (p["r"], SG.fp32(spec["r"]))):
        assert np.array_equal(got, np.asarray(want, dtype=np.float64))
    out, m = np.full((n + 1, 3), -7.0), C.c_int64()
    dp = out.ctypes.data_as(C.POINTER(C.c_double))
    assert T.lib().get_particles(g.h, 0, None, dp, None, None, C.byref(m)) == 0
    assert m.value == n and np.array_equal(out[:n], np.asarray(v, dtype=np.float64)) and (out[n] == -7.0).all()
    rad = np.full(n + 1, -7.0)
    assert T.lib().get_particles(g.h, 0, None, None, None, rad.ctypes.data_as(C.POINTER(C.c_double)), None) == 0
    assert np.array_equal(rad[:n], p["r"]) and rad[n] == -7.0

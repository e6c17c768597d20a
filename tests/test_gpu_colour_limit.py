"""The colouring at its limit of 64 colours: a sphere with 64 contacts gets
all of them, one with more makes the step fail with the colour flag (and no
other), whether the contacts are keyed by the sphere (lowest id) or by the
others (highest id) and whether they lie in its own range of 1,024 spheres or
in another, with which a block agrees on a colour through memory."""
import re

import numpy as np
import pytest

import pyoracle as O
from paper_2011_00459_amd import scenegen as SG

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")

COLOURS, COLOURING_FAILED = 4, 8  # flags of a step's failure


def big_sphere(contacts, across, first):
    """A sphere of radius 0.5 with small ones at its lower half, in cells (of
    1.001) before its own so that each of them finds its contact; across:
    1,331 loose spheres whose cell comes between."""
    big = np.array([1.5, 1.5, 2.01])
    k = np.arange(contacts)
    c = 1.0 - (k + 0.5) / contacts * (1.0 - np.cos(np.radians(75.0)))  # a spiral over the cap
    s, a = np.sqrt(1.0 - c * c), np.pi * (3.0 - np.sqrt(5.0)) * k
    x = [big + 0.519 * np.stack([s * np.cos(a), s * np.sin(a), -c], 1)]
    if across:
        g = 3.1 + 0.08 * np.arange(11)
        x.append(np.stack(np.meshgrid(g, g, g - 2.0, indexing="ij"), -1).reshape(-1, 3))
    x = np.concatenate(x)
    r = np.full(len(x), 0.02)
    x, r = (np.vstack([[big], x]), np.append(0.5, r)) if first else (np.vstack([x, [big]]), np.append(r, 0.5))
    n = len(x)
    return dict(x=SG.fp32(x), r=SG.fp32(r), v=np.zeros((n, 3)), w=np.zeros((n, 3)), rho=None,
                id=np.arange(n, dtype=np.int64), bodies=[SG.walls_body(50.0, 50.0, -1.0, True)],
                material=SG.material(0.5, 0.0), dt=1.0 / 60.0, gravity=(0.0, 0.0, -9.81), max_sweeps=3, tol=0.0,
                warm_start="cold", grid_lo=(0.0, 0.0, 0.0), grid_hi=(4.0, 4.0, 4.0), r_ref=0.02)


@pytest.mark.parametrize("first", [False, True])
@pytest.mark.parametrize("across", [False, True])
@pytest.mark.parametrize("contacts", [64, 65, 90])
def test_sphere_at_the_limit_of_colours(contacts, across, first):
    spec = big_sphere(contacts, across, first)
    g = T.scene_from_specs(spec)
    if contacts <= 64:
        st = g.step(1)[0]
        o = O.OracleScene(spec).step()
        assert np.array_equal(g.get_contacts(0)[0], o["keys"]) and len(o["keys"]) == contacts
        assert st["colours"] == o["colours"] == 64
        assert np.array_equal(g.get_colours(0), o["colour"])
    else:
        with pytest.raises(T.TerrainError) as e:
            g.step(1)
        assert e.value.code == T.TR_E_CAPACITY
        flags = int(re.search(r"flags (0x[0-9a-f]+), (\d+) contacts", str(e.value)).group(1), 16)
        assert flags & COLOURS and not flags & COLOURING_FAILED
        assert f" {contacts} contacts found" in str(e.value)
    g.close()

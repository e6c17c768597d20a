"""The colouring where its work splits: ranges of 1,024 spheres per block with
contacts across two and more of them, several envs in one range, spheres with
more contacts than a thread ranks in registers (a big sphere among small
ones), and the state kept in memory."""
import numpy as np
import pytest

import pyoracle as O
from helpers import jammed_bed, with_

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")


def check(specs, cap_contacts=None):
    g = T.scene_from_specs(specs, cap_contacts=cap_contacts)
    cap = max(len(s["x"]) for s in specs)
    st = g.step(1)
    for e, s in enumerate(specs):
        o = O.OracleScene(dict(s, id=np.arange(len(s["x"]), dtype=np.int64) + e * cap))
        oo = o.step()
        assert np.array_equal(g.get_contacts(e)[0], oo["keys"])
        assert np.array_equal(g.get_colours(e), oo["colour"]), e
        assert st[e]["colours"] == oo["colours"]
    g.close()


@pytest.mark.parametrize("dims", [(1, 1, 1), (8, 8, 16), (16, 16, 4), (41, 5, 5), (25, 19, 11)])
def test_ranges_of_one_env(dims):
    check([jammed_bed(seed=41, nx=dims[0], ny=dims[1], nz=dims[2], sweeps=1, blade=dims[0] > 20)])


def test_envs_share_a_range():
    specs = [jammed_bed(seed=50 + e, nx=3 + e, ny=7, nz=5, sweeps=1, blade=False) for e in range(12)]
    check([with_(s, material=specs[0]["material"]) for s in specs])


@pytest.mark.parametrize("first", [False, True])
def test_more_contacts_than_a_thread_ranks(first):
    # one sphere three radii large in the middle of a bed, the last id (its
    # contacts are keyed by the others) or the first (by itself)
    s = jammed_bed(seed=42, nx=20, ny=20, nz=14, r0=0.03, sweeps=1, blade=False)
    c = np.array([0.0, 0.0, 0.42])
    keep = np.linalg.norm(s["x"] - c, axis=1) > 0.1 + 0.5 * s["r"]
    x = np.concatenate([s["x"][keep], [c]])
    r = np.concatenate([s["r"][keep], [0.1]])
    if first:
        x, r = x[::-1], r[::-1]
    x, r = (np.asarray(a, np.float32).astype(np.float64) for a in (x, r))
    n = len(x)
    spec = with_(s, x=x, r=r, v=np.zeros((n, 3)), w=np.zeros((n, 3)), id=np.arange(n, dtype=np.int64))
    o = O.OracleScene(spec)
    keys = o.step()["keys"]
    ends = np.concatenate([keys >> np.uint64(32), keys & np.uint64(0xffffffff)])
    assert 16 < np.sum(ends == (0 if first else n - 1)) < 64
    check([spec], cap_contacts=16 * n)


def splitmix64(x):
    z = x + np.uint64(0x9E3779B97F4A7C15)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def test_more_spheres_than_lds_holds():
    # 2.7 million spheres: more than 256 blocks keep in LDS.  Every contact
    # must hold the least colour that its spheres' contacts of higher priority
    # leave free, which fixes the whole colouring by induction.
    spec = jammed_bed(seed=43, nx=300, ny=150, nz=60, r0=0.02, sweeps=1, blade=False)
    n = len(spec["x"])
    g = T.scene_from_specs(spec, cap_contacts=4 * n)
    st = g.step(1)[0]
    keys, _ = g.get_contacts(0)
    col = g.get_colours(0).astype(np.int64)
    g.close()
    assert st["contacts"] == len(keys) > 2.5 * n
    a, low = (keys >> np.uint64(32)).astype(np.int64), keys & np.uint64(0xffffffff)
    pair = low < np.uint64(0x80000000)
    rank = np.empty(len(keys), np.int64)  # by decreasing (hash, key)
    rank[np.lexsort((keys, splitmix64(keys)))[::-1]] = np.arange(len(keys))
    who = np.concatenate([a, low[pair].astype(np.int64)])
    con = np.concatenate([np.arange(len(keys)), np.nonzero(pair)[0]])
    order = np.argsort(who * len(keys) + rank[con], kind="stable")
    who, con = who[order], con[order]
    place = np.arange(len(who)) - np.searchsorted(who, who, "left")  # place in the sphere's list
    bits = np.uint64(1) << col[con].astype(np.uint64)
    used = np.zeros(n, np.uint64)
    first = np.zeros(len(keys), np.uint64)
    second = np.zeros(len(keys), np.uint64)
    is_first = order < len(keys)
    for k in range(int(place.max()) + 1):
        at = np.nonzero(place == k)[0]
        f, s = at[is_first[at]], at[~is_first[at]]
        first[con[f]] = used[who[f]]
        second[con[s]] = used[who[s]]
        used[who[at]] |= bits[at]
    free = ~(first | second)
    least = np.log2((free & (~free + np.uint64(1))).astype(np.float64)).astype(np.int64)
    assert np.array_equal(col, least)
    assert st["colours"] == col.max() + 1

"""Staged scatter at the edges of its dispatch, bit for bit against the oracle.

Column counts from one to beyond the staggered kernel's, depth rows from one
to all of them (and beyond what one word's trailing zero count tells), tiles
of one vertex to ragged last tiles, items of a few records, of several parts,
and one hot vertex.  Batches hold more than 4,096 updates, so that none takes
the small-batch path, and name a lane layout, so that they take the tiles; the
direct scatter of medium batches has cases of its own below.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cupk():
    import torch
    assert torch.cuda.is_available(), "GPU test on a machine without a GPU"
    import paper_2509_14433_amd as m
    return m


def _edges(V, n, seed, hot=False):
    """n distinct edges in random order (all at vertex 5 when hot)."""
    rng = np.random.default_rng(seed)
    if hot:
        o = rng.permutation(V - 1)[:n].astype(np.uint32)
        o[o >= 5] += 1
        return np.full(o.shape, 5, np.uint32), o
    k = np.unique(rng.integers(0, V, (int(n * 2.8) + 64, 2)), axis=0)
    k = k[k[:, 0] < k[:, 1]]
    k = k[rng.permutation(len(k))[:n]].astype(np.uint32)
    swap = rng.random(len(k)) < 0.5
    k[swap] = k[swap][:, ::-1]
    return k[:, 0].copy(), k[:, 1].copy()


CASES = [
    # V, edges, C, D, context options
    (300, 9000, 1, 2, {}),
    (300, 9000, 9, 3, dict(tile_vertices=4, lds_rows=3)),        # every depth in LDS
    (300, 9000, 14, 28, dict(tile_vertices=16, lds_rows=1, chunk_records=64)),
    (300, 9000, 17, 34, dict(tile_vertices=16, chunk_records=511)),
    (301, 9000, 20, 40, dict(tile_vertices=8, lds_rows=10)),
    (301, 9000, 24, 48, {}),
    (301, 9000, 25, 50, {}),                                     # the pair kernel
    (301, 9000, 8, 64, dict(tile_vertices=1, lds_rows=31)),
    (301, 9000, 4, 64, dict(tile_vertices=1, lds_rows=40)),      # depths beyond the low word
    (40003, 6000, 16, 32, {}),                                   # less than a record a vertex
    (16001, 200_000, 14, 28, dict(tile_grid=7)),                 # few blocks, many items each
    (5003, 5000, 13, 26, dict(chunk_records=128, hot=True)),     # one tile, many parts
    (5003, 5000, 13, 26, dict(hot=True)),
]


@pytest.mark.parametrize("V,n,C,D,kw", CASES)
def test_staged_scatter_edges(cupk, V, n, C, D, kw):
    kw = dict(kw)
    S = 0x5CA77E2 + C
    u, v = _edges(V, n, V + C, kw.pop("hot", False))
    assert len(u) > 4096
    print(f"case V={V} n={len(u)} C={C} D={D} {kw}", flush=True)
    ctx = cupk.Context(V, C, D, S, scatter_mode=cupk.SCATTER_STAGED, time_kernels=True,
                       tile_layout=cupk.LAYOUT_RECORD, **kw)
    ref = oracle.Sketch(V, C, D, S)
    z = np.zeros(len(u), np.uint8)
    ctx.apply_updates(u, v, z)
    ref.apply(u, v)
    a, g = ctx.get_sketch()
    assert np.array_equal(a, ref.alpha) and np.array_equal(g, ref.gamma)
    # the launch changed at least the buckets that are nonzero now
    assert ctx.counters()["timed_buckets"] >= np.count_nonzero(ref.alpha | ref.gamma)
    k = len(u) - 137  # delete all but a few (XOR takes them out again)
    ctx.apply_updates(u[:k], v[:k], z[:k] + 1)
    ref.apply(u[:k], v[:k])
    a, g = ctx.get_sketch()
    assert np.array_equal(a, ref.alpha) and np.array_equal(g, ref.gamma)
    assert ctx.digest() == ref.digest()
    ctx.close()


WIDTHS = [
    # V, edges, C, tile_vertices: where a vertex id and a place in a bin take
    # 32 bits (records of one word) and where they take more (of two words)
    (1 << 20, 300_000, 2, 16),        # 32 bits in the coarse bins
    ((1 << 20) + 9, 300_000, 2, 16),  # 34 in the coarse bins, 25 in the tiles
    (1 << 22, 40_000, 1, 1024),       # 38 in the coarse bins, 32 in the tiles
    ((1 << 22) + 1, 40_000, 1, 1024),  # 39, 33
    (1 << 21, 300_000, 2, 2048),      # one level: 32
    ((1 << 21) + 5, 300_000, 2, 2048),  # one level: 33
]


@pytest.mark.parametrize("V,n,C,tv", WIDTHS)
def test_record_widths(cupk, V, n, C, tv):
    S = 0x3BD + tv
    D = 3
    u, v = _edges(V, n, V + C)
    # half of them at the last vertices: the largest places and ids, long bins
    u[::2] = V - 1 - u[::2] % 40
    v[::2] = v[::2] % (V - 50)
    print(f"widths V={V} n={len(u)} C={C} tv={tv}", flush=True)
    ctx = cupk.Context(V, C, D, S, tile_vertices=tv, lds_rows=1,
                       tile_layout=cupk.LAYOUT_RECORD)
    ref = oracle.Sketch(V, C, D, S)
    ctx.apply_updates(u, v, np.zeros(len(u), np.uint8))
    ref.apply(u, v)
    a, g = ctx.get_sketch()
    assert np.array_equal(a, ref.alpha) and np.array_equal(g, ref.gamma)
    ctx.close()


DIRECT = [
    # V, edges, C, D: within the direct scatter's range; 16,384 and 16,385 on
    # either side of the one-block classification, a star, many and few columns
    (40003, 4100, 16, 32, False),
    (40003, 16384, 16, 32, False),
    (40003, 16385, 16, 32, False),
    (20011, 9000, 15, 30, True),
    (3001, 5000, 20, 5, False),
    (60013, 20000, 1, 2, False),
]


@pytest.mark.parametrize("timed", [False, True])
@pytest.mark.parametrize("V,n,C,D,hot", DIRECT)
def test_direct_scatter(cupk, V, n, C, D, hot, timed):
    S = 0xD14EC7 + C
    u, v = _edges(V, n, V + n, hot)
    assert len(u) == n
    print(f"direct V={V} n={n} C={C} D={D} hot={hot} timed={timed}", flush=True)
    ctx = cupk.Context(V, C, D, S, time_kernels=timed)
    ref = oracle.Sketch(V, C, D, S)
    z = np.zeros(n, np.uint8)
    ctx.apply_updates(u, v, z)
    ref.apply(u, v)
    a, g = ctx.get_sketch()
    assert np.array_equal(a, ref.alpha) and np.array_equal(g, ref.gamma)
    assert ctx.num_components() == oracle.uf_components(V, u, v)[0]
    if timed:
        assert ctx.counters()["timed_buckets"] >= np.count_nonzero(ref.alpha | ref.gamma)
    # an invalid update rejects the batch
    bad = v.copy()
    bad[n - 1] = u[n - 1]
    with pytest.raises(cupk.CupkError):
        import torch
        ctx.apply_updates_device(torch.from_numpy(
            cupk.pack_updates(u, bad, z).view(np.int64)).cuda())
        ctx.sync()
    assert ctx.digest() == ref.digest()
    ctx.close()


def test_exact_mode_one_block(cupk):
    """Exact mode needs the flags' positions: batches classified by one block
    and through the tiles give the same forest, cuts and sketch."""
    V, n = 12007, 14000
    u, v = _edges(V, n, 3)
    got = []
    for kw in ({}, dict(tile_layout=cupk.LAYOUT_RECORD)):
        ctx = cupk.Context(V, seed=77, exact=True, **kw)
        ctx.apply_updates(u, v, np.zeros(n, np.uint8))
        fu, fv = (x.astype(np.uint32) for x in np.array(sorted(ctx.forest_edges())).T)
        rng = np.random.default_rng(4)  # 12 forest edges among 12,000 of the others
        pick = rng.permutation(len(fu))[:12]
        forest = set(zip(fu.tolist(), fv.tolist()))
        rest = [(a, b) for a, b in zip(u.tolist(), v.tolist())
                if (min(a, b), max(a, b)) not in forest]
        k = min(len(rest), 3000)
        e = [(int(fu[i]), int(fv[i])) for i in pick] + rest[:k]
        new = [(int(a), int(b)) for a, b in zip(*_edges(V, 9000, 5))
               if (a, b) not in set(zip(u.tolist(), v.tolist()))][:6000] if not got else got[0][3]
        d = np.array([1] * len(e) + [0] * len(new), np.uint8)
        p = np.random.default_rng(6).permutation(len(d))
        x = np.array(e + new, np.uint32)[p]
        ctx.apply_updates(x[:, 0], x[:, 1], d[p])
        c = ctx.counters()
        got.append((ctx.forest_edges(), ctx.digest(), c["cuts"], new, c["reverts"]))
        ctx.close()
    assert got[0][0] == got[1][0] and got[0][1] == got[1][1] and got[0][2] == got[1][2]
    assert got[0][4] > 0

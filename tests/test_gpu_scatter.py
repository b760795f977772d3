"""Staged scatter at the edges of its dispatch, bit for bit against the oracle.

Column counts from one to beyond the staggered kernel's, depth rows from one
to all of them (and beyond what one word's trailing zero count tells), tiles
of one vertex to ragged last tiles, items of a few records, of several parts,
and one hot vertex.  Batches hold more than 4,096 updates, so that none takes
the small-batch path.
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
    k = np.unique(rng.integers(0, V, (int(n * 1.4) + 64, 2)), axis=0)
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
    ctx = cupk.Context(V, C, D, S, scatter_mode=cupk.SCATTER_STAGED, time_kernels=True, **kw)
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

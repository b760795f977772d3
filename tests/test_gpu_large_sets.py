"""Reductions whose lists or results are too large to pass through pinned
memory: more than 2^20 words of members and work items, and more than 256 KiB
of sketches."""
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


def _graph(cupk, V, C, D, n, seed):
    rng = np.random.default_rng(seed)
    k = np.unique(np.sort(rng.integers(0, V, (n, 2)), axis=1), axis=0)
    k = k[k[:, 0] < k[:, 1]].astype(np.uint32)
    u, v = k[:, 0].copy(), k[:, 1].copy()
    ctx = cupk.Context(V, C, D, seed)
    ref = oracle.Sketch(V, C, D, seed)
    ctx.apply_updates(u, v, np.zeros(len(u), np.uint8))
    ref.apply(u, v)
    return ctx, ref, rng


def _xor(ref, s):
    """Sum of the members' sketches (duplicates cancel in pairs)."""
    s = np.asarray(s, np.int64)
    once = np.flatnonzero(np.bincount(s, minlength=ref.alpha.shape[0]) % 2)
    return (np.bitwise_xor.reduce(ref.alpha[once], axis=0),
            np.bitwise_xor.reduce(ref.gamma[once], axis=0))


@pytest.mark.parametrize("sizes", [
    [1_100_000],                          # one set of many items
    [1_048_400, 3, 0, 64, 65],            # members and items beyond the limit together
    [7] * 1000,                           # a large result from a short list
    [300_000] * 3 + [0, 1] * 500 + [200_001],
])
def test_lists_and_results_beyond_pinned_memory(cupk, sizes):
    import torch
    V, C, D = 3000, 6, 12
    ctx, ref, rng = _graph(cupk, V, C, D, 9000, 0x1A56E + len(sizes))
    sets = [rng.integers(0, V, n).astype(np.uint32) for n in sizes]
    print(f"sets of {sizes[:5]} members", flush=True)
    a, g = ctx.component_sketch_batch(sets)
    out = torch.empty(len(sets) * C * D * 2, dtype=torch.int64, device="cuda")
    ctx.component_sketch_batch(sets, out=out)
    dev = out.cpu().numpy().view(np.uint64).reshape(len(sets), C, D, 2)
    for j, s in enumerate(sets):
        xa, xg = _xor(ref, s)
        assert np.array_equal(a[j], xa) and np.array_equal(g[j], xg), j
        assert np.array_equal(dev[j, ..., 0], xa) and np.array_equal(dev[j, ..., 1], xg), j
    ctx.close()


def test_levels_pass_beyond_pinned_memory(cupk):
    """Every vertex alone at the lowest level: 2^18 sets of one member are
    1.3e6 words of lists and more results than are published."""
    V, C, D, S = 1 << 18, 3, 12, 0x1E7E15
    rng = np.random.default_rng(8)
    # paths of 16 vertices (3 of 4 edges), then some edges gone and new ones between paths
    w = np.arange(V - 1, dtype=np.uint32)
    w = w[(w % 16 != 15) & (w % 4 != 3)]
    u0, v0 = w, w + 1
    gone = rng.random(len(w)) < 0.02
    x = rng.integers(0, V // 2, 3000).astype(np.uint32)
    nu, nv = x, (x + V // 2 - 5).astype(np.uint32)
    key = np.unique(nu.astype(np.int64) * V + nv)
    nu, nv = (key // V).astype(np.uint32), (key % V).astype(np.uint32)
    ctx = cupk.Context(V, C, D, S, levels=True)
    sk = oracle.Sketch(V, C, D, S)
    fr = oracle.LevelsReplay(sk)
    for u, v, d in ((u0, v0, np.zeros(len(u0), np.uint8)),
                    (np.concatenate([u0[gone], nu]), np.concatenate([v0[gone], nv]),
                     np.concatenate([np.ones(gone.sum(), np.uint8), np.zeros(len(nu), np.uint8)]))):
        print(f"levels batch of {len(u)}", flush=True)
        ctx.apply_updates(u, v, d)
        fr.apply_batch(u, v, d)
        for j in range(1, C + 1):
            assert ctx.level_forest_edges(j) == fr.forest_edges(j), j
    assert ctx.digest() == sk.digest()
    ctx.close()

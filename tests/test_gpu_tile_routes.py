"""Scatter routes against the oracle: exact and levels mode on each, and batches
around the sizes where a route ends.

By default a staged context sends a batch of a few thousand updates to HBM
directly; naming a lane layout sends it through the tiles.  Exact mode then
undoes its speculation with whole passes through the tiles: a random edge of
a sparse graph is toggled at every step, so that cuts fall all along a batch
and most of them leave more than 4,096 updates to undo.
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


def _toggles(V, pairs, n, seed):
    """n updates, each toggling one of `pairs` vertex pairs drawn at random."""
    rng = np.random.default_rng(seed)
    k = rng.permutation(V * (V - 1) // 2)[:pairs]
    a, b = (x[k] for x in np.triu_indices(V, 1))
    live = np.zeros(pairs, bool)
    pick = rng.integers(0, pairs, n)
    d = np.zeros(n, np.uint8)
    for i, q in enumerate(pick):
        d[i] = live[q]
        live[q] = not live[q]
    return a[pick].astype(np.uint32), b[pick].astype(np.uint32), d


ROUTES = {"direct": {}, "tiles": dict(tile_layout=1), "pair": dict(tile_layout=2, lds_rows=4),
          "two_levels": dict(tile_layout=1, tile_vertices=1, coarse_tiles=64),
          "atomic": dict(scatter_mode=0)}


@pytest.fixture(scope="module")
def exact_ref():
    V, C, D, S = 2500, 9, 18, 0x5EED4000
    u, v, d = _toggles(300, 900, 10_000, 5)
    u, v = u * 8 + 3, v * 8 + 3  # spread over V
    sk = oracle.Sketch(V, C, D, S)
    fr = oracle.ForestReplay(sk)
    for i in range(len(u)):
        fr.apply_batch(u[i:i + 1], v[i:i + 1], d[i:i + 1])
    return dict(V=V, C=C, D=D, S=S, u=u, v=v, d=d, sk=sk, fr=fr)


@pytest.mark.parametrize("route", sorted(ROUTES))
def test_exact_mode_undoes_on_every_route(cupk, exact_ref, route):
    R = exact_ref
    n = len(R["u"])
    print(f"exact route={route} n={n}", flush=True)
    ctx = cupk.Context(R["V"], R["C"], R["D"], R["S"], exact=True, **ROUTES[route])
    ctx.apply_updates(R["u"], R["v"], R["d"])
    a, g = ctx.get_sketch()
    assert np.array_equal(a, R["sk"].alpha) and np.array_equal(g, R["sk"].gamma)
    assert ctx.forest_edges() == R["fr"].forest_edges()
    c = ctx.counters()
    fr = R["fr"]
    assert fr.n_failed == 0 and c["sample_failed"] == 0
    assert (c["links"], c["cuts"], c["rounds"]) == (fr.n_links, fr.n_cuts, fr.n_rounds)
    if route in ("tiles", "pair", "two_levels"):
        # the passes through the tiles scatter whole and are undone
        assert c["reverts"] > 1000
    ctx.close()


@pytest.mark.parametrize("route", sorted(ROUTES))
def test_levels_mode_on_every_route(cupk, route):
    V, C, D, S = 2500, 9, 18, 0x5EED5000
    u, v, d = _toggles(300, 1100, 15_000, 6)
    u, v = u * 8 + 3, v * 8 + 3
    print(f"levels route={route} n={len(u)}", flush=True)
    ctx = cupk.Context(V, C, D, S, levels=True, **ROUTES[route])
    sk = oracle.Sketch(V, C, D, S)
    fr = oracle.LevelsReplay(sk)
    for s in range(0, len(u), 5000):
        ctx.apply_updates(u[s:s + 5000], v[s:s + 5000], d[s:s + 5000])
        fr.apply_batch(u[s:s + 5000], v[s:s + 5000], d[s:s + 5000])
        for j in range(1, C + 1):
            assert ctx.level_forest_edges(j) == fr.forest_edges(j), (s, j)
    assert ctx.digest() == sk.digest()
    ctr = ctx.counters()
    assert (ctr["links"], ctr["cuts"]) == (fr.n_links, fr.n_cuts)
    ctx.close()


@pytest.mark.parametrize("hub", [False, True])
@pytest.mark.parametrize("V,C,n", [
    # one block classifies up to 16,384 updates
    (65536, 16, 16384), (65536, 16, 16385),
    # the direct scatter ends: n * (C + 1) against 100,000 + V + C * V / 4
    (65536, 16, 25158), (65536, 16, 25159), (3001, 20, 5619), (3001, 20, 5620),
    # a block takes 32, 64, 128, 256 updates
    (65536, 4, 32768), (65536, 4, 32769), (300_000, 3, 65537), (300_000, 3, 131073),
    (70_001, 1, 20_000)])
def test_batches_where_routes_meet(cupk, V, C, n, hub):
    S, D = 0x10AD + n, 12
    rng = np.random.default_rng(n)
    k = np.unique(rng.integers(0, V, (2 * n, 2)), axis=0)
    if hub:
        k[: len(k) // 4, 0] = 11
        k = np.unique(k, axis=0)
    k = k[k[:, 0] != k[:, 1]]
    # one direction of each pair
    key = np.minimum(k[:, 0], k[:, 1]) * V + np.maximum(k[:, 0], k[:, 1])
    k = k[np.unique(key, return_index=True)[1]]
    k = k[rng.permutation(len(k))[:n]].astype(np.uint32)
    assert len(k) == n
    u, v = k[:, 0].copy(), k[:, 1].copy()
    print(f"routes V={V} C={C} n={n} hub={hub}", flush=True)
    ctx = cupk.Context(V, C, D, S)
    ref = oracle.Sketch(V, C, D, S)
    ctx.apply_updates(u, v, np.zeros(n, np.uint8))
    ref.apply(u, v)
    a, g = ctx.get_sketch()
    assert np.array_equal(a, ref.alpha) and np.array_equal(g, ref.gamma)
    assert ctx.num_components() == oracle.uf_components(V, u, v)[0]
    ctx.close()

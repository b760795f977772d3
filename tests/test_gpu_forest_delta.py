"""Small passes bring the device forest the few vertices that changed, larger
ones the pages (and block labels) of everything written since: batches of both
kinds in turn, on both sides of the list's length, against the oracle's replay.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,small,cuts,exact", [
    (3001, 60, 3, False),      # short lists
    (3001, 900, 200, False),   # lists beyond 1,024 writes: pages after all
    (16384, 300, 20, False),
    (3001, 60, 3, True),
])
def test_small_and_large_batches_in_turn(V, small, cuts, exact):
    import torch
    assert torch.cuda.is_available(), "GPU test on a machine without a GPU"
    import paper_2509_14433_amd as cupk
    C = max(1, int(np.ceil(np.log2(V))))
    S = 0xDE17A + V
    rng = np.random.default_rng(V + small)
    # (a lane layout named: batches beyond 4,096 updates take the tiles)
    ctx = cupk.Context(V, C, 2 * C, S, exact=exact, tile_layout=cupk.LAYOUT_RECORD)
    ref = oracle.Sketch(V, C, 2 * C, S)
    fr = oracle.ForestReplay(ref)
    live = set()

    def step(dels, n_new):
        ups = [(a, b, 1) for a, b in dels]
        live.difference_update(dels)
        while n_new:
            a, b = sorted(int(x) for x in rng.integers(0, V, 2))
            if a != b and (a, b) not in live and (a, b) not in gone:
                live.add((a, b))
                ups.append((a, b, 0))
                n_new -= 1
        p = rng.permutation(len(ups))
        u, v, d = (np.array([ups[i][k] for i in p]) for k in range(3))
        if exact:
            for x, y, z in zip(u, v, d):
                fr.apply_batch(np.array([x], np.uint32), np.array([y], np.uint32),
                               np.array([z], np.uint8))
        else:
            fr.apply_batch(u.astype(np.uint32), v.astype(np.uint32), d.astype(np.uint8))
        ctx.apply_updates(u.astype(np.uint32), v.astype(np.uint32), d.astype(np.uint8))
        assert ctx.forest_edges() == fr.forest_edges()
        assert ctx.num_components() == V - len(fr.forest_edges())

    gone = set()
    step([], 2 * V)
    for i in range(8):
        fe = sorted(fr.forest_edges())
        gone = {fe[j] for j in rng.choice(len(fe), cuts, replace=False)}
        n = 4200 if i % 3 == 2 and not exact else small
        print(f"V={V} batch {i} of {n} updates, {cuts} cuts", flush=True)
        step(sorted(gone), n - cuts)
    assert ctx.digest() == ref.digest()
    ctx.close()

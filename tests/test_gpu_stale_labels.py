"""A piece relabelled by the first replacement round reaches the device forest.

Two trees of several label pages each are joined by one edge.  The batch that
deletes it leaves two components, one of which takes a new label; an edge
inserted between them later, at vertices whose pages nothing else wrote, must
be seen as joining two trees.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split_rounds", [False, True])
def test_relabelled_piece_is_uploaded(split_rounds):
    import torch
    assert torch.cuda.is_available(), "GPU test on a machine without a GPU"
    import paper_2509_14433_amd as cupk
    V, n = 65536, 8192
    ctx = cupk.Context(V, seed=9, split_rounds=split_rounds)
    a = np.arange(1, n, dtype=np.uint32)
    u = np.concatenate([a // 2, n + a // 2, [5]]).astype(np.uint32)
    v = np.concatenate([a, n + a, [n + 7]]).astype(np.uint32)
    ctx.apply_updates(u, v, np.zeros(len(u), np.uint8))
    assert ctx.connected(0, 2 * n - 1)
    one = lambda x, y, d: ctx.apply_updates([x], [y], [d])  # noqa: E731
    one(5, n + 7, 1)
    assert not ctx.connected(0, 2 * n - 1)
    for x, y in ((4097, n + 5000), (3000, 2 * n - 3), (n - 1, n + 2049)):
        print(f"edge {x} {y}", flush=True)
        one(x, y, 0)
        assert ctx.connected(x, y) and ctx.connected(0, 2 * n - 1)
        one(x, y, 1)
        assert not ctx.connected(x, y) and not ctx.connected(0, 2 * n - 1)
    assert ctx.num_components() == V - 2 * n + 2
    ctx.close()

"""The build's radix sort and its pass over the unique keys at the edges of their tiles and tile sizes: the
particle order against a stable sort of the keys' definition in numpy, and the leaf counts (exact), for one
tree and for forests."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bh():
    import paper_1112_4539_amd as bh
    bh.load()
    assert torch.cuda.is_available()
    return bh


def _keys(pos):
    lo, hi = pos.min(0), pos.max(0)
    L = (hi - lo).max()
    L = L if L > 0 else 1.0
    q = np.clip(np.floor((pos - lo) * (2.0 ** 21 / L)), 0, 2 ** 21 - 1).astype(np.uint64)
    key = np.zeros(len(pos), np.uint64)
    for b in range(21):
        for d in range(3):
            key |= ((q[:, d] >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + 2 - d)
    return key


def _order(pos, off):
    return np.concatenate([b + np.argsort(_keys(pos[b:e]), kind="stable") if e > b else np.zeros(0, np.int64)
                           for b, e in zip(off[:-1], off[1:])])


@pytest.mark.parametrize("kind", ["random", "few"])
@pytest.mark.parametrize("n", [4097, 5119, 5120, 5121, (1 << 17) - 1, 1 << 17, (1 << 17) + 1, (1 << 19) - 3, 1 << 19,
                               (1 << 19) + 1, 3000001])
def test_sorted_order(bh, n, kind):
    print(f"[sort] n={n} {kind}", flush=True)
    rng = np.random.default_rng(n)
    # few: 37 distinct places, so that digits are shared by many items and order is by index
    pos = rng.random((n, 3)) if kind == "random" else rng.random((37, 3))[rng.integers(0, 37, n)]
    T = bh.Tree(torch.tensor(pos, device="cuda"), torch.ones(n, dtype=torch.float64, device="cuda"))
    for _ in range(2):          # a rebuild in the same workspace meets the words of the last one
        _, perm = T.export()
        np.testing.assert_array_equal(perm, _order(pos, [0, n]))
        assert T.stats()["n_leaves"] == len(np.unique(_keys(pos)))
        T = bh.Tree(T.pos, T.mass, T.workspace)
    w = T.walk_order().cpu().numpy()
    np.testing.assert_array_equal(np.sort(w), np.arange(n))


@pytest.mark.parametrize("K,per", [(3, 2000), (300, 40), (2047, 9), (2048, 9), (70000, 4)])
def test_sorted_order_forest(bh, K, per):
    print(f"[sort] forest of {K} clusters", flush=True)
    rng = np.random.default_rng(K)
    off = np.concatenate([[0], np.cumsum(rng.integers(0, 2 * per, K))]).astype(np.int64)
    pos = rng.random((off[-1], 3)).astype(np.float32)
    T = bh.build_forest(torch.tensor(pos, device="cuda"), torch.ones(off[-1], device="cuda"),
                        torch.tensor(off, device="cuda"))
    T.check()
    _, perm = T.export()
    np.testing.assert_array_equal(perm, _order(pos.astype(np.float64), off))
    np.testing.assert_array_equal(np.sort(T.walk_order().cpu().numpy()), np.arange(off[-1]))
    leaves = [len(np.unique(_keys(pos[b:e].astype(np.float64)))) if e > b else 0 for b, e in zip(off[:-1], off[1:])]
    assert T.stats()["n_leaves"] == sum(leaves)
    roots = T.roots().cpu().numpy()
    for k, u in enumerate(leaves):
        assert (roots[k + 1] - roots[k] > 0) == (u > 0)

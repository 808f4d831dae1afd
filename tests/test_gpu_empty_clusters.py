"""Forests with runs of empty clusters, at the start, between particles and at the end: every cluster's
root, and forces against the cluster alone."""
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


def _sizes(first, gaps, last, size):
    s = [0] * first
    for g in gaps:
        s += [size] + [0] * g
    return np.array(s + [size] + [0] * last, np.int64)


@pytest.mark.parametrize("sizes", [
    _sizes(0, [0, 1, 7, 8, 9, 10, 62, 63, 64, 65, 66, 127, 128, 129, 1000], 0, 3),
    _sizes(8, [8, 9], 1, 1), _sizes(9, [], 255, 1), _sizes(300, [7] * 700, 256, 5), _sizes(5000, [70] * 300, 257, 40),
    _sizes(0, [], 70000, 100), _sizes(70000, [], 0, 100)], ids=lambda s: f"{len(s)}c{s.sum()}")
def test_empty_clusters(bh, sizes):
    print(f"[empty] {len(sizes)} clusters, {sizes.sum()} particles", flush=True)
    off = np.concatenate([[0], np.cumsum(sizes)])
    rng = np.random.default_rng(len(sizes))
    pos = torch.tensor(rng.normal(size=(off[-1], 3)), dtype=torch.float32, device="cuda")
    mass = torch.tensor(rng.uniform(0.5, 1.5, off[-1]), dtype=torch.float32, device="cuda")
    T = bh.build_forest(pos, mass, torch.tensor(off, device="cuda"))
    T.check()
    rec = T.export()[0]
    roots = T.roots().cpu().numpy()
    assert roots[0] == 0 and roots[-1] == len(rec)
    full = np.flatnonzero(sizes)
    np.testing.assert_array_equal(roots[:-1][sizes == 0], roots[1:][sizes == 0])
    np.testing.assert_array_equal(rec["first"][roots[full]], off[full])
    np.testing.assert_array_equal(rec["count"][roots[full]], sizes[full])
    a, p = T.forces(0.5, 0.01)
    for k in {int(full[0]), int(full[len(full) // 2]), int(full[-1])}:
        b, e = off[k], off[k + 1]
        a1, p1 = bh.Tree(pos[b:e].contiguous(), mass[b:e].contiguous()).forces(0.5, 0.01)
        assert torch.equal(a[b:e], a1) and torch.equal(p[b:e], p1)

"""A group's walk shared by several waves against one wave per group: the same bits, at the sizes
where the runs of the subtree, the waves and the clusters change (no tolerance: the sums are taken
in the same order)."""
import numpy as np
import pytest
import torch

from paper_1112_4539_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bh():
    import paper_1112_4539_amd as bh
    bh.load()
    assert torch.cuda.is_available()
    return bh


def _same(T, **kw):
    a, p = T.forces(**kw)
    T.set_walk_config(waves_per_block=2)        # one wave per group
    a1, p1 = T.forces(**kw)
    T.set_walk_config(persistent=1)
    a2, p2 = T.forces(**kw)
    T.set_walk_config()
    assert torch.isfinite(a).all() and torch.isfinite(p).all()
    assert torch.equal(a, a1) and torch.equal(p, p1)
    assert torch.equal(a, a2) and torch.equal(p, p2)


@pytest.mark.parametrize("prec", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [1, 2, 3, 9, 63, 64, 65, 500, 1000, 16384, 16385, 32768, 32769, 65536, 65537, 102400, 102401])
def test_split_sizes(bh, n, prec):
    print(f"[split] n={n} {prec}", flush=True)
    pos, mass = inputs.plummer(n, n)
    if n > 400:
        pos[300:340] = pos[299]      # a leaf of many particles
    T = bh.Tree(torch.tensor(pos, dtype=prec, device="cuda"), torch.tensor(mass, dtype=prec, device="cuda"))
    _same(T, theta=0.5, eps=0.01)
    _same(T, theta=1.1, eps=0.0)     # cells that hold their target excluded by range
    T.set_order(2)
    _same(T, theta=0.6, eps=0.01)


@pytest.mark.parametrize("prec", [torch.float32, torch.float64])
def test_split_group_theta(bh, prec):
    print(f"[split] theta per group {prec}", flush=True)
    pos, mass = inputs.clumpy(30_011, 4)
    T = bh.Tree(torch.tensor(pos, dtype=prec, device="cuda"), torch.tensor(mass, dtype=prec, device="cuda"))
    tg = torch.tensor(np.random.default_rng(2).uniform(0.25, 1.1, T.n_groups), dtype=torch.float32, device="cuda")
    for order in (1, 2):
        T.set_order(order)
        _same(T, eps=1e-4, theta_group=tg)


@pytest.mark.parametrize("sizes", [[1, 0, 64, 700, 3, 0, 9000, 62], [5] * 200, [1] * 1025, [65536 - 64, 64]])
def test_split_forest(bh, sizes):
    print(f"[split] forest of {len(sizes)} clusters", flush=True)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rng = np.random.default_rng(len(sizes))
    pos = torch.tensor(rng.normal(size=(off[-1], 3)), dtype=torch.float32, device="cuda")
    mass = torch.tensor(rng.uniform(0.5, 1.5, off[-1]), dtype=torch.float32, device="cuda")
    T = bh.build_forest(pos, mass, torch.tensor(off, device="cuda"))
    _same(T, theta=0.5, eps=0.01)
    k = int(np.argmax(sizes))
    a, p = T.forces(0.5, 0.01)
    b, e = off[k], off[k + 1]
    a1, p1 = bh.Tree(pos[b:e].contiguous(), mass[b:e].contiguous()).forces(0.5, 0.01)
    assert torch.equal(a[b:e], a1) and torch.equal(p[b:e], p1)

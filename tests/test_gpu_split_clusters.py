"""Forests whose groups hold several clusters: small ones are walked by one wave of the workgroup, the
others shared, and both must give the bits of one wave per group (the sums are taken in the same
order).  Clusters around the sizes where the rule changes, alone and among large ones."""
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


def _mixed(K, hi, seed):
    rng = np.random.default_rng(seed)
    s = np.floor(np.exp(rng.uniform(0, np.log(hi), K))).astype(np.int64)
    s[rng.choice(K, K // 8, replace=False)] = 0
    return s


SETS = dict(ones=np.ones(700, np.int64), twos=np.full(300, 2), eights=np.full(128, 8), nines=np.full(1000, 9),
            thirties=np.full(60, 30), large_between=np.array([1, 2, 3000, 4, 5, 6, 1, 1, 9000, 1, 7, 0, 0, 33, 40, 3]),
            mixed=_mixed(1024, 300, 1), mixed_large=_mixed(200, 5000, 2), sparse=np.where(np.arange(1000) % 37 == 5, 11, 0))


@pytest.mark.parametrize("prec", [torch.float32, torch.float64])
@pytest.mark.parametrize("name", SETS)
def test_split_clusters(bh, name, prec):
    sizes = SETS[name]
    print(f"[split clusters] {name}: {len(sizes)} clusters, {sizes.sum()} particles {prec}", flush=True)
    off = np.concatenate([[0], np.cumsum(sizes)])
    rng = np.random.default_rng(len(sizes))
    pos = rng.normal(size=(off[-1], 3))
    pos[off[-1] // 2] = pos[off[-1] // 2 - 1]     # (a leaf of two, if both lie in one cluster)
    T = bh.build_forest(torch.tensor(pos, dtype=prec, device="cuda"),
                        torch.tensor(rng.uniform(0.5, 1.5, off[-1]), dtype=prec, device="cuda"),
                        torch.tensor(off, device="cuda"))
    T.check()
    tg = torch.tensor(rng.uniform(0.25, 1.1, T.n_groups), dtype=torch.float32, device="cuda")
    for order in (1, 2):
        T.set_order(order)
        for kw in (dict(theta=0.5, eps=0.01), dict(theta=1.1, eps=0.0), dict(eps=0.01, theta_group=tg)):
            T.set_walk_config()
            a, p = (x.fill_(float("nan")) for x in T._outs(None, None))
            T.forces(acc=a, pot=p, **kw)
            T.set_walk_config(waves_per_block=2)
            a1, p1 = T.forces(**kw)
            assert torch.isfinite(a).all() and torch.equal(a, a1) and torch.equal(p, p1)

"""Walks never depend on the caller's offsets array: how a cluster's subtree is cut into runs (and the
LDS that holds the runs' sums) follows from the tree as it was built.  Bits against the same tree
built from good offsets."""
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


def _set(n, prec=torch.float32):
    pos, mass = inputs.plummer(n, n)
    return torch.tensor(pos, dtype=prec, device="cuda"), torch.tensor(mass, dtype=prec, device="cuda")


@pytest.mark.parametrize("n", [100, 4097, 32769, 65537, 102400])
@pytest.mark.parametrize("off", [(0, 1), (0, 99), (3, 0), (-5, 1 << 40)])
def test_one_cluster_bad_offsets(bh, n, off):
    print(f"[offsets] one cluster of {n}, offsets {off}", flush=True)
    pos, mass = _set(n)
    good = bh.Tree(pos, mass)
    a, p = good.forces(0.5, 0.01)
    T = bh.build_forest(pos, mass, torch.tensor(off, device="cuda"))
    with pytest.raises(ValueError):
        T.check()
    for cfg in (dict(), dict(waves_per_block=2)):
        T.set_walk_config(**cfg)
        a1, p1 = T.forces(0.5, 0.01)
        assert torch.equal(a, a1) and torch.equal(p, p1)


def test_offsets_changed_after_the_build(bh):
    print("[offsets] the offsets array rewritten between build and walk", flush=True)
    sizes = np.array([40000, 3, 0, 500, 20000])
    off = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]), device="cuda")
    pos, mass = _set(int(sizes.sum()))
    T = bh.build_forest(pos, mass, off)
    T.check()
    a, p = T.forces(0.5, 0.01)
    off.copy_(torch.tensor([0, 9, 10, 11, 12, int(sizes.sum())]))
    for cfg in (dict(), dict(waves_per_block=2)):
        T.set_walk_config(**cfg)
        a1, p1 = T.forces(0.5, 0.01)
        assert torch.equal(a, a1) and torch.equal(p, p1)

"""The one-launch build of small trees at the edges of its range, against the oracle (bit-exact:
node set, order, links, moments, walk order)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import hilbert

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bh():
    import paper_1112_4539_amd as bh
    bh.load()
    assert torch.cuda.is_available()
    return bh


def _set(kind, n):
    rng = np.random.default_rng(n)
    if kind == "random":
        return rng.random((n, 3))
    if kind == "clumps":         # deep chains: pairs 2^-20 of the cube apart, and coincident ones
        p = rng.random((n, 3))
        p[n // 2:] = p[:n - n // 2] + 2.0 ** -20
        p[n - n // 8:] = p[:n // 8]
        return p
    if kind == "lattice":
        k = int(np.ceil(n ** (1 / 3)))
        g = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3)
        return g[rng.permutation(len(g))[:n]] / k
    return np.tile(rng.random((1, 3)), (n, 1))


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kind,n", [("random", n) for n in (1, 2, 63, 64, 65, 256, 257, 1023, 1024, 1025, 4095, 4096,
                                                            4097)] +
                         [("clumps", 1000), ("clumps", 4096), ("lattice", 512), ("lattice", 4096),
                          ("coincident", 4096), ("coincident", 2)])
def test_small_build(bh, kind, n, prec):
    print(f"[small build] {kind} n={n} {prec}", flush=True)
    dt = np.float32 if prec == "fp32" else np.float64
    pos = _set(kind, n).astype(dt)
    mass = np.random.default_rng(n + 1).uniform(0.5, 1.5, n).astype(dt)
    T = bh.Tree(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"))
    T.check()
    rec, perm = T.export()
    p64, m64 = pos.astype(np.float64), mass.astype(np.float64)
    O = oracle.Tree(p64, m64)
    assert len(rec) == O.n_nodes and T.stats()["n_leaves"] == int(O.leaf.sum())
    np.testing.assert_array_equal(perm, O.perm)
    np.testing.assert_array_equal(rec["meta"] & 1, O.leaf)
    np.testing.assert_array_equal(rec["meta"] >> 8, O.level)
    for f in ("first", "count", "next", "com", "M", "l", "s"):
        np.testing.assert_array_equal(rec[f], getattr(O, f))
    np.testing.assert_array_equal(T.roots().cpu().numpy(), [0, O.n_nodes])
    np.testing.assert_array_equal(T.walk_order().cpu().numpy(), hilbert.walk_order(p64, m64))


def test_small_build_reports(bh):
    """What the build reports of its inputs: offsets that do not cover the particles, non-finite values."""
    print("[small build] reports", flush=True)
    pos, mass = torch.rand((1000, 3), device="cuda"), torch.ones(1000, device="cuda")
    ok = bh.build_forest(pos, mass, torch.tensor([0, 1000], device="cuda"))
    ok.check()
    bad = bh.build_forest(pos, mass, torch.tensor([0, 999], device="cuda"))
    with pytest.raises(ValueError):
        bad.check()
    for x in (float("nan"), float("inf")):
        p, m = pos.clone(), mass.clone()
        p[999, 2] = x
        m[3] = x
        for a, b in ((p, mass), (pos, m)):
            with pytest.raises(ValueError):
                bh.Tree(a, b).check()

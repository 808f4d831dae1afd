"""The small build's sort where many particles share the upper key bits: cells ten levels down with
runs of 15 to 18 particles around the length that is put into order by insertion, longer ones and
cores that hold nearly everything, with distinct and repeated keys in shuffled order.  Bit-exact
against the oracle."""
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


CELL = 2.0 ** -11   # (the upper 32 of 63 key bits: ten levels and two bits of the eleventh)


def _set(kind, n):
    rng = np.random.default_rng(n)
    if kind == "core":       # all but three particles in one such cell
        p = 0.25 + CELL * 0.9 * rng.random((n, 3))
        p[0], p[1], p[2] = 0.0, 1.0, 0.75
        return p[rng.permutation(n)]
    # cells of `k` particles each, every fourth particle of a cell a copy of another's position
    k = int(kind)
    cells = rng.integers(1, 400, (n // k + 1, 3)) * 2 * CELL
    p = np.repeat(cells, k, axis=0)[:n] + CELL * 0.9 * rng.random((n, 3))
    p[3::4] = p[2::4][: len(p[3::4])]
    p[0], p[1] = 0.0, 1.0
    return p[rng.permutation(n)]


def _longest(pos):
    lo, L = pos.min(0), (pos.max(0) - pos.min(0)).max()
    q = np.clip(np.floor((pos - lo) * (2.0 ** 21 / L)), 0, 2 ** 21 - 1).astype(np.uint64)
    key = np.zeros(len(pos), np.uint64)
    for b in range(21):
        for d in range(3):
            key |= ((q[:, d] >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + 2 - d)
    u, c = np.unique(key >> np.uint64(31), return_counts=True)
    return int(c.max()), len(np.unique(key))


CASES = [("core", 20), ("core", 700), ("core", 4096), ("15", 900), ("16", 960), ("17", 1020), ("18", 1080),
         ("16", 4096), ("17", 4096), ("40", 4000), ("300", 3000)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kind,n", CASES)
def test_small_runs(bh, kind, n, prec):
    dt = np.float32 if prec == "fp32" else np.float64
    pos = _set(kind, n).astype(dt)
    longest, keys = _longest(pos.astype(np.float64))
    print(f"[small runs] {kind} n={n} {prec}: longest run {longest}, {keys} keys", flush=True)
    assert longest >= (n - 3 if kind == "core" else int(kind) - 1) and keys > n // 2
    mass = np.random.default_rng(n + 1).uniform(0.5, 1.5, n).astype(dt)
    T = bh.Tree(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"))
    T.check()
    rec, perm = T.export()
    p64, m64 = pos.astype(np.float64), mass.astype(np.float64)
    O = oracle.Tree(p64, m64)
    assert len(rec) == O.n_nodes
    np.testing.assert_array_equal(perm, O.perm)
    np.testing.assert_array_equal(rec["meta"] & 1, O.leaf)
    np.testing.assert_array_equal(rec["meta"] >> 8, O.level)
    for f in ("first", "count", "next", "com", "M", "l", "s"):
        np.testing.assert_array_equal(rec[f], getattr(O, f))
    np.testing.assert_array_equal(T.walk_order().cpu().numpy(), hilbert.walk_order(p64, m64))

"""Walks at the tree sizes where the number of runs changes, in every launch shape: the same bits (the
runs' sums are added in the same order however a group is walked), and FP64 forces within 1e-12 of the
oracle.  The shape that reads records through LDS keeps its place from run to run."""
import numpy as np
import pytest
import torch

import oracle
from paper_1112_4539_amd import inputs
from tests.util import check_forces, pot_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bh():
    import paper_1112_4539_amd as bh
    bh.load()
    assert torch.cuda.is_available()
    return bh


SHAPES = [dict(waves_per_block=4), dict(lds_share=64), dict(waves_per_block=2, lds_share=32), dict(persistent=1),
          dict(persistent=1, lds_share=64), dict(targets_per_lane=2), dict(targets_per_lane=2, lds_share=64)]


@pytest.mark.parametrize("buckets", [False, True])
@pytest.mark.parametrize("prec", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [64, 65, 768, 769, 5000, 32769])
def test_run_edges(bh, n, prec, buckets):
    print(f"[runs] n={n} {prec} buckets={buckets}", flush=True)
    pos, mass = inputs.plummer(n, n)
    if buckets:
        pos[5:25] = pos[4]
        pos[40:43] = pos[39]
    T = bh.Tree(torch.tensor(pos, dtype=prec, device="cuda"), torch.tensor(mass, dtype=prec, device="cuda"))
    tg = torch.tensor(np.random.default_rng(n).uniform(0.25, 1.1, T.n_groups), dtype=torch.float32, device="cuda")
    for order in (1, 2):
        T.set_order(order)
        for kw in (dict(theta=0.5, eps=0.01), dict(theta=1.1, eps=0.0), dict(eps=0.01, theta_group=tg)):
            T.set_walk_config()
            a, p = T.forces(**kw)
            assert torch.isfinite(a).all()
            for shape in SHAPES:
                T.set_walk_config(**shape)
                a1, p1 = T.forces(**kw)
                assert torch.equal(a, a1) and torch.equal(p, p1), (order, kw, shape)
            T.set_walk_config()
            s = T.walk_stats(**kw)
            assert torch.equal(a, s["acc"]) and torch.equal(p, s["pot"])
    if prec == torch.float64 and n < 5000:
        T.set_order(1)
        w = oracle.Tree(pos, mass).walk(0.5, 0.01)
        a, p = T.forces(0.5, 0.01)
        check_forces(a.cpu().numpy(), w["acc"], w["amag"], 1e-12, f"n={n}")
        assert pot_err(p.cpu().numpy(), w["pot"]).max() <= 1e-12

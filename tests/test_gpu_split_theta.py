"""FP64 walks with a theta per group, shared by several waves, for each variant of their loop (cells
that may hold a target of theta > 1, leaves of several particles): the bits of one wave per group,
and of the uniform walk where every group has the same theta."""
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


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("buckets", [False, True])
@pytest.mark.parametrize("theta", [0.5, 1.125])
@pytest.mark.parametrize("n", [70, 5000, 40000])
def test_split_theta_fp64(bh, n, theta, buckets, order):
    print(f"[split theta] n={n} theta={theta} buckets={buckets} order={order}", flush=True)
    pos, mass = inputs.plummer(n, n)
    if buckets:
        pos[10:30] = pos[9]
    T = bh.Tree(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"))
    T.set_order(order)
    tg = torch.full((T.n_groups,), theta, dtype=torch.float32, device="cuda")
    a, p = T.forces(eps=0.01, theta_group=tg)
    u, q = T.forces(theta, 0.01)
    assert torch.isfinite(a).all() and torch.equal(a, u) and torch.equal(p, q)
    T.set_walk_config(waves_per_block=2)
    a1, p1 = T.forces(eps=0.01, theta_group=tg)
    assert torch.equal(a, a1) and torch.equal(p, p1)
    T.check()

"""Range of the FP64 pair term: r^-1 is a refined hardware root, so powers of two must pass through
it exactly from the smallest to the largest distances whose terms are finite, and distances whose
square overflows must add nothing."""
import sys

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
@pytest.mark.parametrize("eps", [0.0, 2.0 ** -6])
@pytest.mark.parametrize("k", [-180, -40, 40, 180, 600])
def test_fp64_terms_scale_exactly(bh, k, eps, order):
    print(f"[fp64 term] positions and eps times 2^{k}, eps {eps}, order {order}", flush=True)
    sys.stdout.flush()
    pos, mass = inputs.plummer(1500, 3)
    pos = torch.tensor(pos, device="cuda")
    mass = torch.tensor(mass, device="cuda")

    def forces(scale):
        t = bh.Tree(pos * scale, mass)
        t.set_order(order)
        return t.forces(0.5, eps * scale)

    if k == 600 and order == 2:
        pytest.skip("second moments overflow")
    a1, p1 = forces(1.0)
    a2, p2 = forces(2.0 ** k)
    if k == 600:
        assert torch.all(a2 == 0) and torch.all(p2 == 0)
    else:
        assert torch.equal(a2 * 2.0 ** k * 2.0 ** k, a1) and torch.equal(p2 * 2.0 ** k, p1)

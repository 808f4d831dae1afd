"""r^-1 of the FP64 pair term within 1 ulp of the exact value, over the exponents and mantissas of r^2.

The bound: half an ulp from the last sum, at most half from the rounding of x y, 2^-12 from the term
left out of the series; and 2^-11 for the 64-bit-mantissa reference."""
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


# (30,000 targets: one lane each; 3000: eight; 700: 32)
@pytest.mark.parametrize("n", [30000, 3000, 700])
@pytest.mark.parametrize("lo,hi", [(0, 0), (-30, 30), (-500, 500)])
def test_root_ulp(bh, n, lo, hi):
    """The potential of a unit mass at the origin is -r^-1; the other sources have no mass."""
    print(f"[root ulp] {n} distances of exponents {lo}..{hi}", flush=True)
    rng = np.random.default_rng(n + hi)
    x = np.ldexp(1.0 + rng.random(n), rng.integers(lo, hi + 1, n))
    pos = np.zeros((n + 1, 3))
    pos[1:, 0] = x
    mass = np.zeros(n + 1)
    mass[0] = 1.0
    _, pot = bh.direct(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"), 0.0,
                       torch.arange(1, n + 1, device="cuda"))
    got = -pot.cpu().numpy()
    ref = 1 / np.sqrt((x * x).astype(np.longdouble))
    assert np.finfo(np.longdouble).nmant >= 63
    err = np.abs(got.astype(np.longdouble) - ref) / np.spacing(ref.astype(np.float64)).astype(np.longdouble)
    print(f"  largest error {float(err.max()):.4f} ulp", flush=True)
    assert err.max() <= 1 + 2.0 ** -12 + 2.0 ** -11

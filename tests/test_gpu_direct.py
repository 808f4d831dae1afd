"""The direct sum at the edges of its launch rules (targets per workgroup, lanes per target, waves
over the sources) against a float64 sum on the CPU.

Bounds: a lane sums at most n/4 sources in a row, so an output is within (n/4 + 32) rounding units
of the sum of its terms' magnitudes A (2^-24 for FP32 terms and sums, 2^-53 for FP64; a term's own
error, at most a dozen units, is in the 32)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bh():
    import paper_1112_4539_amd as bh
    bh.load()
    assert torch.cuda.is_available()
    return bh


@pytest.mark.parametrize("eps", [0.0, 0.01])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,nt", [(1, 1), (3, 2), (127, 64), (1030, 511), (4099, 2047), (4099, 2048), (515, 2113),
                                  (1030, 10239), (1030, 10240), (259, 16449)])
def test_direct_launch_rules(bh, n, nt, prec, eps):
    print(f"[direct] n={n} targets={nt} {prec} eps={eps}", flush=True)
    g = torch.Generator().manual_seed(n + nt)
    dt = torch.float32 if prec == "fp32" else torch.float64
    pos = torch.rand((n, 3), generator=g, dtype=torch.float64)
    if n > 100:
        pos[n - 1] = pos[0]  # a coincident pair
    pos, mass = pos.to(dt), (torch.rand(n, generator=g, dtype=torch.float64) + 0.5).to(dt)
    tg = torch.randint(0, n, (nt,), generator=g)
    tg[0] = 0
    tg[-1] = n - 1
    acc, pot = bh.direct(pos.cuda(), mass.cuda(), eps, tg.cuda())
    x, m = pos.double(), mass.double()
    d = x[None] - x[:, None]
    r2 = (d * d).sum(2) + eps * eps
    w = torch.where(r2 > 0, r2, torch.ones_like(r2)) ** -0.5
    w[r2 == 0] = 0.0
    w.fill_diagonal_(0.0)
    f = (m * w ** 3)[:, :, None] * d
    a_ref, a_mag = f.sum(1), f.norm(dim=2).sum(1)
    p_mag = (m * w).sum(1)
    unit = (n / 4 + 32) * (2.0 ** -24 if prec == "fp32" else 2.0 ** -53)
    assert torch.all((acc.cpu().double() - a_ref[tg]).norm(dim=1) <= 2 * unit * a_mag[tg])
    assert torch.all((pot.cpu().double() + p_mag[tg]).abs() <= unit * p_mag[tg])


def test_direct_target_out_of_range(bh):
    print("[direct] targets outside [0, n) give NaN, the others are untouched", flush=True)
    pos = torch.rand((500, 3), device="cuda", dtype=torch.float64)
    mass = torch.ones(500, device="cuda", dtype=torch.float64)
    tg = torch.tensor([3, -1, 499, 500, 7], device="cuda")
    acc, pot = bh.direct(pos, mass, 0.01, tg)
    ok = torch.tensor([True, False, True, False, True], device="cuda")
    assert torch.all(torch.isnan(pot) == ~ok) and torch.all(torch.isnan(acc).all(1) == ~ok)

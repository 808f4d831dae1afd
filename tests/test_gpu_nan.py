"""Particles that are not numbers: a NaN position reaches every FP64 sum it belongs to, softened or
not, and a coincident pair without softening adds nothing whatever its mass."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bh():
    import paper_1112_4539_amd as bh
    bh.load()
    assert torch.cuda.is_available()
    return bh


# (lanes per target: 32, 8 and 1)
SHAPES = [(67, 5), (300, 511), (1030, 2113), (1030, 10240)]


@pytest.mark.parametrize("eps", [0.0, 0.01])
@pytest.mark.parametrize("n,nt", SHAPES)
def test_direct_nan_position(bh, n, nt, eps):
    print(f"[nan] direct n={n} targets={nt} eps={eps}", flush=True)
    g = torch.Generator().manual_seed(n)
    pos = torch.rand((n, 3), generator=g, dtype=torch.float64)
    pos[n // 2, 1] = float("nan")
    tg = torch.randint(0, n, (nt,), generator=g)
    acc, pot = bh.direct(pos.cuda(), torch.ones(n, dtype=torch.float64, device="cuda"), eps, tg.cuda())
    # (one coordinate is NaN, so r^2 is, and with it every component's factor)
    assert torch.isnan(pot).all() and torch.isnan(acc).all()


@pytest.mark.parametrize("n,nt", SHAPES)
@pytest.mark.parametrize("m", [float("inf"), float("nan")])
def test_direct_coincident_mass(bh, n, nt, m):
    print(f"[nan] direct n={n} targets={nt} coincident mass {m}", flush=True)
    g = torch.Generator().manual_seed(n)
    pos = torch.rand((n, 3), generator=g, dtype=torch.float64)
    pos[n - 1] = pos[0]
    tg = torch.zeros(nt, dtype=torch.int64)
    mass = torch.ones(n, dtype=torch.float64)
    a, p = bh.direct(pos.cuda(), mass.cuda(), 0.0, tg.cuda())
    mass[n - 1] = m
    a1, p1 = bh.direct(pos.cuda(), mass.cuda(), 0.0, tg.cuda())
    assert torch.isfinite(a).all() and torch.equal(a, a1) and torch.equal(p, p1)


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("eps", [0.0, 0.01])
@pytest.mark.parametrize("n", [500, 5000])
def test_walk_nan_position(bh, n, eps, order):
    """Three NaN coordinates take the key of the cube's lowest corner: with a particle there, a leaf of
    two that every target's walk reaches."""
    print(f"[nan] walk n={n} eps={eps} order={order}", flush=True)
    pos = torch.rand((n, 3), generator=torch.Generator().manual_seed(n), dtype=torch.float64)
    pos[3] = 0.0
    pos[n // 2] = float("nan")
    T = bh.Tree(pos.cuda(), torch.ones(n, dtype=torch.float64, device="cuda"))
    with pytest.raises(ValueError):
        T.check()
    T.set_order(order)
    for cfg in (dict(), dict(waves_per_block=2)):
        T.set_walk_config(**cfg)
        acc, pot = T.forces(0.5, eps)
        assert torch.isnan(pot).all() and torch.isnan(acc).all()

"""The work that a user of this library has it do, as cases that can be timed and checked.

Sizes, softenings and opening parameters are those of the benchmark's and the
tests' workloads (Plummer 4K and 1M, clumpy 4M, the forest of 512 clusters, the
neighbour search, the time loop, the learned opening parameter), and generic
ragged sizes between them.  Inputs are drawn on the GPU from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1112_4539_amd as bh
from paper_1112_4539_amd import learn

DTYPE = {"fp32": torch.float32, "fp64": torch.float64}
EPS = {"plummer": 0.005, "clumpy": 1e-4, "cube": 1e-3}


def listed():
    return [
        # the smallest call: a serving loop or a captured program that hands over a thousand
        # particles and may not allocate
        dict(name="noalloc_1k_fp32", kind="noalloc", dist="plummer", n=1000, prec="fp32", theta=0.5, eps=0.01),
        # a small cluster in full precision: tree and forces of one integration step
        dict(name="forces_4k_fp64", kind="forces", dist="plummer", n=4096, prec="fp64", theta=0.5, eps=0.01, order=1),
        # an ordinary mid-size set of ragged size
        dict(name="forces_100k_fp32", kind="forces", dist="plummer", n=100003, prec="fp32", theta=0.5, eps=0.005,
             order=1),
        # the headline: the largest single force calculation, at its accuracy target
        dict(name="forces_clumpy4m_fp32", kind="forces", dist="clumpy", n=4194304, prec="fp32", theta=0.35, eps=1e-4,
             order=1),
        # the same in double precision, for reference-quality runs
        dict(name="forces_plummer1m_fp64", kind="forces", dist="plummer", n=1048576, prec="fp64", theta=0.5, eps=0.005,
             order=1),
        # quadrupole cell terms: fewer, dearer interactions at equal accuracy
        dict(name="quadrupole_1m_fp32", kind="forces", dist="clumpy", n=1000003, prec="fp32", theta=0.59, eps=1e-4,
             order=2),
        # SPH: tree, neighbour search and density
        dict(name="neighbours_4m_fp32", kind="neighbours", dist="clumpy", n=4194304, prec="fp32", radius=2e-3,
             maxlen=0),
        # many independent clusters in one build and one walk
        dict(name="forest_512_fp32", kind="forest", clusters=512, nmin=1024, nmax=65536, prec="fp32", theta=0.5,
             eps=0.01),
        # the time loop: one kick-drift-kick step with its rebuild
        dict(name="leapfrog_1m_fp32", kind="leapfrog", dist="clumpy", n=1048576, prec="fp32", theta=0.35, eps=1e-4,
             dt=1e-5, order=1, reorder=False),
        # the learned opening parameter: tree, features, network, walk with one theta per group
        dict(name="learned_1m_fp32", kind="learned", dist="clumpy", n=1048576, prec="fp32", eps=1e-4, alpha=0.89),
        # one training step of that network on a minibatch
        dict(name="train_4096", kind="train", rows=131072, batch=4096),
        # the direct sum that judges accuracy and makes the labels, for sampled targets
        dict(name="direct_64k_fp64", kind="direct", dist="clumpy", n=262147, targets=65536, prec="fp64", eps=1e-4),
    ]


# interactions of the largest listed force calculation, and pairs of the listed direct sum
_MOST = 1.8e10
_MOST_DIRECT = 262147 * 65536


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["noalloc", "forces", "forces", "forces", "neighbours", "forest", "leapfrog", "learned",
                       "train", "direct"])
    dist = rng.choice(["plummer", "clumpy", "cube"])
    prec = rng.choice(["fp32", "fp64"])
    theta = round(rng.uniform(0.3, 0.75), 2)
    eps = rng.choice([EPS[dist], 0.01])
    if kind == "noalloc":
        return dict(kind=kind, dist=dist, n=size(200, 65536), prec=prec, theta=theta, eps=eps)
    if kind in ("forces", "leapfrog"):
        n = size(1000, 4194304)
        while n * _per_target(n, theta) * (4.0 if prec == "fp64" else 1.0) > _MOST:
            n = size(1000, 4194304)
        c = dict(kind=kind, dist=dist, n=n, prec=prec, theta=theta, eps=eps, order=rng.choice([1, 1, 2]))
        if kind == "leapfrog":
            c.update(dt=1e-5, reorder=rng.choice([False, True]))
        return c
    if kind == "neighbours":
        n = size(20000, 4194304)
        # radii around those that give a few dozen neighbours
        base = 2e-3 if dist == "clumpy" else 0.03 if dist == "plummer" else 0.013
        r = base * (4194304 / n) ** (1 / 3) * rng.uniform(0.6, 1.2)
        return dict(kind=kind, dist=dist, n=n, prec=prec, radius=float("%.3g" % r), maxlen=rng.choice([0, 0, 32]))
    if kind == "forest":
        return dict(kind=kind, clusters=size(2, 400), nmin=size(200, 2000), nmax=size(4000, 60000), prec="fp32",
                    theta=max(theta, 0.5), eps=0.01)
    if kind == "learned":
        return dict(kind=kind, dist="clumpy", n=size(65536, 2097152), prec="fp32", eps=1e-4, alpha=0.89)
    if kind == "train":
        return dict(kind=kind, rows=size(20000, 262144), batch=size(256, 16384))
    n = size(2000, 1048576)
    return dict(kind=kind, dist=dist, n=n, targets=min(n, size(512, max(512, min(65536, _MOST_DIRECT // n)))),
                prec=prec, eps=eps)


# ---------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _plummer(n, g, a=1.0, rmax=10.0):
    """Truncated Plummer sphere, float64 [n, 3] (the inverse of its mass profile)."""
    u, v, w = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) for _ in range(3))
    x = (u * (rmax / a) ** 3 / ((rmax / a) ** 2 + 1.0) ** 1.5).clamp_min(1e-12)
    r = a / torch.sqrt(x ** (-2.0 / 3.0) - 1.0)
    ct = 2.0 * v - 1.0
    st = torch.sqrt((1.0 - ct * ct).clamp_min(0.0))
    ph = 2.0 * math.pi * w
    return torch.stack([r * st * torch.cos(ph), r * st * torch.sin(ph), r * ct], 1)


def _positions(dist, n, g):
    if dist == "plummer":
        return _plummer(n, g)
    if dist == "cube":
        return torch.rand((n, 3), generator=g, device="cuda", dtype=torch.float64)
    # clumpy: a quarter uniform in the unit cube, the rest in 64 small Plummer clumps
    per = (n - int(round(0.25 * n))) // 64
    centres = torch.rand((64, 3), generator=g, device="cuda", dtype=torch.float64)
    clumps = _plummer(64 * per, g, a=0.01, rmax=0.1) + centres.repeat_interleave(per, 0)
    return torch.cat([torch.rand((n - 64 * per, 3), generator=g, device="cuda", dtype=torch.float64), clumps])


def _sizes(case):
    """Cluster sizes of a forest: spread evenly over their logarithm."""
    K = case["clusters"]
    q = (np.arange(K) + 0.5) / K
    return np.floor(np.exp(math.log(case["nmin"]) + q * math.log(case["nmax"] / case["nmin"]))).astype(np.int64)


def _inputs(case, seed):
    """The arrays that a case's program holds (on the GPU), from the seed alone."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "train":
        X = torch.randn((case["rows"], 8), generator=g, device="cuda", dtype=torch.float32)
        target = torch.rand(case["rows"], generator=g, device="cuda", dtype=torch.float32)
        rows = torch.randperm(case["rows"], generator=g, device="cuda")[: case["batch"]].to(torch.int32)
        return dict(X=X, target=target, rows=rows, params=learn.init_params(int(seed)))
    dt = DTYPE[case["prec"]]
    if kind == "forest":
        sizes = _sizes(case)
        sizes = sizes[np.random.default_rng(int(seed)).permutation(len(sizes))]
        n = int(sizes.sum())
        pos = _plummer(n, g).to(dt)
        cl = torch.tensor(sizes, device="cuda")
        off = torch.zeros(len(sizes) + 1, dtype=torch.int64, device="cuda")
        off[1:] = torch.cumsum(cl, 0)
        return dict(pos=pos, mass=(1.0 / cl.double()).repeat_interleave(cl).to(dt), offsets=off)
    n = case["n"]
    d = dict(pos=_positions(case["dist"], n, g).to(dt),
             mass=torch.full((n,), 1.0 / n, dtype=dt, device="cuda"))
    if kind == "leapfrog":
        d["vel"] = (0.01 * torch.randn((n, 3), generator=g, device="cuda", dtype=torch.float64)).to(dt)
    if kind == "direct":
        d["targets"] = torch.randperm(n, generator=g, device="cuda")[: case["targets"]].sort().values
    return d


# ---------------------------------------------------------------- the program
def prepare(case, seed):
    s = dict(case=case, **_inputs(case, seed))
    kind = case["kind"]
    if kind == "train":
        norm = torch.cat([s["X"].mean(0), 1.0 / s["X"].std(0)])
        s["net"] = bh.MLP(s["params"], norm)
        return s
    n, dt = s["pos"].shape[0], s["pos"].dtype
    if kind in ("forces", "neighbours", "forest", "leapfrog", "learned"):
        K = case.get("clusters", 1)
        s["ws"] = torch.empty(bh.forest_workspace_bytes(n, K, bh.FP64 if dt == torch.float64 else bh.FP32),
                              dtype=torch.uint8, device="cuda")
    if kind in ("forces", "forest", "noalloc", "leapfrog", "learned"):
        s["acc"] = torch.empty((n, 3), dtype=dt, device="cuda")
        s["pot"] = torch.empty((n,), dtype=dt, device="cuda")
    if kind == "leapfrog":
        t = bh.build_tree(s["pos"], s["mass"], s["ws"])
        t.set_order(case["order"])
        t.forces(case["theta"], case["eps"], s["acc"], s["pot"])
        s["ids"] = torch.arange(n, dtype=torch.int64, device="cuda")
    if kind == "learned":
        s["net"] = learn.load_net()[0]
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "noalloc":
        return bh.forces_noalloc(s["pos"], s["mass"], case["theta"], case["eps"], s["acc"], s["pot"])
    if kind == "forces":
        t = bh.build_tree(s["pos"], s["mass"], s["ws"])
        if case["order"] != 1:
            t.set_order(case["order"])
        return t.forces(case["theta"], case["eps"], s["acc"], s["pot"])
    if kind == "forest":
        t = bh.build_forest(s["pos"], s["mass"], s["offsets"], s["ws"])
        return t.forces(case["theta"], case["eps"], s["acc"], s["pot"])
    if kind == "neighbours":
        return bh.build_tree(s["pos"], s["mass"], s["ws"]).neighbours(case["radius"], maxlen=case["maxlen"])
    if kind == "leapfrog":
        bh.leapfrog_step(s["pos"], s["vel"], s["mass"], s["acc"], s["pot"], case["dt"], case["theta"], case["eps"],
                         order=case["order"], reorder=case["reorder"], ids=s["ids"], workspace=s["ws"])
        return dict(pos=s["pos"], vel=s["vel"], acc=s["acc"], pot=s["pot"], ids=s["ids"])
    if kind == "learned":
        t = bh.build_tree(s["pos"], s["mass"], s["ws"])
        theta = s["net"].infer(t.features(), alpha=case["alpha"])
        acc, pot = t.forces(eps=case["eps"], acc=s["acc"], pot=s["pot"], theta_group=theta)
        return dict(theta=theta, acc=acc, pot=pot)
    if kind == "train":
        net = s["net"]
        g = net.grad(s["X"], s["target"], s["rows"])
        net.adam(g, 3e-3)
        return dict(grad=g, params=net.params, m=net.m, v=net.v)
    acc, pot = bh.direct(s["pos"], s["mass"], case["eps"], s["targets"])
    return dict(acc=acc, pot=pot)


# ---------------------------------------------------------------- its work
def _per_target(n, theta):
    """Interactions of one target, as measured from Plummer 1M at theta 0.3 to 0.75 (within 10%)
    and clumpy 4M at 0.35 (within 20%)."""
    return min(n - 1.0, 21.0 * theta ** -2.3 * math.log2(max(n, 2)))


def work(case):
    """Inputs read and outputs written once; 22 operations an interaction (offset 3, square 5,
    softening 1, inverse root 1, factors 3, sums 8, test 1), 60 a quadrupole one."""
    kind = case["kind"]
    if kind == "train":
        b = case["batch"]
        return dict(bytes=b * 40.0 + 4801 * 4 * 8, flops=6.0 * b * (8 * 64 + 64 * 64 + 64))
    el = 8.0 if case["prec"] == "fp64" else 4.0
    if kind == "direct":
        return dict(bytes=case["n"] * 4 * el + case["targets"] * (8 + 4 * el), flops=21.0 * case["n"] * case["targets"])
    if kind == "forest":
        sizes = _sizes(case)
        return dict(bytes=float(sizes.sum()) * 8 * el,
                    flops=22.0 * sum(int(k) * _per_target(int(k), case["theta"]) for k in sizes))
    n = case["n"]
    if kind == "neighbours":
        # pairs: those of the field at this radius (55 a particle at clumpy 4M, r = 2e-3)
        base = 2e-3 if case["dist"] == "clumpy" else 0.03 if case["dist"] == "plummer" else 0.013
        pairs = n * 55.0 * (n / 4194304.0) * (case["radius"] / base) ** 3
        return dict(bytes=n * (4 * el + 12 + el + 8 * case["maxlen"]), flops=20.0 * pairs)
    theta = case.get("theta", 0.4)
    per = 60.0 if case.get("order", 1) == 2 else 22.0
    state = 20.0 if kind == "leapfrog" else 8.0
    return dict(bytes=n * state * el, flops=per * n * _per_target(n, theta))


# ---------------------------------------------------------------- the same in 64 bits
def _morton(q):
    key = torch.zeros(q.shape[0], dtype=torch.int64, device=q.device)
    for b in range(21):
        for d in range(3):
            key |= ((q[:, d] >> b) & 1) << (3 * b + 2 - d)
    return key


def _levels(x, m, seg, K, order):
    """The oct-tree level by level, particles sorted by (cluster, Morton key): per level the cells'
    first particle, count, mass, centre of mass, side, offset of the centre of mass, children (and
    second moments).  Returns the sort and the levels."""
    lo = torch.full((K, 3), math.inf, dtype=torch.float64, device=x.device)
    hi = torch.full((K, 3), -math.inf, dtype=torch.float64, device=x.device)
    i3 = seg[:, None].expand(-1, 3)
    lo.scatter_reduce_(0, i3, x, "amin")
    hi.scatter_reduce_(0, i3, x, "amax")
    L = (hi - lo).amax(1)
    L = torch.where(L > 0, L, torch.ones_like(L))
    q = ((x - lo[seg]) * (2.0 ** 21 / L)[seg][:, None]).floor().clamp(0, 2 ** 21 - 1).to(torch.int64)
    key = _morton(q)
    at = torch.argsort(key, stable=True)
    at = at[torch.argsort(seg[at], stable=True)]
    x, m, seg, q, key = x[at], m[at], seg[at], q[at], key[at]
    n = x.shape[0]
    levels = []
    for lv in range(22):
        pre = key >> (63 - 3 * lv)
        new = torch.ones(n, dtype=torch.bool, device=x.device)
        new[1:] = (pre[1:] != pre[:-1]) | (seg[1:] != seg[:-1])
        cell = torch.cumsum(new, 0) - 1
        first = new.nonzero()[:, 0]
        nc = first.shape[0]
        count = torch.bincount(cell, minlength=nc)
        M = torch.zeros(nc, dtype=torch.float64, device=x.device).index_add_(0, cell, m)
        mx = torch.zeros((nc, 3), dtype=torch.float64, device=x.device).index_add_(0, cell, m[:, None] * x)
        side = L[seg[first]] * 2.0 ** -lv
        ctr = lo[seg[first]] + ((q[first] >> (21 - lv)).double() + 0.5) * side[:, None]
        com = torch.where((M != 0)[:, None], mx / M[:, None], ctr)
        com = torch.where((count == 1)[:, None], x[first], com)
        d = dict(first=first, count=count, M=M, com=com, side=side, s=(ctr - com).norm(dim=1))
        if order == 2:
            y = x - com[cell]
            B = torch.stack([y[:, a] * y[:, b] for a, b in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))], 1)
            d["B"] = torch.zeros((nc, 6), dtype=torch.float64, device=x.device).index_add_(0, cell, m[:, None] * B)
        if levels:
            kids = torch.bincount(parent[first], minlength=levels[-1]["first"].shape[0])  # noqa: F821
            levels[-1].update(kids=kids, kid0=torch.cumsum(kids, 0) - kids)
        levels.append(d)
        parent = cell
        if int(count.max()) == 1:
            break
    return at, x, m, seg, levels


def _expand(t, c, first, count):
    """Each pair (t, c) once for every one of the `count` members from `first` on."""
    k = count[c]
    rep = torch.repeat_interleave(torch.arange(t.shape[0], device=t.device), k)
    off = torch.arange(rep.shape[0], device=t.device) - (torch.cumsum(k, 0) - k)[rep]
    return t[rep], first[c][rep] + off


def _term(d, r2, M, B=None):
    ri = torch.where(r2 > 0, r2, torch.ones_like(r2)) ** -0.5
    ri = torch.where(r2 > 0, ri, torch.zeros_like(r2))
    ri3 = ri * ri * ri
    a = (M * ri3)[:, None] * d
    p = -M * ri
    if B is not None:
        x, y, z = d.unbind(1)
        bd = torch.stack([B[:, 0] * x + B[:, 1] * y + B[:, 2] * z, B[:, 1] * x + B[:, 3] * y + B[:, 4] * z,
                          B[:, 2] * x + B[:, 4] * y + B[:, 5] * z], 1)
        dbd, T, ri5 = (d * bd).sum(1), B[:, 0] + B[:, 3] + B[:, 5], ri3 * ri * ri
        a = a - (3.0 * ri5)[:, None] * bd + (7.5 * dbd * ri5 * ri * ri - 1.5 * T * ri5)[:, None] * d
        p = p + 0.5 * (T * ri3 - 3.0 * dbd * ri5)
    return torch.cat([a, p[:, None]], 1)


def _tree_forces(pos, mass, theta, eps, order=1, offsets=None, chunk=16384):
    """Accelerations and potentials of the method in 64 bits: the opening test of Eq. (2) and the
    terms of Eq. (1), breadth first over (target, cell) pairs."""
    x, m = pos.double(), mass.double()
    n = x.shape[0]
    seg = torch.zeros(n, dtype=torch.int64, device=x.device)
    K = 1
    if offsets is not None:
        K = offsets.shape[0] - 1
        seg = torch.repeat_interleave(torch.arange(K, device=x.device), offsets[1:] - offsets[:-1])
    at, x, m, seg, levels = _levels(x, m, seg, K, order)
    root = torch.searchsorted(seg[levels[0]["first"]], seg)
    out = torch.zeros((n, 4), dtype=torch.float64, device=x.device)
    e2 = eps * eps
    for b in range(0, n, chunk):
        t = torch.arange(b, min(n, b + chunk), device=x.device)
        c = root[t]
        for lv, d in enumerate(levels):
            off = d["com"][c] - x[t]
            d2 = (off * off).sum(1)
            one = d["count"][c] == 1
            own = (t >= d["first"][c]) & (t < d["first"][c] + d["count"][c])
            use = ~own & (one | (d2 > (d["side"][c] / theta + d["s"][c]) ** 2))
            u = use.nonzero()[:, 0]
            out.index_add_(0, t[u], _term(off[u], d2[u] + e2, d["M"][c[u]], d["B"][c[u]] if order == 2 else None))
            o = (~use & ~one).nonzero()[:, 0]
            if o.numel() == 0:
                break
            if lv + 1 < len(levels):
                t, c = _expand(t[o], c[o], d["kid0"], d["kids"])
            else:
                # particles that share a cell of the finest grid are taken one by one
                t, j = _expand(t[o], c[o], d["first"], d["count"])
                t, j = t[t != j], j[t != j]
                off = x[j] - x[t]
                out.index_add_(0, t, _term(off, (off * off).sum(1) + e2, m[j]))
    back = torch.empty_like(out)
    back[at] = out
    return back[:, :3].contiguous(), back[:, 3].contiguous()


def _mlp_step(s, lr=3e-3):
    """One training step of the network in 64 bits."""
    P = torch.as_tensor(s["params"], device="cuda").double().requires_grad_(True)
    X = s["X"][s["rows"].long()].double()
    mean, std = s["X"].mean(0).double(), s["X"].std(0).double()
    W1, b1, W2, b2, w3, b3 = (P[a:b] for a, b in ((0, 512), (512, 576), (576, 4672), (4672, 4736), (4736, 4800),
                                                   (4800, 4801)))
    F = torch.nn.functional
    h = F.gelu((X - mean) / std @ W1.view(64, 8).T + b1, approximate="tanh")
    h = F.gelu(h @ W2.view(64, 64).T + b2, approximate="tanh")
    loss = ((torch.sigmoid(h @ w3 + b3) - s["target"][s["rows"].long()].double()) ** 2).mean()
    (g,) = torch.autograd.grad(loss, P)
    P = P.detach()
    m, v = 0.1 * g, 0.001 * g * g
    return dict(grad=torch.cat([g, loss.detach()[None]]), params=P - lr * g / (g.abs() + 1e-8), m=m, v=v)


def exact(case, seed):
    """What run() returns, in 64 bits by plain torch; None where that takes too long, and for the
    learned parameter (rounded to bfloat16 on its way into the walk)."""
    kind = case["kind"]
    if kind == "learned":
        return None
    if kind == "train":
        return _mlp_step(_inputs(case, seed))
    s = _inputs(case, seed)
    n = s["pos"].shape[0]
    if kind == "direct":
        x, m = s["pos"].double(), s["mass"].double()
        out = []
        step = max(1, 100_000_000 // n)
        for b in range(0, case["targets"], step):
            ti = s["targets"][b:b + step]
            d = x[None, :, :] - x[ti][:, None, :]
            r2 = (d * d).sum(2) + case["eps"] ** 2
            w = r2 ** -0.5
            w[torch.arange(ti.shape[0], device="cuda"), ti] = 0.0
            w[r2 == 0] = 0.0
            out.append(torch.cat([((m * w ** 3)[:, :, None] * d).sum(1), -(m * w).sum(1, keepdim=True)], 1))
        out = torch.cat(out)
        return dict(acc=out[:, :3].contiguous(), pot=out[:, 3].contiguous())
    if kind == "neighbours":
        if n > 150_000:
            return None
        x, m = s["pos"].double(), s["mass"].double()
        h = 0.5 * case["radius"]
        rho = torch.empty(n, dtype=torch.float64, device="cuda")
        step = max(1, 100_000_000 // n)
        for b in range(0, n, step):
            d2 = sum((x[None, :, a] - x[b:b + step, None, a]) ** 2 for a in range(3))
            q = d2.sqrt() / h
            w = torch.where(q < 1, 1 - 1.5 * q * q + 0.75 * q ** 3, 0.25 * (2 - q).clamp_min(0.0) ** 3)
            rho[b:b + step] = (m * w).sum(1) / (math.pi * h ** 3)
        return dict(count=None, hash=None, lists=None, rho=rho)
    if n * _per_target(n, case["theta"]) > 3e9:
        return None
    args = (case["theta"], case["eps"])
    if kind == "leapfrog":
        # the state is held in its own precision: every update rounds to it
        dt, half = s["pos"].dtype, 0.5 * case["dt"]
        if case["reorder"]:
            return None
        a, _ = _tree_forces(s["pos"], s["mass"], *args, order=case["order"])
        v = (s["vel"].double() + half * a).to(dt)
        pos = (s["pos"].double() + case["dt"] * v.double()).to(dt)
        a, p = _tree_forces(pos, s["mass"], *args, order=case["order"])
        return dict(pos=pos, vel=(v.double() + half * a), acc=a, pot=p, ids=None)
    return _tree_forces(s["pos"], s["mass"], *args, order=case.get("order", 1), offsets=s.get("offsets"))

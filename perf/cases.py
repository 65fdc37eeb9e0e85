"""The work that a user of this library has it do, as cases to be timed.

A case is a dict of plain values.  Its "kind" says which public entry points one pass calls:

* update   one analysis step of a 1-D Gaussian-model filter: infoesrf_perturbation_update (and
           infoesrf_mean_update where "mean" is true), through the convenience functions
           ("call": "functions", they return host statistics) or a preallocated runner that only
           enqueues ("call": "runner");
* learned  the same update from the learned warm start;
* batch    many independent uneven filters in one infoesrf_update_batched call, means included;
* cycle    one assimilation cycle of the multi-layer Lorenz-96 model (forecast, observation, mean
           and perturbation update, relaxation to prior spread);
* channels one analysis with weighted-channel observations and a fixed iteration budget;
* cov      the localized covariance applied to a block of state vectors;
* train    the gradients of a warm-start training batch.

Inputs are drawn from the seed with torch alone; exact() repeats a pass in 64-bit torch with
direct solves.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2503_00253_amd import infoesrf as ie
from paper_2503_00253_amd.cycle import CycleRunner

F64 = torch.float64


def _update(name, n, N, Q, ell, length, c, *, precision="fp64", domain="lattice", ritz=4, over=4, mean=False,
            call="runner", stride=4, kind="update"):
    d = dict(kind=kind, n=n, N=N, Q=Q, ell=ell, length=length, c=c, stride=stride, precision=precision,
             domain=domain, ritz=ritz, over=over, mean=mean, call=call)
    return dict(d, name=name) if name else d


def listed():
    return [
        # the smallest analysis, with the library's default options: a user's first call, and a
        # small filter cycled on its own, where launches and the host's share count
        _update("small-n256-defaults", 256, 16, 8, 100.0, 10.0, 20.0, domain="state", ritz=10, over=10, mean=True,
                call="functions"),
        # the workload of the benchmark: one large ensemble on a declared lattice, FP32 inner applies
        _update("n4096-mixed", 4096, 40, 16, 1000.0, 40.0, 80.0, precision="fp32"),
        # the same ensemble in FP64 with the default preconditioner, mean and perturbations
        _update("n4096-fp64-mean", 4096, 40, 16, 1000.0, 40.0, 80.0, ritz=10, over=10, mean=True, call="functions"),
        # no lattice declared: the general observation operator in the state space
        _update("n4096-state", 4096, 40, 16, 1000.0, 40.0, 80.0, domain="state", ritz=10, over=10, mean=True,
                call="functions"),
        # an odd size: a bounded (not periodic) domain whose lattice is ragged
        _update("n3001-ragged", 3001, 24, 11, 1000.0, 30.0, 50.0, precision="fp32", ritz=8, over=6, stride=3),
        # the same update from a learned start
        _update("n4096-learned", 4096, 40, 16, 1000.0, 40.0, 80.0, precision="fp32", kind="learned"),
        # uneven independent filters in one call, the largest work here
        dict(name="batch32-mixed", kind="batch", count=32, lo=128, hi=2048, sizes=4, precision="fp32", ritz=4,
             over=4),
        # a few small filters in one call, FP64 and the default preconditioner
        dict(name="batch8-small-fp64", kind="batch", count=8, lo=64, hi=512, sizes=11, precision="fp64", ritz=10,
             over=10),
        # one cycle of the 8 x 480 atmosphere: point observations of every third site
        dict(name="lorenz-8x480", kind="cycle", nz=8, nx=480, N=20, stride=3, c_h=7.5, c_v=1.0, Q=12, ell=1000.0,
             gamma=0.1, ritz=4, over=4),
        # a large state seen through 100 weighted channels, two PCG iterations
        dict(name="channels-n2000", kind="channels", n=2000, N=20, d=100, Q=8, ell=1000.0, length=12.0, ritz=8,
             over=10, iters=2),
        # the covariance alone, on a block of state vectors
        dict(name="cov-n4096-B640", kind="cov", n=4096, N=40, B=640, length=40.0, c=80.0),
        # one training batch of the warm-start network
        dict(name="train-B8", kind="train", B=8, Q=16, m=1024, hidden=64, kernel=9),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["update", "update", "update", "state", "learned", "batch", "batch", "cycle", "channels",
                       "cov", "train"])
    precision = rng.choice(["fp64", "fp32"])
    ritz, over = rng.choice([(4, 4), (4, 4), (10, 10), (8, 6), (0, 0)])
    if kind in ("update", "state", "learned"):
        stride = rng.choice([2, 3, 4, 4, 5])
        n = _log(rng, 240, 4096)
        m = -(-n // stride)
        if m > 1400:
            stride = 4
        if rng.random() < 0.6:
            n -= n % stride                      # periodic axes take whole strides
        c = rng.uniform(6.0, 80.0)
        c = min(c, n / 8.0)
        if kind == "state":
            n = min(n, 2600)
        return _update(None, n, rng.randint(12, 48), rng.randint(6, 18), rng.choice([100.0, 1000.0]),
                       round(rng.uniform(0.3, 0.6) * c, 2), round(c, 2), precision="fp32" if kind == "learned" else
                       "fp64" if kind == "state" else precision, domain="state" if kind == "state" else "lattice",
                       ritz=ritz, over=over, mean=rng.random() < 0.5, call=rng.choice(["runner", "functions"]),
                       stride=stride, kind="learned" if kind == "learned" else "update")
    if kind == "batch":
        lo = _log(rng, 48, 400)
        return dict(kind="batch", count=rng.randint(3, 20), lo=lo, hi=min(2048, lo * rng.randint(2, 8)),
                    sizes=rng.randint(0, 1 << 20), precision=precision, ritz=ritz, over=over)
    if kind == "cycle":
        return dict(kind="cycle", nz=rng.randint(2, 10), nx=3 * rng.randint(20, 120), N=rng.randint(10, 40), stride=3,
                    c_h=round(rng.uniform(4.0, 9.0), 2), c_v=1.0, Q=rng.randint(6, 14), ell=1000.0, gamma=0.1,
                    ritz=ritz, over=over)
    if kind == "channels":
        n = 20 * rng.randint(40, 120)
        return dict(kind="channels", n=n, N=rng.randint(12, 40), d=n // 20, Q=rng.randint(4, 10), ell=1000.0,
                    length=12.0, ritz=rng.choice([4, 8, 12, 20]), over=10, iters=rng.choice([2, 10]))
    if kind == "cov":
        c = rng.uniform(10.0, 80.0)
        n = _log(rng, 1000, 12000)
        return dict(kind="cov", n=n, N=rng.randint(10, 48), B=_log(rng, 1, 640), length=round(c / 2, 2),
                    c=round(min(c, n / 8.0), 2))
    return dict(kind="train", B=rng.randint(2, 12), Q=rng.randint(4, 20), m=_log(rng, 200, 2000), hidden=64, kernel=9)


# ---- inputs ---------------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator().manual_seed(int(seed) * 2654435761 % (1 << 62))


def _gc(r):
    """Gaspari-Cohn fifth-order correlation (torch, 64 bits)."""
    r = r.abs()
    a = -0.25 * r**5 + 0.5 * r**4 + 0.625 * r**3 - (5.0 / 3.0) * r**2 + 1.0
    s = r.clamp(min=1e-300)
    b = r**5 / 12.0 - 0.5 * r**4 + 0.625 * r**3 + (5.0 / 3.0) * r**2 - 5.0 * r + 4.0 - 2.0 / (3.0 * s)
    return torch.where(r <= 1.0, a, torch.where(r < 2.0, b, torch.zeros_like(r)))


def _members(n, k, length, g, pad=0):
    """k fields of a stationary Gaussian prior on a circle of n + pad points, the first n of them (k, n)."""
    full = n + pad
    d = torch.arange(full, dtype=F64)
    d = torch.minimum(d, full - d)
    lam = torch.fft.fft(torch.exp(-(d**2) / (2.0 * length**2))).real.clamp(min=0.0).sqrt()
    xi = torch.randn(k, full, dtype=F64, generator=g)
    return torch.fft.ifft(torch.fft.fft(xi) * lam).real[:, :n].contiguous()


def _line(n, N, stride, length, c, g):
    """A 1-D filter: members, point observations of every stride-th point, localization."""
    periodic = n % stride == 0
    x = _members(n, N + 1, length, g, 0 if periodic else int(8 * length))
    idx = torch.arange(0, n, stride)
    m = idx.numel()
    y = x[N, idx] + 0.5 * torch.randn(m, dtype=F64, generator=g)
    bx = int(math.ceil(2.0 * c)) - 1
    if periodic:
        bx = min(bx, (n - 1) // 2)
    table = _gc(torch.arange(-bx, bx + 1, dtype=F64) / c)
    return SimpleNamespace(n=n, N=N, m=m, x=x[:N], y=y, idx=idx, nz=1, nx=n, px=int(periodic), bz=0, bx=bx,
                           table=table.reshape(1, -1), r=0.25, lattice=(0, 1, 1, 0, stride, m))


def _problem(p):
    m = p.m
    return ie.Problem(p.x.t().cuda(), np.arange(m + 1), p.idx.numpy(), np.ones(m), np.full(m, p.r), nz=p.nz, nx=p.nx,
                      periodic_z=0, periodic_x=p.px, bz=p.bz, bx=p.bx, table=p.table.numpy())


def _opts(case, p, **kw):
    o = dict(precision=ie.MIXED_FP32 if case.get("precision") == "fp32" else ie.FP64, n_ritz=case["ritz"],
             oversample=case["over"], **kw)
    if case.get("domain", "lattice") == "lattice" and p is not None:
        o.update(apply_domain=ie.DOMAIN_OBS_LATTICE, lattice=p.lattice)
    return ie.default_opts(**o)


def _l96_step(s, dt, F, gamma):
    def f(v):
        t = torch.roll(v, 1, 2) * (torch.roll(v, -1, 2) - torch.roll(v, 2, 2)) - v + F
        if v.shape[1] > 1:
            t[:, 1:] += gamma * (v[:, :-1] - v[:, 1:])
            t[:, :-1] += gamma * (v[:, 1:] - v[:, :-1])
        return t
    k1 = f(s)
    k2 = f(s + 0.5 * dt * k1)
    k3 = f(s + 0.5 * dt * k2)
    k4 = f(s + dt * k3)
    return s + (dt / 6.0) * (k1 + 2.0 * k2 + 2.0 * k3 + k4)


def _atmosphere(case, g):
    """Members and truth after a spin-up, the point observations, noise and localization."""
    nz, nx, N, st = case["nz"], case["nx"], case["N"], case["stride"]
    s = 8.0 + torch.randn(1, nz, nx, dtype=F64, generator=g)
    pert = torch.randn(N, nz, nx, dtype=F64, generator=g)
    idx = (torch.arange(nz)[:, None] * nx + torch.arange(0, nx, st)[None, :]).reshape(-1)
    noise = torch.randn(idx.numel(), dtype=F64, generator=g)
    s = s.cuda()
    for _ in range(300):
        s = _l96_step(s, 0.01, 8.0, case["gamma"])
    s = torch.cat([s + pert.cuda(), s]).cpu().reshape(N + 1, nz * nx)
    bz, bx = int(math.ceil(2 * case["c_v"])) - 1, int(math.ceil(2 * case["c_h"])) - 1
    dz, dx = torch.arange(-bz, bz + 1, dtype=F64)[:, None], torch.arange(-bx, bx + 1, dtype=F64)[None, :]
    table = _gc(torch.sqrt((dx / case["c_h"]) ** 2 + (dz / case["c_v"]) ** 2))
    return SimpleNamespace(n=nz * nx, N=N, m=idx.numel(), s=s, idx=idx, noise=noise, nz=nz, nx=nx, px=1, bz=bz, bx=bx,
                           table=table, r=1.0, lattice=(0, 1, nz, 0, st, nx // st))


def _channels(case, g):
    """A Gaussian prior on a circle seen through d Gaussian-weighted channels."""
    n, N, d = case["n"], case["N"], case["d"]
    x = _members(n, N + 1, 10.0, g)
    j = np.arange(n)
    ptr, hi, hw = [0], [], []
    for i in range(1, d + 1):
        w = np.exp(-((n / np.pi) * np.sin(np.pi * np.abs(j - (n // d) * i) / n)) ** 2 / 200.0)
        keep = np.nonzero(w > 1e-17)[0]
        hi.append(keep)
        hw.append(w[keep])
        ptr.append(ptr[-1] + keep.size)
    H = torch.zeros(d, n, dtype=F64)
    for k in range(d):
        H[k, torch.from_numpy(hi[k])] = torch.from_numpy(hw[k])
    r = 36.28
    y = H @ x[N] + math.sqrt(r) * torch.randn(d, dtype=F64, generator=g)
    dx = np.arange(-(n // 2) + 1, n // 2)
    t = np.exp(-((n / np.pi) * np.sin(np.pi * np.abs(dx) / n)) ** 2 / (2 * case["length"] ** 2))
    bx = int(np.max(np.abs(dx[t > 1e-17])))
    dxs = np.arange(-bx, bx + 1)
    table = np.exp(-((n / np.pi) * np.sin(np.pi * np.abs(dxs) / n)) ** 2 / (2 * case["length"] ** 2))
    P = ie.Problem(x[:N].t().cuda(), np.array(ptr), np.concatenate(hi), np.concatenate(hw), np.full(d, r), nz=1, nx=n,
                   periodic_x=1, bx=bx, table=table.reshape(1, -1))
    return P, y


def _specs(case):
    """The uneven sizes of a batch: (n, N, Q) of each instance."""
    r = np.random.RandomState(case["sizes"])
    return [(4 * int(r.randint(case["lo"], case["hi"] + 1)), int(r.choice([16, 32, 48, 64])), int(r.randint(8, 25)))
            for _ in range(case["count"])]


def _batch(case, seed):
    g = _gen(seed)
    return [(_line(n, N, 4, min(40.0, n / 16.0), min(80.0, n / 8.0), g), Q) for n, N, Q in _specs(case)]


def _net_params(case, g):
    """Seeded weights of the trunk in the library's parameter layout, one (weight, bias) pair a layer."""
    H, K, out = case.get("hidden", 64), case.get("kernel", 9), []
    for co, ci in ((H, 1), (H, H), (H, H), (4, H)):
        out.append(torch.randn(co, ci, K, generator=g) * (1.0 / math.sqrt(ci * K)))
        out.append(0.05 * torch.randn(co, generator=g))
    return out


def _net(case, g):
    net = ie.Net.create(case.get("hidden", 64), case.get("kernel", 9), 0)
    net.set_params(torch.cat([t.reshape(-1) for t in _net_params(case, g)]).numpy())
    return net


def _train_batch(case, g):
    B, Q, m = case["B"], case["Q"], case["m"]
    x = _members(m, B, 10.0, g)
    X = (x / x.norm(dim=1, keepdim=True) * math.sqrt(m)).float()
    cq = (1.0 / (1.0 + torch.logspace(-3, 2, Q, dtype=F64))).float()
    T = cq[None, :, None] * X[:, None, :] * 0.5 + 0.1 * torch.randn(B, Q, m, generator=g)
    return X, cq, T


def prepare(case, seed):
    kind = case["kind"]
    g = _gen(seed)
    if kind in ("update", "learned"):
        p = _line(case["n"], case["N"], case["stride"], case["length"], case["c"], g)
        P = _problem(p)
        kw = {}
        s = SimpleNamespace(P=P, y=p.y.cuda(), nodes=ie.quadrature_elliptic(case["Q"], case["ell"]))
        if kind == "learned":
            s.net = _net(case, _gen(seed + 1))
            kw = dict(warm_start=ie.START_LEARNED, net=s.net)
        if case["call"] == "functions":
            s.opts = _opts(case, p, **kw)
        else:
            # a program that enqueues analysis after analysis and waits for none of them
            s.opts = _opts(case, p, host_sync=0, **kw)
            if case["mean"]:
                s.runner = ie.BatchedRunner([P], [s.nodes], s.opts, ys=[s.y],
                                            lattices=[p.lattice] if case["domain"] == "lattice" else None) \
                    if kind == "update" else ie.PerturbationRunner(P, *s.nodes, s.opts)
            else:
                s.runner = ie.PerturbationRunner(P, *s.nodes, s.opts)
        return s
    if kind == "batch":
        ps = _batch(case, seed)
        probs = [_problem(p) for p, _ in ps]
        opts = _opts(dict(case, domain="state"), None, host_sync=0, apply_domain=ie.DOMAIN_OBS_LATTICE)
        run_ = ie.BatchedRunner(probs, [ie.quadrature_elliptic(Q, 1000.0) for _, Q in ps], opts,
                                ys=[p.y.cuda() for p, _ in ps], lattices=[p.lattice for p, _ in ps])
        return SimpleNamespace(runner=run_)
    if kind == "cycle":
        p = _atmosphere(case, g)
        prob = SimpleNamespace(n=p.n, N=p.N, m=p.m, X=p.s[:p.N].t().numpy(), truth=p.s[p.N].numpy(),
                               h_ptr=np.arange(p.m + 1), h_idx=p.idx.numpy(), h_w=np.ones(p.m), r_var=np.full(p.m, p.r),
                               nz=p.nz, nx=p.nx, periodic_z=0, periodic_x=1, bz=p.bz, bx=p.bx, table=p.table.numpy(),
                               Q=case["Q"], ell=case["ell"],
                               meta=dict(gamma=case["gamma"], dt=0.01, steps_per_cycle=5, forcing=8.0))
        c = CycleRunner(prob, opts=_opts(case, p, host_sync=0), noise=p.noise.reshape(1, -1).numpy())
        c.load_noise(0)
        return SimpleNamespace(c=c, first=c.state.clone())
    if kind == "channels":
        P, y = _channels(case, g)
        return SimpleNamespace(P=P, y=y.cuda(), nodes=ie.quadrature_elliptic(case["Q"], case["ell"]),
                               opts=_opts(dict(case, domain="state"), None, fixed_iters=case["iters"]))
    if kind == "cov":
        p = _line(case["n"], case["N"], 4 if case["n"] % 4 == 0 else 1, case["length"], case["c"], g)
        if p.m > 4096:   # the observations do not matter here
            p.m, p.idx = 16, p.idx[:16]
        V = torch.randn(case["B"], case["n"], dtype=F64, generator=g)
        return SimpleNamespace(P=_problem(p), V=V.cuda().t(), opts=ie.default_opts())
    X, cq, T = _train_batch(case, g)
    return SimpleNamespace(net=_net(case, _gen(seed + 1)), X=X.cuda(), cq=cq.cuda(), T=T.cuda())


def run(s):
    if hasattr(s, "c"):
        # the cycle that starts from the first forecast ensemble
        s.c.state.copy_(s.first)
        s.c.cycle_body()
        return s.c.state[:s.c.N], s.c.mean_a, s.c.Xa
    if hasattr(s, "X"):
        return s.net.gradients(s.X, s.cq, s.T)
    if hasattr(s, "V"):
        return ie.cov_apply(s.P, s.V, s.opts)
    if hasattr(s, "runner"):
        s.runner.run()
        if isinstance(s.runner, ie.BatchedRunner):
            return s.runner.results()
        return s.runner.result()
    xa, _ = ie.perturbation_update(s.P, *s.nodes, s.opts)
    mean, _ = ie.mean_update(s.P, s.y, s.opts)
    return xa, mean


# ---- the work of a pass ---------------------------------------------------------------------

# PCG iterations a system of these priors needs to the default residual (means measured on the
# listed cases): dense stretches of observations take more than sparse ones
_ITERS = {"update": 25, "learned": 25, "batch": 27, "cycle": 6}


def _solve_work(n, N, m, nnz_row, ritz, systems, iters):
    by = 8.0 * (2 * n * N + n + 3 * m)
    return by, systems * iters * (2.0 * m * nnz_row + m * (12.0 + 8.0 * ritz)) + 2.0 * N * m * nnz_row


def work(case):
    kind = case["kind"]
    if kind in ("update", "learned"):
        m = -(-case["n"] // case["stride"])
        by, fl = _solve_work(case["n"], case["N"], m, 2 * (2 * case["c"] // case["stride"]) + 1, case["ritz"],
                             case["Q"] * case["N"], _ITERS[kind])
    elif kind == "batch":
        by = fl = 0.0
        for n, N, Q in _specs(case):
            b, f = _solve_work(n, N, n // 4, 2 * (2 * min(80.0, n / 8.0) // 4) + 1, case["ritz"], Q * N, _ITERS[kind])
            by, fl = by + b, fl + f
    elif kind == "cycle":
        n, N = case["nz"] * case["nx"], case["N"]
        m = n // case["stride"]
        by, fl = _solve_work(n, N, m, 3 * (2 * (2 * case["c_h"] // case["stride"]) + 1), case["ritz"], case["Q"] * N,
                             _ITERS[kind])
        fl += 5 * 4 * 12.0 * n * (N + 1)
    elif kind == "channels":
        by, fl = _solve_work(case["n"], case["N"], case["d"], case["d"], case["ritz"], case["Q"] * case["N"],
                             case["iters"])
        by += case["d"] * 178 * 12.0
    elif kind == "cov":
        n, B = case["n"], case["B"]
        w = 2 * int(2 * case["c"]) + 1
        by, fl = 8.0 * (2 * n * B + n * case["N"]), 2.0 * n * w * (B + case["N"])
    else:
        B, Q, m, H, K = case["B"], case["Q"], case["m"], case["hidden"], case["kernel"]
        by, fl = 4.0 * (B * Q * m + B * m) + 8.0 * (2 * H * H * K), 3 * 2.0 * B * m * K * (2 * H * H + 5 * H)
    return {"bytes": by, "flops": fl}


# ---- 64-bit results -------------------------------------------------------------------------


def _nodes64(Q, ell):
    """The elliptic rule by the arithmetic-geometric mean and descending Landen steps."""
    kc = math.sqrt(1.0 / (1.0 + ell))
    a, b, c = [1.0], [kc], [math.sqrt(ell / (1.0 + ell))]
    while abs(c[-1]) > 1e-17 and len(a) < 40:
        a.append(0.5 * (a[-1] + b[-1]))
        c.append(0.5 * (a[-2] - b[-1]))
        b.append(math.sqrt(a[-2] * b[-1]))
    K = math.pi / (2.0 * a[-1])
    s, p = [], []
    for q in range(1, Q + 1):
        phi = 2.0 ** (len(a) - 1) * a[-1] * (q - 0.5) * K / Q
        for i in range(len(a) - 1, 0, -1):
            phi = 0.5 * (phi + math.asin(max(-1.0, min(1.0, c[i] / a[i] * math.sin(phi)))))
        sn, cn = math.sin(phi), math.cos(phi)
        dn = math.sqrt(1.0 - ell / (1.0 + ell) * sn * sn)
        s.append((sn / cn) ** 2)
        p.append((2.0 * K / (math.pi * Q)) * dn / cn**2 / (1.0 + s[-1]))
    return s, p


def _loc(p, a, b):
    """L between state points a and b (index vectors)."""
    za, xa, zb, xb = a // p.nx, a % p.nx, b // p.nx, b % p.nx
    dz, dx = zb[None, :] - za[:, None], xb[None, :] - xa[:, None]
    if p.px:
        dx = (dx + p.nx // 2) % p.nx - p.nx // 2
        dx = torch.where(dx.abs() > p.bx, torch.where((dx - p.nx).abs() <= p.bx, dx - p.nx, dx), dx)
    ok = (dz.abs() <= p.bz) & (dx.abs() <= p.bx)
    t = p.table.reshape(-1)[((dz.clamp(-p.bz, p.bz) + p.bz) * (2 * p.bx + 1) + dx.clamp(-p.bx, p.bx) + p.bx)]
    return torch.where(ok, t, torch.zeros_like(t))


def _analysis64(p, x, y, Q, ell):
    """(analysis deviations (n, N), analysis mean) with direct solves; x: members (N, n)."""
    N, n = x.shape
    mu = x.mean(0)
    Z = (x - mu) / math.sqrt(N - 1)
    W = Z[:, p.idx]
    r = math.sqrt(p.r)
    S = _loc(p, p.idx, p.idx) * (W.t() @ W) / p.r
    PH = _loc(p, torch.arange(n), p.idx) * (Z.t() @ W) / r
    eye = torch.eye(p.m, dtype=F64)
    ub = torch.zeros(p.m, N, dtype=F64)
    for s, w in zip(*_nodes64(Q, ell)):
        ub += w * torch.cholesky_solve(W.t() / r, torch.linalg.cholesky(S + (1.0 + s) * eye))
    u0 = torch.cholesky_solve(((y - mu[p.idx]) / r).reshape(-1, 1), torch.linalg.cholesky(S + eye))
    return math.sqrt(N - 1) * (Z.t() - PH @ ub), mu + (PH @ u0)[:, 0]


def exact(case, seed):
    kind = case["kind"]
    g = _gen(seed)
    if kind in ("update", "learned"):
        p = _line(case["n"], case["N"], case["stride"], case["length"], case["c"], g)
        xa, mean = _analysis64(p, p.x, p.y, case["Q"], case["ell"])
        if case["call"] == "functions":
            return xa, mean
        return ([xa], [mean]) if case["mean"] and kind == "update" else xa
    if kind == "batch":
        got = [_analysis64(p, p.x, p.y, Q, 1000.0) for p, Q in _batch(case, seed)]
        return [a for a, _ in got], [b for _, b in got]
    if kind == "cycle":
        p = _atmosphere(case, g)
        s = p.s.reshape(p.N + 1, p.nz, p.nx)
        for _ in range(5):
            s = _l96_step(s, 0.01, 8.0, case["gamma"])
        s = s.reshape(p.N + 1, p.n)
        xa, mean = _analysis64(p, s[:p.N], s[p.N, p.idx] + p.noise, case["Q"], case["ell"])
        sf, sa = s[:p.N].std(0), xa.t().std(0)
        return mean + (1.0 + 0.01 * (sf - sa) / sa) * xa.t(), mean, xa.t()
    if kind == "channels":
        return None     # a fixed iteration budget with a random sketch: no value of its own
    if kind == "cov":
        p = _line(case["n"], case["N"], 4 if case["n"] % 4 == 0 else 1, case["length"], case["c"], g)
        V = torch.randn(case["B"], case["n"], dtype=F64, generator=g)
        Z = (p.x - p.x.mean(0)) / math.sqrt(p.N - 1)
        out = torch.zeros_like(V)
        for d in range(-p.bx, p.bx + 1):
            out += float(p.table[0, d + p.bx]) * (Z * torch.roll(Z, -d, 1)).sum(0) * torch.roll(V, -d, 1)
        return out.t()
    X, cq, T = _train_batch(case, g)
    X, cq, T = X.double(), cq.double(), T.double()
    ps = [t.float().double().requires_grad_(True) for t in _net_params(case, _gen(seed + 1))]
    h, pad = X[:, None, :], case["kernel"] // 2
    for i in range(4):
        h = torch.nn.functional.conv1d(h, ps[2 * i], ps[2 * i + 1], padding=pad)
        if i < 3:
            h = torch.nn.functional.gelu(h)
    y = torch.einsum("qd,bdt->bqt", torch.stack([cq ** (d + 1) for d in range(4)], 1), h)
    loss = ((y - T).norm(dim=2) / T.norm(dim=2)).mean()
    grads = torch.autograd.grad(loss, ps)
    return torch.cat([t.reshape(-1) for t in grads]), loss.detach().reshape(1)

"""The work that this library's users have it do, as measurable cases.

A case names one pass through a public entry point:

* ``apply``          H psi of a block of vectors (``Plan.apply``)
* ``conv``           the potential block alone (``Plan.conv``)
* ``batch``          a coupling sweep's plans applied together (``Batch.apply``)
* ``eigenfunction``  a state on a physical observation grid
* ``learned_forward``, ``learned_grad``  the learned preconditioner, both ways
* ``eigs``           a whole solve for the lowest eigenvalues

The geometries, couplings and block sizes are those of ``workloads.py``,
``bench.py`` and the tests.  ``exact`` evaluates the definitions (true labels,
wrapped convolution, sums of exponentials) in plain float64 torch.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2404_04507_amd as iw
from paper_2404_04507_amd import workloads as W

DEV = "cuda:0"
HIDDEN = 256
DIMS = (8, HIDDEN, HIDDEN, HIDDEN, 2)


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def _case(name, kind, geom, K, L, **kw):
    c = {"name": name, "kind": kind, "geom": geom, "K": K, "L": L, "lam": 1.0, "precision": "fp64",
         "order": "grid", "nvec": 1, "pairs": 0, "tuned": False, "plans": 1, "nev": 0, "points": 0}
    c.update(kw)
    if not name:
        del c["name"]
    return c


def listed():
    return [
        # one vector on the 1D lattice lifted to 2D (512 points): the smallest
        # call a user makes; launch latency is all of it
        _case("apply_1d_512", "apply", "1d", 8, 16),
        # the ground-state block of the paper's 2D example at Table 6's
        # truncation (100 x 12 x 12), vectors kept in window order
        _case("apply_2d3_window", "apply", "2d3", 6, 50, order="window", nvec=3),
        # the benchmark's workload: 24 x 24 x 32 x 32, 16 vectors, float32
        # convolution, schedule picked by the autotuner
        _case("apply_2d4_fp32", "apply", "2d4", 12, 16, lam=0.5, precision="fp32", nvec=16, tuned=True),
        # an odd block on odd truncations of the same geometry, float64
        _case("apply_2d4_window", "apply", "2d4", 11, 13, lam=5.0, order="window", nvec=7),
        # the 3D workload: 16^6 points, larger than the last-level cache
        _case("apply_3d6_fp32", "apply", "3d6", 8, 8, lam=2.0, precision="fp32", nvec=8),
        # the paper's 3D example (40^3 x 8^3 points): the grid whose leading
        # block fits no workgroup; two complex columns hold its real block
        _case("apply_3d6_paper", "apply", "3d6p", 4, 20, nvec=2),
        # a potential with many modes off the axes (24 pairs and a constant)
        _case("apply_2d4_oblique", "apply", "2d4", 8, 10, lam=2.0, nvec=6, pairs=24),
        # one step of a coupling sweep: eight instances of different sizes
        _case("batch_sweep", "batch", "2d4", 0, 16, lam=5.0, nvec=8, plans=8),
        # the ground state on the paper's 2D observation grid (1001 x 1001)
        _case("eigenfunction_2d", "eigenfunction", "2d3", 6, 20, points=1001),
        # loss and gradient of the learned preconditioner on a training plan
        _case("learned_grad", "learned_grad", "2d4", 8, 8, lam=2.0, nvec=8),
        # Table 3's ground state (120 x 10 points): a solve bound by latency
        _case("eigs_1d_1200", "eigs", "1dp", 5, 60, nev=1),
        # the benchmark's solve: the 16 lowest pairs of the 589,824-point grid
        _case("eigs_2d4", "eigs", "2d4", 12, 16, lam=2.0, precision="fp32", nev=16),
    ]


def _smooth(e):
    """Whether an extent is a product of primes up to 13."""
    for p in (2, 3, 5, 7, 11, 13):
        while e % p == 0:
            e //= p
    return e == 1


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _half_extent(rng, lo, hi):
    """Half an extent, spread over the logarithm of its range."""
    while True:
        v = _log_int(rng, lo, hi)
        if _smooth(2 * v):
            return v


def _grid(rng, geom):
    """(K, L) of one geometry's range."""
    if geom == "1d":    # the paper's tables go from 40 to some 10^5 points
        return _half_extent(rng, 4, 42), _half_extent(rng, 8, 1024)
    if geom == "2d3":   # Ex. 4.2: up to 24 x 24 x 320
        return _half_extent(rng, 3, 12), _half_extent(rng, 10, 160)
    if geom == "2d4":   # the sweep's range of windows
        return rng.randint(6, 14), rng.randint(6, 16)
    return rng.randint(2, 6), rng.randint(3, 7)  # 3d6


def draw(rng):
    kind = rng.choice(["apply"] * 6 + ["conv", "batch", "eigenfunction", "learned_forward", "learned_grad", "eigs"])
    order = rng.choice(["grid", "grid", "window"])
    lam = round(math.exp(rng.uniform(math.log(0.1), math.log(10.0))), 3)
    if kind in ("apply", "conv"):
        nvec = _log_int(rng, 1, 24)
        if rng.random() < 0.25:  # float32 convolution: the benchmark's two workloads
            geom = rng.choice(["2d4", "2d4", "3d6"])
            K, L = (rng.choice([12, 13, 14]), rng.randint(8, 16)) if geom == "2d4" else (8, rng.randint(4, 7))
            return _case("", kind, geom, K, L, lam=round(rng.uniform(0.1, 2.5), 3), precision="fp32",
                         order=order, nvec=nvec if geom == "2d4" else min(nvec, 8))
        geom = rng.choice(["1d", "2d3", "2d4", "3d6"])
        K, L = _grid(rng, geom)
        pairs = 0
        if rng.random() < 0.25:  # modes off the axes, few to many
            pairs = _log_int(rng, 2, 40)
            geom, K, L = rng.choice([("1d", K, min(L, 200)), ("2d4", rng.randint(4, 8), rng.randint(5, 10))])
            K = min(K, 42)
        return _case("", kind, geom, K, L, lam=lam, order=order, nvec=nvec, pairs=pairs)
    if kind == "batch":
        return _case("", kind, "2d4", 0, rng.randint(6, 16), lam=lam, order=order, nvec=rng.randint(1, 8),
                     plans=rng.randint(2, 8))
    if kind == "eigenfunction":
        geom = rng.choice(["1d", "2d3", "2d4"])
        K, L = {"1d": (rng.randint(4, 14), _half_extent(rng, 10, 64)),
                "2d3": (rng.randint(3, 8), _half_extent(rng, 10, 50)),
                "2d4": (rng.randint(4, 6), rng.randint(4, 8))}[geom]
        return _case("", kind, geom, K, L, lam=lam, order=order,
                     points=_log_int(rng, 400, 10001) if geom == "1d" else _log_int(rng, 101, 1001))
    if kind in ("learned_forward", "learned_grad"):
        K, L = rng.randint(4, 10), rng.randint(4, 10)
        return _case("", kind, "2d4", K, L, lam=lam, order=order,
                     nvec=rng.randint(1, 16) if kind == "learned_forward" else rng.randint(2, 12))
    if rng.random() < 0.5:
        return _case("", kind, "1dp", rng.randint(4, 8), _half_extent(rng, 16, 64), nev=rng.randint(1, 4))
    return _case("", kind, "2d4", rng.randint(4, 8), rng.randint(4, 8), lam=round(rng.uniform(0.5, 3.0), 3),
                 precision=rng.choice(["fp32", "fp64"]), nev=rng.randint(4, 16))


# ---------------------------------------------------------------------------
# problems and inputs
# ---------------------------------------------------------------------------

def _problem(case, seed, i=0):
    """The problem of a case; a solve's coupling depends on the seed (it has
    no other input), as do the coefficients of an oblique potential."""
    rng = np.random.default_rng([seed, i, 17])
    lam, K, L = case["lam"], case["K"], case["L"]
    if case["kind"] == "eigs":
        lam *= 1.0 + 0.02 * (rng.random() - 0.5)
    if case["kind"] == "batch":  # the sweep's windows and couplings
        K, lam = 6 + (5 * i + 2) % 9, lam * (0.6 + 0.8 * rng.random())
    if case["pairs"]:
        base = W.c1_1d(K=K, L=L) if case["geom"] == "1d" else W.c2_2d(K=K, L=L)
        fixed = np.random.default_rng(case["pairs"])  # the same modes for every seed
        modes, vhat, seen = [[0] * base.n], [1.5], set()
        while len(seen) < case["pairs"]:
            m = tuple(int(x) for x in fixed.integers(-4, 5, size=base.n))
            if not any(m) or m in seen or tuple(-x for x in m) in seen:
                continue
            seen.add(m)
            c = lam * complex(rng.standard_normal(), rng.standard_normal()) / (1.0 + sum(x * x for x in m))
            modes += [list(m), [-x for x in m]]
            vhat += [c, c.conjugate()]
        return W.Problem("oblique", base.d, base.P, base.K, base.L, np.array(modes), np.array(vhat))
    return {"1d": lambda: W.c1_1d(lam=lam, K=K, L=L),
            "1dp": lambda: W.paper_example_1d(2.5 * lam, K, L),
            "2d3": lambda: W.paper_example_2d(0.8 * math.pi, 0.2 * math.pi, K, L),
            "2d4": lambda: W.c2_2d(lam=lam, K=K, L=L),
            "3d6": lambda: W.c3_3d(lam=lam, K=K, L=L),
            "3d6p": lambda: W.paper_example_3d(math.pi, K, L)}[case["geom"]]()


def _plan(case, prob):
    plan = iw.Plan.from_problem(prob, precision=case["precision"], order=case["order"])
    if case["tuned"]:
        plan.tune(nvec=case["nvec"])
    return plan


def _block(seed, i, m, N):
    """Complex standard normal vectors, as the benchmark applies to."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (int(seed) % (1 << 40)) + i)
    return torch.randn((m, N), dtype=torch.complex128, device=DEV, generator=g)


def _params(seed):
    """A network that has left its initial state: uniform layers, both
    convolution layers switched on."""
    rng = np.random.default_rng([seed, 5])
    out = []
    for l in range(4):
        b = (1.0 if l < 3 else 0.3) / math.sqrt(DIMS[l])
        out += [rng.uniform(-b, b, DIMS[l] * DIMS[l + 1]), rng.uniform(-b, b, DIMS[l + 1])]
    return np.concatenate(out + [[-0.4, 0.6]]).astype(np.float32)


def _smooth_block(seed, prob, m, order):
    """Vectors that decay with the kinetic energy, as iterates and states do."""
    lam = _kinetic(prob, order)
    return _block(seed, 0, m, prob.N) / (1.0 + lam)


def _ritz_targets(prob, m):
    """Stand-ins for the exact eigenvalues: just above the spectrum's lower bound."""
    nu = float(np.abs(prob.vhat).sum())
    return -0.9 * nu + 0.05 * nu * np.arange(m) / m


def prepare(case, seed):
    if case["kind"] == "batch":
        probs = [_problem(case, seed, i) for i in range(case["plans"])]
        plans = [_plan(case, p) for p in probs]
        xs = [_block(seed, i, 1 + (case["nvec"] + 3 * i) % case["nvec"], p.N) for i, p in enumerate(probs)]
        return {"case": case, "plans": plans, "batch": iw.Batch(plans, precision=case["precision"]),
                "x": xs, "y": [torch.empty_like(x) for x in xs]}
    prob = _problem(case, seed)
    plan = _plan(case, prob)
    s = {"case": case, "plan": plan, "seed": int(seed) & 0x7FFFFFFF}
    if case["kind"] in ("apply", "conv"):
        s["x"] = _block(seed, 0, case["nvec"], prob.N)
        s["y"] = torch.empty_like(s["x"])
    elif case["kind"] == "eigenfunction":
        s["x"] = _smooth_block(seed, prob, 1, case["order"])[0].contiguous()
    elif case["kind"] != "eigs":
        net = iw.Learned()
        net.set(_params(seed))
        plan.attach(net)
        s["net"] = net
        s["x"] = _smooth_block(seed, prob, case["nvec"], case["order"])
        s["lam"] = _ritz_targets(prob, case["nvec"])
    return s


def _observation(case, d):
    """[-5a, 5a]^d with a = 10^(3 - d) (Sec. 4), `points` along each axis."""
    half = 5.0 * 10.0 ** (3 - d)
    return [-half] * d, [2.0 * half / (case["points"] - 1)] * d, [case["points"]] * d


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "apply":
        return s["plan"].apply(s["x"], out=s["y"])
    if kind == "conv":
        return s["plan"].conv(s["x"], out=s["y"])
    if kind == "batch":
        return s["batch"].apply(s["x"], s["y"])
    if kind == "eigenfunction":
        return s["plan"].eigenfunction(s["x"], *_observation(case, s["plan"].d))
    if kind == "learned_forward":
        return s["plan"].learned_forward(s["x"])
    if kind == "learned_grad":
        loss, grad = s["plan"].learned_grad(s["x"], s["lam"])
        return {"loss": loss, "grad": grad}
    # the paper's convergence error (Sec. 4.1) on its example, else the benchmark's
    tol = 1e-10 if case["geom"] == "1dp" else 1e-8
    return s["plan"].eigs(case["nev"], tol=tol, maxit=4000, seed=s["seed"], want_vectors=False).evals


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _conv_flops(prob):
    """Per point: the modes' products, or two transforms where those are fewer."""
    return min(8.0 * len(prob.vhat), 10.0 * math.log2(prob.N))


def work(case):
    kind = case["kind"]
    if kind == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        for i in range(case["plans"]):
            p = _problem(case, 0, i)
            pts = p.N * (1 + (case["nvec"] + 3 * i) % case["nvec"])
            total["bytes"] += 32.0 * pts
            total["flops"] += (_conv_flops(p) + 4.0) * pts
        return total
    prob = _problem(case, 0)
    per = _conv_flops(prob) + 4.0
    if kind in ("apply", "conv"):
        return {"bytes": 32.0 * prob.N * case["nvec"], "flops": per * prob.N * case["nvec"]}
    if kind == "eigenfunction":
        # the sum over the last k_I axis first (it is a sum of its own for
        # every other index), then over the rest
        n, rest = case["points"], prob.N / (2 * case["K"])
        out = float(n) ** prob.d
        flops = 8.0 * prob.N * n + (8.0 * rest * out if prob.d > 1 else 8.0 * rest * n)
        return {"bytes": 16.0 * (prob.N + out), "flops": flops}
    if kind == "eigs":
        # twenty block iterations (well preconditioned solves take no fewer):
        # the apply of the new directions, X, W, P and their images read once
        # and X, P and their images written once
        m = case["nev"] + max(2, case["nev"] // 4)
        return {"bytes": 20.0 * 8.0 * prob.N * m * 12.0, "flops": 20.0 * prob.N * m * (per + 2.0 * 15.0 * m)}
    m, mlp = case["nvec"], 2.0 * 1024 * sum(DIMS[l] * DIMS[l + 1] for l in range(4))
    convs = 2 if kind == "learned_forward" else 6
    return {"bytes": 32.0 * prob.N * m * convs, "flops": convs * per * prob.N * m + (1 if convs == 2 else 3) * mlp}


# ---------------------------------------------------------------------------
# the same in plain float64 torch
# ---------------------------------------------------------------------------

def _window(prob):
    """Per k_II slice: the lower window ends a (nslice x d) and k_II itself,
    a_j = -K_j - floor((Q k_II)_j), Q = P_I^-1 P_II (Sec. 3.1-3.2)."""
    d, n = prob.d, prob.n
    k2 = torch.zeros((1, 0), dtype=torch.float64)
    for h in prob.L:
        ax = torch.fft.fftfreq(2 * h, d=1.0 / (2 * h), dtype=torch.float64)
        k2 = torch.cat([k2.repeat_interleave(2 * h, 0), ax.repeat(len(k2))[:, None]], dim=1)
    P = torch.from_numpy(np.ascontiguousarray(prob.P))
    q = k2 @ torch.linalg.solve(P[:, :d], P[:, d:]).T
    near = torch.round(q)
    q = torch.where((q - near).abs() <= 1e-12 * q.abs().clamp(min=1.0), near, q)
    a = -torch.tensor(list(prob.K), dtype=torch.float64) - torch.floor(q)
    return a, k2 @ P[:, d:].T, P


def _labels(prob, order, j):
    """True labels k_j of every entry (nslice x 2K_j), in the vector order."""
    a, _, _ = _window(prob)
    c = torch.arange(2 * prob.K[j], dtype=torch.float64)[None, :]
    aj = a[:, j:j + 1]
    return aj + (c if order == "window" else torch.remainder(c - aj, 2 * prob.K[j]))


def _kinetic(prob, order):
    """1/2 |2 pi P k|^2 of every entry, in the vector order."""
    d = prob.d
    _, off, P = _window(prob)
    k = [_labels(prob, order, j).to(DEV) for j in range(d)]
    off, P = off.to(DEV), P.to(DEV)
    shape = [len(off)] + [2 * x for x in prob.K]
    lam = torch.zeros(shape, dtype=torch.float64, device=DEV)
    for i in range(d):
        v = off[:, i].reshape([-1] + [1] * d)
        for j in range(d):
            v = v + P[i, j] * k[j].reshape([len(off)] + [2 * prob.K[j] if q == j else 1 for q in range(d)])
        lam += v * v
    return 2.0 * math.pi ** 2 * lam.reshape(-1)


def _to_grid(prob):
    """Window-order position of every grid-order entry."""
    d, ns = prob.d, int(np.prod([2 * x for x in prob.L]))
    a, _, _ = _window(prob)
    pos = torch.zeros([ns] + [1] * d, dtype=torch.int64)
    for j in range(d):
        E = 2 * prob.K[j]
        p = torch.remainder(torch.arange(E, dtype=torch.float64)[None, :] - a[:, j:j + 1], E).to(torch.int64)
        pos = pos * E + p.reshape([ns] + [E if q == j else 1 for q in range(d)])
    nk = int(np.prod([2 * x for x in prob.K]))
    return (torch.arange(ns).reshape([ns] + [1] * d) * nk + pos).reshape(-1).to(DEV)


def _conv(prob, order, x):
    """sum_m Vhat_m x[(k* - m) mod ext], one vector at a time."""
    d, n = prob.d, prob.n
    perm = _to_grid(prob) if order == "window" else None
    out = torch.empty_like(x)
    axis = [n - d + j if j < d else j - d for j in range(n)]  # grid axis of paper index j
    for v in range(x.shape[0]):
        g = (x[v][perm] if perm is not None else x[v]).reshape(prob.ext)
        acc = torch.zeros_like(g)
        for m, c in zip(np.asarray(prob.modes), prob.vhat):
            moved = [(int(m[j]), axis[j]) for j in range(n) if m[j]]
            acc += complex(c) * (torch.roll(g, [s for s, _ in moved], [t for _, t in moved]) if moved else g)
        if perm is not None:
            out[v][perm] = acc.reshape(-1)
        else:
            out[v] = acc.reshape(-1)
    return out


def _apply(prob, order, x, lam):
    return lam[None, :] * x + _conv(prob, order, x)


def _exact_eigenfunction(case, prob, u):
    """sum_k U_k exp(i 2 pi (P k) . xi), a block of window points at a time."""
    d = prob.d
    _, off, P = _window(prob)
    shape = [len(off)] + [2 * x for x in prob.K]
    origin, step, npts = _observation(case, d)
    k = [_labels(prob, case["order"], j).reshape([shape[0]] + [shape[1 + j] if q == j else 1 for q in range(d)])
         for j in range(d)]
    f = [sum((P[i, j] * k[j] for j in range(d)), off[:, i].reshape([-1] + [1] * d)).expand(shape).reshape(-1).to(DEV)
         for i in range(d)]
    xi = [origin[j] + step[j] * torch.arange(npts[j], dtype=torch.float64, device=DEV) for j in range(d)]

    def wave(i, lo, hi):
        t = f[i][lo:hi, None] * xi[i][None, :]
        t = 2.0 * math.pi * (t - torch.round(t))
        return torch.complex(torch.cos(t), torch.sin(t))

    out = torch.zeros(npts, dtype=torch.complex128, device=DEV)
    for lo in range(0, prob.N, 2048):
        hi = min(prob.N, lo + 2048)
        a = u[lo:hi, None] * wave(0, lo, hi)
        out += a.sum(0) if d == 1 else torch.matmul(a.T.contiguous(), wave(1, lo, hi))
    return out


def _network(prob, seed, lam, requires_grad):
    """(D0, E, beta coefficients, parameters) of the learned preconditioner;
    weights rounded to bfloat16 as the definition has it."""
    S = 1024
    p32 = torch.from_numpy(_params(seed))
    layers, at = [], 0
    for l in range(4):
        w = p32[at:at + DIMS[l] * DIMS[l + 1]].to(torch.bfloat16).to(torch.float64).reshape(DIMS[l], DIMS[l + 1])
        at += DIMS[l] * DIMS[l + 1]
        b = p32[at:at + DIMS[l + 1]].to(torch.float64)
        at += DIMS[l + 1]
        layers.append([t.to(DEV).requires_grad_(requires_grad) for t in (w, b)])
    beta = p32[at:].to(torch.float64).to(DEV).requires_grad_(requires_grad)
    zero = np.all(np.asarray(prob.modes) == 0, axis=1)
    vh = np.asarray(prob.vhat)
    nu, s2, v0 = np.abs(vh[~zero]).sum(), (np.abs(vh[~zero]) ** 2).sum(), vh[zero].real.sum()
    sigma, emax = max(0.0, nu - v0), float(lam.max())
    c = (torch.arange(S, dtype=torch.float64, device=DEV) + 0.5) / S
    e = emax * c * c
    h = e + v0 + sigma
    F = torch.stack([c, torch.log1p(e) / 8, e / (e + nu), torch.full_like(c, math.log1p(nu) / 4),
                     h * h / (h * h + s2), nu / h, torch.full_like(c, math.log1p(emax) / 8),
                     torch.sqrt(e) / (torch.sqrt(e) + math.sqrt(nu))], dim=1)
    for l, (w, b) in enumerate(layers):
        F = F @ w + b
        if l < 3:
            F = torch.nn.functional.gelu(F)
    shell = torch.floor(S * torch.sqrt(lam / emax)).clamp(max=S - 1).to(torch.int64)
    hk = lam + v0 + sigma
    M = hk / (hk * hk + s2)
    return 0.5 * M * (1.0 + torch.exp(F[shell, 0])), M * torch.exp(F[shell, 1]), beta, layers


def _precondition(prob, order, r, D0, E, beta):
    a, b1 = beta[0], beta[1].clamp(min=0.0)
    A = _conv(prob, order, E[None, :] * r)
    C = _conv(prob, order, E[None, :] * A)
    return (D0 + b1 * a * a * E)[None, :] * r + E[None, :] * (2.0 * a * b1 * A + b1 * C)


class _ConvGrad(torch.autograd.Function):
    """The convolution is Hermitian: its adjoint is itself."""

    @staticmethod
    def forward(ctx, x, prob, order):
        ctx.of = (prob, order)
        return _conv(prob, order, x)

    @staticmethod
    def backward(ctx, g):
        return _conv(*ctx.of, g.contiguous()), None, None


def _exact_grad(case, prob, seed):
    order, lam = case["order"], _kinetic(prob, case["order"])
    X = _smooth_block(seed, prob, case["nvec"], order)
    target = torch.from_numpy(_ritz_targets(prob, case["nvec"]))

    def ritz(S, HS):
        """Ritz pairs of the rows of S, in float64 on the host."""
        B, A = (S.conj() @ S.T).cpu(), (S.conj() @ HS.T).cpu()
        Li = torch.linalg.inv(torch.linalg.cholesky(0.5 * (B + B.mH)))
        return Li, Li @ (0.5 * (A + A.mH)) @ Li.mH

    HX = _apply(prob, order, X, lam)
    Li, small = ritz(X, HX)
    theta, C = torch.linalg.eigh(small)
    C = (Li.mH @ C).to(DEV)
    Y, HY = C.T @ X, C.T @ HX
    R = HY - theta.to(DEV)[:, None] * Y
    D0, E, beta, layers = _network(prob, seed, lam, True)
    a, b1 = beta[0], beta[1].clamp(min=0.0)
    A = _ConvGrad.apply(E[None, :] * R, prob, order)
    CC = _ConvGrad.apply(E[None, :] * A, prob, order)
    T = (D0 + b1 * a * a * E)[None, :] * R + E[None, :] * (2.0 * a * b1 * A + b1 * CC)
    HT = lam[None, :] * T + _ConvGrad.apply(T, prob, order)
    low = torch.linalg.eigvalsh(ritz(torch.cat([Y, T]), torch.cat([HY, HT]))[1])[:case["nvec"]]
    loss = (low - target).sum() / (theta - target).sum()
    flat = [t for wb in layers for t in wb] + [beta]
    grads = torch.autograd.grad(loss, flat)
    return {"loss": float(loss), "grad": torch.cat([g.reshape(-1) for g in grads]).detach()}


def exact(case, seed):
    kind, order = case["kind"], case["order"]
    if kind == "batch":
        out = []
        for i in range(case["plans"]):
            p = _problem(case, seed, i)
            x = _block(seed, i, 1 + (case["nvec"] + 3 * i) % case["nvec"], p.N)
            out.append(_apply(p, order, x, _kinetic(p, order)))
        return out
    prob = _problem(case, seed)
    if kind in ("apply", "conv"):
        x = _block(seed, 0, case["nvec"], prob.N)
        return _conv(prob, order, x) if kind == "conv" else _apply(prob, order, x, _kinetic(prob, order))
    if kind == "eigenfunction":
        return _exact_eigenfunction(case, prob, _smooth_block(seed, prob, 1, order)[0])
    if kind == "learned_forward":
        lam = _kinetic(prob, order)
        D0, E, beta, _ = _network(prob, seed, lam, False)
        return _precondition(prob, order, _smooth_block(seed, prob, case["nvec"], order), D0, E, beta)
    if kind == "learned_grad":
        return _exact_grad(case, prob, seed)
    if prob.N > 4000:  # a dense eigenproblem of more unknowns takes too long
        return None
    eye = torch.eye(prob.N, dtype=torch.complex128, device=DEV)
    H = _conv(prob, order, eye).real.contiguous()  # real symmetric: every Vhat is real
    H += torch.diag(_kinetic(prob, order))
    return np.linalg.eigvalsh(H.cpu().numpy())[:case["nev"]]

"""Potentials of few Fourier modes, applied as the wrapped convolution that
F V F^{-1} equals (App. C), against the CPU oracle's sparse H~ and against the
transforms (a named schedule always runs them).

Tolerance: every product and sum is float64 in either precision of the plan,
with at most 2 x 16 modes and the kinetic term per point, so
||y - H~ x||_2 <= 1e-13 (max Lambda + sum|Vhat|) ||x||_2, the float64 bar of the
transforms, holds with a wide margin (a point's sum of 34 terms rounds by less
than 34 eps = 8e-15 of it).
"""

import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W

pytestmark = pytest.mark.gpu

P1 = np.array([[1.0, W.GOLDEN]])
P3 = np.array([[1.0, 0.1, math.cos(0.7)], [0.0, 1.0, math.sin(0.7)]])
P4 = W.rot_pair_P()
P6 = W.cubic_pair_P()


def star(P, K, L, seed=1, real=False, skip=(), flip=()):
    """One pair of modes +-e_j per axis with its own (complex) coefficient."""
    d, n = P.shape
    rng = np.random.default_rng(seed)
    modes, vhat = [[0] * n], [0.7]
    for j in range(n):
        if j in skip:
            continue
        c = complex(rng.standard_normal(), 0.0 if real else rng.standard_normal())
        e = [0] * n
        e[j] = -1 if j in flip else 1
        modes += [e, [-x for x in e]]
        vhat += [c, c.conjugate()]
    return W.Problem("star", d, P, list(K), list(L), np.array(modes), np.array(vhat))


def pairs(P, K, L, count, seed=2, span=3):
    """`count` random pairs of modes off the axes, coefficients complex."""
    d, n = P.shape
    rng = np.random.default_rng(seed)
    modes, vhat, seen = [[0] * n], [-0.4], set()
    while len(seen) < count:
        m = tuple(int(x) for x in rng.integers(-span, span + 1, size=n))
        if not any(m) or m in seen or tuple(-x for x in m) in seen:
            continue
        seen.add(m)
        c = complex(rng.standard_normal(), rng.standard_normal())
        modes += [list(m), [-x for x in m]]
        vhat += [c, c.conjugate()]
    return W.Problem("pairs", d, P, list(K), list(L), np.array(modes), np.array(vhat))


def block(N, m, seed=3):
    return torch.from_numpy(np.ascontiguousarray(W.random_block(N, m, seed=seed).T)).to("cuda:0")


def check(prob, order, nvec, window="exact", same=True):
    """Against the oracle; both precisions give the same bits when both take
    the convolution; a vector's result does not depend on its block."""
    H = O.hamiltonian_sparse(prob.P, prob.d, prob.K, prob.L, prob.modes, prob.vhat, window)
    with lib.Plan.from_problem(prob, order=order, window=window) as p, \
            lib.Plan.from_problem(prob, order=order, window=window, precision="fp32") as q:
        pos = O.kstar_to_position(O.index_shift(p.indices(), prob.K, prob.L), prob.K, prob.L)
        x = block(prob.N, nvec)
        y = p.apply(x)
        one = torch.stack([p.apply(x[i].contiguous()) for i in (0, nvec - 1)])
        y32 = q.apply(x)
        c = p.conv(x)
        torch.cuda.synchronize()
        assert torch.equal(one[0], y[0]) and torch.equal(one[1], y[-1])
        if same:
            assert torch.equal(y, y32)
        X = x.cpu().numpy().T
        G = np.empty_like(X)
        G[pos] = X                       # grid order
        ref = (H @ G)[pos]
        nb = p.norm_bound()
        bar = 1e-13 * nb * np.linalg.norm(X, axis=0)
        assert np.all(np.linalg.norm(y.cpu().numpy().T - ref, axis=0) <= bar)
        kin = p.kinetic()
        assert np.all(np.linalg.norm(c.cpu().numpy().T - (ref - kin[:, None] * X), axis=0) <= bar)


STARS = {
    # name: (P, K, L, vectors, options); sizes at tile edges and remainders
    "1d": (P1, [21], [300], 3, {}),
    "1d_tiny": (P1, [1], [2], 2, {}),
    "1d_plane_33": (P1, [33], [250], 2, {"real": True}),
    "2d3": (P3, [6, 7], [50], 4, {}),
    "2d3_flip": (P3, [5, 6], [33], 11, {"flip": (0, 2)}),
    "2d3_extent_2": (P3, [12, 11], [1], 40, {}),
    "2d4": (P4, [5, 6], [9, 7], 5, {}),
    "2d4_one_axis": (P4, [4, 4], [6, 5], 9, {"skip": (0, 1, 2)}),
    "2d4_no_first": (P4, [6, 4], [5, 6], 6, {"skip": (2,), "flip": (3,)}),
    "2d4_short_axes": (P4, [8, 7], [1, 1], 40, {}),
    "2d4_wide_plane": (P4, [14, 15], [3, 2], 4, {"real": True}),
    "3d6": (P6, [2, 3, 2], [3, 4, 2], 3, {}),
    "3d6_planes_cut": (P6, [3, 5, 4], [2, 3, 3], 2, {}),
    "3d6_extent_2": (P6, [1, 1, 1], [3, 2, 5], 40, {}),
}


@pytest.mark.parametrize("order", ["grid", "window"])
@pytest.mark.parametrize("name", sorted(STARS))
def test_star(name, order):
    P, K, L, nvec, kw = STARS[name]
    print(f"case: star {name} {order}", flush=True)
    check(star(P, K, L, **kw), order, nvec)


@pytest.mark.parametrize("window", ["rounded", "pm"])
def test_star_other_windows(window):
    print(f"case: star {window}", flush=True)
    check(star(P4, [5, 4], [6, 6]), "window", 4, window=window)


@pytest.mark.parametrize("order", ["grid", "window"])
@pytest.mark.parametrize("P,K,L,counts", [
    (P1, [9], [21], (1, 2, 5, 16)),
    (P3, [4, 5], [13], (3, 7)),
    (P4, [4, 3], [5, 4], (1, 4, 8)),
    (P6, [2, 2, 2], [2, 3, 2], (2, 4)),
], ids=["d1n2", "d2n3", "d2n4", "d3n6"])
def test_pairs(P, K, L, counts, order):
    for count in counts:
        for nvec in (1, 7):
            print(f"case: {count} pairs n={P.shape[1]} {order} nvec={nvec}", flush=True)
            check(pairs(P, K, L, count), order, nvec)


@pytest.mark.parametrize("P,K,L,count", [(P4, [4, 3], [5, 4], 12), (P6, [2, 2, 2], [2, 3, 2], 6)], ids=["d2", "d3"])
def test_pairs_float64_only(P, K, L, count):
    """Counts that only a float64 plan takes this way."""
    check(pairs(P, K, L, count), "window", 3, same=False)


def test_aliases_and_edges():
    """Modes that wrap onto each other or onto the constant, several on one
    axis, a long axis, no modes at all."""
    one = lambda modes, vhat, K=(3,), L=(4,): W.Problem(  # noqa: E731
        "edge", 1, P1, list(K), list(L), np.array(modes).reshape(-1, 2), np.array(vhat, dtype=np.complex128))
    c = 0.3 + 0.2j
    cases = [one([[6, 0], [-6, 0]], [0.5, 0.5]),                                  # 6 = 0 mod 2K
             one([[0, 1], [0, -1], [0, 9], [0, -9]], [c, c.conjugate(), 0.1, 0.1]),  # 9 = 1 mod 2L
             one([[1, 0], [-1, 0], [2, 0], [-2, 0]], [c, c.conjugate(), c, c.conjugate()]),
             one([[0, 4], [0, -4]], [c, c.conjugate()]),                          # half the extent
             one([[0, 2], [0, -2]], [c, c.conjugate()], (5,), (60,)),             # a step of two along axis 0
             one([[0, 1], [0, -1]], [c, c.conjugate()], (42,), (40,)),
             one([], []), one([[0, 0]], [2.5]), one([[1, 0], [-1, 0]], [0.0, 0.0])]
    for k, prob in enumerate(cases):
        for order in ("grid", "window"):
            print(f"case: edge {k} {order}", flush=True)
            check(prob, order, 3)


def test_four_points_per_thread():
    """The widest form of the 6-axis walk (16-point slow axes, many vectors):
    the same bits as one vector at a time, which takes the narrow form."""
    prob = star(P6, [2, 2, 2], [8, 8, 8])
    print("case: four points per thread", flush=True)
    with lib.Plan.from_problem(prob) as p:
        x = torch.randn((66, prob.N), dtype=torch.complex128, device="cuda:0",
                        generator=torch.Generator("cuda:0").manual_seed(4))
        y = p.apply(x)
        for i in (0, 1, 37, 65):
            assert torch.equal(p.apply(x[i].contiguous()), y[i])
    check(prob, "grid", 1)


@pytest.mark.parametrize("make", [lambda: star(P4, [6, 5], [8, 7]), lambda: pairs(P4, [4, 4], [5, 5], 6),
                                  lambda: star(P6, [2, 2, 3], [3, 3, 2])], ids=["star4", "pairs", "star6"])
@pytest.mark.parametrize("order", ["grid", "window"])
def test_equals_the_transforms(make, order):
    prob = make()
    print(f"case: against the transforms N={prob.N} {order}", flush=True)
    with lib.Plan.from_problem(prob, order=order) as p, \
            lib.Plan.from_problem(prob, order=order, schedule="threepass") as t:
        x = block(prob.N, 4)
        diff = (p.apply(x) - t.apply(x)).norm(dim=1)
        assert torch.all(diff <= 2e-13 * p.norm_bound() * x.norm(dim=1))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("graph", [False, True])
def test_batch_of_all_kinds(graph, prec):
    """Walks of every kind, point kernels of several widths and a plan that
    takes the transforms in one batch: each result equals the plan's own
    apply, over replays with other vectors and counts."""
    probs = [star(P4, [5, 4], [6, 5]), star(P4, [3, 6], [4, 7]), star(P1, [20], [64]), star(P3, [5, 5], [24]),
             star(P6, [2, 2, 2], [3, 2, 3]), pairs(P4, [4, 3], [4, 4], 4), pairs(P4, [3, 3], [4, 4], 6),
             pairs(P1, [6], [12], 30, span=6)]
    plans = [lib.Plan.from_problem(p, precision=prec) for p in probs]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        batch = lib.Batch(plans, precision=prec, graph=graph)
        for rep in range(4):
            print(f"case: batch graph={graph} {prec} rep {rep}", flush=True)
            xs = [block(p.N, 1 + (3 * i + 5 * rep) % 7, seed=10 * rep + i) for i, p in enumerate(probs)]
            if rep == 2:
                xs[0] = xs[3] = xs[5] = None
            ys = [None if x is None else torch.empty_like(x) for x in xs]
            batch.apply(xs, ys)
            refs = [None if x is None else p.apply(x) for p, x in zip(plans, xs)]
            torch.cuda.synchronize()
            for i, (y, r) in enumerate(zip(ys, refs)):
                assert y is None or torch.equal(y, r), i
        batch.close()
    for p in plans:
        p.close()


@pytest.mark.parametrize("d,plans", [(1, 9), (2, 9), (2, 3), (3, 5)])
def test_batch_deals_items_over_xcds(d, plans):
    """Items of one kind whose groups end at every XCD, with and without
    vectors: each result equals the plan's own apply."""
    P, K, L = {1: (P1, [9], [40]), 2: (P4, [3, 4], [6, 5]), 3: (P6, [2, 2, 3], [3, 2, 2])}[d]
    probs = [star(P, [K[0] + i % 3] + K[1:], L, seed=i) for i in range(plans)]
    ps = [lib.Plan.from_problem(p) for p in probs]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        batch = lib.Batch(ps, precision="fp64", graph=False)
        for rep in range(3):
            print(f"case: batch over XCDs d={d} plans={plans} rep {rep}", flush=True)
            xs = [None if (i + rep) % 4 == 3 else block(p.N, 1 + (2 * i + rep) % 9, seed=i) for i, p in enumerate(probs)]
            ys = [None if x is None else torch.full_like(x, float("nan")) for x in xs]
            batch.apply(xs, ys)
            refs = [None if x is None else p.apply(x) for p, x in zip(ps, xs)]
            torch.cuda.synchronize()
            for i, (y, r) in enumerate(zip(ys, refs)):
                assert y is None or torch.equal(y, r), i
        batch.close()
    for p in ps:
        p.close()


def test_under_capture_and_tuned():
    """A captured apply replays on new data; tuning a plan that has nothing to
    choose leaves its results alone."""
    prob = star(P4, [6, 6], [8, 8])
    print("case: capture", flush=True)
    with lib.Plan.from_problem(prob, precision="fp32") as p:
        x, y = block(prob.N, 3), torch.empty((3, prob.N), dtype=torch.complex128, device="cuda:0")
        before = p.apply(x).clone()
        assert p.tune(nvec=3) > 0.0
        assert torch.equal(p.apply(x), before)
        z = torch.empty_like(y)
        p.apply_noalloc(x, z)
        assert torch.equal(z, before)
        g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=s):
            p.apply(x, out=y)
        for seed in (5, 6, 7):
            x.copy_(block(prob.N, 3, seed=seed))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, p.apply(x))

"""The rule between the few-mode convolution and the transforms, on both sides of
its lines: which route a plan takes (the profile's stages tell), and that its
results are the transforms' (a named schedule) to the sums' rounding,
2e-13 (max Lambda + sum |Vhat|) ||x|| in float64 and 2e-6 of it in float32,
whose transforms round to 6e-8 over some ten stages."""

import numpy as np
import pytest
import torch

import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W
from test_few_modes_gpu import P1, P3, P4, P6, block

pytestmark = pytest.mark.gpu

P13 = np.array([[1.0, W.GOLDEN, 0.414]])
P14 = np.array([[1.0, W.GOLDEN, 0.414, 0.271]])
P25 = np.concatenate([P4, [[0.3], [0.2]]], axis=1)


def oblique(P, K, L, count, far):
    """`count` pairs off the axes within 4 of the origin, one of them beyond
    that where `far` is set."""
    d, n = P.shape
    rng = np.random.default_rng(count)
    modes, vhat, seen = [[0] * n], [0.5], set()
    while len(seen) < count:
        m = rng.integers(1, 5, size=n) * rng.choice([-1, 1], size=n)
        m[d] = 5 + rng.integers(0, 2) if far and not seen else rng.integers(1, 5)
        if tuple(m) in seen:
            continue
        seen.add(tuple(int(x) for x in m))
        c = complex(rng.standard_normal(), rng.standard_normal())
        modes += [list(m), list(-m)]
        vhat += [c, c.conjugate()]
    return W.Problem("oblique", d, P, list(K), list(L), np.array(modes), np.array(vhat))


def lattice(P, K, L, step):
    d, n = P.shape
    e = np.eye(n, dtype=np.int64)
    e[d, d] = step
    return W.Problem("lattice", d, P, list(K), list(L), np.concatenate([e, -e]), np.full(2 * n, 0.4))


# plan, precision, pairs that take the convolution, pairs that do not; near, then far
LINES = [
    ("fp64", P1, [9], [1000], (16, 17), (16, 17)),
    ("fp32", P1, [9], [1000], (12, 13), (12, 13)),
    ("fp32", P1, [9], [100], (16, 17), (16, 17)),          # at most 16,384 points
    ("fp64", P13, [8], [20, 20], (12, 13), (12, 13)),
    ("fp32", P13, [8], [20, 20], (8, 9), (4, 5)),
    ("fp64", P14, [8], [8, 9, 8], (12, 13), (4, 5)),
    ("fp64", P14, [4], [6, 5, 5], (8, 9), (8, 9)),
    ("fp64", P3, [8, 8], [50], (12, 13), (12, 13)),
    ("fp32", P3, [8, 8], [50], (8, 9), (6, 7)),
    ("fp64", P4, [7, 7], [8, 8], (12, 13), (4, 5)),
    ("fp32", P4, [7, 7], [8, 8], (4, 5), (2, 3)),
    ("fp32", P4, [5, 5], [7, 5], (8, 9), (8, 9)),
    ("fp64", P25, [6, 6], [7, 5, 5], (4, 5), (3, 4)),
    ("fp32", P25, [6, 6], [7, 5, 5], (2, 3), (2, 3)),
    ("fp64", P6, [4, 3, 3], [7, 3, 3], (4, 5), (4, 5)),
    ("fp32", P6, [4, 3, 3], [7, 3, 3], (2, 3), (2, 3)),
]


def takes(prob, precision):
    """Whether a plan's apply takes the convolution; its result is checked."""
    print(f"case: {precision} n={prob.n} N={prob.N} modes={len(prob.vhat)}", flush=True)
    x = block(prob.N, 2)
    with lib.Plan.from_problem(prob, precision=precision) as p, \
            lib.Plan.from_problem(prob, precision=precision, schedule="threepass") as t:
        p.profile(True)
        y = p.apply(x)
        stages = p.profile_read()
        assert not p.schedule()["fused"] or prob.N <= 16384
        diff = (y - t.apply(x)).norm(dim=1)
        assert torch.all(diff <= (2e-13 if precision == "fp64" else 2e-6) * p.norm_bound() * x.norm(dim=1))
        if p.schedule()["fused"]:  # one stage either way: only the convolution is float64 in a float32 plan
            return torch.equal(y, p.apply(x, precision="fp64")) if precision == "fp32" else None
        return stages["fused"]["launches"] > 0


@pytest.mark.parametrize("case", LINES, ids=[f"{c[0]}-d{c[1].shape[0]}n{c[1].shape[1]}-{int(np.prod(c[2] + c[3])) << c[1].shape[1]}"
                                            for c in LINES])
@pytest.mark.parametrize("far", [False, True], ids=["near", "far"])
def test_lines(case, far):
    precision, P, K, L, near_line, far_line = case
    inside, outside = far_line if far else near_line
    assert takes(oblique(P, K, L, inside, far), precision) in (True, None)
    assert takes(oblique(P, K, L, outside, far), precision) in (False, None)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_lattices(precision):
    """One pair an axis: whatever the axes are, as long as the modes are near."""
    assert takes(lattice(P14, [8], [8, 9, 8], 1), precision)
    assert takes(lattice(P25, [6, 6], [7, 5, 5], 4), precision)
    assert not takes(lattice(P25, [6, 6], [7, 5, 5], 5), precision)

"""The transforms' passes on the workloads whose plans choose the few-mode
convolution by themselves: a named schedule runs them (five passes where no
single split fits), as every solve does.  The bars are those of the other
checks of the transforms against the oracle."""

import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W
from test_apply_gpu import check_full, sampled_check, to_dev
from test_few_modes_gpu import P4, pairs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("lam", [0.5, 5.0])
def test_c2_full_size_sampled(prec, lam):
    prob = W.c2_2d(lam=lam)
    print(f"case: 2d_lifted_4d N={prob.N} {prec} lam={lam} passes", flush=True)
    sampled_check(prob, prec, schedule="threepass")


def test_c3_full_size_sampled():
    prob = W.c3_3d(lam=3.0)
    print(f"case: 3d_lifted_6d N={prob.N} fp32 passes", flush=True)
    sampled_check(prob, "fp32", nvec=1, nsample=200, schedule="threepass")


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_five_pass_grid_sampled(prec):
    """40^3 x 10^3 points, which no three passes fit."""
    prob = W.paper_example_3d(math.pi, 5, 20)
    print(f"case: ex4.3 K=5 L=20 N={prob.N} {prec} five passes", flush=True)
    sampled_check(prob, prec, nvec=1, nsample=200, schedule="threepass")


@pytest.mark.timeout(600)
def test_table9_reference_grid_five_pass_sampled():
    """80^3 x 10^3 points: two-stage axes in the middle pass and in the further one."""
    prob = W.paper_example_3d(math.pi, 5, 40)
    print(f"case: ex4.3 K=5 L=40 N={prob.N} fp32 five passes", flush=True)
    sampled_check(prob, "fp32", nvec=1, nsample=200, schedule="threepass")


def test_hermitian_batch_and_deterministic():
    prob = W.c2_2d(lam=5.0)
    print("case: hermitian/batch/determinism, passes", flush=True)
    with lib.Plan.from_problem(prob, precision="fp32", schedule="threepass") as p:
        X = to_dev(W.random_block(prob.N, 4, seed=1))
        HX = p.apply(X)
        assert torch.equal(HX, p.apply(X))
        assert torch.equal(HX, torch.stack([p.apply(X[i].contiguous()) for i in range(4)]))
        a, b = torch.vdot(X[0], HX[1]).item(), torch.vdot(HX[0], X[1]).item()
        vs = float(np.abs(prob.vhat).sum())
        assert abs(a - b) <= 8e-6 * vs * (X[0].norm() * X[1].norm()).item()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("graph", [False, True])
def test_batch_of_transforms(prec, graph):
    """Ragged grids in three passes, fused ones and a potential grid: each result
    equals the plan's own apply over replays, and these the oracle's."""
    probs = [W.c2_2d(lam=0.3 + i, K=K, L=4) for i, K in enumerate([3, 5, 4])]
    probs += [W.c2_2d(lam=3.3, K=3, L=2), W.c2_2d(lam=2.0, K=2, L=2), pairs(P4, [3, 4], [5, 4], 20)]
    schedules = ["threepass"] * 3 + ["fused"] * 2 + ["threepass"]
    plans = [lib.Plan.from_problem(p, precision=prec, schedule=s) for p, s in zip(probs, schedules)]
    with torch.cuda.stream(torch.cuda.Stream()):
        batch = lib.Batch(plans, precision=prec, graph=graph)
        for rep in range(4):
            print(f"case: batch of transforms {prec} graph={graph} rep {rep}", flush=True)
            blocks = [W.random_block(p.N, 1 + (3 * i + rep) % 5, seed=10 * rep + i) for i, p in enumerate(probs)]
            xs = [None if rep == 2 and i in (1, 4) else to_dev(b) for i, b in enumerate(blocks)]
            ys = [None if x is None else torch.full_like(x, float("nan")) for x in xs]
            batch.apply(xs, ys)
            refs = [None if x is None else p.apply(x) for p, x in zip(plans, xs)]
            torch.cuda.synchronize()
            for i, (y, r) in enumerate(zip(ys, refs)):
                assert y is None or torch.equal(y, r), i
        batch.close()
    for p in plans:
        p.close()
    for prob, schedule in zip(probs, schedules):
        check_full(prob, prec, schedule=schedule)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_tuned_schedule_against_the_oracle(prec):
    """The schedule that the tuner picks, through the applies of a plan with too
    many modes for the convolution."""
    prob = pairs(P4, [6, 5], [7, 6], 24)
    print(f"case: tuned N={prob.N} {prec}", flush=True)
    H = O.hamiltonian_sparse(prob.P, prob.d, prob.K, prob.L, prob.modes, prob.vhat, "exact")
    X = W.random_block(prob.N, 4, seed=3)
    with lib.Plan.from_problem(prob, precision=prec) as p:
        assert p.tune(nvec=4) > 0.0
        p.profile(True)
        pos = O.kstar_to_position(O.index_shift(p.indices(), prob.K, prob.L), prob.K, prob.L)
        y = p.apply(to_dev(X[pos])).cpu().numpy().T
        stages = p.profile_read()
        assert p.schedule()["fused"] or stages["pass2"]["launches"] == 1
        nb, vs = p.norm_bound(), float(np.abs(prob.vhat).sum())
    err = np.linalg.norm(y - (H @ X)[pos], axis=0)
    assert np.all(err <= (1e-13 * nb if prec == "fp64" else 4e-6 * vs) * np.linalg.norm(X, axis=0)), err

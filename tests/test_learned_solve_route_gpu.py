"""Solves run the transforms on every plan, with the learned preconditioner too:
a plan of few modes, whose own applies take the wrapped convolution, solves to
the same bits as one whose schedule is named."""

import numpy as np
import pytest

import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W
from test_learned_gpu import random_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("precond", ["plain", "learned"])
@pytest.mark.parametrize("batched", [False, True])
def test_few_mode_plans_solve_by_the_transforms(precision, precond, batched):
    print(f"case: {precision}, {precond}, batched {batched}", flush=True)
    net = lib.Learned(shells=256, seed=3)
    net.set(random_params(21, beta=(0.2, 0.3)))
    out = []
    for schedule in ("auto", "threepass"):
        plans = [lib.Plan.from_problem(W.c2_2d(lam=lam, K=6, L=6), precision=precision, schedule=schedule)
                 for lam in ((1.5, 3.0) if batched else (1.5,))]
        if precond == "learned":
            for p in plans:
                p.attach(net)
        sched = [p.schedule() for p in plans]
        if batched:
            ev, _, st, _ = lib.eigs_batched(plans, 6, tol=1e-8, precond=precond)
            its = [(s["iterations"], s["fallback"]) for s in st]
        else:
            r = plans[0].eigs(6, tol=1e-8, precond=precond, want_vectors=False)
            ev, its = r.evals, [(r.iterations, r.fallback)]
        out.append((sched, its, np.array(ev)))
        for p in plans:
            p.close()
    net.close()
    assert out[0][0] == out[1][0]
    assert out[0][1] == out[1][1], (out[0][1], out[1][1])
    assert np.array_equal(out[0][2], out[1][2])

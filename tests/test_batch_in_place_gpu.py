"""A batch's results written over its vectors: the transforms allow it (single
applies refuse it), and a few-mode plan's item takes them then.  Against calls
with result buffers of their own, to the transforms' bars (2e-13 (max Lambda +
sum |Vhat|) ||x|| in float64, 4e-6 sum |Vhat| ||x|| in float32)."""

import numpy as np
import pytest
import torch

import paper_2404_04507_amd as lib
from test_few_modes_gpu import P1, P4, P6, block, pairs, star

pytestmark = pytest.mark.gpu

PROBLEMS = {"fused": lambda: star(P1, [8], [16]), "star": lambda: star(P4, [6, 5], [8, 7]),
            "points": lambda: pairs(P4, [4, 4], [5, 5], 4), "star6": lambda: star(P6, [2, 3, 2], [3, 2, 3])}


def bar(plan, prob, precision, x):
    scale = 2e-13 * plan.norm_bound() if precision == "fp64" else 4e-6 * float(np.abs(prob.vhat).sum())
    return scale * x.norm(dim=1)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_batch_over_the_vectors(precision):
    probs = [make() for make in PROBLEMS.values()] + [pairs(P4, [4, 4], [5, 5], 20)]
    plans = [lib.Plan.from_problem(p, precision=precision) for p in probs]
    print(f"case: in place batch {precision}", flush=True)
    with torch.cuda.stream(torch.cuda.Stream()):
        batch = lib.Batch(plans, precision=precision, graph=True)
        for rep in range(3):
            xs = [block(p.N, 2 + i, seed=i + rep) for i, p in enumerate(probs)]
            refs = [p.apply(x) for p, x in zip(plans, xs)]
            ys = [x.clone() for x in xs]
            outs = [y if (i + rep) % 2 else torch.empty_like(y) for i, y in enumerate(ys)]
            batch.apply(ys, outs)
            torch.cuda.synchronize()
            for prob, plan, x, out, ref in zip(probs, plans, xs, outs, refs):
                assert torch.all((out - ref).norm(dim=1) <= bar(plan, prob, precision, x))
        batch.close()
    for p in plans:
        p.close()

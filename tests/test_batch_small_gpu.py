"""Batches of small few-mode plans: one kernel for any number of pairs of modes,
and no slower than the same batch by the transforms."""

import numpy as np
import pytest
import torch

import paper_2404_04507_amd as lib
from test_few_modes_gpu import P1, P4, P6, block, pairs, star

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,counts", [(1, (1, 2, 3, 4, 5, 8, 11, 16)), (2, (1, 3, 5, 8, 12)), (3, (1, 2, 4, 6))])
@pytest.mark.parametrize("order", ["grid", "window"])
def test_any_number_of_pairs(d, counts, order):
    """Plans of every number of pairs that share a launch, with a star and plans
    without vectors among them: each result equals the plan's own apply."""
    P, K, L = {1: (P1, [6], [20]), 2: (P4, [3, 4], [4, 3]), 3: (P6, [2, 2, 2], [2, 2, 3])}[d]
    probs = [pairs(P, [K[0] + i % 2] + K[1:], L, c, seed=i) for i, c in enumerate(counts)] + [star(P, K, L)]
    plans = [lib.Plan.from_problem(p, order=order) for p in probs]
    with torch.cuda.stream(torch.cuda.Stream()):
        batch = lib.Batch(plans, precision="fp64", graph=False)
        for rep in range(3):
            print(f"case: any pairs d={d} {order} rep {rep}", flush=True)
            xs = [None if (i + rep) % 5 == 4 else block(p.N, 1 + (2 * i + rep) % 9, seed=i) for i, p in enumerate(probs)]
            ys = [None if x is None else torch.full_like(x, float("nan")) for x in xs]
            batch.apply(xs, ys)
            refs = [None if x is None else p.apply(x) for p, x in zip(plans, xs)]
            torch.cuda.synchronize()
            for i, (y, r) in enumerate(zip(ys, refs)):
                assert y is None or torch.equal(y, r), i
        batch.close()
    for p in plans:
        p.close()


def batch_us(plans, graph):
    xs = [block(p.N, 1, seed=i) for i, p in enumerate(plans)]
    ys = [torch.empty_like(x) for x in xs]
    batch = lib.Batch(plans, precision="fp64", graph=graph)
    best = np.inf
    for rep in range(6):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(20):
            batch.apply(xs, ys)
        end.record()
        torch.cuda.synchronize()
        best = min(best, start.elapsed_time(end) * 50.0)
    batch.close()
    return best


@pytest.mark.parametrize("graph", [False, True])
def test_small_batches_are_not_slower_than_the_transforms(graph):
    """Eight plans of some 600 points with 3 to 12 pairs: launches are all of it."""
    probs = [pairs(P1, [8 + i % 5], [30], 3 + i % 10, seed=i) for i in range(8)]
    few = [lib.Plan.from_problem(p) for p in probs]
    transforms = [lib.Plan.from_problem(p, schedule="fused") for p in probs]
    with torch.cuda.stream(torch.cuda.Stream()):
        us = [batch_us(plans, graph) for plans in (few, transforms)]
    print(f"case: small batch graph={graph}: {us[0]:.1f} us, transforms {us[1]:.1f} us", flush=True)
    for p in few + transforms:
        p.close()
    assert us[0] <= us[1], us

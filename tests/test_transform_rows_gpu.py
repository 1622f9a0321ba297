"""The transform schedules' gather, stage twiddles and kinetic scatter, at the
row counts and axis lengths where their batches end, for one to four k_I axes
(up to three are compiled in), against the CPU oracle's sparse H~.

Tolerance: the bars of the transforms, ||y - H~ x||_2 <= bar (max Lambda +
sum |Vhat|) ||x||_2 with bar 1e-13 in float64 and 2e-6 in float32 (a transform
rounds by a few log2(points) half-ulps).
"""

import numpy as np
import pytest
import torch

import oracle as O
import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W

pytestmark = pytest.mark.gpu


def problem(d, K, L):
    rng = np.random.default_rng(d)
    P = np.hstack([np.eye(d), np.linalg.qr(rng.standard_normal((d, d)))[0]])
    modes, vhat = W.cosine_modes(2 * d, list(0.5 + rng.random(2 * d)))
    return W.Problem("rows", d, P, list(K), list(L), modes, vhat)


CASES = [
    (1, [1], [2]),           # one partial batch
    (1, [4], [33]),          # 66 points: one long axis or one register pencil
    (1, [9], [50]),          # 100 points in two stages: the last batch of twiddles is short
    (1, [50], [4]),          # the long axis is the last one
    (1, [16], [32]),         # whole batches
    (2, [3, 2], [2, 5]),
    (2, [5, 7], [3, 4]),
    (3, [2, 1, 3], [1, 2, 2]),
    (3, [2, 2, 2], [2, 2, 2]),
    (4, [1, 1, 1, 1], [1, 1, 1, 1]),  # four k_I axes: the general loop
    (4, [1, 1, 2, 1], [1, 1, 1, 2]),
]


@pytest.mark.parametrize("precision,bar", [("fp64", 1e-13), ("fp32", 2e-6)])
@pytest.mark.parametrize("schedule", ["fused", "threepass"])
@pytest.mark.parametrize("order", ["grid", "window"])
@pytest.mark.parametrize("d,K,L", CASES)
def test_rows(d, K, L, order, schedule, precision, bar):
    prob = problem(d, K, L)
    print(f"case: rows d={d} K={K} L={L} {order} {schedule} {precision}", flush=True)
    H = O.hamiltonian_sparse(prob.P, prob.d, prob.K, prob.L, prob.modes, prob.vhat, "exact")
    hn = O.norm_bound(prob.P, prob.d, prob.K, prob.L, prob.modes, prob.vhat, "exact")
    with lib.Plan.from_problem(prob, order=order, schedule=schedule, precision=precision) as p:
        pos = O.kstar_to_position(O.index_shift(p.indices(), prob.K, prob.L), prob.K, prob.L)
        X = W.random_block(p.N, 3, seed=d)
        y = p.apply(torch.from_numpy(np.ascontiguousarray(X.T)).to("cuda:0")).cpu().numpy().T
        G = np.empty_like(X)
        G[pos] = X
        ref = (H @ G)[pos]
        assert np.all(np.linalg.norm(y - ref, axis=0) <= bar * hn * np.linalg.norm(X, axis=0))

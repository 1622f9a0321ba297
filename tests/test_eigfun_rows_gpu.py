"""iwfpm_eigenfunction's two contractions: over rows of the last k_I axis where
P_I is diagonal, over window points otherwise, against the CPU oracle.

Bar: |u - u_ref| <= 1e-10 sum_k |U_k|, as the phases' rounding (a few ulps of
|P k| |xi| <= 1e4 turns here, 1e-11 of the term) and the sums allow; summing
one axis first changes the order of the additions only.
"""

import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W

pytestmark = pytest.mark.gpu

DIAG2 = np.array([[0.7, 0.0, math.cos(0.6)], [0.0, -1.3, math.sin(0.6)]])
FULL2 = np.array([[1.0, 0.25, math.cos(0.6)], [0.0, 1.0, math.sin(0.6)]])
FULL3 = np.concatenate([np.eye(3) + 0.1 * np.eye(3, k=1), W.cubic_pair_P()[:, 3:]], axis=1)

CASES = {
    # name: (P, K, L, grid points); rows and positions at the kernels' edges
    "d1_short": (np.array([[1.0, W.GOLDEN]]), [1], [1], [65]),
    "d1_long_last": (np.array([[1.0, W.GOLDEN]]), [50], [9], [130]),
    "d2_rows_2": (DIAG2, [1, 8], [5], [64, 64]),
    "d2_rows_18_last_34": (DIAG2, [9, 17], [3], [65, 63]),
    "d2_two_kII": (W.rot_pair_P(), [3, 4], [3, 2], [9, 200]),
    "d3": (W.cubic_pair_P(), [2, 3, 2], [2, 2, 1], [7, 5, 66]),
    "d2_general": (FULL2, [4, 5], [6], [33, 70]),
    "d3_general": (FULL3, [2, 1, 2], [2, 1, 2], [5, 9, 10]),
}


@pytest.mark.parametrize("order", ["grid", "window"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_rows_and_points(name, order):
    P, K, L, npts = CASES[name]
    d, n = P.shape
    prob = W.Problem(name, d, P, K, L, np.zeros((0, n), dtype=np.int64), np.zeros(0, dtype=np.complex128))
    print(f"case: {name} {order} N={prob.N}", flush=True)
    U = W.random_block(prob.N, 1, seed=5)[:, 0]
    origin, step = [-3.0 + 0.7 * j for j in range(d)], [0.31 - 0.2 * j for j in range(d)]
    ref = O.eigenfunction_on_grid(P, O.grid_labels(P, d, K, L), U, origin, step, npts)
    with lib.Plan.from_problem(prob, order=order) as p:
        pos = O.kstar_to_position(O.index_shift(p.indices(), K, L), K, L)
        u = torch.from_numpy(np.ascontiguousarray(U[pos])).to("cuda:0")
        out = p.eigenfunction(u, origin, step, npts).cpu().numpy()
        again = p.eigenfunction(u, origin, step, npts).cpu().numpy()
    assert np.abs(out - ref).max() <= 1e-10 * np.abs(U).sum()
    assert np.array_equal(out, again)

"""iwfpm_eigenfunction's scratch stays within its table budget (256 MB; grids of
this many tiles take no slice partials) where the rows of one k_II slice need
more: line cuts with a long last axis through windows of many rows.

Bar for the values, as in the other eigenfunction checks: 1e-10 sum_k |U_k|."""

import numpy as np
import pytest
import torch

import oracle as O
import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,npts", [
    ([9, 10, 3], [1, 1, 120001]),  # 360 rows a slice, 136 of them within the budget: parts of 136, 136 and 88
    ([9, 10, 3], [1, 1, 46603]),   # 356 rows within the budget: a part of four rows is left
    ([9, 10, 3], [2, 1, 46500]),   # a whole slice fits
    ([2, 2, 17], [1, 1, 1100000]),  # 16 rows a slice, 12 within the budget; 34 positions a row
])
@pytest.mark.parametrize("order", ["grid", "window"])
def test_line_cut(K, npts, order):
    P = W.cubic_pair_P()[:, :4]
    prob = W.Problem("cut", 3, P, K, [1], np.zeros((0, 4), dtype=np.int64), np.zeros(0, dtype=np.complex128))
    print(f"case: {order} N={prob.N} {npts}", flush=True)
    U = W.random_block(prob.N, 1, seed=5)[:, 0]
    origin, step = [-3.0, 2.3, -1.6], [0.31, 0.11, 0.003]
    with lib.Plan.from_problem(prob, order=order) as p:
        pos = O.kstar_to_position(O.index_shift(p.indices(), K, [1]), K, [1])
        u = torch.from_numpy(np.ascontiguousarray(U[pos])).to("cuda:0")
        out = torch.empty(npts, dtype=torch.complex128, device="cuda:0")
        with lib.Plan.from_problem(prob, order=order) as other:  # code objects are loaded
            other.eigenfunction(u, origin, step, [1, 1, 64])
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        p.eigenfunction(u, origin, step, npts, out=out)
        torch.cuda.synchronize()
        taken = free - torch.cuda.mem_get_info()[0]
        got = out.cpu().numpy()
    k = O.grid_labels(P, 3, K, [1]) @ P.T
    at = np.unique(np.concatenate([[0, 1, 63, 64, npts[2] - 65, npts[2] - 1], np.linspace(0, npts[2] - 1, 7).astype(int)]))
    for i in range(npts[0]):
        for c in at:
            xi = np.array([origin[0] + step[0] * i, origin[1], origin[2] + step[2] * c])
            ref = np.sum(U * np.exp(2j * np.pi * (k @ xi)))
            assert abs(got[i, 0, c] - ref) <= 1e-10 * np.abs(U).sum(), (i, c)
    # frequencies (8 B a row and axis) and allocation granularity beside the budget
    assert taken <= (256 + 32) << 20, taken

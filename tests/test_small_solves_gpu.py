"""Small solves on the GPU: reductions, residuals and combinations that take the
one-workgroup kernels, at the edges of their rules, against the CPU oracle.

The edges: 1024 and 2048 rows (one and two rows a block of the residual), four
columns of a block, 64 entries of a Gram, 256 coefficients of a combination;
real blocks (two vectors a column) and complex ones (a start block is given).
"""

import numpy as np
import pytest
import torch

import oracle as O
import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = {16: (1, 4), 60: (3, 5), 1000: (10, 25), 1024: (16, 16), 1040: (10, 26), 2048: (16, 32), 2080: (20, 26),
         2400: (10, 60)}


@pytest.mark.parametrize("real", [True, False], ids=["real", "complex"])
@pytest.mark.parametrize("N", sorted(SIZES))
def test_small_solve(N, real):
    K, L = SIZES[N]
    prob = W.c1_1d(K=K, L=L)
    H = O.hamiltonian_dense(prob.P, prob.d, prob.K, prob.L, prob.modes, prob.vhat, "exact")
    ref = np.linalg.eigvalsh(H)
    hn = O.norm_bound(prob.P, prob.d, prob.K, prob.L, prob.modes, prob.vhat, "exact")
    with lib.Plan.from_problem(prob) as p:
        assert p.N == N
        for block in (1, 2, 3, 4, 5, 8, 9, 12, 17):
            if 4 * block > N:
                continue
            nev = max(1, block // 2)
            print(f"case: small solve N={N} block={block} real={real}", flush=True)
            kw = {}
            if not real:
                kw["x0"] = torch.from_numpy(np.ascontiguousarray(W.random_block(N, block, seed=block).T)).to("cuda:0")
            r = p.eigs(nev, tol=1e-12, maxit=2000, block=block, **kw)
            # tol bounds the backward error relative to the norm bound: each value
            # lies within the residual (and the rounding of it) of an eigenvalue
            near = np.abs(r.evals[:, None] - ref[None, :]).min(axis=1)
            assert r.converged == nev
            assert np.all(near <= 2e-12 * hn), near
            X = r.evecs.cpu().numpy().T
            assert np.allclose(X.conj().T @ X, np.eye(nev), atol=1e-10)
            res = np.linalg.norm(H @ X - X * r.evals, axis=0)
            assert np.all(res <= 1e-11 * hn), res

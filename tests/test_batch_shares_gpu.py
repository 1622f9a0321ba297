"""Star items of a batch whose steps are longer than one XCD's share (more than
128 tiles, cut into eight parts, the tiles not a multiple of eight), between
small ones that turn their dealing: against each plan's own apply and, for one
of each kind, the oracle's sparse H~ (1e-13 (max Lambda + sum |Vhat|) ||x||)."""

import numpy as np
import pytest
import torch

import oracle as O
import paper_2404_04507_amd as lib
from test_few_modes_gpu import P4, P6, block, star

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["grid", "window"])
@pytest.mark.parametrize("n", [4, 6])
def test_long_steps(n, order):
    if n == 4:   # a tile is one (i0, i1): 132 and 130 of them a step
        probs = [star(P4, [4, 4], [3, 3], seed=1), star(P4, [4, 4], [2, 66], seed=2), star(P4, [3, 6], [4, 5], seed=3),
                 star(P4, [5, 4], [3, 65], seed=4), star(P4, [4, 5], [2, 66], seed=5)]
    else:        # 16 planes of 16 points a tile
        probs = [star(P6, [2, 2, 2], [3, 2, 2], seed=1), star(P6, [2, 2, 2], [2, 66, 2], seed=2),
                 star(P6, [2, 3, 2], [3, 3, 2], seed=3), star(P6, [2, 2, 2], [2, 65, 1], seed=4)]
    plans = [lib.Plan.from_problem(p, order=order) for p in probs]
    big = 1
    with torch.cuda.stream(torch.cuda.Stream()):
        batch = lib.Batch(plans, precision="fp64", graph=False)
        for rep in range(3):
            print(f"case: long steps n={n} {order} rep {rep}", flush=True)
            xs = [None if (i + rep) % 4 == 3 else block(p.N, 1 + (2 * i + 3 * rep) % 5, seed=i) for i, p in enumerate(probs)]
            ys = [None if x is None else torch.full_like(x, float("nan")) for x in xs]
            batch.apply(xs, ys)
            refs = [None if x is None else p.apply(x) for p, x in zip(plans, xs)]
            torch.cuda.synchronize()
            for i, (y, r) in enumerate(zip(ys, refs)):
                assert y is None or torch.equal(y, r), i
            if rep == 0:
                prob, plan = probs[big], plans[big]
                H = O.hamiltonian_sparse(prob.P, prob.d, prob.K, prob.L, prob.modes, prob.vhat, "exact")
                pos = O.kstar_to_position(O.index_shift(plan.indices(), prob.K, prob.L), prob.K, prob.L)
                X, Y = xs[big].cpu().numpy().T, ys[big].cpu().numpy().T
                G = np.empty_like(X)
                G[pos] = X
                err = np.linalg.norm(Y - (H @ G)[pos], axis=0)
                assert np.all(err <= 1e-13 * plan.norm_bound() * np.linalg.norm(X, axis=0))
        batch.close()
    for p in plans:
        p.close()

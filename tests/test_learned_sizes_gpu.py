"""The shell MLP's products at shell counts on the edges of their tiles (16 and
32 rows; 256 values of K per round of a workgroup's waves) and the Rayleigh-Ritz
Grams with and without room for both in one, against the CPU reference.

Tolerances are those of the reference's other checks: the MLP runs in float32
with the same bfloat16-rounded weights (forward 2e-5 relative), its gradient
accumulates over up to S shells of 256-wide layers (2e-3 relative, cosine
0.99999), the loss goes through float64 (1e-5)."""

import numpy as np
import pytest

import oracle.learned_oracle as LO
import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W
from test_learned_gpu import iterate_block, random_params, reference_parts, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,m", [(1, 2), (15, 3), (32, 1), (33, 4), (255, 2), (257, 5), (1024, 17)])
def test_shell_counts(S, m):
    prob = W.c1_1d(lam=1.0, K=8, L=16)
    print(f"case: {S} shells, {m} columns", flush=True)
    H, kin, C, M, shell, amb, X = reference_parts(prob, S)
    net = lib.Learned(shells=S, seed=11)
    with lib.Plan.from_problem(prob, precision="fp64") as plan:
        plan.attach(net)
        shell = np.where(amb, plan.learned_shells(S)[0], shell)
        p = random_params(33, beta=(0.35, 0.45))
        net.set(p)
        layers, beta = LO.unpack(p, round_weights=True)
        O, _ = LO.mlp_forward(layers, X)
        R = W.random_block(plan.N, 3, seed=9)
        ref, _, _ = LO.precond_apply(C, M, shell, O, beta, R)
        T = to_host(plan.learned_forward(to_dev(R)))
        assert np.linalg.norm(T - ref) <= 2e-5 * np.linalg.norm(ref)
        Xb, lam = iterate_block(H, m=m)
        loss_ref, g_ref = LO.rr_loss_and_grad(p, H, C, M, shell, X, Xb, lam, round_weights=True)
        loss, g = plan.learned_grad(to_dev(Xb), lam)
        assert abs(loss - loss_ref) <= 1e-5 * abs(loss_ref)
        g = g.astype(np.float64)
        assert np.linalg.norm(g - g_ref) <= 2e-3 * np.linalg.norm(g_ref)
        assert g @ g_ref >= 0.99999 * np.linalg.norm(g) * np.linalg.norm(g_ref)
    net.close()

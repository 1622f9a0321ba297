"""The learned gradient where the shells' gradients cancel.

With the output layer zero the network's outputs are exactly zero, so the
shells' gradients dO carry no float32 rounding, and the gradient of the output
bias is their plain sum.  Its error is then the rounding of the float32 result,
2^-24 of it, and what the float64 Rayleigh-Ritz steps leave in dO, below 1e-10
of each (the loss of such blocks agrees to 1e-10).  Sums in float32 are off by
up to 2^-24 of sum |dO| a step, some thousand times that bound where sum |dO|
is hundreds of times |sum dO|."""

import numpy as np
import pytest

import oracle.learned_oracle as LO
import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W
from test_learned_gpu import random_params, reference_parts, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lam,K,m", [(0.1, 4, 4), (0.1, 4, 8), (0.35, 5, 2), (2.0, 4, 12)])
def test_output_bias_gradient(lam, K, m, monkeypatch):
    S = 1024
    prob = W.c2_2d(lam=lam, K=K, L=4)
    print(f"case: lambda {lam}, K {K}, {m} columns", flush=True)
    H, kin, C, M, shell, amb, X = reference_parts(prob, S)
    p = random_params(33, beta=(0.35, 0.45))
    lay, _ = LO.layout()
    ow, shp, ob, nb = lay[3]
    p[ow:ow + shp[0] * shp[1]] = 0.0
    p[ob:ob + nb] = 0.0
    rng = np.random.default_rng(3)
    Xb = (rng.standard_normal((prob.N, m)) + 1j * rng.standard_normal((prob.N, m))) / (1.0 + kin)[:, None]
    nu = float(np.abs(prob.vhat).sum())
    lam_m = -0.9 * nu + 0.05 * nu * np.arange(m) / m
    net = lib.Learned(shells=S, seed=11)
    with lib.Plan.from_problem(prob) as plan:
        plan.attach(net)
        net.set(p)
        shell = np.where(amb, plan.learned_shells(S)[0], shell)
        dO = []
        backward = LO.mlp_backward
        monkeypatch.setattr(LO, "mlp_backward", lambda layers, cache, d: dO.append(d) or backward(layers, cache, d))
        _, ref = LO.rr_loss_and_grad(p, H, C, M, shell, X, Xb, lam_m)
        _, g = plan.learned_grad(to_dev(Xb), lam_m)
    net.close()
    total, reach = dO[0].sum(axis=0), np.abs(dO[0]).sum(axis=0)
    assert np.allclose(ref[ob:ob + nb], total)
    err, bound = np.abs(g[ob:ob + nb] - total), 2.0 ** -24 * np.abs(total) + 1e-10 * reach
    assert np.all(err <= bound), (err, bound, reach / np.abs(total))

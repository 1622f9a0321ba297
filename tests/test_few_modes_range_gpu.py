"""The few-mode convolution where the windows' ends come near 2^31: neighbouring
slices' ends have no 32-bit difference there, and the extent (10) does not divide
2^32.  Compared with the transforms on the same plan data; both sum at most a few
dozen products of order one in float64, hence 1e-12."""

import numpy as np
import pytest

import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W
from test_learned_gpu import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["grid", "window"])
def test_ends_near_the_integer_range(order):
    P = np.array([[1.0, 1.3e8 + 0.37]])  # ends from -1.95e9 to 2.08e9
    modes = np.array([[0, 0], [1, 0], [-1, 0], [0, 1], [0, -1], [2, -3], [-2, 3]])
    vhat = np.array([0.5, 1.0, 1.0, 0.7, 0.7, 0.2 + 0.3j, 0.2 - 0.3j])
    prob = W.Problem("far", 1, P, [5], [16], modes, vhat)
    print(f"case: {order}", flush=True)
    X = to_dev(W.random_block(prob.N, 3, seed=4))
    out = []
    for schedule in ("auto", "threepass"):
        with lib.Plan.from_problem(prob, order=order, schedule=schedule) as plan:
            assert abs(plan.indices()[:, 0]).max() > 1.9e9
            plan.profile(True)
            out.append(to_host(plan.conv(X)))
            out.append(to_host(plan.apply(X)))
            assert (plan.profile_read()["fused"]["launches"] > 0) == (schedule == "auto")
    for a, b in zip(out[:2], out[2:]):
        assert np.linalg.norm(a - b) <= 1e-12 * np.linalg.norm(b)

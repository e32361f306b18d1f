"""Two rounds of workgroups where one would leave places empty (plan_rounds in regot.hip): on either side of its rule, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2605_08793_amd import binding as B
from paper_2605_08793_amd import workloads as W
from test_gpu_parity import dev, full_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,rounds", [(1000, 131_500, 2), (999, 131_500, 1), (2001, 90_007, 2), (3001, 59_913, 1)])
def test_fill(n, m, rounds):
    assert B.regot_plan_geometry(n, m, n * m // 100)[2] == rounds
    assert B.regot_plan_geometry(n, m)[2] == 1
    eta = 0.2
    M, a, b, alpha, beta = W.random_small(n, m, seed=n, eta=eta)
    T = oracle.plan_dense(M[:100], alpha[:100], beta, eta)
    full_check(dev(M), M, a, b, alpha, beta, eta, float(np.quantile(T, 0.998)), capacity=n * m // 100, label="rounds")

"""The second stage of the half-steps at the numbers of partial results where it takes another path: one batch per wave
(up to 32 parts), several waves and batches, one part alone; with parts that are empty (nothing but infinite costs)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_08793_amd import binding as B
from paper_2605_08793_amd import workloads as W
from paper_2605_08793_amd.driver import DualPass
from parity_utils import assert_half_step_close

pytestmark = pytest.mark.gpu


# rows = 16 x the parts of a beta half-step while they fit the chip (see regot_plan_geometry)
@pytest.mark.parametrize("parts", [1, 2, 31, 32, 33, 127, 128, 129, 257, 512])
def test_beta_half_step_by_number_of_parts(parts):
    n, m, eta = 16 * parts, 70, 0.05
    assert B.regot_plan_geometry(n, m)[0] == parts
    M, a, b, alpha, beta = W.random_small(n, m, seed=parts, eta=eta)
    if parts > 1:
        M[: n // 2, 3] = np.inf                       # half of a column's parts are empty
        M[:, 5] = np.inf; M[n - 1, 5] = 0.4           # all but the last
        M[n // 3:, 7] = 50.0                          # parts whose maxima lie far apart
    dp = DualPass(n, m)
    out = torch.empty(m, dtype=torch.float64, device="cuda")
    dp.half_step(*(torch.from_numpy(x).cuda() for x in (M, b, alpha, beta)), eta, 1, out)
    torch.cuda.synchronize()
    assert_half_step_close(out.cpu().numpy(), oracle.sinkhorn_half_step(M, b, alpha, beta, eta, 1), eta, f"{parts} parts")


@pytest.mark.parametrize("m", [512 * 32, 512 * 32 + 1, 512 * 140 + 7])
def test_alpha_half_step_by_number_of_panels(m):
    n, eta = 37, 0.05
    M, a, b, alpha, beta = W.random_small(n, m, seed=m, eta=eta)
    M[5, : m // 2] = np.inf
    dp = DualPass(n, m)
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    dp.half_step(*(torch.from_numpy(x).cuda() for x in (M, a, alpha, beta)), eta, 0, out)
    torch.cuda.synchronize()
    assert_half_step_close(out.cpu().numpy(), oracle.sinkhorn_half_step(M, a, alpha, beta, eta, 0), eta, f"m={m}")

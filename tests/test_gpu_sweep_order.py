"""Sweeps whose rows are taken forward and backward in turn (several in a call) and forward alone (one in a call): both
against the oracle, with blocks of rows that do not divide into batches, one member and several, full and partial groups."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_08793_amd import binding as B
from paper_2605_08793_amd import workloads as W
from paper_2605_08793_amd.driver import DualPass
from parity_utils import assert_half_step_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(1031, 1500), (4100, 257), (8209, 1900), (1100, 1921), (283, 4500), (2805, 5760), (71, 61440)])
@pytest.mark.parametrize("sweeps", [3, 4])
def test_one_call_and_several(n, m, sweeps):
    eta = 0.05
    print(f"[sweep order] n={n} m={m} sweeps={sweeps}", flush=True)
    M, a, b, _, beta = W.random_small(n, m, seed=n + m, eta=eta)
    Md, ad, bd = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (M, a, b))
    want = oracle.sinkhorn_sweeps(M, a, b, eta, sweeps, np.zeros(n), beta)
    dp = DualPass(n, m)

    def run(calls):
        al = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
        be = torch.from_numpy(beta.copy()).cuda()
        for count in calls:
            B.regot_sinkhorn_sweeps(Md, ad, bd, al, be, eta, count, workspace=dp.workspace)
        return al.cpu().numpy(), be.cpu().numpy()

    for calls in ([sweeps], [1] * sweeps, [2] + [1] * (sweeps - 2)):
        got, again = run(calls), run(calls)
        assert all(np.array_equal(x, y) for x, y in zip(got, again))
        for g, w, what in zip(got, want, ("alpha", "beta")):
            assert_half_step_close(g, w, eta, f"{calls} {what}")

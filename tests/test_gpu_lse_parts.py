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


def half_step(M, marginal, alpha, beta, eta, which):
    n, m = M.shape
    dp = DualPass(n, m)
    out = torch.zeros(m if which else n, dtype=torch.float64, device="cuda")
    dp.half_step(*(torch.from_numpy(x).cuda() for x in (M, marginal, alpha, beta)), eta, which, out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


# one part and several, of rows and of columns; the last columns by strip workgroups (1060 = 2 x 512 + 36)
@pytest.mark.parametrize("n,m", [(16, 70), (16, 600), (48, 1060), (560, 70), (2100, 1060), (70, 512 * 33 + 5)])
def test_a_nan_comes_out_where_it_contributes(n, m):
    eta = 0.05
    M, a, b, alpha, beta = W.random_small(n, m, seed=n + m, eta=eta)
    for i, j in ((0, 0), (n // 2, m - 1), (n - 1, m // 3)):
        X = M.copy()
        X[i, j] = np.nan
        for which, marginal, at in ((0, a, i), (1, b, j)):
            got, ref = half_step(X, marginal, alpha, beta, eta, which), oracle.sinkhorn_half_step(X, marginal, alpha, beta, eta, which)
            bad = np.arange(len(ref)) == at
            assert np.array_equal(np.isnan(ref), bad) and np.array_equal(np.isnan(got), bad), (which, i, j)
            assert_half_step_close(got[~bad], ref[~bad], eta, f"which={which} NaN at {i},{j}")


def test_a_nan_and_an_empty_row_in_small_sweeps():
    # (fewer than 2^20 entries: the half-steps one after the other)
    n, m, eta = 900, 1000, 0.05
    M, a, b, alpha, beta = W.random_small(n, m, seed=5, eta=eta)
    for bad in (np.nan, np.inf):
        X = M.copy()
        X[411, 17 if bad != np.inf else slice(None)] = bad
        dp = DualPass(n, m)
        al, be = (torch.from_numpy(x.copy()).cuda() for x in (alpha, beta))
        dp.sinkhorn_sweeps(*(torch.from_numpy(x).cuda() for x in (X, a, b)), eta, 1, al, be)
        torch.cuda.synchronize()
        al, be = al.cpu().numpy(), be.cpu().numpy()
        keep = np.arange(n) != 411
        assert_half_step_close(al[keep], oracle.sinkhorn_half_step(M, a, alpha, beta, eta, 0)[keep], eta, "rows without it")
        assert not np.isfinite(al[411]) and np.isnan(be).all()


@pytest.mark.parametrize("far", [1e30, 1e120, 1e300])
@pytest.mark.parametrize("n,m", [(48, 1060), (2100, 1060), (70, 512 * 33 + 5)])
def test_parts_any_distance_apart(n, m, far):
    """Parts that hold nothing but very large finite costs beside ordinary ones, in the merges of waves, strips and parts."""
    eta = 0.05
    M, a, b, alpha, beta = W.random_small(n, m, seed=n * m, eta=eta)
    M[:, : m // 2] = far; M[0, 3] = 0.2
    for which, marginal in ((0, a), (1, b)):
        X = M if which == 0 else np.ascontiguousarray(M[:, ::-1])
        if which:
            X[: n // 2, m // 3:] = far; X[n - 1] = 0.5
        ref = oracle.sinkhorn_half_step(X, marginal, alpha, beta, eta, which)
        assert np.isfinite(ref).all()
        assert_half_step_close(half_step(X, marginal, alpha, beta, eta, which), ref, eta, f"which={which} far={far}")

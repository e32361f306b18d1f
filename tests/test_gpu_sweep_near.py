"""The sweeps of a call behind its first one, whose terms are plan entries at the old alpha (csrc/regot_sweep_near.hpp): blocks of
rows on either side of where they begin, any rest of a round of batches, one member to sixteen; masses for which the maxima have to be found
after all; sums that come out where no bound holds."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_08793_amd import binding as B
from paper_2605_08793_amd import workloads as W
from paper_2605_08793_amd.driver import DualPass
from parity_utils import assert_half_step_close

pytestmark = pytest.mark.gpu


def found_maxima(dp, sweeps):
    """Whether the last sweep of a call of several was told to find its rows' maxima: ints 50 and 51 of the workspace (HDR_SWEEP_FAR), by parity
    of the sweep, are what the kernel that forms beta says to the next one."""
    return dp.workspace[:256].view(torch.int32)[50 + (sweeps - 1) % 2].item() != 0


def check(M, a, b, eta, sweeps, beta0, label, maxima=None):
    """maxima: whether the last sweep has to find them, or None where that is not what is tested"""
    n, m = M.shape
    print(f"[sweep near] {label} n={n} m={m} eta={eta} sweeps={sweeps}", flush=True)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    Md, ad, bd = dev(M), dev(a), dev(b)
    dp = DualPass(n, m)
    dp.workspace.fill_(0x5A)
    out = []
    for looks in (None, 0):     # the second time the members that are not there at the first look are done without
        al, be = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda"), dev(beta0)
        if looks is not None:
            B.regot_sweep_patience(looks)
        B.regot_sinkhorn_sweeps(Md, ad, bd, al, be, eta, sweeps, workspace=dp.workspace)
        out.append((al.cpu().numpy(), be.cpu().numpy()))
        assert maxima is None or found_maxima(dp, sweeps) == maxima, label
    assert all(np.array_equal(x, y, equal_nan=True) for x, y in zip(*out))
    for got, ref, what in zip(out[0], oracle.sinkhorn_sweeps(M, a, b, eta, sweeps, np.zeros(n), beta0), ("alpha", "beta")):
        some = np.isfinite(ref)
        np.testing.assert_array_equal(got[~some], ref[~some], err_msg=what)
        assert_half_step_close(got[some], ref[some], eta, f"{label} {what}")


@pytest.mark.parametrize("n,m", [
    (2048, 600), (2049, 600), (2310, 1919), (3000, 1920),          # one member, one group of columns a wave: 8 rows a block, 9 and 10, 11, 12
    (2049, 1921), (2900, 3839), (4097, 2500),                      # one member, two groups
    (1025, 3841), (1420, 7680), (145, 61440),                      # two, two and sixteen members
    (8193, 300), (9000, 1920), (9473, 1901), (9729, 640),          # batches in rounds of four, one member: 33, 36, 38 and 39 rows a block
    (2805, 5760), (3145, 5001), (1700, 9599), (2005, 8000),        # three and five members
])
def test_blocks_of_rows(n, m):
    eta = 0.05
    M, a, b, _, beta = W.random_small(n, m, seed=n + m, eta=eta)
    near = None if (n, m) == (2048, 600) else False     # (blocks of 8 rows: nobody asks)
    for sweeps in (2, 3):
        check(M, a, b, eta, sweeps, beta, "plain", near)
    M[n // 2:, m // 3] = np.inf
    M[5, : m // 2] = np.inf
    a[::17] = 0.0
    b[m // 4: m // 4 + 64] = 0.0
    # (from -inf where there is no mass, so that the second sweep need not find the maxima)
    check(M, a / a.sum(), b / b.sum(), eta, 4, np.where(b == 0.0, -np.inf, beta), "infinite costs, no mass", near)


@pytest.mark.parametrize("what", ["small a", "small b", "large b", "no mass in a column", "ratio", "large a"])
def test_masses_that_need_the_maxima(what):
    n, m, eta = 3001, 700, 0.01
    M, a, b, _, beta = W.random_small(n, m, seed=5, eta=eta)
    if what == "small a": a[7] = 1e-200
    if what == "small b": b[7] = 1e-200
    if what == "large b": b[7] = 1e150
    if what == "no mass in a column": b[7: 90] = 0.0; beta[:] = 0.0
    if what == "ratio": b[7] = 1e-30
    if what == "large a": a[7] = 1e14
    check(M, a, b, eta, 2, beta, what, True)
    check(M, a, b, eta, 3, beta, what)


def test_duals_that_eta_is_small_against():
    """eta far below the rounding errors of the duals.  They are held to what a few of those are (the costs are of order 1)."""
    n, sweeps = 2560, 3
    rng = np.random.default_rng(3)
    u, v = rng.random(n), rng.random(n)
    M = u[:, None] + v[None, :] + (1.0 - np.eye(n))
    a = rng.random(n) + 0.1
    a /= a.sum()
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    Md, ad = dev(M), dev(a)
    for eta in (1e-19, 1e-17, 1e-15):
        for beta0 in (np.zeros(n), v, v + 1e-16 * rng.standard_normal(n)):
            dp, al, be = DualPass(n, n), torch.zeros(n, dtype=torch.float64, device="cuda"), dev(beta0)
            B.regot_sinkhorn_sweeps(Md, ad, ad, al, be, eta, sweeps, workspace=dp.workspace)
            assert found_maxima(dp, sweeps)
            ra, rb = oracle.sinkhorn_sweeps(M, a, a, eta, sweeps, np.zeros(n), beta0)
            assert np.abs(al.cpu().numpy() - ra).max() <= 2e-15 and np.abs(be.cpu().numpy() - rb).max() <= 2e-15, eta


@pytest.mark.parametrize("n,m,sweeps", [(3001, 700, 2), (3001, 700, 3), (600, 20000, 2), (4097, 2500, 4)])   # rows of a column shared by three workgroups, by one, by five
def test_no_mass_and_no_cost(n, m, sweeps):
    """A column of mass 0 whose costs are all infinite comes out as NaN (-inf + inf) and takes every alpha of the next sweep with it, those
    of the rows without mass too, whose alpha is -inf otherwise."""
    eta = 0.05
    M, a, b, _, beta = W.random_small(n, m, seed=n + m, eta=eta)
    M[:, m // 2] = np.inf
    a[::17] = 0.0
    b[m // 2] = 0.0
    beta[m // 2] = -np.inf
    check(M, a / a.sum(), b / b.sum(), eta, sweeps, beta, "no mass, no cost", True)

"""Sweeps that read M once (regot_sinkhorn_sweeps for n * m >= 2^20) against the oracle's sweeps and against the
half-steps, at the edges of the cut: one member and several, groups of columns that are full, partial and absent, blocks
of rows that do not divide into batches, matrices whose rows do not start at 16-byte boundaries."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_08793_amd import binding as B
from paper_2605_08793_amd import workloads as W
from paper_2605_08793_amd.driver import DualPass
from parity_utils import assert_half_step_close

pytestmark = pytest.mark.gpu
INF = float("inf")


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def sweep_gpu(Md, a, b, eta, sweeps, beta0, dirty=True):
    n, m = Md.shape
    dp = DualPass(n, m)
    if dirty:
        dp.workspace.fill_(0x5A)
    al = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    be = dev(beta0)
    B.regot_sinkhorn_sweeps(Md, dev(a), dev(b), al, be, eta, sweeps, workspace=dp.workspace)
    torch.cuda.synchronize()
    return al.cpu().numpy(), be.cpu().numpy()


def check(M, a, b, eta, sweeps, beta0, label, Md=None):
    n, m = M.shape
    print(f"[sweep] {label} n={n} m={m} eta={eta} sweeps={sweeps}", flush=True)
    assert n * m >= 1 << 20
    got_a, got_b = sweep_gpu(dev(M) if Md is None else Md, a, b, eta, sweeps, beta0)
    ra, rb = oracle.sinkhorn_sweeps(M, a, b, eta, sweeps, np.zeros(n), beta0)
    # every half-step is within 1e-10 * max(|dual|, eta) of the oracle's (parity_utils); the error of one enters the next
    # with a factor of at most 1 (a log-sum-exp does not magnify), so a few sweeps stay within a few of those
    zero_a, zero_b = ~np.isfinite(ra), ~np.isfinite(rb)
    for got, ref, zero, what in ((got_a, ra, zero_a, "alpha"), (got_b, rb, zero_b, "beta")):
        np.testing.assert_array_equal(got[zero], ref[zero], err_msg=what)
        assert_half_step_close(got[~zero], ref[~zero], eta, f"{label} {what}")
    return got_a, got_b


@pytest.mark.parametrize("n,m", [
    (4096, 256), (16384, 64), (64, 16385),        # few columns; the fewest of either
    (1100, 1920), (1101, 1921),                   # the last width with one group of columns a wave, and one more
    (300, 3840), (301, 3841), (283, 3839),        # one member, full; two members
    (200, 7680), (191, 7681), (137, 11000),       # two, three
    (71, 61440),                                  # sixteen members
    (1031, 1500), (2049, 513), (3001, 1111),      # rows that do not divide into batches
])
def test_edges_of_the_cut(n, m):
    eta = 0.05
    M, a, b, _, beta = W.random_small(n, m, seed=n + m, eta=eta)
    check(M, a, b, eta, 2, beta, "edges")


@pytest.mark.parametrize("n,m,ld,shift", [(1200, 1000, 1001, 0), (1200, 1000, 1000, 1), (600, 3841, 3845, 1)])
def test_rows_off_16_byte_boundaries(n, m, ld, shift):
    eta = 0.05
    M, a, b, _, beta = W.random_small(n, m, seed=7, eta=eta)
    store = torch.full((n * ld + shift,), float("nan"), dtype=torch.float64, device="cuda")
    Md = store[shift:].as_strided((n, m), (ld, 1), storage_offset=shift)
    Md.copy_(dev(M))
    # (what lies between the rows and around them is NaN: a read there must not enter a result)
    check(M, a, b, eta, 2, beta, "unaligned", Md=Md)


@pytest.mark.parametrize("n,m", [(1100, 1300), (300, 4500)])
def test_infinite_costs_zero_masses_and_underflow(n, m):
    rng = np.random.default_rng(m)
    M, a, b, _, beta = W.random_small(n, m, seed=m, eta=0.05)
    # infinite costs, among them whole segments of rows, nearly whole rows and columns
    Mi = M.copy()
    Mi[rng.random((n, m)) < 0.02] = INF
    Mi[3, : m // 2] = INF
    Mi[7, :] = INF; Mi[7, m // 3] = 0.3
    Mi[:, 9] = INF; Mi[n - 1, 9] = 0.1
    Mi[n // 2:, m - 1] = INF
    check(Mi, a, b, 0.05, 2, beta, "infinite costs")
    # zero masses: the dual is -inf, and stays it in later sweeps
    az, bz = a.copy(), b.copy()
    az[::17] = 0.0; bz[::13] = 0.0; bz[m - 1] = 0.0
    check(Mi, az / az.sum(), bz / bz.sum(), 0.05, 3, beta, "zero masses")
    # a start from -inf in columns that have mass; columns whose every term underflows at the old beta
    check(M, a, b, 0.05, 2, np.where(np.arange(m) % 5 == 0, -INF, beta), "beta starts at -inf")
    check(M, a, b, 1e-4, 2, np.where(np.arange(m) % 7 == 0, -3.0, beta), "underflow at the old beta")
    check(M, a, b, 2e-4, 2, np.zeros(m), "small eta from zero")


def test_nan_and_empty_rows_come_back():
    n, m, eta = 1100, 1000, 0.05
    M, a, b, _, beta = W.random_small(n, m, seed=3, eta=eta)
    for bad in (float("nan"), INF):
        X = M.copy()
        X[411, 17 if bad != INF else slice(None)] = bad
        al, be = sweep_gpu(dev(X), a, b, eta, 1, beta)
        keep = np.arange(n) != 411
        ref = oracle.sinkhorn_half_step(M, a, np.zeros(n), beta, eta, 0)
        assert_half_step_close(al[keep], ref[keep], eta, "rows without it")
        assert not np.isfinite(al[411]) and np.isnan(be).all()


def test_same_bits_again_and_in_a_graph():
    p = W.make_problem("c2", device="cuda", n=1500, m=4100)      # two members to a cluster
    dp = DualPass(p.n, p.m)
    al = torch.zeros(p.n, dtype=torch.float64, device="cuda"); be = torch.zeros(p.m, dtype=torch.float64, device="cuda")

    def run():
        B.regot_sinkhorn_sweeps(p.M, p.a, p.b, al, be, p.eta, 3, workspace=dp.workspace)

    run(); torch.cuda.synchronize()
    first = (al.clone(), be.clone())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for replay in range(3):
        be.zero_(); al.fill_(float("nan"))
        graph.replay(); torch.cuda.synchronize()
        assert torch.equal(al, first[0]) and torch.equal(be, first[1]), replay
        be.zero_(); dp.workspace.fill_(replay)
        run(); torch.cuda.synchronize()
        assert torch.equal(al, first[0]) and torch.equal(be, first[1]), replay
    # two streams at once, each with its own workspace: the clusters of both complete
    side, dp2 = torch.cuda.Stream(), DualPass(p.n, p.m)
    al2, be2 = torch.zeros_like(al), torch.zeros_like(be)
    be.zero_(); torch.cuda.synchronize()
    for _ in range(5):
        with torch.cuda.stream(side):
            be2.zero_()
            B.regot_sinkhorn_sweeps(p.M, p.a, p.b, al2, be2, p.eta, 3, workspace=dp2.workspace)
        be.zero_(); run()
    torch.cuda.synchronize()
    assert torch.equal(al, first[0]) and torch.equal(be, first[1])
    assert torch.equal(al2, first[0]) and torch.equal(be2, first[1])


@pytest.mark.parametrize("n,m,shift", [
    (8191, 257, 0), (8192, 257, 1), (8449, 1920, 0), (10241, 1919, 1),    # one member: either side of the rule; 33 rows
    (2719, 3841, 0), (2720, 3841, 1), (2805, 5760, 0), (3001, 5759, 1),   # three members, and the two below the rule
    (1631, 7681, 0), (1632, 7682, 0), (1700, 9599, 1), (1640, 9601, 0),   # five members; three of two groups again
])
def test_batches_of_eight_rows(n, m, shift):
    """Blocks of at least 32 rows in one, three or five members: batches of eight rows, an even or an odd number of them."""
    eta = 0.05
    M, a, b, _, beta = W.random_small(n, m, seed=n + m, eta=eta)
    if shift:  # also infinite costs: a segment of a row, a column but for its last entry, single entries
        M[5, : m // 2] = INF
        M[:-1, 7] = INF
        M[np.arange(0, n, 3), np.arange(0, n, 3) * 13 % (m - 64) + 64] = INF
    store = torch.full((n * m + shift,), float("nan"), dtype=torch.float64, device="cuda")
    Md = store[shift:].view(n, m)
    Md.copy_(dev(M))
    got = check(M, a, b, eta, 2, beta, "eight rows", Md=Md)
    again = sweep_gpu(Md, a, b, eta, 2, beta, dirty=False)
    assert all(np.isfinite(x).all() and np.array_equal(x, y) for x, y in zip(got, again))


# the rows of 64 columns in one workgroup's hands (1100), and shared by 3, 2, 4, 10 and 2 of them where they are done again
@pytest.mark.parametrize("n,m", [(1100, 1300), (2113, 1000), (2050, 4500), (4097, 300), (9217, 1300), (5003, 7690)])
def test_columns_that_are_done_again(n, m):
    """Columns without mass next to each other and at the end, columns far below the others, columns without a finite
    cost, a start from -inf: sums that say nothing, so that sweep_finalize_kernel goes back to alpha and M."""
    eta = 1e-3
    rng = np.random.default_rng(n)
    M, a, b, _, beta = W.random_small(n, m, seed=n * m, eta=eta)
    bz = b.copy()
    bz[m // 4: m // 2] = 0.0; bz[m - 70:] = 0.0; bz[::11] = 0.0; bz[3] = 0.5
    check(M, a, bz / bz.sum(), eta, 3, beta, "blocks without mass")
    Mi = M.copy()
    Mi[n // 3:, m // 3] = INF; Mi[: n - 1, m // 3 + 1] = INF      # one without mass whose only finite cost is the last row's
    check(Mi, a, bz / bz.sum(), eta, 3, beta, "blocks without mass, infinite costs")
    check(M, a, b, eta, 1, np.where(rng.random(m) < 0.3, -3.0, beta), "far below")
    check(M, a, b, eta, 2, np.where(np.arange(m) < m // 2, -INF, beta), "from -inf")
    x = rng.standard_normal((n, 10)); y = rng.standard_normal((m, 10)) + 0.5
    far = (x * x).sum(1)[:, None] + (y * y).sum(1) - 2 * x @ y.T
    far = np.ascontiguousarray(np.maximum(far, 0) / far.max())
    for small in (1e-4, 2e-5):                                    # Gaussian clouds from zero
        check(far, a, b, small, 2, np.zeros(m), f"clouds eta={small}")


def test_a_column_without_a_finite_cost():
    n, m, eta = 2113, 1000, 0.05
    M, a, b, _, beta = W.random_small(n, m, seed=3, eta=eta)
    M[:, 500] = INF; M[:, 501] = INF
    b[501] = 0.0; b /= b.sum()
    al, be = sweep_gpu(dev(M), a, b, eta, 1, beta)
    ra, rb = oracle.sinkhorn_sweeps(M, a, b, eta, 1, np.zeros(n), beta)
    keep = (np.arange(m) != 500) & (np.arange(m) != 501)
    assert not np.isfinite(be[500]) and np.isnan(be[501]) and np.isnan(rb[~keep]).all()
    assert_half_step_close(al, ra, eta, "alpha"); assert_half_step_close(be[keep], rb[keep], eta, "beta")


# one, two and five members; batches of four and of eight rows, an even and an odd number of them
@pytest.mark.parametrize("n,m", [(1200, 1000), (283, 4500), (8449, 1920), (10241, 1919), (2805, 5760), (1700, 9599)])
def test_infinite_terms_met_on_the_way(n, m):
    """A wave puts a floor under its terms once it has met an infinite one: at the first row of a block, at the last, in
    some waves and not in others, with large finite costs among them; the results do not depend on it."""
    eta = 0.02
    M, a, b, _, beta = W.random_small(n, m, seed=m, eta=eta)
    clean = check(M, a, b, eta, 1, beta, "none")
    X = M.copy()
    X[n - 1, m - 1] = INF; X[n // 2 + 1, m // 2] = INF; X[0, 0] = INF
    got = check(X, a, b, eta, 1, beta, "three")
    same = np.ones(n, bool); same[[0, n // 2 + 1, n - 1]] = False
    assert np.array_equal(got[0][same], clean[0][same])          # rows behind the first one met: bit for bit
    X[np.arange(n)[:, None] * m // n < np.arange(m)[None, :] - m // 3] = INF
    X[:, 5] = 1e30; X[7, m // 4: m // 2] = 1e30; X[n // 3, : m // 2] = INF
    bz = b.copy(); bz[m // 5: m // 5 + 200] = 0.0; bz[::97] = 0.0
    check(X, a, bz / bz.sum(), eta, 3, beta, "band, large costs, columns without mass")


# two, three, five (batches of eight rows) and sixteen members; two of two groups of columns a wave
@pytest.mark.parametrize("n,m", [(283, 4500), (2805, 5760), (1700, 9599), (71, 61440), (150, 7680)])
def test_members_that_are_done_without(n, m):
    """A workgroup that does not find another's numbers for a row computes them: at the first look, at the second, never.
    The bits are the same, with infinite costs and columns without mass too."""
    eta = 0.05
    M, a, b, _, beta = W.random_small(n, m, seed=m + 1, eta=eta)
    M[n // 2:, m // 3: m // 2] = INF; M[3, :] = INF; M[3, m - 2] = 0.4
    b[m // 4: m // 4 + 300] = 0.0; b /= b.sum()
    want = check(M, a, b, eta, 2, beta, "never")
    Md = dev(M)
    for looks in (0, 1):
        B.regot_sweep_patience(looks)
        got = sweep_gpu(Md, a, b, eta, 2, beta)
        assert all(np.array_equal(x, y) for x, y in zip(got, want)), looks
    got = sweep_gpu(Md, a, b, eta, 2, beta)          # (the request held for one call)
    assert all(np.array_equal(x, y) for x, y in zip(got, want))


# either side of what the single read is used for: 2^20 entries, 64 rows, 64 and 61440 columns, tall narrow matrices
@pytest.mark.parametrize("n,m,halves", [
    (1024, 1023, True), (1024, 1024, False), (63, 17000, True), (64, 17000, False), (17000, 63, True), (17000, 64, False),
    (64, 61441, True), (64, 61439, False), (20000, 128, True), (19999, 128, False), (20000, 129, False),
    (37000, 256, True), (36999, 255, False), (37000, 257, False), (90000, 257, True), (20001, 70, True),
])
def test_which_sweeps_are_the_half_steps(n, m, halves):
    eta, sweeps = 0.05, 2
    M, a, b, _, beta = W.random_small(n, m, seed=n + 3 * m, eta=eta)
    Md, ad, bd = dev(M), dev(a), dev(b)
    got = sweep_gpu(Md, a, b, eta, sweeps, beta)
    dp = DualPass(n, m)
    al, be = torch.zeros(n, dtype=torch.float64, device="cuda"), dev(beta)
    for _ in range(sweeps):
        dp.half_step(Md, ad, al, be, eta, 0, al)
        dp.half_step(Md, bd, al, be, eta, 1, be)
    torch.cuda.synchronize()
    want = (al.cpu().numpy(), be.cpu().numpy())
    assert all(np.array_equal(x, y) for x, y in zip(got, want)) == halves
    for x, y, what in zip(got, want, ("alpha", "beta")):
        assert_half_step_close(x, y, eta, f"{what} n={n} m={m}")


@pytest.mark.parametrize("n,m", [(1100, 1000), (2113, 1000), (283, 4500)])
@pytest.mark.parametrize("big", [1e9, 1e20, 1e60, 1e300])
def test_masses_far_from_one(n, m, big):
    """Marginals need not sum to 1: a column whose sum looks fine although what underflowed in the rows of large mass is
    far more than what is there, sums that overflow, and very small masses."""
    eta = 1e-3
    M, a, b, _, beta = W.random_small(n, m, seed=n, eta=eta)
    M *= 0.1; beta *= 0.0
    a = a * n * big
    a[0] = 1e-270                                      # one row of next to no mass ...
    M[1:, 17] = 0.7465 + 1e-4 * M[1:, 17]; M[0, 17] = 0.0   # ... has nearly all of what can be seen of column 17
    check(M, a, b, eta, 1, beta, f"mass {big}")
    check(M, a, b * m * big, eta, 3, beta, f"mass {big}, three sweeps")
    check(M, np.full(n, 1e-290), np.full(m, 1e-300), eta, 2, beta, "small masses")

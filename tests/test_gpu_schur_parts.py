"""The reduced solve's half products where their cut into parts, slices and trips can go wrong: rows over many slices and
trips, many and empty rows in a part, several rows in a lane, vectors at and beyond what the LDS holds, ends of the arrays.
Against the oracle's reduced iteration and, for the residual, its product."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_08793_amd import binding as B
from paper_2605_08793_amd.driver import DirectionSolver, SparseTerm

pytestmark = pytest.mark.gpu


def pattern(rng, n, m, lengths):
    """CSR with lengths[i] different random columns in row i."""
    cols = [np.sort(rng.choice(m, size=k, replace=False)) for k in lengths]
    row_ptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    return row_ptr, np.concatenate(cols).astype(np.int32) if row_ptr[-1] else np.zeros(0, np.int32)


CASES = {
    "rows of many trips": (3, 40000, lambda rng, n, m: np.array([m, 8193, 20000])),
    "columns of many trips": (30000, 4, lambda rng, n, m: rng.integers(2, 5, n)),
    "mostly empty rows": (70000, 50, lambda rng, n, m: np.where(rng.random(n) < 0.1, rng.integers(1, 40, n), 0)),
    "one entry a row": (5000, 300, lambda rng, n, m: np.ones(n, int)),
    "whole slices": (1024, 2000, lambda rng, n, m: np.full(n, 256)),
    "whole lanes, long and short": (700, 9000, lambda rng, n, m: np.where(np.arange(n) % 100 == 0, 4096, 4)),
    "odd ends": (1001, 777, lambda rng, n, m: rng.integers(0, 8, n) * 2 + 1),
    "as long as the LDS holds": (20000, 20001, lambda rng, n, m: rng.integers(0, 9, n)),
    "one longer": (19999, 20002, lambda rng, n, m: rng.integers(0, 9, n)),
    "both longer": (20001, 20002, lambda rng, n, m: rng.integers(0, 9, n)),
    "one row": (1, 700, lambda rng, n, m: np.array([650])),
    "one column": (500, 1, lambda rng, n, m: rng.integers(0, 2, n)),
    "no entries": (40, 30, lambda rng, n, m: np.zeros(n, int)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_half_products(name):
    n, m, lengths = CASES[name]
    rng = np.random.default_rng(len(name) + n)
    row_ptr, col_idx = pattern(rng, n, m, lengths(rng, n, m))
    nnz = int(row_ptr[-1])
    val = rng.random(nnz) / max(nnz, 1)
    rows = np.repeat(np.arange(n), np.diff(row_ptr))
    # sums of a plan of which the pattern holds about three quarters
    r = np.bincount(rows, val, n) * 1.3 + 0.1 / n
    c = np.bincount(col_idx, val, m) * 1.3 + 0.1 / m
    eta, tau, rtol = 0.05, 1e-3, 1e-9
    N = n + m - 1
    rhs = [rng.standard_normal(N) / N, rng.standard_normal(N) * np.exp(2 * rng.standard_normal(N)) / N]

    def dev(x):
        return torch.from_numpy(np.ascontiguousarray(x)).cuda()

    term = SparseTerm(n, m, dev(row_ptr), dev(col_idx), nnz)
    if nnz:
        term.val[:] = dev(val)
        term.val_csc[term.csc_pos] = term.val
    solver = DirectionSolver(term)
    rd, cd = dev(r), dev(c)
    x, out = [], []
    for g in rhs:
        print(f"[schur] {name} n={n} m={m} nnz={nnz}", flush=True)
        xs = torch.full((N,), float("nan"), dtype=torch.float64, device="cuda")
        its, conv, rel = solver.solve(eta, tau, rd, cd, dev(g), xs, rtol=rtol, portion=7, reduced=True)
        o_x, o_its, _ = oracle.pcg_solve_reduced(n, m, eta, tau, row_ptr, col_idx, val, r, c, g, rtol=rtol, max_iter=1000)
        assert conv and abs(its - o_its) <= 1, (its, o_its)
        got = xs.cpu().numpy()
        res = np.linalg.norm(oracle.hessian_matvec(n, m, eta, tau, row_ptr, col_idx, val, r, c, got) - g) / np.linalg.norm(g)
        assert res <= 1.5 * rtol + 1e-13, res
        # the same recurrences on products that agree to rounding
        if its == o_its:
            assert np.linalg.norm(got - o_x) <= 1e-10 * np.linalg.norm(o_x)
        x.append(xs)
        out.append((its, conv, rel))
    # a pair gives the bits of two single solves, whatever the portions
    for portion in (16, 2):
        xa, xb = torch.empty_like(x[0]), torch.empty_like(x[0])
        pair = solver.solve2(eta, tau, rd, cd, dev(rhs[0]), dev(rhs[1]), xa, xb, rtol=rtol, portion=portion, reduced=True)
        assert list(pair) == out
        assert torch.equal(xa, x[0]) and torch.equal(xb, x[1])


@pytest.mark.parametrize("n,m", [(700, 900), (3, 21000), (21000, 3)])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_arrays_at_multiples_of_their_elements_only(n, m, shift):
    """Columns and rows at multiples of 4 bytes, everything else at multiples of 8: the same bits as at multiples of 256."""
    rng = np.random.default_rng(n)
    row_ptr, col_idx = pattern(rng, n, m, rng.integers(m // 3, m // 2 + 2, n) if m > n else rng.integers(0, min(m, 300), n))
    nnz = len(col_idx)
    val = rng.random(nnz) / nnz
    rows = np.repeat(np.arange(n), np.diff(row_ptr))
    r, c = np.bincount(rows, val, n) * 1.1 + 0.1 / n, np.bincount(col_idx, val, m) * 1.1 + 0.1 / m
    N = n + m - 1
    rhs = rng.standard_normal((2, N)) / N
    print(f"[schur aligned] n={n} m={m} nnz={nnz} shift={shift}", flush=True)

    def dev(x, off=0):
        x = torch.from_numpy(np.ascontiguousarray(x))
        store = torch.zeros(x.numel() + off, dtype=x.dtype, device="cuda")
        store[off:].copy_(x)
        assert store[off:].data_ptr() % 256 == off * x.element_size()
        return store[off:]

    term = SparseTerm(n, m, dev(row_ptr), dev(col_idx), nnz)
    term.val[:] = dev(val)
    term.val_csc[term.csc_pos] = term.val
    arrays = [t.cpu().numpy() for t in (term.row_ptr, term.col_idx, term.val, term.col_ptr, term.row_idx, term.val_csc)]
    workspace = torch.empty(B.regot_pcg_workspace_bytes(n, m), dtype=torch.uint8, device="cuda")

    def solve(off):
        pat, (rd, cd), g = [dev(a, off) for a in arrays], [dev(a, off) for a in (r, c)], [dev(a, off) for a in rhs]
        x, info = [dev(np.full(N, np.nan), off) for _ in range(3)], dev(np.zeros(12), off)
        B.regot_pcg_solve_reduced(n, m, 0.05, 1e-3, *pat, rd, cd, g[0], x[0], 1e-10, 40, True, info[:4], workspace=workspace)
        B.regot_pcg_solve2_reduced(n, m, 0.05, 1e-3, *pat, rd, cd, *g, *x[1:], 1e-10, 40, True, info[4:], workspace=workspace)
        return x + [info]

    for got, want in zip(solve(shift), solve(0)):
        assert torch.equal(got, want) and torch.isfinite(got).all()
    assert torch.equal(got[:8], torch.cat([got[:4]] * 2))

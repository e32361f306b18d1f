"""Values, columns and lower triangle of stored patterns where the tiles of consecutive entries meet rows in all ways: many rows and
rows without entries in a tile, rows over many tiles, few and many entries, last columns dropped; against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_08793_amd import workloads as W
from paper_2605_08793_amd.driver import SparseTerm

pytestmark = pytest.mark.gpu

# (n, m, lengths of the rows): a tile is 512 entries below 393216 of them and 1024 from there on; by rows instead with at most
# 6144 rows, 8192 columns, 96 entries to a row on average and 262144 of them, 256 of a row by its wave, the others by four waves
CASES = {
    "more empty rows than are held": (150000, 8, lambda rng, n, m: np.where(rng.random(n) < 0.01, m, 0)),
    "only the last row": (70000, 9, lambda rng, n, m: np.where(np.arange(n) == n - 1, m, 0)),
    "only the first row": (70000, 9, lambda rng, n, m: np.where(np.arange(n) == 0, m, 0)),
    "one entry a row": (40000, 5, lambda rng, n, m: np.ones(n, int)),
    "whole tiles": (64, 2048, lambda rng, n, m: np.full(n, m // 2)),
    "long and empty rows, many entries": (3000, 400, lambda rng, n, m: np.where(np.arange(n) % 2 == 0, m - 1, rng.integers(0, 3, n))),
    "short rows, many entries": (200000, 6, lambda rng, n, m: rng.integers(2, m + 1, n)),
    "by rows: ends of trips": (1001, 1300, lambda rng, n, m: np.where(np.arange(n) % 25 == 3, np.resize([255, 256, 257, 1279, 1280, 1281, 1300], n), rng.integers(0, 4, n))),
    "by rows: all of a workgroup's rows long": (400, 8192, lambda rng, n, m: np.where(np.arange(n) % 100 == 99, m, 0)),
    "by rows: fewer rows than waves": (3, 700, lambda rng, n, m: np.array([96, 0, 190])),
    "by rows: as many as there may be": (6144, 300, lambda rng, n, m: np.resize([42, 43], n)),
    "one row more": (6145, 300, lambda rng, n, m: np.resize([42, 43], n)),
    "one column more": (500, 8193, lambda rng, n, m: rng.integers(0, 97, n)),
    "one entry more to a row": (1000, 300, lambda rng, n, m: np.where(np.arange(n) == 5, 97, 96)),
    "large tiles just": (3000, 200, lambda rng, n, m: np.where(np.arange(n) < 216, 132, 131)),
    "large tiles not yet": (3000, 200, lambda rng, n, m: np.where(np.arange(n) < 215, 132, 131)),
    "many entries in few rows": (50000, 30, lambda rng, n, m: np.where((np.arange(n) > 20000) & (np.arange(n) < 42000), m, 0)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_tiles(name):
    n, m, lengths = CASES[name]
    rng = np.random.default_rng(n + m)
    eta, tau = 0.3, 1e-3
    M, a, b, alpha, beta = W.random_small(n, m, seed=n + m, eta=eta)
    keep = np.asarray(lengths(rng, n, m))
    # the columns of a row: its `keep` first ones in a random order of the row
    chosen = np.argsort(np.argsort(rng.random((n, m)), axis=1), axis=1) < keep[:, None]
    rows, cols = np.nonzero(chosen)
    rp = np.concatenate([[0], np.cumsum(keep)]).astype(np.int64)
    ci = cols.astype(np.int32)
    print(f"[tiles] {name} n={n} m={m} nnz={len(ci)}", flush=True)

    def dev(x):
        return torch.from_numpy(np.ascontiguousarray(x)).cuda()

    term = SparseTerm(n, m, dev(rp), dev(ci), len(ci))
    term.refresh(dev(M), dev(alpha), dev(beta), eta)
    cp, ri, pos = oracle.pattern_transpose(n, m, rp, ci)
    np.testing.assert_array_equal(term.col_ptr.cpu().numpy(), cp)
    np.testing.assert_array_equal(term.row_idx.cpu().numpy(), ri)
    np.testing.assert_array_equal(term.csc_pos.cpu().numpy(), pos)
    val = oracle.pattern_values(M, alpha, beta, eta, rp, ci)
    got, got_csc = term.val.cpu().numpy(), term.val_csc.cpu().numpy()
    np.testing.assert_allclose(got, val, rtol=1e-10, atol=0)
    np.testing.assert_array_equal(got_csc[pos], got)
    r, c = np.bincount(rows, val, n) + 0.1, np.bincount(cols, val, m) + 0.1
    hp, hi, hv = oracle.hessian_lower_csc(n, m, eta, tau, rp, ci, val, r, c)
    for _ in range(2):      # with the structure, then the values alone
        term.lower_csc(eta, tau, dev(r), dev(c))
        assert term.h_info.cpu().tolist() == [len(hi), 0]
        np.testing.assert_array_equal(term.h_col_ptr.cpu().numpy(), hp)
        np.testing.assert_array_equal(term.h_row_idx.cpu().numpy()[:len(hi)], hi)
        np.testing.assert_allclose(term.h_val.cpu().numpy()[:len(hi)], hv, rtol=1e-10, atol=0)
        assert not term.h_val[len(hi):].any()
        term.h_val[:len(hi)] = float("nan")

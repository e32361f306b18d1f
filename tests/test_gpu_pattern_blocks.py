"""Stored-pattern kernels at the sizes where their blocks of work are dealt to the dies unevenly: fewer blocks than dies, a
last die with fewer or none, more rows than one trip covers; against the oracle, exactly where it is exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_08793_amd import workloads as W
from paper_2605_08793_amd.driver import DualPass, SparseTerm

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# rows in groups of 4, entries in tiles of 2048 and blocks of 256: n = 1 .. 36 rows are 1 .. 9 groups on 8 dies; the last
# shape has more groups of rows than the grid has workgroups
@pytest.mark.parametrize("n,m,keep", [(1, 300, 40), (3, 300, 255), (4, 300, 256), (5, 300, 257), (31, 90, 2047), (32, 90, 2048),
                                      (33, 90, 2049), (36, 700, 9 * 2048), (37, 700, 17000), (257, 129, 16385), (16900, 40, 60000)])
def test_pattern_values_and_lower_triangle(n, m, keep):
    eta, tau = 0.3, 1e-3
    M, a, b, alpha, beta = W.random_small(n, m, seed=n + m, eta=eta)
    T = oracle.plan_dense(M, alpha, beta, eta)
    delta = float(np.partition(T.ravel(), T.size - keep)[T.size - keep]) * (1 - 1e-9)
    rp, ci, val = oracle.sparsify_csr(M, alpha, beta, eta, delta)
    nnz = int(rp[-1])
    assert nnz == keep
    dp = DualPass(n, m, capacity=nnz + 7)
    dp.dual_eval_sparsify(dev(M), dev(a), dev(b), dev(alpha), dev(beta), eta, delta)
    term = SparseTerm(n, m, dp.row_ptr, dp.col_idx, nnz)
    term.refresh(dev(M), dev(alpha), dev(beta), eta)
    cp, ri, pos = oracle.pattern_transpose(n, m, rp, ci)
    np.testing.assert_array_equal(term.col_ptr.cpu().numpy(), cp)
    np.testing.assert_array_equal(term.row_idx.cpu().numpy(), ri)
    np.testing.assert_array_equal(term.csc_pos.cpu().numpy(), pos)
    got, got_csc = term.val.cpu().numpy(), term.val_csc.cpu().numpy()
    np.testing.assert_allclose(got, val, rtol=1e-10, atol=0)
    np.testing.assert_array_equal(got_csc[pos], got)
    r, c = T.sum(1), T.sum(0)
    term.lower_csc(eta, tau, dev(r), dev(c))
    hp, hi, hv = oracle.hessian_lower_csc(n, m, eta, tau, rp, ci, val, r, c)
    assert term.h_info.cpu().tolist() == [len(hi), 0]
    np.testing.assert_array_equal(term.h_col_ptr.cpu().numpy(), hp)
    np.testing.assert_array_equal(term.h_row_idx.cpu().numpy()[:len(hi)], hi)
    np.testing.assert_allclose(term.h_val.cpu().numpy()[:len(hi)], hv, rtol=1e-10, atol=0)

"""The end of the threshold search (the result kernel selecting among the keys that are left) and the range the sample is
searched over: ties of as many entries as the result kernel takes and one more, pools it reads and larger ones, infinite
and far-off entries.  s_k and both counts against a full sort, exactly."""
import numpy as np
import pytest
import torch

from paper_2605_08793_amd import workloads as W
from paper_2605_08793_amd.driver import PatternRefresh, TopK

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def check(M, alpha, beta, eta, k, label):
    n, m = M.shape
    print(f"[topk finish] {label} n={n} m={m} k={k}", flush=True)
    tk = TopK(n, m, k)
    tk.workspace.fill_(0x77)
    tk.threshold(dev(M), dev(alpha), dev(beta), eta)
    delta, s_k, above, equal = tk.result_host()
    s = (((alpha[:, None] + beta[None, :]) - M) + 0.0).ravel()
    want = -np.sort(-s)[k - 1]
    assert s_k == want, (s_k, want)
    assert above == int((s > want).sum()) and equal == int((s == want).sum())


@pytest.mark.parametrize("ties", [1, 2, 255, 256, 257, 300, 20000])
@pytest.mark.parametrize("n,m", [(1100, 1000), (2300, 2100)])
def test_ties_at_the_threshold(n, m, ties):
    rng = np.random.default_rng(ties)
    M = rng.random((n, m))
    k = n * m // 100
    order = np.argsort(M, axis=None)                       # alpha = beta = 0: the k smallest costs are kept
    at = order[k - 1 - ties // 2: k - 1 - ties // 2 + ties]
    M.ravel()[at] = M.ravel()[order[k - 1]]
    check(M, np.zeros(n), np.zeros(m), 0.05, k, f"{ties} ties")


@pytest.mark.parametrize("frac", [1e-6, 1e-3, 0.01, 0.5, 0.999])
def test_outliers_and_forbidden_entries(frac):
    n, m, eta = 1300, 1700, 0.05
    M, a, b, alpha, beta = W.random_small(n, m, seed=11, eta=eta)
    k = max(1, int(frac * n * m))
    check(M, alpha, beta, eta, k, "plain")
    far = M.copy(); far[5, :] = 1e6; far[9, 17] = -1e6; far[:, 3] = 1e-300
    check(far, alpha, beta, eta, k, "far-off entries")
    inf = M.copy(); inf[np.random.default_rng(1).random((n, m)) < 0.0005] = np.inf
    check(inf, alpha, beta, eta, k, "infinite costs")
    zero = alpha.copy(); zero[::400] = -np.inf              # rows without mass
    check(M, zero, beta, eta, min(k, int(0.99 * n * m)), "rows at -inf")
    narrow = 1e5 + 1e-9 * M                                 # keys that share all their leading bits
    check(narrow, alpha * 1e-10, beta * 1e-10, eta, k, "narrow range")


def test_refresh_with_rows_at_minus_infinity():
    n, m, eta = 1300, 1700, 0.05
    M, a, b, alpha, beta = W.random_small(n, m, seed=12, eta=eta)
    alpha[::400] = -np.inf
    k = n * m // 100
    pr = PatternRefresh(n, m, k)
    pr.refresh(dev(M), dev(a), dev(b), dev(alpha), dev(beta), eta)
    torch.cuda.synchronize()
    T = np.exp(((alpha[:, None] + beta[None, :]) - M) / eta)
    want = -np.sort(-T.ravel())[k - 1]
    assert int(pr.info.cpu()[1]) == 0 and int(pr.info.cpu()[0]) == k
    assert abs(float(pr.delta.cpu()[0]) / want - 1) < 1e-12

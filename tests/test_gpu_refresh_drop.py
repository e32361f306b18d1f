"""regot_dual_eval_sparsify_topk where its kernels behind the pass go beyond what they usually meet: segments of several hundred
candidates (ranks counted over many words of the bits of those that stay), and a bin of the k-th value with thousands of keys,
equal ones (more than a thread of the finish kernel asks for ahead)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_2605_08793_amd import workloads as W
from test_gpu_refresh import check_against_oracle, dev, run_refresh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,rows,frac", [(1100, 1000, 60, 0.03), (1100, 1030, 300, 0.2), (2500, 513, 40, 0.01), (1600, 700, 1600, 0.5)])
def test_long_segments(n, m, rows, frac):
    eta = 0.2
    M, a, b, alpha, beta = W.random_small(n, m, seed=n + rows, eta=eta)
    at = np.random.default_rng(rows).permutation(n)[:rows]
    M[at] -= 20.0 * eta if rows < n else 0.0
    k = int(frac * n * m)
    pr, info, delta, got = run_refresh(dev(M), M, a, b, alpha, beta, eta, k, "long segments")
    check_against_oracle(M, a, b, alpha, beta, eta, k, pr, info, delta, got)


@pytest.mark.parametrize("ties", [1, 300, 2500, 6000])
def test_many_keys_in_the_bin(ties):
    n, m, eta, k = 1500, 1400, 0.3, 40000
    rng = np.random.default_rng(17)
    M = rng.random((n, m))
    M.flat[rng.permutation(n * m)[:ties]] = np.sort(M, axis=None)[k - ties // 2]
    a = np.full(n, 1.0 / n); b = np.full(m, 1.0 / m)
    alpha = np.zeros(n); beta = np.zeros(m)
    pr, info, delta, got = run_refresh(dev(M), M, a, b, alpha, beta, eta, k, "many keys")
    check_against_oracle(M, a, b, alpha, beta, eta, k, pr, info, delta, got)

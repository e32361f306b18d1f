"""Several sweeps in one call on matrices whose sweeps all take the rows forward with streaming loads: what a sweep leaves to
the next one of the call (the published numbers, the order of arrival, the marks) with one member and several, batches of four
and of eight rows, infinite costs, columns that are done again, members that are done without, in a graph."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_08793_amd import binding as B
from paper_2605_08793_amd import workloads as W
from paper_2605_08793_amd.driver import DualPass
from parity_utils import assert_half_step_close

pytestmark = pytest.mark.gpu


# sweeps go forward alone beyond 2.7e7 entries for two of them in a call, 3.6e7 for more
@pytest.mark.parametrize("n,m,sweeps", [
    (14300, 1900, 2), (19000, 1900, 3),      # one member: one group of columns a wave
    (18800, 1921, 3),                        #             two groups
    (3600, 7690, 2), (4700, 7690, 3),        # five members, batches of eight rows
    (2260, 16000, 4), (590, 61400, 3),       # five and sixteen members, batches of four
])
def test_several_streaming_sweeps(n, m, sweeps):
    assert n * m > (27000000 if sweeps == 2 else 36000000)
    eta = 0.05
    print(f"[sweep stream] n={n} m={m} sweeps={sweeps}", flush=True)
    M, a, b, _, beta = W.random_small(n, m, seed=n + m, eta=eta)
    M[n // 2:, m // 3: m // 3 + 40] = np.inf
    M[3, :] = np.inf
    M[3, m - 2] = 0.4
    b[m // 4: m // 4 + 300] = 0.0
    b /= b.sum()
    a *= 0.9
    want = oracle.sinkhorn_sweeps(M, a, b, eta, sweeps, np.zeros(n), beta)
    Md, ad, bd = (torch.from_numpy(x).cuda() for x in (M, a, b))
    dp = DualPass(n, m)
    al, be = (torch.zeros(k, dtype=torch.float64, device="cuda") for k in (n, m))
    start = torch.from_numpy(beta).cuda()

    def run():
        be.copy_(start)
        B.regot_sinkhorn_sweeps(Md, ad, bd, al, be, eta, sweeps, workspace=dp.workspace)

    dp.workspace.fill_(0x5A)
    run()
    first = al.clone(), be.clone()
    for got, ref, what in zip(first, want, ("alpha", "beta")):
        got, some = got.cpu().numpy(), np.isfinite(ref)
        np.testing.assert_array_equal(got[~some], ref[~some], err_msg=what)
        assert_half_step_close(got[some], ref[some], eta, what)
    for looks in (0, 1):     # (held for one call, all of its sweeps)
        B.regot_sweep_patience(looks)
        run()
        assert torch.equal(al, first[0]) and torch.equal(be, first[1]), looks
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for replay in range(3):
        al.fill_(float("nan"))
        graph.replay()
        assert torch.equal(al, first[0]) and torch.equal(be, first[1]), replay
        run()
        assert torch.equal(al, first[0]) and torch.equal(be, first[1]), replay

"""Solves in portions with a look at the direction after each: the combination works in the same workspace and must
leave what the next portion goes on from alone."""
import numpy as np
import pytest
import torch

from paper_2605_08793_amd import binding as B
from paper_2605_08793_amd.driver import SparseTerm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reduced", [True, False])
@pytest.mark.parametrize("systems", [1, 2])
@pytest.mark.parametrize("n,m", [(2000, 1500), (70000, 300), (300, 70000), (20100, 20300)])
def test_a_direction_after_every_portion(n, m, systems, reduced):
    rng = np.random.default_rng(n + m)
    N, nnz = n + m - 1, 12 * max(n, m)
    print(f"[schur portions] n={n} m={m} systems={systems} reduced={reduced}", flush=True)
    rows, cols = np.divmod(np.unique(rng.integers(0, n * m, nnz)), m)
    val = rng.random(len(rows)) / len(rows)

    def dev(x):
        return torch.from_numpy(np.ascontiguousarray(x)).cuda()

    rp = dev(np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64))
    term = SparseTerm(n, m, rp, dev(cols.astype(np.int32)), len(rows))
    term.val[:] = dev(val)
    term.val_csc[term.csc_pos] = term.val
    r, c = dev(np.bincount(rows, val, n) * 1.2 + 0.1 / n), dev(np.bincount(cols, val, m) * 1.2 + 0.1 / m)
    rhs = [dev(rng.standard_normal(N) / N) for _ in range(systems)]
    others = [dev(rng.standard_normal(N)) for _ in range(4)]
    workspace = torch.empty(B.regot_pcg_workspace_bytes(n, m), dtype=torch.uint8, device="cuda")
    call = getattr(B, f"regot_pcg_solve{'' if systems == 1 else '2'}{'_reduced' if reduced else ''}")

    def solve(portions, look):
        workspace.fill_(0x55)
        x = [torch.full((N,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(systems)]
        info = torch.zeros(4 * systems, dtype=torch.float64, device="cuda")
        d, used = torch.empty(N, dtype=torch.float64, device="cuda"), torch.zeros(2, dtype=torch.float64, device="cuda")
        seen = []
        for k, its in enumerate(portions):
            call(n, m, 0.05, 1e-3, term.row_ptr, term.col_idx, term.val, term.col_ptr, term.row_idx, term.val_csc, r, c,
                 *rhs, *x, 1e-10, its, k == 0, info, workspace=workspace)
            if look:
                B.regot_splr_direction(n, m, x[0], others[0], others[1], others[2], others[3], d, used, workspace=workspace)
                B.regot_splr_direction(n, m, x[0], None, None, None, None, d, used, workspace=workspace)
                assert torch.equal(d, -x[0])
            seen.append(info.cpu().tolist())
        return x, seen

    portions = [0, 0, 1, 1, 0, 1, 100, 3]
    got, got_info = solve(portions, True)
    want, want_info = solve(portions, False)
    assert got_info == want_info
    # (the portions make no difference either)
    whole, whole_info = solve([sum(portions)], False)
    assert whole_info[0] == want_info[-1] and all(whole_info[0][4 * k + 1] == 1 for k in range(systems))
    assert want_info[3][0] == 2 and want_info[5][0] == 3
    for g, w, a in zip(got, want, whole):
        assert torch.equal(g, w) and torch.equal(g, a)

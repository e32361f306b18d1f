"""regot_pattern_transpose of a CSR structure whose rows hold a column more than once (which a pattern as include/regot.h defines it does not):
every entry is listed, in the order of the entries, whichever way the pattern is transposed; bit for bit against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def pattern(n, m, each, seed):
    rng = np.random.default_rng(seed)
    ci = np.sort(rng.integers(0, m, size=(n, each)), axis=1).astype(np.int32)  # (with replacement)
    return np.arange(n + 1, dtype=np.int64) * each, ci


CASES = {
    "one entry": (300, 2000, 20), "drawn with replacement": (900, 1500, 60), "many in a column": (100, 300, 1000), "wide": (700, 30000, 300),
    "all groups, odd rows": (1023, 4099, 40), "one block": (7, 600, 400), "by sorting": (40, 20600, 300),
}


@pytest.mark.parametrize("name", list(CASES))
def test_repeats(name):
    from paper_2605_08793_amd import binding as B
    n, m, each = CASES[name]
    rp, ci = pattern(n, m, each, seed=n + m)
    if name == "one entry":  # none but the last two of the last row
        ci = np.stack([np.sort(np.random.default_rng(i).permutation(m)[:each]) for i in range(n)]).astype(np.int32)
        ci[-1, -2] = ci[-1, -1]
    if name == "many in a column":  # more than 16 bits hold; and rows in which it is not the only one
        ci[:] = 299
        ci[::3, :500] = 130
    if name == "all groups, odd rows":  # rows of no entries and of many, unsorted ones
        keep = np.ones(n * each, dtype=bool); keep[40 * each: 200 * each] = False
        rows = np.repeat(np.arange(n), each)[keep]
        ci = ci.ravel()[::-1].copy()[keep]
        rp = np.zeros(n + 1, dtype=np.int64); rp[1:] = np.cumsum(np.bincount(rows, minlength=n))
    ci = ci.ravel(); nnz = int(rp[-1])
    o_cp, o_ri, o_pos = oracle.pattern_transpose(n, m, rp, ci)
    ws = torch.empty(B.regot_pattern_transpose_workspace_bytes(n, m, nnz), dtype=torch.uint8, device="cuda")
    print(f"[repeats] {name}: n={n} m={m} nnz={nnz}", flush=True)
    for poison in (0xA5, 0):
        ws.fill_(poison)
        cp = torch.full((m + 1,), -5, dtype=torch.int64, device="cuda")
        ri = torch.full((nnz,), -5, dtype=torch.int32, device="cuda")
        pos = torch.full((nnz,), -5, dtype=torch.int64, device="cuda")
        B.regot_pattern_transpose(n, m, nnz, torch.as_tensor(rp).cuda(), torch.as_tensor(ci).cuda(), cp, ri, pos, workspace=ws)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(cp.cpu().numpy(), o_cp)
        np.testing.assert_array_equal(ri.cpu().numpy(), o_ri)
        np.testing.assert_array_equal(pos.cpu().numpy(), o_pos)


def test_repeats_beside_entries_of_no_column():
    from paper_2605_08793_amd import binding as B
    n, m, each = 400, 700, 50
    rp, ci = pattern(n, m, each, seed=9)
    ci = ci.ravel(); nnz = int(rp[-1])
    bad = np.random.default_rng(1).permutation(nnz)[:2000]
    keep = np.ones(nnz, dtype=bool); keep[bad] = False
    rows = np.repeat(np.arange(n), each)[keep]
    rp2 = np.zeros(n + 1, dtype=np.int64); rp2[1:] = np.cumsum(np.bincount(rows, minlength=n))
    o_cp, o_ri, o_pos = oracle.pattern_transpose(n, m, rp2, ci[keep])
    given = ci.copy(); given[bad] = np.resize(np.array([m, -1, 2 ** 31 - 1, -2 ** 31], dtype=np.int32), bad.size)
    ws = torch.full((B.regot_pattern_transpose_workspace_bytes(n, m, nnz),), 0x7F, dtype=torch.uint8, device="cuda")
    cp = torch.empty(m + 1, dtype=torch.int64, device="cuda")
    ri = torch.full((nnz,), -5, dtype=torch.int32, device="cuda"); pos = torch.full((nnz,), -5, dtype=torch.int64, device="cuda")
    B.regot_pattern_transpose(n, m, nnz, torch.as_tensor(rp).cuda(), torch.as_tensor(given).cuda(), cp, ri, pos, workspace=ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(cp.cpu().numpy(), o_cp)
    np.testing.assert_array_equal(ri.cpu().numpy()[:keep.sum()], o_ri)
    got = pos.cpu().numpy()
    assert (got[bad] == -1).all()
    np.testing.assert_array_equal(got[keep], o_pos)


def test_repeats_on_either_side_of_a_cut():
    """65535 rows, the most that are transposed by counting, with an entry each in one column, and a second one in the rows that two blocks
    share, so that no block has both: more entries of the column than the 16 bits of a column's place count."""
    from paper_2605_08793_amd import binding as B
    n, m, each, column = 65535, 2048, 17, 1000
    nnz = n * each
    share = min(max(nnz // 128, 2048), 16384)  # entries of a block; the entry at position p of row r is block (r / 32 + p / share)'s
    p = np.arange(nnz, dtype=np.int64)
    block = ((p // each) * share + 32 * p) // (32 * share)
    block = block.reshape(n, each)
    ci = np.sort(np.random.default_rng(2).integers(0, 58, size=(n, each)) + 58 * np.arange(each), axis=1).astype(np.int32)   # up to 985
    ci[:, -1] = column
    cut = block[:, 0] != block[:, -1]
    assert cut.sum() > 100
    ci[cut, 0] = column
    rp, ci = np.arange(n + 1, dtype=np.int64) * each, ci.ravel()
    o_cp, o_ri, o_pos = oracle.pattern_transpose(n, m, rp, ci)
    assert o_cp[column + 1] - o_cp[column] > 65535
    ws = torch.full((B.regot_pattern_transpose_workspace_bytes(n, m, nnz),), 0x7F, dtype=torch.uint8, device="cuda")
    cp = torch.empty(m + 1, dtype=torch.int64, device="cuda")
    ri = torch.full((nnz,), -5, dtype=torch.int32, device="cuda"); pos = torch.full((nnz,), -5, dtype=torch.int64, device="cuda")
    print(f"[repeats] cut rows: n={n} m={m} nnz={nnz} cut={int(cut.sum())}", flush=True)
    B.regot_pattern_transpose(n, m, nnz, torch.as_tensor(rp).cuda(), torch.as_tensor(ci).cuda(), cp, ri, pos, workspace=ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(cp.cpu().numpy(), o_cp)
    np.testing.assert_array_equal(ri.cpu().numpy(), o_ri)
    np.testing.assert_array_equal(pos.cpu().numpy(), o_pos)

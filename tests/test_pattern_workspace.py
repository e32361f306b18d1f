"""The size regot_pattern_transpose asks for: it does not fall as the pattern gets more entries, so what was asked for the largest
pattern does for the others of its matrix, and it is no more than include/regot.h says.  A host-side query, without a GPU."""
import pytest

from paper_2605_08793_amd import binding as B


def asked(n, m, nnz):
    return B.regot_pattern_transpose_workspace_bytes(n, m, nnz)


# matrices on either side of each edge of by_counting, and those whose number of blocks used to fall with nnz
SHAPES = [(1023, 40000), (1023, 20000), (319, 30000), (1631, 38091), (20000, 20000), (200, 40000), (1000, 40000), (90, 40001), (65535, 2048), (65536, 2048),
          (20480, 300), (20481, 300), (40, 20480), (39, 20480), (30, 255), (1, 1), (1, 40000), (3000, 3000), (65535, 40000), (50000, 50000)]


def entries(n, m):
    """Up to the full matrix or 4e6: steps of one at the edges (of the entries of a block, of the rule, of a tile of the sort), then odd strides."""
    most = min(n * m, 4_000_000)
    edges = {1, 2048, 262_144, 262_272, 2_097_152, n * m // 512, n * m // 200, 16 * n}
    some = {e + d for e in edges for d in range(-130, 131)} | set(range(0, 700_000, 127)) | set(range(700_000, 4_000_001, 997)) | {317_262, 317_444}
    return sorted(e for e in some if 0 <= e <= most)


@pytest.mark.parametrize("n,m", SHAPES)
def test_does_not_fall_with_more_entries(n, m):
    before = 0
    for nnz in entries(n, m):
        size = asked(n, m, nnz)
        assert size >= before, (nnz, size, before)
        before = size


@pytest.mark.parametrize("n,m", SHAPES)
def test_is_what_the_header_says(n, m):
    p = (m + 127) // 128 * 128
    for nnz in entries(n, m):
        b = n // 32 + max(nnz // 16384, min(nnz // 2048, 128)) + 2
        bound = max(20.5 * nnz, nnz + (3 * p + 24) * b + 5 * p if n < 65536 and m <= 40000 else 0) + 4096
        assert asked(n, m, nnz) <= bound, nnz

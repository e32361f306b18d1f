"""The shares of a vector that the parts of the reduced solve work on, up to the longest vector a call takes: checked by the
compiler, from the kernels' own header."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "regot.h"
#include "regot_kernels.hpp"
#include "regot_schur.hpp"
// one share behind the other, from 0 to the end of the vector, none longer than the others' length
constexpr bool whole(int64_t count)
{
    using namespace regot;
    int64_t end = 0;
    for (int part = 0; part < kSchurParts; ++part) {
        const int64_t begin = schur_share(count, part), next = schur_share(count, part + 1);
        if (begin != end || next < begin || next - begin > (count + kSchurParts - 1) / kSchurParts) return false;
        end = next;
    }
    return end == count;
}
static_assert(whole(COUNT), "shares");
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("count", [0, 1, 255, 257, 20001, 2147483392, 2147483393, 2147483646])
def test_shares_cover_the_vector(tmp_path, count):
    src = tmp_path / "shares.hip"
    src.write_text(PROGRAM)
    done = subprocess.run(["hipcc", "-std=c++17", "--cuda-host-only", "-fsyntax-only", "-w", f"-DCOUNT={count}LL",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2605_08793_amd", "csrc"),
                           str(src)], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr

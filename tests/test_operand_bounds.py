"""Where gemm_split_kernel reads its fp32 operand, asked of the functions that the kernel asks: every 16-byte read of a 32-deep
stage lies inside the stored operand, for rows that end in the middle of a 32-byte chunk too.  Runs on the host."""
import os
import subprocess

import pytest

from paper_2110_15032_amd import build

PROGRAM = r"""
#include <cstdio>
#include "gemm_device.h"
using namespace sbp;
template <int R, int NT>
int check() {   // reduction-major storage: 32 rows of `limit` floats, `ld` apart, the last one not padded
    using T = Tile<R, false, NT, 32, true>;
    int bad = 0;
    for (int limit = 8; limit <= 2 * R + 12; limit += 4)
        for (int ld = limit; ld <= limit + 8; ld += 4)
            for (int first = 0; first < limit; first += R)
                for (int tid = 0; tid < NT; ++tid)
                    for (int it = 0; it < T::PER_THREAD; ++it) {
                        const uint64_t off = 2ull * T::src_offset(ld, first, limit, it * NT + tid), size = 4ull * (31ull * ld + limit);
                        const uint64_t second = off + T::second_half(first, limit, tid);
                        bad += off % 16 || off + 16 > size || second + 16 > size;
                        // the values that count: column c of the chunk comes from float c
                        const int krow = (it * NT + tid) / T::CPR, col = (int)(off / 4 - (uint64_t)krow * ld);
                        if (col + 8 <= limit && second != off + 16) ++bad;
                    }
    return bad;
}
int main() {
    const int bad = check<128, 256>() + check<128, 512>();
    printf("%d\n", bad);
    return bad != 0;
}
"""


def test_the_split_kernel_reads_inside_its_fp32_operand(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    src, exe = tmp_path / "bounds.hip", str(tmp_path / "bounds")
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--cuda-host-only", "-O1", "-std=c++17", "-w", "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"), str(src), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, f"{r.stdout.strip()} reads outside the operand or of the wrong values"

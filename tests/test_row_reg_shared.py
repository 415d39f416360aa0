"""The start of the LDS of the Top-k that holds a row in registers (csrc/topk_row_reg_shared.h), run on the host for every
thread of the workgroup and every length of the register array: what has to be zero is, and nothing else is written,
inside the object or past its end (the kernel's results cannot show that: what it stores there are zeros)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <cstring>
#include "topk_row_reg_shared.h"
using namespace ef21;

constexpr unsigned char kUnwritten = 0xa5;

template <int R>
int check() {
    struct Guarded {
        RegShared<R> sh;
        unsigned char past[4 * 4 * kRegThreads];
    };
    static Guarded got, want;
    std::memset((void *)&got, kUnwritten, sizeof got);
    std::memset((void *)&want, kUnwritten, sizeof want);
    for (int tid = 0; tid < kRegThreads; ++tid) clear_shared(got.sh, tid);
    std::memset(want.sh.hist, 0, sizeof want.sh.hist);
    std::memset(want.sh.bitmap, 0, sizeof want.sh.bitmap);
    std::memset(want.sh.tie_rank, 0, sizeof want.sh.tie_rank);
    std::memset(want.sh.sub, 0, sizeof want.sh.sub);
    want.sh.bin = want.sh.count = want.sh.n_list = want.sh.n_tie = 0;
    const unsigned char *a = (const unsigned char *)&got, *b = (const unsigned char *)&want;
    for (size_t i = 0; i < sizeof got; ++i)
        if (a[i] != b[i]) {
            std::printf("%d quads a thread: byte %zu of an object of %zu is %02x, not %02x\n", R, i, sizeof got.sh, a[i], b[i]);
            return 1;
        }
    return 0;
}

int main() { return check<1>() + check<2>() + check<3>() + check<4>() + check<6>() + check<9>() + check<13>() + check<15>(); }
"""


@pytest.mark.parametrize("optimise", ["-O0", "-O2"])
def test_start_of_the_lds_stays_inside_its_arrays(tmp_path, optimise):
    source, program = tmp_path / "start.cpp", tmp_path / "start"
    source.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", optimise, "-Wall", "-Werror", "-I",
                           os.path.join(ROOT, "paper_2106_05203_amd", "csrc"), str(source), "-o", str(program)])
    done = subprocess.run([str(program)], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stdout

"""How set_state and get_state copy arrays (csrc/copy_way.h), run on the host: by hipMemcpyAsync, or by a kernel through the caches or past them."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "copy_way.h"
int main() {
    long n, d;
    int arrays;
    while (std::scanf("%ld %ld %d", &n, &d, &arrays) == 3)
        std::printf("%d\n", (int)ef21::copy_way((n + 2) * d, arrays == 1 ? d : (n + 2) * d, arrays == 1));
}
"""

# n, d, arrays copied, us with a step by hipMemcpyAsync, through the caches and past them: one card, in turn
MEASURED = [
    # a step with supplied gradients, then x out
    (8, 2000000, 1, 57.2, 57.6, 56.0), (4, 5000000, 1, 76.4, 76.3, 78.6), (2, 6000000, 1, 65.3, 65.7, 70.6), (8, 6000000, 1, 134.5, 135.6, 139.4),
    (8, 7000000, 1, 157.0, 158.0, 162.0), (4, 7000000, 1, 102.5, 102.8, 106.6), (16, 4000000, 1, 186.7, 188.6, 191.6), (20, 5000000, 1, 273.2, 273.7, 277.5),
    (100, 1000000, 1, 299.6, 300.6, 301.7), (1, 9000000, 1, 69.4, 69.8, 70.3), (4, 9000000, 1, 124.3, 124.9, 123.0), (1, 12000000, 1, 89.3, 89.6, 90.9),
    (2, 12000000, 1, 107.7, 108.4, 108.7), (1, 16000000, 1, 104.6, 104.9, 107.6), (1, 18000000, 1, 117.3, 117.8, 118.9), (2, 14000000, 1, 126.6, 127.0, 127.1),
    (4, 12000000, 1, 157.3, 158.5, 157.7), (2, 16000000, 1, 141.5, 142.3, 138.3), (1, 20000000, 1, 136.4, 136.4, 130.1), (5, 11500000, 1, 178.3, 179.1, 175.5),
    (8, 11200000, 1, 248.5, 249.2, 242.5), (8, 12000000, 1, 264.2, 266.4, 255.9), (4, 16000000, 1, 223.4, 224.4, 213.8), (8, 20000000, 1, 472.9, 472.8, 429.3),
    (1, 30000000, 1, 226.4, 216.2, 183.9), (4, 30000000, 1, 451.2, 442.7, 380.1), (1, 50000000, 1, 372.0, 377.8, 329.2), (4, 50000000, 1, 702.4, 711.2, 655.4),
    (1, 100000000, 1, 714.2, 718.9, 658.0), (2, 100000000, 1, 934.3, 942.9, 864.5),
    # a step, then x, g_i and g out
    (8, 2000000, 3, 81.8, 74.8, 75.5), (2, 8000000, 3, 108.7, 100.5, 107.8), (1, 10000000, 3, 101.9, 97.9, 102.8), (4, 5000000, 3, 106.6, 98.5, 105.9),
    (1, 13000000, 3, 142.3, 133.5, 127.2), (2, 10000000, 3, 142.7, 134.7, 125.5), (8, 4000000, 3, 150.2, 138.5, 138.8), (8, 5000000, 3, 188.6, 179.2, 164.7),
    (16, 2200000, 3, 163.5, 151.0, 153.7), (4, 7000000, 3, 163.3, 154.6, 150.5), (4, 8000000, 3, 180.3, 173.1, 158.3), (2, 16000000, 3, 231.3, 229.8, 198.2),
    (4, 12000000, 3, 262.2, 262.7, 225.5),
    # the three in, then a step
    (8, 1000000, 3, 49.7, 47.4, 50.3), (2, 3000000, 3, 53.7, 51.8, 52.3), (2, 6000000, 3, 86.6, 84.7, 98.2), (8, 3000000, 3, 107.2, 103.4, 109.0),
    (1, 9000000, 3, 96.3, 94.4, 105.1), (1, 13000000, 3, 142.1, 125.3, 136.2), (8, 4000000, 3, 155.1, 135.9, 143.0), (8, 5000000, 3, 185.7, 177.6, 171.3),
    (4, 10000000, 3, 223.4, 217.9, 202.6), (8, 7000000, 3, 265.8, 260.1, 241.4), (8, 11200000, 3, 419.1, 417.9, 371.7), (1, 40000000, 3, 416.5, 431.3, 358.8),
]


def test_no_copy_is_slower_than_by_hipmemcpyasync(tmp_path):
    source, program = tmp_path / "way.cpp", tmp_path / "way"
    source.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2106_05203_amd", "csrc"),
                           str(source), "-o", str(program)])
    done = subprocess.run([str(program)], input="\n".join("%d %d %d" % row[:3] for row in MEASURED), capture_output=True, text=True,
                          timeout=60, check=True)
    ways = [int(line) for line in done.stdout.split()]
    assert len(ways) == len(MEASURED)
    for row, way in zip(MEASURED, ways):
        us = row[3:]
        assert us[way] <= 1.005 * us[0], (row, way)           # two runs differ by half a per cent
        # between 39 and 44 million entries in all the copy out is up to 7 per cent faster one way, the copy in up to 9 the other
        assert us[way] <= 1.025 * min(us) or (row[2] == 3 and 39e6 <= (row[0] + 2) * row[1] <= 44e6 and us[way] <= 1.09 * min(us)), (row, way)

"""Which way the stepsize's power iteration goes (csrc/gram_way.h), run on the host: with A, on the Gram matrices in fp32 (the iteration or the
recurrence), or by squaring them."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "gram_way.h"
int main() {
    int n, iterations;
    long m, d;
    while (std::scanf("%d %ld %ld %d", &n, &m, &d, &iterations) == 4) {
        const ef21::GramWay way = ef21::gram_way(n, m, d, iterations);
        const char *name = way.bytes == 0 ? "A" : way.squarings >= 0 ? "squaring" : ef21::lanczos_steps(iterations) ? "recurrence" : "iteration";
        std::printf("%s %d %zu\n", name, way.squarings, way.bytes);
    }
}
"""


@pytest.fixture(scope="module")
def ways(tmp_path_factory):
    """(n, m, d, iterations) .. -> names of the ways."""
    folder = tmp_path_factory.mktemp("ways")
    source, program = folder / "ways.cpp", folder / "ways"
    source.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2106_05203_amd", "csrc"),
                           str(source), "-o", str(program)])

    def ask(cases):
        done = subprocess.run([str(program)], input="\n".join("%d %d %d %d" % tuple(c) for c in cases), capture_output=True, text=True,
                              timeout=60, check=True)
        names = [line.split()[0] for line in done.stdout.splitlines()]
        assert len(names) == len(cases)
        return names
    return ask


# n, m, d, iterations, us a call on G in fp32, us by squaring (the best number of squarings): measured one after the other on one card
MEASURED = [
    (39, 249, 183, 47, 122.3, 134.8), (38, 28, 171, 47, 112.9, 129.1), (49, 422, 203, 47, 167.4, 192.1), (53, 15, 148, 47, 114.2, 130.2),
    (47, 410, 215, 47, 163.5, 181.6), (36, 9, 183, 47, 111.1, 128.5), (46, 108, 823, 1000, 3589.1, 4026.4),
    (32, 1942, 520, 47, 1016.5, 838.8), (34, 342, 548, 47, 769.8, 640.3), (10, 91, 837, 100, 831.9, 674.5), (34, 221, 526, 47, 720.6, 542.2),
    (5, 151, 1004, 47, 669.0, 474.1), (13, 51, 830, 1000, 2533.0, 1199.4), (9, 144, 969, 1000, 2526.7, 1389.6), (12, 36, 683, 100, 672.8, 491.4),
    (8, 18, 292, 2, 72.4, 44.4), (1, 112, 260, 2, 68.1, 39.1),
]


def test_the_faster_way_on_the_matrices_is_taken(ways):
    names = ways([row[:4] for row in MEASURED])
    for row, name in zip(MEASURED, names):
        best = "squaring" if row[5] < row[4] else "fp32"
        assert name == best or (best == "fp32" and name in ("recurrence", "iteration")), (row, name)


def test_up_to_128_columns_nothing_is_squared(ways):
    names = ways([(n, 500, d, t) for n in (1, 20, 300) for d in (1, 64, 128) for t in (1, 47, 48, 2822, 2823, 10**6)])
    assert "squaring" not in names


def test_the_gpu_tests_reach_the_ways_they_are_for(ways):
    """test_gpu_stepsize.py names for its shapes the way that each goes: a rule that sends them elsewhere would empty it."""
    from test_gpu_stepsize import MANY_PRODUCTS, REACHED
    cases = [(n, d, d, t, way) for n, d, way, iterations in REACHED for t in iterations]
    cases += [(n, 1024, 1024, t, "squaring") for n, t in MANY_PRODUCTS]
    names = ways([case[:4] for case in cases])
    assert names == [case[4] for case in cases], [(case, name) for case, name in zip(cases, names) if name != case[4]]

"""Workgroups that hand work over by a ticket (draw_ticket in csrc/device_utils.h): every wavefront's stores have to have arrived before
the ticket is drawn.  One thread draws it, and what the compiler makes of a barrier does not wait for the other wavefronts' stores, so the
compiled code is looked at: no run shows the order of two stores that are nearly always a microsecond apart."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2106_05203_amd", "csrc")

SOURCE = r"""
#include "device_utils.h"
extern "C" __global__ __launch_bounds__(1024) void publish(uint32_t *out, uint32_t *sums, uint32_t *counter, uint32_t *total) {
    __shared__ uint32_t last;
    out[blockIdx.x * 1024 + threadIdx.x] = threadIdx.x;
    atomicAdd(sums + threadIdx.x, threadIdx.x);
    if (ef21::draw_ticket(counter, gridDim.x, &last)) total[threadIdx.x] = sums[threadIdx.x];
}
"""


def test_stores_arrive_before_the_ticket(tmp_path):
    from paper_2106_05203_amd import build
    source, listing = tmp_path / "publish.hip", tmp_path / "publish.s"
    source.write_text(SOURCE)
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared") and not f.startswith("-parallel-jobs")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-I", CSRC, "--cuda-device-only", "-S", "-o", str(listing),
                           str(source)], stderr=subprocess.DEVNULL)
    code = listing.read_text().split("publish:", 1)[1].split("s_endpgm", 1)[0]
    lines = [line.split(";")[0].strip() for line in code.splitlines()]
    barrier = next(i for i, line in enumerate(lines) if line.startswith("s_barrier"))
    stores = [i for i, line in enumerate(lines[:barrier]) if re.match(r"(global|flat)_(store|atomic)", line)]
    assert len(stores) == 2, lines[:barrier]
    assert any(re.match(r"s_waitcnt .*vmcnt\(0\)", line) for line in lines[stores[-1]:barrier]), lines[stores[-1]:barrier + 1]


def test_tickets_are_drawn_in_one_place():
    """A fence of the device's scope is in draw_ticket alone: what hands work over by other means would need a look of its own."""
    with_fence = sorted(name for name in os.listdir(CSRC) if "__threadfence" in open(os.path.join(CSRC, name)).read())
    assert with_fence == ["device_utils.h"], with_fence

"""A copy from memory straight into LDS takes its destination from m0 and must not follow the scalar instruction that
writes m0 without a wait state in between.  The compiler keeps to that for its own instructions and does not look into
assembly, so the listing of the copies is checked.  (m0 is written nowhere else, so that these are all there are.)"""
import os
import re
import subprocess

import pytest

from paper_2305_12213_amd import build

KERNEL = """
#include <hip/hip_runtime.h>
#include "lds_async.h"
__global__ void copies(const char* from, float* out) {
  __shared__ uint4 area[256];
  const uint32_t to = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&area[0];
  dynb::async_copy_1k(from + threadIdx.x * 16, to);
  dynb::async_copy_1k_from(from + 1024, threadIdx.x * 16, to + 1024);
  dynb::async_copy_1k_buffer(dynb::buffer_resource(from, 4096), 2048 + threadIdx.x * 16, to + 2048);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  out[threadIdx.x] = ((const float*)area)[threadIdx.x];
}
"""


def is_copy(l):
    return l.startswith("global_load_lds") or l.startswith("buffer_load") and l.endswith("lds")


def too_early(lines):
    """Copies right behind the instruction that writes their m0."""
    return [b for a, b in zip(lines, lines[1:]) if is_copy(b) and re.match(r"s_\w+ m0,", a)]


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    d = tmp_path_factory.mktemp("copies")
    (d / "copies.hip").write_text(KERNEL)
    subprocess.run(["hipcc", *build.HIP_FLAGS, "-I", build.CSRC, "--cuda-device-only", "-S", str(d / "copies.hip"),
                    "-o", str(d / "copies.s")], check=True, capture_output=True)
    lines = [l.split(";")[0].strip() for l in (d / "copies.s").read_text().splitlines()]
    return [l for l in lines if re.match(r"[a-z]\w+( |$)", l)]


def test_copies_wait_for_their_destination(listing):
    assert sum(map(is_copy, listing)) == 3
    assert not too_early(listing)
    assert len(too_early([l for l in listing if not l.startswith("s_nop")])) == 3     # the check itself


def test_only_the_copies_write_m0():
    for name in sorted(os.listdir(build.CSRC)):
        with open(os.path.join(build.CSRC, name)) as f:
            text = f.read()
        assert name == "lds_async.h" or not re.search(r'"[^"\n]*\bm0,', text), name

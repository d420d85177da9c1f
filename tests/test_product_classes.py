"""Which class a bf16 product is timed in, asked of the library's own rule through a small program linked against it:
every tile size is a kernel of its own, and a class's average launch is one kernel's."""
import pytest

from test_result_routes import ask

PROGRAM = """
#include <cstdio>
#include "dynb_internal.h"
int main() {
  int mode, m, n, k;
  while (std::scanf("%d %d %d %d", &mode, &m, &n, &k) == 4) {
    dynb::GemmArgs a = {};
    a.mode = mode; a.M = m; a.N = n; a.K = (int)dynb::round_up(k, 64);
    std::printf("%s\\n", dynb_profile_name(dynb::gemm_class(DYNB_BF16, a)));
  }
}
"""
FWD, DGRAD, WGRAD = range(3)

CALLS = [
    (FWD, 4096, 4096, 4096, "gemm_fwd"), (DGRAD, 4096, 4096, 1000, "gemm_dgrad"), (WGRAD, 4096, 4096, 0, "gemm_wgrad"),
    (FWD, 3329, 3585, 64, "gemm_fwd"),                                           # 14 x 15 tiles of 256
    (FWD, 4096, 1000, 4096, "gemm_small_tiles"), (DGRAD, 1400, 1409, 65, "gemm_small_tiles"),
    (FWD, 1025, 1100, 1030, "gemm_128x64_tiles"), (DGRAD, 1531, 777, 2112, "gemm_128x64_tiles"),
    (FWD, 1531, 777, 128, "gemm_64_tiles"), (FWD, 1024, 10, 1024, "gemm_64_tiles"), (DGRAD, 1024, 1024, 1024, "gemm_64_tiles"),
    (WGRAD, 1000, 4096, 0, "gemm_wgrad_small_tiles"),
]


@pytest.fixture(scope="module")
def classes(tmp_path_factory):
    return ask(tmp_path_factory.mktemp("classes"), PROGRAM, "".join("%d %d %d %d\n" % c[:4] for c in CALLS))


@pytest.mark.parametrize("i", range(len(CALLS)))
def test_tile_sizes_are_timed_apart(classes, i):
    assert classes[i] == CALLS[i][-1], CALLS[i]

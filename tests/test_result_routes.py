"""Rules of launches that were measured on both sides, asked of the library itself through a small program linked against
it: whether the weight gradients of a launch of 64 x 64 tiles leave past the caches, and how tall the tiles of an update
are."""
import os
import subprocess

import pytest

from paper_2305_12213_amd import build


def ask(directory, program, calls):
    (directory / "main.cpp").write_text(program)
    if not os.path.exists(build.LIB):
        build.build_library(verbose=False)
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(directory / "main.cpp"), build.LIB, "-o",
                    str(directory / "main"), "-Wl,--allow-shlib-undefined", "-Wl,-rpath," + os.path.dirname(build.LIB)],
                   check=True)
    return subprocess.run([str(directory / "main")], input=calls, check=True, capture_output=True, text=True).stdout.split()


# dense layers (inputs, outputs, whether the launch forms the average), workers, whether past the caches was faster
RESULTS = [
    ([(960, 160, 0), (160, 192, 0)], 8, False),        # 6 MB
    ([(672, 160, 0), (160, 1024, 0)], 16, True),       # 17 MB
    ([(448, 224, 0), (224, 96, 0)], 64, True),         # 31 MB
    ([(1024, 1024, 0)], 8, False),                     # 34 MB
    ([(544, 1248, 0), (1248, 256, 0)], 64, False),     # 256 MB
    ([(1440, 1088, 0), (1088, 1920, 0), (1920, 32, 0)], 64, True),   # 952 MB
    ([(3072, 1024, 1), (1024, 1024, 1)], 8, True),     # 134 MB, averaged in the launch
    ([(1024, 500, 0)], 8, False),                      # 16 MB, but rows that are not whole lines
    ([(1024, 500, 1)], 8, False),
    ([(1440, 1088, 0), (1088, 1900, 0)], 64, False),   # ... the larger part of a launch
    ([(3072, 1024, 1), (1024, 10, 1)], 8, True),       # ... the smaller
]

PROGRAM = """
#include <cstdio>
#include "dynb_internal.h"
int main() {
  int layers, K;
  while (std::scanf("%d %d", &layers, &K) == 2) {
    dynb::GemmArgs a[8] = {};
    for (int q = 0; q < layers; ++q) {
      int in, out, folded;
      if (std::scanf("%d %d %d", &in, &out, &folded) != 3) return 1;
      a[q].mode = dynb::MODE_WGRAD; a[q].M = out; a[q].N = in; a[q].ldcf = out;
      a[q].Cf = (float*)(1 << 20);
      a[q].agg = folded ? a[q].Cf : nullptr;
    }
    std::printf("%d\\n", (int)dynb::wgrad_small_past(a, layers, K));
  }
}
"""


@pytest.fixture(scope="module")
def results(tmp_path_factory):
    calls = "".join("%d %d %s\n" % (len(layers), K, " ".join("%d %d %d" % l for l in layers)) for layers, K, _ in RESULTS)
    return ask(tmp_path_factory.mktemp("results"), PROGRAM, calls)


@pytest.mark.parametrize("i", range(len(RESULTS)))
def test_results_leave_the_faster_way(results, i):
    assert (results[i] == "1") == RESULTS[i][-1], RESULTS[i]


# layers (rows, columns, taps), workers whose average is folded into the update (0: none), rows of the faster tiles
CHAIN = [(33, 44, 1), (44, 253, 1), (253, 173, 1), (173, 26, 1), (26, 152, 1), (152, 143, 1), (143, 300, 1)]
TILES = [
    ([(785, 301, 1), (301, 97, 1), (97, 10, 1)], 0, 16), ([(3072, 512, 1), (512, 512, 1), (512, 10, 1)], 0, 64),
    ([(256, 256, 9)], 0, 16),
    ([(320, 320, 9)], 2, 16), ([(1495, 1200, 1)], 7, 16),                              # few workers
    ([(416, 1000, 1)], 64, 16), ([(586, 471, 1), (471, 10, 1)], 64, 16),               # one or two layers
    ([(682, 203, 1), (203, 788, 1)], 64, 16), ([(1344, 1000, 1)], 16, 16),
    ([(919, 836, 1), (836, 300, 1), (300, 10, 1)], 16, 64),                            # more: 128 tiles and more
    ([(600, 700, 1), (700, 300, 1), (300, 10, 1)], 16, 16),
    ([(600, 700, 1), (700, 300, 1), (300, 10, 1)], 32, 64),                            # 81 MB of gradients
    ([(256, 256, 9), (256, 256, 9)], 8, 64), ([(128, 128, 9), (128, 128, 9)], 32, 16),
    ([(192, 192, 9)], 32, 16), ([(256, 256, 9)], 32, 64),                              # 42 and 75 MB, convolutions
    (CHAIN[:5], 32, 16), (CHAIN[:6], 32, 64), (CHAIN[:6], 8, 16), (CHAIN, 8, 64),
]

TILE_PROGRAM = """
#include <cstdio>
#include "dynb_internal.h"
int main() {
  int layers, K;
  while (std::scanf("%d %d", &layers, &K) == 2) {
    dynb::CastMats m = {};
    m.n = layers;
    for (int q = 0; q < layers; ++q)
      if (std::scanf("%d %d %d", &m.R[q], &m.C[q], &m.taps[q]) != 3) return 1;
    std::printf("%d\\n", dynb::cast_tile_rows(m, K > 0 ? 128 : 64, K));
  }
}
"""


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    calls = "".join("%d %d %s\n" % (len(layers), K, " ".join("%d %d %d" % l for l in layers)) for layers, K, _ in TILES)
    return ask(tmp_path_factory.mktemp("tiles"), TILE_PROGRAM, calls)


@pytest.mark.parametrize("i", range(len(TILES)))
def test_updates_take_the_faster_tiles(tiles, i):
    assert int(tiles[i]) == TILES[i][-1], TILES[i]

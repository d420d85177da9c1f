"""How weight gradients of convolutions are worked on, asked of the library's own rule through a small program linked
against it: with how many groups of threads the chunks of a worker are added up (the three forms were timed at these
sizes), and which layers share a launch."""
import random

import pytest

from test_gpu_layers_of_one_geometry import CALLS
from test_result_routes import ask

TAPS, ROWS, FLAT = range(3)

PROGRAM = """
#include <cstdio>
#include "dynb_internal.h"
int main() {
  int layers, h, w, cin, cout, K, most_images;
  long long at_least;
  while (std::scanf("%d %d %d %d %d %d %lld %d", &layers, &h, &w, &cin, &cout, &most_images, &at_least, &K) == 8) {
    dynb::Segs s = {};
    s.K = K;
    for (int k = 0; k < K; ++k) {
      int images;
      if (std::scanf("%d", &images) != 1) return 1;
      s.off[k + 1] = s.off[k] + images * h * w;
    }
    const int64_t rows = (int64_t)most_images * h * w;
    int64_t scratch = dynb::conv_wgrad_scratch_floats(rows, K, cin, cout);
    scratch = scratch < at_least ? at_least : scratch;
    auto pitch = [](int c) { return c <= 32 ? 32 : dynb::round_up(c, 64); };
    const dynb::ConvWgradPlan p = dynb::conv_wgrad_plan(
        layers, pitch(cin), cin, h, w, pitch(cout), cout, h, w, 1, dynb::conv_wgrad_chunk_rows(rows), scratch, s);
    const int64_t blocks = (int64_t)((cin + 63) / 64) * ((cout + 63) / 64);
    const bool flat = p.kernel == dynb::CONV_WGRAD_FLAT;
    const int64_t floats = (int64_t)p.layers * p.ch.first[K] * blocks * (flat ? p.ci32 * p.co32 * 10 * 1024 : 40 * 1024);
    std::printf("%d,%d,%d,%d,%d,%d\\n", p.kernel, (int)p.paired, p.layers, p.sum_groups, p.ch.rows,
                (int)(floats <= scratch));
  }
}
"""


def plans(directory, calls):
    """(kernel, paired, layers, sum_groups, rows of a chunk, whether its results fit in the scratch area) of every (layers,
    image, channels in and out, batch bound, batches, floats of the scratch area if that is larger for another layer)."""
    lines = "".join("%d %d %d %d %d %d %d %d %s\n" % (n, *image, *channels, most, (at_least or [0])[0], len(b), " ".join(map(str, b)))
                    for n, image, channels, most, b, *at_least in calls)
    return [tuple(int(v) for v in l.split(",")) for l in ask(directory, PROGRAM, lines)]


# channels, images of 16 x 16 pixels of the workers (a chunk each), groups of the faster sum
SUMS = [
    (24, [1] * 64, 1), (24, [32] + [1] * 63, 1), (24, [190] + [1] * 63, 4), (24, [64] + [1] * 63, 4),
    (24, [24] + [1] * 7, 4), (24, [6] * 64, 1), (24, [400] + [1] * 15, 16), (24, [48] * 8, 4), (24, [4], 1), (24, [64], 4),
    (64, [8] * 8, 1), (64, [24] * 8, 4), (64, [190, 1, 1, 1], 16), (64, [190] + [1] * 63, 4), (64, [6] * 16, 1),
    (128, [12] * 4, 1), (128, [1, 1, 1, 1, 1, 1, 1, 64], 1),
    (24, [0, 0], 1), (24, [0, 190, 0], 16),
]


@pytest.fixture(scope="module")
def sums(tmp_path_factory):
    return plans(tmp_path_factory.mktemp("sums"), [(1, (16, 16), (c, c), sum(b) or 1, b) for c, b, _ in SUMS])


@pytest.mark.parametrize("i", range(len(SUMS)))
def test_chunks_are_added_up_the_faster_way(sums, i):
    assert sums[i][3] == SUMS[i][-1], SUMS[i]


# layers, image, channels, most images, batches, how many share the first launch: all of them, also where the results
# of one layer at chunks of its own length are few, unless the workers' last chunks alone are too many
SHARED = [
    (6, (32, 32), (64, 64), 48, [20, 12, 8, 5, 3], 6), (6, (16, 16), (64, 64), 128, [70, 58], 6), (6, (32, 32), (64, 64), 4, [4], 6),
    (4, (28, 28), (24, 24), 167, [64, 45, 33, 18, 7], 4), (6, (32, 32), (64, 64), 512, [139, 139, 69, 69, 35, 35, 17, 9], 6),
    (8, (16, 16), (64, 64), 64, [1] * 64, 2), (8, (1, 1), (64, 524353), 8, [8] + [0] * 63, 4),     # (more blocks of eight than a grid takes)
]


@pytest.fixture(scope="module")
def shared(tmp_path_factory):
    return plans(tmp_path_factory.mktemp("shared"), [s[:-1] for s in SHARED])


@pytest.mark.parametrize("i", range(len(SHARED)))
def test_layers_of_one_geometry_share_launches(shared, i):
    assert shared[i][2] == SHARED[i][-1], SHARED[i]


def test_plans_fit_in_the_scratch_area(tmp_path):
    rng = random.Random(7)
    calls = []
    for _ in range(2000):
        b = [rng.choice([0, 1, 2, rng.randint(0, 60)]) for _ in range(rng.choice([1, 2, 5, 16, 64]))]
        calls.append((rng.randint(1, 8), (rng.randint(1, 40), rng.randint(1, 40)), (rng.randint(1, 300), rng.randint(1, 300)),
                      max(1, sum(b)) * rng.choice([1, 1, 1, 2, 9]), b))
    for call, (kernel, paired, layers, groups, rows, fits) in zip(calls, plans(tmp_path, calls)):
        assert fits and 1 <= layers <= call[0] and groups in (1, 4, 16) and rows > 0, call
        assert rows % (call[1][1] if kernel == ROWS else 32) == 0, call
        assert not paired or kernel != FLAT, call


def launches(directory, image, channels, b, most):
    """(kernel, paired, layers, sum_groups) of every launch that takes more than one layer of such a model."""
    widths = [image[2], *channels]
    # (the last layer divides its reduction where it has few tiles: at most 64 results of each worker)
    dense = -(-widths[-1] * 7 // 64) * 64 * 64 * len(b)
    todo = {}
    for i, o in zip(widths, widths[1:]):
        todo[i, o] = todo.get((i, o), 0) + 1
    got = []
    for shape, n in todo.items():
        while n > 0:
            p = plans(directory, [(min(n, 8), image[:2], shape, most, b, dense)])[0]
            got.append(p[:4])
            n -= p[2]
    return got


def test_the_calls_run_on_the_device_reach_every_form(tmp_path):
    by_call = [launches(tmp_path, *call) for call in CALLS]
    several = [p for got in by_call for p in got if p[2] > 1]
    assert {p[:2] for p in several} == {(FLAT, 0), (ROWS, 0), (ROWS, 1), (TAPS, 0), (TAPS, 1)}
    assert {p[3] for p in several} == {1, 4, 16}
    assert [p[2] for p in by_call[0] if p[2] > 1] == [8, 2]
    assert [p[2] for p in by_call[11] if p[2] > 1] == [4, 4] and all(p[2] == 1 for p in by_call[12])

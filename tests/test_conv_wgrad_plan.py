"""How weight gradients of convolutions are worked on, asked of the library's own rule through a small program linked
against it: with how many groups of threads the chunks of a worker are added up (the three forms were timed at these
sizes)."""
import pytest

from test_result_routes import ask

PROGRAM = """
#include <cstdio>
#include "dynb_internal.h"
int main() {
  int layers, h, w, cin, cout, K, most_images;
  while (std::scanf("%d %d %d %d %d %d %d", &layers, &h, &w, &cin, &cout, &most_images, &K) == 7) {
    dynb::Segs s = {};
    s.K = K;
    for (int k = 0; k < K; ++k) {
      int images;
      if (std::scanf("%d", &images) != 1) return 1;
      s.off[k + 1] = s.off[k] + images * h * w;
    }
    const int64_t rows = (int64_t)most_images * h * w;
    auto pitch = [](int c) { return c <= 32 ? 32 : dynb::round_up(c, 64); };
    const dynb::ConvWgradPlan p = dynb::conv_wgrad_plan(
        layers, pitch(cin), cin, h, w, pitch(cout), cout, h, w, 1, dynb::conv_wgrad_chunk_rows(rows),
        dynb::conv_wgrad_scratch_floats(rows, K, cin, cout), s);
    std::printf("%d,%d,%d,%d\\n", p.kernel, (int)p.paired, p.layers, p.sum_groups);
  }
}
"""


def plans(directory, calls):
    """(kernel, paired, layers, sum_groups) of every (layers, image, channels in and out, batch bound, batches)."""
    lines = "".join("%d %d %d %d %d %d %d %s\n" % (n, *image, *channels, most, len(b), " ".join(map(str, b)))
                    for n, image, channels, most, b in calls)
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
    assert sums[i][-1] == SUMS[i][-1], SUMS[i]

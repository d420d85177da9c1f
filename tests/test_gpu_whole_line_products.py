"""The bf16 products on large tiles at the edges of their tiles, ring and dispatch: rows and columns around multiples
of 64, 128 and 256, one stage and more stages than the ring holds, odd numbers of them, with and without a ReLU mask.
They are held bit for bit against the same rows in pieces small enough for the 64 x 64 tiles, whose sums run
in the same order: a row's results depend on nothing but the row.  (The 64 x 64 tiles are compared with
the float64 oracle in test_gpu_small_products.py.)"""
import numpy as np
import pytest

from paper_2305_12213_amd import synth
from gpu_harness import DeviceRun, worker_grads_as_lists

pytestmark = pytest.mark.gpu


def compare_rows(spec, rows, layers):
    rng = np.random.default_rng(41)
    params = [(W, (rng.standard_normal(b.shape) * 0.1).astype(np.float32)) for W, b in synth.init_params(spec, "he", 5)]
    x, y = synth.make_batch(spec, "normal", rows, 6, 0)
    looked_at = sorted({0, 1, 63, 127, 128, 255, 256, rows // 2, rows - 129, rows - 2, rows - 1})
    # the rows looked at are workers of their own, what lies between them belongs to other workers
    b, at = [], []
    for r in looked_at:
        if r > sum(b):
            b.append(r - sum(b))
        at.append(len(b))
        b.append(1)
    whole = DeviceRun(spec, params, rows, len(b))
    got = worker_grads_as_lists(spec, whole.forward_backward(x, y, b).cpu().numpy(), whole.P)
    few = DeviceRun(spec, params, len(looked_at), len(looked_at))
    ref = worker_grads_as_lists(spec, few.forward_backward(x[looked_at], y[looked_at], [1] * len(looked_at)).cpu().numpy(), few.P)
    for k, r in enumerate(looked_at):
        for layer in range(layers):
            assert np.array_equal(got[at[k]][layer][1], ref[k][layer][1]), (r, layer, "bias")
            assert np.array_equal(got[at[k]][layer][0], ref[k][layer][0]), (r, layer, "weights")


# One row per worker makes a layer's bias gradient the row of the gradient wrt its output, and the next layer's weight
# gradient the outer product of its output with that: both products show in full.
@pytest.mark.parametrize("n_in,width,classes,rows", [
    (64, 1409, 65, 1400),        # 11 x 12 tiles of 128: one stage forward, two stages back
    (200, 1664, 300, 1290),      # 11 x 13: four and five stages
    (320, 1535, 64, 1409),       # five and one
    (64, 3585, 65, 3329),        # 14 x 15 tiles of 256: one and two stages
    (190, 3328, 130, 3584),      # whole tiles, three stages each
    (450, 4095, 64, 3073),       # 13 x 16: eight and one
    (1030, 1100, 1025, 1025),    # 9 x 18 tiles of 128 x 64: seventeen stages each
    (1024, 1089, 10, 1024),      # 8 x 18: sixteen, and 64 x 64 tiles back
])
def test_rows_of_large_products_equal_rows_of_small_ones(n_in, width, classes, rows):
    spec = synth.mlp_spec([n_in, width, classes], "bf16")
    compare_rows(spec, rows, 2)


# A dense layer whose output goes over a residual branch as well: the input gradient of the layer behind it adds the
# branch's gradient, before the mask or without one.
@pytest.mark.parametrize("relu", [True, False])
@pytest.mark.parametrize("width,rows", [
    (3585, 3329),                # 14 x 15 tiles of 256
    (1535, 1400),                # 11 x 12 of 128
    (1089, 1025),                # 9 x 18 of 128 x 64
])
def test_rows_of_large_products_with_an_addend(width, rows, relu):
    spec = {"dtype": "bf16", "input": (70,), "classes": 33,
            "layers": [synth.dense(70, width, relu=relu), synth.dense(width, width, relu=False), synth.add(0, relu=True),
                       synth.dense(width, 33, relu=False)]}
    compare_rows(spec, rows, 3)

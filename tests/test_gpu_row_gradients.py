"""Weight gradients of stride-1 convolutions by whole image rows (17 to 32 pixels, more than 32 channels on
both sides; 32 pixels: on one): against the float64 oracle with bf16 rounding emulated, on rows that do not
fill the two 16-pixel steps, images one row high, chunks that cross images and end anywhere, workgroups that
divide a chunk; and infinities stay with their worker and their taps."""
import numpy as np
import pytest

from oracle import network as on
from paper_2305_12213_amd import synth
from gpu_harness import DeviceRun, worker_grads_as_lists, worst_pair_relerr
import test_gpu_nonfinite as nonfinite

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("image,channels,b", [
    ((5, 17, 4), (40, 33), [3, 0, 1]),
    ((1, 20, 4), (64, 64), [7, 1]),              # one row per image: only the middle kernel row
    ((2, 31, 4), (36, 70), [5, 2, 1]),           # two blocks of output channels
    ((13, 28, 4), (48, 48), [9, 1, 4]),          # several chunks, image borders inside them
    ((7, 32, 4), (24, 64), [4, 3]),
    ((28, 28, 4), (33, 40), [80, 61, 1]),        # chunks divided between two halves of a workgroup
])
def test_weight_gradients_by_rows(image, channels, b):
    # no ReLU, so there are no 0/1 decisions to resolve; bound of the other bf16 parity tests
    c1, c2 = channels
    spec = {"dtype": "bf16", "input": image, "classes": 4,
            "layers": [synth.conv3x3(image[2], c1, 1, relu=False), synth.conv3x3(c1, c2, 1, relu=False),
                       synth.gap(), synth.dense(c2, 4, relu=False)]}
    params = synth.init_params(spec, "he", 81)
    x, y = synth.make_batch(spec, "normal", sum(b), 82, 0)
    run = DeviceRun(spec, params, sum(b), len(b))
    got = worker_grads_as_lists(spec, run.forward_backward(x, y, b).cpu().numpy(), run.P)
    _, ref = on.worker_gradients(spec, params, x, y, b, emulate_bf16=True)
    for k in range(len(b)):
        assert worst_pair_relerr(got[k], ref[k]) < 8e-3, (image, channels, k)


@pytest.mark.parametrize("width", [17, 28, 32])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_worker_does_not_see_its_neighbours(width, value):
    nonfinite.test_a_worker_does_not_see_its_neighbours((4, width, 4), (40, 40), value)


@pytest.mark.parametrize("width", [17, 20, 28, 31, 32])
def test_a_tap_does_not_see_the_other_side_of_the_image(width):
    nonfinite.test_a_tap_does_not_see_the_other_side_of_the_image((4, width, 36), 40)

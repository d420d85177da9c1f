"""Convolutions whose operand is gathered pixel by pixel (stride 2, and channels or images that no other kernel takes):
channels that are a power of two or not, at either stride, and images of one row or column."""
import numpy as np
import pytest

from oracle import network as on
from paper_2305_12213_amd import synth
from gpu_harness import DeviceRun, worker_grads_as_lists, worst_pair_relerr

pytestmark = pytest.mark.gpu


def spec_of(image, layers, classes):
    made, c = [], image[2]
    for n, stride in layers:
        made.append(synth.conv3x3(c, n, stride, relu=False))
        c = n
    return {"dtype": "bf16", "input": image, "layers": made + [synth.gap(), synth.dense(c, classes, relu=False)], "classes": classes}


# Against the float64 oracle with bf16 rounding emulated, without ReLU: the bound of the other parity tests, 8e-3.
@pytest.mark.parametrize("image,layers,b", [
    ((9, 7, 3), [(40, 1), (72, 2), (96, 1)], [5, 0, 3]),       # 40 and 72 channels, three and two taps to a stage
    ((12, 12, 3), [(96, 1), (96, 1), (200, 2)], [7, 4]),
    ((1, 9, 3), [(136, 1), (136, 1), (136, 2)], [6, 1]),       # one row: taps outside above and below
    ((7, 1, 3), [(64, 1), (128, 2), (24, 1)], [3, 9]),         # one column; whole stages of a tap
    ((6, 6, 3), [(8, 1), (300, 1), (8, 2)], [30, 1, 2]),
])
def test_gathered_convolutions(image, layers, b):
    spec = spec_of(image, layers, 7)
    rng = np.random.default_rng(61)
    params = [(W, (rng.standard_normal(bb.shape) * 0.1).astype(np.float32)) for W, bb in synth.init_params(spec, "he", 62)]
    x, y = synth.make_batch(spec, "normal", sum(b), 63, 0)
    run = DeviceRun(spec, params, sum(b), len(b))
    g = run.forward_backward(x, y, b).cpu().numpy()
    _, ref = on.worker_gradients(spec, params, x, y, b, emulate_bf16=True)
    got = worker_grads_as_lists(spec, g, run.P)
    for k in range(len(b)):
        assert worst_pair_relerr(got[k], ref[k]) < 8e-3, (image, k, worst_pair_relerr(got[k], ref[k]))

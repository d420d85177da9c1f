"""Input gradients of stride-2 convolutions in launches of the sizes that the kernel on runs of pixels takes for each
number of channels: workers of a few samples at the start, in the middle and at the end of a batch that is large
enough, against the float64 oracle with bf16 rounding emulated (bound of the other bf16 parity tests)."""
import numpy as np
import pytest

from paper_2305_12213_amd import synth
from gpu_harness import DeviceRun, worker_grads_as_lists, worst_pair_relerr
from relu_ties import resolved_worker_references

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("image,channels,b", [
    ((9, 35, 4), (33, 32), [2, 70, 1, 0, 64, 2]),      # two blocks of input channels, the second almost empty
    ((9, 35, 4), (16, 40), [2, 1]),                    # a quarter of the last 64 channels of dy
    ((15, 16, 4), (40, 72), [2, 210, 1, 212, 3]),      # one workgroup per compute unit
    ((3, 128, 4), (8, 120), [1, 2]),                   # ... on the widest images
    ((6, 40, 4), (72, 48), [1, 150, 2, 140, 2]),       # three blocks of input channels
    ((6, 10, 4), (200, 24), [3, 240, 0, 236, 1]),      # seven
    ((7, 7, 4), (128, 8), [1, 520, 2, 520, 3]),        # more than half a round of workgroups
])
def test_strided_input_gradient_in_launches_of_its_sizes(image, channels, b):
    # with a residual branch into the strided layer's input: addend and mask
    c1, c2 = channels
    spec = {"dtype": "bf16", "input": image, "classes": 3,
            "layers": [synth.conv3x3(image[2], c1, 1), synth.conv3x3(c1, c1, 1, relu=False), synth.add(0, True),
                       synth.conv3x3(c1, c2, 2), synth.gap(), synth.dense(c2, 3, relu=False)]}
    params = synth.init_params(spec, "he", 91)
    x, y = synth.make_batch(spec, "normal", sum(b), 92, 0)
    run = DeviceRun(spec, params, sum(b), len(b))
    g = run.forward_backward(x, y, b).cpu().numpy()
    assert np.isfinite(g).all()
    off = np.concatenate([[0], np.cumsum(b)])
    for k, n in enumerate(b):
        if n > 4:
            continue
        got = worker_grads_as_lists(spec, g[k:k + 1], run.P)
        rows = slice(off[k], off[k + 1])
        refs, _, _, _ = resolved_worker_references(spec, params, x[rows], y[rows], [n], got, True)
        assert worst_pair_relerr(got[0], refs[0]) < 8e-3, (image, channels, k)

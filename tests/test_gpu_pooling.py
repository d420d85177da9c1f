"""Global average pooling over images whose pixels end at every edge of the rows that a lane fetches at once (1, 2, 4
or 8 times 32), in 64-byte and 128-byte rows, against the float64 oracle with bf16 rounding emulated (bound of the
other bf16 parity tests)."""
import numpy as np
import pytest

from paper_2305_12213_amd import synth
from test_gpu_parity import check_worker_gradients

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("channels", [20, 72])
@pytest.mark.parametrize("image", [
    (1, 2), (1, 31), (4, 8), (3, 11), (8, 8), (5, 13), (8, 16), (3, 43),   # up to 128 pixels, and one more
    (16, 16), (1, 257), (9, 32), (17, 17), (5, 64), (3, 107), (16, 24), (5, 77),   # 256 and a rest of each kind
])
def test_pooling_of_every_number_of_rows(image, channels):
    spec = {"dtype": "bf16", "input": image + (4,), "classes": 5,
            "layers": [synth.conv3x3(4, channels, 1), synth.gap(), synth.dense(channels, 5, relu=False)]}
    params = synth.init_params(spec, "he", 71)
    rng = np.random.default_rng(8)
    params = [(W, (rng.standard_normal(bb.shape) * 0.1).astype(np.float32)) for W, bb in params]
    b = [2, 0, 3]
    x, y = synth.make_batch(spec, "normal", sum(b), 72, 0)
    check_worker_gradients(spec, params, x, y, b, label="pooling %s %d" % (image, channels))

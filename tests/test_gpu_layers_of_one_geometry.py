"""Weight gradients of convolutions that share a launch because they have one geometry, and the sums over their chunks:
more such layers than a launch takes, layers of another geometry between them, so many workers that the
results of all layers at once do not fit in the scratch area, idle workers, and one, several and many
chunks per worker (the three forms of the sum), on each of the kernels (test_conv_wgrad_plan.py asks the library which
ones the calls take).  Against the float64 oracle with
bf16 rounding emulated, without ReLU (no 0/1 decisions to resolve): the bound of the other parity tests, 8e-3, and
behind more than four convolutions, where a stored value that rounded the other way has spread, the
2e-2 stated for bf16."""
import numpy as np
import pytest

from oracle import network as on
from paper_2305_12213_amd import synth
from gpu_harness import DeviceRun, worker_grads_as_lists, worst_pair_relerr, worst_relerr

pytestmark = pytest.mark.gpu


# image, channels of the layers one after the other, batches, the batch that the model is bound for
CALLS = [
    ((9, 8, 4), [8] * 11, [5, 0, 3], 8),                   # runs of pixels; ten of one geometry: eight and two
    ((3, 20, 4), [40, 40, 40, 40], [90, 0, 31, 1], 122),   # by rows, chunks lengthened until all three fit
    ((5, 6, 4), [40, 40, 33, 40, 40], [60, 17, 0], 77),    # by taps; 40 -> 33 and 33 -> 40 in between
    ((8, 8, 4), [8, 8, 8, 8, 8], [1] * 64, 64),            # one chunk per worker
    ((9, 8, 4), [12, 12, 12], [700], 700),                 # some 200 chunks of one worker
    ((16, 16, 4), [33, 33, 33], [20, 13], 33),             # by taps, several per worker, mostly channels that do not exist
    ((3, 20, 4), [40, 40, 40, 40], [90, 0, 31, 1], 400),   # bound for more: all three at chunks of their own
    ((5, 6, 4), [40, 40, 40], [60, 17, 0], 200),
    ((3, 20, 4), [40, 40, 40], [500, 300, 90], 890),       # halves of chunks in two groups of waves, by rows
    ((16, 16, 4), [33, 33, 33], [200, 130, 1], 331),       # ... and by taps
    ((9, 8, 4), [40, 8, 40, 8, 40], [70, 33], 103),        # runs of pixels, narrow on either side
    ((8, 8, 4), [8] * 9, [1] * 64, 64),                    # eight in halves: too many last chunks
    ((2, 32, 4), [64, 64, 64], [1] * 64, 64),              # ... and each alone
]


@pytest.mark.parametrize("image,channels,b,most", CALLS)
def test_convolutions_of_one_geometry(image, channels, b, most):
    layers, c = [], image[2]
    for n in channels:
        layers.append(synth.conv3x3(c, n, 1, relu=False))
        c = n
    layers += [synth.gap(), synth.dense(c, 7, relu=False)]
    spec = {"dtype": "bf16", "input": image, "layers": layers, "classes": 7}
    rng = np.random.default_rng(51)
    params = [(W, (rng.standard_normal(bb.shape) * 0.1).astype(np.float32)) for W, bb in synth.init_params(spec, "he", 52)]
    x, y = synth.make_batch(spec, "normal", sum(b), 53, 0)
    run = DeviceRun(spec, params, most, len(b))
    g = run.forward_backward_aggregate(x, y, b).cpu().numpy()
    _, ref = on.worker_gradients(spec, params, x, y, b, emulate_bf16=True)
    got = worker_grads_as_lists(spec, g, run.P)
    bound = 8e-3 if len(channels) <= 4 else 2e-2
    for k in range(len(b)):
        assert worst_pair_relerr(got[k], ref[k]) < bound, (image, channels, k, worst_pair_relerr(got[k], ref[k]))
        assert b[k] or np.all(g[k] == 0.0)
    assert worst_relerr(run.out.cpu().numpy(), spec, on.weighted_aggregate(ref, b)) < bound

"""Convolutions with resident weights in launches of several tiles per workgroup, so that its two groups of waves take
turns, the halo of a tile is fetched over the results of another, and a run of tiles ends raggedly.  A worker's gradients do
not depend on the other workers: each is compared with the same samples alone, whose launches have one tile per
workgroup (these are compared with the oracle elsewhere).  Activations and their gradients then agree bit for bit; the
weight gradients are sums of at most 5000 products in fp32, cut into parts elsewhere: 2e-5 of the largest is 20 times the
rounding error of such a sum in random order."""
import numpy as np
import pytest

from paper_2305_12213_amd import synth
from gpu_harness import DeviceRun, worker_grads_as_lists, worst_pair_relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("image,channels,b", [
    ((40, 43, 4), 130, [3, 1, 2] * 17),         # the widest images: 102 samples, 686 tiles of 256 pixels, the last of 80;
                                                # three blocks of outputs, 8 or 9 tiles a workgroup; one block, 2 or 3
    ((9, 14, 4), 100, [28, 30, 17, 31, 25] * 11),      # 710 tiles, the last of 162: 5 or 6, 2 or 3
    ((32, 32, 4), 64, [4, 3, 5] * 15),          # tiles that end with images: 2 or 3
    ((5, 31, 4), 64, [30, 20, 7] * 20),         # 691 tiles, rows that do not divide a tile
    ((16, 16, 4), 64, [7, 1, 9, 3] * 14),       # 280 tiles: one or two
])
def test_resident_weights_over_several_tiles(image, channels, b):
    # 64 reduction channels, stride 1, forward and input gradient, with a residual branch (addend and mask)
    spec = {"dtype": "bf16", "input": image, "classes": 4,
            "layers": [synth.conv3x3(image[2], 64, 1), synth.conv3x3(64, channels, 1),
                       synth.conv3x3(channels, 64, 1), synth.conv3x3(64, 64, 1, relu=False), synth.add(0, True),
                       synth.conv3x3(64, 64, 1), synth.gap(), synth.dense(64, 4, relu=False)]}
    params = synth.init_params(spec, "he", 97)
    rng = np.random.default_rng(7)
    params = [(W, (rng.standard_normal(bb.shape) * 0.1).astype(np.float32)) for W, bb in params]
    x, y = synth.make_batch(spec, "normal", sum(b), 98, 0)
    run = DeviceRun(spec, params, sum(b), len(b))
    g = run.forward_backward(x, y, b).cpu().numpy().copy()
    assert np.isfinite(g[:, :run.P]).all()
    together = worker_grads_as_lists(spec, g, run.P)
    off = np.concatenate([[0], np.cumsum(b)])
    for k, n in enumerate(b):
        rows = slice(off[k], off[k + 1])
        alone = worker_grads_as_lists(spec, run.forward_backward(x[rows], y[rows], [n])[:1].cpu().numpy(), run.P)
        assert worst_pair_relerr(together[k], alone[0]) < 2e-5, (image, channels, k)

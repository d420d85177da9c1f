"""The fp32 matrix products where their tiling can go wrong: widths and batches around 16 and 32
(tile sides, the two tile counts per wave), reductions shorter than the ring of blocks, idle and
one-row workers, workers that end inside a 16-row block, and inputs that are read in place or, for
their width or alignment, packed first.  Gradients, biases and their weighted average against the
float64 oracle; 1e-4 is the fp32 bound of the other parity tests."""
import numpy as np
import pytest

from oracle import network as on
from paper_2305_12213_amd import binding, synth
from gpu_harness import DeviceRun, worker_grads_as_lists, worst_pair_relerr, worst_relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,b,shift", [
    ([15, 16, 17], [1], 0),
    ([31, 33, 2], [16, 0, 17, 1], 0),
    ([64, 65, 3], [15, 33], 0),              # read in place
    ([64, 31, 3], [15, 33], 1),              # ... unless the rows are not 16-byte aligned
    ([320, 48, 16], [0, 0, 31, 3], 0),       # more blocks than the ring holds
    ([1024, 1056, 5], [7, 40, 0, 2], 0),     # 2 x 2 tiles per wave, with an edge of one 16-wide tile
    ([1000, 1041, 5], [3, 18], 0),           # ... and one that leaves less than a tile
    ([48, 2], [1] * 64, 0),
    ([20, 17, 16, 40, 33, 9, 18, 16, 15, 12, 10, 3], [5, 0, 18], 0),   # more layers than one launch takes
])
def test_fp32_products_at_the_edges_of_their_tiles(dims, b, shift):
    import torch
    spec = synth.mlp_spec(dims, "f32")
    for L in spec["layers"]:
        L["relu"] = False                    # (no 0/1 decisions: the oracle needs no resolving)
    params = synth.init_params(spec, "he", 7)
    rng = np.random.default_rng(11)
    params = [(W, (rng.standard_normal(bb.shape) * 0.1).astype(np.float32)) for W, bb in params]
    x, y = synth.make_batch(spec, "normal", sum(b), 8, 0)
    run = DeviceRun(spec, params, sum(b), len(b))
    xd = torch.zeros(x.size + 4, device="cuda")[shift:shift + x.size].view(x.shape)
    xd.copy_(torch.from_numpy(x))
    g = run.forward_backward_aggregate(xd, y, b).cpu().numpy()
    _, ref = on.worker_gradients(spec, params, x, y, b)
    got = worker_grads_as_lists(spec, g, run.P)
    for k in range(len(b)):
        assert worst_pair_relerr(got[k], ref[k]) < 1e-4, (dims, b, k)
        assert np.all(g[k, run.P:] == 0.0)
    assert worst_relerr(run.out.cpu().numpy(), spec, on.weighted_aggregate(ref, b)) < 1e-4
    # the two-call form gives the same gradients bit for bit
    two = run.forward_backward(xd, y, b).cpu().numpy()
    assert np.array_equal(two, g)

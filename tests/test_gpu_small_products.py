"""The 64 x 64-tile bf16 products at the edges of their tiles, ring and dispatch: widths around 64,
reductions shorter and longer than the ring, idle and one-row workers, workers that end inside a
32-row stage, averages folded in (many tiles, one worker, few rows and workers) and left to another
pass, and batches on both sides of the row counts from which a reduction is divided instead or the
large tiles take over.  Gradients and
their average against the float64 oracle with bf16 rounding emulated; bound of the other parity
tests (8e-3; without ReLU, so there are no 0/1 decisions to resolve)."""
import numpy as np
import pytest

from oracle import network as on
from paper_2305_12213_amd import synth
from gpu_harness import DeviceRun, worker_grads_as_lists, worst_pair_relerr, worst_relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,b", [
    ([63, 65, 2], [1]),
    ([64, 64, 64], [33, 0, 31, 1]),
    ([700, 129, 3], [40, 2]),                    # eleven stages against a ring of four
    ([520, 530, 10], [200, 0, 100, 7]),          # 81 tiles: folded
    ([520, 530, 10], [300, 0, 260, 7]),          # ... average by a pass over the matrix, behind the shared launch
    ([130, 70, 5], [400, 1, 0, 150]),            # 6 tiles, 551 rows: workers side by side, average apart
    ([130, 70, 5], [600]),                       # ... one worker: folded
    ([72, 40, 3], [4090, 6]),                    # the last batch that is walked ...
    ([72, 40, 3], [4090, 7]),                    # ... and the first that is divided
    ([512, 256, 10], [500, 100]),
    ([130, 70, 5], [3] * 64),                    # 64 workers of a few rows: side by side
    ([1000, 1024, 10], [2100, 1996]),            # large tiles, average by a pass
    ([1000, 1056, 10], [2100, 1996]),            # ... only without the average: small tiles walk for it
    ([24, 65, 40, 33, 64, 70, 48, 20, 66, 34, 12, 4], [20, 0, 33]),   # more layers than one launch takes
])
def test_small_products_at_the_edges_of_their_tiles(dims, b):
    spec = synth.mlp_spec(dims, "bf16")
    for L in spec["layers"]:
        L["relu"] = False
    params = synth.init_params(spec, "he", 7)
    rng = np.random.default_rng(12)
    params = [(W, (rng.standard_normal(bb.shape) * 0.1).astype(np.float32)) for W, bb in params]
    x, y = synth.make_batch(spec, "normal", sum(b), 9, 0)
    run = DeviceRun(spec, params, sum(b), len(b))
    g = run.forward_backward_aggregate(x, y, b).cpu().numpy()
    _, ref = on.worker_gradients(spec, params, x, y, b, emulate_bf16=True)
    got = worker_grads_as_lists(spec, g, run.P)
    for k in range(len(b)):
        assert worst_pair_relerr(got[k], ref[k]) < 8e-3, (dims, b, k)
    assert worst_relerr(run.out.cpu().numpy(), spec, on.weighted_aggregate(ref, b)) < 8e-3
    two = run.forward_backward(x, y, b).cpu().numpy()
    assert np.array_equal(two, g)

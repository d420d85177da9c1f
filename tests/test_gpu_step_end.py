"""Where an iteration's end (mean losses, zero padding) and the weighted averages are formed: along with the
grouped weight gradients or in a last launch, averages of all, some or no layers folded in.  Whatever the
route, the average has to be the ascending sum over the workers' written gradients (fp32 rounding of K
terms: K 2^-24), the losses those of the float64 oracle, and all padding zero."""
import numpy as np
import pytest

from oracle import network as on
from paper_2305_12213_amd import synth
from gpu_harness import DeviceRun, worker_grads_as_lists, worst_pair_relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dims,b", [
    ([64, 10], [43, 21]),                        # every walk is short: all layers fold, no last launch
    ([33, 7], [600]),                            # one worker, more rows than a round of its loss sum
    ([130, 70, 5], [400, 1, 0, 150]),            # longer walks
    ([785, 301, 97, 10], [401, 203, 99, 0, 50, 25, 7]),   # the first layer's walk is worth it
    ([40, 24, 5], [2] * 64),                     # 64 workers: averages in the last launch
    ([24, 65, 40, 33, 64, 70, 48, 20, 66, 34], [20, 0, 33]),   # nine layers: one more than a launch takes
])
def test_end_of_an_iteration(dims, b, dtype):
    spec = synth.mlp_spec(dims, dtype)
    params = synth.init_params(spec, "he", 7)
    x, y = synth.make_batch(spec, "normal", sum(b), 9, 0)
    run = DeviceRun(spec, params, sum(b), len(b))
    g = run.forward_backward_aggregate(x, y, b).cpu().numpy()
    out = run.out.cpu().numpy()
    assert np.isfinite(g).all() and np.isfinite(out).all()
    assert not g[:, run.P:].any() and not out[run.P:].any()
    lam = np.asarray(b, np.float64) / sum(b)
    terms = lam[:, None] * g.astype(np.float64)
    bound = len(b) * 2.0 ** -24 * np.abs(terms).sum(axis=0)      # (lambda_k itself is rounded to fp32 too)
    assert (np.abs(out - terms.sum(axis=0)) <= 2 * bound).all()
    losses, _ = on.worker_gradients(spec, params, x, y, b, emulate_bf16=dtype == "bf16")
    assert np.allclose(run.losses(len(b)), losses, rtol=4e-3 if dtype == "bf16" else 1e-5, atol=1e-6)
    two = run.forward_backward(x, y, b).cpu().numpy()
    assert np.array_equal(two, g)


@pytest.mark.parametrize("dtype,classes", [
    ("f32", 1), ("f32", 16), ("f32", 17),        # whole rows in a 16 x 16 tile, and one class more
    ("bf16", 3), ("bf16", 16), ("bf16", 17), ("bf16", 64), ("bf16", 65),
])
def test_loss_in_the_last_product(dtype, classes):
    # rows that end inside a tile, idle and one-row workers; no hidden layer, so no 0/1 decisions.  Bounds
    # of the other parity tests: fp32 sums 1e-4, one bf16 rounding of the stored gradient 8e-3.
    spec = synth.mlp_spec([70, classes], dtype)
    params = synth.init_params(spec, "he", 5)
    rng = np.random.default_rng(8)
    params = [(W, (rng.standard_normal(bb.shape) * 0.1).astype(np.float32)) for W, bb in params]
    b = [65, 0, 1, 30]
    x, y = synth.make_batch(spec, "normal", sum(b), 4, 0)
    run = DeviceRun(spec, params, sum(b), len(b))
    got = worker_grads_as_lists(spec, run.forward_backward(x, y, b).cpu().numpy(), run.P)
    losses, ref = on.worker_gradients(spec, params, x, y, b, emulate_bf16=dtype == "bf16")
    for k in range(len(b)):
        assert worst_pair_relerr(got[k], ref[k]) < (8e-3 if dtype == "bf16" else 1e-4), (classes, k)
    assert np.allclose(run.losses(len(b)), losses, rtol=1e-4, atol=1e-5)

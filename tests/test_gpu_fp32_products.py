"""The fp32 matrix products where their tiling can go wrong: widths and batches around 16 and 32
(tile sides, the tile counts per wave), reductions shorter than the ring of blocks, idle and
one-row workers, workers walked by one wave and divided over waves, workers that end inside a 16-row
block, and inputs that are read in place or, for their width or alignment, packed first.  Gradients, biases and their weighted average against the
float64 oracle; 1e-4 is the fp32 bound of the other parity tests."""
import numpy as np
import pytest

from oracle import network as on
from paper_2305_12213_amd import binding, synth
from gpu_harness import DeviceRun, worker_grads_as_lists, worst_pair_relerr, worst_relerr
from test_gpu_parity import check_worker_gradients

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
    ([70, 20, 5], [900, 0, 300, 1, 17, 64, 30], 0),       # workers side by side, average in the last launch
    ([300, 320, 5], [300, 0, 300, 1, 17, 64, 30], 0),     # ... two per wave and one left, average by a pass
    ([520, 530, 5], [7, 40, 0, 18], 0),      # 2 x 2 tiles, a worker per wave; single ones where the average is folded in
    ([1024, 1056, 520, 5], [7, 40, 0, 2], 0),             # ... 2 x 2 with it too beside a layer that fills the chip
    ([130, 1030, 5], [0, 40] + [16, 17, 15] * 20 + [33, 0], 0),   # 2 x 2 tiles, six workers per wave, the last with four
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


def test_two_by_two_tiles_in_forward_and_input_gradient():
    # 33 x 33 tiles of 32 x 32 in four products, with ragged edges and ReLU masks; reductions of 60
    # and 5 (two blocks, against a ring of five) and of 1041 and 1030
    spec = synth.mlp_spec([60, 1041, 1030, 5], "f32")
    params = synth.init_params(spec, "he", 17)
    b = [515, 0, 498, 17]
    x, y = synth.make_batch(spec, "normal", sum(b), 18, 0)
    check_worker_gradients(spec, params, x, y, b, label="fp32 2 x 2 tiles")


# The products as one chain of fused multiply-adds in ascending order of the reduction index, bit for
# bit.  Operands of at most 13 bits in [1, 2) make every step exact in float64, so rounding its result
# to float32 is the fused operation.  Each product is read off a gradient that only scales it by a
# power of two: equal logits of 2^n classes make dz = (2^-n - onehot) / b exact.
def chain(a, b):
    acc = np.zeros((a.shape[0], b.shape[1]), np.float32)
    for k in range(a.shape[1]):
        acc = (acc.astype(np.float64) + a[:, k:k + 1].astype(np.float64) * b[k].astype(np.float64)).astype(np.float32)
    return acc


def few_bits(rng, *shape):
    return ((1 + rng.integers(0, 4096, shape) / 4096) * rng.choice([-1.0, 1.0], shape)).astype(np.float32)


def dz_of(y, b, classes):
    dz = np.full((len(y), classes), 1.0 / classes)
    dz[np.arange(len(y)), y] -= 1.0
    return (dz / np.repeat(b, b)[:, None]).astype(np.float32)


def linear_run(dims, params, x, y, b):
    spec = synth.mlp_spec(dims, "f32")
    for L in spec["layers"]:
        L["relu"] = False
    run = DeviceRun(spec, params, len(x), len(b))
    g = run.forward_backward(x, y, b).cpu().numpy()
    return worker_grads_as_lists(spec, g, run.P)


@pytest.mark.parametrize("n,m", [(300, 50), (70, 16370)])     # 2 x 2 tiles from 16353 columns on
def test_forward_is_one_chain(n, m):
    rng = np.random.default_rng(31)
    rows, W = 33, few_bits(rng, n, m)
    x, y = few_bits(rng, rows, n), rng.integers(0, 2, rows).astype(np.int32)
    zeros = np.zeros
    params = [(W, zeros(m, np.float32)), (zeros((m, 2), np.float32), zeros(2, np.float32))]
    got = linear_run([n, m, 2], params, x, y, [1] * rows)     # one row per worker: dW of layer 2 is h dz
    want = chain(x, W)
    for k in range(rows):
        assert np.array_equal(got[k][1][0][:, 1 - y[k]], 0.5 * want[k]), k


@pytest.mark.parametrize("m,classes", [(50, 64), (16370, 32)])
def test_input_gradient_is_one_chain(m, classes):
    rng = np.random.default_rng(32)
    rows, W = 33, few_bits(rng, m, classes)
    x, y = np.zeros((rows, 1), np.float32), rng.integers(0, classes, rows).astype(np.int32)
    zeros = np.zeros
    params = [(zeros((1, m), np.float32), zeros(m, np.float32)), (W, zeros(classes, np.float32))]
    got = linear_run([1, m, classes], params, x, y, [1] * rows)   # bias gradient of layer 1: dz W'
    want = chain(dz_of(y, [1] * rows, classes), np.ascontiguousarray(W.T))
    for k in range(rows):
        assert np.array_equal(got[k][0][1], want[k]), k


@pytest.mark.parametrize("n,classes,b", [
    (77, 16, [64, 32, 8]),
    (1000, 1024, [64, 16]),          # 2 x 2 tiles
    (40, 4, [1024, 512, 2048]),
    (200, 1024, [64] * 14 + [128] + [1]),   # 2 x 2 tiles, two workers per wave
])
def test_weight_gradient_is_one_chain_per_worker(n, classes, b):
    rng = np.random.default_rng(33)
    x, y = few_bits(rng, sum(b), n), rng.integers(0, classes, sum(b)).astype(np.int32)
    params = [(np.zeros((n, classes), np.float32), np.zeros(classes, np.float32))]
    got = linear_run([n, classes], params, x, y, b)
    dz, off = dz_of(y, b, classes), 0
    for k, bk in enumerate(b):
        assert np.array_equal(got[k][0][0], chain(x[off:off + bk].T, dz[off:off + bk])), k
        off += bk


def test_weight_gradient_of_rows_beyond_32_bit_offsets():
    # 2^24 outputs: 32 rows of the gradient are 2 GiB.  Equal logits and small whole inputs make every column without a
    # label exact, in any order; a label's is a chain of at most 32 additions of partial sums below 8.
    import torch
    bound = 32 * 8 * 2.0 ** -24
    n, m, b = 17, 1 << 24, [32, 0, 2]
    rng = np.random.default_rng(34)
    x, y = rng.integers(-8, 9, (sum(b), n)).astype(np.float32), rng.integers(0, m, sum(b)).astype(np.int32)
    y[:3] = [0, m - 1, 17]
    spec = synth.mlp_spec([n, m], "f32")
    run = DeviceRun(spec, [(np.zeros((n, m), np.float32), np.zeros(m, np.float32))], sum(b), len(b))
    g = run.forward_backward_aggregate(x, y, b)
    mean, off = torch.zeros(n + 1, m, dtype=torch.float64, device="cuda"), 0
    for k, bk in enumerate(b):
        got = g[k, :n * m + m].view(n + 1, m)                    # (the biases follow the weights)
        xk = torch.from_numpy(np.hstack([x[off:off + bk], np.ones((bk, 1), np.float32)])).cuda().double()
        labels = torch.from_numpy(y[off:off + bk].astype(np.int64)).cuda()
        want = (xk.sum(0) / (m * max(bk, 1)))[:, None].repeat(1, m)
        plain = torch.ones(m, dtype=torch.bool, device="cuda")
        plain[labels] = False
        want.index_add_(1, labels, -xk.t().contiguous() / max(bk, 1))
        assert bool((got.double() == want)[:, plain].all()), k
        assert float((got.double() - want).abs().max()) <= bound, k
        mean += want * (bk / sum(b))
        off += bk
    out = run.out[:n * m + m].view(n + 1, m).double()
    assert float((out - mean).abs().max()) <= 2 * bound      # (three more, of the workers' shares)

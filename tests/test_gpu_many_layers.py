"""Dense models of more layers than one launch takes: which weight gradients form their average is decided launch by
launch, the aggregate is the weighted sum of the workers' gradients either way; and the static call of as many layers as
its preparation takes in one launch, all of their tensors padded."""
import numpy as np
import pytest

from paper_2305_12213_amd import binding, synth
from gpu_harness import DeviceRun

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,dtype,K,B,finalizes", [
    ([767, 932, 9, 14, 557, 55, 46, 45, 8, 17], "f32", 32, 58, True),   # the ninth layer alone: not worth a walk
    ([767, 932, 9, 14, 557, 55, 46, 45, 8], "f32", 32, 58, False),      # eight layers: free beside the first one's
    ([67, 92, 9, 14, 57, 55, 46, 45, 8, 17], "f32", 2, 9, False),       # worth it in both launches
    ([64, 72, 80, 40, 96, 64, 33, 72, 80, 48, 10], "bf16", 2, 40, None),
    ([64, 72, 80, 40, 96, 64, 33, 72, 80, 48, 10], "bf16", 64, 200, None),
])
def test_aggregate_of_more_layers_than_a_launch_takes(dims, dtype, K, B, finalizes):
    spec = synth.mlp_spec(dims, dtype)
    params = synth.init_params(spec, "he", 5)
    b = [0 if k % 7 == 3 else 1 for k in range(K)]
    b[0] += B - sum(b)
    x, y = synth.make_batch(spec, "normal", B, 6, 0)
    run = DeviceRun(spec, params, B, K)
    run.forward_backward_aggregate(x, y, b)
    binding.profile_enable(True)
    binding.profile_reset()
    g = run.forward_backward_aggregate(x, y, b).cpu().numpy().astype(np.float64)
    launches = binding.profile_read()["finalize"]["launches"]
    binding.profile_enable(False)
    want = sum(n / B * g[k] for k, n in enumerate(b))
    got = run.out.cpu().numpy()
    assert np.abs(got[:run.P] - want[:run.P]).max() <= K * 2.0 ** -24 * max(np.abs(g).max(), 1e-30)
    assert not got[run.P:].any()
    if finalizes is not None:
        assert (launches > 0) == finalizes


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dims,b", [
    ([10, 7, 5, 8, 17], [6, 0, 5, 4]),
    ([33, 65, 1, 70, 9, 130, 66, 3, 5], [40, 1, 37]),       # eight layers, four padded tensors each
    ([1, 1], [3]),
    ([64, 64, 64], [7, 2]),                                 # nothing to pad but the batch
])
def test_static_call_pads_every_tensor(dims, b, dtype):
    import torch
    # scratch full of another model's finite and infinite values
    other = binding.Model(synth.mlp_spec([200, 130, 90], dtype))
    n = other.padded_params()
    p = torch.full((n,), 3e38, device="cuda")
    binding.forward_backward_static(other, p, torch.full((64, 200), 3e38, device="cuda"),
                                    torch.zeros(64, dtype=torch.int32, device="cuda"), [64],
                                    torch.empty(1, n, device="cuda"))
    spec = synth.mlp_spec(dims, dtype)
    params = synth.init_params(spec, "he", 7)
    x, y = synth.make_batch(spec, "normal", sum(b), 8, 0)
    run = DeviceRun(spec, params, sum(b), len(b))
    want = run.forward_backward(x, y, b).clone()
    got = torch.full_like(want, float("nan"))
    binding.forward_backward_static(run.model, run.params, torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda(),
                                    torch.from_numpy(np.ascontiguousarray(y, np.int32)).cuda(), b, got)
    torch.cuda.synchronize()
    assert torch.equal(got[:, :run.P], want[:, :run.P])

"""The workspace-free gradient call right after one that left NaN everywhere in the static scratch, in another
layout: against the call with a workspace of its own, bit for bit (the same kernels over the same values).
Widths that need padding everywhere or nowhere, rows that are read in place, more layers than one preparing
launch takes, a convolutional model, idle workers."""
import numpy as np
import pytest

from paper_2305_12213_amd import binding, synth
from gpu_harness import DeviceRun

pytestmark = pytest.mark.gpu


def cnn_spec():
    return {"dtype": "bf16", "input": (6, 5, 3), "classes": 4,
            "layers": [synth.conv3x3(3, 12, 1), synth.conv3x3(12, 20, 2), synth.gap(),
                       synth.dense(20, 4, relu=False)]}


@pytest.mark.parametrize("dtype,dims", [
    ("f32", [70, 33, 5]), ("f32", [64, 128, 10]), ("f32", [128, 17]), ("f32", [785, 30, 70, 9]),
    ("bf16", [70, 33, 5]), ("bf16", [64, 128, 64]), ("bf16", [7, 66, 2, 90]),
    ("bf16", [24, 65, 40, 33, 64, 70, 48, 20, 66, 34]), ("bf16", None),
])
def test_static_call_on_scratch_full_of_nan(dtype, dims):
    import torch
    b = [19, 0, 5]
    spoil = synth.mlp_spec([200, 600, 300, 50], dtype)
    model = binding.Model(spoil)
    nan = torch.full((256, 200), float("nan"), device="cuda")
    params = torch.full((model.padded_params(),), float("nan"), device="cuda")
    grads = torch.empty(1, model.padded_params(), device="cuda")
    binding.forward_backward_static(model, params, nan, torch.zeros(256, dtype=torch.int32, device="cuda"),
                                    [256], grads)
    spec = synth.mlp_spec(dims, dtype) if dims else cnn_spec()
    p = synth.init_params(spec, "he", 3)
    x, y = synth.make_batch(spec, "normal", sum(b), 6, 0)
    run = DeviceRun(spec, p, sum(b), len(b))
    ref = run.forward_backward(x, y, b).cpu().numpy()
    got = torch.full((len(b), run.Pp), float("nan"), device="cuda")
    binding.forward_backward_static(run.model, run.params, torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(),
                                    b, got)
    torch.cuda.synchronize()
    assert np.isfinite(ref).all()
    assert np.array_equal(got.cpu().numpy(), ref)

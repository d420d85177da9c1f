"""The update launch where its accesses change: widths that are and are not multiples of 4 (whole
16-byte accesses or single elements), matrices narrower and a little wider than a tile, offsets that
are no multiple of 4, all three optimizers, with a finished gradient and with the average folded in,
dense layers and convolutions (nine taps each).  Parameters and state against the definition in
float64; the 16-bit copies through the gradients computed from them, which must equal those of a
model bound afresh to the updated parameters."""
import numpy as np
import pytest

from paper_2305_12213_amd import binding, synth

pytestmark = pytest.mark.gpu


def conv_spec(c1, c2):
    return {"dtype": "bf16", "input": (6, 5, 3), "classes": 3,
            "layers": [synth.conv3x3(3, c1, 1), synth.conv3x3(c1, c2, 2), synth.gap(),
                       synth.dense(c2, 3, relu=False)]}


SPECS = {
    "odd": lambda: synth.mlp_spec([67, 129, 65, 5], "bf16"),
    "aligned": lambda: synth.mlp_spec([64, 132, 68, 8], "bf16"),
    "odd f32": lambda: synth.mlp_spec([3, 131, 7], "f32"),
    "conv odd": lambda: conv_spec(9, 13),
    "conv wide": lambda: conv_spec(72, 68),
    "ten layers": lambda: synth.mlp_spec([9] * 11, "bf16"),      # more tensors than one launch takes
    "many tiles odd": lambda: synth.mlp_spec([2050, 2051, 5], "bf16"),   # (tiles of 64 rows, not of 16)
    "many tiles aligned": lambda: synth.mlp_spec([2052, 2060, 8], "f32"),
}


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("kind", ["sgd", "momentum", "adam"])
@pytest.mark.parametrize("name", list(SPECS))
def test_update_and_copies(name, kind, fold):
    import torch
    spec, b = SPECS[name](), [5, 2, 0, 3, 1]
    K = len(b)
    model = binding.Model(spec)
    P, n = model.num_params(), model.padded_params()
    gen = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    params = rnd(n) * 0.2
    params[P:] = 0
    nbytes = model.workspace_bytes(sum(b), K)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    model.bind(params, ws, nbytes, sum(b), K)
    g, s1, s2 = rnd(K, n), rnd(n), rnd(n).abs()
    lam = torch.tensor(b, dtype=torch.float64, device="cuda") / sum(b)
    gd = (lam[:, None] * g.double()).sum(0) if fold else g[0].double()
    p0, m0, v0 = params.double(), s1.double(), s2.double()
    rule = binding.make_optimizer(kind, lr=0.1, momentum=0.9, step=3)
    if fold:
        binding.model_aggregate_update(model, g, b, rule, s1, s2)
    else:
        binding.model_update(model, g[0].contiguous(), rule, s1, s2)
    if kind == "sgd":
        ref = p0 - 0.1 * gd
    elif kind == "momentum":
        m0 = 0.9 * m0 + gd
        ref = p0 - 0.1 * m0
    else:
        m0 = 0.9 * m0 + 0.1 * gd
        v0 = 0.999 * v0 + 0.001 * gd * gd
        ref = p0 - 0.1 * (m0 / (1 - 0.9 ** 3)) / ((v0 / (1 - 0.999 ** 3)).sqrt() + 1e-8)
    close = lambda a, r: float((a[:P].double() - r[:P]).abs().max()) <= 2e-6 * float(r[:P].abs().max())
    assert close(params, ref)                    # (a dozen fp32 roundings of 6e-8 each)
    if kind != "sgd":
        assert close(s1, m0)
    if kind == "adam":
        assert close(s2, v0)
    x = torch.rand((sum(b),) + tuple(spec["input"]), generator=gen, device="cuda")
    y = torch.zeros(sum(b), dtype=torch.int32, device="cuda")
    fresh = binding.Model(spec)
    ws2 = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    fresh.bind(params, ws2, nbytes, sum(b), K)
    got, want = torch.zeros(K, n, device="cuda"), torch.zeros(K, n, device="cuda")
    binding.forward_backward(model, x, y, b, got)
    binding.forward_backward(fresh, x, y, b, want)
    torch.cuda.synchronize()
    assert torch.isfinite(want).all() and torch.equal(got, want)

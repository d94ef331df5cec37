"""Reductions so wide that the rows of one pass reach 2^32 bytes: the LM head
then takes its general kernel, the draft layer's projections fewer rows per
pass.

The inputs are built so that few channels count and the references are small:
in the LM head, whole numbers in the first and the last channels (exact in
float32); in the draft layer, a gate / up projection that picks single
channels and a down projection with weights at both ends of its rows."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

WIDE = 1 << 24          # 128 rows x 2^24 bf16 channels: 2^32 bytes


def test_lm_head_wide_rows():
    import torch
    import paper_2505_12728_amd as sd
    R, V, n, tau = 128, 20, 512, 16.0
    g = torch.Generator(device="cuda").manual_seed(3)
    hidden = torch.zeros(R, WIDE, dtype=torch.bfloat16, device="cuda")
    weight = torch.zeros(V, WIDE, dtype=torch.bfloat16, device="cuda")
    z = torch.zeros(R, V, dtype=torch.float64, device="cuda")
    for cols in (slice(0, n), slice(WIDE - n, WIDE)):
        h = torch.randint(-2, 3, (R, n), generator=g, device="cuda")
        w = torch.randint(-2, 3, (V, n), generator=g, device="cuda")
        hidden[:, cols], weight[:, cols] = h.bfloat16(), w.bfloat16()
        z += h.double() @ w.double().T
    p = sd.sd_lm_head_probs(hidden, weight, tau)
    # float32 exponentials of exact logits, as PROB_TOL's float32 entry
    assert torch.allclose(p.double(), torch.softmax(z / tau, -1), rtol=1e-5, atol=1e-12)


def test_layer_wide_intermediate():
    import torch
    import paper_2505_12728_amd as sd
    B, r, hq, D, I, n = 8, 16, 4, 64, WIDE, 2048
    d, dev = hq * D, "cuda"
    g = torch.Generator(device=dev).manual_seed(5)
    i8 = dict(dtype=torch.int8, device=dev)
    W = {"fc_w": torch.zeros(d, 2 * d, **i8), "wqkv": torch.zeros(3 * d, d, **i8), "wo": torch.zeros(d, d, **i8),
         "wgu": torch.zeros(2 * I, d, **i8), "wdown": torch.zeros(d, I, **i8)}
    W["fc_w"][:, :d].fill_diagonal_(1)                       # x0 = x1 = the first half of u
    # gate i picks channel i (times 8), up i channel i + 5, both modulo d
    gate = torch.arange(d, device=dev)
    W["wgu"][:I].view(I // d, d, d)[:, gate, gate] = 1
    W["wgu"][I:].view(I // d, d, d)[:, gate, (gate + 5) % d] = 1
    for name in list(W):
        W[name + "_s"] = torch.ones(W[name].shape[0], device=dev)
    W["wgu_s"][:I] = 8.0
    W["wdown_s"].fill_(1.0 / 64)
    W["fc_b"], W["ln1"], W["ln2"] = torch.zeros(d, device=dev), torch.ones(d, device=dev), torch.ones(d, device=dev)
    x = torch.randint(0, 2, (B * r, d), generator=g, device=dev).float() * 2 - 1
    u = torch.cat([x, torch.zeros_like(x)], -1).bfloat16().view(B, r, 2 * d)
    ref = x.double()
    act = torch.nn.functional.silu(8 * x.double()) * x.double().roll(-5, -1)
    for cols in (slice(0, n), slice(I - n, I)):
        w = torch.randint(-127, 128, (d, n), generator=g, device=dev)
        W["wdown"][:, cols] = w.to(torch.int8)
        ref = ref + act.repeat(1, n // d) @ w.double().T / 64
    kc = torch.zeros(B, 32, hq, D, dtype=torch.bfloat16, device=dev)
    out = sd.sd_semi_ar_layer_q8(u, W, kc, kc.clone(), torch.zeros(B, dtype=torch.int32, device=dev), hq, hq, 1e-6, 1e4)
    err = (out.view(B * r, d).double() - ref).abs().max() / ref.square().mean().sqrt()
    # the activations are rounded to bf16 (2^-9 of 8), 4096 of them summed
    assert float(err) <= 2.5e-2
    assert np.isfinite(float(err))

"""The projection stream (sd_linear, sd_linear_q8) at the edges of its tiles:
rows around the 16-row blocks and the 128-row pass, reductions of one chunk,
of an odd number of chunks and of ranges that do not fill the register
groups, columns around the 32-column unit and the 224-column work-group; and
33 to 64 work-groups, which start at different chunks of their range (one to
four splits of 3 to 19 chunks, equal ranges and unequal ones).

Reference: the products in float64.  Every product of two bf16 (or int8 and
bf16) values is exact in float32, so the error is that of the float32 sums:
at most K 2^-24 of the sum of the products' magnitudes.  Whole-number int8
weights have the same bits as bf16, and both types sum in the same order, so
their results agree bit for bit."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,K,N", [
    (1, 256, 1), (6, 256, 33), (16, 512, 31), (17, 768, 224), (33, 2304, 225), (48, 1280, 96),
    (64, 4352, 449), (65, 2816, 64), (80, 256, 7169), (96, 11008, 130), (112, 1024, 57), (128, 512, 448),
    (129, 1536, 225), (300, 768, 70),
    (6, 768, 4001), (40, 1280, 2500), (17, 2304, 4000), (100, 3328, 3001), (128, 4864, 3900), (5, 4864, 2049)])
def test_linear_stream_edges(R, K, N):
    import torch
    import paper_2505_12728_amd as sd
    g = torch.Generator(device="cuda").manual_seed(R * 7919 + K * 31 + N)
    x = torch.randn(R, K, generator=g, device="cuda").bfloat16()
    wq = torch.randint(-127, 128, (N, K), generator=g, device="cuda").to(torch.int8)
    w = wq.bfloat16()
    bias = torch.randn(N, generator=g, device="cuda")
    ref = x.double() @ w.double().T
    # K 2^-24 of the magnitudes for the sum, one rounding for the bias
    bound = K * 2.0 ** -24 * (x.double().abs() @ w.double().abs().T) + 2.0 ** -23 * (ref.abs() + bias.abs() + 1)
    y = sd.sd_linear(x, w, bias=bias)
    assert bool(((y.double() - (ref + bias.double())).abs() <= bound).all())
    yq = sd.sd_linear_q8(x, wq, torch.ones(N, device="cuda"), bias=bias)
    assert torch.equal(y, yq)

"""Rows of the draft layer that hold an infinity, or whose mean square
overflows float32.

An infinite row has no RMSNorm (inf / inf): its keys, values and output are
NaN in the oracle, and must be NaN here rather than finite numbers that the
later rows of the block would attend to.  A finite row whose mean square
overflows float32 is normalised with a factor of 0: its keys and values are
0, and nothing of it is NaN.

The infinite row is the first new row of its sequence, so that every row of
the sequence sees its key; the other sequences stay within the bounds of
tests/test_gpu_draft.py."""

import numpy as np
import pytest

import oracle
from paper_2505_12728_amd import synth
from tests.gpu_util import np_to_device, to_device
from tests.test_gpu_draft import LAYER_MAX, LAYER_RMS

pytestmark = pytest.mark.gpu


def _run(inp, q8):
    import torch
    import paper_2505_12728_amd as sd
    W = {k: (to_device(v) if isinstance(v, synth.Tensor) else np_to_device(v)) for k, v in inp["weights"].items()}
    kc, vc = to_device(inp["k_cache"]), to_device(inp["v_cache"])
    layer = sd.sd_semi_ar_layer_q8 if q8 else sd.sd_semi_ar_layer
    out = layer(to_device(inp["u"]), W, kc, vc, np_to_device(inp["pos"]), inp["hq"], inp["hkv"], inp["eps"], inp["theta"])
    torch.cuda.synchronize()
    return out.cpu().numpy(), kc.float().cpu().numpy(), vc.float().cpu().numpy()


# SwiGLU fused into the gate / up projection and not, one wave and two per
# unit, one and several row blocks and passes
@pytest.mark.parametrize("B,r,hq,hkv,D,I", [(3, 2, 4, 2, 64, 512), (3, 6, 16, 4, 128, 256), (9, 9, 4, 4, 64, 768),
                                            (20, 7, 4, 1, 64, 512)])
@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("value", [np.inf, -np.inf, 2.0 ** 120])
def test_layer_row_without_finite_norm(B, r, hq, hkv, D, I, q8, value):
    w = synth.Workload("edge", "bf16", batch=B, hq=hq, hkv=hkv, head_dim=D, kv_len=64, block=r - 1,
                       draft_ffn=I, draft_ctx=5)
    inp = synth.draft_inputs(w, seed=41 + B + r, q8=q8)
    bad = 1                                     # sequence whose first new row holds the value
    u = inp["u"].values.copy()
    u[bad, 0, 3] = value
    inp["u"] = synth.Tensor(u, "bf16")
    out, kc, vc = _run(inp, q8)
    W = {k: (v.values if isinstance(v, synth.Tensor) else v) for k, v in inp["weights"].items()}
    layer = oracle.semi_ar_layer_q8 if q8 else oracle.semi_ar_layer
    with np.errstate(all="ignore"):
        ref, rk, rv = layer(u, W, inp["k_cache"].values, inp["v_cache"].values, inp["pos"], hq, hkv, inp["eps"],
                            inp["theta"])
    p = int(inp["pos"][bad])
    if np.isinf(value):
        assert np.isnan(ref[bad]).all() and np.isnan(rk[bad, p]).all() and np.isnan(rv[bad, p]).all()
        for got, want in ((out, ref), (kc, rk), (vc, rv)):
            assert np.array_equal(np.isnan(got), np.isnan(want))
    else:
        assert not kc[bad, p].any() and not vc[bad, p].any()
        assert not np.isnan(out).any() and not np.isnan(kc).any() and not np.isnan(vc).any()
    good = np.arange(B) != bad
    rms = float(np.sqrt(np.mean(ref[good] ** 2)))
    assert np.max(np.abs(out[good] - ref[good])) <= LAYER_MAX * rms
    assert np.sqrt(np.mean((out[good] - ref[good]) ** 2)) <= LAYER_RMS * rms

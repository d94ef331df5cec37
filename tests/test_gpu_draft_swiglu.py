"""The draft layer with SwiGLU in the gate / up projection, at the edges of
its tiles: rows around the 16-row blocks and the 128-row pass; intermediate widths whose
16-pair units fill the last work-group, leave it ragged, or are fewer than
the compute units; 3 and 5 chunks of the reduction, at each of which some
work-group starts; one shape whose reduction is split instead.

Reference: the oracle, with the bounds of tests/test_gpu_draft.py.  Int8
weights with power-of-two scales are exact in bf16 and both types sum in the
same order, so their layers agree bit for bit, although the gate and the up
products meet in one wave for bf16 and in two for int8."""

import numpy as np
import pytest

import oracle
from paper_2505_12728_amd import synth
from tests.gpu_util import np_to_device, to_device
from tests.test_gpu_draft import _check_layer, _run_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,r,hq,hkv,D,I", [
    (1, 1, 4, 4, 64, 256), (1, 16, 4, 2, 64, 11008), (17, 1, 4, 4, 64, 768), (6, 8, 2, 1, 128, 4352),
    (8, 8, 4, 4, 64, 11008), (5, 13, 4, 1, 64, 4352), (10, 11, 4, 2, 64, 8448), (8, 16, 4, 4, 64, 512),
    (43, 3, 4, 4, 64, 4352), (3, 2, 16, 4, 128, 256),
    (2, 5, 12, 4, 64, 11008), (9, 9, 20, 4, 64, 4352), (6, 16, 10, 2, 128, 8448)])
def test_fused_swiglu_edges(B, r, hq, hkv, D, I):
    import torch
    import paper_2505_12728_amd as sd
    w = synth.Workload("edge", "bf16", batch=B, hq=hq, hkv=hkv, head_dim=D, kv_len=64, block=r - 1,
                       draft_ffn=I, draft_ctx=20)
    inp = synth.draft_inputs(w, seed=77 + B + r, q8=True)
    q8 = inp["weights"]
    inp["weights"] = {k: v for k, v in q8.items() if not k.endswith("_s")}
    for name in oracle.draft_layer.Q8_WEIGHTS:
        q8[name + "_s"] = np.exp2(np.floor(np.log2(q8[name + "_s"]))).astype(np.float32)
        inp["weights"][name] = synth.Tensor(q8[name].astype(np.float32) * q8[name + "_s"][:, None], "bf16")
    got = _run_layer(inp)
    _check_layer(inp, got)
    W = {k: (to_device(v) if isinstance(v, synth.Tensor) else np_to_device(v)) for k, v in q8.items()}
    out = sd.sd_semi_ar_layer_q8(to_device(inp["u"]), W, to_device(inp["k_cache"]), to_device(inp["v_cache"]),
                                 np_to_device(inp["pos"]), hq, hkv, inp["eps"], inp["theta"])
    torch.cuda.synchronize()
    assert np.array_equal(got[0], out.cpu().numpy())

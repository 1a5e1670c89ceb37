"""silu in the grouped GEMM's two epilogues (whole tiles and fix-up of pieces) where exp(-a) nears
the end of the fp32 range: silu(a) = a / (1 + exp(-a)) is a normal number down to a = -88.7."""
import numpy as np
import pytest
import torch

import moe_inputs as mi
from gpu_util import pack_layer, to_dev, to_host

pytestmark = pytest.mark.gpu


# d = 256: one reduction of 8 steps, whole tiles; d = 2048: 64 steps, every tile goes out in pieces
@pytest.mark.parametrize("d", [256, 2048])
@pytest.mark.parametrize("a", [-88.5, -87.5, -80.0, -3.0, 0.0, 40.0])
def test_silu_over_the_fp32_range(d, a):
    import paper_2402_07033_amd as moe
    f, N = 512, 40
    b = 2.0 ** 100 if a < -60 else 1.0
    bf16 = mi.f32_to_bf16_bits
    x = np.zeros((N, d), np.float32)
    x[:, 0] = 1.0
    w1, w3 = np.zeros((1, d, f), np.float32), np.zeros((1, d, f), np.float32)
    w1[0, 0, :] = a      # exact in bf16, so x.w1 = a and x.w3 = b exactly
    w3[0, 0, :] = b
    w2 = np.zeros((1, f, d), np.float32)
    w2[0, np.arange(f), np.arange(f) % d] = 1.0   # at most two h per output
    W = pack_layer(mi.LayerInputs(None, None, None, bf16(w1), bf16(w3), bf16(w2)))
    off = torch.tensor([0, N], dtype=torch.int32, device="cuda")
    yg = to_host(moe.moe_expert_ffn(W, to_dev(bf16(x)), off, path=moe.MOE_FFN_GROUPED))
    per_out = np.bincount(np.arange(f) % d, minlength=d)
    ref = per_out[None, :] * (a / (1.0 + np.exp(-a)) * b)
    # h rounds to the 8 significant bits of bf16: at most half a unit of the last, 2^-8 of the
    # value; before that exp in fp32 of an argument up to 88.5 (88.5 * 2^-23 < 2^-16)
    err = np.max(np.abs(yg - ref) - (2.0 ** -8 + 2.0 ** -15) * np.abs(ref))
    assert err <= 0, (yg[0, 0], ref[0, 0])
    W.free()

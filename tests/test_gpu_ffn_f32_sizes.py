"""The all-fp32 expert FFN at the edges of its row tiles (16, 32, 64 and 128 rows by the mean
number of rows per expert) and with reductions shorter than a workgroup's waves can share."""
import numpy as np
import pytest
import torch

import moe_inputs as mi
from gpu_util import max_rel, pack_layer, to_dev, to_host
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,f", [(64, 64), (192, 320), (576, 128)])
@pytest.mark.parametrize("counts", [[0, 1, 15, 16, 17], [33, 31, 0, 32, 1], [65, 63, 64, 1, 48],
                                    [257, 129, 128, 127, 0], [300]])
def test_ffn_f32_tile_edges(counts, d, f):
    import paper_2402_07033_amd as moe
    E, N = len(counts), sum(counts)
    cfg = mi.small_config("f32e", 1, d, f, E, 1, 5000 + N + d)
    w1, w3, w2 = mi.make_weights(cfg, threads=1)
    xg = mi.normal_f32(cfg.seed, 90, (N, d))
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    W = pack_layer(mi.LayerInputs(cfg, None, None, w1, w3, w2))
    buf = torch.full((N + 4, d), float("nan"), device="cuda")
    moe.moe_expert_ffn(W, to_dev(xg), to_dev(offsets), yg=buf[:N])
    torch.cuda.synchronize()
    out = to_host(buf)
    assert np.isnan(out[N:]).all() and np.isfinite(out[:N]).all()
    # fp32 sums of up to 576 products in two layers: 1e-5 as the tiny fp32 layer
    assert max_rel(out[:N], orc.expert_ffn(xg.astype(np.float64), offsets, w1, w3, w2)) <= 1e-5
    W.free()

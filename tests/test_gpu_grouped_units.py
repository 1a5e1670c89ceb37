"""Grouped GEMM at the edges of its token units (64 rows) and tiles, for every tile shape: the
step loop exists once per number of units, an expert's units are dealt evenly to its tiles, and
rows past an expert's end are dropped stores."""
import numpy as np
import pytest
import torch

import moe_inputs as mi
from gpu_util import max_rel, pack_layer, to_dev, to_host
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu
# bf16 rows and intermediate, fp32 sums: 2^-9 relative per rounding, as every grouped test
TOL_BF16 = 2e-2

EDGES = {
    # mean rows > 256: 256-row tiles of 1..4 units; 257, 513 and 769 rows leave 1-unit remainders
    # to be dealt over 2, 3 and 4 tiles
    "256 x 256": ([1024, 769, 513, 257, 256, 255, 1, 0], (256, 256)),
    # mean rows 97..256: 192-row tiles of 1..3 units
    "192 x 256": ([385, 193, 192, 191, 129, 128, 65, 16], (192, 256)),
    # up to 96 rows: 128-row tiles of 1..2 units, 512 features
    "128 x 512": ([257, 129, 128, 65, 64, 63, 17, 0], (128, 512)),
}


# d, f: 512 / 1024 one round of few tiles; 2048 / 512 and 512 / 2304 cut left-over tiles along the
# reduction of the first and of the second projection
@pytest.mark.parametrize("d,f", [(512, 1024), (2048, 512), (512, 2304)])
@pytest.mark.parametrize("name", list(EDGES))
def test_grouped_unit_edges(name, d, f):
    import paper_2402_07033_amd as moe
    counts, tile = EDGES[name]
    E, N = len(counts), sum(counts)
    plan = moe.moe_expert_ffn_plan(N, E, d, f, path=moe.MOE_FFN_GROUPED)
    assert (plan["up_tile_rows"], plan["up_tile_features"]) == tile
    assert (plan["down_tile_rows"], plan["down_tile_features"]) == tile
    cfg = mi.small_config("units", 1, d, f, E, 1, 4000 + d + f, w_dtype=mi.BF16, x_dtype=mi.BF16)
    w1, w3, w2 = mi.make_weights(cfg, threads=8)
    xg = mi.f32_to_bf16_bits(mi.normal_f32(cfg.seed, 90, (N, d)))
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    W = pack_layer(mi.LayerInputs(cfg, None, None, w1, w3, w2))
    guard = 16  # rows behind yg that no store may reach
    buf = torch.full((N + guard, d), float("nan"), device="cuda")
    out = []
    for _ in range(2):
        moe.moe_expert_ffn(W, to_dev(xg), to_dev(offsets), yg=buf[:N], path=moe.MOE_FFN_GROUPED)
        torch.cuda.synchronize()
        out.append(to_host(buf).copy())
    assert np.isnan(out[0][N:]).all(), "a store behind the last row"
    assert (out[0][:N] == out[1][:N]).all()
    ref = orc.expert_ffn(mi.to_f64(xg), offsets, w1, w3, w2)
    assert np.isfinite(out[0][:N]).all() and max_rel(out[0][:N], ref) <= TOL_BF16
    W.free()


# MID: GROUPED's tiles (here the 128 x 512 one, 256 x 256 where f % 256 or d % 512 is not 0, and 192 x 256 at
# 140 rows per expert), and f = 128, whose second projection is too short for the pipelined kernel
@pytest.mark.parametrize("d,f", [(256, 128), (512, 128), (512, 384), (1024, 512)])
@pytest.mark.parametrize("counts", [[33, 0, 17, 1], [1, 2, 0, 3], [130, 300, 64, 65]])
def test_mid_path_shapes(d, f, counts):
    import paper_2402_07033_amd as moe
    E, N = len(counts), sum(counts)
    cfg = mi.small_config("mid", 1, d, f, E, 1, 4500 + N + d + f, w_dtype=mi.BF16)
    w1, w3, w2 = mi.make_weights(cfg, threads=8)
    xg = mi.normal_f32(cfg.seed, 90, (N, d))
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    W = pack_layer(mi.LayerInputs(cfg, None, None, w1, w3, w2))
    buf = torch.full((N + 16, d), float("nan"), device="cuda")
    moe.moe_expert_ffn(W, to_dev(xg), to_dev(offsets), yg=buf[:N], path=moe.MOE_FFN_MID)
    torch.cuda.synchronize()
    out = to_host(buf)
    assert np.isnan(out[N:]).all() and np.isfinite(out[:N]).all()
    ref = orc.expert_ffn(xg.astype(np.float64), offsets, w1, w3, w2)
    assert max_rel(out[:N], ref) <= TOL_BF16
    if f == 128:  # GROUPED has no kernel for this reduction, as before
        with pytest.raises(moe.MoeError):
            moe.moe_expert_ffn(W, to_dev(xg), to_dev(offsets), path=moe.MOE_FFN_GROUPED)
    W.free()

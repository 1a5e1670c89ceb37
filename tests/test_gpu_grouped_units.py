"""Grouped GEMM at the edges of its token units (64 rows) and tiles, for every tile shape: the
step loop exists once per number of units, an expert's units are dealt evenly to its tiles, and
rows past an expert's end are dropped stores."""
import numpy as np
import pytest
import torch

import gg_schedule
import moe_inputs as mi
from gpu_util import Scratch, max_rel, pack_layer, to_dev, to_host
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu
# bf16 rows and intermediate (each rounded by up to 2^-8 of itself), fp32 sums, as every grouped test
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
# reduction of the first and of the second projection; 2048 / 1536 leaves 192 of 256 (256-row tiles: too
# many to cut); 2048 / 2560 a round of whole tiles and pieces behind it
@pytest.mark.parametrize("d,f", [(512, 1024), (2048, 512), (512, 2304), (2048, 1536), (2048, 2560)])
@pytest.mark.parametrize("name", list(EDGES))
def test_grouped_unit_edges(name, d, f):
    import paper_2402_07033_amd as moe
    counts, tile = EDGES[name]
    E, N = len(counts), sum(counts)
    if name == "128 x 512" and f == 2560:
        f = 1792  # (larger matrices have tiles of 160 rows there)
    tiles = moe.moe_expert_ffn_tiles(counts, d, f, path=moe.MOE_FFN_GROUPED)
    assert all((t["rows"], t["features"]) == tile for t in tiles.values())
    cfg = mi.small_config("units", 1, d, f, E, 1, 4000 + d + f, w_dtype=mi.BF16, x_dtype=mi.BF16)
    w1, w3, w2 = mi.make_weights(cfg, threads=8)
    xg = mi.f32_to_bf16_bits(mi.normal_f32(cfg.seed, 90, (N, d)))
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    W = pack_layer(mi.LayerInputs(cfg, None, None, w1, w3, w2))
    guard = 16  # rows behind yg that no store may reach
    buf = torch.full((N + guard, d), float("nan"), device="cuda")
    scratch = Scratch(N, E, d, f)
    out = []
    for _ in range(2):
        moe.moe_expert_ffn(W, to_dev(xg), to_dev(offsets), workspace=scratch.ws, yg=buf[:N], path=moe.MOE_FFN_GROUPED)
        torch.cuda.synchronize()
        out.append(to_host(buf).copy())
    assert np.isnan(out[0][N:]).all(), "a store behind the last row"
    assert (out[0][:N] == out[1][:N]).all()
    assert scratch.pieces() == any(t["pieces"] for t in tiles.values())
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


# Several rounds of whole tiles per workgroup, then pieces: the operand requests of a tile's last
# steps are the next tile's, and the waits of its first steps count the stores of the tile before,
# so neighbours of different numbers of units matter.  The step loop exists per number of units and, for
# tiles that are their expert's only one, with the weights past L2.  64 steps in the long projection, and 136 with 128 x 512
# tiles, which give way to those of 160 rows in shorter ones.
ROUNDS = {
    # name: rows per expert (repeated), repeats, tile rows, features of the long projection, its (rounds, cut, turned)
    "256 x 256, several tiles": ([641, 64, 257, 190, 1, 385, 256, 513], 1, 256, 10240, (2, True, False)),
    "256 x 256, one tile each": ([201, 190, 256, 130, 64, 255, 240, 232], 1, 256, 18432, (2, True, False)),
    "256 x 256, turned": ([900, 100, 300, 257, 1, 700, 200, 513], 1, 256, 16384, (4, True, True)),
    "256 x 256, turned, whole": ([900, 100, 300, 257, 1, 700, 200, 513], 1, 256, 18432, (4, False, True)),
    "256 x 256, 8 rounds": ([900, 100, 300, 257, 1, 700, 200, 513], 1, 256, 31744, (8, True, True)),
    "192 x 256, several tiles": ([385, 193, 64, 128, 17, 130, 192, 65], 1, 192, 12800, (2, True, False)),
    "192 x 256, several tiles, whole": ([385, 193, 64, 128, 17, 130, 192, 65], 1, 192, 16384, (2, False, False)),
    "192 x 256, nearly one tile each": ([200, 190, 128, 65, 17, 130, 192, 64], 1, 192, 16384, (2, True, False)),
    "192 x 256, turned": ([385, 193, 64, 128, 17, 130, 192, 65], 1, 192, 24576, (4, True, True)),
    "192 x 256, 8 rounds": ([385, 193, 64, 128, 17, 130, 192, 65], 2, 192, 24576, (8, True, True)),
    "128 x 512, several tiles": ([384, 300, 0, 0, 0, 17, 0, 0], 4, 128, 11264, (2, True, False)),
    "128 x 512, nearly one tile each": ([129, 128, 64, 17, 1, 65, 100, 90], 4, 128, 8704, (2, True, False)),
    "128 x 512, nearly one tile each, whole": ([129, 128, 64, 17, 1, 65, 100, 90], 4, 128, 13824, (3, False, False)),
    "128 x 512, turned": ([300, 0, 17, 129, 64, 1, 200, 30], 2, 128, 24576, (4, True, True)),
    "128 x 512, 8 rounds": ([300, 0, 17, 129, 64, 1, 200, 30], 4, 128, 25600, (8, True, True)),
}


def short_side(tile_rows):
    return 4352 if tile_rows == 128 else 2048


def long_branch(name, up, cus=256):
    counts, repeats, tile_rows, long, _ = ROUNDS[name]
    return gg_schedule.branch(counts * repeats, tile_rows, 512 if tile_rows == 128 else 256, long,
                              short_side(tile_rows) // 32, up, cus)


@pytest.mark.parametrize("long_side", ["f", "d"])  # many tiles in the first / second projection
@pytest.mark.parametrize("name", list(ROUNDS))
def test_rounds_of_whole_tiles_and_pieces(name, long_side):
    import paper_2402_07033_amd as moe
    counts, repeats, tile_rows, long, want = ROUNDS[name]
    counts = counts * repeats
    E, N = len(counts), sum(counts)
    short = short_side(tile_rows)
    d, f = (short, long // 2) if long_side == "f" else (long, short)
    features = 512 if tile_rows == 128 else 256
    tiles = moe.moe_expert_ffn_tiles(counts, d, f, path=moe.MOE_FFN_GROUPED)
    t = tiles["up" if long_side == "f" else "down"]
    assert (t["rows"], t["features"], bool(t["pieces"])) == (tile_rows, features, want[1])
    b = long_branch(name, long_side == "f", torch.cuda.get_device_properties(0).multi_processor_count)
    assert (b.rounds, b.cut, b.turned) == want and b.left > 0 and len(b.once | b.shared) > 1

    g = torch.Generator(device="cuda")
    g.manual_seed(4700 + N)
    normal = lambda *s: torch.randn(s, device="cuda", generator=g)  # noqa: E731
    w1, w3 = ((normal(E, d, f) * d ** -0.5).to(torch.bfloat16) for _ in range(2))
    w2 = (normal(E, f, d) * f ** -0.5).to(torch.bfloat16)
    xg = normal(N, d).to(torch.bfloat16)
    bounds = [0]
    for n in counts:
        bounds.append(bounds[-1] + n)
    off = torch.tensor(bounds, dtype=torch.int32, device="cuda")
    W, scratch = moe.moe_weights_pack(w1, w3, w2), Scratch(N, E, d, f)
    buf = torch.full((N + 16, d), float("nan"), device="cuda")
    moe.moe_expert_ffn(W, xg, off, workspace=scratch.ws, yg=buf[:N], path=moe.MOE_FFN_GROUPED)
    torch.cuda.synchronize()
    assert bool(torch.isnan(buf[N:]).all()), "a store behind the last row"
    assert scratch.pieces() == any(t["pieces"] for t in tiles.values())
    # every row in 64 bits, h rounded to bf16 as the kernels do
    worst = 0.0
    for e in range(E):
        lo, hi = bounds[e], bounds[e + 1]
        if lo == hi:
            continue
        x = xg[lo:hi].double()
        h = torch.nn.functional.silu(x @ w1[e].double()) * (x @ w3[e].double())
        ref = h.to(torch.bfloat16).double() @ w2[e].double()
        err = (buf[lo:hi].double() - ref).norm(dim=1) / ref.norm(dim=1)
        assert bool(torch.isfinite(err).all())
        worst = max(worst, float(err.max()))
    print(f"{name}, long {long_side}: {b.rounds} rounds, {b.left} tiles left, error {worst:.2e}")
    # 2-norm of a row.  An h whose fp32 value (relative error about 2^-20: sums of 2048 and more
    # products) lies that close to a rounding boundary of bf16 rounds the other way and moves by 2^-7
    # of itself at most, about one in 2^11.  The largest h of a row of 2048 has about half of the row's
    # norm, so two of that size move yg by less than 8e-3 of its norm; one step's operands from the
    # wrong tile move it by 1/sqrt(steps), 0.04 and more.
    assert worst <= 8e-3
    W.free()

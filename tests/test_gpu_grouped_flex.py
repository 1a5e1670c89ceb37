"""Grouped GEMM's tiles of up to 160 rows x 4..32 fragment rows (csrc/moe_gg_sched.h, gg_flex) at the edges of their token blocks, full and narrowed rounds, both sides of the rule, and the row count beside the line."""
import pytest
import torch

from test_grouped_flex import L, feature_tiles  # noqa: F401

pytestmark = pytest.mark.gpu

EDGE = [160, 129, 1, 96, 65, 33, 16, 128]   # every copy of the step loop: 1..4, 5..6, 7..8, 9..10 blocks
CASES = {
    # rows per expert, d, f, then per projection: feature tiles of an expert (0: the launch's own tiles)
    "128 x 512 launch, better cut": (EDGE, 2048, 2048, 0, 0),
    "128 x 512 launch, narrowed": (EDGE * 4, 2048, 1280, 8, 8),
    "128 x 512 launch, two rounds": (EDGE * 8, 2048, 1536, 8, 4),
    "128 x 512 launch, reductions too short to cut": (EDGE * 8, 1024, 1024, 4, 4),
    "128 x 512 launch, small matrices": (EDGE * 4, 512, 1024, 0, 0),
    "128 x 512 launch, empty experts": ([0, 160, 0, 0, 17, 0, 1, 0] * 8, 2048, 1280, 10, 10),
    "192 x 256 launch, narrowed": ([160, 120, 130, 97] * 8, 2048, 1280, 8, 0),
    "192 x 256 launch, full": ([160, 120, 130, 97] * 8, 2048, 2048, 8, 0),
    "192 x 256 launch, second projection": ([160, 120, 130, 97] * 12, 2048, 1280, 5, 5),
    "192 x 256 launch, better cut": ([160, 120, 130, 97], 2048, 2048, 0, 0),
    "256 x 256 launch, 11 half tiles": ([28, 30, 160, 1] * 16, 2048, 1408, 8, 4),
    "256 x 256 launch, second projection": ([28, 30, 160, 1] * 12, 2304, 1280, 5, 5),
    "128 x 512 launch, experts of several tiles": ([161, 320, 16, 17, 90, 0, 0, 100] * 3, 2048, 2560, 10, 10),
    "128 x 512 launch, 64 experts, skewed": ([480, 170, 40, 20, 9, 3, 1, 0] * 8, 1024, 1536, 6, 3),
    "161 rows": ([161, 120, 130, 97] * 8, 2048, 1280, 0, 0),
}


def planned(L, counts, d, f, up, only_wide, wgs):  # noqa: F811
    """Feature tiles of an expert, 0 for the launch's own tiles."""
    E, N, n_tok = len(counts), sum(counts), sum(-(-n // 160) for n in counts)
    KS, FR = (d // 32, f // 8) if up else (f // 32, d // 16)
    if E * FR * KS < 128 << 10:  # the projection's weights in KiB: they stay in the last-level cache
        return 0
    if up and N <= 96 * E:
        slim = KS <= 128 and feature_tiles(L, 33 * E, E, FR // 4, wgs, KS, up, False)
        return L.fill(n_tok, FR // 4, wgs) if slim else 0
    if N > 160 * E or (only_wide and max(counts) > 160):
        return 0
    tiles = [feature_tiles(L, N, n, FR // 4, wgs, KS, up, only_wide)
             for n in [n_tok, *range(E, E + (0 if only_wide else N // 160) + 1)]]
    return tiles[0] if any(tiles[1:]) else 0  # (the host takes the kernel that holds both if it expects them)


@pytest.mark.parametrize("name", list(CASES))
def test_small_experts(L, name):  # noqa: F811
    import paper_2402_07033_amd as moe
    counts, d, f, *want = CASES[name]
    E, N = len(counts), sum(counts)
    plan = moe.moe_expert_ffn_plan(N, E, d, f, path=moe.MOE_FFN_GROUPED)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for up, w in zip((1, 0), want):
        only_wide = plan["up_tile_features" if up else "down_tile_features"] == 256
        NT = planned(L, counts, d, f, up, only_wide, (cus + 7) // 8)
        assert cus != 256 or NT == w, (up, NT)

    g = torch.Generator(device="cuda")
    g.manual_seed(5100 + N)
    normal = lambda *s: torch.randn(s, device="cuda", generator=g)  # noqa: E731
    w1, w3 = ((normal(E, d, f) * d ** -0.5).to(torch.bfloat16) for _ in range(2))
    w2 = (normal(E, f, d) * f ** -0.5).to(torch.bfloat16)
    xg = normal(N, d).to(torch.bfloat16)
    bounds = [0]
    for n in counts:
        bounds.append(bounds[-1] + n)
    off = torch.tensor(bounds, dtype=torch.int32, device="cuda")
    W = moe.moe_weights_pack(w1, w3, w2)
    bufs = []
    for _ in range(2):
        buf = torch.full((N + 16, d), float("nan"), device="cuda")
        moe.moe_expert_ffn(W, xg, off, yg=buf[:N], path=moe.MOE_FFN_GROUPED)
        torch.cuda.synchronize()
        bufs.append(buf)
    assert bool(torch.isnan(bufs[0][N:]).all()), "a store behind the last row"
    assert torch.equal(bufs[0][:N], bufs[1][:N])
    worst = 0.0
    for e in range(E):
        lo, hi = bounds[e], bounds[e + 1]
        if lo == hi:
            continue
        x = xg[lo:hi].double()
        h = torch.nn.functional.silu(x @ w1[e].double()) * (x @ w3[e].double())
        ref = h.to(torch.bfloat16).double() @ w2[e].double()
        err = (bufs[0][lo:hi].double() - ref).norm(dim=1) / ref.norm(dim=1)
        assert bool(torch.isfinite(err).all())
        worst = max(worst, float(err.max()))
    print(f"{name}: error {worst:.2e}")
    # 2-norm of a row: an h close to a rounding boundary of bf16 rounds the other way and moves by 2^-7 of itself at
    # most, about one in 2^11; the largest h of a row of 1024 and more has less than 0.6 of the row's norm, so two
    # of that size move yg by less than 1e-2 of its norm.  One step's operands from the wrong tile move it by
    # 1 / sqrt(steps), 0.08 and more.
    assert worst <= 1e-2
    W.free()

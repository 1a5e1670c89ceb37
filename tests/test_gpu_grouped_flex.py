"""Grouped GEMM's tiles of up to 160 rows x 12..32 fragment rows (csrc/moe_gg_sched.h, gg_small_tiles) at the edges of their token
blocks, full and narrowed rounds, both sides of the rule, and the row count beside the line."""
import pytest
import torch

from gpu_util import Scratch

pytestmark = pytest.mark.gpu

EDGE = [160, 129, 1, 96, 65, 33, 16, 128]   # every copy of the step loop: 1..4, 5..6, 7..8, 9..10 blocks
CASES = {
    # rows per expert, d, f, then per projection: feature tiles of an expert (0: the launch's own tiles)
    "128 x 512 launch, better cut": (EDGE, 2048, 2048, 0, 0),
    "128 x 512 launch, narrowed": (EDGE * 4, 2048, 1280, 8, 0),
    "128 x 512 launch, narrowed, one tile each": ([128, 97, 1, 96, 65, 33, 16, 17] * 4, 2048, 1280, 8, 8),
    "128 x 512 launch, two rounds": (EDGE * 8, 2048, 1536, 8, 4),
    "128 x 512 launch, reductions too short to cut": (EDGE * 8, 1024, 1024, 4, 0),
    "128 x 512 launch, small matrices": (EDGE * 4, 512, 1024, 0, 0),
    "128 x 512 launch, empty experts": ([0, 160, 0, 0, 17, 0, 1, 0] * 8, 2048, 1280, 10, 0),
    "192 x 256 launch, narrowed": ([160, 120, 130, 97] * 8, 2048, 1280, 8, 0),
    "192 x 256 launch, full": ([160, 120, 130, 97] * 8, 2048, 2048, 8, 0),
    "192 x 256 launch, second projection": ([160, 120, 130, 97] * 12, 2048, 1280, 5, 5),
    "192 x 256 launch, better cut": ([160, 120, 130, 97], 2048, 2048, 0, 0),
    "256 x 256 launch, 11 half tiles": ([28, 30, 160, 1] * 16, 2048, 1408, 8, 4),
    "256 x 256 launch, second projection": ([28, 30, 160, 1] * 12, 2304, 1280, 5, 5),
    "128 x 512 launch, experts of several tiles": ([161, 320, 16, 17, 90, 0, 0, 100] * 3, 2048, 2560, 10, 10),
    "128 x 512 launch, 64 experts, skewed": ([480, 170, 40, 20, 9, 3, 1, 0] * 8, 1024, 1536, 6, 0),
    "161 rows": ([161, 120, 130, 97] * 8, 2048, 1280, 0, 0),
    "256 x 256 launch, second projection, 161 rows": ([28, 30, 161, 1] * 10, 2304, 2560, 10, 0),
}


def layer(E, d, f, N, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    normal = lambda *s: torch.randn(s, device="cuda", generator=g)  # noqa: E731
    w1, w3 = ((normal(E, d, f) * d ** -0.5).to(torch.bfloat16) for _ in range(2))
    w2 = (normal(E, f, d) * f ** -0.5).to(torch.bfloat16)
    return w1, w3, w2, normal(N, d).to(torch.bfloat16)


def bounds_of(counts):
    bounds = [0]
    for n in counts:
        bounds.append(bounds[-1] + n)
    return bounds


def worst_row(yg, xg, bounds, w1, w3, w2):
    """Largest error of a row, 2-norm over 2-norm, against 64 bits with h rounded to bf16."""
    worst = 0.0
    for e in range(len(bounds) - 1):
        lo, hi = bounds[e], bounds[e + 1]
        if lo == hi:
            continue
        x = xg[lo:hi].double()
        h = torch.nn.functional.silu(x @ w1[e].double()) * (x @ w3[e].double())
        ref = h.to(torch.bfloat16).double() @ w2[e].double()
        err = (yg[lo:hi].double() - ref).norm(dim=1) / ref.norm(dim=1)
        assert bool(torch.isfinite(err).all())
        worst = max(worst, float(err.max()))
    return worst


@pytest.mark.parametrize("name", list(CASES))
def test_small_experts(name):
    import paper_2402_07033_amd as moe
    counts, d, f, *want = CASES[name]
    E, N = len(counts), sum(counts)
    tiles = moe.moe_expert_ffn_tiles(counts, d, f, path=moe.MOE_FFN_GROUPED)
    small = [t["feature_tiles"] if t["rows"] == 160 else 0 for t in (tiles["up"], tiles["down"])]
    assert torch.cuda.get_device_properties(0).multi_processor_count != 256 or small == want

    w1, w3, w2, xg = layer(E, d, f, N, 5100 + N)
    bounds = bounds_of(counts)
    off = torch.tensor(bounds, dtype=torch.int32, device="cuda")
    W, scratch = moe.moe_weights_pack(w1, w3, w2), Scratch(N, E, d, f)
    bufs = []
    for _ in range(2):
        buf = torch.full((N + 16, d), float("nan"), device="cuda")
        moe.moe_expert_ffn(W, xg, off, workspace=scratch.ws, yg=buf[:N], path=moe.MOE_FFN_GROUPED)
        torch.cuda.synchronize()
        bufs.append(buf)
    assert bool(torch.isnan(bufs[0][N:]).all()), "a store behind the last row"
    assert torch.equal(bufs[0][:N], bufs[1][:N])
    # the device went the way that the host's query says
    assert scratch.pieces() == bool(tiles["up"]["pieces"] or tiles["down"]["pieces"])
    worst = worst_row(bufs[0], xg, bounds, w1, w3, w2)
    print(f"{name}: error {worst:.2e}")
    # 2-norm of a row: an h close to a rounding boundary of bf16 rounds the other way and moves by 2^-7 of itself at
    # most, about one in 2^11; the largest h of a row of 1024 and more has less than 0.6 of the row's norm, so two
    # of that size move yg by less than 1e-2 of its norm.  One step's operands from the wrong tile move it by
    # 1 / sqrt(steps), 0.08 and more.
    assert worst <= 1e-2
    W.free()


# Few experts in use: the second projection (fewer than 64 steps) is never cut, so pieces are the first's.
FEW = [
    # rows of the experts in use, f, experts, are there pieces
    ([90], 1536, 16, True),         # 16 narrow tiles for all CUs
    ([24] * 8, 1536, 16, True),
    ([24] * 12, 1536, 16, False),   # 192 of them
    ([90] * 16, 1536, 16, False),
    ([150], 1536, 16, True),        # two of the launch's token tiles in place of one
    ([150] * 8, 1536, 16, False),   # ... and matrices that the last-level cache does not keep
    ([24] * 6, 1408, 32, True),     # tiles of 256 features, as wide as the narrow ones
    ([90] * 24, 1408, 32, False),
    ([90] * 37, 1792, 64, True),    # a round of the launch's own tiles, and three of the next
    ([60] * 37, 1792, 64, False),
]


@pytest.mark.parametrize("rows,f,E,pieces", FEW)
def test_few_experts_in_use(rows, f, E, pieces):
    import paper_2402_07033_amd as moe
    d, N, counts = 4096, sum(rows), rows + [0] * (E - len(rows))
    w1, w3, w2, xg = layer(E, d, f, N, 5300 + N)
    bounds = bounds_of(counts)
    W, scratch = moe.moe_weights_pack(w1, w3, w2), Scratch(N, E, d, f)
    buf = torch.full((N + 16, d), float("nan"), device="cuda")
    tiles = moe.moe_expert_ffn_tiles(counts, d, f, path=moe.MOE_FFN_GROUPED)
    moe.moe_expert_ffn(W, xg, torch.tensor(bounds, dtype=torch.int32, device="cuda"), workspace=scratch.ws, yg=buf[:N],
                       path=moe.MOE_FFN_GROUPED)
    torch.cuda.synchronize()
    assert bool(torch.isnan(buf[N:]).all()), "a store behind the last row"
    assert worst_row(buf, xg, bounds, w1, w3, w2) <= 1e-2  # (as above)
    assert scratch.pieces() == bool(tiles["up"]["pieces"]) and not tiles["down"]["pieces"]
    assert torch.cuda.get_device_properties(0).multi_processor_count != 256 or scratch.pieces() == pieces
    W.free()


def test_fewer_experts_than_a_token_has():
    """Without a fix-up launch, since every token has two experts, and then all rows are one expert's: nothing is cut."""
    import paper_2402_07033_amd as moe
    E, d, f, T, k = 8, 4096, 8192, 73, 2
    N = T * k
    assert not moe.moe_expert_ffn_tiles([N] + [0] * 7, d, f, k=k)["up"]["fixup"]
    assert moe.moe_expert_ffn_tiles([N] + [0] * 7, d, f)["up"]["pieces"]
    w1, w3, w2, x = layer(E, d, f, T, 5400)
    bounds = bounds_of([0, 0, N, 0, 0, 0, 0, 0])
    W, perm = moe.moe_weights_pack(w1, w3, w2), torch.arange(N, dtype=torch.int32, device="cuda")
    buf = torch.full((N + 16, d), float("nan"), device="cuda")
    moe.moe_expert_ffn_tokens(W, x, k, perm, torch.tensor(bounds, dtype=torch.int32, device="cuda"), yg=buf[:N])
    torch.cuda.synchronize()
    assert bool(torch.isnan(buf[N:]).all())
    assert worst_row(buf, x.repeat_interleave(k, dim=0), bounds, w1, w3, w2) <= 1e-2
    W.free()

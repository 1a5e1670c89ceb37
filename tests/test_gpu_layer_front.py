"""moe_layer's routing and batching in one launch (up to 512 slots, a workgroup per token, few passes): the bits of the two
calls at the edges of its groups of lanes and slots, on both sides of its limit, and with outputs over its inputs."""
import ctypes as C

import pytest
import torch

import moe_inputs as mi
from gpu_util import pack_layer, to_dev

pytestmark = pytest.mark.gpu


# One launch: 1, 2, 4, 8 and 64 lanes per token; 64 slots and one more, groups that end inside a token, 512 slots, as many tokens
# as CUs; three passes of the workgroup over the tokens; fewer logits than experts; rows of 256 B, and longer than one request of a
# wave (8 KiB).  Two: the first slots beyond 512, one token more than CUs, a fourth pass, two passes of 64 lanes.
@pytest.mark.parametrize("T,E,EL,k,d,w,x", [
    (1, 1, 1, 1, 64, mi.F32, mi.F32), (16, 8, 8, 2, 256, mi.F32, mi.F32), (64, 2, 2, 1, 64, mi.F32, mi.F32),
    (65, 3, 3, 1, 64, mi.F32, mi.F32), (8, 64, 64, 8, 256, mi.BF16, mi.BF16), (8, 64, 33, 8, 256, mi.BF16, mi.F32),
    (128, 4, 4, 4, 64, mi.F32, mi.F32), (256, 2, 2, 2, 64, mi.F32, mi.F32), (192, 8, 8, 2, 64, mi.F32, mi.F32),
    (29, 16, 9, 7, 64, mi.F32, mi.F32), (5, 4, 3, 2, 2112, mi.F32, mi.F32),
    (129, 4, 4, 4, 64, mi.F32, mi.F32), (257, 4, 4, 1, 64, mi.F32, mi.F32), (193, 8, 8, 2, 64, mi.F32, mi.F32),
    (9, 64, 64, 8, 256, mi.BF16, mi.BF16)])
def test_layer_front(T, E, EL, k, d, w, x):
    import paper_2402_07033_amd as moe
    cfg = mi.small_config("front", T, d, 128, E, k, 30 + T + E, w_dtype=w, x_dtype=x, zipf_s=1.2)
    li = mi.make_layer(cfg, threads=4)
    W, xd, lg = pack_layer(li), to_dev(li.x), to_dev(li.logits)[:, :EL].contiguous()
    lg[0].fill_(0.5)  # ties go to the lower expert
    if EL > 2:
        lg[T // 2, 1] = float("-inf")
    path = moe.MOE_FFN_AUTO if w == mi.F32 else moe.MOE_FFN_MID
    out = moe.moe_layer(W, xd, lg, k, path=path)
    idx, wt = moe.moe_route(lg, k)
    counts, offsets, perm, inv_perm, xg = moe.moe_permute(idx, E, xd)
    y = moe.moe_combine(moe.moe_expert_ffn(W, xg, offsets, path=path), inv_perm, wt)
    want = dict(idx=idx, w=wt, counts=counts, offsets=offsets, perm=perm, inv_perm=inv_perm, xg=xg, y=y)
    for n, v in want.items():
        assert torch.equal(out[n], v), n
    W.free()


def call(W, xd, lg, T, E, k, d, over=None, guard=0):
    """moe_layer on buffers of the caller's (logits in `over`'s memory), with `guard` rows behind xg."""
    import paper_2402_07033_amd as moe
    N = T * k
    i32 = dict(dtype=torch.int32, device="cuda")
    bufs = dict(idx=torch.empty(N, **i32), w=torch.empty(N, device="cuda"), counts=torch.empty(E, **i32),
                offsets=torch.empty(E + 1, **i32), perm=torch.empty(T * E, **i32), inv_perm=torch.empty(N, **i32),
                xg=torch.full((N + guard, d), float("nan"), device="cuda"), yg=torch.empty((N, d), device="cuda"),
                y=torch.empty((T, d), device="cuda"))
    ws = torch.empty(moe.moe_expert_ffn_workspace(N, E, d, 128, moe.MOE_F32), dtype=torch.uint8, device="cuda")
    logits = lg
    if over:
        logits = bufs[over].reshape(-1).view(torch.float32)[:T * E]
        logits.copy_(lg.reshape(-1))
    p = {n: t.data_ptr() for n, t in bufs.items()}
    stage = C.c_int(-1)
    torch.cuda.synchronize()
    rc = moe.lib().moe_layer(W.handle, xd.data_ptr(), moe.MOE_F32, d, logits.data_ptr(), T, E, k, moe.MOE_FFN_AUTO,
                             p["idx"], p["w"], p["counts"], p["offsets"], p["perm"], p["inv_perm"], p["xg"],
                             ws.data_ptr(), ws.numel(), p["yg"], p["y"], C.byref(stage), None)
    torch.cuda.synchronize()
    assert rc == 0
    return bufs


@pytest.mark.parametrize("over", ["xg", "perm"])
def test_outputs_over_the_logits(over):
    """The logits are dead once the tokens are routed: an output of the batching may lie over them."""
    import paper_2402_07033_amd as moe
    T, E, k, d = 16, 8, 2, 256
    cfg = mi.small_config("front", T, d, 128, E, k, 77)
    li = mi.make_layer(cfg, threads=4)
    W, xd, lg = pack_layer(li), to_dev(li.x), to_dev(li.logits)
    want = moe.moe_layer(W, xd, lg, k)
    bufs = call(W, xd, lg, T, E, k, d, over)
    for n in ("idx", "w", "counts", "offsets", "inv_perm", "xg", "yg", "y"):
        assert torch.equal(bufs[n].reshape(-1), want[n].reshape(-1)), n
    assert torch.equal(bufs["perm"][:T * k], want["perm"])
    W.free()


# One launch and (over) the two: NaN in the first, the last and all of a token's logits, beside -inf, and in every token.
@pytest.mark.parametrize("over", [None, "perm"])
@pytest.mark.parametrize("T,E,k", [(16, 8, 2), (9, 5, 3), (1, 8, 8)])
def test_nan_logits(T, E, k, over):
    """A NaN logit is compared with nothing: its token's ids may be none, which count as the last expert's, and every
    slot still has a row of its own."""
    import paper_2402_07033_amd as moe
    d, N = 256, T * k
    cfg = mi.small_config("front", T, d, 128, E, k, 90 + T)
    li = mi.make_layer(cfg, threads=4)
    W, xd, lg = pack_layer(li), to_dev(li.x), to_dev(li.logits)
    nan = float("nan")
    lg[0, 0] = nan
    lg[T // 2] = nan
    lg[T - 1, 1:] = float("-inf")
    lg[T - 1, E - 1] = nan
    lg[::3, 2] = nan
    bufs = call(W, xd, lg, T, E, k, d, over, guard=4)
    idx, wt = moe.moe_route(lg, k)
    counts, offsets, perm, inv_perm, xg = moe.moe_permute(idx, E, xd)
    assert torch.equal(bufs["idx"], idx.reshape(-1))
    assert torch.equal(torch.nan_to_num(bufs["w"], nan=-1.0), torch.nan_to_num(wt.reshape(-1), nan=-1.0))
    for n, v in dict(counts=counts, offsets=offsets, inv_perm=inv_perm).items():
        assert torch.equal(bufs[n], v), n
    assert torch.equal(bufs["perm"][:N], perm) and torch.equal(bufs["xg"][:N], xg)
    assert bool(torch.isnan(bufs["xg"][N:]).all()), "a row behind the last one"
    assert sorted(perm.tolist()) == list(range(N)) and int(offsets[E]) == N
    W.free()

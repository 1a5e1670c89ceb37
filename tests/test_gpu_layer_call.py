"""moe_layer, the four calls in one: the bits of the four calls, and the error of the one that fails."""
import pytest
import torch

import moe_inputs as mi
from gpu_util import pack_layer, to_dev

pytestmark = pytest.mark.gpu


def _layer(T, E, k, w, x):
    cfg = mi.small_config("layer_call", T, 256, 512, E, k, 70 + T, w_dtype=w, x_dtype=x, zipf_s=1.2)
    li = mi.make_layer(cfg, threads=4)
    return pack_layer(li), to_dev(li.x), to_dev(li.logits)


# all-fp32; decode sized; the grouped kernels with either row type
@pytest.mark.parametrize("T,E,k,w,x", [(1, 8, 2, mi.F32, mi.F32), (16, 8, 2, mi.F32, mi.F32), (7, 16, 4, mi.BF16, mi.F32),
                                       (300, 8, 2, mi.BF16, mi.BF16), (301, 3, 1, mi.BF16, mi.F32)])
def test_layer_is_the_four_calls(T, E, k, w, x):
    import paper_2402_07033_amd as moe
    W, xd, lg = _layer(T, E, k, w, x)
    out = moe.moe_layer(W, xd, lg, k)
    idx, wt = moe.moe_route(lg, k)
    counts, offsets, perm, inv_perm, xg = moe.moe_permute(idx, E, xd)
    yg = moe.moe_expert_ffn(W, xg, offsets)
    y = moe.moe_combine(yg, inv_perm, wt)
    want = dict(idx=idx, w=wt, counts=counts, offsets=offsets, perm=perm, inv_perm=inv_perm, xg=xg, yg=yg, y=y)
    assert set(out) == set(want)
    for n, v in want.items():
        assert out[n].dtype == v.dtype and torch.equal(out[n], v), n
    W.free()


def test_layer_names_the_call_that_failed():
    import paper_2402_07033_amd as moe
    W, xd, lg = _layer(8, 8, 2, mi.BF16, mi.F32)
    with pytest.raises(moe.MoeError, match="moe_route"):
        moe.moe_layer(W, xd, lg, 9)
    with pytest.raises(moe.MoeError, match="moe_expert_ffn"):
        moe.moe_layer(W, xd, lg, 2, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    with pytest.raises(TypeError):
        moe.moe_layer(W, xd.t(), lg, 2)
    W.free()
    with pytest.raises(moe.MoeError, match="moe_expert_ffn"):
        moe.moe_layer(W, xd, lg, 2)


@pytest.mark.parametrize("k", [9, 300, 0, -1])
def test_refused_k_allocates_no_rows(k):
    """The call that refuses is the router's, at the router's price: T*k indices and weights."""
    import paper_2402_07033_amd as moe
    W, xd, lg = _layer(64, 8, 2, mi.BF16, mi.F32)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    with pytest.raises(RuntimeError if k < 0 else moe.MoeError, match=None if k < 0 else "moe_route"):
        moe.moe_layer(W, xd, lg, k)
    assert torch.cuda.max_memory_allocated() - before <= 2 * (64 * max(k, 0) * 4 + 512)
    W.free()


def test_layer_sizes_that_do_not_fit():
    """Fewer rows than logits, another row length, more logits than experts: refused.  More rows than
    logits (the first T are used) and fewer logits than experts are ordinary calls."""
    import paper_2402_07033_amd as moe
    W, xd, lg = _layer(64, 8, 2, mi.BF16, mi.F32)
    for x, logits in ((xd[:63], lg), (xd[:, :192].contiguous(), lg), (torch.cat([xd, xd], dim=1), lg),
                      (xd, torch.cat([lg, lg[:, :1]], dim=1))):
        with pytest.raises(moe.MoeError, match="moe_permute"):
            moe.moe_layer(W, x, logits, 2)
    five = lg[:37, :5].contiguous()
    out = moe.moe_layer(W, xd, five, 2)
    want = moe.moe_layer(W, xd[:37].contiguous(), five, 2)
    assert all(torch.equal(out[n], want[n]) for n in want)
    assert (out["counts"][5:] == 0).all() and int(out["offsets"][-1]) == 74
    idx, w = moe.moe_route(five, 2)
    _, offsets, _, inv_perm, xg = moe.moe_permute(idx, 8, xd[:37])
    assert torch.equal(out["y"], moe.moe_combine(moe.moe_expert_ffn(W, xg, offsets), inv_perm, w))
    W.free()


def test_refused_layer_has_enqueued_nothing():
    import ctypes as C

    import paper_2402_07033_amd as moe
    W, xd, lg = _layer(8, 8, 2, mi.BF16, mi.F32)
    T, E, k, N = 8, 8, 2, 16
    idx, counts, perm, inv_perm = (torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (N, E, N, N))
    offsets = torch.full((E + 1,), -7, dtype=torch.int32, device="cuda")
    w, xg, yg, y = (torch.full(s, -7.0, device="cuda") for s in ((N,), (N, 256), (N, 256), (T, 256)))
    ws = torch.empty(moe.moe_expert_ffn_workspace(N, E, 256, 512, moe.MOE_F32), dtype=torch.uint8, device="cuda")
    stage = C.c_int(-1)
    for ws_bytes, y_ptr, want in ((ws.numel() - 1, y.data_ptr(), (-3, 2)), (ws.numel(), y.data_ptr() + 4, (-1, 3))):
        rc = moe.lib().moe_layer(W.handle, xd.data_ptr(), moe.MOE_F32, 256, lg.data_ptr(), T, E, k, moe.MOE_FFN_AUTO,
                                 idx.data_ptr(), w.data_ptr(), counts.data_ptr(), offsets.data_ptr(), perm.data_ptr(),
                                 inv_perm.data_ptr(), xg.data_ptr(), ws.data_ptr(), ws_bytes, yg.data_ptr(), y_ptr,
                                 C.byref(stage), None)
        torch.cuda.synchronize()
        assert (rc, stage.value) == want
        for t in (idx, counts, offsets, perm, inv_perm, w, xg, yg, y):
            assert (t == -7).all()
    W.free()

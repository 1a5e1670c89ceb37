"""moe_permute where its launch changes: one token per workgroup and several, groups of 64 slots
that end inside a token, 4096 slots (from there the first rows are requested before the slots are counted), 15 tokens per CU
(with more the rows go past L2; 3840 | 3841 on 256 CUs), slots beyond what a workgroup keeps for the row copy (the copy is
then a launch of its own), rows that are no multiple of the copy's 8 KiB, expert ids out of range."""
import numpy as np
import pytest

import moe_inputs as mi
from gpu_util import to_dev, to_host
from oracle import moe_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k,d,xdt", [
    (1, 1, 1, 64, "bf16"), (255, 8, 2, 4160, "f32"), (256, 64, 8, 64, "bf16"), (257, 64, 7, 2112, "f32"),
    (2500, 3, 3, 64, "f32"), (2047, 8, 2, 4160, "f32"), (2049, 8, 2, 4160, "f32"), (3840, 8, 2, 2112, "bf16"), (3841, 8, 2, 2112, "bf16"), (4099, 5, 1, 64, "bf16"), (4099, 8, 2, 4160, "f32"), (32768, 16, 8, 64, "bf16"), (33000, 16, 8, 64, "f32")])
def test_permute_at_launch_edges(T, E, k, d, xdt):
    import paper_2402_07033_amd as moe
    rng = np.random.default_rng(T + E)
    idx = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    x32 = mi.normal_f32(700 + T, 0, (T, d))
    x = mi.f32_to_bf16_bits(x32) if xdt == "bf16" else x32
    rc, ro, rp, ri, _ = orc.permute(idx, E, np.zeros((T, 1)))
    c, o, p, ip, xg = moe.moe_permute(to_dev(idx), E, to_dev(x))
    assert (to_host(c) == rc).all() and (to_host(o) == ro).all()
    assert (to_host(p) == rp).all() and (to_host(ip) == ri).all()
    assert (to_host(xg) == x[rp // k]).all()
    c, o, p, ip, _ = moe.moe_permute(to_dev(idx), E, None)
    assert (to_host(o) == ro).all() and (to_host(p) == rp).all() and (to_host(ip) == ri).all()


def test_permute_clamps_expert_ids():
    import paper_2402_07033_amd as moe
    idx = np.array([[-3, 2], [7, 100], [0, 1], [5, -1]], dtype=np.int32)
    rc, ro, rp, ri, _ = orc.permute(np.clip(idx, 0, 5), 6, np.zeros((4, 1)))
    c, o, p, ip, _ = moe.moe_permute(to_dev(idx), 6, None)
    assert (to_host(c) == rc).all() and (to_host(o) == ro).all()
    assert (to_host(p) == rp).all() and (to_host(ip) == ri).all()

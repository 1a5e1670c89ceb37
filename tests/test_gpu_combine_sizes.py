"""moe_combine on either side of the size from which its rows go past L2 (y of 32 MiB), row
lengths, against the sum in fp64: k products and sums in fp32, each rounded by 2^-24 of what was added."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,k", [(2048, 4096, 2), (2049, 4096, 2), (3, 4160, 8), (65600, 192, 1)])
def test_combine_sizes(T, d, k):
    import paper_2402_07033_amd as moe
    g = torch.Generator(device="cuda").manual_seed(T + d)
    yg = torch.empty((T * k, d), device="cuda").normal_(generator=g)
    w = torch.rand((T, k), device="cuda", generator=g)
    inv = torch.randperm(T * k, device="cuda", generator=g).to(torch.int32)
    buf = torch.full((T + 1, d), float("nan"), device="cuda")
    y = moe.moe_combine(yg, inv, w, buf[:T])
    rows = yg.double()[inv.long()].reshape(T, k, d) * w.double()[:, :, None]
    bound = 2.0 ** -24 * (k + 1) * rows.abs().sum(dim=1)
    assert ((y.double() - rows.sum(dim=1)).abs() <= bound).all()
    assert torch.isnan(buf[T:]).all(), "a store behind the last row"

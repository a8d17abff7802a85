"""The orientation stencil's two tilings give the same map, bit for bit: single
images take small tiles where large ones would leave compute units idle, a
batch takes large ones, and both sum the taps of a pixel in the same order.
Sides that are no multiple of either tile or of 16; small and large
stencils; the side at the line between the tilings."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sigma", [1.5, 2.0, 4.0, 5.0])
@pytest.mark.parametrize("M", [16, 24, 64, 72, 216, 648, 1024])
def test_small_and_large_tiles_agree(M, sigma):
    from paper_1304_2062_amd import se2n
    print(f"orient tiles {M} {sigma}", flush=True)
    N = 12
    g = torch.Generator().manual_seed(M)
    f = torch.rand(M, M, generator=g).cuda()
    mask = (torch.rand(M, M, generator=g) < 0.4).to(torch.uint8).cuda()
    plan = se2n.Plan(M, N, torch.float32)
    small = plan.orient(f, mask, sigma)
    item = se2n.BatchItem(f, mask, N, 0.5, 1.0, 10, sigma=sigma)
    ws = se2n.batch_workspace([item])
    se2n.inpaint_batched([item], ws)
    assert torch.equal(small, item.rmap_out)
    se2n.batch_clear()
    plan.close()

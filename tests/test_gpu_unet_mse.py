"""The loss over voxel counts around one and several rounds of its workgroups (512 of 256).

Tolerance: a sum of n FP32 products in chains of at most n / 131072 + 1 terms per thread, 6
and 4 pairings and 512 workgroups' sums; each product rounds three times."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("nvox", [1, 255, 257, 131072, 131073, 700001])
def test_loss_and_gradient(hip, nvox, weighted):
    import torch

    from paper_1410_1914_amd import unet as U

    g = torch.Generator("cuda").manual_seed(nvox)
    pred, target = (torch.randn(nvox, generator=g, device="cuda") for _ in range(2))
    mask = (torch.rand(nvox, generator=g, device="cuda") < 0.7).to(torch.uint8)
    mask[0] = 1
    weight = torch.rand(nvox, generator=g, device="cuda") * 4 if weighted else None
    dout, loss, count = torch.full((nvox,), 7.0, device="cuda"), torch.zeros(1, device="cuda"), int(mask.sum())
    U.unet_mse(pred, target, mask, dout, loss, nvox, count, weight)
    torch.cuda.synchronize()
    d = torch.where(mask != 0, pred - target, torch.zeros_like(pred)).double()
    wd = d * (weight.double() if weighted else 1.0)
    want = float((wd * d).sum()) / count
    assert abs(float(loss) - want) <= (nvox // 131072 + 1 + 10 + 512 + 4) * 2.0 ** -24 * want
    assert torch.allclose(dout.double(), 2.0 * wd / count, rtol=4 * 2.0 ** -24, atol=0.0)

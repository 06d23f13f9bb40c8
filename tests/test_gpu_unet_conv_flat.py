"""The 3x3x3 convolution on grids of few rows, whose tiles lie flat: a workgroup's waves side
by side in x.  Values against FP64 products of shifted copies; the head and the masked
backward forms against the layers they are made of; and no slower than the same number of
voxels standing.

Tolerance: as for the other tiles (BF16 rounding of the result, 27 cin FP32 additions)."""
import time

import pytest

import test_gpu_unet_backward as backward
from test_gpu_unet_conv import _check, _data, _reference

pytestmark = pytest.mark.gpu

# rows that end inside the first, second and last wave of a tile, or leave some of them empty
SHAPES = [(1, 1, 65), (5, 2, 130), (9, 4, 79), (7, 8, 64), (13, 3, 17), (6, 20, 193), (70, 4, 260), (160, 8, 300), (90, 7, 513)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("cin,cout", [(16, 16), (48, 16), (16, 32), (32, 32), (64, 64), (32, 48)])
def test_flat_tiles(hip, shape, cin, cout):
    import torch

    from paper_1410_1914_amd import unet as U

    ldx, offx, ldy, offy = cin + 16, 8, cout + 24, 16
    x, w, b = _data(shape, ldx, cin, cout, sum(shape) + cin)
    y = torch.full((x.shape[0], ldy), 7.0, dtype=torch.bfloat16, device="cuda")
    y32 = torch.zeros((x.shape[0], cout), device="cuda")
    U.unet_conv3d_fwd(x, ldx, offx, w, b, y, ldy, offy, y32, shape, cin, cout, True)
    torch.cuda.synchronize()
    ref, mag = _reference(x[:, offx:offx + cin], w, b, shape, True)
    _check(y[:, offy:offy + cout], ref, mag, cin)
    assert torch.equal(y32.bfloat16(), y[:, offy:offy + cout])
    assert (y[:, :offy] == 7).all() and (y[:, offy + cout:] == 7).all()


@pytest.mark.parametrize("shape,c1,c2,cout", [((20, 4, 130), 32, 64, 64), ((40, 8, 200), 16, 32, 16), ((8, 2, 66), 16, 32, 32)])
def test_concatenation(hip, shape, c1, c2, cout):
    import torch

    from paper_1410_1914_amd import unet as U

    nz, ny, nx = shape
    x, w, b = _data(shape, c1, c1 + c2, cout, 5)
    x2 = _data((nz // 2, ny // 2, nx // 2), c2, 16, 16, 6)[0]
    up = x2.view(nz // 2, ny // 2, nx // 2, c2)
    for d in range(3):
        up = up.repeat_interleave(2, d)
    y = torch.zeros((nz * ny * nx, cout), dtype=torch.bfloat16, device="cuda")
    U.unet_conv3d_fwd_cat(x, c1, 0, c1, x2, c2, 0, w, b, y, cout, 0, None, shape, c1 + c2, cout, True)
    torch.cuda.synchronize()
    ref, mag = _reference(torch.cat([x, up.reshape(-1, c2)], 1), w, b, shape, True)
    _check(y, ref, mag, c1 + c2)


@pytest.mark.parametrize("shape", [(1, 4, 70), (160, 8, 300), (50, 3, 100), (300, 4, 513)])
@pytest.mark.parametrize("base", [False, True])
def test_head_is_the_convolution_then_the_head(hip, shape, base):
    import torch

    from paper_1410_1914_amd import unet as U

    x, w, b = _data(shape, 16, 16, 16, 3)
    V = x.shape[0]
    g = torch.Generator("cuda").manual_seed(4)
    hw, hb, add = (torch.randn(n, generator=g, device="cuda") for n in (16, 1, V))
    y, want, got = torch.zeros_like(x), torch.zeros(V, device="cuda"), torch.full((V,), 7.0, device="cuda")
    U.unet_conv3d_fwd(x, 16, 0, w, b, y, 16, 0, None, shape, 16, 16, True)
    U.unet_head_fwd(y, 16, hw, hb, add if base else None, want, V, 16)
    for _ in range(5):
        got.fill_(7.0)
        U.unet_conv3d_fwd_head(x, 16, 0, w, b, hw, hb, add if base else None, got, shape)
        torch.cuda.synchronize()
        assert torch.equal(got, want)


@pytest.mark.parametrize("shape", [(8, 8, 136), (80, 8, 512), (16, 16, 520)])
def test_network(hip, shape):
    import torch

    from paper_1410_1914_amd import unet as U

    backward.test_network_gradient_is_the_chain_of_layers(hip, shape)
    net = U.UNet(seed=3)
    feat = backward._bf((shape[0] * shape[1] * shape[2], 16), 5)
    assert torch.equal(net.forward(feat, shape, train=True), net.forward(feat, shape))


@pytest.mark.parametrize("shape", [(8, 20, 40), (90, 8, 300)])
def test_values_that_are_not_finite_stay_within_reach(hip, shape):
    import torch

    from paper_1410_1914_amd import unet as U

    nz, ny, nx = shape
    x, w, b = _data(shape, 16, 16, 16, 7)
    z, yy, xx = nz // 2, 3, 16
    x[(z * ny + yy) * nx + xx, 1] = float("inf")
    x[-1, 0] = float("nan")
    y = torch.zeros((nz * ny * nx, 16), dtype=torch.bfloat16, device="cuda")
    U.unet_conv3d_fwd(x, 16, 0, w, b, y, 16, 0, None, shape, 16, 16, False)
    torch.cuda.synchronize()
    want = torch.zeros((nz, ny, nx), dtype=torch.bool, device="cuda")
    want[z - 1:z + 2, yy - 1:yy + 2, xx - 1:xx + 2] = True
    want[nz - 2:, ny - 2:, nx - 2:] = True
    assert torch.equal(~torch.isfinite(y.float()).all(1).view(nz, ny, nx), want)


@pytest.mark.parametrize("cin,cout", [(16, 16), (48, 16), (16, 48)])
def test_few_rows_take_about_as_long_as_few_planes(hip, cin, cout):
    import torch

    from paper_1410_1914_amd import unet as U

    us = []
    for shape in ((512, 4, 512), (4, 512, 512)):
        x, w, b = _data(shape, cin, cin, cout, 1)
        y = torch.zeros((x.shape[0], cout), dtype=torch.bfloat16, device="cuda")
        best = float("inf")
        for _ in range(7):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(20):
                U.unet_conv3d_fwd(x, cin, 0, w, b, y, cout, 0, None, shape, cin, cout, True)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        us.append(best * 5e4)
    print(us, flush=True)
    assert us[0] <= 1.5 * us[1]

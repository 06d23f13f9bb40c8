"""The weight gradient on grids that are thin in one direction or very small: values in the
marching form's runs of any number, and no route slower than the general one (inputs off the
16-byte boundaries take that one).

Tolerance: a chain of n FP32 additions is off by at most n 2^-24 of the sum of magnitudes;
the longest here adds the rows of a run, 32 products of an instruction and up to 256 runs."""
import pytest

from test_gpu_unet_wgrad import _data, _reference, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(300, 8, 32), (11, 77, 1), (9, 38, 3), (19, 1, 28), (40, 8, 20), (17, 7, 7), (16, 8, 8), (64, 8, 8), (90, 2, 5), (33, 9, 3),
                                   (20, 5, 4), (1000, 1, 1)])
@pytest.mark.parametrize("cin,cout", [(16, 16), (32, 64)])
def test_values_on_thin_grids(hip, shape, cin, cout):
    x, dy = _data(shape, cin, cout, sum(shape))
    dw, db = _run(x, dy, shape, cin, cout, cin, 0, cout, 0)
    ref, mag = _reference(x, dy, shape)
    n = (8 * 16 + 32 + 256) * 2.0 ** -24
    assert ((dw - ref).abs() <= n * mag).all()
    assert ((db - dy.double().sum(0)).abs() <= n * dy.double().abs().sum(0)).all()


@pytest.mark.parametrize("shape", [(2000, 8, 32), (100, 8, 32), (64, 8, 8), (200, 4, 16), (2000, 1, 1), (1000, 1, 1),
                                   (256, 256, 1), (256, 256, 2), (60, 4, 4), (2000, 1, 8), (500, 2, 6),
                                   (11, 77, 1), (5, 38, 3), (19, 1, 28), (3000, 1, 5), (2000, 3, 5)])
@pytest.mark.parametrize("cin,cout", [(16, 16), (32, 64)])
def test_no_slower_than_the_general_form(hip, shape, cin, cout):
    import time

    import torch

    from paper_1410_1914_amd import unet as U

    x, dy = _data(shape, cin, cout, 1)
    store = torch.zeros(x.numel() + 8, dtype=torch.bfloat16, device="cuda")
    off = store[4:4 + x.numel()].view(x.shape)
    off.copy_(x)
    dw, db = torch.zeros(cout, U.unet_kpad(cin), device="cuda"), torch.zeros(cout, device="cuda")

    def us(a):
        best = float("inf")
        for _ in range(7):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(20):
                U.unet_conv3d_wgrad(a, cin, 0, dy, cout, 0, shape, cin, cout, dw, db)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best * 5e4

    assert us(x) <= 1.35 * us(off)

"""Weight gradient of the 3x3x3 convolution where its tiling can go wrong: rows that end
inside a tile, one plane, several runs of planes per tile, channel slices of wider rows,
inputs that are not finite at the ends of the rows, and inputs off the 16-byte boundaries
(another kernel).  Reference: FP64 products of shifted copies in plain torch.

Tolerance: a sum of n terms added one after another in FP32 is off by at most n 2^-24 of
the sum of magnitudes; no chain here is longer than 170 (rows of a run, 32 products of an
instruction, runs and tiles)."""
import pytest

pytestmark = pytest.mark.gpu

TOL = 170 * 2.0 ** -24


def _reference(x, dy, shape):
    import torch

    nz, ny, nx = shape
    X = torch.nn.functional.pad(x.double().view(nz, ny, nx, -1), (0, 0, 1, 1, 1, 1, 1, 1))
    D = dy.double()
    taps = [X[t // 9:t // 9 + nz, t // 3 % 3:t // 3 % 3 + ny, t % 3:t % 3 + nx].reshape(nz * ny * nx, -1) for t in range(27)]
    return torch.cat([D.T @ s for s in taps], 1), torch.cat([D.abs().T @ s.abs() for s in taps], 1)


def _run(x, dy, shape, cin, cout, ldx, offx, ldd, offd):
    import torch

    from paper_1410_1914_amd import unet as U

    dw = torch.zeros(cout, U.unet_kpad(cin), device="cuda")
    db = torch.zeros(cout, device="cuda")
    U.unet_conv3d_wgrad(x, ldx, offx, dy, ldd, offd, shape, cin, cout, dw, db)
    torch.cuda.synchronize()
    assert not dw[:, 27 * cin:].any()
    return dw[:, :27 * cin].double(), db.double()


def _data(shape, ldx, ldd, seed):
    import torch

    g = torch.Generator("cuda").manual_seed(seed)
    V = shape[0] * shape[1] * shape[2]
    return (torch.randn((V, ldx), generator=g, device="cuda").bfloat16(),
            torch.randn((V, ldd), generator=g, device="cuda").bfloat16())


@pytest.mark.parametrize("shape", [(1, 8, 32), (1, 9, 33), (5, 7, 31), (13, 17, 70), (3, 1, 1), (50, 8, 64), (7, 16, 96)])
@pytest.mark.parametrize("cin,cout,ldx,offx,ldd,offd", [(16, 16, 16, 0, 16, 0), (48, 32, 64, 16, 48, 8),
                                                        (32, 48, 32, 0, 48, 0), (128, 64, 128, 0, 96, 32)])
def test_weight_gradient_tiles(hip, shape, cin, cout, ldx, offx, ldd, offd):
    x, dy = _data(shape, ldx, ldd, sum(shape) + cin)
    dw, db = _run(x, dy, shape, cin, cout, ldx, offx, ldd, offd)
    xs, ds = x[:, offx:offx + cin], dy[:, offd:offd + cout]
    ref, mag = _reference(xs, ds, shape)
    assert ((dw - ref).abs() <= TOL * mag).all()
    assert ((db - ds.double().sum(0)).abs() <= TOL * ds.double().abs().sum(0)).all()


@pytest.mark.parametrize("shape", [(2, 3, 40), (1, 8, 32)])
def test_values_that_are_not_finite_stay_in_their_own_taps(hip, shape):
    import torch

    x, dy = _data(shape, 16, 16, 3)
    x[-1] = float("inf")  # the last voxel: taps that would step past the grid never meet it
    dw, _ = _run(x, dy, shape, 16, 16, 16, 0, 16, 0)
    ref, _ = _reference(x, dy, shape)
    nz, ny, nx = shape
    # tap t reads the voxel at (z, y, x) + t - 1: met where its partner lies inside the grid
    met = torch.tensor([nz - t // 9 in range(nz) and ny - t // 3 % 3 in range(ny) and nx - t % 3 in range(nx)
                        for t in range(27)], device="cuda")
    assert torch.equal(torch.isfinite(dw).view(16, 27, 16).all(2).all(0), ~met)
    fine = torch.isfinite(ref)
    assert torch.allclose(dw[fine], ref[fine], rtol=1e-5, atol=1e-3)


def test_weight_gradient_of_inputs_off_the_16_byte_boundaries(hip):
    import torch

    shape, c = (5, 9, 40), 16
    x, dy = _data(shape, c, c, 4)
    store = torch.zeros(x.numel() + 4, dtype=torch.bfloat16, device="cuda")
    off = store[4:].view(x.shape)
    off.copy_(x)
    dw, db = _run(off, dy, shape, c, c, c, 0, c, 0)
    ref, mag = _reference(x, dy, shape)
    assert ((dw - ref).abs() <= TOL * mag).all()
    assert ((db - dy.double().sum(0)).abs() <= TOL * dy.double().abs().sum(0)).all()

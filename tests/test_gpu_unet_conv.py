"""The 3x3x3 convolution where its tilings can go wrong: grids smaller than a tile, rows and
planes that end inside one, every number of planes per workgroup, one to four channel slices
per workgroup, the marching form and the ring, channel slices of wider rows, a concatenation
with an upsampled tensor, and inputs that are not finite at a corner.  Reference: FP64
products of shifted copies in plain torch.

Tolerance: BF16 rounding of the result (2^-8 of it covers half a unit) and FP32 sums of
27 cin products, off by at most 27 cin 2^-24 of the sum of magnitudes."""
import pytest

pytestmark = pytest.mark.gpu


def _reference(x, w, b, shape, relu):
    import torch

    nz, ny, nx = shape
    cin = x.shape[1]
    out = torch.zeros((nz * ny * nx, w.shape[0]), dtype=torch.float64, device="cuda")
    mag = torch.zeros_like(out)
    X = torch.nn.functional.pad(x.double().view(nz, ny, nx, cin), (0, 0, 1, 1, 1, 1, 1, 1))
    for t in range(27):
        s = X[t // 9:t // 9 + nz, t // 3 % 3:t // 3 % 3 + ny, t % 3:t % 3 + nx].reshape(-1, cin)
        k = w[:, t * cin:(t + 1) * cin].double().T.contiguous()
        out += s @ k
        mag += s.abs() @ k.abs()
    out += b.double()
    return out.clamp_min(0) if relu else out, mag + b.double().abs()


def _data(shape, ld, cin, cout, seed):
    import torch

    from paper_1410_1914_amd import unet as U

    g = torch.Generator("cuda").manual_seed(seed)
    x = torch.randn((shape[0] * shape[1] * shape[2], ld), generator=g, device="cuda").bfloat16()
    w = torch.zeros((cout, U.unet_kpad(cin)), device="cuda")
    w[:, :27 * cin] = torch.randn((cout, 27 * cin), generator=g, device="cuda") * (27 * cin) ** -0.5
    return x, w.bfloat16(), torch.randn(cout, generator=g, device="cuda")


def _check(got, ref, mag, cin):
    tol = 2.0 ** -8 * ref.abs() + 27 * cin * 2.0 ** -24 * mag
    assert ((got.double() - ref).abs() <= tol).all()


# (shape, cin, cout): the comment names the form taken
CASES = [((1, 1, 1), 16, 16), ((3, 5, 17), 32, 16), ((2, 17, 15), 48, 64), ((7, 4, 16), 64, 96),  # one plane per slab
         ((12, 40, 70), 16, 16), ((9, 33, 50), 32, 32),                                              # one or two
         ((30, 50, 50), 64, 64), ((23, 47, 49), 32, 64), ((47, 30, 49), 48, 32),                     # three or four
         ((50, 90, 70), 32, 48), ((21, 100, 130), 16, 48),                                           # one slice; march
         ((37, 130, 135), 16, 16), ((70, 90, 60), 16, 32), ((29, 121, 97), 16, 64),                  # march
         ((66, 250, 262), 32, 16)]                                                                   # ring


@pytest.mark.parametrize("shape,cin,cout", CASES)
@pytest.mark.parametrize("relu", [False, True])
def test_tiles(hip, shape, cin, cout, relu):
    import torch

    from paper_1410_1914_amd import unet as U

    ldx, offx, ldy, offy = (cin, 0, cout, 0) if relu else (cin + 16, 8, cout + 24, 16)
    x, w, b = _data(shape, ldx, cin, cout, sum(shape) + cin)
    y = torch.full((x.shape[0], ldy), 7.0, dtype=torch.bfloat16, device="cuda")
    y32 = torch.zeros((x.shape[0], cout), device="cuda") if relu else None
    U.unet_conv3d_fwd(x, ldx, offx, w, b, y, ldy, offy, y32, shape, cin, cout, relu)
    torch.cuda.synchronize()
    ref, mag = _reference(x[:, offx:offx + cin], w, b, shape, relu)
    _check(y[:, offy:offy + cout], ref, mag, cin)
    if relu:
        assert torch.equal(y32.bfloat16(), y)
        assert ((y32 - ref).abs() <= (27 * cin + 2) * 2.0 ** -24 * mag).all()
    else:
        assert (y[:, :offy] == 7).all() and (y[:, offy + cout:] == 7).all()


@pytest.mark.parametrize("shape,c1,c2,cout", [((6, 10, 14), 32, 64, 64), ((40, 46, 50), 16, 32, 32),
                                              ((64, 250, 262), 16, 32, 16)])
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


@pytest.mark.parametrize("shape,cin,cout", [((6, 20, 40), 32, 64), ((37, 130, 135), 16, 16), ((66, 250, 262), 32, 16)])
def test_values_that_are_not_finite_stay_within_reach(hip, shape, cin, cout):
    """An infinity and a NaN reach the 27 voxels around them and nothing else."""
    import torch

    from paper_1410_1914_amd import unet as U

    nz, ny, nx = shape
    x, w, b = _data(shape, cin, cin, cout, 7)
    z, yy, xx = nz // 2, 3, 15
    v = (z * ny + yy) * nx + xx
    x[v, 1] = float("inf")
    x[x.shape[0] - 1, 0] = float("nan")
    y = torch.zeros((nz * ny * nx, cout), dtype=torch.bfloat16, device="cuda")
    U.unet_conv3d_fwd(x, cin, 0, w, b, y, cout, 0, None, shape, cin, cout, False)
    torch.cuda.synchronize()
    bad = ~torch.isfinite(y.float()).all(1).view(nz, ny, nx)
    want = torch.zeros_like(bad)
    want[z - 1:z + 2, yy - 1:yy + 2, xx - 1:xx + 2] = True
    want[nz - 2:, ny - 2:, nx - 2:] = True
    assert torch.equal(bad, want)

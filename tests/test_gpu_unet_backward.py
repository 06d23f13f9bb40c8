"""The backward steps in 16-byte pieces and the ReLU masks applied where a gradient is
written.

Single layers: pooling's and upsampling's adjoints and the head's input gradient round one
FP32 expression to BF16, so torch's FP32 gives the same bits; the head's weight gradient is
a sum of n products in FP32, off by at most n 2^-24 of the sum of magnitudes along its
longest chain (here at most 64 additions).

Network: its gradient against the same chain of public layer calls with every mask a call
of its own.  All tensors of the chain have the same bits; only the FP32 sums of the weight
gradients meet in another order (chains of at most 170 terms)."""
import pytest

pytestmark = pytest.mark.gpu


def _bf(shape, seed):
    import torch

    return torch.randn(shape, generator=torch.Generator("cuda").manual_seed(seed), device="cuda").bfloat16()


# rows of whole 16-byte pieces, and rows that are not (another kernel)
@pytest.mark.parametrize("shape", [(2, 2, 2), (4, 6, 10), (2, 18, 34)])
@pytest.mark.parametrize("c,ldf,offf,ldc,offc", [(16, 16, 0, 16, 0), (8, 24, 16, 32, 8), (32, 48, 16, 32, 0),
                                                 (12, 20, 4, 12, 0), (16, 33, 1, 17, 1)])
def test_pool_and_up_adjoints(hip, shape, c, ldf, offf, ldc, offc):
    import torch

    from paper_1410_1914_amd import unet as U

    nz, ny, nx = shape
    fine, coarse = _bf((nz, ny, nx, ldf), 1), _bf((nz // 2, ny // 2, nx // 2, ldc), 2)
    want = fine.clone()
    spread = coarse[..., offc:offc + c].float()
    for d in range(3):
        spread = spread.repeat_interleave(2, d)
    want[..., offf:offf + c] = (fine[..., offf:offf + c].float() + 0.125 * spread).bfloat16()
    got = fine.clone()
    U.unet_pool_bwd(coarse, ldc, offc, got, ldf, offf, shape, c)
    torch.cuda.synchronize()
    assert torch.equal(got, want)

    want = coarse.clone()
    s = torch.zeros((nz // 2, ny // 2, nx // 2, c), device="cuda")
    for d in range(8):
        s = s + fine[d >> 2::2, (d >> 1) & 1::2, d & 1::2, offf:offf + c].float()
    want[..., offc:offc + c] = s.bfloat16()
    got = coarse.clone()
    U.unet_up_bwd(fine, ldf, offf, got, ldc, offc, shape, c)
    torch.cuda.synchronize()
    assert torch.equal(got, want)


@pytest.mark.parametrize("nvox", [1, 255, 257, 5000, 140000])
@pytest.mark.parametrize("ldx,c", [(16, 16), (48, 16), (20, 16), (8, 8)])
def test_head_adjoint(hip, nvox, ldx, c):
    import torch

    from paper_1410_1914_amd import unet as U

    x = _bf((nvox, ldx), 3)
    g = torch.Generator("cuda").manual_seed(4)
    w, dout = (torch.randn(n, generator=g, device="cuda") for n in (c, nvox))
    dx = torch.full((nvox, c), 7.0, dtype=torch.bfloat16, device="cuda")
    dw, db = torch.zeros(c, device="cuda"), torch.zeros(1, device="cuda")
    U.unet_head_bwd(x, ldx, w, dout, dx, dw, db, nvox, c)
    torch.cuda.synchronize()
    assert torch.equal(dx, (dout[:, None] * w).bfloat16())
    p = x[:, :c].double() * dout.double()[:, None]
    # per thread nvox / (256 * 512) + 1 terms, 6 + 3 pairings, at most 1024 workgroups' sums
    tol = (nvox // (256 * 512) + 10 + min(1024, nvox // 256 + 1)) * 2.0 ** -24
    assert ((dw - p.sum(0)).abs() <= tol * p.abs().sum(0)).all()
    assert (db - dout.double().sum()).abs() <= tol * dout.double().abs().sum()


@pytest.mark.parametrize("shape", [(8, 8, 8), (8, 24, 40), (16, 16, 136)])
def test_network_gradient_is_the_chain_of_layers(hip, shape):
    import torch

    from paper_1410_1914_amd import unet as U

    net = U.UNet(seed=8)
    for t, (name, _, cout) in enumerate(net.specs):
        net.B[name].copy_(torch.linspace(-0.1, 0.1, cout))
    net.touch()
    dims = [tuple(s >> l for s in shape) for l in range(4)]
    vox = [d[0] * d[1] * d[2] for d in dims]
    feat = _bf((vox[0], 16), 9)
    dout = torch.randn(vox[0], generator=torch.Generator("cuda").manual_seed(10), device="cuda")
    net.forward(feat, shape, train=True)
    net.backward(feat, dout, shape)
    got = net.grads(shape).clone()

    spec = {n: (ci, co) for n, ci, co in net.specs}
    wb = {n: net.W[n].bfloat16() for n in spec}
    ref = torch.zeros_like(net.params)
    act, grad = {"feat": feat}, {}

    def buf(lev, c):
        return torch.zeros((vox[lev], c), dtype=torch.bfloat16, device="cuda")

    # (layer, input, output, level); the skip tensors live in their concatenations
    order = [("e1a", "feat", "a1", 0), ("e1b", "a1", "cat1", 0), ("e2a", "p2", "a2", 1), ("e2b", "a2", "cat2", 1),
             ("e3a", "p3", "a3", 2), ("e3b", "a3", "cat3", 2), ("b4a", "p4", "b4a", 3), ("b4b", "b4a", "b4b", 3),
             ("d3a", "cat3", "d3a", 2), ("d3b", "d3a", "d3b", 2), ("d2a", "cat2", "d2a", 1), ("d2b", "d2a", "d2b", 1),
             ("d1a", "cat1", "d1a", 0), ("d1b", "d1a", "d1b", 0)]
    pooled = {"e1b": ("cat1", "p2", 16, 0), "e2b": ("cat2", "p3", 32, 1), "e3b": ("cat3", "p4", 64, 2)}
    upped = {"b4b": ("b4b", "cat3", 128, 64, 2), "d3b": ("d3b", "cat2", 64, 32, 1), "d2b": ("d2b", "cat1", 32, 16, 0)}
    cat_ch = {"cat1": 48, "cat2": 96, "cat3": 192}
    for name, i, o, lev in order:
        ci, co = spec[name]
        act[o] = buf(lev, cat_ch.get(o, co))
        U.unet_conv3d_fwd(act[i], ci, 0, wb[name], net.B[name], act[o], cat_ch.get(o, co), 0, None, dims[lev], ci, co, True)
        if name in pooled:
            s, d, c, l = pooled[name]
            act[d] = buf(l + 1, c)
            U.unet_pool_fwd(act[s], cat_ch[s], 0, act[d], c, 0, dims[l], c)
        if name in upped:
            s, d, c, off, l = upped[name]
            U.unet_up_fwd(act[s], c, 0, act[d], cat_ch[d], off, dims[l], c)
    wo, wc, bo, _ = net._layout["head"]
    grad["d1b"] = buf(0, 16)
    U.unet_head_bwd(act["d1b"], 16, net.W["head"], dout, grad["d1b"], ref[wo:wo + wc], ref[bo:bo + 1], vox[0], 16)
    for name, i, o, lev in reversed(order):
        ci, co = spec[name]
        ldo = cat_ch.get(o, co)
        if name in upped:  # the gradient of this output comes from the concatenation
            s, d, c, off, l = upped[name]
            grad[s] = buf(l + 1, c)
            U.unet_up_bwd(grad[d], cat_ch[d], off, grad[s], c, 0, dims[l], c)
        if name in pooled:
            s, d, c, l = pooled[name]
            U.unet_pool_bwd(grad[d], c, 0, grad[s], cat_ch[s], 0, dims[l], c)
        U.unet_relu_bwd(act[o], ldo, 0, grad[o], ldo, 0, vox[lev], co)
        wo, wc, bo, _ = net._layout[name]
        U.unet_conv3d_wgrad(act[i], ci, 0, grad[o], ldo, 0, dims[lev], ci, co, ref[wo:wo + wc], ref[bo:bo + co])
        if i != "feat":
            wt = torch.zeros(ci * U.unet_kpad(co), dtype=torch.bfloat16, device="cuda")
            U.unet_conv3d_wtrans(wb[name], wt, ci, co)
            grad[i] = buf(lev, ci)
            U.unet_conv3d_fwd(grad[o], ldo, 0, wt, None, grad[i], ci, 0, None, dims[lev], co, ci, False)
    torch.cuda.synchronize()
    # the weight gradients' magnitudes are not at hand: by Cauchy-Schwarz the sum of
    # magnitudes of an entry is at most |x| |dy| over the layer's tensors
    for name, i, o, lev in order:
        ci, co = spec[name]
        wo, wc, bo, _ = net._layout[name]
        mag = act[i][:, :ci].double().norm(dim=0).max() * grad[o][:, :co].double().norm(dim=0).max()
        assert (got[wo:wo + wc] - ref[wo:wo + wc]).abs().max() <= 2 * 170 * 2.0 ** -24 * mag
        assert (got[bo:bo + co] - ref[bo:bo + co]).abs().max() <= 2 * 170 * 2.0 ** -24 * grad[o].double().abs().sum(0).max()
    wo, wc, bo, _ = net._layout["head"]
    p = act["d1b"].double() * dout.double()[:, None]
    assert ((got[wo:wo + wc] - p.sum(0)).abs() <= 600 * 2.0 ** -24 * p.abs().sum(0)).all()

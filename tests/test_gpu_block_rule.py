"""Which calls step a grid in blocks of planes: those that move enough steps through a block
of enough planes, and no shorter ones; and that cut grids step like whole ones in every
tiling, with planes that hold nothing, in middle blocks and in rounds of every length."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _map(shape, seed):
    u = np.random.default_rng(seed).integers(0, 64, shape, dtype=np.uint8)
    return np.where(u < 3, 1, np.where(u < 4, 2, np.where(u < 8, 3, 0))).astype(np.uint8)


def _params(hip, mode, knudsen):
    return hip.lbm_params_default(mode=hip.MODE_REACT if mode == "react" else hip.MODE_DEFF, knudsen=knudsen,
                                  k_lat=0.01 if mode == "react" else 0.0, check_every=20, tol_flux=0.0)


def test_short_calls_and_thin_blocks_walk_the_whole_grid(hip):
    s = hip.Solver(_map((90, 300, 300), 1), _params(hip, "deff", 0), device_prep=True)
    n, _ = s.blocks(200)
    assert n >= 3  # 90 // n planes to a block, a quarter of them steps to a round
    most = 90 // n // 4
    for k in range(1, 3 * most):
        rounds = -(-k // most)
        assert s.blocks(k) == ((n, -(-k // rounds)) if k // rounds >= 5 else (1, 1))
    s.set_tiling(1, 4, 0)  # without the XCD-aware order there are no slabs
    assert s.blocks(200) == (1, 1)
    s.close()
    thin = hip.Solver(_map((16, 530, 640), 2), _params(hip, "deff", 0), device_prep=True)
    small = hip.Solver(_map((60, 60, 60), 2), _params(hip, "deff", 0), device_prep=True)
    assert thin.blocks(200) == (1, 1) and small.blocks(200) == (1, 1)


@pytest.mark.parametrize("shape,mode,knudsen", [((90, 300, 300), "deff", 0), ((97, 230, 384), "react", 1)])
def test_every_tiling_on_a_cut_grid(hip, shape, mode, knudsen):
    import torch

    ph = _map(shape, 3)
    ph[:, shape[1] // 3:shape[1] // 3 + 30] = 1  # a slab of y with nothing to step in most planes
    ph[30:45] = 1  # planes with nothing in them, inside a block and at a block's end
    if mode == "deff":
        ph[:, 5, :] = 0
    a = hip.Solver(ph, _params(hip, mode, knudsen), device_prep=True)
    assert a.blocks(40)[0] >= 3
    c0 = torch.rand(a.shape, generator=torch.Generator().manual_seed(1))
    b = hip.Solver(ph, _params(hip, mode, knudsen), device_prep=True)
    b.set_tiling(1, 4, 0)
    b.set_initial_concentration(c0)
    b.step(7)
    want7 = b.populations()
    b.step(33)
    want40 = b.populations()
    for spw in (1, 2, 4):
        for waves in (1, 2, 4, 8):
            a.set_tiling(spw, waves, 1)
            a.set_initial_concentration(c0)
            a.step(7)
            assert a.blocks(7)[0] >= 3 and a.blocks(33)[0] >= 3
            assert torch.equal(a.populations(), want7), (spw, waves)
            a.step(33)
            assert torch.equal(a.populations(), want40), (spw, waves)


def test_d3q19_short_calls_thin_blocks_and_uneven_slabs_walk_the_whole_grid(hip):
    s = hip.Solver19(_map((90, 210, 220), 1), _params(hip, "deff", 1))
    n, _ = s.blocks(200)
    assert n >= 3
    most = min(12, 90 // n // 4)
    for k in range(1, 3 * most):
        rounds = -(-k // most)
        assert s.blocks(k) == ((n, -(-k // rounds)) if k // rounds >= 4 else (1, 1))
    s.close()
    for shape in ((16, 350, 400), (300, 9, 800), (50, 50, 50)):
        s = hip.Solver19(_map(shape, 2), _params(hip, "deff", 1))
        assert s.blocks(200) == (1, 1)
        s.close()


@pytest.mark.parametrize("shape,mode,steps", [((121, 170, 160), "react", 29), ((90, 210, 220), "deff", 41)])
def test_d3q19_middle_blocks_and_empty_planes(hip, shape, mode, steps):
    import torch

    ph = _map(shape, 4)
    ph[:, shape[1] // 3:shape[1] // 3 + 10] = 1
    ph[40:48] = 1
    if mode == "deff":
        ph[:, 5, :] = 0
    a, b = (hip.Solver19(ph, _params(hip, mode, 1)) for _ in range(2))
    assert a.blocks(steps)[0] >= 3
    c0 = torch.rand(a.shape, generator=torch.Generator().manual_seed(2))
    for s in (a, b):
        s.set_initial_concentration(c0)
    a.step(steps)
    for _ in range(steps):
        b.step(1)
    assert torch.equal(a.populations(), b.populations())
    assert a.measure().as_dict() == b.measure().as_dict()


@pytest.mark.parametrize("every", [20, 34])
def test_windows_of_a_cut_grid(hip, every):
    """Check windows, of even and uneven rounds, equal single steps; the time of their launches is
    reported as for small grids."""
    import torch

    ph = _map((90, 300, 300), 6)
    p = hip.lbm_params_default(check_every=every, tol_flux=0.0, max_steps=1 << 40)
    a, b = (hip.Solver(ph, p, device_prep=True) for _ in range(2))
    assert a.blocks(every)[0] >= 3
    c0 = torch.rand(a.shape, generator=torch.Generator().manual_seed(3))
    for s in (a, b):
        s.set_initial_concentration(c0)
    for _ in range(2):
        _, info = a.advance(3 * every)
    for _ in range(6 * every):
        b.step(1)
    assert torch.equal(a.populations(), b.populations())
    assert info.steps == 6 * every and info.kernel_launches == 6 * every and info.kernel_ms > 0


def test_no_steps_on_a_cut_grid(hip):
    """A call of no steps, and the none that are left after steps taken two to a launch."""
    import torch

    ph = _map((90, 300, 300), 7)
    s = hip.Solver(ph, _params(hip, "deff", 0), device_prep=True)
    assert s.blocks(200)[0] >= 3
    f = s.populations()
    s.step(0)
    assert torch.equal(s.populations(), f)
    s.set_temporal(6, 16)
    s.step(8)
    two = s.populations()
    s.set_temporal(0)
    s.set_populations(f)
    s.step(8)
    assert torch.equal(s.populations(), two)
    s.close()
    s = hip.Solver19(_map((90, 210, 220), 7), _params(hip, "deff", 1))
    assert s.blocks(200)[0] >= 3
    f = s.populations()
    s.step(0)
    assert torch.equal(s.populations(), f)

"""Steps taken in blocks of planes (grids whose lattices exceed the last-level cache)
against single steps over the whole grid: the same lattice, bit for bit.

A single ``step(1)`` walks the whole grid; ``step(n)`` on a large grid takes the steps
block by block.  Shapes cover the fewest planes that are still cut, rows in their own
windows and windows running on across row ends, rows that do not divide by eight, and
step counts that leave either lattice current."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (nz, ny, nx), mode, Knudsen, steps: about 5 M simulated voxels, two or three blocks
D7 = [((16, 530, 640), "deff", 1, 7), ((61, 131, 700), "react", 0, 38), ((187, 99, 320), "react", 1, 33),
      ((212, 203, 192), "deff", 0, 120)]
# D3Q19: about 2 M simulated voxels
D19 = [((16, 350, 400), "deff", 9), ((73, 131, 256), "react", 26), ((150, 121, 130), "react", 31)]


def _map(shape, seed):
    """Mostly pore, with carbon, Pt and ionomer voxels spread at random."""
    u = np.random.default_rng(seed).integers(0, 64, shape, dtype=np.uint8)
    return np.where(u < 3, 1, np.where(u < 4, 2, np.where(u < 8, 3, 0))).astype(np.uint8)


def _params(hip, mode, knudsen):
    return hip.lbm_params_default(mode=hip.MODE_REACT if mode == "react" else hip.MODE_DEFF, knudsen=knudsen,
                                  k_lat=0.01 if mode == "react" else 0.0, check_every=20, tol_flux=0.0)


@pytest.mark.parametrize("shape,mode,knudsen,steps", D7)
def test_d3q7_blocks_equal_whole_steps(hip, shape, mode, knudsen, steps):
    import torch

    ph = _map(shape, shape[0])
    a = hip.Solver(ph, _params(hip, mode, knudsen), device_prep=True)
    assert 56 * a.info.n_active > 240 << 20  # both lattices past the limit of whole steps
    b = hip.Solver(ph, _params(hip, mode, knudsen), device_prep=True)
    c0 = torch.rand(a.shape, generator=torch.Generator().manual_seed(1))
    for s in (a, b):
        s.set_initial_concentration(c0)
    a.step(steps)
    for _ in range(steps):
        b.step(1)
    assert torch.equal(a.populations(), b.populations())
    # the same in a captured check window, from the lattice the steps left current
    a.advance(40)
    for _ in range(40):
        b.step(1)
    assert torch.equal(a.populations(), b.populations())


@pytest.mark.parametrize("shape,mode,steps", D19)
def test_d3q19_blocks_equal_whole_steps(hip, shape, mode, steps):
    import torch

    ph = _map(shape, shape[1])
    a = hip.Solver19(ph, _params(hip, mode, 1))
    assert 152 * a.info.n_active > 240 << 20
    b = hip.Solver19(ph, _params(hip, mode, 1))
    c0 = torch.rand(a.shape, generator=torch.Generator().manual_seed(2))
    for s in (a, b):
        s.set_initial_concentration(c0)
    a.step(steps)
    for _ in range(steps):
        b.step(1)
    assert torch.equal(a.populations(), b.populations())
    assert a.measure().as_dict() == b.measure().as_dict()

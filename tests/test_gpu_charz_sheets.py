"""Structure characterisation by sheets, where its layouts can go wrong: runs longer than
a window, than a ring's margin and than the stored counts; rows that do not fill a word;
cross-sections whose yz diagonals close late; sheets that do not fit on chip (walked or
swept instead); maps that start at odd addresses.  Against the oracle, value for value."""
import numpy as np
import pytest

from oracle import lbm as O

pytestmark = pytest.mark.gpu

SHAPES = [
    (5, 5, 31), (64, 64, 64), (33, 33, 97), (40, 60, 63),  # lcm 120
    (130, 130, 129), (97, 31, 40),                         # rings of 130 and 3007 rows
    (300, 300, 8), (1, 260, 260), (260, 1, 33),
    (2, 700, 700),                                         # sheets too large for LDS
]


def _sparse(shape, seed, share):
    """Solid at random with the given share, and two slabs of pore for long runs."""
    m = np.random.default_rng(seed).random(shape) >= share
    m[shape[0] // 2] = True
    m[:, shape[1] // 2] = True
    return m


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("share", [0.004, 0.4])
def test_pore_size(hip, shape, share):
    m = _sparse(shape, sum(shape), share)
    assert np.array_equal(hip.pore_size_device(m).cpu().numpy(), O.pore_chords(m))


def test_pore_size_of_a_long_all_pore_map(hip):
    m = np.ones((150, 150, 140), bool)
    m[3, 4, 5] = False
    assert np.array_equal(hip.pore_size_device(m).cpu().numpy(), O.pore_chords(m))


@pytest.mark.parametrize("shape", SHAPES + [(3, 700, 1000)])
@pytest.mark.parametrize("faces", [1, 2, 3])
def test_reach(hip, shape, faces):
    m = np.random.default_rng(sum(shape)).random(shape) >= 0.42
    seed = np.zeros(shape, bool)
    seed[:, :, 0] = bool(faces & 1)
    if faces & 2:
        seed[:, :, -1] = True
    want = O.flood(m, seed & m)
    got, cycles = hip.reach_device(m, faces)
    assert np.array_equal(got.cpu().numpy(), want.astype(np.uint8))
    again, cycles2 = hip.reach_device(m, faces, static_scratch=True)
    assert np.array_equal(again.cpu().numpy(), want.astype(np.uint8))
    if shape[1] * shape[2] < 400_000 and shape[0] * shape[2] < 400_000:
        assert cycles2 == cycles  # sheets; the line sweeps of larger planes race on purpose


@pytest.mark.parametrize("nx", [64, 61])
def test_reach_of_maps_at_odd_addresses(hip, nx):
    import torch

    shape = (20, 30, nx)
    m = np.random.default_rng(nx).random(shape) >= 0.4
    seed = np.zeros(shape, bool)
    seed[:, :, 0] = True
    store = torch.zeros(2, m.size + 8, dtype=torch.uint8, device="cuda")
    a, out = (store[k, 1:1 + m.size].view(shape) for k in (0, 1))
    a.copy_(torch.from_numpy(m.astype(np.uint8) * 200))  # any non-zero byte passes
    got, _ = hip.reach_device(a, 1, out=out)
    assert np.array_equal(got.cpu().numpy(), O.flood(m, seed & m).astype(np.uint8))
    assert not store[1, 0] and not store[1, 1 + m.size:].any()

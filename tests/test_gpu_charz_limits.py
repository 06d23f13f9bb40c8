"""Structure characterisation at the limits of what a workgroup's LDS holds: the reach's
largest sheets, the first ones past them (line sweeps) and the sizes between, where a sheet
alone would still fit 160 KB but not together with the kernel's own LDS."""
import numpy as np
import pytest

from oracle import lbm as O

pytestmark = pytest.mark.gpu


# nx / 64 rounded up times the rows of a sheet: 6784, 6785, 6816, 6820, 6826, 6827; 6822, 6824
@pytest.mark.parametrize("shape", [(1, 6784, 64), (1, 6785, 64), (1, 6816, 64), (1, 6820, 60), (1, 6826, 64),
                                   (1, 6827, 64), (2, 1137, 384), (1706, 2, 256)])
def test_reach_of_the_largest_sheets(hip, shape):
    m = np.random.default_rng(sum(shape)).random(shape) >= 0.3
    seed = np.zeros(shape, bool)
    seed[:, :, 0] = seed[:, :, -1] = True
    got, _ = hip.reach_device(m, 3)
    assert np.array_equal(got.cpu().numpy(), O.flood(m, seed & m).astype(np.uint8))


def test_threads_with_different_sizes(hip):
    """Calls of two host threads, one with small and one with large sheets, on streams of
    their own: none is refused and each gives what it gives alone."""
    import threading

    import torch

    maps = [np.random.default_rng(n).random((n, n, 60)) >= 0.4 for n in (8, 140)]
    want = [(hip.pore_size_device(m).cpu(), hip.reach_device(m, 1)[0].cpu()) for m in maps]
    errors = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(150 if k == 0 else 40):
                    assert torch.equal(hip.pore_size_device(maps[k]).cpu(), want[k][0])
                    assert torch.equal(hip.reach_device(maps[k], 1)[0].cpu(), want[k][1])
        except Exception as e:  # handed to the test's own thread
            errors.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def _us(f):
    """Microseconds of a call, the best of five rounds of ten."""
    import time

    import torch

    f()
    best = float("inf")
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(10):
            f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best * 1e5


@pytest.mark.parametrize("shape", [(52, 50, 50), (48, 50, 50), (32, 31, 100), (1, 200, 200), (3, 300, 100)])
def test_pore_size_of_long_rings_takes_no_longer_than_of_a_cube(hip, shape):
    """A few rings of many rows (their y and z edges have a small common divisor, or one of
    them is short) are not laid out by a few workgroups; these maps have no more voxels than
    the cube, which takes both routes about as long."""
    import torch

    def pore(s):
        return (torch.rand(s, generator=torch.Generator("cuda").manual_seed(1), device="cuda") < 0.45).to(torch.uint8)

    cube, m = pore((51, 51, 50)), pore(shape)
    assert np.array_equal(hip.pore_size_device(m).cpu().numpy(), O.pore_chords(m.cpu().numpy().astype(bool)))
    assert _us(lambda: hip.pore_size_device(m)) <= 1.6 * _us(lambda: hip.pore_size_device(cube))


@pytest.mark.parametrize("shape", [(40, 50, 50), (16, 24, 240), (2, 100, 100), (10, 100, 64), (12, 30, 33), (7, 14, 300)])
@pytest.mark.parametrize("share", [0.05, 0.5])
def test_pore_size_with_several_workgroups_to_a_sheet(hip, shape, share):
    m = np.random.default_rng(sum(shape)).random(shape) >= share
    m[shape[0] // 2] = True
    assert np.array_equal(hip.pore_size_device(m).cpu().numpy(), O.pore_chords(m))

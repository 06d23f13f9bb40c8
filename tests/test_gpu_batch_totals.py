"""An instance's measured totals do not depend on the batch it is in: added in one order by
itself, among others, in groups of any size and after others have finished."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(96, 90, 70), (20, 30, 40), (64, 64, 130), (96, 96, 65)]


def _map(shape):
    u = np.random.default_rng(sum(shape)).integers(0, 64, shape, dtype=np.uint8)
    return np.where(u < 6, 1, np.where(u < 8, 2, np.where(u < 14, 3, 0))).astype(np.uint8)


def _params(hip, mode, max_steps):
    react = mode == "react"
    return hip.lbm_params_default(mode=hip.MODE_REACT if react else hip.MODE_DEFF, k_lat=0.01 if react else 0.0,
                                  check_every=20, max_steps=max_steps, tol_flux=0.0)


@pytest.mark.parametrize("mode", ["deff", "react"])
@pytest.mark.parametrize("group", [0, 1, 192 << 20])
def test_totals_of_an_instance_are_its_own(hip, mode, group):
    limits = [200, 40, 200, 120]  # two instances finish before the others
    maps = [_map(s) for s in SHAPES]
    b = hip.Batch(maps, [_params(hip, mode, n) for n in limits], device_prep=True)
    b.set_group_bytes(group)
    _, infos = b.run()
    for m, n, got in zip(maps, limits, infos):
        s = hip.Solver(m, _params(hip, mode, n), device_prep=True)
        _, want = s.run_to_steady()
        assert got.steps == want.steps == n
        for k in ("j_in", "j_out", "j_vol", "rate", "mass", "residual"):
            assert getattr(got, k) == getattr(want, k), k

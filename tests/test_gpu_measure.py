"""The measured totals over grids from a few row segments to more than a wave takes at once
in any split of them: the mass against the sum of the field that is read back.

Tolerance: the field is read back in FP32 (2^-24 of each value), the totals are FP64 sums of
at most 6 M terms (n 2^-53, below 1e-9)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["deff", "react"])
@pytest.mark.parametrize("shape", [(2, 3, 5), (4, 8, 70), (32, 32, 32), (70, 63, 57), (96, 130, 128), (170, 160, 200)])
def test_mass_is_the_sum_of_the_field(hip, shape, mode):
    import torch

    u = np.random.default_rng(shape[2]).integers(0, 64, shape, dtype=np.uint8)
    ph = np.where(u < 3, 1, np.where(u < 4, 2, 0)).astype(np.uint8)
    react = mode == "react"
    s = hip.Solver(ph, hip.lbm_params_default(mode=hip.MODE_REACT if react else hip.MODE_DEFF, knudsen=0,
                                              k_lat=0.01 if react else 0.0), device_prep=True)
    s.set_initial_concentration(torch.rand(s.shape, generator=torch.Generator().manual_seed(2)))
    s.step(3)
    info = s.measure()
    total = float(s.concentration().double().sum())
    assert abs(info.mass - total) <= (2.0 ** -24 + 1e-9) * total
    again = s.measure()
    assert again.mass == info.mass and again.j_vol == info.j_vol  # one fixed order of addition

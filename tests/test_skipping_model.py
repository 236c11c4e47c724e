"""The skipping rule itself, on the CPU: what a certified tile leaves out moves
no posterior mean by more than the stated bound, and the count of the skipped
weight stays inside its 32 bits."""
import numpy as np
import pytest

from paper_1706_07263_amd import synth
from tests.skip_model import SkipModel, scaled_attenuation, skip_rule

MASS_DEPTH_LOG2 = 12.0   # unit of the kernels' count below the first depth


def _mu_ref():
    s = synth.plan_settings(0, 8)
    thb, so2 = 0.5 * (s["thb_min"] + s["thb_max"]), 0.5 * (s["so2_min"] + s["so2_max"])
    return scaled_attenuation(thb * (1.0 - so2), thb * so2, 1.0, 0.0) / np.sqrt(np.log2(np.e) / 2.0)


@pytest.mark.parametrize("grid,sigma,tol", [(64, 0.02, 1e-6), (128, 0.01, 1e-2), (256, 0.015, 3e-3), (256, 0.01, 1e-9),
                                            (128, 0.02, 100.0)])
def test_certified_tiles_hold_the_bound(grid, sigma, tol):
    s = dict(synth.plan_settings(0, grid, sigma=sigma), posterior_tolerance=tol)
    skip_log2, bound = skip_rule(s)
    assert 0 < bound <= tol
    mu_ref = _mu_ref()
    model = SkipModel(s, mu_ref, skip_log2, bound)
    rng = np.random.default_rng(grid)
    for spread in (3.0, 40.0):
        thb = rng.uniform(110 - spread, 110 + spread, (8, 16))
        so2 = rng.uniform(0.7 - 0.004 * spread, 0.7 + 0.004 * spread, (8, 16))
        fr = synth.noisy_frame(*synth.hb_hbo2(thb, so2), synth.spectra(), 5).astype(np.float64)
        z = (-np.log(fr) - mu_ref).reshape(128, 3) * np.sqrt(np.log2(np.e) / (2.0 * sigma ** 2))
        for tile in model.tiles(z):
            p = model.passes(tile)
            assert p.moved <= bound
            units = np.array(p.skipped) + model.depth0 + MASS_DEPTH_LOG2
            assert units.max() < 31.0

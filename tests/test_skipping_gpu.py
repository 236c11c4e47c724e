"""The posterior kernels' certified skipping against a float64 model of its
rule: how many chunks a tile evaluates tells which passes ran."""
import numpy as np
import pytest

from paper_1706_07263_amd import synth
from tests import hbtest
from tests.skip_model import SkipModel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def tissue_frame(seed, h, w):
    """Pixels of random tissue, more or less spread over the grid."""
    rng = np.random.default_rng(seed)
    spread, centre = (10, 25, 40, 60)[seed % 4], (60, 100, 140, 190)[seed // 4 % 4]
    thb = rng.uniform(max(20, centre - spread), min(200, centre + spread), (h, w))
    so2 = rng.uniform(max(0.3, 0.7 - spread * 0.004), min(1.0, 0.7 + spread * 0.004), (h, w))
    return synth.noisy_frame(*synth.hb_hbo2(thb, so2), synth.spectra(), seed)


# Frames whose first depth does not suffice (margins of the model's decisions
# 0.2 and more in log2).  With the tolerances above 1e-3 the skipped weight lies
# above 2^-10: no count in units fixed for the default tolerance holds it.
@pytest.mark.parametrize("grid,sigma,tol,seed", [(256, 0.01, 1e-6, 28), (256, 0.015, 3e-3, 13), (256, 0.015, 3e-3, 29),
                                                 (256, 0.014, 5e-3, 30), (512, 0.02, 2e-3, 30), (512, 0.02, 2e-3, 45)])
def test_certificate_follows_its_model(torch_cuda, grid, sigma, tol, seed):
    """One region of 16 x 8 pixels, four tiles: some need a second pass, and the
    evaluated chunks are the model's.  About ten chunks a tile lie in a unit of
    depth and bounds round far below that unit: a quarter of what the further
    passes add is room enough."""
    from paper_1706_07263_amd import hb
    s = dict(synth.plan_settings(0, grid, sigma=sigma), posterior_tolerance=tol)
    run = hbtest.GpuRun(16, 8, s, grid_split=1)
    info = run.plan.info()
    assert info["posterior_kernel"] == "mfma"
    hb.hb_plan_set_timing(run.plan.handle, True)
    run(tissue_frame(seed, 8, 16)[None])
    chunks = hb.hb_plan_get_work(run.plan.handle)[0] / (32 * 16)
    obs = run.debug(hb.HB_DEBUG_LOWPASS_OBS).astype(np.float64)
    run.close()
    model = SkipModel(s, info["mu_ref"], info["skip_log2"], info["skip_bound"])
    z = (obs[0] + obs[1]).T * np.sqrt(np.log2(np.e) / (2.0 * sigma ** 2))
    passes = [model.passes(t) for t in model.tiles(z)]
    first, want = sum(p.kept[0] for p in passes), sum(p.kept[-1] for p in passes)
    print(f"{grid} {sigma} {tol}: chunks {chunks:.0f}, model {want} ({first} in the first pass), passes "
          f"{[len(p.kept) for p in passes]}")
    assert max(p.moved for p in passes) <= info["skip_bound"]
    assert want > 1.03 * first
    assert abs(chunks - want) <= 0.25 * (want - first)


@pytest.mark.parametrize("tol", [1e-12, 1e-9, 1e-6])
def test_first_depth_certifies_at_any_tolerance(torch_cuda, tol):
    """Smooth tissue certifies at the first depth: the unit of the skipped weight
    follows the depth, so that a tight tolerance does not drown in what counting
    whole units adds."""
    from paper_1706_07263_amd import hb
    s = dict(synth.plan_settings(0, 512), posterior_tolerance=tol)
    run = hbtest.GpuRun(16, 8, s, grid_split=1)
    info = run.plan.info()
    thb = np.full((8, 16), 90.0) + np.linspace(0.0, 4.0, 16)[None]
    fr = synth.noisy_frame(*synth.hb_hbo2(thb, np.full((8, 16), 0.7)), synth.spectra(), 3)
    hb.hb_plan_set_timing(run.plan.handle, True)
    run(fr[None])
    chunks = hb.hb_plan_get_work(run.plan.handle)[0] / (32 * 16)
    obs = run.debug(hb.HB_DEBUG_LOWPASS_OBS).astype(np.float64)
    run.close()
    model = SkipModel(s, info["mu_ref"], info["skip_log2"], info["skip_bound"])
    passes = [model.passes(t) for t in model.tiles((obs[0] + obs[1]).T * np.sqrt(np.log2(np.e) / 2e-4))]
    assert [len(p.kept) for p in passes] == [1] * 4
    assert abs(chunks - sum(p.kept[0] for p in passes)) <= 0.01 * chunks

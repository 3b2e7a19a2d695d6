"""The FP16 collision works on the stored binary16 values directly.  One step
from a state that binary16 holds exactly is the FP32 form's step, rounded once:
both run the same arithmetic (scaled by powers of two), so a result is off by
half a unit of binary16 and what FP32 arithmetic itself leaves."""
import numpy as np
import pytest
import torch

from paper_1507_02509_amd import inputs
from paper_1507_02509_amd.sim import Sim, beta_from_nu

pytestmark = pytest.mark.gpu

W = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None, None]
SCALE = np.array([2.0] + [8.0] * 4 + [32.0] * 4)[:, None, None]


@pytest.mark.parametrize("nx,ny", [(5, 3), (65, 7), (130, 66)])
@pytest.mark.parametrize("variant", ["A", "B", "C", "D"])
@pytest.mark.parametrize("gamma_mode", ["estimate", "fixed", "exact"])
def test_one_step_is_the_f32_step_rounded(nx, ny, variant, gamma_mode):
    ux, uy = inputs.spectral(256, 8, 0.1, seed=nx + ny)
    ux, uy = ux[:ny, :nx].copy(), uy[:ny, :nx].copy()
    kw = dict(collision="kbc", variant=variant, gamma_mode=gamma_mode, device="cuda")
    if gamma_mode == "fixed":
        kw["gamma_fixed"] = 1.3
    beta = beta_from_nu(1e-2)
    s16 = Sim(nx, ny, beta, form="f16", **kw).init(ux, uy).step(3)
    f = s16.get_populations()
    s32 = Sim(nx, ny, beta, form="f32", **kw).init(ux, uy)
    s32.set_populations(f)
    h16 = (s16.step(1).get_populations().cpu().numpy() - W) * SCALE
    h32 = (s32.step(1).get_populations().cpu().numpy() - W) * SCALE
    half = 0.5 * np.spacing(np.abs(h16).astype(np.float16)).astype(np.float64)
    assert np.isfinite(h16).all()
    assert (np.abs(h16 - h32) <= half + 2.0 ** -20 * np.abs(h32).max()).all()

"""The spectra's shell sums are collected in tiles of 256 x 8 wavevectors
(k_x, |k_y|): sizes at and around the tile edges (half = N/2 of 255 .. 257
and 7 .. 9), the smallest lattice, and more shells than the lattice has,
against the oracle's full-plane definition."""
import numpy as np
import pytest
import torch

from paper_1507_02509_amd.sim import Sim, beta_from_nu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 14, 16, 17, 18, 510, 512, 513, 514])
def test_shell_tiles(orc, n):
    print("shell tiles", n, flush=True)
    rng = np.random.default_rng(n)
    f = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None, None] * (1 + 0.01 * rng.standard_normal((9, n, n)))
    s = Sim(n, n, beta_from_nu(1e-3), form="f64").init(np.zeros((n, n)), np.zeros((n, n)), mode="eq")
    s.set_populations(f)
    _, gx, gy = (t.cpu().numpy() for t in s.moments())
    kmax = n + 3                        # the corner's shell is round(n / sqrt 2)
    ek, zk = (t.cpu().numpy() for t in s.spectra(kmax))
    oe, oz = orc.spectra(gx, gy, kmax)
    # FP64 sums of up to n^2 terms in another order, and the transforms'
    # rounding (log2 n stages): 1e-12 of the largest shell
    assert np.abs(ek - oe).max() < 1e-12 * oe.max()
    assert np.abs(zk - oz).max() < 1e-12 * oz.max()
    last = int(np.floor(np.hypot(n // 2, n // 2) + 0.5))
    assert not ek[last + 1:].any() and not zk[last + 1:].any()
    only_e = torch.empty(kmax + 1, dtype=torch.float64, device="cuda")
    from paper_1507_02509_amd import _lib as L
    L.check(s.lib.lbm_spectra(s.ctx, kmax, only_e.data_ptr(), None))
    assert np.abs(only_e.cpu().numpy() - ek).max() < 1e-12 * oe.max()

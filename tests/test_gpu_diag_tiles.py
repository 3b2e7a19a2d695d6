"""The one-pass diagnostics kernel works on 64 x 8 and 64 x 16 tiles extended
by two nodes on every side: lattices at and around the tile edges and the
smallest one against the oracle; populations beyond a factor two of their
weights (the general logarithm) and non-finite ones."""
import numpy as np
import pytest

from paper_1507_02509_amd.sim import Sim, beta_from_nu

pytestmark = pytest.mark.gpu
W = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)[:, None, None]


def restarted(nx, ny, f, rho0=1.0, **kw):
    s = Sim(nx, ny, beta_from_nu(1e-3), rho0=rho0, **kw).init(np.zeros((ny, nx)), np.zeros((ny, nx)), mode="eq")
    s.set_populations(f)
    return s


def compare(orc, s, f, nx, ny, rho0, tol):
    p = orc.Params(nx, ny, beta_from_nu(1e-3), collision=orc.KBC, variant=orc.VARIANTS["B"])
    o = orc.diagnostics(p, f)
    d = s.diagnostics()
    for k in ("mass", "E", "E_std", "Z", "Z_std", "P", "P_std", "S", "gamma", "gamma_std"):
        assert d[k] == pytest.approx(o[k], rel=tol, abs=tol * (1 + abs(o["S"]))), k
    assert d["n_nonfinite"] == o["n_nonfinite"] and d["n_feq_nonpos"] == o["n_feq_nonpos"]
    return d


# sums of at most 2e5 terms of one sign in another order (1e-15 each) and the
# logarithm's and quotient's last places: 1e-11 leaves room for the
# cancellation in the standard deviations
@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 4), (62, 7), (63, 8), (64, 9), (65, 16), (66, 17), (130, 15),
                                   (2049, 500), (2048, 512)])
@pytest.mark.parametrize("rho0", [1.0, 1.3])
def test_tile_edges(orc, nx, ny, rho0):
    print("diag tiles", nx, ny, rho0, flush=True)
    rng = np.random.default_rng(nx * 7 + ny)
    f = rho0 * W * (1 + 0.05 * rng.standard_normal((9, ny, nx)))
    compare(orc, restarted(nx, ny, f, rho0, form="f64"), f, nx, ny, rho0, 1e-11)


def test_far_from_equilibrium(orc):
    print("diag far", flush=True)
    nx, ny = 70, 20
    rng = np.random.default_rng(5)
    f = W * np.exp(rng.uniform(-3, 3, (9, ny, nx)))     # factors 0.05 .. 20: both logarithms, |u|^2 above 1/6
    compare(orc, restarted(nx, ny, f, form="f64"), f, nx, ny, 1.0, 1e-11)


def test_nonfinite_counts():
    print("diag nonfinite", flush=True)
    nx, ny = 67, 19
    f = np.repeat(np.repeat(W, ny, 1), nx, 2)
    f[3, 5, 6], f[0, 18, 66], f[7, 0, 0], f[8, 0, 0] = np.nan, np.inf, np.inf, -np.inf
    for form in ("f32", "f64"):
        d = restarted(nx, ny, f, form=form).diagnostics()
        assert d["n_nonfinite"] == 3
        assert np.isnan(d["S"])

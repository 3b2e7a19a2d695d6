"""Two adjoint steps per launch (lbm_adjoint_segment, lbm_adjoint_rollout) on
4-, 8- and 16-row tiles, ragged in both directions, short and long segments,
with the dL/dbeta sums direct and folded: lambda bitwise equal to single
adjoint steps over recomputed states, dL/dbeta to summation order, and the
rollout bitwise equal to its segments in turn."""
import pytest
import torch

from paper_1507_02509_amd import inputs
from paper_1507_02509_amd.sim import Sim, beta_from_nu

pytestmark = pytest.mark.gpu

LATTICES = [(3, 5), (64, 4), (70, 33), (65, 512), (520, 261), (1801, 1001)]


@pytest.mark.parametrize("nx,ny", LATTICES)
@pytest.mark.parametrize("form,kw,frozen", [("f32", dict(variant="D", gamma_guard=1e-4), False),
                                            ("f32", dict(variant="B"), True), ("f16", dict(variant="C"), False),
                                            ("f64", dict(variant="A"), False), ("f64", dict(collision="lbgk"), False),
                                            ("f32", dict(variant="B", gamma_mode="fixed", gamma_fixed=1.1), False)])
@pytest.mark.parametrize("nsteps,K", [(7, 7), (11, 4)])
def test_pairs(nx, ny, form, kw, frozen, nsteps, K):
    print("adjoint pairs", nx, ny, form, kw, frozen, nsteps, K, flush=True)
    ux, uy = inputs.uniform_noise(nx, ny, 0.03, seed=nx + ny, device="cuda")
    s = Sim(nx, ny, beta_from_nu(1e-3), form=form, fusion=1, **kw).init(ux, uy)
    s.set_adjoint_gamma(frozen)
    states = [s.state_buffer().clone()]
    for _ in range(nsteps):
        states.append(s.step(1).state_buffer().clone())
    g = torch.Generator(device="cuda").manual_seed(3)
    lam0 = torch.randn((ny, 9, s.pitch), generator=g, dtype=s.adjoint_dtype, device="cuda")

    def acc():
        return torch.zeros(1, dtype=torch.float64, device="cuda")

    # one step at a time, over the states themselves; sum of |terms| for the bar
    a, b, db, scale = lam0.clone(), s.new_adjoint(), acc(), 0.0
    for n in range(nsteps - 1, -1, -1):
        one = acc()
        s.adjoint_step(states[n], a, b, one)
        db += one
        scale += float(s.planes(a).abs().max()) * nx * ny
        a, b = b, a
    want = s.planes(a).clone()

    def slots():
        return [s.new_state() for _ in range(K - 1)]

    # segment by segment
    la, lb, dseg, sl = lam0.clone(), s.new_adjoint(), acc(), slots()
    for first in reversed(range(0, nsteps, K)):
        if s.adjoint_segment(states[first], sl, min(K, nsteps - first), la, lb, dseg):
            la, lb = lb, la
    assert torch.equal(s.planes(la), want)
    # FP64 sums of the same terms in another order
    assert abs(dseg.item() - db.item()) <= 1e-13 * scale
    # the whole rollout
    ra, rb, droll = lam0.clone(), s.new_adjoint(), acc()
    if s.adjoint_rollout([states[n] for n in range(0, nsteps, K)], nsteps, K, slots(), slots(), ra, rb, droll):
        ra, rb = rb, ra
    assert torch.equal(s.planes(ra), want)
    assert droll.item() == dseg.item()

"""Ensembles advanced by four fused steps per launch (their default where the
members have many tiles per CU together): bitwise equal to stepping every
member by single steps, ragged members included, and the states end in the
buffers they end in with pairs of steps."""
import pytest
import torch

from paper_1507_02509_amd import inputs
from paper_1507_02509_amd.ensemble import Ensemble
from paper_1507_02509_amd.sim import Sim, beta_from_nu

pytestmark = pytest.mark.gpu

# sizes of the members by the bytes of all their buffers: few tiles, inside the
# last-level cache (plain stores), beyond it
FEW = [(70, 33), (128, 200)]
INSIDE = [(700, 333), (65, 1200), (512, 512), (130, 77)]
BEYOND = [(1500, 1301), (2000, 901), (70, 33)]


def members(sizes, fusion, **kw):
    out = []
    for k, (nx, ny) in enumerate(sizes):
        beta = beta_from_nu(1e-3 * (k + 1))
        ux, uy = inputs.uniform_noise(nx, ny, 0.03, seed=k, device="cuda")
        out.append(Sim(nx, ny, beta, gamma_fixed=1.0 / beta, fusion=fusion, **kw).init(ux, uy))
    return out


@pytest.mark.parametrize("sizes", [FEW, INSIDE, BEYOND])
@pytest.mark.parametrize("kw", [dict(form="f32", variant="B"), dict(form="f32", collision="lbgk"),
                                dict(form="f32", variant="D", gamma_mode="fixed"), dict(form="f64", variant="C"),
                                dict(form="f64", collision="lbgk"), dict(form="f64", variant="A", gamma_mode="fixed"),
                                dict(form="f16", variant="A"), dict(form="f16", collision="lbgk"),
                                dict(form="f32", variant="B", gamma_mode="exact")])
def test_equals_single_steps(sizes, kw):
    print("ensemble4", sizes, kw, flush=True)
    a, b = members(sizes, None, **kw), members(sizes, 1, **kw)
    ens = Ensemble(a)
    ens.step(19)                     # 16 by fours where they pay, a pair, a single step
    for s, r in zip(a, b):
        r.step(19)
        assert s.steps == 19
        assert torch.equal(s.planes(s.state_buffer()), r.planes(r.state_buffer()))
        assert s.state_buffer() is s.buf_a      # nine pairs and one single step
    ens.free()

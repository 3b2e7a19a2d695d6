"""Four fused steps per launch (taken by lbm_step in its default configuration
on small lattices and where memory binds): bitwise equal to single steps at
the edges of every launch shape's range, ragged in both directions, and the
state ends in the buffer it ends in without them."""
import pytest
import torch

from paper_1507_02509_amd import inputs
from paper_1507_02509_amd.sim import Sim, beta_from_nu

pytestmark = pytest.mark.gpu

# (lattice, tile height it takes): one tile per CU of 2, 4, 8, 12, 16 or 28
# rows (28 not for FP64), the next size beyond each
SMALL = [(3, 5), (64, 64), (65, 33), (64, 256), (64, 258), (200, 130), (128, 514), (320, 313), (384, 380), (400, 400),
         (512, 509), (640, 637)]
KINDS = [("f32", "kbc", "B", "estimate"), ("f16", "kbc", "D", "estimate"), ("f64", "kbc", "A", "estimate"),
         ("f32", "lbgk", "B", "estimate"), ("f64", "kbc", "C", "fixed"), ("f32", "kbc", "B", "exact")]
# many tiles per CU: memory-bound collisions with plain and non-temporal stores
LARGE = [(900, 701, "f32", "lbgk", "estimate"), (2240, 1700, "f32", "kbc", "fixed"), (2240, 1701, "f32", "kbc", "estimate"),
         (700, 601, "f64", "lbgk", "estimate"), (1500, 1301, "f64", "kbc", "fixed"), (901, 900, "f16", "lbgk", "estimate"),
         (1700, 1601, "f16", "kbc", "fixed")]


def pair(nx, ny, form, collision, variant, gamma):
    beta = beta_from_nu(1e-3)
    ux, uy = inputs.uniform_noise(nx, ny, 0.03, seed=nx + ny, device="cuda")
    return [Sim(nx, ny, beta, collision=collision, variant=variant, form=form, gamma_mode=gamma, gamma_fixed=1.0 / beta,
                fusion=f).init(ux, uy) for f in (None, 1)]


def same(a, b):
    return torch.equal(a.planes(a.state_buffer()), b.planes(b.state_buffer()))


@pytest.mark.parametrize("nx,ny", SMALL)
@pytest.mark.parametrize("form,collision,variant,gamma", KINDS)
def test_small(nx, ny, form, collision, variant, gamma):
    print("step4 small", nx, ny, form, collision, variant, gamma, flush=True)
    a, b = pair(nx, ny, form, collision, variant, gamma)
    a.step(11)                    # two launches of four steps, a pair, a single step
    b.step(11)
    assert a.steps == b.steps == 11 and same(a, b)


@pytest.mark.parametrize("nx,ny,form,collision,gamma", LARGE)
def test_large(nx, ny, form, collision, gamma):
    print("step4 large", nx, ny, form, collision, gamma, flush=True)
    a, b = pair(nx, ny, form, collision, "B", gamma)
    a.step(16)
    b.step(16)
    assert same(a, b)


def test_buffer_and_splits():
    """Every step count ends in the buffer that pairs of steps end in, and a
    caller's own tile height or store kind keeps the pairs."""
    print("step4 buffers", flush=True)
    ux, uy = inputs.uniform_noise(130, 70, 0.03, seed=1, device="cuda")
    for n in range(1, 19):
        a, b = (Sim(130, 70, 0.99, form="f32", fusion=f).init(ux, uy) for f in (None, (2, 16)))
        a.step(n)
        b.step(n)
        assert (a.state_buffer() is a.buf_a) == (b.state_buffer() is b.buf_a) and same(a, b), n
    c = Sim(130, 70, 0.99, form="f32", tile=(256, 1, False)).init(ux, uy).step(18)
    assert same(c, a)


def test_graph_replay():
    print("step4 graph", flush=True)
    ux, uy = inputs.uniform_noise(96, 80, 0.03, seed=2, device="cuda")
    a = Sim(96, 80, 0.99, form="f32", graph=10).init(ux, uy)
    b = Sim(96, 80, 0.99, form="f32", fusion=1).init(ux, uy)
    for k in (10, 20, 7, 33):
        a.step(k)
        b.step(k)
        torch.cuda.synchronize()
        assert same(a, b)

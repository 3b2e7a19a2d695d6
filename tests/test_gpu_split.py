"""Which launches run: lbm_get_split / lbm_ensemble_get_split against the
launch shapes documented for lbm_step (four steps per launch, kbc_step4.hip),
and every shape of many tiles per CU compared bitwise with single steps.  A
dispatch that never takes four steps, or another height, fails here."""
import pytest
import torch

from paper_1507_02509_amd import _lib as L
from paper_1507_02509_amd import inputs
from paper_1507_02509_amd.ensemble import Ensemble
from paper_1507_02509_amd.sim import Sim, beta_from_nu

pytestmark = pytest.mark.gpu


def make(nx, ny, form="f32", collision="kbc", gamma="estimate", variant="B", **kw):
    beta = beta_from_nu(1e-3)
    ux, uy = inputs.uniform_noise(nx, ny, 0.03, seed=nx + ny, device="cuda")
    return Sim(nx, ny, beta, collision=collision, variant=variant, form=form, gamma_mode=gamma, gamma_fixed=1.0 / beta,
               **kw).init(ux, uy)


def same(a, b):
    return torch.equal(a.planes(a.state_buffer()), b.planes(b.state_buffer()))


# at most one tile per CU: rows and waves by lattice (FP32 and FP16, FP64), at the
# edges of each height's range
ONE = [(3, 5, (2, 10), (2, 10)), (64, 256, (2, 10), (2, 10)), (64, 258, (4, 12), (4, 12)), (128, 512, (4, 12), (4, 12)),
       (128, 514, (8, 16), (8, 16)), (320, 313, (8, 16), (8, 16)), (384, 380, (12, 16), (12, 12)),
       (512, 509, (16, 16), (16, 12)), (640, 637, (28, 12), None)]


@pytest.mark.parametrize("nx,ny,single,double", ONE)
def test_one_tile_per_cu(nx, ny, single, double):
    print("split one", nx, ny, flush=True)
    for form, collision, gamma in (("f32", "kbc", "estimate"), ("f16", "kbc", "estimate"), ("f32", "lbgk", "estimate"),
                                   ("f32", "kbc", "exact"), ("f64", "kbc", "estimate"), ("f64", "kbc", "exact")):
        s = make(nx, ny, form, collision, gamma)
        want = double if form == "f64" else single
        if form == "f64" and gamma == "exact" and single != (2, 10):
            assert s.split(19) == {4: 0, 2: 18, 1: 1, "tile4": None}
        elif want is not None:
            assert s.split(19) == {4: 16, 2: 2, 1: 1, "tile4": want + (True,)}, (form, collision, gamma, s.split(19))
        assert s.split(7)[4] == 0 and s.split(0) == {4: 0, 2: 0, 1: 0, "tile4": None}


# many tiles per CU: the height whose busiest CU has the least to do (FP32), and
# the shapes of the other forms; None: pairs of steps
MANY = [(768, 767, "f32", "kbc", "estimate", (12, 8, True)), (1020, 1023, "f32", "kbc", "estimate", (16, 8, True)),
        (1601, 1537, "f32", "kbc", "estimate", (20, 8, True)), (1201, 1199, "f32", "kbc", "estimate", (24, 8, True)),
        (1281, 1279, "f32", "kbc", "estimate", (28, 12, True)), (900, 701, "f32", "lbgk", "estimate", (12, 8, False)),
        (2900, 2601, "f16", "kbc", "estimate", (40, 12, True)), (1401, 1403, "f16", "kbc", "estimate", None),
        (901, 900, "f16", "lbgk", "estimate", (24, 8, True)), (1700, 1601, "f16", "kbc", "fixed", (24, 8, False)),
        (1401, 1403, "f64", "lbgk", "estimate", (12, 12, True)), (700, 601, "f64", "lbgk", "estimate", (12, 12, False)),
        (701, 703, "f64", "kbc", "estimate", (12, 8, True)), (700, 601, "f64", "kbc", "fixed", (12, 8, False)),
        (1401, 1403, "f64", "kbc", "fixed", (12, 8, True)), (1020, 1023, "f32", "kbc", "exact", None)]


@pytest.mark.parametrize("nx,ny,form,collision,gamma,tile", MANY)
def test_many_tiles_per_cu(nx, ny, form, collision, gamma, tile):
    print("split many", nx, ny, form, collision, gamma, flush=True)
    a = make(nx, ny, form, collision, gamma)
    b = make(nx, ny, form, collision, gamma, fusion=1)
    assert a.split(11) == ({4: 8, 2: 2, 1: 1, "tile4": tile} if tile else {4: 0, 2: 10, 1: 1, "tile4": None})
    assert b.split(11) == {4: 0, 2: 0, 1: 11, "tile4": None}
    a.step(11)
    b.step(11)
    assert same(a, b)


# members of an ensemble: few tiles, inside the last-level cache, beyond it
FEW = [(70, 33), (128, 200)]
INSIDE = [(700, 333), (65, 1200), (512, 512), (130, 77)]
BEYOND = [(2100, 2001), (1900, 1801), (70, 33)]
ENS = [(FEW, "f32", "kbc", None), (INSIDE, "f32", "kbc", (24, 8, True)), (INSIDE, "f32", "lbgk", (12, 8, False)),
       (BEYOND, "f32", "kbc", (28, 12, True)), (INSIDE, "f16", "kbc", None), (BEYOND, "f16", "kbc", (40, 12, True)),
       (BEYOND, "f64", "lbgk", (12, 12, True))]


@pytest.mark.parametrize("sizes,form,collision,tile", ENS)
def test_ensemble(sizes, form, collision, tile):
    print("split ensemble", sizes, form, collision, flush=True)
    a, b = ([make(nx, ny, form, collision, **kw) for nx, ny in sizes] for kw in ({}, {"fusion": 1}))
    e = Ensemble(a)
    assert e.split(11) == ({4: 8, 2: 2, 1: 1, "tile4": tile} if tile else {4: 0, 2: 10, 1: 1, "tile4": None})
    assert e.split(11, persistent=True) == {4: 0, 2: 10, 1: 1, "tile4": None}
    e.step(11)
    for s, r in zip(a, b):
        r.step(11)
        assert same(s, r)
    e.free()


def test_settings():
    """The division follows the settings: the caller's own fused tile, single
    steps, graph replays chunk by chunk, a slab."""
    print("split settings", flush=True)
    s = make(130, 70)
    assert s.split(18)[4] == 16
    rows = s.fusion_rows
    s.set_fusion(2, 24)
    assert s.split(18) == {4: 0, 2: 18, 1: 0, "tile4": None}
    s.set_fusion(2, rows)
    assert s.split(18)[4] == 16
    s.set_graph(10)
    assert {k: s.split(37)[k] for k in (4, 2, 1)} == {4: 24, 2: 12, 1: 1}   # 3 x (8 + 2), then 7
    s.set_graph(0)
    s.set_fusion(1)
    assert s.split(9) == {4: 0, 2: 0, 1: 9, "tile4": None}
    s.set_fusion(2, 8)
    lo, hi = s.halo_buffers()
    s.set_halo(lo, hi)
    assert s.split(2)[2] == 2
    for n in (3, -1):
        with pytest.raises(L.KbcError) as e:
            s.split(n)
        assert e.value.code == L.LBM_EINVAL


def test_store_kind_of_the_caller():
    """A store kind set against the default is kept: pairs where the four-step
    kernels do not have it, their other kind where they do."""
    print("split store kind", flush=True)
    s = make(130, 70)                                       # default: non-temporal
    assert s.tile[2] and s.split(16)[4] == 16
    s.set_tile(256, 1, False)
    assert s.split(16) == {4: 0, 2: 16, 1: 0, "tile4": None}
    s.set_tile(256, 1, True)
    assert s.split(16)[4] == 16
    s = make(1020, 1023)                                    # default: plain; the kernels write non-temporally
    assert not s.tile[2] and s.split(16)["tile4"] == (16, 8, True)
    s.set_tile(256, 1, True)
    assert s.split(16)["tile4"] == (16, 8, True)
    s = make(900, 701, collision="lbgk")                    # both kinds
    assert s.split(16)["tile4"] == (12, 8, False)
    s.set_tile(256, 1, True)
    assert s.split(16)["tile4"][2] and s.split(16)[4] == 16
    e = Ensemble([make(nx, ny) for nx, ny in BEYOND])
    assert e.split(16)["tile4"] == (28, 12, True)
    e.set_tile(256, 1, False)
    assert e.split(16) == {4: 0, 2: 16, 1: 0, "tile4": None}
    e.set_tile(256, 1, True)
    assert e.split(16)[4] == 16
    e.free()

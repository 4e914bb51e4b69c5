"""The linked-subcell form of the list build (3^d stencil).  Small systems take
the circle form, so the lists of test_gpu_nlist.py that put pairs at their list
radius, or atoms into one subcell, no longer reach it by size: the same
properties here with HDMD_CIRCLE=0 and the grid of side >= r_l,max requested,
in the sparse and the dense form (more than 16 atoms per subcell).  Lists are
sets of pairs decided in FP64: they equal the definition's exactly.  Batches
of systems that are linked by size equal the lone runs bit for bit."""
import numpy as np
import pytest
import torch

from paper_2112_12271_amd import hdmd as H
from paper_2112_12271_amd import inputs
from tests.gpu_util import csr_equal, dev, force_err, gpu_list, partnered
from tests.test_gpu_nlist import _boundary

pytestmark = pytest.mark.gpu
FULL = H.HDMD_SUBCELLS_FULL
BOTH = (H.HDMD_FP64, H.HDMD_MIXED)


@pytest.fixture
def linked(monkeypatch):
    monkeypatch.setenv("HDMD_CIRCLE", "0")


def _system(d, x, L, sig_max, prec=H.HDMD_FP64, cut=1.0, skin=0.25, width=8):
    return H.System(d=d, n=len(x), box_l=L, potential=H.HDMD_HARMONIC, cutoff=cut, skin=skin,
                    sigma_max=sig_max, precision=prec, max_neighbors=width, subcells=FULL)


def test_the_switch_selects_the_form(monkeypatch):
    """The forms list a row in different orders, so that the force sums differ
    in their last bits: the switch these tests rely on does select."""
    d, n = 3, 600
    sig = inputs.bidisperse(n, 1.0, 1.4, 1)
    L = inputs.box_for_packing(d, sig, 0.6)
    x = inputs.uniform_positions(n, d, L, 2)
    out = []
    for env in ("1", "0", "0"):
        monkeypatch.setenv("HDMD_CIRCLE", env)
        s = _system(d, x, L, 1.4, width=200)
        assert H.hdmd_cells_per_axis(s) >= 3
        out.append(H.hdmd_forces(s, dev(x), dev(sig), H.workspace(s))[0])
    assert torch.equal(out[1], out[2]) and not torch.equal(out[0], out[1])
    assert force_err(out[0].cpu().numpy(), out[1].cpu().numpy()) < 1e-12


@pytest.mark.parametrize("d", [2, 3, 4, 6, 8])
@pytest.mark.parametrize("nc,pairs", [(3, 200), (5, 200), (3, 2000)])
def test_boundary_band(orc, linked, d, nc, pairs):
    """Pairs at r_l +- a few ulps across subcell and periodic faces and corners
    (4000 atoms: the dense form for d <= 4)."""
    rl = 1.25
    L = nc * rl * (1.0 + 4e-9)
    # (d = 8: atoms enough for 3^8 subcells, at most four per atom)
    x = _boundary(d, L, rl, max(pairs, 900) if d == 8 else pairs, seed=31 * d + nc + pairs)
    sig = np.ones(len(x))
    ref = orc.nlist_brute(x, sig, L, 1.0, 0.25)
    for prec in BOTH:
        s = _system(d, x, L, 1.0, prec)
        assert H.hdmd_cells_per_axis(s) >= 3
        got, _, _ = gpu_list(s, x, sig)
        assert csr_equal(got, ref), prec


@pytest.mark.parametrize("d,nc,pairs", [(3, 3, 300), (4, 3, 300), (6, 3, 300), (3, 5, 300), (5, 4, 300),
                                        (3, 5, 1500), (4, 3, 1500), (5, 3, 2200), (7, 3, 1500),
                                        (9, 3, 3000)])
def test_pair_radius_band(orc, linked, d, nc, pairs):
    """Pairs at their own list radius c sigma_ij + s, a few ulps either side,
    with diameters 1 and 2 mixed: the per-atom shares of the pair threshold
    keep every pair the definition lists, sparse and dense."""
    c, skin = 1.0, 0.25
    L = nc * (2.0 * c + skin) * (1.0 + 4e-9)
    g = np.random.default_rng(53 * d + nc + pairs)
    h = 0.5 * L
    a = g.uniform(-h, h, (pairs, d))
    sig = g.choice([1.0, 2.0], size=(pairs, 2))
    u = g.normal(size=(pairs, d))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    rl = c * sig.mean(axis=1) + skin
    b = a + (rl + g.integers(-4, 5, pairs) * np.spacing(rl))[:, None] * u
    b = np.where(b >= h, b - L, b)
    b = np.where(b < -h, b + L, b)
    b = np.where(b >= h, -h, b)
    x, sig = np.stack([a, b], 1).reshape(-1, d), sig.reshape(-1)
    sig[0] = 2.0
    ref = orc.nlist_brute(x, sig, L, c, skin)
    assert len(ref[1]) > 300
    for prec in BOTH:
        s = _system(d, x, L, 2.0, prec)
        assert H.hdmd_cells_per_axis(s) == nc
        got, _, _ = gpu_list(s, x, sig)
        assert csr_equal(got, ref), prec


@pytest.mark.parametrize("d,n,L", [(3, 1600, 13.0), (5, 1500, 7.0)])
@pytest.mark.parametrize("prec", BOTH)
def test_one_crowded_subcell(orc, linked, d, n, L, prec):
    """A sparse system with 90 atoms in one subcell: the segments that reach it
    walk its blocks in several passes, and its home atoms take three."""
    g = np.random.default_rng(50 + d)
    x = inputs.uniform_positions(n, d, L, 40 + d)
    lsc = L / orc.ncell(L, 1.7)
    x[:90] = -L / 2 + g.uniform(0.05, 0.95, size=(90, d)) * lsc
    sig = inputs.bidisperse(n, 1.0, 1.4, 60 + d)
    ref = orc.nlist_brute(x, sig, L, 1.0, 0.3)
    s = _system(d, x, L, 1.4, prec, skin=0.3, width=128)
    assert n <= 16 * H.hdmd_cells_per_axis(s) ** d
    got, _, _ = gpu_list(s, x, sig)
    assert csr_equal(got, ref)


@pytest.mark.parametrize("d,nc,n", [(6, 3, 7290), (4, 3, 8000), (2, 5, 1000), (7, 3, 8000)])
@pytest.mark.parametrize("waves", [1, 2, 4])
def test_waves_per_subcell(orc, linked, monkeypatch, d, nc, n, waves):
    monkeypatch.setenv("HDMD_BUILD_BLK", str(waves))
    c, skin = inputs.WCA_CUT, 0.3
    rlmax = c * 1.4 + skin
    L = nc * rlmax * 1.02
    x, sig = partnered(d, n, L, 77 * d + nc, rlmax)
    ref = orc.nlist_brute(x, sig, L, c, skin)
    for prec in BOTH:
        s = _system(d, x, L, 1.4, prec, cut=c, skin=skin, width=16)
        assert H.hdmd_cells_per_axis(s) == nc
        got, _, _ = gpu_list(s, x, sig)
        assert csr_equal(got, ref), prec


# linked by size: sparse and dense in d = 3, sparse d = 5 and 8, d = 9 (a launch of
# its own); then circle-form systems of the same batch
BATCH = [(3, 5000, 0.55, 0.25), (3, 5003, 0.9, 1.4), (5, 9001, 0.3, 0.25), (8, 7000, 0.0044, 0.1),
         (9, 20000, 0.0015, 0.1), (3, 700, 0.6, 0.25), (4, 500, 0.45, 0.25), (6, 900, 0.03, 0.1)]


@pytest.mark.parametrize("prec", BOTH)
@pytest.mark.parametrize("per_class", [False, True])
def test_batch_of_linked_systems_equals_alone(orc, monkeypatch, prec, per_class):
    """FIRE in one batch, in one build launch over the classes and in a launch
    per class: the bits of the lone runs, whose positions agree with the
    oracle's (1e-9, FP64) in d = 3, sparse and dense."""
    if per_class:
        monkeypatch.setenv("HDMD_BUILD_PER_CLASS", "1")
    params = H.hdmd_fire_defaults(0.05, 1e-12, 40)
    systems, alone = [], []
    for k, (d, n, phi, skin) in enumerate(BATCH):
        sig = inputs.bidisperse(n, 1.0, 1.4, k + 1)
        L = inputs.box_for_packing(d, sig, phi)
        x = inputs.uniform_positions(n, d, L, 10 * k + 2)
        s = _system(d, x, L, 1.4, prec, skin=skin, width=64)
        nc = H.hdmd_cells_per_axis(s)
        assert nc >= 3
        if k < 5:
            assert d >= 8 or n > min(8192, 128 * 3 ** d)
            assert (n > 16 * nc ** d) == (k == 1)
        X = dev(x)
        s, res = H.fire_auto(s, X, dev(sig), params, slack=2.0)
        assert res.builds > 1, k  # rebuilt on the way
        if k < 2 and prec == H.HDMD_FP64 and not per_class:
            xo, _ = orc.fire(x, sig, L, H.HDMD_HARMONIC, 1.0, skin, 1.0,
                             orc.fire_params(dt0=0.05, ftol=1e-12, maxiter=40))
            dx = X.cpu().numpy() - xo
            dx -= L * np.round(dx / L)
            assert np.abs(dx).max() < 1e-9, k
        systems.append((s, x, sig))
        alone.append((X.cpu().numpy(), res))
    B = H.Batch(max_slots=8, max_atoms=60000, max_cells=200000)
    keep = []
    for k, (s, x, sig) in enumerate(systems):
        keep.append((dev(x), dev(sig), H.workspace(s)))
        B.hdmd_batch_add_fire(k, s, *keep[k], params)
    for _ in range(4):
        B.hdmd_batch_run(12)
    state, _ = B.hdmd_batch_poll()
    assert (np.asarray(state[:len(systems)]) == H.HDMD_SLOT_DONE).all()
    for k in range(len(systems)):
        pos, _, res = B.hdmd_batch_take(k)
        assert np.array_equal(pos.cpu().numpy(), alone[k][0]), k
        assert (res.iterations, res.builds, res.energy) == \
            (alone[k][1].iterations, alone[k][1].builds, alone[k][1].energy), k

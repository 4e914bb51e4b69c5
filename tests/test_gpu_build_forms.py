"""The list build's forms at the sizes where each can go wrong: subcells of
15, 16, 17, 80, 81, 128 and 129 atoms (edges of the 16-candidate blocks, of a
segment's five blocks per subcell and of the 128 home atoms of a pass), both
sides of the sparse / dense line (16 atoms per subcell), clusters whose every
pair survives (the survivor queues fill and a segment is interrupted and
resumed), and the circle form of n_cell <= 2 at the edges of its 64-atom
tiles and 128-candidate chunks, in d = 7 (16 slots) and d = 8 (24).  Lists are
sets of pairs decided in FP64: they equal the definition's exactly."""
import numpy as np
import pytest

from paper_2112_12271_amd import hdmd as H
from paper_2112_12271_amd import inputs
from tests.gpu_util import csr_equal, gpu_list

pytestmark = pytest.mark.gpu
CUT, SKIN = 1.0, 0.25


@pytest.fixture(autouse=True)
def linked_subcells(monkeypatch):
    """These systems are small: the circle form only where n_cell <= 2."""
    monkeypatch.setenv("HDMD_CIRCLE", "0")


def _check(orc, x, sig, L, nc, d, width=256):
    ref = orc.nlist_brute(x, sig, L, CUT, SKIN)
    s = H.System(d=d, n=len(x), box_l=L, potential=H.HDMD_HARMONIC, cutoff=CUT, skin=SKIN,
                 sigma_max=float(sig.max()), max_neighbors=width, subcells=H.HDMD_SUBCELLS_FULL)
    assert H.hdmd_cells_per_axis(s) in nc
    got, _, _ = gpu_list(s, x, sig)
    assert csr_equal(got, ref)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("occ", [15, 16, 17, 80, 81, 128, 129])
def test_subcells_of_exact_occupancy(orc, d, occ):
    nc = 3
    L = nc * (CUT * 1.4 + SKIN) * 1.01
    lsc = L / nc
    g = np.random.default_rng(10 * occ + d)
    cells = np.stack(np.meshgrid(*[np.arange(nc)] * d, indexing="ij"), -1).reshape(-1, d)
    x = ((cells[:, None, :] + g.uniform(1e-6, 1 - 1e-6, size=(len(cells), occ, d))) * lsc - L / 2)
    x = x.reshape(-1, d)
    sig = g.choice([1.0, 1.4], size=len(x))
    sig[0] = 1.4
    _check(orc, x, sig, L, (nc,), d, width=9 * occ)


@pytest.mark.parametrize("d,nc,n", [(3, 4, 1023), (3, 4, 1025), (4, 3, 1296), (4, 3, 1297)])
def test_sparse_dense_line(orc, d, nc, n):
    L = nc * (CUT * 1.4 + SKIN) * 1.01
    x = inputs.uniform_positions(n, d, L, 7 * n)
    _check(orc, x, inputs.bidisperse(n, 1.0, 1.4, n), L, (nc,), d)


@pytest.mark.parametrize("d,nc,n,k", [(3, 3, 900, 300), (3, 5, 700, 120), (5, 3, 5000, 200),
                                      (6, 2, 700, 260), (8, 2, 600, 200)])
def test_clusters_fill_the_survivor_queues(orc, d, nc, n, k):
    """k atoms within a small ball across a corner of subcells and of the box."""
    L = nc * (CUT * 1.4 + SKIN) * 1.01
    g = np.random.default_rng(d + n)
    x = inputs.uniform_positions(n, d, L, 3 * n)
    u = g.normal(size=(k, d))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    x[:k] = L / 2 + 0.5 * g.uniform(size=(k, 1)) * u
    x[x >= L / 2] -= L
    _check(orc, x, inputs.bidisperse(n, 1.0, 1.4, n), L, (nc,), d, width=k + 100)


@pytest.mark.parametrize("d", [7, 8])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 127, 128, 129, 1000])
def test_circle_form_edges(orc, d, n):
    L = 2 * (CUT * 1.4 + SKIN) * 1.001
    g = np.random.default_rng(100 * d + n)
    # pairs at their list radius up to a few ulps, across the box faces
    x = inputs.uniform_positions(n, d, L, n + d)
    sig = np.full(n, 1.4)
    sig[: n // 2] = 1.0
    for p in range(0, n - 1, 2):
        v = g.normal(size=d)
        v /= np.linalg.norm(v)
        r = CUT * 0.5 * (sig[p] + sig[p + 1]) + SKIN
        x[p + 1] = x[p] + (r + g.integers(-3, 4) * np.spacing(r)) * v
    x = np.where(x >= L / 2, x - L, x)
    x = np.where(x < -L / 2, x + L, x)
    x = np.where(x >= L / 2, -L / 2, x)
    # (few atoms: one subcell, at most four per atom)
    _check(orc, x, sig, L, (1, 2), d, width=n)

"""Distance shells of the Verlet rows: forces right after a build (shell 0
alone) and along runs whose displacement grows through the shells, against the
oracle, with rows at the edges of the in-place ordering (32 rows of 64 entries
down to one of 2048, and rows too long for it; also of the export's, whose
rows past 512 entries take another sort), a skin of zero, one lane and
several per atom."""
import os

import numpy as np
import pytest
import torch

from paper_2112_12271_amd import hdmd as H
from paper_2112_12271_amd import inputs
from tests.gpu_util import csr_equal, dev, force_err, gpu_list

pytestmark = pytest.mark.gpu


def _ball(n, d, r, L, seed):
    g = np.random.default_rng(seed)
    u = g.normal(size=(n, d))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    x = 0.3 * L * np.ones(d) + r * g.uniform(size=(n, 1)) ** (1.0 / d) * u
    return np.where(x >= L / 2, x - L, x)


@pytest.mark.parametrize("n", [2, 64, 65, 66, 129, 257, 512, 513, 514, 1025, 2049, 2050, 2600])
def test_rows_of_every_ordering_width(orc, n):
    """All atoms within the list radius of each other: rows of n - 1 entries,
    in every shell."""
    d, L, cut, skin = 3, 8.0, 1.0, 0.5
    x = _ball(n, d, 0.74, L, n)
    sig = np.ones(n)
    s = H.System(d=d, n=n, box_l=L, potential=H.HDMD_HARMONIC, cutoff=cut, skin=skin, sigma_max=1.0,
                 max_neighbors=n)
    ref = orc.nlist_brute(x, sig, L, cut, skin)
    assert (np.diff(ref[0]) == n - 1).all()
    got, s, ws = gpu_list(s, x, sig)
    assert csr_equal(got, ref)
    F, E = H.hdmd_forces(s, dev(x), dev(sig), ws)
    Fo, _, Eo = orc.forces(x, sig, L, H.HDMD_HARMONIC, cut, 1.0, *ref)
    if n == 2:
        assert np.abs(F.cpu().numpy() - Fo).max() < 1e-12
    else:
        assert force_err(F.cpu().numpy(), Fo) < 1e-12
    assert abs(float(E) - Eo) <= 1e-12 * abs(Eo)
    # the list is the same after the force kernel has ordered its rows
    rp, cols = H.hdmd_nlist_export(s, ws)
    assert csr_equal((rp.cpu().numpy(), cols.cpu().numpy()), ref)


@pytest.mark.parametrize("d,n,phi", [(2, 700, 0.6), (4, 900, 0.35), (7, 3000, 0.08)])
@pytest.mark.parametrize("lpa", [1, 2, 4])
@pytest.mark.parametrize("skin", [0.0, 0.4])
def test_run_through_the_shells(orc, d, n, phi, lpa, skin):
    """60 steps of a hot liquid: the displacement passes through every shell
    and several rebuilds (skin 0: a rebuild at every step, no shells)."""
    sig = inputs.bidisperse(n, 1.0, 1.2, n)
    L = inputs.box_for_packing(d, sig, phi)
    x = inputs.uniform_positions(n, d, L, 5 * n)
    v = inputs.gaussian_velocities(n, d, 4.0, 7 * n)
    os.environ["HDMD_LPA"] = str(lpa)
    try:
        s = H.System(d=d, n=n, box_l=L, potential=H.HDMD_HARMONIC, cutoff=1.0, skin=skin,
                     sigma_max=1.2, max_neighbors=n)
        ws = H.workspace(s)
        X, V = dev(x), dev(v)
        st, _ = H.hdmd_step(s, X, V, dev(sig), ws, 60, 0.01)
    finally:
        del os.environ["HDMD_LPA"]
    xo, vo, _, _ = orc.vv(x, v, sig, L, H.HDMD_HARMONIC, 1.0, skin, 1.0, 60, 0.01)
    assert st.builds >= (60 if skin == 0 else 3)
    dx = X.cpu().numpy() - xo
    dx -= L * np.round(dx / L)
    assert np.abs(dx).max() < 1e-9
    assert np.abs(V.cpu().numpy() - vo).max() < 1e-9

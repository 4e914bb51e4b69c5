"""A lone system's circle form takes four home atoms per wave where at least an
eightieth of the box lies within the list radius, up to 8192 atoms, and sixteen
otherwise: lists and forces on both sides of either line, with last groups that
are not full."""
import numpy as np
import pytest

from paper_2112_12271_amd import hdmd as H
from paper_2112_12271_amd import inputs
from tests.gpu_util import csr_equal, dev, force_err, gpu_list

pytestmark = pytest.mark.gpu
CUT, SKIN = 1.0, 0.25


@pytest.mark.parametrize("d,n,nc", [
    (3, 3, 2), (4, 65, 2), (3, 1022, 2), (8, 1027, 2), (6, 8192, 2), (6, 8193, 2),
    (3, 1021, 5), (3, 1024, 5), (5, 1025, 3), (7, 1023, 3), (2, 6, 4), (6, 900, 2.7), (6, 901, 2.75),
])
def test_lists_and_forces(orc, d, n, nc):
    L = nc * (CUT * 1.4 + SKIN) * 1.01
    x = inputs.uniform_positions(n, d, L, 17 * n + d)
    sig = inputs.bidisperse(n, 1.0, 1.4, n)
    ref = orc.nlist_brute(x, sig, L, CUT, SKIN)
    s = H.System(d=d, n=n, box_l=L, potential=H.HDMD_HARMONIC, cutoff=CUT, skin=SKIN, sigma_max=1.4,
                 max_neighbors=max(int(np.diff(ref[0]).max()), 1), subcells=H.HDMD_SUBCELLS_FULL)
    got, s, ws = gpu_list(s, x, sig)
    assert csr_equal(got, ref)
    # 1e-12 of F_rms: the bound of every FP64 force test here
    F, E = H.hdmd_forces(s, dev(x), dev(sig), ws)
    Fo, _, Eo = orc.forces(x, sig, L, H.HDMD_HARMONIC, CUT, 1.0, *ref)
    if np.abs(Fo).max() > 0:
        assert force_err(F.cpu().numpy(), Fo) < 1e-12
        assert abs(float(E) - Eo) <= 1e-12 * abs(Eo)
    else:
        assert np.abs(F.cpu().numpy()).max() == 0 and float(E) == 0
    # the rows in shells hold the same list
    rp, cols = H.hdmd_nlist_export(s, ws)
    assert csr_equal((rp.cpu().numpy(), cols.cpu().numpy()), ref)

"""The circle form of small systems with three subcells per axis and more: both
sides of its size limit (128 * 3^d atoms, 8192 at most), quarters of tiles that
are not full, boxes of many list radii (where the f16 margin of the chord test
is a large part of the list radius), pairs at their list radius up to a few
ulps and across the box faces, and batches whose systems rebuild in few waves
and in many.  Lists are sets of pairs decided in FP64: they equal the
definition's exactly."""
import numpy as np
import pytest

from paper_2112_12271_amd import hdmd as H
from paper_2112_12271_amd import inputs
from tests.gpu_util import csr_equal, dev, gpu_list

pytestmark = pytest.mark.gpu
CUT, SKIN = 1.0, 0.25


def _system(d, n, nc, seed):
    """Atoms in pairs at their list radius up to a few ulps."""
    L = nc * (CUT * 1.4 + SKIN) * 1.01
    g = np.random.default_rng(seed)
    x = inputs.uniform_positions(n, d, L, seed + 1)
    sig = np.full(n, 1.4)
    sig[: n // 2] = 1.0
    for p in range(0, n - 1, 2):
        v = g.normal(size=d)
        v /= np.linalg.norm(v)
        r = CUT * 0.5 * (sig[p] + sig[p + 1]) + SKIN
        x[p + 1] = x[p] + (r + g.integers(-3, 4) * np.spacing(r)) * v
    x -= L * np.floor(x / L + 0.5)
    x[x >= L / 2] = -L / 2
    return x, sig, L


@pytest.mark.parametrize("d,n,nc", [
    (2, 1152, 20), (2, 1153, 20), (3, 3456, 9), (3, 3457, 9), (3, 17, 3), (3, 79, 30), (4, 8191, 6),
    (4, 8193, 6), (5, 2063, 3), (6, 3000, 3), (7, 1000, 3),
])
def test_list_of_small_systems(orc, d, n, nc):
    x, sig, L = _system(d, n, nc, 10 * n + d)
    ref = orc.nlist_brute(x, sig, L, CUT, SKIN)
    s = H.System(d=d, n=n, box_l=L, potential=H.HDMD_HARMONIC, cutoff=CUT, skin=SKIN, sigma_max=1.4,
                 max_neighbors=min(max(int(np.diff(ref[0]).max()), 1), 1 << 20),
                 subcells=H.HDMD_SUBCELLS_FULL)
    got, _, _ = gpu_list(s, x, sig)
    assert csr_equal(got, ref)


@pytest.mark.parametrize("copies", [1, 40])
def test_batch_of_quarter_and_whole_tiles(copies):
    """FIRE alone and in a batch, bit for bit: one system rebuilds in quarters
    of tiles, forty of them at once (2600 tiles) in whole ones."""
    d, n = 4, 4129
    sig = inputs.bidisperse(n, 1.0, 1.4, 3)
    L = inputs.box_for_packing(d, sig, 0.5)
    x = inputs.uniform_positions(n, d, L, 4)
    s = H.System(d=d, n=n, box_l=L, potential=H.HDMD_HARMONIC, cutoff=1.0, skin=0.1, sigma_max=1.4,
                 max_neighbors=400)
    params = H.hdmd_fire_defaults(f_tol=1e-30)
    params.max_iter = 40
    X, SG, ws = dev(x), dev(sig), H.workspace(s)
    H.hdmd_fire_minimize(s, X, SG, ws, params)
    want = X.cpu().numpy()
    B = H.Batch(max_slots=copies, max_atoms=copies * (n + 64), max_cells=copies * 8192)
    keep = []
    for k in range(copies):
        keep.append((dev(x), H.workspace(s)))
        B.hdmd_batch_add_fire(k, s, keep[k][0], SG, keep[k][1], params)
    B.hdmd_batch_run(45)
    state, _ = B.hdmd_batch_poll()
    assert (np.asarray(state[:copies]) == H.HDMD_SLOT_DONE).all()
    for k in range(copies):
        assert np.array_equal(B.hdmd_batch_take(k)[0].cpu().numpy(), want)

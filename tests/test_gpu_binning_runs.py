"""The binning's last workgroup takes the prefix sums (up to 65536 subcells) and
the scatter (up to 8192 atoms) in the rebuilds of a run; a first build past
1024 atoms has launches of their own for them.  Runs that rebuild at every
step, from both kinds of first build, against the oracle."""
import numpy as np
import pytest

from paper_2112_12271_amd import hdmd as H
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,L", [
    (2, 1024, 40.0),      # the last size of the fused first build
    (2, 1025, 40.0),
    (2, 8192, 110.0),     # scatter by the binning in the run, in a launch at first
    (2, 8193, 110.0),     # scatter in a launch always
    (2, 70000, 352.0),    # 251^2 subcells: the binning's prefix, several passes
    (2, 70000, 360.0),    # 257^2 subcells: past it
])
def test_rebuilds_at_every_step(orc, d, n, L):
    """10 steps with skin 0: the positions agree within rounding (1e-9) as long
    as every rebuild lists every pair."""
    rng = np.random.default_rng(n + int(L))
    x = rng.uniform(-L / 2, L / 2, size=(n, d))
    v = rng.normal(size=(n, d))
    sig = np.ones(n)
    s = H.System(d=d, n=n, box_l=L, potential=H.HDMD_HARMONIC, cutoff=1.4, skin=0.0, sigma_max=1.0,
                 max_neighbors=64, subcells=H.HDMD_SUBCELLS_FULL)
    X, V = dev(x), dev(v)
    st, _ = H.hdmd_step(s, X, V, dev(sig), H.workspace(s), 10, 0.01)
    xo, vo, _, _ = orc.vv(x, v, sig, L, H.HDMD_HARMONIC, 1.4, 0.0, 1.0, 10, 0.01)
    assert st.builds >= 10
    dx = X.cpu().numpy() - xo
    dx -= L * np.round(dx / L)
    assert np.abs(dx).max() < 1e-9
    assert np.abs(V.cpu().numpy() - vo).max() < 1e-9

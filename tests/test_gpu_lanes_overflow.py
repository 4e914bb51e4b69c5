"""The lanes per atom of the force kernels are chosen on a list that holds: a
first build whose rows overflow (the usual way to a row width) leaves the
choice to the next; and on a list of about the system's own size."""
import dataclasses

import pytest

from paper_2112_12271_amd import hdmd as H
from paper_2112_12271_amd import inputs
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [H.HDMD_FP64, H.HDMD_MIXED])
def test_an_overflowed_build_does_not_settle_the_lanes(prec):
    """d = 2, 18000 atoms, rows of about 360 (a key no other test uses): 282
    waves of one lane per atom leave most SIMDs without work while each walks
    its row, so that any timing on the list gives more lanes."""
    d, n, rl = 2, 18000, 1.6
    L = (n * 3.14159 * rl * rl / 360.0) ** 0.5
    x, sig = dev(inputs.uniform_positions(n, d, L, 5)), dev(inputs.bidisperse(n, 1.0, 1.2, 6))
    s = H.System(d=d, n=n, box_l=L, potential=H.HDMD_HARMONIC, cutoff=1.0, skin=0.4, sigma_max=1.2,
                 precision=prec, max_neighbors=32)
    rc, rw = H.hdmd_build_nlist(s, x, sig, H.workspace(s))
    assert rc == H.HDMD_ERR_NLIST_OVERFLOW and rw > 300
    assert H.hdmd_build_config(s)[4] == 1
    s = dataclasses.replace(s, max_neighbors=rw + 8)
    rc, _ = H.hdmd_build_nlist(s, x, sig, H.workspace(s))
    assert rc == H.HDMD_OK
    assert H.hdmd_build_config(s)[4] > 1


def test_the_lanes_of_one_size_do_not_bind_another():
    """Rows of the same length in a system eight times as large fill the SIMDs
    with one lane per atom: its lanes are its own to time."""
    rl = 1.6

    def make(n):
        L = (n * 3.14159 * rl * rl / 250.0) ** 0.5
        x, sig = dev(inputs.uniform_positions(n, 2, L, 7)), dev(inputs.bidisperse(n, 1.0, 1.2, 8))
        return H.System(d=2, n=n, box_l=L, potential=H.HDMD_HARMONIC, cutoff=1.0, skin=0.4, sigma_max=1.2,
                        max_neighbors=400), x, sig

    small, x, sig = make(18000)
    assert H.hdmd_build_nlist(small, x, sig, H.workspace(small))[0] == H.HDMD_OK
    assert H.hdmd_build_config(small)[4] > 1
    large, x, sig = make(144000)
    assert H.hdmd_build_config(large)[4] == 1
    assert H.hdmd_build_nlist(large, x, sig, H.workspace(large))[0] == H.HDMD_OK
    assert H.hdmd_build_config(large)[4] in (1, 2, 4)

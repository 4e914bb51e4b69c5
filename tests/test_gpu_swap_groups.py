"""SWAP's search of the linked subcells in groups of 64: groups with one atom to
several hundred, a last group that is not full (3^6 and 5^2 subcells), empty
subcells, and attempts of every word of a batch put off by others."""
import numpy as np
import pytest
import torch

from paper_2112_12271_amd import hdmd as H
from paper_2112_12271_amd import inputs
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,L,crowd", [
    (2, 900, 18.0, 0),
    (2, 1500, 30.0, 400),   # 400 atoms in one subcell
    (3, 60, 12.0, 0),       # mostly empty subcells
    (6, 3000, 5.2, 0),
])
@pytest.mark.parametrize("half", [False, True])
def test_swap_in_groups(orc, d, n, L, crowd, half):
    if half and d == 6:
        pytest.skip("five half-size subcells per axis do not fit")
    g = np.random.default_rng(n + d)
    x = inputs.uniform_positions(n, d, L, n)
    x[:crowd] = 0.1 + 1.2 * g.uniform(size=(crowd, d))
    sig = g.choice([1.0, 1.2, 1.4], size=n)
    natt = 700
    pairs = g.integers(0, n, size=(natt, 2)).astype(np.int32)
    u = g.uniform(size=natt)
    T = 0.3
    sig_o, acc_o, de_o, na_o = orc.swap(x, sig, L, H.HDMD_HARMONIC, 1.0, 1.0, pairs, u, T)
    # no decision of the oracle sits within rounding of the Metropolis threshold
    thr = np.where(de_o <= 0, 2.0, np.exp(-np.maximum(de_o, 0) / T))
    assert np.all((de_o <= 0) | (np.abs(u - thr) > 1e-9))
    s = H.System(d=d, n=n, box_l=L, potential=H.HDMD_HARMONIC, cutoff=1.0, skin=0.2, sigma_max=1.4,
                 max_neighbors=n, subcells=H.HDMD_SUBCELLS_HALF if half else H.HDMD_SUBCELLS_FULL)
    D = dev(sig)
    acc, na = H.hdmd_swap(s, dev(x), D, H.workspace(s), torch.as_tensor(pairs, device="cuda"), dev(u), T)
    assert na == na_o
    assert np.array_equal(acc.cpu().numpy(), acc_o)
    assert np.array_equal(D.cpu().numpy(), sig_o)

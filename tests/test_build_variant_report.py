"""CPU test: hdmd_build_config reports the list-build variant that runs, also
where HDMD_BUILD_BLK asks for one that there is not."""
import pytest

from paper_2112_12271_amd import hdmd as H


@pytest.mark.parametrize("asked,linked", [("1", 1), ("2", 2), ("4", 4), ("3", 4), ("64", 4), ("1026", 4), ("0", 1)])
def test_variant_is_one_that_runs(monkeypatch, asked, linked):
    monkeypatch.setenv("HDMD_BUILD_BLK", asked)
    big = H.System(d=3, n=9000, box_l=30.0, subcells=H.HDMD_SUBCELLS_FULL)
    assert H.hdmd_build_config(big)[3] == linked
    half = H.System(d=3, n=900, box_l=12.0, subcells=H.HDMD_SUBCELLS_HALF)
    assert H.hdmd_build_config(half)[1:4:2] == (2, linked)
    # the circle form (small systems, n_cell <= 2) has one variant
    small = H.System(d=3, n=900, box_l=12.0, subcells=H.HDMD_SUBCELLS_FULL)
    assert H.hdmd_build_config(small)[3] == 1
    wide = H.System(d=8, n=90000, box_l=3.2, subcells=H.HDMD_SUBCELLS_FULL)
    assert H.hdmd_build_config(wide)[2:4] == (2, 1)

"""The largest sizes that are taken and the first past them: bands and padded grids on both sides of the joint
rule, the longest rows of the image grid (host-only)."""

import pytest

from paper_1807_11560_amd import lddmm as L

TAKEN = [
    # grid, band, spectral
    ((64, 64, 64), (64, 64, 64), (96, 113, 96)),
    ((64, 64, 64), (64, 64, 64), (96, 96, 240)),
    ((8, 8, 8), (4, 4, 4), (256, 57, 6)),
    ((8, 8, 256), (4, 4, 4), (6, 256, 256)),
    ((64, 64, 256), (64, 64, 64), (96, 96, 96)),
    ((2048, 8, 256), (64, 8, 64), (96, 12, 96)),
]
REFUSED = [
    ((64, 64, 64), (64, 64, 64), (96, 114, 96)),
    ((64, 64, 64), (64, 64, 64), (96, 96, 241)),
    ((8, 8, 8), (4, 4, 4), (256, 58, 6)),
    ((8, 8, 257), (4, 4, 4), (6, 6, 6)),
    ((8, 8, 8), (4, 4, 4), (6, 257, 6)),
]


@pytest.mark.parametrize("grid,band,spectral", TAKEN)
def test_taken(grid, band, spectral):
    assert L.Problem(grid=grid, band=band, spectral=spectral, time_steps=1).workspace_bytes() > 0


@pytest.mark.parametrize("grid,band,spectral", REFUSED)
def test_refused(grid, band, spectral):
    with pytest.raises(L.LddmmError) as e:
        L.Problem(grid=grid, band=band, spectral=spectral, time_steps=1).workspace_bytes()
    assert e.value.code == L.E_SHAPE
    assert "LDS" not in str(e.value)  # no kernel's tile is the reason

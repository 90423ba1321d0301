"""Instance norms by the length of a row: 256 threads up to 9 216 points, 1024 up to 36 864, rows that are read again above."""
import pytest

import test_gpu_layers as layers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nlat,nlon,theta", [(192, 192, 0.04), (193, 192, 0.04), (5, 16, 1.2), (96, 96, 0.08), (97, 96, 0.08)])
def test_row_lengths(monkeypatch, nlat, nlon, theta):
    gd = dict(grid_type=1, nlat_in=nlat, nlon_in=nlon, nlat_out=nlat, nlon_out=nlon, theta=theta)
    monkeypatch.setattr(layers, "MHA_CASES", [(gd, 1, 16, 1)])
    layers.test_mha_block(0)

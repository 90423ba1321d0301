"""Global attention launches whose units of 128 tokens do not share out evenly over the compute units: the rest goes in halves (at most 16 of
32 units left), or stays (17); the last unit of a slice full, half full and with a single token; against float64."""
import pytest

from test_gpu_global import run_global
from test_gpu_global_split import _inputs

pytestmark = pytest.mark.gpu


# units of a die: 41 (9 left), 44 (12), 48 (16), 49 (17), 65 (1)
@pytest.mark.parametrize("nlat,nlon,B,H", [(13, 24, 12, 9), (4, 64, 2, 88), (3, 43, 8, 24), (3, 64, 4, 49), (10, 32, 1, 130)])
def test_rest(nlat, nlon, B, H):
    run_global(0, nlat, nlon, B, H, _inputs(nlat, nlon, B * H, 12), [0, B * H // 2, B * H - 1], case="rest %dx%d" % (nlat, nlon))

"""Owners that are the two classes of a finer grid (kPairs), taken in and written four columns of a latitude at a time: rows that end
within a patch or a workgroup, fewer columns than a patch, patches of one, two and four owner rows, a segment left incomplete, both
directions; against the float64 oracle."""
import pytest

from paper_2505_11157_amd.workloads import make_inputs
from test_gpu_nattn import C_DERIVED, run_case
from test_gpu_nattn_bf16 import run_bf16

pytestmark = pytest.mark.gpu

# coarse latitudes and longitudes, fine latitudes, theta
SHAPES = [(9, 4, 17, 1.3), (9, 20, 17, 0.5), (10, 36, 19, 0.3), (7, 68, 13, 1.2), (17, 64, 33, 0.25), (6, 12, 11, 3.1)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [16, 32, 64])
@pytest.mark.parametrize("up", [True, False])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_pairs(i, up, d, dtype):
    lat, lon, fine, theta = SHAPES[i]
    sizes = (lat, lon, fine, 2 * lon) if up else (fine, 2 * lon, lat, lon)
    c = dict(zip(("nlat_in", "nlon_in", "nlat_out", "nlon_out"), sizes), kind="nattn", grid_type=0, theta=theta, batch=1, heads=3, d=d, dtype=dtype)
    c, arrs = make_inputs(c, seed=6300 + 10 * i + d)
    run = (lambda *a: run_bf16(*a)) if dtype == "bf16" else (lambda c, a, s, n: run_case(c, a, s, C=C_DERIVED, case=n))
    run(c, arrs, [0, 2], "pairs%d%s[d%d]" % (i, "up" if up else "down", d))

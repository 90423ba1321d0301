"""The patch kernels (float32 and bf16 tensors on the bf16 matrix cores) where their tables and stages have edges: fewer columns than a
patch or a workgroup owns, owner rows that leave a segment incomplete, whole circles of a length that is and is not a multiple of
four, arcs over several stages, a last chunk that reaches around the circle, classes on either side, more walked rows than a table holds;
every width they are built for."""
import pytest

from paper_2505_11157_amd.workloads import make_inputs
from test_gpu_nattn import C_DERIVED, run_case
from test_gpu_nattn_bf16 import run_bf16

pytestmark = pytest.mark.gpu


def _c(gt, lat_in, lon_in, lat_out, lon_out, theta):
    return dict(kind="nattn", grid_type=gt, nlat_in=lat_in, nlon_in=lon_in, nlat_out=lat_out, nlon_out=lon_out, theta=theta,
                batch=1, heads=9, dtype="f32")


SHAPES = [_c(1, 6, 4, 6, 4, 1.2), _c(1, 9, 7, 9, 7, 0.9), _c(0, 9, 12, 9, 12, 3.1), _c(0, 18, 35, 18, 35, 0.5), _c(0, 37, 72, 37, 72, 0.2),
          _c(0, 21, 132, 21, 132, 0.45), _c(0, 19, 57, 9, 19, 0.6), _c(0, 9, 20, 17, 40, 0.5), _c(0, 300, 8, 300, 8, 1.6)]


@pytest.mark.parametrize("d", [16, 20, 32, 64])
@pytest.mark.parametrize("ci", range(len(SHAPES)))
def test_patches(ci, d):
    # nine slices: eight of them are dealt out to the XCDs whole, the last one by workgroups
    c, arrs = make_inputs(dict(SHAPES[ci], d=d), seed=5200 + 10 * ci + d)
    run_case(c, arrs, [0, 7, 8], C=C_DERIVED, case="patch%d[d%d]" % (ci, d))


@pytest.mark.parametrize("d", [16, 20, 32, 64])
@pytest.mark.parametrize("ci", range(len(SHAPES)))
def test_patches_bf16(ci, d):
    c, arrs = make_inputs(dict(SHAPES[ci], d=d, dtype="bf16"), seed=5300 + 10 * ci + d)
    run_bf16(c, arrs, [0, 7, 8], "patch-bf16-%d[d%d]" % (ci, d))

"""The patch kernels on circles of an even length that is no multiple of four, whose pieces astride the end of a row are loaded in halves: fewer
columns than a piece, whole circles and arcs over the seam, finer grids on either side, channels that are not the kernel's."""
import pytest

import paper_2505_11157_amd as S
from paper_2505_11157_amd.workloads import make_inputs
from test_gpu_nattn import C_DERIVED, debug_switches, run_case
from test_gpu_nattn_bf16 import run_bf16

pytestmark = pytest.mark.gpu

SHAPES = [(9, 2, 9, 2, 2.0), (9, 6, 9, 6, 1.2), (12, 22, 12, 22, 3.1), (24, 46, 24, 46, 0.5), (11, 130, 11, 130, 0.5), (21, 42, 11, 14, 0.6),
          (11, 22, 21, 66, 0.5), (13, 26, 13, 13, 0.7)]


@pytest.mark.parametrize("own", [False, True])
@pytest.mark.parametrize("d", [16, 24, 32, 64])
@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_even_rows(i, d, own):
    sizes = dict(zip(("nlat_in", "nlon_in", "nlat_out", "nlon_out", "theta"), SHAPES[i]))
    with debug_switches(S.S2_DEBUG_OWN_PATCHES if own else 0):
        for dtype in ("f32", "bf16"):
            c, arrs = make_inputs(dict(sizes, kind="nattn", grid_type=1, batch=1, heads=3, d=d, dtype=dtype), seed=6500 + 10 * i + d)
            if dtype == "bf16":
                run_bf16(c, arrs, [0, 2], "even%d[d%d]" % (i, d))
            else:
                run_case(c, arrs, [0, 2], C=C_DERIVED, case="even%d[d%d]" % (i, d))

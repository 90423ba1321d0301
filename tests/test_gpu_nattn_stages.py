"""dk and dv of float32 tensors with 32 channels: stages of 24 chunks, 48 looked up at once.  Disks that hold the sphere, with numbers of
chunks next to one and two stages, against the float64 oracle.  By default these small launches may share patches, in stages of 32 chunks;
test_gpu_nattn_shared_patches runs them with a patch for every wavefront, on the 24."""
import math

import pytest

import paper_2505_11157_amd as S
from paper_2505_11157_amd.workloads import make_inputs
from test_gpu_nattn import C_DERIVED, debug_switches, run_case

pytestmark = pytest.mark.gpu


# rows x chunks of a row: 22 23 24 25 | 47 48 49 | 95 96 97 (and 24 and 48 in another way)
@pytest.mark.parametrize("rows,chunks", [(22, 1), (23, 1), (6, 4), (5, 5), (47, 1), (6, 8), (7, 7), (19, 5), (12, 8), (97, 1), (3, 8), (2, 24)])
def test_chunk_counts(rows, chunks):
    c = dict(kind="nattn", grid_type=1, nlat_in=rows, nlon_in=4 * chunks, nlat_out=rows, nlon_out=4 * chunks, theta=math.pi, batch=1, heads=2,
             d=32, dtype="f32")
    c, arrs = make_inputs(c, seed=6100 + 100 * rows + chunks)
    run_case(c, arrs, [0, 1], C=C_DERIVED, case="stages%dx%d" % (rows, chunks))


@pytest.mark.parametrize("ratio", [3, 4])
@pytest.mark.parametrize("rows,chunks", [(23, 1), (6, 4), (7, 7), (12, 8), (16, 6)])
def test_owners_of_three_and_four_classes(rows, chunks, ratio):
    # owners are the classes of a grid of three or four times the longitudes, each with a patch of its own
    c = dict(kind="nattn", grid_type=1, nlat_in=rows, nlon_in=4 * chunks * ratio, nlat_out=rows, nlon_out=4 * chunks, theta=math.pi, batch=1, heads=2,
             d=32, dtype="f32")
    c, arrs = make_inputs(c, seed=6200 + 100 * rows + chunks)
    with debug_switches(S.S2_DEBUG_OWN_PATCHES):
        run_case(c, arrs, [0, 1], C=C_DERIVED, case="classes%d-%dx%d" % (ratio, rows, chunks))

"""Random grids, whole circles and infinities on the patch kernels of large launches, with a patch for every wavefront, and on those that share patches:
the grids are small, so that by default the rule for small launches has some on either."""
import pytest

import paper_2505_11157_amd as S
import test_gpu_nattn as nattn
import test_gpu_nattn_band as band
import test_gpu_nattn_nonfinite_kinds as kinds
import test_gpu_nattn_whole_circles as circles
from test_gpu_nattn import debug_switches

pytestmark = pytest.mark.gpu
MODES = {"own": S.S2_DEBUG_OWN_PATCHES, "quarters": S.S2_DEBUG_QUARTERS}


def _params(test):
    """The parameters of a test, by name"""
    out = [{}]
    for mark in getattr(test, "pytestmark", []):
        if mark.name == "parametrize":
            names = mark.args[0].split(",")
            out = [dict(o, **dict(zip(names, v if len(names) > 1 else (v,)))) for o in out for v in mark.args[1]]
    return out


@pytest.mark.parametrize("seed", range(64))
@pytest.mark.parametrize("mode", MODES)
def test_random_small_grids(mode, seed):
    with debug_switches(MODES[mode]):
        nattn.test_random_small_grids(seed)


@pytest.mark.parametrize("seed", range(48))
def test_random_tuned_shapes(seed):
    with debug_switches(S.S2_DEBUG_OWN_PATCHES):
        nattn.test_random_tuned_shapes(seed)


@pytest.mark.parametrize("seed", range(16))
def test_random_tuned_upsampling(seed):
    with debug_switches(S.S2_DEBUG_OWN_PATCHES):
        nattn.test_random_tuned_upsampling(seed)


@pytest.mark.parametrize("seed", range(30))
def test_random_shapes(seed):
    with debug_switches(S.S2_DEBUG_OWN_PATCHES):
        band.test_band_kernels_random_shapes(seed)


@pytest.mark.parametrize("p", _params(circles.test_whole_circles), ids=str)
@pytest.mark.parametrize("mode", MODES)
def test_whole_circles(mode, p):
    with debug_switches(MODES[mode]):
        circles.test_whole_circles(**p)


@pytest.mark.parametrize("p", _params(kinds.test_infinities), ids=str)
@pytest.mark.parametrize("mode", MODES)
def test_infinities(mode, p):
    with debug_switches(MODES[mode]):
        kinds.test_infinities(**p)

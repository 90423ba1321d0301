"""Small launches of the patch kernels, whose heavy workgroups go in parts that two or all four wavefronts share: the edge cases of the
patch kernels with a patch for every wavefront, by halves and by quarters (by default they run on any of these), the sizes at which
the default changes from one to the next, and non-finite values where only one of the sharing wavefronts meets them."""
import math

import pytest
import torch

import paper_2505_11157_amd as S
import test_gpu_nattn_nonfinite as nonfinite
import test_gpu_nattn_pairs as pairs
import test_gpu_nattn_patch as patch
import test_gpu_nattn_stages as stages
from paper_2505_11157_amd.workloads import make_inputs
from test_gpu_nattn import C_DERIVED, debug_switches, run_case

pytestmark = pytest.mark.gpu
MODES = {"own": S.S2_DEBUG_OWN_PATCHES, "halves": S.S2_DEBUG_HALVES, "quarters": S.S2_DEBUG_QUARTERS}


@pytest.mark.parametrize("d", [16, 20, 32, 64])
@pytest.mark.parametrize("ci", range(len(patch.SHAPES)))
@pytest.mark.parametrize("mode", MODES)
def test_patches(mode, ci, d):
    with debug_switches(MODES[mode]):
        patch.test_patches(ci, d)
        patch.test_patches_bf16(ci, d)


@pytest.mark.parametrize("d,dtype", [(16, "bf16"), (32, "f32"), (64, "bf16"), (64, "f32")])
@pytest.mark.parametrize("i", range(len(pairs.SHAPES)))
@pytest.mark.parametrize("mode", MODES)
def test_pairs(mode, i, d, dtype):
    with debug_switches(MODES[mode]):
        pairs.test_pairs(i, True, d, dtype)
        pairs.test_pairs(i, False, d, dtype)


@pytest.mark.parametrize("rows,chunks", [(22, 1), (23, 1), (6, 4), (5, 5), (47, 1), (6, 8), (7, 7), (19, 5), (12, 8), (97, 1), (3, 8), (2, 24)])
def test_chunk_counts(rows, chunks):
    with debug_switches(S.S2_DEBUG_OWN_PATCHES):
        stages.test_chunk_counts(rows, chunks)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["k", "v-inf", "dout"])
@pytest.mark.parametrize("ci", range(len(nonfinite.SHAPES)))
@pytest.mark.parametrize("mode", MODES)
def test_non_finite_values(mode, ci, where, dtype):
    with debug_switches(MODES[mode]):
        nonfinite.test_non_finite_values_stay_in_their_neighborhoods(ci, where, dtype)


@pytest.mark.parametrize("heads", [1, 2, 4, 5, 8])
def test_sizes_between_the_lists(heads):
    # 24 x 48, disks of five latitudes: quarters, halves, and a patch for every wavefront, by slices
    c = dict(kind="nattn", grid_type=1, nlat_in=24, nlon_in=48, nlat_out=24, nlon_out=48, theta=5 * math.pi / 24, batch=2, heads=heads, d=32, dtype="f32")
    c, arrs = make_inputs(c, seed=6400 + heads)
    run_case(c, arrs, [0, 2 * heads - 1], C=C_DERIVED, case="shares%d" % heads)


def test_logits_far_apart_in_the_parts():
    # references of the softmax that differ by far more than an exponential holds from one wavefront's keys to the next one's
    g = S.s2_grid_init(S.S2_GRID_LEGENDRE_GAUSS, 12, 32, 12, 32, math.pi)
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn(1, 1, 32, 12, 32, generator=gen, device="cuda") for _ in range(3))
    q = 40 * q
    out, lse = S.s2_nattn_fwd(g, q, k, v, 1.0)
    with debug_switches(S.S2_DEBUG_OWN_PATCHES):
        own, own_lse = S.s2_nattn_fwd(g, q, k, v, 1.0)
    assert (lse - own_lse).abs().max() <= 1e-5 * own_lse.abs().max()
    # logits of some 600 carry 600 * 2^-23 * a few of rounding into the weights
    assert (out - own).abs().max() <= 1e-3

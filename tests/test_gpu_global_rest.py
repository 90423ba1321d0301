"""Global attention launches whose units of 128 tokens do not share out evenly over the compute units: the rest goes in halves (at most 16 of
32 units left), or stays (17); the last unit of a slice full, half full and with a single token; against float64, and one slice against another."""
import math

import numpy as np
import pytest
import torch

import paper_2505_11157_amd as S
from test_gpu_global import run_global
from test_gpu_global_split import _inputs

pytestmark = pytest.mark.gpu


# units of a die: 41 (9 left), 44 (12), 48 (16), 49 (17), 49 (17)
@pytest.mark.parametrize("nlat,nlon,B,H", [(13, 24, 12, 9), (4, 64, 2, 88), (3, 43, 8, 24), (3, 64, 4, 49), (10, 32, 1, 130)])
def test_rest(nlat, nlon, B, H):
    run_global(0, nlat, nlon, B, H, _inputs(nlat, nlon, B * H, 12), [0, B * H // 2, B * H - 1], case="rest %dx%d" % (nlat, nlon))


def test_a_single_unit_left_that_is_half_full():
    # 192 tokens, 260 slices: two units a slice, 65 of a die; the last ones of a die go in halves, units 64, 129 and so on up to 519: the first
    # of slice 32, and the second of slices 64 and 259, whose second half would begin at the token count
    run_global(0, 3, 64, 4, 65, _inputs(3, 64, 260, 13), [0, 32, 64, 259], case="rest 3x64")


@pytest.mark.parametrize("nlat,nlon,B,H", [(13, 24, 12, 9), (4, 64, 2, 88), (3, 64, 4, 65), (31, 62, 3, 11)])
def test_equal_slices(nlat, nlon, B, H):
    # Units in halves sum their keys in two chains, from the same reference as the others, so that the same probabilities are rounded alike:
    # results differ by the order of float32 sums, some 4e-7, which moves a share 4e-7 / 2^-8 of the bf16 results by one step of 2^-8, that is
    # sqrt(4e-7 2^-8) = 4e-5 of the norm; four times that.  (With a reference for each chain: 1e-3 and more.)
    a = [torch.from_numpy(x).to("cuda:0").to(torch.bfloat16).reshape(1, 1, nlat * nlon, 64) for x in _inputs(nlat, nlon, 1, 14)]
    q, k, v = (x.expand(B, H, -1, -1).contiguous() for x in a[:3])
    g = S.s2_grid_init(0, nlat, nlon, nlat, nlon, math.pi)
    out, lse = S.s2_attn_global_fwd(g, q, k, v, 0.125)
    out, lse = out.double().reshape(B * H, -1), lse.double().reshape(B * H, -1)
    apart = ((out - out[0]).norm(dim=1) / out[0].norm()).cpu().numpy()
    print("%dx%d: %d of %d slices apart, at most %.1e, lse %.1e" % (nlat, nlon, (apart > 0).sum(), B * H, apart.max(), (lse - lse[0]).abs().max()))
    assert np.isfinite(apart).all() and apart.max() <= 1.6e-4
    assert (lse - lse[0]).abs().max() <= 1e-6 * (1 + lse[0].abs().max())

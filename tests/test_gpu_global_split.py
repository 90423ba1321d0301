"""Small global attention launches share the streamed side among the wavefronts of a workgroup; against float64.

Sizes at the edges of that split: one token tile, a last workgroup without a live query, token counts below and above a
stage of 64, 32-token tiles that do and do not straddle latitudes, pole rows of weight zero, and launches just below and
above the lines of 256 and 320 blocks.  Tolerances are those of the other global tests (bf16 results, float32 lse).
"""
import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_2505_11157_amd as S
from paper_2505_11157_amd.workloads import round_to_bf16
from test_gpu_global import run_global

pytestmark = pytest.mark.gpu


def _inputs(nlat, nlon, nbh, seed):
    rng = np.random.default_rng(seed)
    return [round_to_bf16(rng.standard_normal((nbh, nlat * nlon, 64)).astype(np.float32)) for _ in range(4)]


@pytest.mark.parametrize("gt,nlat,nlon,B,H", [(0, 3, 5, 1, 1), (0, 3, 32, 1, 1), (1, 4, 16, 1, 2), (0, 5, 13, 2, 1),
                                              (0, 9, 21, 1, 3), (1, 6, 32, 1, 1), (0, 46, 90, 1, 1),
                                              (0, 9, 32, 5, 17), (0, 9, 32, 2, 43), (0, 13, 24, 2, 53),
                                              (0, 13, 24, 12, 9)])
def test_split_launches(gt, nlat, nlon, B, H):
    # fifteen tokens average the rounding of a probability over a short sum only: twice the bound
    run_global(gt, nlat, nlon, B, H, _inputs(nlat, nlon, B * H, 11), [0, B * H - 1], case="split %dx%d" % (nlat, nlon),
               rel=4e-2 if nlat * nlon < 32 else 2e-2)


@pytest.mark.parametrize("tile", [0, 1])
def test_a_key_tile_of_logits_at_minus_infinity(tile):
    """Thirty-two keys at minus infinity, all that one pair of wavefronts meets in its first stage: exp gives 0."""
    nlat, nlon = 9, 32
    q, k, v, _ = _inputs(nlat, nlon, 1, 5)
    q[..., 0] = np.abs(q[..., 0]) + 0.5
    k[0, 32 * tile:32 * tile + 32, 0] = -np.inf
    ref, ref_lse = O.global_fwd(0, nlat, nlon, *(a.astype(np.float64) for a in (round_to_bf16(q), k, v)), 0.125)
    dev = torch.device("cuda:0")
    fold = lambda a: torch.from_numpy(a).reshape(1, 1, nlat * nlon, 64).to(dev).to(torch.bfloat16).contiguous()
    g = S.s2_grid_init(0, nlat, nlon, nlat, nlon, math.pi)
    out, lse = S.s2_attn_global_fwd(g, *(fold(a) for a in (q, k, v)), 0.125)
    out, lse = out.float().cpu().numpy().reshape(ref.shape), lse.cpu().numpy().reshape(ref_lse.shape)
    assert np.isfinite(ref).all()
    assert (np.abs(out - ref) <= 2e-2 * np.abs(ref) + 2e-2 * np.sqrt((ref ** 2).mean())).all()
    assert (np.abs(lse - ref_lse) <= 1e-6 + 1e-5 * np.abs(ref_lse)).all()

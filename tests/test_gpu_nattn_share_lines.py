"""Launches of which wavefronts share patches take no longer than with a patch for every wavefront: on either side of the lines of the rule, where
the lines of one kernel would cost another one up to two fifths."""
import math

import pytest
import torch

import paper_2505_11157_amd as S
from test_gpu_nattn import debug_switches

pytestmark = pytest.mark.gpu
E, G = S.S2_GRID_EQUIANGULAR, S.S2_GRID_LEGENDRE_GAUSS
F32, BF16 = torch.float32, torch.bfloat16


def _us(f):
    f()
    torch.cuda.synchronize()
    best = 1e9
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 20 * 1e3)
    return best


# forward; by halves against unsplit 1.35, 1.23 and 1.26 (bf16, 64 channels), 1.41, 1.25 and 1.12 (owners of a finer grid); and two that gain
@pytest.mark.parametrize("grid,sizes,theta,slices,d,dtype", [
    (E, (118, 235, 118, 235), 0.061, 2, 64, BF16), (G, (25, 51, 25, 51), 0.36, 9, 64, BF16), (E, (64, 126, 64, 126), 0.2725, 4, 64, BF16),
    (E, (39, 75, 77, 150), 0.1238, 3, 64, BF16), (E, (39, 75, 77, 150), 0.1238, 3, 16, F32), (E, (39, 75, 77, 150), 0.1238, 3, 32, F32),
    (G, (64, 128, 64, 128), 7 * math.pi / 64, 1, 32, F32), (G, (64, 128, 64, 128), 7 * math.pi / 64, 1, 64, BF16)])
def test_no_slower_than_unsplit(grid, sizes, theta, slices, d, dtype):
    g = S.s2_grid_init(grid, *sizes, theta)
    gen = torch.Generator(device="cuda").manual_seed(1)
    q = torch.randn(slices, 1, d, *sizes[2:], generator=gen, device="cuda").to(dtype)
    k, v = (torch.randn(slices, 1, d, *sizes[:2], generator=gen, device="cuda").to(dtype) for _ in range(2))
    step = lambda: S.s2_nattn_fwd(g, q, k, v, d ** -0.5)
    with debug_switches(S.S2_DEBUG_OWN_PATCHES):
        unsplit = _us(step)
    us = _us(step)
    print("%s %d slices d = %d %s: unsplit %.1f us, as the rule has it %.1f" % (sizes, slices, d, dtype, unsplit, us), flush=True)
    assert us <= 1.1 * unsplit

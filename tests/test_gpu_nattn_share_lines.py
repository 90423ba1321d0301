"""Which launches of the patch kernels share the patches of heavy workgroups, told by the bits of their results: sums in parts are added in another
order.  On either side of the lines of the rule; the times beside the launches that do not share are by halves (or quarters) against unsplit."""
import math

import pytest
import torch

import paper_2505_11157_amd as S
from test_gpu_nattn import debug_switches

pytestmark = pytest.mark.gpu
E, G, L = S.S2_GRID_EQUIANGULAR, S.S2_GRID_LEGENDRE_GAUSS, S.S2_GRID_LEGENDRE_GAUSS_LOBATTO
F32, BF16 = torch.float32, torch.bfloat16


def _bits(g, t, flags):
    q, k, v, dout = t
    with debug_switches(flags):
        out, lse = S.s2_nattn_fwd(g, q, k, v, q.shape[2] ** -0.5)
        return [x.float().flatten() for x in (out, lse) + tuple(S.s2_nattn_bwd(g, q, k, v, out, lse, dout, q.shape[2] ** -0.5))]


def _same(a, b):
    return [torch.equal(x, y) for x, y in zip(a, b)]


@pytest.mark.parametrize("grid,sizes,theta,slices,d,dtype,shares", [
    # much work for kernels that fit several workgroups on a compute unit: forward 1.35, 1.23, 1.26
    (E, (118, 235, 118, 235), 0.061, 2, 64, BF16, 0), (G, (25, 51, 25, 51), 0.36, 9, 64, BF16, 0), (E, (64, 126, 64, 126), 0.2725, 4, 64, BF16, 0),
    (G, (145, 290, 145, 290), 0.05265, 1, 40, BF16, 0),      # channels that are not the kernel's: 1.10
    # disks of a spacing or two: backward 1.45, 1.36, 1.15, 1.35
    (G, (100, 200, 100, 200), 0.01605, 1, 40, BF16, 0), (G, (121, 240, 121, 240), 0.01182, 1, 32, F32, 0), (E, (53, 104, 53, 104), 0.05715, 1, 40, BF16, 0),
    (L, (46, 93, 46, 93), 0.03557, 8, 16, F32, 0),
    # launches that gain
    (G, (64, 128, 64, 128), 7 * math.pi / 64, 1, 32, F32, 2), (G, (64, 128, 64, 128), 7 * math.pi / 64, 2, 32, F32, 1),
    (G, (64, 128, 64, 128), 7 * math.pi / 64, 1, 64, BF16, 2), (G, (64, 128, 64, 128), 7 * math.pi / 64, 1, 16, F32, 2)])
def test_lines(grid, sizes, theta, slices, d, dtype, shares):
    g = S.s2_grid_init(grid, *sizes, theta)
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    t = [torch.randn(slices, 1, d, *(sizes[2:] if i in (0, 3) else sizes[:2]), generator=gen, device="cuda:0").to(dtype) for i in range(4)]
    got = _bits(g, t, 0)
    lists = [_bits(g, t, f) for f in (S.S2_DEBUG_OWN_PATCHES, S.S2_DEBUG_HALVES, S.S2_DEBUG_QUARTERS)]
    print(sizes, slices, d, dtype, [_same(got, x) for x in lists], flush=True)
    assert all(_same(got, lists[shares]))
    for i in {0, 1, 2} - {shares}:
        assert not all(_same(got, lists[i]))     # (the lists can be told apart here)


# forward by halves: owners of a finer grid 1.41, 1.25, 1.12; up to 100 chunks with much work 1.28 (68 chunks)
@pytest.mark.parametrize("grid,sizes,theta,slices,d,dtype", [
    (E, (39, 75, 77, 150), 0.1238, 3, 64, BF16), (E, (39, 75, 77, 150), 0.1238, 3, 16, F32), (E, (39, 75, 77, 150), 0.1238, 3, 32, F32),
    (S.S2_GRID_EQUIANGULAR_TRAPEZOID, (58, 117, 58, 117), 0.08028, 4, 8, F32), (L, (113, 226, 226, 452), 0.01829, 1, 16, F32)])
def test_lines_of_the_forward(grid, sizes, theta, slices, d, dtype):
    g = S.s2_grid_init(grid, *sizes, theta)
    gen = torch.Generator(device="cuda:0").manual_seed(2)
    t = [torch.randn(slices, 1, d, *(sizes[2:] if i in (0, 3) else sizes[:2]), generator=gen, device="cuda:0").to(dtype) for i in range(4)]
    got, own, halves = (_bits(g, t, f)[:2] for f in (0, S.S2_DEBUG_OWN_PATCHES, S.S2_DEBUG_HALVES))
    assert all(_same(got, own)) and not all(_same(got, halves))

"""The float32 forward of d = e = 32 on upsampling grids, by columns: parity with the float64 oracle, and the same bits when everything is
rolled by whole steps of the coarse circle; two to four classes, whole circles, an incomplete last segment, a last workgroup beyond the circle."""
import math

import pytest
import torch

import paper_2505_11157_amd as S
from paper_2505_11157_amd.workloads import make_inputs
from test_gpu_nattn import C_DERIVED, run_case

pytestmark = pytest.mark.gpu

SHAPES = [(0, 17, 72, 33, 144, 0.4), (1, 12, 76, 20, 228, 0.9), (0, 9, 80, 17, 320, 3.1), (0, 33, 128, 65, 256, 0.12), (2, 20, 72, 40, 144, 0.5),
          (3, 21, 84, 42, 168, 0.6), (0, 90, 72, 60, 144, 2.6)]


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_columns(i):
    gt, lat_in, lon_in, lat_out, lon_out, theta = SHAPES[i]
    c = dict(kind="nattn", grid_type=gt, nlat_in=lat_in, nlon_in=lon_in, nlat_out=lat_out, nlon_out=lon_out, theta=theta, batch=1, heads=2, d=32, dtype="f32")
    c, arrs = make_inputs(c, seed=6400 + i)
    run_case(c, arrs, [0, 1], C=C_DERIVED, case="columns%d" % i)


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_rolled_bit_for_bit(i):
    gt, lat_in, lon_in, lat_out, lon_out, theta = SHAPES[i]
    g, r = S.s2_grid_init(gt, lat_in, lon_in, lat_out, lon_out, theta), lon_out // lon_in
    gen = torch.Generator(device="cuda").manual_seed(i)
    q, k, v = (torch.randn(1, 3, 32, *s, generator=gen, device="cuda") for s in ((lat_out, lon_out), (lat_in, lon_in), (lat_in, lon_in)))
    out, lse = S.s2_nattn_fwd(g, q, k, v, 1 / math.sqrt(32))
    for s in (1, 5, lon_in - 1):
        o, l = S.s2_nattn_fwd(g, torch.roll(q, r * s, 4), torch.roll(k, s, 4), torch.roll(v, s, 4), 1 / math.sqrt(32))
        assert torch.equal(o, torch.roll(out, r * s, 4)) and torch.equal(l, torch.roll(lse, r * s, 3))

"""GPU parity of the patch kernels away from the longitude counts and grid pairs they were first written for: the edges of
tiles, stages, classes and row tables, float32 and bf16 tensors, against the float64 oracle."""
import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_2505_11157_amd as S
from paper_2505_11157_amd.workloads import grid_dict, make_inputs, round_to_bf16
from test_gpu_nattn import C_DERIVED, run_case
from test_gpu_nattn_bf16 import run_bf16

pytestmark = pytest.mark.gpu


def _c(gt, lat_in, lon_in, lat_out, lon_out, theta, heads=2, d=16):
    return dict(kind="nattn", grid_type=gt, nlat_in=lat_in, nlon_in=lon_in, nlat_out=lat_out, nlon_out=lon_out, theta=theta,
                batch=1, heads=heads, d=d, dtype="f32")


SHAPES = [
    # odd longitude counts: short arcs only / arcs on the common grid / whole circles with a ragged last tile
    _c(0, 33, 65, 33, 65, 0.25), _c(0, 19, 129, 19, 129, 0.5, d=32), _c(1, 12, 101, 12, 101, 1.3, d=64),
    # fewer longitudes than a tile, than 32, than a stage; one longitude
    _c(0, 9, 10, 9, 10, 0.9), _c(0, 9, 17, 9, 17, 0.6, d=64), _c(1, 16, 31, 16, 31, 0.8, d=32), _c(0, 17, 33, 17, 33, math.pi),
    _c(1, 4, 1, 4, 1, 0.9),
    # channel counts between the instantiated ones
    _c(0, 17, 40, 17, 40, 0.4, d=24), _c(0, 17, 45, 17, 45, 0.4, d=7), _c(1, 12, 26, 12, 26, 0.6, d=50),
    # classes of a finer grid: ratio 2 with even and odd counts, 3, whole circles, either direction
    _c(0, 33, 66, 17, 33, 0.4), _c(0, 17, 33, 33, 66, 0.4), _c(1, 24, 96, 12, 48, 0.5, d=64), _c(1, 12, 48, 24, 96, 0.5, d=64),
    _c(0, 25, 93, 13, 31, 0.45, d=32), _c(0, 13, 31, 25, 93, 0.45, d=32), _c(0, 9, 24, 5, 12, math.pi), _c(3, 5, 12, 9, 24, math.pi),
    # more than 64 walked rows per workgroup (two registers per lane), and exactly 64
    _c(0, 97, 16, 97, 16, 1.2), _c(0, 66, 12, 66, 12, math.pi), _c(0, 65, 32, 33, 16, 1.2), _c(1, 64, 8, 64, 8, math.pi),
    # a zero-weight pole row on a grid pair with classes
    _c(2, 24, 56, 12, 28, 0.5), _c(2, 12, 28, 24, 56, 0.6),
]


@pytest.mark.parametrize("ci", range(len(SHAPES)))
def test_any_grid_f32(ci):
    c, arrs = make_inputs(SHAPES[ci], seed=4100 + ci)
    run_case(c, arrs, range(2), C=C_DERIVED, case="any%d" % ci)


@pytest.mark.parametrize("ci", range(len(SHAPES)))
def test_any_grid_bf16(ci):
    c, arrs = make_inputs(dict(SHAPES[ci], dtype="bf16"), seed=4200 + ci)
    run_bf16(c, arrs, range(2), "any-bf16-%d" % ci)


@pytest.mark.parametrize("batch,heads,d", [(4, 8, 16), (4, 8, 32), (4, 8, 64), (3, 5, 16)])
def test_any_grid_many_slices(batch, heads, d):
    # enough workgroups for several owner tiles per wavefront, on an odd longitude count
    c, arrs = make_inputs(dict(_c(0, 41, 75, 41, 75, 0.3, d=d), batch=batch, heads=heads), seed=4300 + d)
    run_case(c, arrs, [0, batch * heads - 1], C=C_DERIVED, case="any-many[d%d]" % d)


def _launches(f):
    S.s2_trace_reset()
    S.s2_trace_enable(True)
    try:
        f()
        return {n for n, _, _ in S.s2_trace_entries()}
    finally:
        S.s2_trace_enable(False)
        S.s2_trace_reset()


@pytest.mark.parametrize("batch", [3, 12])
@pytest.mark.parametrize("lon,d", [(76, 16), (75, 16), (75, 7), (76, 32), (75, 32), (76, 24), (76, 64), (75, 64), (75, 50)])
def test_any_grid_many_slices_bf16(lon, d, batch):
    # 24 slices make two owner tiles per wavefront, 96 make four (forward and, for 16 channels, backward), in each way a row is
    # staged: four columns at a time (76 longitudes), column by column (75), and with channels missing
    c, arrs = make_inputs(dict(_c(0, 41, lon, 41, lon, 0.3, heads=8, d=d), batch=batch, dtype="bf16"), seed=4600 + d)
    names = _launches(lambda: run_bf16(c, arrs, [0, 8 * batch - 1], "any-many-bf16[%d,d%d,b%d]" % (lon, d, batch)))
    assert names == {"nattn_fwd_patch", "nattn_bwd_dq_patch", "nattn_bwd_dkdv_patch"}, names


@pytest.mark.parametrize("lon", [76, 75])
@pytest.mark.parametrize("d", [16, 32, 64])
def test_any_grid_many_slices_f32(lon, d):
    # 32 slices: two owner tiles per wavefront (16 channels: in the forward and dq)
    c, arrs = make_inputs(dict(_c(0, 41, lon, 41, lon, 0.3, heads=8, d=d), batch=4), seed=4700 + d)
    names = _launches(lambda: run_case(c, arrs, [0, 31], C=C_DERIVED, case="any-many[%d,d%d]" % (lon, d)))
    assert names == {"nattn_fwd_patch", "nattn_bwd_dq_patch", "nattn_bwd_dkdv_patch"}, names


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,e", [(16, 32), (32, 16), (64, 8), (5, 64), (24, 17)])
def test_value_width_other_than_key_width(d, e, dtype):
    for ci, heads in ((0, 2), (17, 2), (1, 24)):
        c, arrs = make_inputs(dict(SHAPES[ci], d=max(d, e), heads=heads, dtype=dtype), seed=4800 + d)
        c["d"] = d
        arrs = [np.ascontiguousarray(a[:, :n]) for a, n in zip(arrs, (d, d, e, e))]
        run = (lambda: run_bf16(c, arrs, [0, heads - 1], "e%d-bf16" % ci)) if dtype == "bf16" else \
            (lambda: run_case(c, arrs, [0, heads - 1], C=C_DERIVED, case="e%d" % ci))
        assert _launches(run) == {"nattn_fwd_patch", "nattn_bwd_dq_patch", "nattn_bwd_dkdv_patch"}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,e", [(65, 65), (80, 24), (16, 128), (128, 128)])
def test_more_than_64_channels(d, e, dtype):
    # grids on which the lanes of a wavefront leave the walk over a disk at different times (3:1, upsampling), equal ones, and
    # a partly filled wavefront; 33 .. 128 channels in one to four blocks of dk and dv
    for ci, c in enumerate((_c(0, 12, 15, 7, 5, 1.1), _c(0, 9, 12, 9, 24, 0.6), _c(1, 8, 70, 8, 70, 0.5))):
        c, arrs = make_inputs(dict(c, d=max(d, e), dtype=dtype), seed=4900 + d)
        c["d"] = d
        arrs = [np.ascontiguousarray(a[:, :n]) for a, n in zip(arrs, (d, d, e, e))]
        if dtype == "bf16":
            run_bf16(c, arrs, range(2), "wide%d[%d,%d]" % (ci, d, e))
        else:
            run_case(c, arrs, range(2), C=C_DERIVED, case="wide%d[%d,%d]" % (ci, d, e))


@pytest.mark.parametrize("lon,d", [(80, 16), (75, 32), (80, 64), (75, 24)])
def test_bf16_sums_carry_float32_weights(lon, d):
    # The weights of the bf16 sums (probabilities) are float32 values.  A relative error u of a sum moves its rounding to 8 bits
    # with a probability of about u / 2^-8: float32 sums (u of some 2^-24 .. 2^-21) give shares of 1e-4 to 4e-4 of results that
    # are not the correctly rounded ones, weights of 16 or 17 bits (u of about 2^-17) 2e-3.
    c, arrs = make_inputs(dict(_c(0, 41, lon, 41, lon, 0.3, heads=4, d=d), dtype="bf16"), seed=4500 + d)
    arrs, gd, scale = [round_to_bf16(a) for a in arrs], grid_dict(c), 1 / math.sqrt(d)
    g = S.s2_grid_init(0, 41, lon, 41, lon, 0.3)
    q, k, v, dout = (torch.from_numpy(a).to("cuda:0")[None].to(torch.bfloat16).contiguous() for a in arrs)
    out, lse = S.s2_nattn_fwd(g, q, k, v, scale)
    dv = S.s2_nattn_bwd(g, q, k, v, out, lse, dout, scale)[2]
    a64 = [a.astype(np.float64) for a in arrs]
    for name, x, ref in (("out", out, O.nattn_fwd(gd, *a64[:3], scale)[0]), ("dv", dv, O.nattn_bwd(gd, *a64, scale)[2])):
        share = (x[0].float().cpu().numpy() != round_to_bf16(ref.astype(np.float32))).mean()
        print("not correctly rounded: %s %.2e" % (name, share))
        assert share < 8e-4, (name, share)


@pytest.mark.parametrize("dtype,d", [(torch.float32, 16), (torch.float32, 64), (torch.bfloat16, 64)])
def test_slices_of_more_than_four_gigabytes_stay_on_the_tiles(dtype, d):
    # 16.8 million points: 64 float32 channels of a slice are more than 32-bit offsets reach (staged column by column then, 16
    # channels four columns at a time).  Against the shape-agnostic kernels; both are held to 1e-6 + 1e-5 |ref| elsewhere.
    nlat, nlon = 2900, 5800
    g = S.s2_grid_init(0, nlat, nlon, nlat, nlon, 1.5 * math.pi / (nlat - 1))
    gen = torch.Generator(device="cuda:0").manual_seed(46)
    q, k, v, dout = (torch.randn((1, 1, d, nlat, nlon), generator=gen, device="cuda:0", dtype=dtype) for _ in range(4))
    res, scale = [], 1 / math.sqrt(d)
    for flag in (0, S.S2_DEBUG_NO_BAND):
        S.s2_debug_control(flag, S.S2_DEBUG_NO_BAND & ~flag)
        S.s2_trace_reset()
        S.s2_trace_enable(True)
        try:
            out, lse = S.s2_nattn_fwd(g, q, k, v, scale)
            saved = res[0][:2] if res else (out, lse)   # one forward result for both backward passes
            res.append((out, lse) + S.s2_nattn_bwd(g, q, k, v, *saved, dout, scale))
            names = {n for n, _, _ in S.s2_trace_entries()}
        finally:
            S.s2_trace_enable(False)
            S.s2_trace_reset()
            S.s2_debug_control(0, S.S2_DEBUG_NO_BAND)
        assert all(("generic" in n) == bool(flag) for n in names), names
    for name, a, b in zip(("out", "lse", "dq", "dk", "dv"), *res):
        rel = 2e-2 if a.dtype == torch.bfloat16 else 2e-5
        for x, y in zip(a.reshape(-1, nlat, nlon), b.reshape(-1, nlat, nlon)):
            x, y = x.float(), y.float()
            assert bool(((x - y).abs() <= 2e-6 + rel * (y.abs() + y.square().mean().sqrt())).all()), name

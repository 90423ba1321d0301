"""Non-finite inputs on the patch kernels: a NaN or an infinity at a point reaches the points whose disk holds
it and no others.  The pattern of finite results must be the oracle's, and the finite results must be right, to the bounds
of the plain cases (bf16: with the allowance that test_gpu_nattn_bf16 derives for D formed from the rounded `out`)."""
import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_2505_11157_amd as S
from paper_2505_11157_amd.workloads import grid_dict, make_inputs, round_to_bf16

pytestmark = pytest.mark.gpu


def _c(gt, lat_in, lon_in, lat_out, lon_out, theta, d=16):
    return dict(kind="nattn", grid_type=gt, nlat_in=lat_in, nlon_in=lon_in, nlat_out=lat_out, nlon_out=lon_out, theta=theta,
                batch=1, heads=2, d=d, dtype="f32")


SHAPES = [
    # staged four columns at a time, column by column, and with channels missing; short arcs, long arcs, whole circles
    _c(0, 17, 32, 17, 32, 0.5), _c(0, 19, 129, 19, 129, 0.5, d=32), _c(0, 17, 40, 17, 40, 0.4, d=24), _c(1, 12, 101, 12, 101, 1.3, d=64),
    # classes of a finer grid, either direction
    _c(0, 33, 66, 17, 33, 0.4), _c(0, 17, 33, 33, 66, 0.4),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["k", "v", "v-inf", "q", "dout", "k-channel"])
@pytest.mark.parametrize("ci", range(len(SHAPES)))
def test_non_finite_values_stay_in_their_neighborhoods(ci, where, dtype):
    c, arrs = make_inputs(dict(SHAPES[ci], dtype=dtype), seed=4400 + ci)
    if dtype == "bf16":
        arrs = [round_to_bf16(a) for a in arrs]
    gd, d = grid_dict(c), c["d"]
    scale = 1 / math.sqrt(d)
    arrs = [a.copy() for a in arrs]
    x = dict(zip(("q", "k", "v", "dout"), arrs))[where.split("-")[0]]
    h, w = x.shape[2] // 2 - 1, x.shape[3] // 3
    x[0, 3 if where == "k-channel" else slice(None), h, w] = np.inf if where == "v-inf" else np.nan
    x[0, 1, 0, 0] = np.nan                              # and one at the pole, in one channel
    g = S.s2_grid_init(gd["grid_type"], gd["nlat_in"], gd["nlon_in"], gd["nlat_out"], gd["nlon_out"], gd["theta"])
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k, v, dout = (torch.from_numpy(a).to("cuda:0").reshape((1, 2) + a.shape[1:]).to(dt).contiguous() for a in arrs)
    out, lse = S.s2_nattn_fwd(g, q, k, v, scale)
    got = (out, lse) + tuple(S.s2_nattn_bwd(g, q, k, v, out, lse, dout, scale))
    a64 = [a.astype(np.float64) for a in arrs]
    brute = gd["nlon_in"] % gd["nlon_out"] != 0
    ref = tuple(O.nattn_fwd(gd, *a64[:3], scale, brute=brute)) + tuple(O.nattn_bwd(gd, *a64, scale, brute=brute))
    assert not all(np.isfinite(r).all() for r in ref)
    extra = {}
    if dtype == "bf16":
        dD = 2.0 ** -9 * np.abs(a64[3] * ref[0]).sum(axis=1, keepdims=True)
        extra["dq"] = abs(scale) * dD * O.nattn_fwd(gd, a64[0], a64[1], np.abs(a64[1]), scale, brute=brute)[0]
        extra["dk"] = abs(scale) * O.nattn_bwd(gd, a64[0], a64[1], a64[1], dD * np.abs(a64[0]), scale, brute=brute)[2]
    for name, a, r in zip(("out", "lse", "dq", "dk", "dv"), got, ref):
        a = a.float().reshape(r.shape).cpu().numpy().astype(np.float64)
        fin = np.isfinite(r)
        assert np.array_equal(np.isfinite(a), fin), "%s: %d of %d spoiled, %d expected" % (
            name, (~np.isfinite(a)).sum(), a.size, (~fin).sum())
        a, r, more = a[fin], r[fin], np.nan_to_num(extra[name])[fin] if name in extra else 0.0
        rms = np.sqrt((r ** 2).mean())
        rel = 2e-2 if dtype == "bf16" and name != "lse" else 1e-5
        # float32: the stated bound 1e-6 + 1e-5 |r|, with 1e-5 rms for the larger sums of the coarse grids' backward
        assert (np.abs(a - r) <= 1e-6 + rel * (np.abs(r) + rms) + more).all(), (name, np.abs(a - r).max())

"""Infinities beside the NaN of test_gpu_nattn_nonfinite, the upsampling forward of d = 32, and what values that are not finite cost."""
import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_2505_11157_amd as S
import test_gpu_nattn_nonfinite as base
from paper_2505_11157_amd.workloads import grid_dict, make_inputs, round_to_bf16

pytestmark = pytest.mark.gpu
INF, NAN = float("inf"), float("nan")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["k", "v", "v-inf", "q", "dout", "k-channel"])
def test_upsampling_forward_of_32_channels(monkeypatch, where, dtype):
    # float32: the forward by columns, the patches behind it
    monkeypatch.setattr(base, "SHAPES", [base._c(0, 9, 72, 17, 144, 0.5, d=32)])
    base.test_non_finite_values_stay_in_their_neighborhoods(0, where, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["q", "k", "v", "dout"])
@pytest.mark.parametrize("d", [16, 24, 32, 64])
def test_infinities(where, d, dtype):
    # one channel of one point infinite, of another minus infinite: the same results are finite as in float64, and they are right
    c, arrs = make_inputs(base._c(0, 17, 40, 17, 40, 0.4, d=d), seed=4500 + d)
    if dtype == "bf16":
        arrs = [round_to_bf16(a) for a in arrs]
    gd, scale = grid_dict(c), 1 / math.sqrt(d)
    arrs = [a.copy() for a in arrs]
    x = dict(zip(("q", "k", "v", "dout"), arrs))[where]
    x[0, 3, 8, 11], x[1, d - 1, 5, 39], x[1, 0, 0, 0] = INF, -INF, INF
    g = S.s2_grid_init(*(gd[n] for n in ("grid_type", "nlat_in", "nlon_in", "nlat_out", "nlon_out", "theta")))
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q, k, v, dout = (torch.from_numpy(a).to("cuda:0").reshape((1, 2) + a.shape[1:]).to(dt).contiguous() for a in arrs)
    out, lse = S.s2_nattn_fwd(g, q, k, v, scale)
    got = (out, lse) + tuple(S.s2_nattn_bwd(g, q, k, v, out, lse, dout, scale))
    a64 = [a.astype(np.float64) for a in arrs]
    with np.errstate(all="ignore"):
        ref = tuple(O.nattn_fwd(gd, *a64[:3], scale)) + tuple(O.nattn_bwd(gd, *a64, scale))
    assert not all(np.isfinite(r).all() for r in ref)
    for name, a, r in zip(("out", "lse", "dq", "dk", "dv"), got, ref):
        a = a.float().reshape(r.shape).cpu().numpy().astype(np.float64)
        fin = np.isfinite(r)
        if where == "k" and name == "dq":
            # the oracle leaves a logit of minus infinity out; here its weight of zero meets the infinite channel of the key, and 0 inf is NaN
            for b, ch in ((0, 3), (1, d - 1), (1, 0)):
                fin[b, ch] &= np.isfinite(a[b, ch])
        assert np.array_equal(np.isfinite(a), fin), "%s: %d of %d not finite, %d expected" % (name, (~np.isfinite(a)).sum(), a.size, (~fin).sum())
        # bf16: twice the usual bound, for D formed from the rounded out
        rel = 4e-2 if dtype == "bf16" and name != "lse" else 1e-5
        a, r = a[fin], r[fin]
        assert (np.abs(a - r) <= 1e-6 + rel * (np.abs(r) + np.sqrt((r ** 2).mean()))).all(), (name, np.abs(a - r).max())


def _ms(f):
    f()
    torch.cuda.synchronize()
    best = 1e9
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["one of k", "one of v", "one of dout", "all of q", "all of k", "all of v", "all of dout", "everything"])
def test_cost_of_nan(where, dtype):
    # (every owner that meets a NaN summed one neighbor and one channel after the other: 14 to 100 steps)
    B, H, d, nlat, nlon = 2, 8, 32, 129, 256
    g = S.s2_grid_init(0, nlat, nlon, nlat, nlon, 4 * math.pi / 128)
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    cast = torch.float32 if dtype == "f32" else torch.bfloat16
    t = {n: torch.randn(B, H, d, nlat, nlon, generator=gen, device="cuda:0").to(cast) for n in ("q", "k", "v", "dout")}

    def step():
        out, lse = S.s2_nattn_fwd(g, t["q"], t["k"], t["v"], d ** -0.5)
        S.s2_nattn_bwd(g, t["q"], t["k"], t["v"], out, lse, t["dout"], d ** -0.5)

    plain = _ms(step)
    if where.startswith("one"):
        t[where.split()[-1]][1, 2, 3, 40, 100] = NAN
    for n in t:
        if where in ("everything", "all of " + n):
            t[n].fill_(NAN)
    spoiled = _ms(step)
    print("%s %s: %.3f -> %.3f ms" % (dtype, where, plain, spoiled), flush=True)
    assert spoiled <= 5 * plain, (plain, spoiled)

"""Grids of 2^15 and more longitudes, whose arcs the tables of the patch kernels do not hold, and grids of fewer next to one of more, whose
rows stay classes of a finer latitude there: against a softmax over the neighbor lists in float64, its gradients from autograd."""
import math

import numpy as np
import pytest
import torch

import paper_2505_11157_amd as S

pytestmark = pytest.mark.gpu


def reference(g, q, k, v, dout, scale):
    """(out, lse, dq, dk, dv) of tensors [slices][channels][latitudes][longitudes] in float64."""
    q, k, v = (x.detach().double().requires_grad_() for x in (q, k, v))
    omega = torch.from_numpy(S.s2_grid_get_weights(g)[1]).to(q.device)
    m, (nlat_out, nlon_out), (nlat_in, nlon_in) = min(q.shape[3], k.shape[3]), q.shape[2:], k.shape[2:]
    up, down = nlon_out // m, nlon_in // m
    shift = down * torch.arange(m, device=q.device)
    out = torch.empty(v.shape[:2] + q.shape[2:], dtype=torch.float64, device=q.device)
    lse = torch.empty(q.shape[:1] + q.shape[2:], dtype=torch.float64, device=q.device)
    dq, dk, dv = (torch.zeros_like(x) for x in (q, k, v))
    for h in range(nlat_out):
        for s in range(up):
            at = torch.from_numpy(np.asarray(S.s2_grid_get_neighbors_at(g, h, s), dtype=np.int64)).to(q.device)
            lat, col = at // nlon_in, (at % nlon_in)[:, None] + shift
            index = lat[:, None] * nlon_in + col % nlon_in                    # [neighbors][output columns of the class]
            K, V = (x.flatten(2)[:, :, index] for x in (k, v))
            logit = scale * (q[:, :, h, s::up].unsqueeze(2) * K).sum(1) + torch.log(omega[lat])[:, None]
            L = torch.logsumexp(logit, 1)
            o = (torch.exp(logit - L.unsqueeze(1)).unsqueeze(1) * V).sum(2)
            grads = torch.autograd.grad((o * dout[:, :, h, s::up].double()).sum(), (q, k, v))
            for x, y in zip((dq, dk, dv), grads):
                x += y
            out[:, :, h, s::up], lse[:, h, s::up] = o.detach(), L.detach()
    return out, lse, dq, dk, dv


# cutoffs of a few and of some hundred offsets; equal grids, 2:1, 1:2, either side of 2^15; what runs (of the forward: of all three)
@pytest.mark.parametrize("lon_in,lon_out,d,dtype,theta,kernels", [
    (32768, 32768, 32, "f32", 0.0015, "stream"), (32768, 32768, 32, "f32", 0.012, "tiled<8 waves>"),
    (65536, 32768, 32, "f32", 0.0015, "tiled<1 wave>"), (65536, 32768, 32, "f32", 0.012, "tiled<8 waves>"),
    (32768, 65536, 32, "f32", 0.0015, "tiled<1 wave>"), (32768, 65536, 32, "f32", 0.012, "tiled<8 waves>"),
    (32772, 32772, 16, "f32", 0.0015, "generic"), (32768, 32768, 32, "bf16", 0.012, "generic"),
    (40000, 20000, 32, "f32", 0.0015, "patch"), (40000, 20000, 32, "f32", 0.012, "patch"), (40000, 20000, 16, "bf16", 0.012, "patch"),
    (20000, 40000, 24, "f32", 0.0015, "patch"), (20000, 40000, 24, "f32", 0.012, "patch"), (20000, 40000, 32, "bf16", 0.012, "patch"),
    (32764, 32764, 32, "f32", 0.0015, "patch"), (32764, 32764, 32, "f32", 0.012, "patch")])
def test_long_circles(lon_in, lon_out, d, dtype, theta, kernels):
    nlat, B = 3, 2
    g = S.s2_grid_init(1, nlat, lon_in, nlat, lon_out, theta)
    cast = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda:0").manual_seed(lon_in + d)
    rnd = lambda n: torch.randn(1, B, d, nlat, n, generator=gen, device="cuda:0").to(cast)
    q, k, v, dout = rnd(lon_out), rnd(lon_in), rnd(lon_in), rnd(lon_out)
    scale = 1 / math.sqrt(d)
    S.s2_trace_reset()
    S.s2_trace_enable(True)
    try:
        out, lse = S.s2_nattn_fwd(g, q, k, v, scale)
        got = (out, lse) + tuple(S.s2_nattn_bwd(g, q, k, v, out, lse, dout, scale))
        torch.cuda.synchronize()
        names = {n for n, _, _ in S.s2_trace_entries()}
    finally:
        S.s2_trace_enable(False)
        S.s2_trace_reset()
    assert "nattn_fwd_" + kernels in names and all(kernels.split("<")[0] in n or "dkdv2_tiled" in n for n in names), names
    want = reference(g, *(x[0] for x in (q, k, v, dout)), scale)
    assert S.s2_grid_device_flags(g) == 0
    for name, a, r in zip(("out", "lse", "dq", "dk", "dv"), got, want):
        a = a[0].double()
        rms = float((r ** 2).mean().sqrt())
        # float32: the bound of the plain cases, 1e-6 + 1e-5 |r|, with 1e-5 rms for sums over several hundred points; bf16: as elsewhere
        # (twice for dq and dk, whose D comes from the rounded out)
        rel = 1e-5 if dtype == "f32" or name == "lse" else 4e-2 if name in ("dq", "dk") else 2e-2
        assert bool(((a - r).abs() <= 1e-6 + rel * (r.abs() + rms)).all()), (name, float((a - r).abs().max()))

"""Finite float32 values near either end of the range, on the kernels that cut them into three bf16 terms.  The last term of a value
below 2^-110 ends at bf16's smallest number, 2^-133: such a factor is held to 2^-134, larger ones to their last bit.  A value of
(1 - 2^-9) 2^128 or more rounds to an infinite first term, and the sums it enters are evaluated without terms."""
import math

import pytest
import torch

import paper_2505_11157_amd as S
from test_gpu_nattn_long_circles import reference

pytestmark = pytest.mark.gpu
CUT = 2.0 ** -134            # how far the terms of a small factor are from it
FLOOR = 2.0 ** -149          # the rounding of a small result


def _nattn(d, seed):
    g = S.s2_grid_init(0, 17, 40, 17, 40, 0.4)
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    return g, [torch.randn(1, 2, d, 17, 40, generator=gen, device="cuda:0") for _ in range(4)], 1 / math.sqrt(d)


@pytest.mark.parametrize("e", [-120, -60, 60, 104, 110, 114, 118, 122, 125])
@pytest.mark.parametrize("d", [16, 24, 32, 64])
def test_attention_is_linear_down_to_small_values(d, e):
    # out is linear in v, the gradients are linear in dout: scaled by 2^-e they keep the plain bound, scaled too, and beyond that what
    # the cut of a factor leaves of it
    g, (q, k, v, dout), scale = _nattn(d, 4900 + d)
    s = 2.0 ** -e
    out, lse = S.s2_nattn_fwd(g, q, k, v, scale)
    small = S.s2_nattn_fwd(g, q, k, v * s, scale)[0]
    grads = S.s2_nattn_bwd(g, q, k, v, out, lse, dout * s, scale)
    ref = reference(g, q[0], k[0], v[0], dout[0], scale)
    weight = reference(g, q[0], k[0], v[0], torch.ones_like(dout[0]), scale)[4][:, :1]      # sum_i p_ij of an input point
    points = max(S.s2_grid_get_neighbors_at(g, h, 0).size for h in range(17))
    most_v = float(v[0].abs().sum(1).max())
    # a sum over p_ij of what each factor may be off; dS, whose weight is omega <= 1, is a factor of its own
    cut = {"out": CUT, "dv": CUT * weight, "dq": CUT * scale * float(k.abs().max()) * (most_v + points),
           "dk": CUT * scale * float(q.abs().max()) * (most_v * weight + points)}
    assert torch.equal(S.s2_nattn_fwd(g, q, k, v * s, scale)[1], lse)
    for name, a, r in zip(("out", "dq", "dk", "dv"), (small,) + tuple(grads), (ref[0],) + ref[2:]):
        rms = float((r ** 2).mean().sqrt())
        bound = s * (1e-6 + 1e-5 * (r.abs() + rms)) + cut[name] + FLOOR
        err = (a[0].double() - s * r).abs()
        assert bool((err <= bound).all()), (name, float((err / bound).max()))
    if e <= 110:
        # and nothing of the last bit is lost before 2^-110: the same as without the factor, within 2^-20
        err = float((small[0].double() - s * ref[0]).norm() / (s * ref[0]).norm())
        assert err < 2.0 ** -20, err


@pytest.mark.parametrize("d", [16, 24, 32, 64])
def test_attention_with_the_largest_values(d):
    g, (q, k, v, dout), scale = _nattn(d, 4950 + d)
    v, dout = v.clone(), dout.clone()
    v[0, 0, 3, 8, 11], v[0, 1, 0, 0, 5] = 3.4e38, -3.4e38
    out, lse = S.s2_nattn_fwd(g, q, k, v, scale)
    ref = reference(g, q[0], k[0], v[0], dout[0], scale)
    err = (out[0].double() - ref[0]).abs()
    assert bool((ref[0].abs() > 1e30).any()) and bool((err <= 2e-6 + 2e-5 * ref[0].abs()).all()), float((err / (ref[0].abs() + 0.1)).max())
    assert bool(((lse[0].double() - ref[1]).abs() <= 1e-6 + 1e-5 * ref[1].abs()).all())
    v[0, 0, 3, 8, 11], v[0, 1, 0, 0, 5] = 0.0, 0.0
    dout[0, 0, 5, 8, 11], dout[0, 1, 0, 16, 39] = 3.4e38, -3.4e38
    out, lse = S.s2_nattn_fwd(g, q, k, v, scale)
    dv = S.s2_nattn_bwd(g, q, k, v, out, lse, dout, scale)[2]
    ref = reference(g, q[0], k[0], v[0], dout[0], scale)
    err = (dv[0].double() - ref[4]).abs()
    assert bool((ref[4].abs() > 1e30).any()) and bool((err <= 2e-6 + 2e-5 * ref[4].abs() + 1e-5 * float(ref[4][0, 0].abs().max())).all())


@pytest.mark.parametrize("e", [-60, 60, 104, 110, 114, 118, 122, 125])
@pytest.mark.parametrize("cin,cout", [(16, 16), (128, 64), (48, 96), (16, 160)])
def test_channel_products_down_to_small_values(cin, cout, e):
    # on a grid with a cutoff below its spacing a point's only neighbor is itself: z = omega x, y = W z, dx = omega W^T dy, dW = sum dy z
    nlat, nlon, B = 9, 48, 2
    g = S.s2_grid_init(1, nlat, nlon, nlat, nlon, 0.01)
    omega = torch.from_numpy(S.s2_grid_get_weights(g)[1]).reshape(1, 1, nlat, 1)
    gen = torch.Generator().manual_seed(cin + cout)
    rnd = lambda *n: torch.randn(*n, generator=gen)
    x, w, dy = rnd(B, cin, nlat, nlon), rnd(cout, cin, 1), rnd(B, cout, nlat, nlon)
    dc = S.s2_disco_init(g, 1)
    flat = lambda t: t.transpose(0, 1).reshape(t.shape[1], -1)
    back = lambda t: t.reshape(-1, B, nlat, nlon).transpose(0, 1)
    s = 2.0 ** -e
    y, ws = S.s2_disco_fwd(dc, x.to("cuda:0"), (w * s).to("cuda:0"), None)
    dx = S.s2_disco_bwd(dc, x.to("cuda:0"), (w * s).to("cuda:0"), dy.to("cuda:0"), ws)[0]
    dw = S.s2_disco_bwd(dc, x.to("cuda:0"), (w * s).to("cuda:0"), (dy * s).to("cuda:0"), ws)[1]
    z, w, dy = (omega * x.double()).float().double(), w.double()[:, :, 0], dy.double()
    for name, a, r, factors in (("y", y, back(w @ flat(z)), back(torch.ones_like(w) @ flat(z).abs())),
                                ("dx", dx, omega * back(w.t() @ flat(dy)), omega * back(torch.ones_like(w.t()) @ flat(dy).abs())),
                                ("dw", dw[:, :, 0], flat(dy) @ flat(z).t(), torch.ones_like(flat(dy)) @ flat(z).abs().t())):
        rms = float((r ** 2).mean().sqrt())
        err = (a.double().cpu() - s * r).abs()
        # (128 sums at most, and what the mixing leaves of dz is itself a small value that psi^T takes from memory)
        bound = s * (1e-6 * rms + 1e-5 * (r.abs() + rms)) + CUT * factors + 2 * FLOOR
        assert bool((err <= bound).all()), (name, float((err / bound).max()))

"""Channel products with factors that are not finite: what float32 arithmetic makes of them, NaN and either infinity, at every result they
enter; at no other; and at the cost of a second pass, not of a sum per result.  On a Gaussian grid with a cutoff below its spacing a
point's only neighbor is itself, so that with one basis function z = omega x, y = W z + bias, dx = omega W^T dy, dW = sum dy z."""
import pytest
import torch

import paper_2505_11157_amd as S

pytestmark = pytest.mark.gpu
INF, NAN = float("inf"), float("nan")


# (32 | 64, 16) and (128, 64) take psi^T first in the backward, the others the channel mixing; one to four row blocks, and two of them
@pytest.mark.parametrize("cin,cout", [(16, 16), (32, 16), (64, 16), (48, 96), (128, 64), (64, 128), (16, 160)])
def test_kinds_of_results(cin, cout):
    nlat, nlon, B = 9, 48, 2
    g = S.s2_grid_init(1, nlat, nlon, nlat, nlon, 0.01)
    omega = torch.from_numpy(S.s2_grid_get_weights(g)[1]).reshape(1, 1, nlat, 1)
    gen = torch.Generator().manual_seed(cin + cout)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    x, w, dy = rnd(B, cin, nlat, nlon), rnd(cout, cin, 1), rnd(B, cout, nlat, nlon)
    w[4, 1], w[6, 3], w[6, 7], w[7, 2], w[9, 9] = 3.4e38, INF, -INF, NAN, -INF       # 3.4e38: rounds to an infinite first term
    w[12, 5] = 1e30                                                                # overflows only with large values of x
    x[0, 2, 4, 5], x[0, 5, 4, 5] = INF, -INF
    x[1, 11, 2, 40] = -INF
    x[1, 3, 5, 17] = NAN
    x[0, 3, 1, 1] = x[0, 9, 1, 2] = 0.0
    x[1, 5, 8, 47] = -1e20
    dy[0, 3, 3, 3], dy[1, 3, 6, 6], dy[1, 8, 2, 2], dy[0, 10, 7, 30] = INF, -INF, NAN, -INF
    dc = S.s2_disco_init(g, 1)
    dev = [t.to("cuda:0") for t in (x, w, dy)]
    y, ws = S.s2_disco_fwd(dc, dev[0], dev[1], None)
    dx, dw, _ = S.s2_disco_bwd(dc, dev[0], dev[1], dev[2], ws)
    x, w, dy = x.double(), w.double()[:, :, 0], dy.double()
    z = (omega * x).float().double()
    flat = lambda t: t.transpose(0, 1).reshape(t.shape[1], -1)
    # every sum from its single products: a matrix product need not take zero times infinity
    product = lambda a, b: torch.stack([(a[i][:, None] * b).sum(0) for i in range(a.shape[0])])
    back = lambda t: t.reshape(-1, B, nlat, nlon).transpose(0, 1)
    most = torch.finfo(torch.float32).max
    for name, got, want, terms in (("y", y, back(product(w, flat(z))), back(product(w.abs(), flat(z).abs()))),
                                   ("dx", dx, omega * back(product(w.t(), flat(dy))), omega * back(product(w.t().abs(), flat(dy).abs()))),
                                   ("dw", dw[:, :, 0], product(flat(dy), flat(z).t()), product(flat(dy).abs(), flat(z).abs().t()))):
        got = got.double().cpu()
        if name == "dx" and cout >= cin:
            # the channels are mixed first, and psi^T takes the halves of +d and -d = 0 and a spare term of weight zero from the planes:
            # an infinity, or twice a value that is too large, may be NaN there
            want = torch.where(want.abs() <= omega * most / 2, want, NAN)
            got = torch.where(torch.isfinite(got), got, NAN)
        want = torch.where(want.abs() > most, want.sign() * INF, want)
        assert torch.isnan(want).any() and torch.isfinite(want).any(), name
        assert torch.equal(torch.isnan(got), torch.isnan(want)), name
        assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)]), name
        fin = torch.isfinite(want)
        # 128 float32 roundings of the largest partial sum at most
        assert ((got - want).abs() <= 2.0 ** -17 * terms)[fin].all(), name


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


@pytest.mark.parametrize("value", [NAN, INF])
@pytest.mark.parametrize("where", ["x", "weight", "dy", "all of x", "all of the weight"])
def test_cost_of_values_that_are_not_finite(where, value):
    # a step of four is what the second pass may take of a training step (summed one by one: 6 to 28 steps)
    B, c, nlat, nlon = 4, 64, 129, 256
    dc = S.s2_disco_init(S.s2_grid_init(0, nlat, nlon, nlat, nlon, 0.05), 9)
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda:0")
    t = {"x": rnd(B, c, nlat, nlon), "weight": rnd(c, c, 9) / 24, "dy": rnd(B, c, nlat, nlon)}

    def step():
        _, ws = S.s2_disco_fwd(dc, t["x"], t["weight"], None)
        S.s2_disco_bwd(dc, t["x"], t["weight"], t["dy"], ws)

    plain = _ms(step)
    if where.startswith("all"):
        t[where.split()[-1]].fill_(value)
    else:
        t[where].view(-1)[t[where].numel() // 2 + 17] = value
    spoiled = _ms(step)
    assert spoiled <= 4 * plain, (plain, spoiled)

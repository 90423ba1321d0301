"""Channel products on grids of so many points that the rows of a tile lie further apart than 32-bit offsets reach.  On a grid with a
cutoff below its spacing a point's only neighbor is itself: z = omega x, y = W z, dx = omega W^T dy, dW = sum dy z."""
import pytest
import torch

import paper_2505_11157_amd as S

pytestmark = pytest.mark.gpu


def _disco(nlat, cin, cout):
    nlon = 65536
    g = S.s2_grid_init(1, nlat, nlon, nlat, nlon, 3e-8)
    gen = torch.Generator(device="cuda:0").manual_seed(nlat)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda:0")
    x, w, dy = rnd(1, cin, nlat, nlon), rnd(cout, cin, 1), rnd(1, cout, nlat, nlon)
    omega = torch.from_numpy(S.s2_grid_get_weights(g)[1]).to("cuda:0").reshape(nlat, 1)
    return S.s2_disco_init(g, 1), omega, x, w, dy


def test_products_of_far_rows():
    # a lane's offset, nine rows of 4 bytes a point, passes 2^32 from 119 304 648 points on
    nlat = 1821
    dc, omega, x, w, dy = _disco(nlat, 16, 16)
    assert 36 * nlat * 65536 >= 2 ** 32
    y, ws = S.s2_disco_fwd(dc, x, w, None)
    dx = S.s2_disco_bwd(dc, x, w, dy, ws)[0]
    w = w.double()[:, :, 0]
    for lat in (0, 1, nlat // 2, nlat - 1):
        for cols in (slice(0, 200), slice(65536 - 200, 65536)):
            z, d = omega[lat] * x[0, :, lat, cols].double(), dy[0, :, lat, cols].double()
            for a, r, terms in ((y, w @ z, w.abs() @ z.abs()), (dx, omega[lat] * (w.t() @ d), omega[lat] * (w.abs().t() @ d.abs()))):
                # 16 products and z itself, each rounded once
                assert bool(((a[0, :, lat, cols].double() - r).abs() <= 18 * 2.0 ** -24 * terms).all()), (lat, cols)


def test_weight_gradients_of_far_rows():
    # 128 rows of dy, offsets counted in points
    nlat = 513
    dc, omega, x, w, dy = _disco(nlat, 16, 128)
    assert 128 * nlat * 65536 >= 2 ** 32
    _, ws = S.s2_disco_fwd(dc, x, w, None)
    dw, db = S.s2_disco_bwd(dc, x, w, dy, ws)[1:3]
    ref, sums = torch.zeros(128, 16, dtype=torch.float64, device="cuda:0"), torch.zeros(128, dtype=torch.float64, device="cuda:0")
    for lat in range(0, nlat, 27):
        d, z = dy[0, :, lat:lat + 27].double(), omega[lat:lat + 27] * x[0, :, lat:lat + 27].double()
        ref += d.flatten(1) @ z.flatten(1).t()
        sums += d.flatten(1).sum(1)
    # sums of 33 million random products: of the order of their root mean square where a row is mistaken for another
    for a, r in ((dw[:, :, 0], ref), (db, sums)):
        assert float((a.double() - r).abs().max()) <= 1e-3 * float((r ** 2).mean().sqrt())

"""The channel products of the DISCO convolution at the edges of their tiles against the float64 oracle: 1 to 5 row blocks
of the output, contraction lengths that end inside a tile of the weight gradient, 144 points (half a slice over)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2505_11157_amd as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,K,cout", [(16, 9, 32), (64, 3, 64), (16, 8, 64), (16, 4, 48), (48, 5, 96), (16, 9, 128), (80, 3, 160), (208, 2, 16)])
def test_channel_tiles(cin, K, cout):
    gd = dict(grid_type=0, nlat_in=9, nlon_in=16, nlat_out=9, nlon_out=16, theta=0.8)
    B = 2
    rng = np.random.default_rng(cin + 7 * K + 31 * cout)
    d64 = lambda *s: rng.standard_normal(s).astype(np.float32).astype(np.float64)
    x, dy, weight, bias = d64(B, cin, 9, 16), d64(B, cout, 9, 16), d64(cout, cin, K), d64(cout)
    g = S.s2_grid_init(0, 9, 16, 9, 16, gd["theta"])
    dc = S.s2_disco_init(g, K)
    T = lambda a: torch.from_numpy(a.astype(np.float32)).to("cuda:0").contiguous()
    y, ws = S.s2_disco_fwd(dc, T(x), T(weight), T(bias))
    dx, dw, db = S.s2_disco_bwd(dc, T(x), T(weight), T(dy), ws)
    r_y, r_z = O.disco_fwd(gd, K, x, weight, bias)
    r_dx, r_dw, r_db = O.disco_bwd(gd, K, x, weight, bias, dy)
    sums = {"dw": np.einsum("bohw,bckhw->ock", np.abs(dy), np.abs(r_z)), "db": np.abs(dy).sum((0, 2, 3))}
    for name, got, ref in (("y", y, r_y), ("dx", dx, r_dx), ("dw", dw, r_dw), ("db", db, r_db)):
        err = np.abs(got.cpu().numpy().astype(np.float64) - ref)
        bound = 1e-6 + 1e-5 * np.abs(ref) + 2e-5 * np.sqrt((ref ** 2).mean()) + 8 * 2.0 ** -24 * sums.get(name, 0.0)
        assert (err <= bound).all(), (name, float(err.max()))

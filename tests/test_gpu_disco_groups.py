"""The DISCO contraction by groups of four owner latitudes: numbers of latitudes that leave 1, 2 or 3 of a group, basis counts on
either side of the line up to which two entries are taken at a time, one and two owners per lane, resampling both ways."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2505_11157_amd as S
from test_gpu_layers import close

pytestmark = pytest.mark.gpu


# nlat_in, nlon_in, nlat_out, nlon_out, theta, K
@pytest.mark.parametrize("size", [(5, 32, 5, 32, 0.9, 3), (6, 16, 6, 16, 1.2, 9), (7, 64, 7, 64, 0.8, 1), (9, 128, 9, 128, 0.6, 13),
                                  (9, 128, 9, 128, 0.6, 14), (10, 160, 10, 160, 0.5, 16), (17, 128, 9, 64, 0.4, 9),
                                  (13, 128, 4, 32, 0.7, 4), (11, 48, 6, 16, 3.1, 5)])
def test_groups(size):
    a, b, c, d, theta, K = size
    gd = dict(grid_type=0, nlat_in=a, nlon_in=b, nlat_out=c, nlon_out=d, theta=theta)
    B, cin, cout = 1, 16, 16
    rng = np.random.default_rng(sum(size[:4]) + K)
    f32 = lambda *s: rng.standard_normal(s).astype(np.float32)
    x, dy, weight, bias = f32(B, cin, a, b), f32(B, cout, c, d), f32(cout, cin, K), f32(cout)
    dc = S.s2_disco_init(S.s2_grid_init(0, a, b, c, d, theta), K)
    T = lambda v: torch.from_numpy(v).to("cuda:0")
    y, ws = S.s2_disco_fwd(dc, T(x), T(weight), T(bias))
    dx, dw, db = S.s2_disco_bwd(dc, T(x), T(weight), T(dy), ws)
    torch.cuda.synchronize()
    d64 = [v.astype(np.float64) for v in (x, weight, bias, dy)]
    r_y, r_z = O.disco_fwd(gd, K, *d64[:3])
    r_dx, r_dw, _ = O.disco_bwd(gd, K, *d64)
    case = "disco group %s K%d" % (size[:4], K)
    close(y.cpu().numpy(), r_y, "y", case)
    close(dx.cpu().numpy(), r_dx, "dx", case)
    close(dw.cpu().numpy(), r_dw, "dweight", case, np.einsum("bohw,bckhw->ock", np.abs(d64[3]), np.abs(r_z)))

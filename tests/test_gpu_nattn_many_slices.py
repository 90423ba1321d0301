"""More (batch, head) slices than one launch takes (2^32 threads): the launches are split, and every slice has the results that it has in a launch of a
few: bit for bit where none of them share patches, which few slices may, and up to rounding where they do."""
import pytest
import torch

import paper_2505_11157_amd as S
from test_gpu_nattn import debug_switches

pytestmark = pytest.mark.gpu


def test_more_threads_than_a_launch_takes():
    # 60 x 20 points are 30 workgroups of 256 threads of the patch kernels, 16.8 million of them (27 GB of tensors)
    B, H, nlat, nlon, d, e, dtype = 700, 801, 60, 20, 1, 1, torch.float32
    g = S.s2_grid_init(1, nlat, nlon, nlat, nlon, 0.1)
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    q, k, v, dout = (torch.empty(B, H, c, nlat, nlon, dtype=dtype, device="cuda:0").normal_(generator=gen) for c in (d, d, e, e))
    out, lse = S.s2_nattn_fwd(g, q, k, v, 1.0)
    got = (out, lse) + tuple(S.s2_nattn_bwd(g, q, k, v, out, lse, dout, 1.0))
    n = B * H
    at = torch.tensor(sorted({0, 7, n // 8 - 1, n // 8, n // 4, n // 2 - 1, n // 2, n // 2 + 1, 559240, 559241, n - 9, n - 1}), device="cuda:0")
    few = [x.reshape((n,) + x.shape[2:])[at].unsqueeze(0).contiguous() for x in (q, k, v, dout)]
    for flags, exact in ((S.S2_DEBUG_OWN_PATCHES, True), (0, False), (S.S2_DEBUG_QUARTERS, False)):
        with debug_switches(flags):
            o, l = S.s2_nattn_fwd(g, *few[:3], 1.0)
            want = (o, l) + tuple(S.s2_nattn_bwd(g, *few[:3], o, l, few[3], 1.0))
        for name, a, b in zip(("out", "lse", "dq", "dk", "dv"), got, want):
            a = a.reshape((n,) + a.shape[2:])[at]
            b = b.reshape(a.shape)
            # by parts: the order of a few float32 sums
            assert torch.equal(a, b) if exact else ((a - b).abs() <= 1e-6 + 1e-5 * b.abs()).all(), (name, flags)

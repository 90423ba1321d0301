"""More (batch, head) slices than one launch takes (2^32 threads): the launches are split, and every slice has the results that it has in a launch of
twelve, bit for bit.  In a launch of fewer, whose wavefronts may share patches, it has them up to rounding."""
import pytest
import torch

import paper_2505_11157_amd as S
from test_gpu_nattn import debug_switches

pytestmark = pytest.mark.gpu
FLAGS = {"default": 0, "halves": S.S2_DEBUG_HALVES, "quarters": S.S2_DEBUG_QUARTERS}


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
    o, l = S.s2_nattn_fwd(g, *few[:3], 1.0)
    want = (o, l) + tuple(S.s2_nattn_bwd(g, *few[:3], o, l, few[3], 1.0))
    for name, a, b in zip(("out", "lse", "dq", "dk", "dv"), got, want):
        a = a.reshape((n,) + a.shape[2:])[at]
        assert torch.equal(a, b.reshape(a.shape)), name


@pytest.mark.parametrize("mode", ["default", "halves", "quarters"])
def test_fewer_slices(mode):
    # 64 x 128 for 12 slices has a patch for every wavefront; by default two and three go by halves, one by quarters
    g = S.s2_grid_init(1, 64, 128, 64, 128, 0.344)
    gen = torch.Generator(device="cuda:0").manual_seed(10)
    q, k, v, dout = (torch.empty(1, 12, 32, 64, 128, device="cuda:0").normal_(generator=gen) for _ in range(4))

    def results(n, flags):
        t = [x[:, :n].contiguous() for x in (q, k, v, dout)]
        with debug_switches(flags):
            out, lse = S.s2_nattn_fwd(g, *t[:3], 0.2)
            return (out, lse) + tuple(S.s2_nattn_bwd(g, *t[:3], out, lse, t[3], 0.2))

    for n in (1, 2, 3, 12):
        for name, a, b, c in zip(("out", "lse", "dq", "dk", "dv"), results(12, 0), results(n, S.S2_DEBUG_OWN_PATCHES), results(n, FLAGS[mode])):
            a = a[:, :n]
            assert torch.equal(a, b), (name, n)
            if mode == "default" and n == 12:
                assert torch.equal(a, c), name
            # by parts: some 300 float32 terms of a point are added up in another order, 2^-24 of the sum of their sizes each, which is no more
            # than 16 times the largest result
            assert (a - c).abs().max() <= 300 * 2.0 ** -24 * 16 * a.abs().max(), (name, n)

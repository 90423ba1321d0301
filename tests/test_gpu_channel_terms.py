"""Channel products on the bf16 matrix cores: an infinite factor is not cut into terms (infinity and NaN): the sums it enters are what
float32 arithmetic gives, infinite with the sign of the product, and the sums it does not enter stay what they are.  Widths of one to
four row blocks, a number of points that leaves the last workgroup partly empty."""
import pytest
import torch

import paper_2505_11157_amd as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout", [(16, 16), (32, 64), (48, 96), (16, 128), (16, 160)])
def test_infinite_factors_of_the_mixing(cin, cout):
    gen = torch.Generator(device="cuda:0").manual_seed(cin + cout)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda:0")
    d = S.s2_disco_init(S.s2_grid_init(0, 11, 16, 11, 16, 0.9), 4)
    x, w, dy = rnd(2, cin, 11, 16), rnd(cout, cin, 4), rnd(2, cout, 11, 16)
    run = lambda x, w, dy: S.s2_disco_fwd(d, x, w, None)[:1] + S.s2_disco_bwd(d, x, w, dy, S.s2_disco_fwd(d, x, w, None)[1])[:2]
    y0, dx0, dw0 = run(x, w, dy)
    # one infinite weight: its output channel is infinite with the sign of that one (point, basis function) value
    z = S.s2_disco_fwd(d, x, torch.zeros_like(w).index_put_((torch.tensor(3), torch.tensor(5), torch.tensor(1)), torch.ones((), device="cuda:0")), None)[0]
    w1 = w.clone()
    w1[3, 5, 1] = float("inf")
    y1 = S.s2_disco_fwd(d, x, w1, None)[0]
    rest = [i for i in range(cout) if i != 3]
    assert torch.allclose(y1[:, rest], y0[:, rest], rtol=1e-5, atol=1e-5)     # (summed in another order)
    known = z[:, 3].abs() > 0                     # (a value of exactly zero times infinity is NaN)
    assert torch.equal(y1[:, 3][known], torch.full_like(y1[:, 3][known], float("inf")) * z[:, 3][known].sign())
    # one infinite output gradient: the weight gradients of its channel are infinite with the signs of the values at its point
    one = torch.zeros_like(dy)
    one[1, 2, 4, 7] = 1.0
    at = run(x, w, one)[2][2]
    dy1 = dy.clone()
    dy1[1, 2, 4, 7] = float("inf")
    dw1 = run(x, w, dy1)[2]
    rest = [i for i in range(cout) if i != 2]
    assert torch.allclose(dw1[rest], dw0[rest], rtol=1e-5, atol=1e-4)
    known = at.abs() > 0
    assert torch.equal(dw1[2][known], torch.full_like(dw1[2][known], float("inf")) * at[known].sign())

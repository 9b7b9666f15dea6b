"""GPU test of the masked data gradient for every channel count of dout that the convolution takes:
8 and 16 channels go through a kernel without a mask of its own, 128 through the direct one.  The
reference is the FP64 convolution on the same BF16 values, 0 where the ReLU output is not positive."""
import numpy as np
import pytest

from oracle import surrogate_ref as R
from paper_1705_03141_amd import surrogate as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cout", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("n,d,h,w", [(1, 3, 5, 7), (2, 17, 9, 40)])
def test_masked(cout, n, d, h, w):
    import torch
    cin = 32
    gen = torch.Generator().manual_seed(cout + d)
    bf = lambda *s: torch.randn(s, generator=gen).to(torch.bfloat16)  # noqa: E731
    dout, w_t, y = bf(n, d, h, w, cout), bf(27, cin, cout), torch.relu(bf(n, d, h, w, cin))
    dev = lambda t: t.cuda().view(torch.int16)  # noqa: E731
    f64 = lambda t: t.double().numpy()  # noqa: E731
    dd, wd, yd = dev(dout), dev(w_t), dev(y)
    din = torch.full((n, d, h, w, cin), -1, dtype=torch.int16, device="cuda")
    assert S._lib().surr_conv3d_dgrad(S._p(dd), S._p(wd), S._p(yd), S._p(din), n, d, h, w, cin, cout, None) == 0
    want = np.where(f64(y) > 0, R.conv3d(f64(dout), f64(w_t), np.zeros(cin)), 0.0)
    got = din.view(torch.bfloat16).double().cpu().numpy()
    # one BF16 rounding of values up to max |want|, on top of FP32 sums of 27 cout products
    assert np.abs(got - want).max() <= np.abs(want).max() * 2.0 ** -8 + 1e-3
    assert not got[f64(y) <= 0].any()

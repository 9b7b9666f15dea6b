"""GPU test of the convolutions at the edges of the tiles of the sliding kernel (32 and 64 channels)
and the box kernel (8 and 16): volumes thinner than a tile or one voxel past it in every
direction, one z plane up to several z ranges, volumes on both sides of the lines above which 64
channels take the sliding kernel and boxes have two planes.  The reference is the FP64
convolution on the same BF16 values."""
import numpy as np
import pytest

from oracle import surrogate_ref as R
from paper_1705_03141_amd import surrogate as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin", [8, 16, 32, 64])
@pytest.mark.parametrize("n,d,h,w,cout", [(1, 1, 1, 1, 32), (1, 2, 9, 33, 32), (2, 3, 17, 31, 64), (1, 5, 8, 65, 32),
                                          (1, 40, 3, 5, 32), (1, 16, 15, 33, 32), (1, 17, 15, 33, 32),
                                          (2, 9, 17, 31, 64), (1, 33, 31, 65, 32)])
def test_edges(cin, n, d, h, w, cout):
    import torch
    gen = torch.Generator().manual_seed(cin + 10 * d + w)
    bf = lambda *s: torch.randn(s, generator=gen).to(torch.bfloat16)  # noqa: E731
    x, wt, b = bf(n, d, h, w, cin), bf(27, cout, cin), torch.randn(cout, generator=gen)
    dev = lambda t: t.cuda().view(torch.int16) if t.dtype == torch.bfloat16 else t.cuda()  # noqa: E731
    f64 = lambda t: t.double().numpy()  # noqa: E731
    L = S._lib()
    xd, wd, bd = dev(x), dev(wt), dev(b)
    y = torch.full((n, d, h, w, cout), float("nan"), device="cuda")
    assert L.surr_conv3d_fwd(S._p(xd), S._p(wd), S._p(bd), None, S._p(y), n, d, h, w, cin, cout, 1, None) == 0
    want = np.maximum(R.conv3d(f64(x), f64(wt), f64(b)), 0.0)
    # FP32 sums of 27 cin products of magnitude about 1: n u sqrt(n) is below 2e-3 absolute at n = 1728
    assert np.abs(y.cpu().numpy() - want).max() < 27 * cin * 2.0 ** -24 * np.sqrt(27 * cin) + 1e-5
    # data gradient of a layer cout -> cin' read the other way: dout has cin channels, din cout
    mask = torch.relu(bf(n, d, h, w, cout))
    md = dev(mask)
    din = torch.full((n, d, h, w, cout), -1, dtype=torch.int16, device="cuda")
    if cin % 32 == 0:
        for m in (None, md):
            assert L.surr_conv3d_dgrad(S._p(xd), S._p(wd), S._p(m), S._p(din), n, d, h, w, cout, cin, None) == 0
            ref = R.conv3d(f64(x), f64(wt), np.zeros(cout))
            if m is not None:
                ref = np.where(f64(mask) > 0, ref, 0.0)
            got = din.view(torch.bfloat16).double().cpu().numpy()
            # one BF16 rounding (2^-9) of values up to max |ref|, on top of the FP32 sum
            assert np.abs(got - ref).max() <= np.abs(ref).max() * 2.0 ** -8 + 1e-3
            if m is not None:
                assert not got[f64(mask) <= 0].any()

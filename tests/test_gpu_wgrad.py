"""GPU test of the weight gradient at the edges of its tiles (16 rows x 32 voxels, the upper half
of the rows and the right half of the voxels passed over where the lattice ends before them) and
on both sides of 256 (tile, plane) steps, above which 8 channels are packed.  Inputs are whole
numbers of magnitude up to 4, so every FP32 sum (below 16 x 90000 < 2^24) is exact in any order."""
import numpy as np
import pytest

from oracle import surrogate_ref as R
from paper_1705_03141_amd import surrogate as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,h,w,cin,cout", [
    (1, 1, 1, 1, 8, 32), (1, 3, 5, 5, 8, 32), (1, 256, 4, 17, 8, 32),
    (1, 257, 4, 16, 8, 32), (1, 300, 7, 17, 8, 64), (1, 65, 17, 40, 8, 32), (1, 65, 31, 33, 8, 32),
    (1, 2, 8, 16, 32, 32), (1, 2, 9, 17, 32, 64), (2, 70, 17, 33, 64, 32), (1, 40, 24, 50, 24, 32), (1, 5, 33, 20, 128, 64)])
def test_edges(n, d, h, w, cin, cout):
    import torch
    gen = torch.Generator().manual_seed(cin + 10 * d + w)
    ints = lambda c: torch.randint(-4, 5, (n, d, h, w, c), generator=gen)  # noqa: E731
    x, dout = ints(cin), ints(cout)
    dev = lambda t: t.to(torch.bfloat16).cuda().view(torch.int16)  # noqa: E731
    L = S._lib()
    xd, dd = dev(x), dev(dout)
    dw = torch.full((27, cout, cin), float("nan"), device="cuda")
    db = torch.full((cout,), float("nan"), device="cuda")
    size = L.surr_conv3d_wgrad_scratch_bytes(n, d, h, w, cin, cout)
    scratch = torch.full((size // 4,), float("nan"), device="cuda")
    assert L.surr_conv3d_wgrad(S._p(xd), S._p(dd), S._p(dw), S._p(db), S._p(scratch), n, d, h, w, cin, cout, None) == 0
    want_w, want_b = R.conv3d_wgrad(x.double().numpy(), dout.double().numpy())
    assert np.array_equal(dw.cpu().numpy(), want_w) and np.array_equal(db.cpu().numpy(), want_b)

"""GPU test of convolutions with more blocks than one launch takes (2^32 threads along x): many
volumes of one voxel, each an item of its own, of which only the centre tap contributes.  The
reference is the product with that tap in FP64 on the same BF16 values."""
import pytest

from paper_1705_03141_amd import surrogate as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,n", [(8, 2 ** 24 + 9), (32, 2 ** 23 + 9), (64, 2 ** 23 + 9)])
def test_many_volumes(cin, n):
    import torch
    cout = 32
    gen = torch.Generator(device="cuda").manual_seed(cin)
    bf = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)  # noqa: E731
    x, wt, b = bf(n, cin), bf(27, cout, cin), torch.randn(cout, generator=gen, device="cuda")
    y = torch.full((n, cout), -1, dtype=torch.int16, device="cuda")
    bits = lambda t: t.view(torch.int16)  # noqa: E731
    assert S._lib().surr_conv3d_fwd(S._p(bits(x)), S._p(bits(wt)), S._p(b), S._p(y), None, n, 1, 1, 1, cin, cout, 0,
                                    None) == 0
    want = x.double() @ wt[13].double().T + b.double()
    got = y.view(torch.bfloat16).double()
    # one BF16 rounding on top of an FP32 sum of cin products of magnitude about 1
    assert bool(((got - want).abs() <= want.abs() * 2.0 ** -8 + 1e-4).all())


def test_long_volume_is_enqueued_at_once():
    """The host's part of a call does not grow with the number of planes: 2^22 planes, for which a
    search over every split into ranges takes over 20 ms."""
    import time

    import torch
    d, c = 2 ** 22, 32
    x = torch.zeros((d, c), dtype=torch.int16, device="cuda")
    wt = torch.zeros((27, c, c), dtype=torch.int16, device="cuda")
    y = torch.empty_like(x)
    host = []
    for _ in range(4):
        torch.cuda.synchronize()
        t = time.perf_counter()
        assert S._lib().surr_conv3d_fwd(S._p(x), S._p(wt), None, S._p(y), None, 1, d, 1, 1, c, c, 0, None) == 0
        host.append(time.perf_counter() - t)
    torch.cuda.synchronize()
    assert min(host) < 5e-3

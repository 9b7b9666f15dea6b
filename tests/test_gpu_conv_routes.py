"""GPU tests of what the convolutions owe to whoever calls them, whichever kernel they take: tensors
and weights at any alignment (views that begin on an odd element), small and large volumes of 64
channels, which take different kernels, bitwise alike, and input planes of 2^31 elements."""
import pytest

from paper_1705_03141_amd import surrogate as S

pytestmark = pytest.mark.gpu


def _odd(t):
    """A copy of t that begins one element after a 16-byte boundary."""
    import torch
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
    v = buf[1:1 + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == t.element_size()
    return v


@pytest.mark.parametrize("cin", [8, 16, 32, 64, 128])
@pytest.mark.parametrize("n,d,h,w,cout", [(1, 3, 5, 7, 32), (1, 20, 9, 70, 64)])
def test_alignment(cin, n, d, h, w, cout):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(cin + d)
    bf = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16).view(torch.int16)  # noqa: E731
    x, wt, dout, y = bf(n, d, h, w, cin), bf(27, cout, cin), bf(n, d, h, w, cout), bf(n, d, h, w, cout)
    b = torch.randn(cout, generator=gen, device="cuda")
    L, p, dims = S._lib(), S._p, (n, d, h, w)
    scratch = torch.empty(L.surr_conv3d_wgrad_scratch_bytes(*dims, cin, cout) // 4 + 8, device="cuda")

    def run(f):
        o16, o32 = f(torch.zeros_like(dout)), f(torch.zeros((n, d, h, w, cout), device="cuda"))
        din = f(torch.zeros_like(dout))
        dw, db = f(torch.zeros((27, cout, cin), device="cuda")), f(torch.zeros(cout, device="cuda"))
        xs, ws, bs, ds, ys = f(x), f(wt), f(b), f(dout), f(y)
        assert L.surr_conv3d_fwd(p(xs), p(ws), p(bs), p(o16), None, *dims, cin, cout, 1, None) == 0
        assert L.surr_conv3d_fwd(p(xs), p(ws), p(bs), None, p(o32), *dims, cin, cout, 0, None) == 0
        # the data gradient of a layer cout -> cin: its dout has cin channels, its input cout
        assert L.surr_conv3d_dgrad(p(xs), p(ws), p(ys), p(din), *dims, cout, cin, None) == 0
        assert L.surr_conv3d_wgrad(p(xs), p(ds), p(dw), p(db), p(f(scratch)), *dims, cin, cout, None) == 0
        return o16, o32, din, dw, db

    for a, c in zip(run(lambda t: t.clone()), run(_odd)):
        assert torch.equal(a, c)


def test_small_and_large_volumes_of_64_channels_agree():
    """Alone each volume has few tiles and takes the staged kernel, all of them the sliding one."""
    import torch
    n, d, h, w, cin, cout = 6, 4, 11, 33, 64, 64
    gen = torch.Generator(device="cuda").manual_seed(1)
    bf = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16).view(torch.int16)  # noqa: E731
    x, wt, b, y = bf(n, d, h, w, cin), bf(27, cout, cin), torch.randn(cout, generator=gen, device="cuda"), bf(n, d, h, w, cout)
    assert d * 2 * 6 * 2 <= 256 < n * d * 2 * 6 * 2
    L, p = S._lib(), S._p
    outs = []
    for per in (n, 1):
        o32 = torch.zeros((n, d, h, w, cout), device="cuda")
        din = torch.zeros((n, d, h, w, cout), dtype=torch.int16, device="cuda")
        for k in range(0, n, per):
            s = slice(k, k + per)
            assert L.surr_conv3d_fwd(p(x[s]), p(wt), p(b), None, p(o32[s]), per, d, h, w, cin, cout, 1, None) == 0
            assert L.surr_conv3d_dgrad(p(x[s]), p(wt), p(y[s]), p(din[s]), per, d, h, w, cout, cin, None) == 0
        outs.append((o32, din))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("cin,h,w", [(8, 16386, 16384), (32, 8194, 8192), (64, 4098, 8192)])
def test_planes_of_2_to_31_elements(cin, h, w):
    """One plane against its two halves, each with the rows next to it.  With 8 and 64 channels the
    order of the sums is the same, with 32 the large plane takes a kernel with another."""
    import torch
    cout = 32
    assert h * w * cin >= 2 ** 31
    gen = torch.Generator(device="cuda").manual_seed(cin)
    x = torch.randint(-2 ** 15, 2 ** 15 - 1, (1, 1, h, w, cin), generator=gen, device="cuda", dtype=torch.int16)
    x = (x & 0x3FF) | 0x3F00 | (x & -2 ** 15)  # BF16 of magnitude 0.5 to 8
    wt = torch.randn((27, cout, cin), generator=gen, device="cuda").to(torch.bfloat16).view(torch.int16)
    L, p = S._lib(), S._p
    out = torch.empty((1, 1, h, w, cout), dtype=torch.int16, device="cuda")
    assert L.surr_conv3d_fwd(p(x), p(wt), None, p(out), None, 1, 1, h, w, cin, cout, 0, None) == 0
    mid = h // 4 * 2
    for first, last, skip in ((0, mid + 1, 0), (mid - 2, h, 2)):
        part = torch.empty((last - first, w, cout), dtype=torch.int16, device="cuda")
        assert L.surr_conv3d_fwd(p(x[0, 0, first:last]), p(wt), None, p(part), None, 1, 1, last - first, w, cin, cout, 0,
                                 None) == 0
        got, want = out[0, 0, first + skip:last if skip else mid], part[skip:None if skip else mid]
        if cin != 32:
            assert torch.equal(got, want)
            continue
        for r in range(0, got.shape[0], 1024):
            a, c = (t[r:r + 1024].view(torch.bfloat16).float() for t in (got, want))
            # FP32 sums of 27 cin products of magnitude up to 20, then one BF16 rounding each
            assert bool(((a - c).abs() <= c.abs() * 2.0 ** -7 + 27 * cin * 20 * 2.0 ** -22).all())

"""fp32 convolutions as six bf16 products per fp32 product (K-split kernels, general weight gradient): against fp64 at the edges of
the scheme's ranges -- operands far from one, operands whose first part rounds to infinity, long sums of one sign -- and of the
kernels' tiles and chunks.

Bounds.  A sum of K fp32 products formed in any order of fp32 additions is off by a few 2^-24 of the sum of magnitudes; with
random signs and K <= 2048 the 2-norm over a tensor stays below 4 * 2^-24 = 2.4e-7 of its own (the fp32 matrix instructions measured
0.6e-7 to 4.2e-7 over these layers, these kernels 0.3e-7 to 2.9e-7; the weight gradient of 100352 pixels, where both are
bound by the sums of chunks, 2.0e-7): 5e-7 holds either way and not for a part left out (2^-17 = 7.6e-6)."""
import pytest
import torch

from paper_1910_00932_amd import binding as B

pytestmark = pytest.mark.gpu
BOUND = 5e-7


def _run(F, H, W, cin, cout, xs, ws_, gs, seed=0, positive=False):
    g = torch.Generator().manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=g)   # noqa: E731
    x, w, dy = rnd(F, H, W, cin), rnd(cout, cin, 1, 1), rnd(F, H, W, cout)
    if positive:
        x, w, dy = x.abs(), w.abs(), dy.abs()
    return x * xs, w * ws_, dy * gs


def _layer(x, w, dy):
    F, H, W, cin = x.shape
    cout = w.shape[0]
    d = B.ConvDesc(N=1, T=F, Cin=cin, H=H, W=W, Cout=cout, kh=1, kw=1, stride=1, pad=0, fold_div=0, dtype=B.TSM_F32, layout=B.TSM_NTHWC)
    xd, wd, dyd = x.cuda(), w.cuda(), dy.cuda()
    y, dx, dw = torch.empty_like(dyd), torch.empty_like(xd), torch.empty_like(wd)
    s1, s2 = torch.empty(cout, device="cuda"), torch.empty(cout, device="cuda")
    ws = torch.empty(max(16, B.tsm_conv_workspace_bytes(d)), dtype=torch.uint8, device="cuda")
    B.tsm_conv_fwd(d, xd, wd, y, s1, s2, ws)
    B.tsm_conv_dgrad(d, dyd, wd, dx, ws)
    B.tsm_conv_wgrad(d, xd, dyd, dw, 0, ws)
    torch.cuda.synchronize()
    x2, w2, g2 = x.double().reshape(-1, cin), w.double().reshape(cout, cin), dy.double().reshape(-1, cout)
    refs = {"y": x2 @ w2.t(), "dx": g2 @ w2, "dw": g2.t() @ x2}
    return {k: (t.cpu().double().reshape(refs[k].shape), refs[k]) for k, t in (("y", y), ("dx", dx), ("dw", dw))}


# scales of x, w and dy: all three kinds of products (and their smallest parts, 2^-18 of them) stay inside fp32's range
@pytest.mark.parametrize("scale", [(1.0, 1.0, 1.0), (1e-15, 1e15, 1e-15), (1e15, 1e-15, 1e15), (3e-30, 1e20, 1e12), (1e-3, 1e3, 1.0)])
@pytest.mark.parametrize("shape", [(2, 5, 7, 32, 32), (3, 9, 9, 64, 36), (8, 14, 14, 256, 128), (1, 3, 3, 2048, 96), (8, 33, 31, 40, 72)])
def test_against_64_bits(shape, scale):
    for name, (got, ref) in _layer(*_run(*shape, *scale)).items():
        err = float((got - ref).norm() / ref.norm())
        assert err < BOUND, (name, err)


def test_sums_of_one_sign_over_many_pixels():
    for name, (got, ref) in _layer(*_run(32, 56, 56, 64, 64, 1.0, 1.0, 1.0, positive=True)).items():
        # one sign: the sums' own roundings all weigh in; the fp32 instructions' chain over a chunk of 1792 pixels is off by 1e-6
        assert float((got - ref).norm() / ref.norm()) < 2e-6, name


def test_values_whose_first_part_is_infinite():
    x, w, dy = _run(2, 4, 4, 64, 64, 1e-3, 1e-3, 1e-3)
    big = 3.4e38   # above the largest bf16, below the largest fp32
    x[0, 0, 0, 5], dy[1, 2, 3, 7] = big, -big
    for name, (got, ref) in _layer(x, w, dy).items():
        assert torch.isfinite(got).all(), name
        rows = (got - ref).abs() / ref.abs().amax(dim=1, keepdim=True)
        assert float(rows.max()) < 1e-5, name

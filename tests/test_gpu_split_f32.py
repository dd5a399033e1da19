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


# Operands with bits that three bf16 parts cannot hold (below 2^-110) go through the fp32 instruction, whose sums keep BOUND.  The
# shapes: every number of wavefronts per tile, whole and ragged chunks, the weight gradient's tiles, one and two groups.
TINY_SHAPES = [(2, 5, 7, 32, 32), (8, 14, 14, 64, 128), (8, 33, 31, 40, 72), (32, 28, 28, 128, 64), (16, 56, 56, 64, 192),
               (33, 33, 31, 67, 67)]


@pytest.mark.parametrize("power", [-112, -118, -125])
@pytest.mark.parametrize("shape", TINY_SHAPES)
def test_operands_below_the_range_of_the_parts(shape, power):
    """All of x, then of dy and w, between 2^(power-3) and 2^(power+3); the partner brings the sums back."""
    for tiny in ("x", "dy", "w"):
        x, w, dy = _run(*shape, 1.0, 1.0, 1.0)
        s = {k: torch.tensor(float(power if k == tiny else -power - 20)) for k in ("x", "w", "dy")}
        x, w, dy = (torch.exp2(s[k]) * v for k, v in (("x", x), ("w", w), ("dy", dy)))
        for name, (got, ref) in _layer(x, w, dy).items():
            if not torch.isfinite(ref.float()).all():      # (the product of the two large ones)
                continue
            err = float((got - ref).norm() / ref.norm())
            assert err < BOUND, (tiny, name, err)


@pytest.mark.parametrize("shape", TINY_SHAPES)
def test_a_few_operands_below_the_range(shape):
    """Single tiny values with a huge partner of their own among ordinary ones: the results that they reach."""
    F, H, W, cin, cout = shape
    x, w, dy = _run(*shape, 1.0, 1.0, 1.0)
    small, large = 1.2345678 * 2.0 ** -124, 2.0 ** 124
    w[:, 3], x[..., 3] = 0.0, 0.0
    x[-1, -1, -1, 3], w[cout - 1, 3] = small, large
    dy[..., 5], dy[0, 0, 0, 5] = 0.0, small
    w[5] = 0.0
    w[5, cin - 1] = large
    out = _layer(x, w, dy)
    for name in ("y", "dx"):
        got, ref = out[name]
        keep = ref.abs() < 1e30
        err = float((got - ref)[keep].norm() / ref[keep].norm())
        assert err < BOUND, (name, err)
    got, ref = out["y"]
    assert abs(float(got[-1, cout - 1] - ref[-1, cout - 1])) < 1e-5 * max(1.0, abs(float(ref[-1, cout - 1])))


def test_results_at_the_top_of_the_range():
    """x*y = 2^128 (1 - 2^-23), just inside fp32, where the product of the first parts is 2^128."""
    v = 2.0 ** 64 * (1 - 2.0 ** -24)
    x, w, dy = torch.zeros(2, 4, 4, 64), torch.zeros(64, 64, 1, 1), torch.zeros(2, 4, 4, 64)
    x[0, 1, 2, 5], w[7, 5], dy[1, 2, 3, 9], w[9, 11], dy[0, 1, 2, 20] = v, v, v, v, v
    for name, (got, ref) in _layer(x, w, dy).items():
        assert torch.isfinite(got).all() and float(ref.abs().max()) > 3.4e38, name
        assert torch.equal(got.float(), ref.float()), name


# The matrix core's sums lean towards minus infinity, by 6e-8 of the mean magnitude over 2048 products and 6e-8 over 100352 pixels
# where nothing is done about it.  Half of all sums are formed of the negated operand, so the mean over a tensor, of N results that
# are off by 1e-7 to 3e-7 of it at random, stays within 5 * 3e-7 / sqrt(N) (3e-9 .. 2e-8); fp32 instructions: 1e-9.
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("shape,names,bound", [((8, 14, 14, 2048, 64), ("y",), 6e-9), ((8, 14, 14, 64, 2048), ("dx",), 6e-9),
                                               ((2, 14, 14, 2048, 32), ("y",), 2e-8), ((1, 12, 12, 1024, 36), ("y",), 2e-8),
                                               ((32, 56, 56, 64, 64), ("y", "dx", "dw"), 2.5e-8), ((4, 28, 28, 64, 64), ("dw",), 2.5e-8),
                                               ((33, 33, 31, 67, 67), ("dw",), 2.5e-8)])
def test_sums_do_not_lean(shape, names, bound, relu):
    x, w, dy = _run(*shape, 1.0, 1.0, 1.0)
    out = _layer(x.relu() if relu else x, w, dy)
    for name in names:
        got, ref = out[name]
        lean = float((got - ref).mean() / ref.abs().mean())
        assert abs(lean) < bound, (name, lean)


@pytest.mark.parametrize("shape", [(2, 7, 7, 4608, 32), (8, 14, 14, 2048, 64), (4, 14, 14, 64, 2048), (16, 28, 28, 256, 256)])
def test_long_sums_of_one_sign(shape):
    """Forward and data gradient over up to 4608 products of one sign: a sum per 32 of them, whose additions are off by
    sqrt(K/32/8) * 2^-25 at most in each of up to eight partial sums, and one rounding: 8e-8 (fp32 instructions: 1.0e-7 .. 1.8e-7)."""
    out = _layer(*_run(*shape, 1.0, 1.0, 1.0, positive=True))
    for name in ("y", "dx"):
        got, ref = out[name]
        assert float((got - ref).norm() / ref.norm()) < 8e-8, name


def test_products_whose_left_out_parts_have_one_sign():
    """x = 1 + 2^-8 + ..: of all operands the one whose square loses most, 2^-24 of it, by the three part products that are left
    out; with as much for the rounding of the sum."""
    v = torch.tensor([0x3f807fc0], dtype=torch.int32).view(torch.float32)
    x, w, dy = (t * 0 + v for t in _run(8, 14, 14, 256, 128, 1.0, 1.0, 1.0))
    for name, (got, ref) in _layer(x, w, dy).items():
        assert float(((got - ref) / ref).abs().max()) <= 2.0 ** -23, name

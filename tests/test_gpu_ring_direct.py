"""The ring kernel's tiles that load straight into LDS, with several tiles per block: K ranges of one to a few steps (fewer than the
stages hold, as many, more), whole and ragged last tiles (the waits count the stores of whole tiles), 256- and 128-row tiles, both
column widths (each case names the tiles it runs), the statistics, and the data gradient of the same layers -- against fp32
products of the same bf16 values.

Bound per element: one rounding to bf16 of a sum of at most 1152 products in fp32, 2^-8 of its size and of the tensor's root mean
square (twice the rounding); per-channel sums, of the values as stored, 1e-5 of the sum of their magnitudes."""
import pytest
import torch
import torch.nn.functional as nnf

from paper_1910_00932_amd import binding as B

pytestmark = pytest.mark.gpu

CASES = [
    # frames, height, width, cin, cout, kernel; tiles of the forward convolution and of the data gradient
    (45, 56, 56, 128, 128, 1, "256x128", "256x128"),     # two steps, 551 whole tiles and a ragged one on 256 CUs
    (64, 48, 48, 192, 128, 1, "256x128", "256x128"),     # three steps, whole tiles only
    (45, 56, 56, 64, 128, 3, "256x128", "256x64"),       # nine steps
    (45, 56, 56, 64, 64, 1, "256x64", "256x64"),         # one step of data
    (64, 48, 56, 128, 64, 1, "256x64", "256x128"),       # two steps, whole tiles only
    (45, 56, 56, 64, 64, 3, "256x64", "256x64"),
    (62, 28, 28, 320, 128, 1, "r128x128", "256x128"),    # 380 tiles
    (63, 28, 28, 64, 128, 3, "256x128", "256x64"),
    (61, 28, 27, 192, 192, 1, "256x128", "256x128"),     # a column tile with half of its columns
    # 128 x 64: 32769 to 49151 pixels, so that some CUs have two tiles
    (12, 56, 56, 64, 64, 1, "r128x64", "r128x64"),       # one step of data, 294 whole tiles
    (13, 53, 53, 64, 128, 1, "r128x128", "r128x64"),     # the data gradient's two steps; a ragged last tile
    (14, 54, 55, 192, 64, 1, "r128x64", "256x128"),      # three
    (12, 56, 56, 64, 64, 3, "r128x64", "r128x64"),       # nine
    (13, 53, 53, 128, 64, 3, "r128x64", "r128x128"),     # eighteen, ragged
    # short in K and three, five and seven parts wide: not for the short-K kernels, whose blocks fall into streams of one block per part
    (12, 50, 56, 64, 768, 1, "256x256", "r128x64"),
    (8, 50, 56, 768, 128, 1, "r128x64", "256x128"),
    (8, 50, 56, 256, 640, 1, "256x128", "r128x128"),
    (8, 50, 56, 896, 256, 1, "r128x128", "256x128"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_several_tiles_per_block(case):
    F, H, W, cin, cout, k, fwd_tile, dgrad_tile = case
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")   # noqa: E731
    x, dy = rnd(F, H, W, cin).bfloat16(), rnd(F, H, W, cout).bfloat16()
    w = (rnd(cout, cin, k, k) * (cin * k * k) ** -0.5).bfloat16()
    d = B.ConvDesc(N=1, T=F, Cin=cin, H=H, W=W, Cout=cout, kh=k, kw=k, stride=1, pad=k // 2, fold_div=0, dtype=B.TSM_BF16, layout=B.TSM_NTHWC)
    ws = torch.empty(max(16, B.tsm_conv_workspace_bytes(d)), dtype=torch.uint8, device="cuda")
    y, dx = torch.empty_like(dy), torch.empty_like(x)
    s1, s2 = torch.empty(cout, device="cuda"), torch.empty(cout, device="cuda")
    B.tsm_profile_begin()
    for _ in range(2):            # (the second call finds the first one's values in LDS and in the result)
        B.tsm_conv_fwd(d, x, w, y, s1, s2, ws)
        B.tsm_conv_dgrad(d, dy, w, dx, ws)
    ran = B.tsm_profile_end()
    assert {"igemm_fwd_" + fwd_tile, "igemm_dgrad_" + dgrad_tile} <= set(ran), sorted(ran)

    def products(a, wt):          # [F,H,W,C] x [N,C,k,k], tap by tap in fp32
        p = k // 2
        ap = nnf.pad(a.float(), (0, 0, p, p, p, p))
        out = torch.zeros(F * H * W, wt.shape[0], device="cuda")
        for i in range(k):
            for j in range(k):
                out += ap[:, i:i + H, j:j + W].reshape(F * H * W, -1) @ wt[:, :, i, j].float().t().contiguous()
        return out.reshape(F, H, W, -1)

    for name, got, ref in (("y", y, products(x, w)), ("dx", dx, products(dy, w.transpose(0, 1).flip(2, 3)))):
        err = (got.float() - ref).abs() / (ref.pow(2).mean().sqrt() + ref.abs())
        assert float(err.max()) < 2.0 ** -8, (name, float(err.max()))
    yd = y.double().reshape(-1, cout)
    assert float(((s1.double() - yd.sum(0)).abs() / yd.abs().sum(0)).max()) < 1e-5
    assert float(((s2.double() - yd.pow(2).sum(0)).abs() / yd.pow(2).sum(0)).max()) < 1e-5

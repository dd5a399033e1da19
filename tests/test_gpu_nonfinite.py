"""Infinite and NaN operands of fp32 layers and of layers whose channel counts or shift groups are no multiples of eight: a tap
outside the frame or the clip adds nothing, whatever it would be multiplied with.  The reference sums, in 64 bits, the
products of the taps inside and no others; NaN and infinities have to lie where it has them, everything else agrees as
in test_gpu_general_conv.py."""
import numpy as np
import pytest
import torch

from paper_1910_00932_amd import binding as B
from paper_1910_00932_amd import inputs as I
from gpu_util import CDT, dev_vec, empty_act, from_dev, to_dev, workspace

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _off_the_plain_kernels(monkeypatch):
    monkeypatch.setenv("TSM_PLAIN_CONV", "0")


CASES = [  # N,T,Cin,H,W,Cout,k,stride,pad,fold_div,dtype
    (1, 2, 8, 9, 7, 12, 3, 1, 1, 0, "f32"),        # K-split, chunks that cross taps
    (2, 3, 64, 5, 6, 36, 3, 1, 1, 8, "f32"),       # K-split, whole chunks, shifted
    (1, 2, 32, 9, 9, 40, 3, 2, 1, 0, "f32"),       # parity classes
    (1, 3, 5, 8, 7, 7, 3, 1, 1, 4, "f32"),         # general kernels, element by element
    (1, 3, 5, 8, 7, 7, 3, 2, 1, 4, "bf16"),
    (1, 3, 12, 6, 9, 140, 1, 1, 0, 5, "bf16"),     # groups of 2 of 12 channels: 1x1, only the clip's ends are outside
    (2, 3, 72, 6, 5, 72, 3, 1, 1, 8, "bf16"),      # groups of 9 of 72 channels: the source is a shifted copy
    (1, 4, 64, 7, 6, 64, 1, 1, 0, 6, "bf16"),      # groups of 10 of 64 channels
    (2, 4, 24, 29, 30, 260, 1, 1, 0, 8, "bf16"),   # groups of 3 of 24 channels, 545 tiles: the general kernel on a shifted copy
    (1, 2, 24, 6, 7, 132, 7, 2, 3, 0, "f32"),      # 7x7, wide result
]


def _reference(case, x, w, dy):
    """y, dx and dw over the taps inside; x, dy [F, rows, columns, channels]."""
    N, T, Cin, H, W, Cout, k, s, p, fd, _ = case
    F, Ho, Wo = N * T, dy.shape[1], dy.shape[2]
    fold = Cin // fd if fd else 0
    dt = np.where(np.arange(Cin) < fold, 1, np.where(np.arange(Cin) < 2 * fold, -1, 0))
    f = np.arange(F)
    fs = f[:, None] + dt[None, :]                                             # source frame per (frame, channel)
    t_ok = (f[:, None] % T + dt >= 0) & (f[:, None] % T + dt < T)
    y, dx, dw = np.zeros((F, Ho, Wo, Cout)), np.zeros((F, H, W, Cin)), np.zeros((Cout, Cin, k, k))
    oh, ow = np.arange(Ho), np.arange(Wo)
    for kh in range(k):
        for kw in range(k):
            ih, iw = oh * s + kh - p, ow * s + kw - p
            inside = ((ih >= 0) & (ih < H))[:, None] & ((iw >= 0) & (iw < W))[None, :]
            ok = inside[None, :, :, None] & t_ok[:, None, None, :]             # [F, Ho, Wo, Cin]
            at = (np.where(t_ok, fs, 0)[:, None, None, :], np.clip(ih, 0, H - 1)[None, :, None, None],
                  np.clip(iw, 0, W - 1)[None, None, :, None], np.arange(Cin)[None, None, None, :])
            xs = x[at]
            for co in range(Cout):
                wt, g = w[co, :, kh, kw], dy[..., co][..., None]
                y[..., co] += np.where(ok, xs * wt, 0).sum(-1)
                np.add.at(dx, at, np.where(ok, g * wt, 0))
                dw[co, :, kh, kw] += np.where(ok, g * xs, 0).sum((0, 1, 2))
    return y, dx, dw


def _compare(got, ref, rel, what):
    assert np.array_equal(np.isnan(got), np.isnan(ref)), (what, int(np.isnan(got).sum()), int(np.isnan(ref).sum()))
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf]) and np.array_equal(np.isinf(got), inf), what
    ok = np.isfinite(ref)
    scale = np.sqrt(np.mean(ref[ok] ** 2))
    assert (np.abs(got[ok] - ref[ok]) <= rel * (scale + np.abs(ref[ok]))).all(), what


@pytest.mark.parametrize("case", CASES)
def test_taps_outside_add_nothing(case):
    N, T, Cin, H, W, Cout, k, s, p, fd, dtype = case
    Ho, Wo = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
    x, w = I.normal((N, T, Cin, H, W), 0, dtype), I.kaiming_conv((Cout, Cin, k, k), 1, dtype)
    dy = I.normal((N, T, Cout, Ho, Wo), 3, dtype)
    wi, dyi = w.copy(), dy.copy()
    wi[1, 0, 0, 0], wi[2, Cin - 1, k - 1, k // 2], wi[Cout - 1, 1, k - 1, 0] = np.inf, -np.inf, np.nan
    dyi[0, 0, 1, 0, 0], dyi[N - 1, T - 1, 2, Ho - 1, Wo // 2], dyi[0, T - 1, Cout - 1, 1, Wo - 1] = np.inf, -np.inf, np.nan
    d = B.ConvDesc(N=N, T=T, Cin=Cin, H=H, W=W, Cout=Cout, kh=k, kw=k, stride=s, pad=p, fold_div=fd, dtype=CDT[dtype],
                   layout=B.TSM_NTHWC)
    ws = workspace(B.tsm_conv_workspace_bytes(d))
    y, dx = empty_act((N, T, Cout, Ho, Wo), dtype, "nthwc"), empty_act((N, T, Cin, H, W), dtype, "nthwc")
    dw = torch.empty((Cout, Cin, k, k), dtype=torch.float32, device="cuda")
    B.tsm_conv_fwd(d, to_dev(x, dtype, "nthwc"), dev_vec(wi, dtype), y, None, None, ws)
    B.tsm_conv_dgrad(d, to_dev(dy, dtype, "nthwc"), dev_vec(wi, dtype), dx, ws)
    B.tsm_conv_wgrad(d, to_dev(x, dtype, "nthwc"), to_dev(dyi, dtype, "nthwc"), dw, 0, ws)
    torch.cuda.synchronize()
    rows = lambda a: a.astype(np.float64).transpose(0, 1, 3, 4, 2).reshape(N * T, a.shape[3], a.shape[4], a.shape[2])   # noqa: E731
    with np.errstate(invalid="ignore"):
        ry, rdx, _ = _reference(case, rows(x), wi.astype(np.float64), rows(dy))
        _, _, rdw = _reference(case, rows(x), w.astype(np.float64), rows(dyi))
    rel = 2.0 ** -8 if dtype == "bf16" else 1e-4
    _compare(rows(from_dev(y, "nthwc")), ry, rel, "fwd")
    _compare(rows(from_dev(dx, "nthwc")), rdx, rel, "dgrad")
    _compare(dw.cpu().numpy().astype(np.float64), rdw, 1e-3, "wgrad")
    assert np.isinf(ry).any() and np.isinf(rdw).any() and np.isfinite(rdx).any()

"""The K-split convolutions (fp32 layers, bf16 layers with few tiles) against the oracle, element by element, at every tile
the library picks by the number of 64 x 64 tiles per CU, with remainders in pixels, channels and K chunks, shifted and
strided, and shift groups whose border splits a vector.  Bounds: those of test_gpu_conv.py (one rounding of an fp32 sum, with
a factor of two; 1e-4 in fp32)."""
import os
import subprocess
import sys

import numpy as np
import pytest

import test_gpu_block as TB
import test_gpu_block_infer as TI
import test_gpu_conv as TC
import test_gpu_sweep as TS
from conftest import ROOT, rel_l2
from gpu_util import compare_act
from paper_1910_00932_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _off_the_plain_kernels(monkeypatch):
    monkeypatch.setenv("TSM_PLAIN_CONV", "0")


CASES = [  # N,T,Cin,H,W,Cout,k,stride,pad,fold_div
    (1, 1, 64, 1, 1, 64, 1, 1, 0, 0),          # one pixel, one chunk: seven of eight wavefronts have nothing to add
    (1, 2, 512, 5, 5, 64, 3, 1, 1, 8),         # 32 x 32 tiles, nine chunks per wavefront
    (1, 4, 64, 33, 17, 128, 3, 1, 1, 0),       # 70 tiles: 32 x 64
    (2, 4, 128, 31, 33, 72, 1, 1, 0, 8),       # 256 tiles: 64 x 64 over eight wavefronts; result ends inside a tile
    (2, 8, 64, 35, 31, 64, 1, 1, 0, 8),        # 272 tiles: 64 x 64 over four
    (2, 8, 64, 51, 50, 64, 3, 1, 1, 0),        # 638 tiles (fp32: over four, just below the line)
    (2, 8, 64, 52, 52, 64, 1, 1, 0, 8),        # 676 tiles (fp32: over two)
    (1, 3, 128, 13, 9, 64, 3, 2, 1, 0),        # parity classes
    (1, 2, 256, 14, 13, 128, 1, 2, 0, 0),      # parity classes without taps
    (1, 3, 72, 9, 8, 136, 3, 1, 1, 8),         # groups of nine channels, chunks that cross taps
    (4, 8, 24, 24, 22, 40, 3, 1, 1, 0),        # 16896 pixels, ragged: the general weight gradient in both types
    (1, 2, 24, 7, 6, 40, 3, 1, 1, 8),          # groups of three: one vector of channels holds all of them
]


GENERAL_IN_BF16 = (CASES[5], CASES[6])   # more than two 64 x 64 tiles per CU


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_ksplit_parity(case, dtype):
    B.tsm_profile_begin()
    TC._run(case, dtype, "nthwc")
    classes = B.tsm_profile_end()
    both = {"ksplit_fwd_" + dtype, "ksplit_dgrad_" + dtype}
    if dtype == "bf16" and case in GENERAL_IN_BF16:
        assert not both & set(classes), sorted(classes)
    else:
        assert both <= set(classes), sorted(classes)


@pytest.mark.parametrize("case,split", [  # strided 1x1: three parity classes of dx receive nothing
    ((8, 8, 512, 7, 7, 128, 1, 2, 0, 8), False),    # 400 tiles for 256 CUs, 128 products
    ((2, 8, 512, 7, 7, 128, 1, 2, 0, 8), True),     # 104 tiles
    ((4, 8, 256, 14, 14, 1024, 1, 2, 0, 8), True),  # 400 tiles, 1024 products
])
def test_strided_one_tap_data_gradients_on_both_sides_of_the_line(case, split):
    B.tsm_profile_begin()
    TC._run(case, "bf16", "nthwc")
    classes = B.tsm_profile_end()
    assert ("ksplit_dgrad_bf16" in classes) == split, sorted(classes)


def test_ksplit_with_two_wavefronts_per_tile_in_bf16():
    """Groups of 17 of 136 channels: the data gradient (699 tiles) stores vectors that straddle two groups from the tile two
    wavefronts share; the forward pass (932 tiles) reads a shifted copy on the general kernel."""
    B.tsm_profile_begin()
    TC._run((2, 8, 136, 30, 31, 200, 1, 1, 0, 8), "bf16", "nthwc")
    classes = B.tsm_profile_end()
    assert "ksplit_dgrad_bf16" in classes and "gen_fwd_bf16" in classes, sorted(classes)


# ---- the fused epilogues, at every tile --------------------------------------------------------------------------------
# Bottlenecks with 16 middle channels (one column tile) whose pixel counts end inside a tile, by tiles of 64 x 64 per 256 CUs:
# 32x32 and 32x64 tiles, 64x64 over eight, four and two wavefronts.  Switches take the library's own line away for bf16.
TILES = [  # N,T,H,W
    (1, 3, 19, 17),     # 16 tiles
    (1, 5, 41, 29),     # 93
    (1, 8, 41, 35),     # 180
    (2, 8, 35, 36),     # 315
    (4, 8, 36, 37),     # 666
]


def _bottleneck(frames, dtype, monkeypatch, proj=False, stride=1, mid=16):
    monkeypatch.setenv("TSM_KSPLIT", "1")
    monkeypatch.setenv("TSM_KSPLIT_MAX_TILES", "1000000")
    N, T, H, W = frames
    cin = 4 * mid
    B.tsm_profile_begin()
    TB.run_block("bottleneck", N, T, cin, H, W, mid, 4 * mid, stride, proj, 8 if mid > 8 else 4, dtype, "nthwc")
    classes = B.tsm_profile_end()
    assert "ksplit_fwd_" + dtype in classes and "ksplit_dgrad_" + dtype in classes, sorted(classes)
    assert not any(k.startswith(("igemm", "gen_fwd", "gen_dgrad")) for k in classes), sorted(classes)
    # (masks and BatchNorm sums rode in the data gradients: one reduction is left, the last stage's)
    assert classes["relu_bn_bwd_reduce"][0] == 1, classes


@pytest.mark.parametrize("frames", TILES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_mask_sums_and_addend_in_the_data_gradient(frames, dtype, monkeypatch):
    """(fp32 takes half the channels: an fp32 decision at zero that falls the other way moves a gradient by its own size.)"""
    _bottleneck(frames, dtype, monkeypatch, mid=16 if dtype == "bf16" else 8)


@pytest.mark.parametrize("frames", TILES)
def test_compact_addend_in_the_data_gradient(frames, monkeypatch):
    """Strided projection blocks: the projection's gradient is added from its compact form, on odd and even maps."""
    _bottleneck(frames, "bf16", monkeypatch, proj=True, stride=2)


@pytest.mark.parametrize("frames", TILES)
@pytest.mark.parametrize("proj", [False, True])
def test_affine_residual_and_relu_in_the_forward_pass(frames, proj, monkeypatch):
    monkeypatch.setenv("TSM_KSPLIT_MAX_TILES", "1000000")
    N, T, H, W = frames
    got, ref, refq, classes = TI.run_infer_block(N, T, 64, H, W, 16, 64, 2 if proj else 1, proj, 8, "bf16", "nthwc")
    assert set(k for k in classes if k.startswith(("igemm", "ksplit", "fused", "bn_relu", "block_tail"))) == {"ksplit_fwd_bf16"}, sorted(classes)
    # (bounds of test_gpu_block_infer.py)
    compare_act(got, refq, 2e-2, "vs bf16-storage oracle", "bf16", rtol=2.0 ** -5, atol_rel=2.0 ** -5)
    compare_act(got, ref, 2e-2, "vs fp64 oracle", "bf16", rtol=2.0 ** -5, atol_rel=2.0 ** -5)


BITS_CHILD = """
import sys
sys.path[:0] = [%r, %r]
import numpy as np, test_gpu_step
from paper_1910_00932_amd import binding as B
B.tsm_profile_begin()
r = test_gpu_step.run_step(2, 4, 64, "bf16")
assert "ksplit_dgrad_bf16" in B.tsm_profile_end()
np.save(sys.argv[1], r["grads"])
""" % (ROOT, os.path.join(ROOT, "tests"))


def test_mask_bits_and_activation_decide_alike(tmp_path):
    """The train step's data gradients with the decision bits and, TSM_MASK_BITS=0, with the activation as mask: the same step up
    to the order in which the weight gradients' atomic additions arrive."""
    grads = []
    for bits in ("1", "0"):
        out = str(tmp_path / ("bits%s.npy" % bits))
        r = subprocess.run([sys.executable, "-c", BITS_CHILD, out], cwd=ROOT, env=dict(os.environ, TSM_MASK_BITS=bits),
                           capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
        grads.append(np.load(out))
    assert np.isfinite(grads[0]).all() and rel_l2(grads[1], grads[0]) < 1e-5


# ---- the kernels for larger layers, which layers of these sizes would not reach ----------------------------------------

@pytest.mark.parametrize("case,dtype", [(c, "bf16") for c in TC.CASES + TS._conv_cases(11, 16)] + [(c, "f32") for c in TC.CASES])
def test_small_layers_without_the_ksplit_kernels(case, dtype, monkeypatch):
    """The convolutions of test_gpu_conv.py and the random sweep on the kernels that take larger ones."""
    monkeypatch.setenv("TSM_KSPLIT", "0")
    B.tsm_profile_begin()
    TC._run(case, dtype, "nthwc")
    classes = B.tsm_profile_end()
    cin, cout, fold = case[2], case[5], case[2] // case[9] if case[9] else 0
    kind = "igemm_%s_" if dtype == "bf16" and cin % 8 == 0 and cout % 8 == 0 and fold % 8 == 0 else "gen_%s_" + dtype
    for way in ("fwd", "dgrad"):
        assert any(k.startswith(kind % way) for k in classes), (way, sorted(classes))


@pytest.mark.parametrize("case", [  # channel counts that are no multiples of 64, more than two 64 x 64 tiles per CU either way
    (2, 8, 72, 47, 45, 136, 1, 1, 0, 9),      # shifted 1x1, groups of eight; rows and columns end inside a tile
    (2, 8, 40, 51, 49, 72, 3, 1, 1, 5),       # 3x3, K steps that straddle taps
    (2, 8, 72, 91, 90, 72, 3, 2, 1, 0),       # parity classes
])
def test_large_layers_with_ragged_channels(case):
    B.tsm_profile_begin()
    TC._run(case, "bf16", "nthwc")
    classes = B.tsm_profile_end()
    for way in ("fwd", "dgrad"):
        cd = case[5] if way == "fwd" else case[2]
        assert "igemm_%s_128x%d" % (way, 64 if cd <= 64 else 128) in classes, sorted(classes)

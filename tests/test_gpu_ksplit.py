"""The K-split convolutions (fp32 layers, bf16 layers with few tiles) against the oracle, element by element, at every tile
the library picks by the number of 64 x 64 tiles per CU, with remainders in pixels, channels and K chunks, shifted and
strided, and shift groups whose border splits a vector.  Bounds: those of test_gpu_conv.py (one rounding of an fp32 sum, with
a factor of two; 1e-4 in fp32)."""
import pytest

import test_gpu_conv as TC
from paper_1910_00932_amd import binding as B

pytestmark = pytest.mark.gpu

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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_ksplit_parity(case, dtype):
    B.tsm_profile_begin()
    TC._run(case, dtype, "nthwc")
    classes = B.tsm_profile_end()
    if dtype == "f32":
        assert "ksplit_fwd_" + dtype in classes and "ksplit_dgrad_" + dtype in classes, sorted(classes)

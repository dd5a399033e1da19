"""BatchNorm's sums finished inside the elementwise passes (bn_fold_use: up to 128 partial rows, whole slabs of 128 bytes of
channels) and, beyond either line, in launches of their own: blocks on both sides against the oracle, at the edges of the pass's
128-row turns and of its grid, with identity and projection shortcuts, in both storage types."""
import pytest

import test_gpu_block as TB

pytestmark = pytest.mark.gpu

CASES = [
    # kind, N, T, Cin, H, W, Cmid, Cout, stride, projection, fold_div, dtype
    ("basic", 1, 1, 32, 1, 1, 32, 32, 1, False, 8, "f32"),         # one pixel, one slab
    ("basic", 1, 2, 64, 3, 3, 64, 64, 1, False, 8, "f32"),         # fewer rows than one turn of a block
    ("basic", 1, 1, 32, 127, 1, 32, 32, 1, False, 8, "f32"),       # one row short of a turn
    ("basic", 1, 1, 32, 43, 3, 32, 32, 1, False, 8, "f32"),        # one row beyond it
    ("basic", 1, 8, 96, 32, 32, 96, 96, 1, False, 8, "f32"),       # 64-row tiles: 128 partial rows, the last that are folded
    ("basic", 1, 8, 96, 33, 32, 96, 96, 1, False, 8, "f32"),       # 132 partial rows: launches of their own
    ("basic", 1, 2, 40, 7, 7, 40, 40, 1, False, 8, "f32"),         # channels that fill no slab
    ("bottleneck", 1, 4, 64, 9, 7, 64, 256, 1, True, 8, "bf16"),   # two BatchNorms in the tail and in the last stage's backward pass
    ("bottleneck", 2, 4, 256, 13, 11, 64, 256, 1, False, 8, "bf16"),
    ("bottleneck", 1, 8, 256, 21, 19, 128, 512, 2, True, 8, "bf16"),
    ("bottleneck", 1, 4, 32, 9, 7, 32, 128, 1, True, 8, "f32"),
    ("bottleneck", 1, 2, 48, 9, 9, 24, 72, 1, True, 8, "bf16"),    # ragged channels
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_blocks_on_both_sides_of_the_rule(case):
    TB.run_block(*case, "nthwc")

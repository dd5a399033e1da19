"""BatchNorm's sums finished inside the elementwise passes (bn_fold_use: up to 128 partial rows, whole slabs of 128 bytes of
channels) and, beyond either line, in launches of their own: blocks on both sides against the oracle, at the edges of the pass's
128-row turns and with more rows than its grid takes in one turn, with identity and projection shortcuts, in both storage
types."""
import numpy as np
import pytest

from paper_1910_00932_amd import binding as B

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

# More rows than 512 blocks over all slabs take at 128 each: the loop's later turns, whose rows are loaded before the earlier ones'
# are stored (in place in the backward pass of a middle stage), the last of them ragged.
TURNS = [   # block, and the passes that have to be among its kernels
    # 968 rows of 128 slabs, four blocks each: two turns
    (("bottleneck", 1, 8, 4096, 11, 11, 32, 4096, 1, False, 8, "f32"), {"bn_fold_relu", "bn_fold_tail", "bn_fold_bwd"}),
    # two BatchNorms in the tail and in its backward pass
    (("bottleneck", 1, 8, 64, 11, 11, 32, 4096, 1, True, 8, "f32"), {"bn_fold_relu", "bn_fold_tail", "bn_fold_bwd"}),
    # (the forward sums have more partial rows)
    (("bottleneck", 1, 8, 64, 11, 11, 64, 8192, 1, True, 8, "bf16"), {"bn_fold_bwd"}),
    # middle stages of 7938 rows, 9 slabs, 56 blocks each: two turns, in place backward
    (("bottleneck", 1, 2, 32, 63, 63, 288, 32, 1, True, 8, "f32"), {"bn_fold_relu", "bn_fold_bwd"}),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_blocks_on_both_sides_of_the_rule(case):
    TB.run_block(*case, "nthwc")


@pytest.mark.parametrize("case,names", TURNS, ids=lambda c: "-".join(str(v) for v in c) if isinstance(c, tuple) else "")
def test_several_turns_of_the_grid(case, names, monkeypatch):
    """The values in front of a ReLU are spread around 2 and -2: of millions around zero fp32 takes one or two ReLU decisions other
    than the oracle, and each moves dx by a few 1e-4."""
    make_params = TB.make_params

    def far_from_zero(*args, **kw):
        p = make_params(*args, **kw)
        for k in p:
            if k.startswith("b"):
                p[k] = p[k] + np.where(np.arange(p[k].size) % 4 == 3, -2, 2).astype(np.float32)
        return p

    monkeypatch.setattr(TB, "make_params", far_from_zero)
    B.tsm_profile_begin()
    TB.run_block(*case, "nthwc")
    ran = B.tsm_profile_end()
    assert names <= set(ran) and not {"bn_bwd_coeffs", "bn_bwd_apply2"} & set(ran), sorted(ran)

"""The feature generator where its launches change shape: tokens that do not fill a workgroup's 16 or a chunk's 256,
heads staged in several groups, more columns than two grid rows of lanes.  Same oracle and bounds as
test_gpu_features.py (fp32 sums of at most 64 terms forward, of N terms relative to the largest gradient backward)."""
import pytest

pytestmark = pytest.mark.gpu

import test_gpu_features as base

SHAPES = [  # (M, heads, r, L, d_h)
    (11, 9, 33, 10, 32),        # 121 tokens: 7 full workgroups and 9 tokens, less than half a chunk; 594 columns; heads in groups of 4
    (4, 1, 2, 16, 1),           # exactly one workgroup, a single hidden unit
    (8, 13, 17, 0, 64),         # one lane's share of a chunk, no Fourier bands, groups of 2
    (16, 2, 64, 16, 64),        # exactly one chunk; the most LDS
    (17, 2, 5, 3, 33),          # a chunk and 33 tokens
    (25, 3, 3, 1, 3),           # two chunks and 113 tokens; slices of fewer elements than lanes
    (41, 13, 3, 9, 27),         # two rows a lane: 7 chunks, slices of 16 and 11 rows
    (50, 16, 5, 4, 45),         # four rows a lane: 10 chunks, slices of 32 and 13 rows, 18 input features
]


@pytest.mark.parametrize("M,heads,r,L,d_h", SHAPES)
def test_generator_shapes(M, heads, r, L, d_h):
    for dtype in ("f32", "bf16"):
        base.test_generator_forward(M, heads, r, L, d_h, dtype)
    base.test_generator_backward(M, heads, r, L, d_h)

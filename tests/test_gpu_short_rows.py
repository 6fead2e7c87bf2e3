"""The bf16 kernels for RIB rows of a single pair and for none (r = 2, r = 0), which have kernels of their own, at the sizes
where the workgroup's shape changes: one and several tiles of 32 and 64 tokens, partial ones, window sides that are and
are not multiples of 8, all three places of the denominator, LSE and delta.  Same oracle and bounds as the general
shape tests, which derive them for logits of a few units: heads of 16 channels and more here.  (With 2 or 4 channels a
logit of these many rows reaches 10 to 15, and 2^-9 of that, the rounding of the scaled q, is past the bound of 2e-2;
the general tests have such heads on few rows.)"""
import pytest

pytestmark = pytest.mark.gpu

import test_gpu_backward_shapes as backward
import test_gpu_forward_shapes as forward


@pytest.mark.parametrize("d,r", [(30, 2), (16, 2), (32, 2), (30, 0), (20, 0), (32, 0), (28, 2)])
@pytest.mark.parametrize("M,s", [(8, 3), (9, 4), (15, 7), (16, 0), (24, 12), (25, 1)])
def test_short_rib_rows(oracle, d, r, M, s):
    for many in (False, True) if M in (9, 16) else (False,):
        forward.test_forward_shapes(oracle, d, r, M, s, 1, 2, many)
    for packed in (False, True):
        backward.test_backward_shapes(oracle, d, r, M, s, 1, 2, packed)

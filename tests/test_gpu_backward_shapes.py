"""The bf16 backward kernels where their dispatch changes hands, against the oracle, every element: padded
widths 32 / 48 / 64 with LSE and delta in columns, in the C operand or mixed; window sides that are and are not
multiples of 8; workgroups of 2, 3 and 4 waves, with waves wholly or half past the window's end; rows of a single
dword and no RIB at all.

Tolerance: bf16 operands round P, dS and the gradients to 2^-8 relative, and a gradient element of these shapes is a
sum of about N terms of size P <= 1 whose roundings add at random; 2e-2 absolute is the bound the parity tests
derive for logits of this size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import binding as rb
from paper_2603_06738_amd import workloads as wk
from helpers import geometry

REL = 1e-2      # roundings to bf16, of at most 2^-8 each, of Q_aug (through the logits), of P or dS and of the result: 2.6 times 2^-8

SHAPES = [  # (d, r, M, shift, H / M, W / M)
    (16, 14, 8, 3, 1, 2),       # one 64-token block: the second wave idles; width 32, extras in columns
    (16, 16, 24, 12, 1, 1),     # 3 workgroups of 3 waves; width 32, LSE in the C operand
    (30, 2, 40, 7, 1, 1),       # width 32, single-dword RIB rows, 25 blocks over 7 workgroups: idle waves
    (30, 16, 24, 5, 2, 1),      # width 48, columns
    (32, 8, 16, 0, 1, 2),       # width 48, delta in the C operand, LSE in columns
    (30, 18, 40, 9, 1, 1),      # width 48, LSE in the C operand
    (32, 16, 24, 0, 1, 1),      # width 48, both in the C operand
    (30, 34, 8, 4, 2, 2),       # width 64, LSE in the C operand
    (32, 32, 40, 0, 1, 1),      # width 64, both
    (24, 20, 9, 4, 1, 2),       # 81 tokens: two waves, the second in its first block
    (30, 16, 11, 10, 1, 1),     # 121 tokens
    (30, 18, 13, 6, 1, 1),      # 169 tokens: three waves
    (28, 36, 15, 1, 1, 1),      # 225 tokens: four waves, width 64
    (32, 30, 17, 16, 1, 1),     # 289 tokens: two workgroups of three
    (30, 34, 25, 3, 1, 1),      # 625 tokens: ten blocks over three workgroups of four
    (2, 2, 9, 0, 1, 1),         # single-dword content and RIB rows
    (4, 0, 10, 2, 1, 1),        # no RIB
    (2, 44, 12, 5, 1, 1),       # RIB rows of more than 32 values
]


@pytest.mark.parametrize("d,r,M,s,ny,nx", SHAPES)
@pytest.mark.parametrize("packed", [False, True], ids=["dense", "packed"])
def test_backward_shapes(oracle, d, r, M, s, ny, nx, packed):
    import gpu_helpers as gh
    wl = wk.custom(f"bwd-d{d}r{r}m{M}", "bf16", 2, ny * M, nx * M, 2, d, r, M, s, 7000 + 64 * M + d + r, backward=True)
    assert rb.kernel_name(rb.params_of(wl), True) == "mfma-bf16"
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x, packed=packed)
    out, lse = gh.gpu_fwd(wl, t, packed=packed)
    got = gh.gpu_bwd(wl, t, out, lse, packed=packed)
    again = gh.gpu_bwd(wl, t, out, lse, packed=packed)
    ref = oracle.bwd(geometry(oracle, wl), x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    names = ("dQ", "dK", "dV", "dF_q", "dF_k") if r > 0 else ("dQ", "dK", "dV")
    for name, a, a2, b in zip(names, got, again, ref):
        assert bool((a == a2).all()), name                  # fixed summation order
        assert gh.max_abs(gh.host(a), b) <= gh.TOL["bf16"], name


def check_gradients(got, again, ref):
    """Run to run the same, every element within the parity tests' bound, and within REL in the 2-norm: gradients of few
    channels and sums over windows are themselves not much larger than that bound."""
    import gpu_helpers as gh
    for name, a, a2, b in zip(("dQ", "dK", "dV", "dF_q", "dF_k"), got, again, ref):
        assert bool((a == a2).all()), name
        assert gh.max_abs(gh.host(a), b) <= gh.TOL["bf16"], name
        assert gh.rel(gh.host(a), b) <= REL, name


@pytest.mark.parametrize("d,r,M,s,B,ny,nx,heads", [
    (30, 34, 32, 16, 8, 2, 2, 8),       # 64 columns, LSE in the C operand; two whole workgroups a unit
    (32, 32, 45, 3, 4, 2, 4, 4),        # both in the C operand; 2025 tokens: a partial last block and tile
    (4, 56, 32, 0, 16, 2, 2, 4),        # a long RIB row beside 4-value content rows
], ids=["whole", "partial", "short-content"])
def test_eight_wave_workgroups(oracle, d, r, M, s, B, ny, nx, heads):
    """Grids large enough for the 64-column dkv kernel's workgroups of 512 keys."""
    import gpu_helpers as gh
    wl = wk.custom(f"bwd8-d{d}r{r}m{M}", "bf16", B, ny * M, nx * M, heads, d, r, M, s, 7900 + M, backward=True)
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x)
    out, lse = gh.gpu_fwd(wl, t)
    got = gh.gpu_bwd(wl, t, out, lse)
    again = gh.gpu_bwd(wl, t, out, lse)
    ref = oracle.bwd(geometry(oracle, wl), x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    check_gradients(got, again, ref)


@pytest.mark.parametrize("d,r,M,s,B,ny,nx,heads", [
    (30, 18, 23, 4, 1, 1, 1, 1),        # 529 tokens, two groups: the third workgroup's rows end in its first wave
    (30, 16, 24, 0, 1, 1, 2, 2),        # 576, whole tiles of 64
    (32, 32, 31, 9, 1, 1, 1, 3),        # 961: the last tile a single token of the second group's block
    (16, 14, 32, 0, 1, 1, 1, 2),        # 1024, four groups, whole tiles of 128
    (30, 34, 33, 8, 1, 1, 1, 1),        # 1089: a last tile of 65
    (30, 8, 40, 13, 1, 1, 1, 1),        # 1600 = 12.5 tiles, a window side that is a multiple of 8
    (24, 24, 41, 0, 1, 1, 1, 2),        # 1681
    (32, 16, 48, 5, 1, 1, 1, 2),        # 2304
    (30, 34, 32, 0, 4, 2, 2, 2),        # 32 units: the last grid of one round in four groups
    (30, 34, 32, 0, 3, 1, 11, 1),       # 33: two groups
    (16, 16, 24, 7, 4, 3, 7, 1),        # 84 units: two groups
    (16, 16, 24, 7, 1, 2, 43, 1),       # 86: none
    (6, 4, 28, 0, 1, 1, 1, 1),          # rows of 8-byte pieces
    # the other combinations of width, extras and alignment, in two groups and in four
    (16, 16, 25, 0, 1, 1, 1, 2), (32, 8, 25, 3, 1, 1, 1, 2), (32, 16, 25, 0, 1, 1, 1, 2), (24, 34, 25, 1, 1, 1, 1, 2),
    (32, 24, 25, 0, 1, 1, 1, 2), (32, 24, 24, 5, 1, 1, 1, 2), (16, 14, 33, 0, 1, 1, 1, 1), (16, 16, 33, 2, 1, 1, 1, 1),
    (32, 8, 33, 0, 1, 1, 1, 1), (32, 8, 32, 7, 1, 1, 1, 1), (32, 16, 33, 0, 1, 1, 1, 1), (24, 34, 33, 0, 1, 1, 1, 1),
    (32, 24, 33, 9, 1, 1, 1, 1), (32, 24, 32, 0, 1, 1, 1, 1),
])
def test_streamed_side_shared_by_groups(oracle, d, r, M, s, B, ny, nx, heads):
    """Small grids, whose waves share the streamed side in two or four groups, around the rule's edges; run to run the same."""
    import gpu_helpers as gh
    wl = wk.custom(f"bwdg-d{d}r{r}m{M}", "bf16", B, ny * M, nx * M, heads, d, r, M, s, 8100 + 64 * M + d, backward=True)
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x)
    out, lse = gh.gpu_fwd(wl, t)
    got = gh.gpu_bwd(wl, t, out, lse)
    again = gh.gpu_bwd(wl, t, out, lse)
    ref = oracle.bwd(geometry(oracle, wl), x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    check_gradients(got, again, ref)

"""The bf16 token-row forward kernels where their dispatch changes hands, against the oracle, every element: padded
widths 32 / 48 / 64, full and with columns to spare; denominators from the ones columns and from fp32 sums (d = 32);
window sides that are and are not multiples of 8; workgroups of 2, 3, 4 waves of 64 queries (grids that fill the chip)
and 4 to 8 waves of 32 (grids that do not), with waves wholly or half past the window's end; single-dword rows and no
RIB; the walk with the running maximum.

Tolerance: the parity tests' 2e-2 absolute for logits of this size; bf16 rounds the scaled Q row and P to 2^-8
relative each, and O is an average of values of size one."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import binding as rb
from paper_2603_06738_amd import workloads as wk
from helpers import geometry

SHAPES = [  # (d, r, M, shift, H / M, W / M); `many` repeats the image until 64-query waves outnumber 1024 SIMDs
    (16, 14, 8, 3, 1, 2),       # one 64-token block; width 32, two columns to spare
    (16, 16, 24, 12, 1, 1),     # 3 waves of 64, 6 of 32; width 32, full
    (30, 2, 40, 7, 1, 1),       # width 32, single-dword RIB rows
    (30, 16, 24, 5, 2, 1),      # width 48, two columns to spare
    (32, 8, 16, 0, 1, 2),       # fp32 sums, eight columns to spare
    (30, 18, 40, 9, 1, 1),      # width 48, full
    (32, 16, 24, 0, 1, 1),      # fp32 sums, full
    (30, 34, 8, 4, 2, 2),       # width 64, two RIB pieces a lane
    (24, 20, 9, 4, 1, 2),       # 81 tokens: a 64-token tile and 17
    (30, 16, 11, 10, 1, 1),     # 121 tokens
    (30, 18, 13, 6, 1, 1),      # 169 tokens: three waves of 64, six of 32
    (28, 36, 15, 1, 1, 1),      # 225 tokens
    (32, 30, 17, 16, 1, 1),     # 289 tokens: two workgroups of three waves, or of five
    (30, 34, 25, 3, 1, 1),      # 625 tokens
    (30, 16, 32, 16, 1, 1),     # whole 512-query items that do not fill the chip
    (2, 2, 9, 0, 1, 1),         # single-dword content and RIB rows
    (4, 0, 10, 2, 1, 1),        # no RIB
    (2, 44, 12, 5, 1, 1),       # RIB rows of more than 32 values
]


@pytest.mark.parametrize("many", [False, True], ids=["few", "many"])
@pytest.mark.parametrize("d,r,M,s,ny,nx", SHAPES)
def test_forward_shapes(oracle, d, r, M, s, ny, nx, many):
    import torch
    import gpu_helpers as gh
    per_image = 2 * ny * nx * ((M * M + 63) // 64)
    B = 1 + 1024 // per_image if many else 2
    wl = wk.custom(f"fwd-d{d}r{r}m{M}", "bf16", B, ny * M, nx * M, 2, d, r, M, s, 8000 + 64 * M + d + r)
    assert rb.kernel_name(rb.params_of(wl), False) == "mfma-bf16"
    x = wk.make_inputs(wl)
    O_ref, lse_ref = oracle.fwd(geometry(oracle, wl), x["q"], x["k"], x["v"], x["f_q"], x["f_k"])
    for packed in (False, True):
        t = gh.device_inputs(wl, x, packed=packed)
        for flags in (0, rb.RIB_FLAG_FORCE_ROW_MAX):
            out, lse = gh.gpu_fwd(wl, t, flags=flags, packed=packed)
            assert gh.max_abs(gh.host(out), O_ref) <= gh.TOL["bf16"], flags
            assert gh.max_abs(gh.host(lse), lse_ref) <= gh.TOL["bf16"], flags
    # logits far outside the optimistic walk's range: the second walk, element by element the forced one's
    t = gh.device_inputs(wl, x)
    hot = dict(t, q=t["q"] * 64)
    (a, la), (b, lb) = (gh.gpu_fwd(wl, hot, flags=f, packed=False) for f in (0, rb.RIB_FLAG_FORCE_ROW_MAX))
    assert bool(torch.isfinite(a).all()) and bool(torch.isfinite(la).all())
    assert gh.max_abs(gh.host(a), gh.host(b)) <= gh.TOL["bf16"] and gh.max_abs(gh.host(la), gh.host(lb)) <= gh.TOL["bf16"]


@pytest.mark.parametrize("flags", [0, rb.RIB_FLAG_FORCE_ROW_MAX], ids=["optimistic", "row-max"])
@pytest.mark.parametrize("d,r,M,s,B,ny,nx,heads", [
    (16, 14, 32, 3, 1, 1, 2, 2),        # whole tiles of 128; 32 columns
    (30, 18, 33, 0, 1, 1, 1, 1),        # 1089: a last tile of 65, blocks without keys in two groups
    (32, 16, 40, 9, 1, 1, 1, 1),        # 1600 = 12.5 tiles, fp32 sums
    (30, 34, 45, 11, 1, 1, 1, 1),       # 2025, 64 columns
    (30, 16, 32, 0, 4, 4, 2, 1),        # 32 units: the last grid of one round
    (30, 16, 32, 0, 3, 1, 11, 1),       # 33: no groups
    (6, 4, 36, 35, 1, 1, 1, 1),         # rows of 8-byte pieces
])
def test_streamed_side_shared_by_groups(oracle, d, r, M, s, B, ny, nx, heads, flags):
    """Small grids, whose waves share the keys in four groups; then with one row whose logits need the second walk."""
    import gpu_helpers as gh
    wl = wk.custom(f"fwdg-d{d}r{r}m{M}", "bf16", B, ny * M, nx * M, heads, d, r, M, s, 8600 + 64 * M + d)
    x = wk.make_inputs(wl)
    g = geometry(oracle, wl)
    O_ref, lse_ref = oracle.fwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"])
    t = gh.device_inputs(wl, x)
    out, lse = gh.gpu_fwd(wl, t, flags=flags)
    out2, _ = gh.gpu_fwd(wl, t, flags=flags)
    assert bool((out == out2).all())
    assert gh.max_abs(gh.host(out), O_ref) <= gh.TOL["bf16"] and gh.max_abs(gh.host(lse), lse_ref) <= gh.TOL["bf16"]
    if flags:
        return
    # q of one token 256 times as large (exact in bf16): its logits overflow exp2, and its workgroup walks again
    import torch
    t["q"][0, M // 2, M // 2] *= 256.0
    got = gh.gpu_fwd(wl, t)[0]
    ref = gh.gpu_fwd(wl, t, flags=rb.RIB_FLAG_FORCE_ROW_MAX)[0]
    # both walks multiply the same operands; P and the sums differ by their rounding to 2^-8
    assert bool(torch.isfinite(got).all()) and float((got.float() - ref.float()).abs().max()) <= gh.TOL["bf16"]

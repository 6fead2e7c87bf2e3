"""The fp32 kernels on three bf16 parts a value, where their staging and dispatch change hands, against the oracle, every
element: padded widths 16 to 64, odd head dims and ranks (rows padded to even lengths), a second RIB slot a lane, no
RIB, windows with a partial last block, packed projections; and the rows that go back to fp32 products because a value
leaves the range of the parts.

Tolerance: products keep 24 bits and sums are fp32.  A logit is a sum of up to 64 products of size one, good to
about 64 * 2^-24 = 4e-6; O, LSE and the gradients (sums of size one over softmax weights) follow it linearly, with a
factor of a few: 3e-5 absolute, relative above one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import binding as rb
from paper_2603_06738_amd import workloads as wk
from helpers import geometry

SHAPES = [  # (d, r, M, shift, H / M, W / M)
    (8, 6, 8, 3, 1, 2),         # width 16, one 64-token tile
    (7, 9, 9, 4, 1, 1),         # both odd: 8 + 10 columns of 32; 81 tokens
    (30, 2, 12, 7, 1, 1),       # width 32, a single RIB pair; two tiles and a quarter
    (31, 1, 10, 0, 1, 1),       # odd single-value RIB rows; the last block has 4 keys
    (16, 0, 8, 5, 2, 1),        # no RIB
    (30, 18, 16, 5, 1, 1),      # width 48, full
    (15, 20, 11, 3, 1, 1),      # odd d: RIB starts on the next even column
    (32, 32, 13, 6, 1, 1),      # width 64, full
    (30, 33, 14, 1, 1, 1),      # width 64, odd rank in the second slot
    (5, 47, 9, 2, 1, 1),        # long RIB rows
    (31, 33, 9, 0, 1, 1),       # both odd and 64 together: the fp32-product kernels
    (30, 16, 24, 12, 1, 1),     # 576 tokens, five workgroups
]
NAMES = ("dQ", "dK", "dV", "dF_q", "dF_k")


def _close(gh, a, b, name):
    scale = max(1.0, float(np.abs(b).max())) if b.size else 1.0
    assert gh.max_abs(a, b) <= 3e-5 * scale, name


@pytest.mark.parametrize("packed", [False, True], ids=["dense", "packed"])
@pytest.mark.parametrize("d,r,M,s,ny,nx", SHAPES)
def test_f32_shapes(oracle, d, r, M, s, ny, nx, packed):
    import gpu_helpers as gh
    wl = wk.custom(f"f32-d{d}r{r}m{M}", "f32", 2, ny * M, nx * M, 2, d, r, M, s, 9000 + 64 * M + d + r, backward=True)
    assert rb.kernel_name(rb.params_of(wl), True) == "mfma-f32"
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x, packed=packed)
    out, lse = gh.gpu_fwd(wl, t, packed=packed)
    got = gh.gpu_bwd(wl, t, out, lse, packed=packed)
    g = geometry(oracle, wl)
    O_ref, lse_ref = oracle.fwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"])
    ref = oracle.bwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    _close(gh, gh.host(out), O_ref, "O")
    _close(gh, gh.host(lse), lse_ref, "LSE")
    for name, a, b in zip(NAMES if r else NAMES[:3], got, ref):
        _close(gh, gh.host(a), b, name)


@pytest.mark.parametrize("tensor,value", [("v", float("inf")), ("v", float("nan")), ("v", 2.0 ** 40), ("d_out", 2.0 ** 40),
                                          ("d_out", float("-inf")), ("k", float("nan")), ("q", float("inf"))])
def test_f32_values_outside_the_parts(tensor, value):
    """One element that three bf16 parts cannot carry: where the vector kernels are finite, infinite or NaN, so are
    these, and the finite values agree to fp32 rounding (relative to the element's tensor)."""
    import torch
    import gpu_helpers as gh
    wl = wk.custom("f32-range", "f32", 1, 12, 24, 2, 30, 17, 12, 5, 9900, backward=True)
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x)
    t[tensor][0, 3, 5, 7] = value
    res = []
    for flags in (0, rb.RIB_FLAG_VECTOR_ONLY):
        out, lse = gh.gpu_fwd(wl, t, flags=flags)
        res.append((out, lse, *gh.gpu_bwd(wl, t, out, lse, flags=flags)))
    for name, a, b in zip(("O", "LSE") + NAMES, *res):
        assert torch.equal(torch.isnan(a), torch.isnan(b)), name
        inf = torch.isinf(b)
        assert torch.equal(torch.isinf(a), inf) and torch.equal(a[inf], b[inf]), name
        fin = torch.isfinite(b)
        if bool(fin.any()):
            assert float((a[fin] - b[fin]).abs().max()) <= 3e-5 * max(1.0, float(b[fin].abs().max())), name


@pytest.mark.parametrize("tensor,power", [("v", 118), ("d_out", 118), ("k", 120), ("q", 120), ("f_k", 120), ("f_q", 120)])
@pytest.mark.parametrize("part", ["all", "channel"])
def test_f32_values_too_small_for_the_parts(oracle, tensor, power, part):
    """A tensor, or one channel of it, so small that its third bf16 part would leave the exponent range: the outputs it
    scales keep fp32's relative accuracy, here 3e-6 of the largest element (of the channel)."""
    import gpu_helpers as gh
    wl = wk.custom("f32-small", "f32", 1, 12, 24, 2, 30, 17, 12, 5, 9910, backward=True)
    x = wk.make_inputs(wl)
    pick = slice(None) if part == "all" else slice(4, 5)
    x[tensor] = x[tensor].copy()
    x[tensor][..., pick] *= np.float32(2.0) ** -power
    t = gh.device_inputs(wl, x)
    out, lse = gh.gpu_fwd(wl, t)
    got = [out, *gh.gpu_bwd(wl, t, out, lse)]
    g = geometry(oracle, wl)
    args = [x[n].astype(np.float64) for n in ("q", "k", "v", "f_q", "f_k")]
    ref = [oracle.fwd(g, *args)[0], *oracle.bwd(g, *args, x["d_out"].astype(np.float64))]
    scaled = {"v": ("O",), "d_out": ("dV",), "k": ("dQ",), "q": ("dK",), "f_k": ("dF_q",), "f_q": ("dF_k",)}[tensor]
    if part == "all" and tensor in ("v", "d_out"):
        scaled += ("dQ", "dK")
    for name, a, b in zip(("O",) + NAMES, got, ref):
        if name in scaled:
            a, b = gh.host(a)[..., pick], b[..., pick]
            assert np.abs(a - b).max() <= 3e-6 * np.abs(b).max(), name


MANY = [  # (d, r, M, shift, units): grids that fill the chip take workgroups of up to eight waves and tiles of 64 tokens
    (30, 16, 12, 6, 256),       # five waves, tiles of 32 still; width 48
    (7, 9, 13, 4, 256),         # six waves, 169 tokens, both odd; width 32
    (16, 0, 14, 3, 256),        # seven waves, no RIB; width 16
    (31, 1, 15, 0, 256),        # eight waves, 225 tokens, odd, a single-value RIB row; width 48
    (30, 2, 16, 5, 256),        # eight waves, whole tiles; width 32
    (30, 33, 13, 6, 256),       # six waves, a second RIB slot, odd; width 64
    (32, 32, 15, 1, 256),       # eight waves; width 64, full
    (8, 6, 20, 9, 256),         # two workgroups of seven; width 16
    (15, 20, 18, 2, 128),       # two workgroups of six, odd d; width 48
    (30, 18, 25, 24, 256),      # three workgroups of seven, the last partly past the window's end
]


@pytest.mark.parametrize("d,r,M,s,units", MANY)
def test_f32_shapes_of_large_batches(oracle, d, r, M, s, units):
    import gpu_helpers as gh
    wl = wk.custom(f"f32-many-d{d}r{r}m{M}", "f32", units // 4, M, 2 * M, 2, d, r, M, s, 9300 + 64 * M + d + r, backward=True)
    assert rb.kernel_name(rb.params_of(wl), True) == "mfma-f32"
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x, packed=True)
    out, lse = gh.gpu_fwd(wl, t, packed=True)
    got = gh.gpu_bwd(wl, t, out, lse, packed=True)
    g = geometry(oracle, wl)
    O_ref, lse_ref = oracle.fwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"])
    ref = oracle.bwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    _close(gh, gh.host(out), O_ref, "O")
    _close(gh, gh.host(lse), lse_ref, "LSE")
    for name, a, b in zip(NAMES if r else NAMES[:3], got, ref):
        _close(gh, gh.host(a), b, name)


@pytest.mark.parametrize("tensor,value", [("v", float("inf")), ("v", 2.0 ** -118), ("d_out", 2.0 ** 40), ("k", 2.0 ** -118), ("q", 2.0 ** 40)])
@pytest.mark.parametrize("d,r,M", [(30, 17, 12), (30, 16, 14), (30, 33, 15)], ids=["five-waves", "seven-waves", "eight-waves"])
def test_f32_fallback_in_large_workgroups(d, r, M, tensor, value):
    """The rows that go back to fp32 products, where a workgroup has more waves than those were written for: one value in
    one window; every output of every window as the vector kernels have it."""
    import torch
    import gpu_helpers as gh
    wl = wk.custom(f"f32-wide-m{M}", "f32", 64, M, 2 * M, 2, d, r, M, 5, 9400 + M, backward=True)
    t = gh.device_inputs(wl, wk.make_inputs(wl))
    t[tensor][3, 3, 5, 7] = value
    res = []
    for flags in (0, rb.RIB_FLAG_VECTOR_ONLY):
        out, lse = gh.gpu_fwd(wl, t, flags=flags)
        res.append((out, lse, *gh.gpu_bwd(wl, t, out, lse, flags=flags)))
    for name, a, b in zip(("O", "LSE") + NAMES, *res):
        assert torch.equal(torch.isnan(a), torch.isnan(b)), name
        inf = torch.isinf(b)
        assert torch.equal(torch.isinf(a), inf) and torch.equal(a[inf], b[inf]), name
        fin = torch.isfinite(b)
        if bool(fin.any()):
            assert float((a[fin] - b[fin]).abs().max()) <= 3e-5 * max(1.0, float(b[fin].abs().max())), name


@pytest.mark.parametrize("d,r,M", [(30, 16, 6), (31, 33, 9), (30, 16, 9)], ids=["36-tokens", "fp32-products", "parts"])
def test_f32_logits_far_below_zero(oracle, d, r, M):
    """Every logit near -160, so that LSE is too: the rows past a partial block's end (logit 0) must not come in as
    exp(0 - LSE), which is infinite."""
    import gpu_helpers as gh
    wl = wk.custom("f32-low", "f32", 1, M, 2 * M, 2, d, r, M, 0, 9500 + M, backward=True)
    x = wk.make_inputs(wl)
    x["f_q"], x["f_k"] = x["f_q"].copy(), x["f_k"].copy()
    x["f_q"][..., 0], x["f_k"][..., 0] = 20.0, -8.0 / wl.scale_p
    t = gh.device_inputs(wl, x)
    out, lse = gh.gpu_fwd(wl, t)
    got = gh.gpu_bwd(wl, t, out, lse)
    g = geometry(oracle, wl)
    O_ref, lse_ref = oracle.fwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"])
    ref = oracle.bwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    # (a logit of 160 in base 2 is good to 2^-16: ten times the bound of logits of size one)
    for name, a, b in zip(("O", "LSE") + NAMES, (out, lse, *got), (O_ref, lse_ref, *ref)):
        assert gh.max_abs(gh.host(a), b) <= 3e-4 * max(1.0, float(np.abs(b).max())), name


@pytest.mark.parametrize("d,r,M,s,B,ny,nx,heads", [
    (5, 3, 8, 1, 1, 1, 1, 1),           # 16 columns, 64 tokens: half of the four streamed groups have none
    (14, 4, 9, 8, 1, 1, 1, 1),          # 32 columns, 81: the third group a partial block, the second workgroup a partial wave
    (30, 17, 11, 0, 1, 1, 2, 1),        # 48 columns, 121: just under a tile
    (30, 8, 12, 5, 1, 2, 1, 2),         # 144: a second tile with one partial block
    (32, 32, 13, 2, 1, 1, 1, 3),        # 64 columns: two groups, tiles of 64
    (31, 33, 20, 0, 1, 1, 1, 1),
    (16, 16, 32, 9, 1, 1, 1, 1),        # eight whole tiles
    (30, 16, 16, 0, 4, 4, 2, 2),        # 64 units of 256: the last grid of one round
    (30, 16, 16, 0, 1, 5, 13, 1),       # 65: four waves, no groups
    (32, 30, 12, 3, 2, 4, 4, 3),        # 96 units of 144, 64 columns: two workgroups of 128 each, one round
    (30, 8, 12, 3, 2, 4, 4, 3),         # 48 columns: three of 64, past one round
])
def test_streamed_side_shared_by_groups(oracle, d, r, M, s, B, ny, nx, heads):
    """Small grids, whose waves share the streamed side, around the rule's edge, against the oracle; run to run the same."""
    import gpu_helpers as gh
    wl = wk.custom(f"f32-groups-m{M}d{d}", "f32", B, ny * M, nx * M, heads, d, r, M, s, 9500 + 64 * M + d, backward=True)
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x)
    runs = []
    for _ in range(2):
        out, lse = gh.gpu_fwd(wl, t)
        runs.append((out, lse, *gh.gpu_bwd(wl, t, out, lse)))
    g = geometry(oracle, wl)
    ref = oracle.fwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"]) + oracle.bwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    for name, a, a2, b in zip(("O", "LSE") + NAMES, *runs, ref):
        assert bool((a == a2).all()), name
        assert gh.max_abs(gh.host(a), b) <= gh.TOL["f32"], name


@pytest.mark.parametrize("tensor", ["q", "v", "d_out"])
@pytest.mark.parametrize("B,heads", [(1, 2), (16, 3)], ids=["groups", "four-waves"])
def test_rows_done_again_stay_in_their_workgroup(tensor, B, heads):
    """One value the parts cannot carry in the window's second block of rows: every row is written by its own workgroup."""
    import torch
    import gpu_helpers as gh
    wl = wk.custom("f32-redo", "f32", B, 12, 24, heads, 30, 16, 12, 5, 9930, backward=True)
    t = gh.device_inputs(wl, wk.make_inputs(wl))
    t[tensor][0, 11, 10, 3] = 2.0 ** 33
    res = []
    for flags in (0, 0, rb.RIB_FLAG_VECTOR_ONLY):
        out, lse = gh.gpu_fwd(wl, t, flags=flags)
        res.append((out, lse, *gh.gpu_bwd(wl, t, out, lse, flags=flags)))
    for name, a, a2, b in zip(("O", "LSE") + NAMES, *res):
        assert torch.equal(a, a2) or bool(torch.isnan(a).any()), name
        assert torch.equal(torch.isfinite(a), torch.isfinite(b)), name
        fin = torch.isfinite(b)
        # fp32 sums of up to 144 terms in another order: 144 * 2^-24 of the largest
        assert float((a[fin] - b[fin]).abs().max()) <= 3e-5 * max(1.0, float(b[fin].abs().max())), name


@pytest.mark.parametrize("d,r,M,grouped", [
    (30, 16, 8, False), (16, 14, 8, False),     # two blocks for four groups
    (30, 16, 9, True),                          # three
    (30, 34, 8, True),                          # 64 columns: two groups
])
def test_groups_only_where_most_have_a_block(d, r, M, grouped):
    import gpu_helpers as gh
    wl = wk.custom("f32-route", "f32", 2, 2 * M, M, 3, d, r, M, 1, 9940 + M + r, backward=True)
    t = gh.device_inputs(wl, wk.make_inputs(wl))
    out, lse = gh.gpu_fwd(wl, t)
    names = gh.kernels_of(lambda: gh.gpu_fwd(wl, t)) + gh.kernels_of(lambda: gh.gpu_bwd(wl, t, out, lse))
    kinds = [any(k in n for n in names) for k in ("fwd_keys_kernel", "dq_keys_kernel", "dkv_keys_kernel")]
    assert not names or kinds == [grouped] * 3, names

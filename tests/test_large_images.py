"""bf16 problems whose offsets inside one image need more than 32 bits (images of 2^24 pixels or 2^32 bytes, token
strides of 2^24 bytes): they stay on the matrix cores, forward and backward, with 64-bit offsets.  The GPU tests reach
these kernels through the stride, with one or two windows whose q, k, v are views 2^23 elements apart."""
import numpy as np
import pytest

from paper_2603_06738_amd import binding as rb
from paper_2603_06738_amd import workloads as wk
from helpers import geometry

STRIDE = 1 << 23


@pytest.mark.parametrize("kw", [dict(H=2048, W=2048, token_stride=3 * 192), dict(H=4096, W=4096),
                                dict(H=16, W=16, token_stride=STRIDE), dict(H=16, W=16, token_stride=STRIDE, r=0),
                                dict(H=18, W=18, window=9, token_stride=STRIDE, d=32, r=32)])
def test_selection(kw):
    base = dict(B=1, heads=6, d=30, r=16, window=16, shift=0, scale_c=0.1, scale_p=0.1, dtype="bf16")
    base.update(kw)
    for backward in (False, True):
        assert rb.kernel_name(rb.make_params(**base), backward=backward) == "mfma-bf16"


def spread(tensors):
    """q, k, v as views into one buffer, a token every STRIDE elements."""
    import torch
    B, H, W, C = tensors[0].shape
    buf = torch.empty((B * H * W - 1) * STRIDE + 3 * C, dtype=torch.bfloat16, device="cuda:0")
    views = []
    for i, t in enumerate(tensors):
        view = buf.as_strided((B, H, W, C), (H * W * STRIDE, W * STRIDE, STRIDE, 1), i * C)
        view.copy_(t)
        views.append(view)
    return views


@pytest.mark.gpu
@pytest.mark.parametrize("d,r,M,nx,s", [(30, 16, 9, 1, 4), (32, 8, 8, 2, 3), (30, 30, 8, 1, 0), (32, 32, 9, 1, 2), (24, 0, 9, 1, 0),
                                        (16, 14, 11, 1, 10), (30, 34, 8, 2, 7), (2, 2, 9, 1, 0)])
def test_forward_and_backward(oracle, d, r, M, nx, s):
    import torch
    import gpu_helpers as gh
    wl = wk.custom(f"big-d{d}r{r}m{M}", "bf16", 1, M, nx * M, 2, d, r, M, s, 8800 + 64 * M + d + r, backward=True)
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x)
    t["q"], t["k"], t["v"] = spread([t[n] for n in ("q", "k", "v")])
    g = geometry(oracle, wl)
    O_ref, lse_ref = oracle.fwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"])
    ref = oracle.bwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    for flags in (0, rb.RIB_FLAG_FORCE_ROW_MAX):
        p = rb.params_of(wl, flags=flags, token_stride=STRIDE)
        assert rb.kernel_name(p) == rb.kernel_name(p, backward=True) == "mfma-bf16"
        out = torch.full((wl.B, wl.H, wl.W, wl.C), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        lse = torch.full((wl.n_windows, wl.heads, wl.N), float("nan"), device="cuda:0")
        rb.rib_window_attn_fwd(p, t["q"], t["k"], t["v"], t["f_q"], t["f_k"], out, lse)
        assert gh.max_abs(gh.host(out), O_ref) <= gh.TOL["bf16"], flags
        assert gh.max_abs(gh.host(lse), lse_ref) <= gh.TOL["bf16"], flags
    dq, dk, dv = (torch.full_like(out, float("nan")) for _ in range(3))
    df = [torch.full((wl.heads, wl.N, wl.r), float("nan"), device="cuda:0") for _ in range(2)]
    rb.rib_window_attn_bwd(p, t["q"], t["k"], t["v"], t["f_q"], t["f_k"], out, t["d_out"], lse, dq, dk, dv, *df, rb.alloc_workspace(p))
    for name, a, b in zip(("dQ", "dK", "dV", "dF_q", "dF_k") if r else ("dQ", "dK", "dV"), (dq, dk, dv, *df), ref):
        assert gh.max_abs(gh.host(a), b) <= gh.TOL["bf16"], name


@pytest.mark.gpu
def test_gated_backward_matches_the_dense_layout():
    """The gated pair on spread views against the same call on dense tensors (32-bit offsets)."""
    import torch
    import gpu_helpers as gh
    wl = wk.custom("big-gated", "bf16", 1, 9, 9, 2, 30, 16, 9, 4, 8899, backward=True)
    t = gh.device_inputs(wl, wk.make_inputs(wl))
    gate = torch.rand(t["q"].shape, device="cuda:0").to(torch.bfloat16)
    res = []
    for views, stride in (([t["q"], t["k"], t["v"]], 0), (spread([t["q"], t["k"], t["v"]]), STRIDE)):
        p = rb.params_of(wl, token_stride=stride)
        out, raw, dq, dk, dv, dg = (torch.empty_like(t["q"]) for _ in range(6))
        lse = torch.empty((wl.n_windows, wl.heads, wl.N), device="cuda:0")
        df = [torch.empty((wl.heads, wl.N, wl.r), device="cuda:0") for _ in range(2)]
        ws = torch.empty(rb.rib_window_attn_gated_bwd_workspace_bytes(p), dtype=torch.uint8, device="cuda:0")
        rb.rib_window_attn_gated_fwd(p, *views, t["f_q"], t["f_k"], gate, out, raw, lse)
        rb.rib_window_attn_gated_bwd(p, *views, t["f_q"], t["f_k"], gate, raw, t["d_out"], lse, dq, dk, dv, dg, *df, ws)
        res.append((out, raw, lse, dq, dk, dv, dg, *df))
    for i, (a, b) in enumerate(zip(*res)):
        assert gh.max_abs(gh.host(a), gh.host(b)) <= gh.TOL["bf16"], i

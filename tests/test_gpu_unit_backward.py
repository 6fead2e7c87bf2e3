"""The bf16 backward that does a whole (window, head) unit in one workgroup (windows of 64 to 512 tokens), against the
oracle, every element: workgroups of 2, 4 and 8 waves, full, with a partial last wave and with waves that have no keys;
2, 3 and 4 column blocks of dQ_aug dealt to them; LSE and delta in columns, in the C operand and mixed; partial last
tiles of queries; plain and gated; dense and packed.

Tolerance: as for the pair of kernels (test_gpu_backward_shapes.py): the same operands are rounded to 2^-8, sums are fp32."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import binding as rb
from paper_2603_06738_amd import workloads as wk
from helpers import geometry

SHAPES = [  # (d, r, M, shift, H / M, W / M)
    (30, 16, 8, 0, 1, 3),       # 64 tokens: the second wave has no keys
    (30, 18, 9, 4, 2, 1),       # 81
    (16, 14, 11, 3, 1, 2),      # 121: width 32, columns
    (32, 32, 11, 0, 1, 1),      # width 64, four column blocks on two waves
    (30, 16, 12, 6, 1, 2),      # 144: three of four waves, the third a quarter full
    (20, 8, 14, 9, 1, 1),       # 196: width 32
    (32, 8, 15, 2, 1, 1),       # 225: width 48, delta in the C operand
    (30, 18, 16, 8, 2, 2),      # 256, LSE in the C operand
    (16, 16, 16, 0, 1, 1),      # width 32, LSE in the C operand
    (30, 34, 16, 5, 1, 2),      # width 64
    (32, 16, 17, 1, 1, 1),      # 289: five of eight waves, the fifth half full
    (24, 34, 18, 0, 1, 1),      # 324: width 64 (58 columns)
    (16, 12, 20, 7, 1, 1),      # 400
    (30, 16, 21, 20, 1, 1),     # 441
    (32, 32, 22, 11, 1, 1),     # 484: the last wave's second block starts past the end
    # the other combinations of width, extras, alignment and waves
    (16, 16, 9, 0, 1, 1), (16, 16, 12, 5, 1, 1), (16, 16, 20, 0, 1, 1), (32, 8, 9, 1, 1, 1), (32, 8, 20, 0, 1, 1), (32, 8, 8, 3, 1, 1),
    (30, 18, 20, 9, 1, 1), (32, 16, 8, 0, 1, 2), (32, 16, 16, 4, 1, 1), (24, 34, 9, 0, 1, 1), (24, 34, 12, 7, 1, 1), (24, 34, 8, 0, 1, 2),
    (32, 24, 9, 2, 1, 1), (32, 24, 12, 0, 1, 1), (32, 24, 8, 5, 1, 1), (30, 34, 20, 0, 1, 1), (32, 32, 12, 6, 1, 1), (32, 32, 8, 0, 1, 2),
]


@pytest.mark.parametrize("d,r,M,s,ny,nx", SHAPES)
@pytest.mark.parametrize("packed", [False, True], ids=["dense", "packed"])
def test_unit_backward(oracle, d, r, M, s, ny, nx, packed):
    import gpu_helpers as gh
    wl = wk.custom(f"unit-d{d}r{r}m{M}", "bf16", 2, ny * M, nx * M, 3, d, r, M, s, 9000 + 64 * M + d + r, backward=True)
    assert rb.kernel_name(rb.params_of(wl), True) == "mfma-bf16"
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x, packed=packed)
    out, lse = gh.gpu_fwd(wl, t, packed=packed)
    got = gh.gpu_bwd(wl, t, out, lse, packed=packed)
    again = gh.gpu_bwd(wl, t, out, lse, packed=packed)
    ref = oracle.bwd(geometry(oracle, wl), x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    for name, a, a2, b in zip(("dQ", "dK", "dV", "dF_q", "dF_k"), got, again, ref):
        assert bool((a == a2).all()), name                  # fixed summation order
        assert gh.max_abs(gh.host(a), b) <= gh.TOL["bf16"], name


@pytest.mark.parametrize("d,r,M,s", [(30, 16, 9, 4), (30, 18, 16, 8), (32, 32, 21, 3)])
def test_unit_backward_gated_is_the_plain_one_of_the_gated_gradient(d, r, M, s):
    """dO = dO' * gate, formed in bf16 by the caller, through the plain entry point: bit for bit the gated call."""
    import torch
    import gpu_helpers as gh
    wl = wk.custom(f"unitg-m{M}", "bf16", 1, M, 2 * M, 2, d, r, M, s, 9900 + M, backward=True)
    t = gh.device_inputs(wl, wk.make_inputs(wl))
    p = rb.params_of(wl)
    out, lse = gh.gpu_fwd(wl, t)
    gen = torch.Generator(device=gh.DEV)
    gen.manual_seed(7)
    gate = torch.rand(out.shape, generator=gen, device=gh.DEV).to(torch.bfloat16)
    plain = dict(t, d_out=(t["d_out"].float() * gate.float()).to(torch.bfloat16))
    ref = gh.gpu_bwd(wl, plain, out, lse)
    dq, dk, dv, dg = (torch.full_like(out, float("nan")) for _ in range(4))
    dfq, dfk = (torch.full((wl.heads, wl.N, wl.r), float("nan"), dtype=torch.float32, device=gh.DEV) for _ in range(2))
    ws = torch.empty(rb.rib_window_attn_gated_bwd_workspace_bytes(p), dtype=torch.uint8, device=gh.DEV)
    rb.rib_window_attn_gated_bwd(p, t["q"], t["k"], t["v"], t["f_q"], t["f_k"], gate, out, t["d_out"], lse, dq, dk, dv, dg, dfq, dfk, ws)
    torch.cuda.synchronize()
    for name, a, b in zip(("dQ", "dK", "dV", "dF_q", "dF_k"), (dq, dk, dv, dfq, dfk), ref):
        assert torch.equal(a, b), name


@pytest.mark.parametrize("M,made", [(16, False), (24, True)], ids=["one-kernel", "pair"])
def test_gated_call_makes_delta_once(M, made):
    """The pass over dO', gate and O writes delta into the workspace for the pair of kernels only."""
    import torch
    import gpu_helpers as gh
    wl = wk.custom(f"unitd-m{M}", "bf16", 1, M, 2 * M, 2, 30, 16, M, 3, 9950 + M, backward=True)
    t = gh.device_inputs(wl, wk.make_inputs(wl))
    p = rb.params_of(wl)
    out, lse = gh.gpu_fwd(wl, t)
    dq, dk, dv, dg = (torch.empty_like(out) for _ in range(4))
    dfq, dfk = (torch.empty((wl.heads, wl.N, wl.r), dtype=torch.float32, device=gh.DEV) for _ in range(2))
    ws = torch.full((rb.rib_window_attn_gated_bwd_workspace_bytes(p),), 0x5A, dtype=torch.uint8, device=gh.DEV)
    rb.rib_window_attn_gated_bwd(p, t["q"], t["k"], t["v"], t["f_q"], t["f_k"], torch.ones_like(out), out, t["d_out"], lse,
                                 dq, dk, dv, dg, dfq, dfk, ws)
    torch.cuda.synchronize()
    delta = ws[:wl.n_units * wl.N * 4]          # (the workspace begins with it)
    assert bool((delta == 0x5A).all()) == (not made)

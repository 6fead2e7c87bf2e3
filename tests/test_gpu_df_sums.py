"""The sums of the RIB gradients over windows where their dispatch changes: rows of 16, 8 and 4 bytes a lane, one slice
of windows and several with a short last one, a last workgroup that is partly idle, many heads.  fp32 storage: the
partials are those of the fp32 kernels, so the bound of 1e-4 of the parity tests holds for sums of unit-size terms too."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import workloads as wk
from helpers import geometry

SHAPES = [  # (dtype, B, windows down, across, heads, d, r, M)
    ("f32", 1, 3, 5, 1, 6, 4, 6),           # 15 windows: one slice; 144 values a head, 16 bytes a lane
    ("f32", 3, 5, 9, 2, 6, 4, 6),           # 135 windows: 16 slices, the last ones short
    ("f32", 1, 17, 1, 3, 5, 3, 3),          # 27 values a head: 4 bytes a lane, 2 slices of 9 and 8
    ("f32", 2, 4, 9, 2, 4, 2, 3),           # 18: 8 bytes a lane
    ("f32", 1, 8, 5, 37, 2, 6, 2),          # 37 heads
    ("bf16", 2, 3, 6, 2, 30, 18, 9),        # 1458: 8 bytes a lane, several workgroups a head
    ("bf16", 4, 4, 4, 1, 16, 16, 8),        # 64 windows of 64 tokens
]


@pytest.mark.parametrize("dtype,B,ny,nx,heads,d,r,M", SHAPES)
def test_rib_gradient_sums(oracle, dtype, B, ny, nx, heads, d, r, M):
    import gpu_helpers as gh
    wl = wk.custom(f"df-{dtype}m{M}r{r}", dtype, B, ny * M, nx * M, heads, d, r, M, 1, 3300 + ny * nx + M, backward=True)
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x)
    out, lse = gh.gpu_fwd(wl, t)
    got = gh.gpu_bwd(wl, t, out, lse)
    again = gh.gpu_bwd(wl, t, out, lse)
    ref = oracle.bwd(geometry(oracle, wl), x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    for name, a, a2, b in zip(("dF_q", "dF_k"), got[3:], again[3:], ref[3:]):
        assert bool((a == a2).all()), name
        if dtype == "f32":
            assert gh.max_abs(gh.host(a), b) <= gh.TOL["f32"], name
        else:       # a window left out of 36 or 64 would be an eighth of the sum and more
            assert gh.rel(gh.host(a), b) <= 1e-2, name


@pytest.mark.parametrize("dtype,B,ny,nx,heads,d,r,M", [
    ("bf16", 4, 4, 4, 4, 30, 16, 16),       # one kernel a unit; 64 windows: slices for whole rows and for 4 bytes a lane differ
    ("bf16", 8, 2, 2, 4, 30, 16, 32),       # the pair, 128 units: past one round, rows and the f_q table in 16-byte pieces
    ("bf16", 1, 2, 4, 1, 30, 34, 32),       # the pair in groups, a second RIB piece
    ("bf16", 2, 6, 7, 2, 6, 6, 25),         # rows of 8-byte pieces
    ("f32", 4, 3, 3, 5, 7, 3, 9),           # 243 values a head: 4 bytes a lane wherever dF lies
    ("f32", 4, 4, 4, 3, 30, 16, 16),
], ids=["unit", "pair", "groups", "short-rows", "odd", "f32"])
def test_rib_gradients_do_not_depend_on_where_they_lie(dtype, B, ny, nx, heads, d, r, M):
    """dF_q and dF_k at 16-, 8- and 4-byte aligned addresses of a flat buffer: the same bits, and nothing beside them written."""
    import torch
    import gpu_helpers as gh
    from paper_2603_06738_amd import binding as rb
    wl = wk.custom(f"df-at-m{M}r{r}", dtype, B, ny * M, nx * M, heads, d, r, M, 1, 3700 + M, backward=True)
    t = gh.device_inputs(wl, wk.make_inputs(wl))
    p = rb.params_of(wl)
    out, lse = gh.gpu_fwd(wl, t)
    want = gh.gpu_bwd(wl, t, out, lse)
    dq, dk, dv = (torch.empty_like(out) for _ in range(3))
    n = wl.heads * wl.N * wl.r
    for at_q, at_k in ((4, 4), (1, 1), (2, 2), (4, 3), (2, 4)):     # in values; the allocation itself is 16-byte aligned
        flat = torch.full((2, (n // 8 + 2) * 8), 7.0, dtype=torch.float32, device=gh.DEV)
        dfq, dfk = flat[0, at_q:at_q + n], flat[1, at_k:at_k + n]
        rb.rib_window_attn_bwd(p, t["q"], t["k"], t["v"], t["f_q"], t["f_k"], out, t["d_out"], lse, dq, dk, dv, dfq, dfk,
                               rb.alloc_workspace(p, gh.DEV))
        torch.cuda.synchronize()
        for name, a, b in zip(("dQ", "dK", "dV", "dF_q", "dF_k"), (dq, dk, dv, dfq, dfk), want):
            assert torch.equal(a.reshape(-1), b.reshape(-1)), (name, at_q, at_k)
        rest = flat.clone()
        rest[0, at_q:at_q + n], rest[1, at_k:at_k + n] = 7.0, 7.0
        assert bool((rest == 7.0).all()), (at_q, at_k)

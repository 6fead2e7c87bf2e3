"""Which form of the backward pair a call runs on, by the names of the kernels it launches, where the rule between them was
not what its comment says.  (Grids for a chip of 256 compute units.)"""
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import workloads as wk


def dkv_threads(d, r, M, B, ny, nx, heads):
    """Threads of the dkv kernel's workgroups and whether it stages 16-byte pieces (None: no profiler, other chip)."""
    import re
    import torch
    import gpu_helpers as gh
    wl = wk.custom("route", "bf16", B, ny * M, nx * M, heads, d, r, M, 3, 1, backward=True)
    t = gh.device_inputs(wl, wk.make_inputs(wl))
    out, lse = gh.gpu_fwd(wl, t)
    names = gh.kernels_of(lambda: gh.gpu_bwd(wl, t, out, lse))
    if not names or torch.cuda.get_device_properties(0).multi_processor_count != 256:
        return None
    found = [re.search(r"dkv_kernel<\d+, (\d+), .*?, (\d), (?:true|false), (\d+), (\d+)>", n) for n in names]
    (m,) = [f for f in found if f]
    return m.group(1), int(m.group(3)) if m.group(1) == "64" else 192, m.group(2) == "0"


@pytest.mark.parametrize("d,r,M,B,ny,nx,heads,want", [
    (30, 34, 40, 7, 2, 2, 6, 256),      # 25 blocks in 32, 3 rounds of eight waves against 5 of four
    (30, 34, 40, 8, 2, 2, 6, 512),      # 3 against 6
    (30, 34, 32, 12, 2, 2, 6, 256),     # 16 in 16: 3 against 5
    (30, 34, 32, 16, 2, 2, 6, 512),     # 3 against 6
    (32, 32, 48, 8, 2, 2, 6, 512),      # 36 in 40: 4 against 7
    (30, 34, 45, 9, 2, 2, 6, 256),      # an odd side: 4 against 7
])
def test_eight_wave_dkv_where_it_takes_no_more_rounds(d, r, M, B, ny, nx, heads, want):
    got = dkv_threads(d, r, M, B, ny, nx, heads)
    if got is not None:
        assert got[:2] == ("64", want), got


@pytest.mark.parametrize("d,r,M,B,ny,nx,heads,tile,wide", [
    (32, 32, 24, 16, 2, 2, 6, "32", False),     # aligned, both extras in the C operand, three waves
    (30, 34, 24, 16, 2, 2, 6, "32", True),      # LSE alone
    (32, 32, 40, 6, 2, 2, 6, "64", False),      # aligned, four waves
    (32, 32, 41, 7, 2, 2, 6, "64", True),       # an odd side
])
def test_dkv_pieces_of_64_columns(d, r, M, B, ny, nx, heads, tile, wide):
    """8-byte pieces where those of 16 bytes spill more."""
    got = dkv_threads(d, r, M, B, ny, nx, heads)
    if got is not None:
        assert (got[0], got[2]) == (tile, wide), got


@pytest.mark.parametrize("M,B", [(9, 1), (24, 1), (24, 43), (33, 1)], ids=["unit", "groups", "pair", "four-groups"])
@pytest.mark.parametrize("d", range(2, 33, 2))
def test_every_rank_is_served(d, M, B):
    """Every even rank beside every even head dimension, against the vector-ALU kernels: the forms are chosen by both."""
    import torch
    import gpu_helpers as gh
    from paper_2603_06738_amd import binding as rb
    for r in range(0, 65 - d, 2):
        wl = wk.custom("rank", "bf16", B, M, M, 2, d, r, M, 1, 14000 + 64 * d + r, backward=True)
        gen = torch.Generator(device=gh.DEV)
        gen.manual_seed(wl.seed)
        grid, feat = (B, M, M, 2 * d), (2, M * M, r)
        t = {n: torch.randn(grid, generator=gen, device=gh.DEV).to(torch.bfloat16) for n in ("q", "k", "v", "d_out")}
        t.update({n: (0.5 * torch.randn(feat, generator=gen, device=gh.DEV)).to(torch.bfloat16) for n in ("f_q", "f_k")})
        res = []
        for flags in (0, rb.RIB_FLAG_VECTOR_ONLY):
            out, lse = gh.gpu_fwd(wl, t, flags=flags)
            res.append((out, lse) + gh.gpu_bwd(wl, t, *(res[0][:2] if res else (out, lse)), flags=flags))
        for name, a, b in zip(gh.NAMES, *res):
            if a.numel():
                # as the bound of test_gpu_large_grids.py; the vector kernels round their results to 2^-8 too
                assert float((a.float() - b.float()).norm() / b.float().norm()) <= 1.4e-2, (name, r)

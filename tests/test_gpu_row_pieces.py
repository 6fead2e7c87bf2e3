"""How rows are cut into the pieces lanes move: 16-byte pieces (d, r >= 8) that fill a row, slide back over a neighbour or
stand alone, 8-byte pieces for rows of 4 and 6 values, RIB rows of more than 32 values; window sides whose 16-row runs
lie in one window row, in two, and are gathered one by one; forward, and the backward pair with its table of scaled RIB
rows (several windows: only the first one writes it).  Against the oracle, every element, at the bound of the parity tests:
on small grids, whose backward past 512 tokens runs in groups of waves and moves 8-byte pieces, and on grids of more than
one round of the chip, where it moves 16."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import binding as rb
from paper_2603_06738_amd import workloads as wk
from helpers import geometry

SHAPES = [  # (d, r, M, shift)
    (8, 8, 24, 5),          # one whole piece of four lanes' worth; 16 rows cross window rows
    (10, 12, 32, 0),        # slid pieces
    (26, 22, 40, 31),
    (30, 10, 25, 4),        # gathered rows, partial last tile
    (16, 44, 24, 0),        # a second RIB piece
    (24, 40, 23, 22),
    (4, 8, 24, 3),          # 8-byte pieces
    (30, 4, 32, 16),
    (6, 6, 25, 0),
    (4, 58, 24, 7),
    (32, 6, 24, 0),
    (12, 4, 8, 1),          # 64 tokens: one workgroup a unit in the backward
]


@pytest.mark.parametrize("d,r,M,s", SHAPES)
@pytest.mark.parametrize("packed", [False, True], ids=["dense", "packed"])
def test_row_pieces(oracle, d, r, M, s, packed):
    import gpu_helpers as gh
    wl = wk.custom(f"rows-d{d}r{r}m{M}", "bf16", 2, M, 2 * M, 2, d, r, M, s, 4100 + 64 * M + d + r, backward=True)
    assert rb.kernel_name(rb.params_of(wl), True) == "mfma-bf16"
    x = wk.make_inputs(wl)
    t = gh.device_inputs(wl, x, packed=packed)
    out, lse = gh.gpu_fwd(wl, t, packed=packed)
    g = geometry(oracle, wl)
    got = (out, lse) + tuple(gh.gpu_bwd(wl, t, out, lse, packed=packed))
    ref = oracle.fwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"]) + oracle.bwd(g, x["q"], x["k"], x["v"], x["f_q"], x["f_k"], x["d_out"])
    for name, a, b in zip(("O", "LSE", "dQ", "dK", "dV", "dF_q", "dF_k"), got, ref):
        assert gh.max_abs(gh.host(a), b) <= gh.TOL["bf16"], name


@pytest.mark.parametrize("d,r,M,s", [c for c in SHAPES if c[2] ** 2 > 512])
def test_row_pieces_of_large_grids(oracle, d, r, M, s):
    import re
    import torch
    import gpu_helpers as gh
    wl = wk.custom(f"rows-many-d{d}r{r}m{M}", "bf16", 1, M, 2 * M, 2, d, r, M, s, 4500 + 64 * M + d + r)
    got, ref, names = gh.many_images(oracle, wl, 24)
    if names and torch.cuda.get_device_properties(0).multi_processor_count == 256:
        kind = 0 if d >= 8 and r >= 8 else 4
        assert any(re.search(rf"dq_kernel<\d+, \d+, \w+, \w+, \w+, {kind}, false, 256, 1>", n) for n in names), names
    for name, a, b in zip(gh.NAMES, got, ref):
        if name[:2] != "dF":
            assert gh.max_abs(gh.host(a), b) <= gh.TOL["bf16"], name
        assert gh.rel(gh.host(a), b) <= 1e-2, name

"""Infinities in the bf16 inputs: where the vector kernels are finite, infinite or NaN the matrix-core kernels are too.
Windows whose last tile is partial (its rows past the window's end must not bring the last token's infinity back in) and
whole ones, narrow and wide rows, denominators from the matrix cores and from the vector ALU, both forward walks."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import binding as rb
from paper_2603_06738_amd import workloads as wk

INF = float("inf")
SHAPES = [(30, 16, 9), (32, 16, 9), (30, 34, 11), (16, 14, 13), (24, 0, 15), (30, 16, 17), (30, 18, 8), (30, 16, 24),
          (30, 16, 33), (32, 16, 40), (30, 34, 41)]     # four groups of waves, blocks of the last tile past the window


def both(wl, t, names, flags=0):
    import torch
    import gpu_helpers as gh
    res = []
    for f in (flags, rb.RIB_FLAG_VECTOR_ONLY):
        out, lse = gh.gpu_fwd(wl, t, flags=f)
        res.append(dict(zip(("O", "LSE", "dQ", "dK", "dV", "dF_q", "dF_k"), (out, lse, *gh.gpu_bwd(wl, t, out, lse, flags=f)))))
    for name in names:
        a, b = (x[name].float() for x in res)
        assert torch.equal(torch.isnan(a), torch.isnan(b)), name
        inf = torch.isinf(b)
        assert torch.equal(torch.isinf(a), inf) and torch.equal(a[inf], b[inf]), name
        fin = torch.isfinite(b)
        assert float((a[fin] - b[fin]).abs().max()) <= gh.TOL["bf16"], name


def problem(d, r, M, seed):
    import gpu_helpers as gh
    wl = wk.custom(f"inf-d{d}r{r}m{M}", "bf16", 1, M, 2 * M, 2, d, r, M, 0, seed, backward=True)
    return wl, gh.device_inputs(wl, wk.make_inputs(wl))


@pytest.mark.parametrize("flags", [0, rb.RIB_FLAG_FORCE_ROW_MAX], ids=["optimistic", "row-max"])
@pytest.mark.parametrize("d,r,M", SHAPES)
def test_last_token(d, r, M, flags):
    """An infinity in the last token of a window: of v, it is the whole channel of O; of dO, of dV."""
    wl, t = problem(d, r, M, 500 + M)
    t["v"][0, M - 1, M - 1, 1] = INF
    both(wl, t, ("O", "LSE"), flags)
    wl, t = problem(d, r, M, 600 + M)
    t["d_out"][0, M - 1, M - 1, 1] = -INF
    both(wl, t, ("dV",), flags)


@pytest.mark.parametrize("flags", [0, rb.RIB_FLAG_FORCE_ROW_MAX], ids=["optimistic", "row-max"])
@pytest.mark.parametrize("d,r,M", SHAPES + [(30, 16, 32)])
def test_keys_masked_by_an_infinity(d, r, M, flags):
    """Keys taken out by minus infinity in a channel where every q is positive: P is 0 at them, O, LSE and every
    gradient but that channel of dQ (0 times infinity) finite.  Masked keys in the first block and, in the larger
    windows, whole later ones."""
    wl, t = problem(d, r, M, 700 + M)
    C = wl.C
    for hd in range(wl.heads):
        t["q"][..., hd * d] = t["q"][..., hd * d].abs() + 0.5
    keys = t["k"].view(wl.H * wl.W, C)
    for n in [3, 7, 20, 30] + list(range(40, M * M - 1 if M < 16 else 130)):
        keys[(n // M) * wl.W + n % M, ::d] = -INF           # the first window's token n, channel 0 of every head
    both(wl, t, ("O", "LSE", "dQ", "dK", "dV"), flags)

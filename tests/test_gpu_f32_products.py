"""The rounding of one product in the fp32 kernels that multiply three bf16 parts a value.  Every sum here has a single
non-zero term, and one of its factors is 1 in channel 0, so channel c is channel 0 times a known value.

Bound, in units of 2^-24: the part products left out are at most 2.5 (x1 y2 + x2 y1 + x2 y2 with one factor's parts
rounded to nearest and the other's truncated; up to 6.8 with both truncated), and both channels are rounded once, 1
each: 4.5."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import binding as rb

M, HEADS, D, R = 9, 2, 30, 16
N, C = M * M, HEADS * D


def gradients(one_query):
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(31 + one_query)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda:0")
    q, k, v, g = (rand(N, HEADS, D) for _ in range(4))
    fq, fk = rand(HEADS, N, R), rand(HEADS, N, R)
    n = 44
    if one_query:               # a single upstream row: one term in dV and dK
        q[n, :, 0] = g[n, :, 0] = 1.0
        g[torch.arange(N, device="cuda:0") != n] = 0.0
    else:                       # a single key row: one term in dQ
        k[n, :, 0] = 1.0
        k[torch.arange(N, device="cuda:0") != n] = 0.0
    t = [a.view(1, M, M, C).contiguous() for a in (q, k, v)]
    p = rb.make_params(1, M, M, HEADS, D, R, M, 0, 1.0, 0.25, "f32")
    out, dq, dk, dv = (torch.empty_like(t[0]) for _ in range(4))
    lse = torch.empty((1, HEADS, N), device="cuda:0")
    df = [torch.empty((HEADS, N, R), device="cuda:0") for _ in range(2)]
    rb.rib_window_attn_fwd(p, *t, fq, fk, out, lse)
    rb.rib_window_attn_bwd(p, *t, fq, fk, out, g.view(1, M, M, C).contiguous(), lse, dq, dk, dv, *df, rb.alloc_workspace(p))
    grad = lambda a: a.view(N, HEADS, D).double()
    return n, q.double(), k.double(), g.double(), grad(dq), grad(dk), grad(dv)


def worst(got, factors):
    """Largest error of channel c against channel 0 times factors[head][c], in units of 2^-24."""
    want = got[..., :1] * factors
    return float(((got - want).abs() / want.abs())[..., 1:].max()) * 2.0 ** 24


def test_products_keep_24_bits():
    n, q, k, g, dq, dk, dv = gradients(one_query=True)
    assert worst(dv, g[n]) <= 4.5
    assert worst(dk, q[n]) <= 4.5
    n, q, k, g, dq, dk, dv = gradients(one_query=False)
    assert worst(dq, k[n]) <= 4.5

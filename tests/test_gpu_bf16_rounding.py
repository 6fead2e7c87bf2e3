"""How the bf16 kernels for windows of any size turn fp32 probabilities and score gradients into matrix operands: rounded
to nearest, with nothing added beforehand, and for d = 32, where the denominator is summed on the vector ALU, in fp32.

Logits are exact here (scale_c = ln 2 makes the base-2 logit q.k itself, with q a unit row and k small multiples of a
power of two), so every value that gets rounded is known and the results follow bit by bit or within the rounding of
the fp32 sums.  None of the rounded values lies near a tie: at least 0.03 of a bf16 step away, where the kernels' own
error (LSE carried as two bf16 parts, 2^-17 of at most 10) is under 0.01."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import binding as rb

LN2 = float(np.float32(np.log(2.0)))


def rne(x):
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)


def forward(d, r, M, q, k, v, flags=0):
    import torch
    C, N = d, M * M
    grid = lambda a: torch.tensor(a, dtype=torch.bfloat16, device="cuda:0").view(1, M, M, C).contiguous()
    f = torch.zeros((1, N, r), dtype=torch.bfloat16, device="cuda:0")
    p = rb.make_params(1, M, M, 1, d, r, M, 0, LN2, 1.0, "bf16", flags=flags)
    t = [grid(a) for a in (q, k, v)] + [f, f]
    out = torch.empty((1, M, M, C), dtype=torch.bfloat16, device="cuda:0")
    lse = torch.empty((1, 1, N), device="cuda:0")
    rb.rib_window_attn_fwd(p, *t, out, lse)
    return p, t, out, lse, grid


@pytest.mark.parametrize("flags", [0, rb.RIB_FLAG_FORCE_ROW_MAX], ids=["optimistic", "row-max"])
@pytest.mark.parametrize("d,r,M", [(30, 16, 9), (16, 14, 12), (30, 34, 11), (24, 0, 15), (30, 18, 16), (30, 16, 24),
                                   (32, 16, 9), (32, 30, 12), (32, 0, 16), (32, 16, 24)])
def test_denominator(d, r, M, flags):
    N = M * M
    steps = np.random.default_rng(M).integers(0, 129, N)        # logits 0, -1/32, .. -4; the first one the maximum
    steps[0] = 0
    q, k, v = (np.zeros((N, d), np.float32) for _ in range(3))
    q[:, 0], k[:, 0] = 1.0, -steps / 32.0
    _, _, _, lse, _ = forward(d, r, M, q, k, v, flags)
    P = np.exp2(k[:, 0].astype(np.float64))
    want = np.log((P if d == 32 else rne(P).astype(np.float64)).sum())
    # N fp32 additions, a logarithm and its product with ln 2
    tol = N * 2.0 ** -24 + 4 * 2.0 ** -24 * abs(want)
    assert float((lse.double().cpu() - want).abs().max()) <= tol


@pytest.mark.parametrize("d,r", [(30, 16), (30, 18), (32, 16), (30, 34), (16, 14), (24, 0)])
@pytest.mark.parametrize("M,a", [(9, 4), (11, 2), (15, 16), (24, 4)])
def test_probabilities_and_score_gradients(d, r, M, a):
    """One query row has a logit log2(a) at key 0 and 0 elsewhere, and is the only one with an upstream gradient (1 in
    channel 1): its P is 1 / Z, Z = N - 1 + a, at every key but the first.  v is 1 in channel 1 of key j0 alone, so
    dS = P (0 - delta) at the other keys, delta = bf16(1 / Z)."""
    import torch
    N, i, j0, j1 = M * M, 7, 5, 50
    q, k, v, g = (np.zeros((N, d), np.float32) for _ in range(4))
    q[i, 0], k[0, 0], v[j0, 1], g[i, 1] = 1.0, np.log2(a), 1.0, 1.0
    k[j1, 2] = 1.0                                              # (meets zeros of q: dQ[i][2] = scale_c dS[i][j1])
    p, t, out, lse, grid = forward(d, r, M, q, k, v)
    dq, dk, dv = (torch.empty_like(out) for _ in range(3))
    df = [torch.empty((1, N, r), device="cuda:0") for _ in range(2)]
    rb.rib_window_attn_bwd(p, *t, out, grid(g), lse, dq, dk, dv, *df, rb.alloc_workspace(p))
    P = np.float32(1.0 / (N - 1 + a))
    others = [j for j in range(1, N) if j != j0]
    host = lambda x: x.float().cpu().numpy().reshape(N, d)
    assert (host(dv)[others, 1] == rne(P)).all()
    dS = rne(-P * rne(P))
    assert (host(dk)[others, 0] == rne(dS * np.float32(LN2))).all()
    assert host(dq)[i, 2] == rne(dS * np.float32(LN2))

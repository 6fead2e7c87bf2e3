"""The work whose time counts: window attention with RIB as a user of this library has it done.

Every case goes through the public entry points of `paper_2603_06738_amd.binding`, on the current
stream, with buffers and workspaces that a program keeps for the lifetime of a layer.  Three kinds:

    infer   one attention forward without LSE (serving)
    train   forward with LSE, then backward: O, LSE, dQ, dK, dV, dF_q, dF_k
    layer   one training step of a whole gated layer: feature tables from the generator's weights,
            gated forward, gated backward, generator backward

A case is a dict of plain values: kind, dtype ("bf16" / "f32"), grid B x H x W, heads, head dim d,
rank r, window side M, cyclic shift s, and whether q, k, v are views of one packed [B, H, W, 3C]
projection.  The sizes are those of the repository's own workloads (configs 1-5 and the paper's
layer schedule), with ragged window sides (24, 12) beside the powers of two.
"""
import math

import torch

from paper_2603_06738_amd import binding as rb

DEV = "cuda:0"
GEN_L, GEN_DH = 10, 32          # Fourier bands and hidden width of the generator (the paper's)

MAX_FLOP = 2.0e12               # of a drawn case; a third of the largest listed one
MAX_FLOP_F32 = 1.2e11           # fp32 arithmetic is an order slower per operation
MAX_TOKENS = 262144


def _case(name, kind, dtype, B, H, W, heads, d, r, M, s, packed=False):
    return {"name": name, "kind": kind, "dtype": dtype, "B": B, "H": H, "W": W, "heads": heads, "d": d, "r": r,
            "M": M, "s": s, "packed": packed}


def listed():
    return [
        # serving one 64 x 64 tile through a shifted 16-window layer: the smallest call, all latency
        _case("infer_w16_tile", "infer", "bf16", 1, 64, 64, 6, 30, 16, 16, 8),
        # config 1: a small fp32 layer, the precision the paper quotes its costs in
        _case("infer_w16_f32", "infer", "f32", 1, 48, 48, 2, 30, 8, 16, 0),
        # 12 x 12 windows (144 tokens: no whole tile), packed projection, an ordinary serving batch
        _case("infer_w12_packed", "infer", "bf16", 4, 96, 144, 6, 30, 16, 12, 6, packed=True),
        # config 3 with its shift: the headline forward at 32 x 32 windows
        _case("infer_w32", "infer", "bf16", 8, 96, 96, 6, 30, 16, 32, 16),
        # config 4: one large photograph at 64 x 64 windows
        _case("infer_w64_photo", "infer", "bf16", 1, 512, 512, 6, 30, 16, 64, 32),
        # config 5: the benchmark's training step
        _case("train_w32", "train", "bf16", 16, 96, 96, 6, 30, 16, 32, 16),
        # the first layer of the paper's schedule: small windows, many of them
        _case("train_w16_r18", "train", "bf16", 16, 96, 96, 6, 30, 18, 16, 0),
        # 24 x 24 windows (576 tokens: whole 64-token tiles but no whole 256-query blocks), packed projection
        _case("train_w24_packed", "train", "bf16", 8, 96, 96, 6, 30, 18, 24, 12, packed=True),
        # the large variant's second cycle: d = 32, d + r = 64
        _case("train_w48_d32", "train", "bf16", 8, 96, 96, 6, 32, 32, 48, 0),
        # the schedule's largest layer: one 96 x 96 window per patch
        _case("train_w96_r34", "train", "bf16", 16, 96, 96, 6, 30, 34, 96, 0),
        # config 5's layer in fp32 storage, a quarter of its batch
        _case("train_w32_f32", "train", "f32", 4, 96, 96, 6, 30, 16, 32, 16),
        # the light variant's gated layer with its feature generator, one whole step
        _case("layer_w48_light", "layer", "bf16", 8, 96, 96, 3, 16, 16, 48, 0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case anywhere in the ranges above: window sides 8 to 96 (odd ones too), batches and grids of
    any number of windows, heads 1 to 8, even d of 16 to 32, even r of 8 to 34 (any r in fp32)."""
    while True:
        kind = rng.choice(["infer", "train", "train", "layer"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        M = _log_int(rng, 8, 96)
        d = rng.choice([16, 20, 24, 28, 30, 30, 30, 32, 32])
        r = rng.randrange(8, 35) if dtype == "f32" else 2 * rng.randrange(4, 18)
        if d + r > 64:
            continue
        heads = rng.choice([1, 2, 3, 4, 6, 6, 8])
        windows = _log_int(rng, 1, MAX_TOKENS / (M * M))
        nwy = rng.randrange(1, max(1, int(math.sqrt(windows))) + 1)
        nwx = rng.randrange(1, max(1, windows // nwy) + 1)
        B = max(1, windows // (nwy * nwx))
        s = rng.choice([0, M // 2, rng.randrange(M)])
        case = _case(None, kind, dtype, B, nwy * M, nwx * M, heads, d, r, M, s, packed=rng.random() < 0.4)
        del case["name"]
        if work(case)["flops"] <= (MAX_FLOP if dtype == "bf16" else MAX_FLOP_F32):
            return case


def _dims(case):
    N = case["M"] ** 2
    tokens = case["B"] * case["H"] * case["W"]
    units = tokens // N * case["heads"]
    return N, tokens, units, case["heads"] * case["d"]


def work(case):
    """Bytes of every input once and every output once, and the operations of the unpadded contractions:
    forward 2 N^2 (2d + r) per (window, head), backward 2 N^2 (5d + 3r); exponentials are not counted."""
    N, tokens, units, C = _dims(case)
    e = 4 if case["dtype"] == "f32" else 2
    d, r, heads = case["d"], case["r"], case["heads"]
    grid, table, dtable = tokens * C * e, heads * N * r * e, heads * N * r * 4
    nbytes = 3 * grid + 2 * table + grid
    flops = 2.0 * N * N * (2 * d + r) * units
    if case["kind"] != "infer":
        nbytes += units * N * 4 + grid + 3 * grid + 2 * dtable          # LSE; dO; dQ, dK, dV; dF_q, dF_k
        flops += 2.0 * N * N * (5 * d + 3 * r) * units
    if case["kind"] == "layer":
        n_in, proj = 2 + 4 * GEN_L, 2 * heads * GEN_DH * r
        weights = n_in * GEN_DH + GEN_DH + proj
        nbytes += 2 * grid + grid + 2 * weights * 4                     # gate, dgate; ungated O; weights and their gradients
        flops += 3 * 2.0 * N * (n_in * GEN_DH + proj)                   # products forward, and both of them backward
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # Measured over the listed cases and 14 drawn ones, every output of the matrix-core path against the same call
    # on the vector-ALU kernels (fp32 arithmetic, sums in another order), and about four times the worst seen:
    # fp32 storage 7.1e-7 (2-norm) and 7.1e-6 (largest); bf16 storage 4e-3 (dK; 5.6e-3 on the generator's db_h,
    # a sum with cancellation) and 0.11 (dK, an element against the tensor's root mean square).
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 3e-5}
    return {"rel": 1.6e-2, "max": 0.4}


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    td = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    N, _, units, C = _dims(case)
    B, H, W, heads, d, r = (case[n] for n in ("B", "H", "W", "heads", "d", "r"))

    def normal(*shape, std=1.0, dtype=td):
        return (torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32) * std).to(dtype)

    def empty(*shape, dtype=td):
        return torch.empty(shape, device=DEV, dtype=dtype)

    f32 = torch.float32
    grid = (B, H, W, C)
    st = {"kind": case["kind"]}
    # scale of the content and positional logits: 1/sqrt(d) and 1/sqrt(r), as the paper has them
    st["p"] = rb.make_params(B, H, W, heads, d, r, case["M"], case["s"], d ** -0.5, r ** -0.5, case["dtype"],
                             token_stride=3 * C if case["packed"] else 0)
    if case["packed"]:
        qkv = normal(B, H, W, 3 * C)
        st["q"], st["k"], st["v"] = qkv[..., :C], qkv[..., C:2 * C], qkv[..., 2 * C:]
    else:
        st["q"], st["k"], st["v"] = normal(*grid), normal(*grid), normal(*grid)
    if case["kind"] == "layer":
        n_in = 2 + 4 * GEN_L
        st["gp"] = rb.make_gen_params(case["M"], heads, r, GEN_L, GEN_DH, case["dtype"])
        st["W_h"] = normal(n_in, GEN_DH, std=n_in ** -0.5, dtype=f32)
        st["b_h"] = normal(GEN_DH, std=0.1, dtype=f32)
        st["W_pq"] = normal(heads, GEN_DH, r, std=0.25, dtype=f32)
        st["W_pk"] = normal(heads, GEN_DH, r, std=0.25, dtype=f32)
        st["f_q"], st["f_k"] = empty(heads, N, r), empty(heads, N, r)
        st["gate"] = torch.rand(grid, generator=gen, device=DEV, dtype=f32).to(td)
        st["raw"], st["dgate"] = empty(*grid), empty(*grid)
        st["dW_h"], st["db_h"] = empty(n_in, GEN_DH, dtype=f32), empty(GEN_DH, dtype=f32)
        st["dW_pq"], st["dW_pk"] = empty(heads, GEN_DH, r, dtype=f32), empty(heads, GEN_DH, r, dtype=f32)
        st["gws"] = empty(max(rb.rib_features_bwd_workspace_bytes(st["gp"]), 256), dtype=torch.uint8)
        st["ws"] = empty(max(rb.rib_window_attn_gated_bwd_workspace_bytes(st["p"]), 256), dtype=torch.uint8)
    else:
        st["f_q"], st["f_k"] = normal(heads, N, r, std=0.5), normal(heads, N, r, std=0.5)
    st["out"] = empty(*grid)
    if case["kind"] != "infer":
        st["dout"] = normal(*grid)
        st["lse"] = empty(units // heads, heads, N, dtype=f32)
        st["dq"], st["dk"], st["dv"] = empty(*grid), empty(*grid), empty(*grid)
        st["df_q"], st["df_k"] = empty(heads, N, r, dtype=f32), empty(heads, N, r, dtype=f32)
        if case["kind"] == "train":
            st["ws"] = rb.alloc_workspace(st["p"], DEV)
    return st


def run(st):
    p, q, k, v, fq, fk, out = (st[n] for n in ("p", "q", "k", "v", "f_q", "f_k", "out"))
    if st["kind"] == "infer":
        rb.rib_window_attn_fwd(p, q, k, v, fq, fk, out)
        return out
    if st["kind"] == "train":
        rb.rib_window_attn_fwd(p, q, k, v, fq, fk, out, st["lse"])
        rb.rib_window_attn_bwd(p, q, k, v, fq, fk, out, st["dout"], st["lse"], st["dq"], st["dk"], st["dv"],
                               st["df_q"], st["df_k"], st["ws"])
        return {n: st[n] for n in ("out", "lse", "dq", "dk", "dv", "df_q", "df_k")}
    weights = (st["W_h"], st["b_h"], st["W_pq"], st["W_pk"])
    rb.rib_features_fwd(st["gp"], *weights, fq, fk)
    rb.rib_window_attn_gated_fwd(p, q, k, v, fq, fk, st["gate"], out, st["raw"], st["lse"])
    rb.rib_window_attn_gated_bwd(p, q, k, v, fq, fk, st["gate"], st["raw"], st["dout"], st["lse"], st["dq"], st["dk"],
                                 st["dv"], st["dgate"], st["df_q"], st["df_k"], st["ws"])
    rb.rib_features_bwd(st["gp"], *weights, st["df_q"], st["df_k"], st["dW_h"], st["db_h"], st["dW_pq"], st["dW_pk"],
                        st["gws"])
    return {n: st[n] for n in ("out", "raw", "lse", "dq", "dk", "dv", "dgate", "f_q", "f_k", "df_q", "df_k", "dW_h",
                               "db_h", "dW_pq", "dW_pk")}

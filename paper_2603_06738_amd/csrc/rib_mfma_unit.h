// RIB window attention, backward, bf16 matrix cores: windows of up to 512 tokens, a whole (window, head)
// unit in one workgroup.  Gradient formulas: include/rib_attn.h.
//
// Where one workgroup holds all keys of a unit, scores, dP and exponentials need making only once: 11 MFMAs
// (32x32x16) a 32x32 block and the equivalent of 3 (48 columns) for dQ, where the pair of kernels in
// rib_mfma_bwd.h makes 20, and 16 exponentials for 32.  Above all, under 512 tokens a workgroup spends half of
// its life on its start and its end (16x16 windows: 9 and 12 us of 19 and 22 in the pair), and here there is one of each.
//
// A wave owns 64 keys (K_aug, V as MFMA B operands, dK_aug^T and dV^T as accumulators), the queries stream in tiles of
// 32, as in the pair's dkv kernel.  dS leaves the accumulators key by key: it is already the B operand of dK, and
// goes to LDS as one row of 32 queries a key.  dQ_aug^T = K_aug^T dS^T contracts over keys, so both of its
// operands are read transposed (ds_read_b64_tr_b16) from rows of keys, dS and an image of K_aug; its 16x16 blocks
// are dealt to the waves, each over ALL keys, so no sum crosses waves and every output has one fixed order.
// One barrier a tile: dQ of a tile is made while the next one's scores are, from the other of two dS buffers.
// Rows are swizzled in 16- and 32-byte pieces so that eight rows of a block tile the 64 banks.
//
// delta = dO . O is made by the 8 lanes that stage a query row, which have its dO words already.
//
// Workgroups of 2, 4 and 8 waves: up to 128, 256, 512 tokens.  246 to 256 registers, two waves a SIMD; spilled are none with 32
// columns, up to 5 with 48 and up to 22 with 64 (two waves; up to 7 with four and eight).  LDS with 32 / 48 / 64 columns: 35 / 41 / 48 KB
// up to 128 tokens, 60 / 70 / 80 KB up to 256, so that two workgroups share a CU, 109 / 127 / 146 KB up to 512.  What bounds it (16x16 windows, d = 30, r = 18; clk of
// a workgroup, two on the CU): start 10 000, a tile 4 200 (dQ 1 500, scores and gradients 2 400, barrier 200; the SIMD's
// MFMAs 1 800, the CU's LDS accesses 1 800), end 7 800.  Forward + backward, us, with the pair / here / here
// with the sums of RIB gradients as they are now (d = 30 and 6 heads unless said): 16 images 96 x 96 of 16x16, r = 18 432 / 348 / 329; 96 x 96
// of 12x12, r = 16 728 / 389 / 340 (144 tokens: the pair gives each wave a half-empty tile); 96 x 96 of 8x8, r = 16 595 / 462 / 344; 8
// images 66 x 66 of 22x22, d = r = 32, 8 heads 331 / 239 / 223; one 22x22 window of 2 heads 60 / 55, one 8x8 25 / 20.  On grids of one round the pair shares its streamed side
// in two groups of waves, and is slower all the same (backward, d = 30, r = 16, groups / here: one 16x16 window of 2 heads 27 / 20, one
// 22x22 45 / 42, 32 of 17x17, 4 heads 43 / 33).  Past 512 tokens a second group of keys would need dQ kept
// in memory between the two, and the pair's loops take no longer a block than this one's.
#pragma once

#include <type_traits>

#include "rib_mfma_bwd.h"

namespace rib {
namespace unit {

using namespace rows;
using bwd::Args;
using bwd::StatRegs;
using bwd::stat_request;

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int DQK>
struct ULay {
    using L = Lay<DQK, 32>;
    static constexpr int RC = DQK / 16;                     // 16-column blocks of K_aug
    static constexpr int KB = DQK * 2;                      // bytes of a K row
    static constexpr size_t k_bytes(int waves) { return (size_t)waves * 64 * KB; }
    static constexpr size_t ds_bytes(int waves) { return (size_t)waves * 64 * 64; }         // one tile of 32 queries
    static constexpr size_t bytes(int waves) { return k_bytes(waves) + 2 * ds_bytes(waves) + 2 * L::STAGE * sizeof(bf16_t); }
    // Byte offset of 16-column block `c` inside K row `row`: the blocks are permuted so that eight consecutive
    // rows of one block tile the 64 banks.
    static __device__ __forceinline__ int block(int row, int c)
    {
        return 32 * (DQK == 64 ? c ^ ((row >> 1) & 3) : DQK == 32 ? c ^ ((row >> 2) & 1) : c);
    }
    // ... of dword `w` of row `row`
    static __device__ __forceinline__ int dword(int row, int w) { return row * KB + block(row, w >> 3) + 4 * (w & 7); }
};

// Raw words of a streamed 32-query tile: 8 lanes a token, NP tokens a lane.
template <int DQK, int NP>
struct QRegs {
    dword2 x[NP], y[NP], o[NP], fa[NP], fb[DQK == 64 ? NP : 1];
    float lse[NP];
};
template <int DQK, int NP, bool ALN>
__device__ __forceinline__ void q_request(QRegs<DQK, NP> &rg, const Geo &g, const Win &win, const Stream &s, const char *ob, int tile,
                                          int nt, int wave)
{
    const int lane = opaque_tid() & 63, l = lane >> 3;
    const Piece pc = piece_of<kLong8>(g, lane & 7);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int slot = p * nt + wave * 64;
        if (NP == 1 ? nt == 256 || slot < 256 : slot < 256) {
            const int n0 = tile * 32 + (slot >> 3);
            const uint32_t t = win.token<ALN>(n0, l);
            rg.x[p] = get8(s.xb, token_offset<false>(t, s.xs) + 4u * pc.dc, false);
            const uint32_t yo = token_offset<false>(t, s.ys) + 4u * pc.dc;
            rg.y[p] = get8(s.yb, yo, false);
            rg.o[p] = get8(ob, yo, false);
            const int n = n0 + l, nc = ALN ? n : (n < win.last ? n : win.last);
            const uint32_t fr = __umul24((uint32_t)nc, s.frow);
            rg.fa[p] = get8(s.fb, fr + 4u * pc.f0, false);
            if (DQK == 64) rg.fb[p] = get8(s.fb, fr + 4u * pc.f1, false);
            rg.lse[p] = *(const float *)((const char *)s.lse + 4u * (uint32_t)nc);
        }
    }
}

template <int DQK, int NP, bool XS, bool XD, bool ALN>
__device__ __forceinline__ void q_commit(const QRegs<DQK, NP> &rg, const Geo &g, bf16_t *S, float sc, float sp, int left, int nt, int wave)
{
    using L = Lay<DQK, 32>;
    const int lane = opaque_tid() & 63, l = lane >> 3, j = lane & 7;
    const Piece pc = piece_of<kLong8>(g, j);
    bf16_t *xr = S + __mul24(l, L::XS) + 2 * pc.dc, *yr = S + L::YR + __mul24(l, L::YS) + 2 * pc.dc;
    bf16_t *fr = S + __mul24(l, L::XS) + g.d + 2 * pc.f0, *fr1 = S + __mul24(l, L::XS) + g.d + 2 * pc.f1;
    const int hp = g.d >> 1;
    const float m0 = 2 * j + 1 < hp ? 1.f : 0.f, m1 = 2 * j < hp ? 1.f : 0.f;      // (a slid pair counts its new half only)
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int slot = p * nt + wave * 64;
        if (NP == 1 ? nt == 256 || slot < 256 : slot < 256) {
            const int r0 = slot >> 3;
            dword2 x = rg.x[p], y = rg.y[p], f = rg.fa[p];
            x.x = scale_pair(x.x, sc), x.y = scale_pair(x.y, sc);
            f.x = scale_pair(f.x, sp), f.y = scale_pair(f.y, sp);
            // delta of this lane's row (paper Sec. 2.2 backward): 8 lanes share it
            const float a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, y.x), __builtin_bit_cast(bf16x2, rg.o[p].x), 0.f, false);
            const float b = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, y.y), __builtin_bit_cast(bf16x2, rg.o[p].y), 0.f, false);
            float dl = (m0 != 0.f ? a : 0.f) + (m1 != 0.f ? b : 0.f);
#define RIB_DPP_ADD(x, ctrl) (x) += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, (x)), (ctrl), 0xF, 0xF, true))
            RIB_DPP_ADD(dl, 0xB1);      // quad_perm [1,0,3,2]: lane ^ 1
            RIB_DPP_ADD(dl, 0x4E);      // quad_perm [2,3,0,1]: lane ^ 2
            RIB_DPP_ADD(dl, 0x141);     // row_half_mirror: lane ^ 7
#undef RIB_DPP_ADD
            if (!ALN && r0 + l >= left) y.x = y.y = 0u;
            put8(xr + r0 * L::XS, x, false);
            put8(yr + r0 * L::YS, y, false);
            put8(fr + r0 * L::XS, f, false);
            if (DQK == 64) {
                f = rg.fb[p];
                f.x = scale_pair(f.x, sp), f.y = scale_pair(f.y, sp);
                put8(fr1 + r0 * L::XS, f, false);
            }
            // the row's -delta by its first lane, -LSE * log2 e by its second
            const float e = j ? -rg.lse[p] * kLog2e : -dl;
            const uint32_t pk = split_bf16(e);
            const int row = r0 + l, xo = XS ? L::EX + 2 * row : row * L::XS + DQK - 2, yo = XD ? L::EX + 64 + 2 * row : L::YR + row * L::YS + L::DVK - 2;
            const uint32_t word = (j ? XS : XD) ? __float_as_uint(e) : pk;
            if (j < 2) *(uint32_t *)(S + (j ? xo : yo)) = word;
        }
    }
}

// The wave's 64 K / V rows: K_aug into its rows of the K image (`K`, rows row0 ..), V through `W`; both read back as
// MFMA B operands.  Rows past the window's end are zero in the image.
template <int DQK, bool XS, bool XD, bool ALN>
__device__ __forceinline__ void kv_stage(const StatRegs<DQK, false, kLong8> &r, const Geo &g, char *K, bf16_t *W, int row0, int left,
                                         bf16x8 (&Kb)[2][DQK / 16], bf16x8 (&Vb)[2][2])
{
    using U = ULay<DQK>;
    constexpr int YS = Lay<DQK, 32>::YS;
    const int lane = threadIdx.x & 63, l = lane >> 3, col = lane & 31, hf = lane >> 5;
    const Piece pc = piece_of<kLong8>(g, lane & 7);
    const int hp = g.d >> 1;
    {
        const int row = row0 + lane;
        const bool in = ALN ? left > 0 : lane < left;
        for (int c = hp + (g.r >> 1); c < DQK / 2; ++c)
            *(uint32_t *)(K + U::dword(row, c)) = (c == DQK / 2 - 1 && !XS && in) ? 0x3f803f80u : 0u;
        for (int c = hp; c < 16; ++c) *(uint32_t *)(W + lane * YS + 2 * c) = (c == 15 && !XD) ? 0x3f803f80u : 0u;
    }
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const int rr = p * 8 + l, row = row0 + rr;
        const bool in = ALN ? left > 0 : rr < left;
        const Words<kLong8> x = r.x[p], f = r.fa[p];
        *(uint32_t *)(K + U::dword(row, pc.dc)) = in ? x.w[0] : 0u;
        *(uint32_t *)(K + U::dword(row, pc.dc + 1)) = in ? x.w[1] : 0u;
        *(uint32_t *)(K + U::dword(row, hp + pc.f0)) = in ? f.w[0] : 0u;
        *(uint32_t *)(K + U::dword(row, hp + pc.f0 + 1)) = in ? f.w[1] : 0u;
        if (DQK == 64) {
            const Words<kLong8> f1 = r.fb[p];
            *(uint32_t *)(K + U::dword(row, hp + pc.f1)) = in ? f1.w[0] : 0u;
            *(uint32_t *)(K + U::dword(row, hp + pc.f1 + 1)) = in ? f1.w[1] : 0u;
        }
        put<kLong8>(W + rr * YS + 2 * pc.dc, r.y[p], false);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int row = row0 + b * 32 + col;
#pragma unroll
        for (int t = 0; t < DQK / 16; ++t) Kb[b][t] = *(const bf16x8 *)(K + row * U::KB + U::block(row, t) + 16 * hf);
        read_rows<2>(Vb[b], W + (b * 32 + col) * YS + 8 * hf);
    }
}

// W waves; every value of a template below that depends on it is a constant.
template <int DQK, bool XS, bool XD, bool ALN, int W>
__global__ __launch_bounds__(W * 64, 2) void unit_kernel(Geo g, const bf16_t *__restrict__ q, const bf16_t *__restrict__ k,
                                                     const bf16_t *__restrict__ v, const bf16_t *__restrict__ fq,
                                                     const bf16_t *__restrict__ fk, const bf16_t *__restrict__ out,
                                                     const bf16_t *__restrict__ dout, const float *__restrict__ lse,
                                                     bf16_t *__restrict__ dq, bf16_t *__restrict__ dk,
                                                     bf16_t *__restrict__ dv, float *__restrict__ dfq_part, float *__restrict__ dfk_part)
{
    using L = Lay<DQK, 32>;
    using U = ULay<DQK>;
    constexpr int NP = W == 2 ? 2 : 1, nt = W * 64, NKS = 2 * W;
    constexpr int TPW = (2 * U::RC + W - 1) / W;            // most 16x16 blocks of dQ_aug a wave makes of a tile
    extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, col = lane & 31, hf = lane >> 5;
    char *const kimg = (char *)smem;
    char *const dsb = kimg + U::k_bytes(W);
    constexpr int dsz = (int)U::ds_bytes(W);
    bf16_t *const stages = (bf16_t *)(dsb + 2 * dsz);
    int *const map = (int *)(stages + 2 * L::STAGE);

    int64_t u;
    int zero, b;
    block_coords(1, u, zero);
    const int w = (int)u / g.heads, hd = (int)u - w * g.heads;
    const float sc2 = g.scale_c * kLog2e, sp2 = g.scale_p * kLog2e;
    const int ntiles = (g.N + 31) / 32;
    const Win win = window_of<ALN>(g, w, nt, map, b);
    const int64_t img = (int64_t)b * g.H * g.W;
    Stream ks, qs;
    ks.xb = (const char *)(k + img * g.tstride + hd * g.d);
    ks.yb = (const char *)(v + img * g.tstride + hd * g.d);
    ks.fb = (const char *)(fk + (int64_t)hd * g.N * g.r);
    ks.xs = ks.ys = qs.xs = g.tstride * 2;
    ks.frow = qs.frow = (uint32_t)g.r * 2u;
    qs.xb = (const char *)(q + img * g.tstride + hd * g.d);
    qs.yb = (const char *)(dout + img * g.C + hd * g.d);
    qs.fb = (const char *)(fq + (int64_t)hd * g.N * g.r);
    qs.ys = (int64_t)g.C * 2;
    ks.lse = qs.lse = lse + u * g.N;
    ks.delta = qs.delta = nullptr;
    const char *ob = (const char *)(out + img * g.C + hd * g.d);
    if (!ALN) __syncthreads();

    const int n0 = wave * 64;                               // this wave's first key
    const bool active = n0 < g.N;
    QRegs<DQK, NP> rg;
    bf16x8 Kb[2][L::KS], Vb[2][L::VS];
    {
        StatRegs<DQK, false, kLong8> sr;
        stat_request<DQK, false, false, ALN, kLong8, false>(sr, g, win, ks, n0, nullptr, false);
        q_request<DQK, NP, ALN>(rg, g, win, qs, ob, 0, nt, wave);
        init_pads<DQK, 32, true, XS, XD, 2>(g, stages, nt);
        kv_stage<DQK, XS, XD, ALN>(sr, g, kimg, (bf16_t *)dsb + wave * 64 * L::YS, n0, active ? g.N - n0 : 0, Kb, Vb);
    }
    q_commit<DQK, NP, XS, XD, ALN>(rg, g, stages, sc2, sp2, g.N, nt, wave);
    q_request<DQK, NP, ALN>(rg, g, win, qs, ob, ntiles > 1 ? 1 : 0, nt, wave);
    __syncthreads();

    f32x16 accV[2], accK[2][L::RB];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int i = 0; i < 16; ++i) accV[kb][i] = 0.f;
#pragma unroll
        for (int mb = 0; mb < L::RB; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) accK[kb][mb][i] = 0.f;
    }

    // dQ_aug of a tile: 16x16 blocks (16 columns c, the 16 queries of half wave & 1), dealt to the waves
    auto dq_blocks = [&](auto count, int t) {
        constexpr int CNT = decltype(count)::value, CH = CNT == 1 ? 4 : 2;
        // lane constants of the 16x16x32 products: a = row / column, gq = group of four keys
        const int ln = opaque_tid() & 63, a = ln & 15, gq = ln >> 4, krow = 4 * gq + (a >> 2);
        const char *pd = dsb + (t & 1) * dsz + krow * 64 + (((a & 3) * 8) ^ ((gq >> 1) * 16)) + (((wave & 1) ^ (gq & 1)) * 32);
        const char *pk[CNT];
        f32x4 acc[CNT][2];
#pragma unroll
        for (int i = 0; i < CNT; ++i) {
            pk[i] = kimg + krow * U::KB + (a & 3) * 8 + U::block(krow, (wave + i * W) >> 1);
            acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        bf16x8 A[2][CH][CNT], B[2][CH];
        auto fetch = [&](int buf, int s0) {
#pragma unroll
            for (int s = 0; s < CH; ++s) {
                union { s16x4 h[2]; bf16x8 v; } x;
                x.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(pd + (s0 + s) * 2048));
                x.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(pd + (s0 + s) * 2048 + 1024));
                B[buf][s] = x.v;
#pragma unroll
                for (int i = 0; i < CNT; ++i) {
                    x.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(pk[i] + (s0 + s) * 32 * U::KB));
                    x.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(pk[i] + ((s0 + s) * 32 + 16) * U::KB));
                    A[buf][s][i] = x.v;
                }
            }
        };
        fetch(0, 0);
#pragma unroll
        for (int s0 = 0; s0 < NKS; s0 += CH) {
            const int buf = (s0 / CH) & 1;
            if (s0 + CH < NKS) fetch(buf ^ 1, s0 + CH);
            RIB_FENCE();
#pragma unroll
            for (int s = 0; s < CH; ++s)
#pragma unroll
                for (int i = 0; i < CNT; ++i) acc[i][s & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[buf][s][i], B[buf][s], acc[i][s & 1], 0, 0, 0);
        }
        RIB_FENCE();
        const int n = t * 32 + 8 * (a >> 2) + 4 * (wave & 1) + (a & 3);
        if (ALN || n < g.N) {
#pragma unroll
            for (int i = 0; i < CNT; ++i) {
                const int c = (wave + i * W) >> 1, rc = 16 * c + 4 * gq - g.d;
                const f32x4 x = acc[i][0] + acc[i][1];
                if (16 * c < g.d) {
                    char *dst = (char *)dq + ((img * g.C + hd * g.d) * 2 + (int64_t)(token_offset<false>(win.any(n), (int64_t)g.C * 2) + 32u * c + 8u * gq));
                    dword2 z;
                    z.x = pack_bf16(x[0] * g.scale_c, x[1] * g.scale_c);
                    z.y = pack_bf16(x[2] * g.scale_c, x[3] * g.scale_c);
                    if (rc <= -4) *(dword2 *)dst = z;
                    else if (rc == -2) *(uint32_t *)dst = z.x;
                }
                if (16 * c + 16 > g.d) {
                    float *fp = dfq_part + (u * g.N + n) * g.r + rc;
                    const float2 lo = {x[0] * g.scale_p, x[1] * g.scale_p}, hi = {x[2] * g.scale_p, x[3] * g.scale_p};
                    if (rc >= 0 && rc < g.r) *(float2 *)fp = lo;
                    if (rc >= -2 && rc + 2 < g.r) *(float2 *)(fp + 2) = hi;
                }
            }
        }
    };
    auto dq_tile = [&](int t) {
        if constexpr (2 * U::RC % W == 0) {
            dq_blocks(std::integral_constant<int, TPW>(), t);
        } else {
            if (wave + (TPW - 1) * W < 2 * U::RC) dq_blocks(std::integral_constant<int, TPW>(), t);
            else if constexpr (TPW > 1) dq_blocks(std::integral_constant<int, TPW - 1>(), t);
        }
    };

    const int trx = tr_lane_offset<L::XS>(lane), try_ = L::YR + tr_lane_offset<L::YS>(lane);
    const int aqo = col * L::XS + 8 * hf, ago = L::YR + col * L::YS + 8 * hf;
    const int ds_out = col * 64 + ((hf ^ ((col >> 2) & 1)) * 32) + ((col >> 3) & 1) * 16;   // (second half: ^ 16)
#pragma unroll 1
    for (int t = 0; t < ntiles; ++t) {
        const bf16_t *cur = stages + (t & 1) * L::STAGE;
        char *const dsw = dsb + (t & 1) * dsz + wave * 4096;
        if (t > 0) dq_tile(t - 1);
        q_commit<DQK, NP, XS, XD, ALN>(rg, g, stages + ((t + 1) & 1) * L::STAGE, sc2, sp2, rows_left<32>(g, t + 1), nt, wave);
        q_request<DQK, NP, ALN>(rg, g, win, qs, ob, t + 2 < ntiles ? t + 2 : ntiles - 1, nt, wave);
        if (active) {
            bf16x8 Aq[L::KS], Ag[L::VS], Aqt[L::RB][2], Agt[2];
            read_rows<L::KS>(Aq, cur + aqo);
            read_rows<L::VS>(Ag, cur + ago);
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                f32x16 S = {0}, D = {0};
                if (XS || XD) {
                    const float *ex = (const float *)(cur + L::EX) + 4 * hf;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (XS) {
                            const float4 e = *(const float4 *)(ex + 8 * j);
                            S[4 * j] = e.x, S[4 * j + 1] = e.y, S[4 * j + 2] = e.z, S[4 * j + 3] = e.w;
                        }
                        if (XD) {
                            const float4 e = *(const float4 *)(ex + 32 + 8 * j);
                            D[4 * j] = e.x, D[4 * j + 1] = e.y, D[4 * j + 2] = e.z, D[4 * j + 3] = e.w;
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < L::KS; ++i) S = mfma(Aq[i], Kb[kb][i], S);
#pragma unroll
                for (int i = 0; i < L::VS; ++i) D = mfma(Ag[i], Vb[kb][i], D);
                RIB_FENCE();
                if (kb == 0) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        Agt[i] = read_tr<L::YS>(cur + 16 * i * L::YS, try_, 0);
#pragma unroll
                        for (int mb = 0; mb < L::RB; ++mb) Aqt[mb][i] = read_tr<L::XS>(cur + 16 * i * L::XS, trx, 32 * mb);
                    }
                }
                RIB_FENCE();
                if (!ALN && t == ntiles - 1) mask_rows(S, t * 32, g.N, hf);
                uint32_t wp[8], wds[8];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int i = 8 * h; i < 8 * h + 8; ++i) S[i] = __builtin_amdgcn_exp2f(S[i]);
                    RIB_FENCE();
#pragma unroll
                    for (int i = 8 * h; i < 8 * h + 8; ++i) D[i] *= S[i];
#pragma unroll
                    for (int i = 8 * h; i < 8 * h + 8; i += 2) wp[i >> 1] = pack_bf16(S[i], S[i + 1]);
#pragma unroll
                    for (int i = 8 * h; i < 8 * h + 8; i += 2) wds[i >> 1] = pack_bf16(D[i], D[i + 1]);
                    if (!ALN) {                 // keys past the window's end
#pragma unroll
                        for (int i = 4 * h; i < 4 * h + 4; ++i) wds[i] = n0 + kb * 32 + col < g.N ? wds[i] : 0u;
                    }
                    RIB_FENCE();
                    const bf16x8 B = as_bf16x8(wds[4 * h], wds[4 * h + 1], wds[4 * h + 2], wds[4 * h + 3]);
                    *(bf16x8 *)(dsw + kb * 2048 + (h ? ds_out ^ 16 : ds_out)) = B;
                    accV[kb] = mfma(Agt[h], as_bf16x8(wp[4 * h], wp[4 * h + 1], wp[4 * h + 2], wp[4 * h + 3]), accV[kb]);
#pragma unroll
                    for (int mb = 0; mb < L::RB; ++mb) accK[kb][mb] = mfma(Aqt[mb][h], B, accK[kb][mb]);
                }
            }
        } else if (t < 2) {     // no keys: the products over all waves' keys meet zeros
#pragma unroll
            for (int i = 0; i < 4; ++i) *(uint4 *)(dsw + (i * 64 + lane) * 16) = uint4{0u, 0u, 0u, 0u};
        }
        RIB_FENCE();
        __syncthreads();
    }
    // (the streamed Q_aug rows carry scale * log2 e: undo the log2 e here)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const int n = n0 + kb * 32 + col;
        if (n < g.N) {
            const int64_t base = (img + win.any(n)) * g.C + hd * g.d;
            char *pd = (char *)(dfk_part + (u * g.N + n) * g.r);
#pragma unroll
            for (int mb = 0; mb < L::RB; ++mb) bwd::store_block(accK[kb][mb], mb, hf, g, kLn2, kLn2, (char *)(dk + base), pd);
            bwd::store_block(accV[kb], 0, hf, g, 1.f, 1.f, (char *)(dv + base), nullptr);
        }
    }
    dq_tile(ntiles - 1);
}

template <int DQK, bool XS, bool XD, bool ALN, int W>
hipError_t launch_unit(const Geo &g, const Args &a)
{
    const size_t smem = ULay<DQK>::bytes(W) + (ALN ? 0 : (size_t)2 * g.M * sizeof(int));
    if (smem > (size_t)kMaxDynLds) return hipErrorInvalidValue;
    auto kern = unit_kernel<DQK, XS, XD, ALN, W>;
    const hipError_t e = prepare_kernel((const void *)kern, nullptr);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)g.units), dim3(W * 64), smem, a.st, g, a.q, a.k, a.v, a.fq, a.fk,
                       a.out, a.dout, a.lse, a.dq, a.dk, a.dv, a.pq, a.pk);
    return hipGetLastError();
}
template <int DQK, bool XS, bool XD>
hipError_t unit_width(const Geo &g, const Args &a)
{
    if (g.M % 8 == 0)       // (8 or 16)
        return g.N <= 128 ? launch_unit<DQK, XS, XD, true, 2>(g, a) : launch_unit<DQK, XS, XD, true, 4>(g, a);
    return g.N <= 128 ? launch_unit<DQK, XS, XD, false, 2>(g, a) : g.N <= 256 ? launch_unit<DQK, XS, XD, false, 4>(g, a)
                                                                               : launch_unit<DQK, XS, XD, false, 8>(g, a);
}
template <int DQK>
hipError_t unit_flags(const Geo &g, const Args &a)
{
    const bool xs = g.d + g.r + 2 > DQK, xd = g.d + 2 > 32;
    if constexpr (DQK == 32) {
        return xs ? unit_width<DQK, true, false>(g, a) : unit_width<DQK, false, false>(g, a);
    } else {
        if (xd) return xs ? unit_width<DQK, true, true>(g, a) : unit_width<DQK, false, true>(g, a);
        return xs ? unit_width<DQK, true, false>(g, a) : unit_width<DQK, false, false>(g, a);
    }
}
hipError_t launch32(const Geo &g, const Args &a);
hipError_t launch48(const Geo &g, const Args &a);
hipError_t launch64(const Geo &g, const Args &a);

}  // namespace unit
}  // namespace rib

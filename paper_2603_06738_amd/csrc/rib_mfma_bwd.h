// RIB window attention, backward, on the gfx950 matrix cores (bf16 MFMA, fp32
// accumulation).  Gradient formulas: include/rib_attn.h (chain rule through paper
// Sec. 2.2 and Sec. 3.1 Eq. 5-6).
//
// Two kernels, both free of atomics so that every output is run-to-run identical:
//
//   dq kernel   -- a wave owns 64 queries (MFMA B operands in registers) and the workgroup
//     streams the unit's keys through LDS.  Per 32x32 block it forms the TRANSPOSED scores
//     S^T = K_aug Q_aug^T and dP^T = V dO^T (a lane owns a QUERY column), so dS^T is the B
//     operand of dQ_aug^T += K_aug^T dS^T (contraction over keys).
//   dkv kernel  -- a wave owns 64 keys and the workgroup streams the queries; S = Q_aug K_aug^T
//     and dP = dO V^T with a lane owning a KEY column, so P and dS, packed to bf16, are the B
//     operands of dV^T += dO^T P and dK_aug^T += Q_aug^T dS (contractions over queries).
//
//   In both kernels it is Q_aug that carries scale * log2(e), rounded to bf16 exactly as the
//   forward rounds it, so the recomputed logits are the forward's bit for bit.  P is recomputed
//   as exp2(S - LSE) and dS = P (dP - delta).  Where the padding of the augmented rows has two
//   free columns neither subtraction costs a vector instruction: -LSE*log2(e), split into a bf16
//   high and low part, rides in the last two columns of Q_aug against ones in K_aug, and -delta
//   rides the same way in the padding of dO against ones in V.  Without free columns (template
//   flags XS for the scores, XD for dP) they enter as the C operand of the first MFMA (dkv: a
//   lane's accumulator rows are queries) or as a lane constant added to the result (dq: a lane
//   is one query).
//
//   What bounds them: neither pipe by itself.  By counters (32 x 32 windows, d = 30, r = 16) the matrix pipe
//   (11 MFMAs a 32x32 block in dkv, 9 in dq) is busy 36 / 36 % of the SIMD-cycles and the vector ALU (89 / 75
//   instructions a block, of which exp2, multiplies and packs are 48 / 40) 42 / 45 %; for 44 / 39 % of its time a
//   wave waits on its previous instruction, and only two waves of 256 registers share a SIMD.  What both pipes
//   need less of is staging (a build without it is 14 to 20 % faster).  So the streamed
//   tiles are kept as plain rows in LDS, written in 16-byte pieces, and the operands of the
//   products that contract over tokens are read TRANSPOSED from the same rows
//   (ds_read_b64_tr_b16): no transposed image, no byte permutes to build one.  One pair of kernels
//   serves every window of more tokens than one workgroup holds (rib_mfma_unit.h), and of 64 and more where those do not: a last partial tile repeats the window's last token
//   and masks its rows of S (the separate kernels for windows that were not whole 256-token blocks,
//   with their predicated staging, took 656 us where these take about 280 us: 24 x 24 windows, 8 x 96 x 96
//   tokens, 6 heads, d = 30, r = 18).  Registers spilled: none with 32 columns, and none with 48 where the window side
//   is a multiple of 8.  With 64 dkv spills 4 to 13 (odd sides 9 to 26), in eight waves and in groups up to 12; dq, on sides that are no multiple of 8
//   only, 17 to 45 with 48 columns and 29 to 69 with 64 (two-channel heads 95).
//
//   The last r columns of dQ_aug / dK_aug are this unit's contribution to dF_q /
//   dF_k (Sec. 3.1: the RIB features are shared by all windows); they go to a
//   per-unit fp32 scratch and are summed over windows in a fixed order afterwards.
#pragma once

#include "rib_rows.h"

namespace rib {
namespace bwd {

using namespace rows;

// Raw words of a wave's 64 stationary rows between their request and their staging, 64 / LANES rows a pass.
template <int DQK, bool WITH_O, int TINY>
struct StatRegs {
    static constexpr int P = Moved<TINY>::LANES;        // passes
    Words<TINY> x[P], y[P], fa[P], fb[DQK == 64 ? P : 1], o[WITH_O ? P : 1];
    float e0, e1;
};
template <int DQK, bool QDO, bool WITH_O, bool ALN, int TINY, bool BIG>
__device__ __forceinline__ void stat_request(StatRegs<DQK, WITH_O, TINY> &r, const Geo &g, const Win &win, const Stream &s, int n0,
                                             const char *ob, bool from_o)
{
    using M = Moved<TINY>;
    const int lane = threadIdx.x & 63, l = lane / M::LANES;
    const Piece pc = piece_of<TINY>(g, lane % M::LANES);
#pragma unroll
    for (int p = 0; p < M::LANES; ++p) {
        // (a wave past the window's end repeats its last rows)
        const int nf = n0 + p * M::ROWS, nb = ALN && nf > win.last - (M::ROWS - 1) ? win.last - (M::ROWS - 1) : nf, n = nb + l;
        const uint32_t t = win.token<ALN, M::ROWS>(nb, l);
        r.x[p] = get<TINY>(s.xb, token_offset<BIG>(t, s.xs) + 4u * pc.dc, pc.c1);
        r.y[p] = get<TINY>(s.yb, token_offset<BIG>(t, s.ys) + 4u * pc.dc, pc.c1);
        if (WITH_O && from_o) r.o[p] = get<TINY>(ob, token_offset<BIG>(t, s.ys) + 4u * pc.dc, pc.c1);
        if (!pc.fnone) {
            const uint32_t fr = __umul24((uint32_t)(n < win.last ? n : win.last), s.frow);
            r.fa[p] = get<TINY>(s.fb, fr + 4u * pc.f0, pc.f1d);
            if (DQK == 64) r.fb[p] = get<TINY>(s.fb, fr + 4u * pc.f1, pc.f1d);
        }
    }
    r.e0 = r.e1 = 0.f;
    if (QDO) {
        const int n = n0 + lane, nc = n < win.last ? n : win.last;
        r.e0 = s.lse[nc];
        if (!WITH_O || !from_o) r.e1 = s.delta[nc];
    }
}

// delta_i = dO_i . O_i (paper Sec. 2.2 backward; the softmax Jacobian's row term) of the wave's 64
// rows from the words the lanes hold: each lane multiplies its channel pairs, halving
// steps over the lanes of a row (lane ^ 7, ^ 2, ^ 1: DPP patterns; four lanes: the last two) leave lane j of a row's lanes
// with the row of pass j, and a lane permute hands row `lane` its value.
template <int DQK, int TINY>
__device__ __forceinline__ float make_delta(const StatRegs<DQK, true, TINY> &r, const Geo &g)
{
    using M = Moved<TINY>;
    const int lane = threadIdx.x & 63, j = lane % M::LANES;
    const Piece pc = piece_of<TINY>(g, j);
    float part[M::LANES];
#pragma unroll
    for (int p = 0; p < M::LANES; ++p) {
        part[p] = 0.f;
#pragma unroll
        for (int i = 0; i < M::WORDS; ++i) {
            // (a slid piece counts its new words only)
            const bool own = pc.c1 ? i == 0 && j == 0 : pc.dc + i >= M::WORDS * j;
            const float a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, r.y[p].w[i]), __builtin_bit_cast(bf16x2, r.o[p].w[i]), 0.f, false);
            part[p] += own ? a : 0.f;
        }
    }
#define RIB_DPP(x, ctrl) __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, (x)), (ctrl), 0xF, 0xF, true))
    const bool b2 = (j & 4) != 0, b1 = (j & 2) != 0, b0 = (j & 1) != 0;
    float h4[4], h2[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (M::LANES == 8) {
            const float keep = b2 ? part[4 + i] : part[i], give = b2 ? part[i] : part[4 + i];
            h4[i] = keep + RIB_DPP(give, 0x141);        // row_half_mirror: lane ^ 7
        } else {
            h4[i] = part[i];
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float keep = b1 ? h4[2 + i] : h4[i], give = b1 ? h4[i] : h4[2 + i];
        h2[i] = keep + RIB_DPP(give, 0x4E);         // quad_perm [2,3,0,1]: lane ^ 2
    }
    const float keep = b0 ? h2[1] : h2[0], give = b0 ? h2[0] : h2[1];
    const float mine = keep + RIB_DPP(give, 0xB1);  // quad_perm [1,0,3,2]: lane ^ 1
#undef RIB_DPP
    return __shfl(mine, (lane % M::ROWS) * M::LANES + lane / M::ROWS);
}

// Stage the wave's 64 rows through its private LDS area and read them back as MFMA B operands.  `ftab` (QDO, may be
// null): where this head's scaled RIB rows go for the dkv kernel.
template <int DQK, bool QDO, bool XS, bool XD, bool WITH_O, int TINY>
__device__ __forceinline__ void stat_stage(const StatRegs<DQK, WITH_O, TINY> &r, const Geo &g, bf16_t *W, float sc, float sp, float nl,
                                           float nd, bf16x8 (&Xb)[2][DQK / 16], bf16x8 (&Yb)[2][2], char *ftab = nullptr,
                                           int n0 = 0, bool aln = false)
{
    using L = Lay<DQK, 64>;
    using M = Moved<TINY>;
    const int lane = threadIdx.x & 63, l = lane / M::LANES, col = lane & 31, hf = lane >> 5;
    const Piece pc = piece_of<TINY>(g, lane % M::LANES);
    bf16_t *Xs = W, *Ys = W + 64 * L::XS;
    {   // padding columns and extras of row `lane`
        bf16_t *xr = Xs + lane * L::XS, *yr = Ys + lane * L::YS;
        for (int c = g.d + g.r; c < DQK - (XS ? 0 : 2); c += 2) *(uint32_t *)(xr + c) = 0u;
        for (int c = g.d; c < L::DVK - (XD ? 0 : 2); c += 2) *(uint32_t *)(yr + c) = 0u;
        if (!XS) *(uint32_t *)(xr + DQK - 2) = QDO ? split_bf16(nl) : 0x3f803f80u;
        if (!XD) *(uint32_t *)(yr + L::DVK - 2) = QDO ? split_bf16(nd) : 0x3f803f80u;
    }
    bf16_t *xr = Xs + l * L::XS + 2 * pc.dc, *yr = Ys + l * L::YS + 2 * pc.dc;
    bf16_t *fr = Xs + l * L::XS + g.d + 2 * pc.f0, *fr1 = Xs + l * L::XS + g.d + 2 * pc.f1;
#pragma unroll
    for (int p = 0; p < M::LANES; ++p) {
        put<TINY>(xr + p * M::ROWS * L::XS, QDO ? scaled<TINY>(r.x[p], sc) : r.x[p], pc.c1);
        put<TINY>(yr + p * M::ROWS * L::YS, r.y[p], pc.c1);
        if (!pc.fnone) {
            const Words<TINY> fa = QDO ? scaled<TINY>(r.fa[p], sp) : r.fa[p];
            Words<TINY> fb;
            if (DQK == 64) fb = QDO ? scaled<TINY>(r.fb[p], sp) : r.fb[p];
            put<TINY>(fr + p * M::ROWS * L::XS, fa, pc.f1d);
            if (DQK == 64) put<TINY>(fr1 + p * M::ROWS * L::XS, fb, pc.f1d);
            if (QDO && has_table(TINY) && ftab) {
                const int n = n0 + p * M::ROWS + l, last = g.N - 1, nb = aln && n0 + p * M::ROWS > last - (M::ROWS - 1) ? last - (M::ROWS - 1) + l : n;
                char *row = ftab + __umul24((uint32_t)(nb < last ? nb : last), (uint32_t)g.r * 2u);
                put<TINY>((bf16_t *)(row + 4u * pc.f0), fa, pc.f1d);
                if (DQK == 64) put<TINY>((bf16_t *)(row + 4u * pc.f1), fb, pc.f1d);
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        read_rows<L::KS>(Xb[b], Xs + (b * 32 + col) * L::XS + 8 * hf);
        read_rows<L::VS>(Yb[b], Ys + (b * 32 + col) * L::YS + 8 * hf);
    }
}

// One 32-row accumulator block of a gradient: this lane's token, rows 32*mb + 8*a + 4*hf + 0..3 in
// registers 4a .. 4a+3.  Columns below d go to the grid tensor (bf16, times sc), the next r to this
// unit's RIB partial (fp32, times sp).
__device__ __forceinline__ void store_block(const f32x16 &acc, int mb, int hf, const Geo &g, float sc, float sp, char *grid_dst,
                                            char *part_dst)
{
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int c = 32 * mb + 8 * a + 4 * hf;
        const float v0 = acc[4 * a], v1 = acc[4 * a + 1], v2 = acc[4 * a + 2], v3 = acc[4 * a + 3];
        if (c + 2 <= g.d) {
            dword2 w;
            w.x = pack_bf16(v0 * sc, v1 * sc);
            w.y = pack_bf16(v2 * sc, v3 * sc);
            if (c + 4 <= g.d) {
                *(dword2 *)(grid_dst + 2 * c) = w;
            } else {            // the head's last pair, then the first two RIB columns
                *(uint32_t *)(grid_dst + 2 * c) = w.x;
                if (g.r > 0 && part_dst) *(float2u *)part_dst = float2u{v2 * sp, v3 * sp};
            }
        } else if (part_dst && c + 2 <= g.d + g.r) {
            char *dst = part_dst + 4 * (c - g.d);
            if (c + 4 <= g.d + g.r) *(float4u *)dst = float4u{v0 * sp, v1 * sp, v2 * sp, v3 * sp};
            else *(float2u *)dst = float2u{v0 * sp, v1 * sp};
        }
    }
}

// Sums of groups of waves that share stationary rows: accumulators through LDS, a row of 64 lanes a register.
template <int DQK, bool DQ>
constexpr int sums_of() { return (2 * Lay<DQK, 64>::RB + (DQ ? 0 : 2)) * 16 * 64; }    // floats a wave
template <int N>
__device__ __forceinline__ void give_sums(const f32x16 (&acc)[N], float *part)
{
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) part[(b * 16 + i) * 64] = acc[b][i];
}
template <int N>
__device__ __forceinline__ void take_sums(f32x16 (&acc)[N], const float *part)
{
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[b][i] += part[(b * 16 + i) * 64];
}
template <int N, int M>
__device__ __forceinline__ void give_sums(const f32x16 (&acc)[N][M], float *part)
{
#pragma unroll
    for (int b = 0; b < N; ++b) give_sums(acc[b], part + b * M * 1024);
}
template <int N, int M>
__device__ __forceinline__ void take_sums(f32x16 (&acc)[N][M], const float *part)
{
#pragma unroll
    for (int b = 0; b < N; ++b) take_sums(acc[b], part + b * M * 1024);
}

// Common start of both kernels.
#define RIB_BWD_SETUP                                                                                      \
    using L = Lay<DQK, T>;                                                                                 \
    extern __shared__ __attribute__((aligned(16))) bf16_t smem[];                                          \
    const int nt = T >= 64 ? NT : (int)blockDim.x, waves = nt >> 6;                                        \
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);                                     \
    const int lane = threadIdx.x & 63, col = lane & 31, hf = lane >> 5;                                    \
    int64_t u;                                                                                             \
    int blk, b;                                                                                            \
    block_coords(nblk, u, blk);                                                                            \
    const int w = (int)(u / g.heads), hd = (int)(u - (int64_t)w * g.heads);                                \
    const Win win = window_of<ALN>(g, w, nt, (int *)((char *)smem + L::bytes(waves)), b);                  \
    const int64_t img = (int64_t)b * g.H * g.W;                                                            \
    Stream ks, qs;                                                                                         \
    ks.xb = (const char *)(k + img * g.tstride + hd * g.d);                                                \
    ks.yb = (const char *)(v + img * g.tstride + hd * g.d);                                                \
    ks.fb = (const char *)(fk + (int64_t)hd * g.N * g.r);                                                  \
    ks.xs = ks.ys = qs.xs = g.tstride * 2;                                                                 \
    ks.frow = qs.frow = (uint32_t)g.r * 2u;                                                                \
    qs.xb = (const char *)(q + img * g.tstride + hd * g.d);                                                \
    qs.yb = (const char *)(dout + img * g.C + hd * g.d);                                                   \
    qs.fb = (const char *)(fq + (int64_t)hd * g.N * g.r);                                                  \
    qs.ys = (int64_t)g.C * 2;                                                                              \
    ks.lse = qs.lse = lse + u * g.N;                                                                       \
    ks.delta = qs.delta = delta + u * g.N;                                                                 \
    const float sc2 = g.scale_c * kLog2e;                                                                  \
    /* G groups share the stationary rows of waves / G waves */                                             \
    const int own = waves / G, grp = G == 1 ? 0 : wave / own, n0 = (blk * own + (G == 1 ? wave : wave % own)) * 64;   \
    const int ntiles = (g.N + T - 1) / T;                                                                  \
    if (!ALN) __syncthreads();

// dQ (+ dF_q partial).  A lane stages at most two tokens a tile: T = 64 with 4 waves (NT = 256 lanes; dkv also 8), T = 32 with 2 or 3;
// in two groups of waves T = 64 and in four T = 128, with 8 (both kernels).
//
// One step is one 32x32 block s = (key block, query block); its instructions are written in the
// order they should issue and pinned with scheduling fences: the 5 score MFMAs of block s + 1 and
// the 2 * RB gradient MFMAs of block s - 1 are spread between the exponentials, products and packs
// of block s, so that the matrix pipe and the vector ALU always have independent work (left alone,
// the compiler chains exp2 -> multiply -> pack element by element and waits for every LDS read
// where it is issued).
template <int DQK, int T, bool XS, bool XD, bool ALN, int TINY, bool BIG, int NT, int G>
__global__ __launch_bounds__(T >= 64 ? NT : 192, 2) void dq_kernel(Geo g, int nblk, const bf16_t *__restrict__ q, const bf16_t *__restrict__ k,
                                                      const bf16_t *__restrict__ v, const bf16_t *__restrict__ fq,
                                                      const bf16_t *__restrict__ fk, const bf16_t *__restrict__ out,
                                                      const bf16_t *__restrict__ dout, const float *__restrict__ lse,
                                                      float *__restrict__ delta, bf16_t *__restrict__ dq,
                                                      float *__restrict__ dfq_part, bf16_t *__restrict__ ftab)
{
    RIB_BWD_SETUP
    constexpr int NB = T / 32 / G, NS = 2 * NB;             // key blocks of a tile: of this wave's group
    const float sp2 = g.scale_p * kLog2e;

    // one exposed memory latency: the wave's rows and the first two tiles are requested together
    Regs<DQK, TINY> rg, rg1;
    bf16x8 Qb[2][L::KS], Gb[2][L::VS];
    float nl[2] = {0.f, 0.f}, nd[2] = {0.f, 0.f};
    {
        StatRegs<DQK, true, TINY> sr;
        const bool from_o = g.gate == nullptr;          // a gated call's pass over dO', G and O has made delta already
        stat_request<DQK, true, true, ALN, TINY, BIG>(sr, g, win, qs, n0, (const char *)(out + img * g.C + hd * g.d), from_o);
        request<DQK, T, false, ALN, TINY, BIG>(rg, g, win, ks, 0, nt, wave);
        request<DQK, T, false, ALN, TINY, BIG>(rg1, g, win, ks, ntiles > 1 ? 1 : 0, nt, wave);
        float dl = sr.e1;
        if (from_o) {
            dl = make_delta<DQK, TINY>(sr, g);
            if (n0 + lane < g.N && grp == 0) delta[u * g.N + n0 + lane] = dl;   // for the dkv kernel, which runs second
        }
        const float l2 = -sr.e0 * kLog2e;
        stat_stage<DQK, true, XS, XD, true, TINY>(sr, g, smem + wave * L::WAVE_STAT, sc2, sp2, l2, -dl, Qb, Gb,
                                                      w == 0 && grp == 0 ? (char *)(ftab + (int64_t)hd * g.N * g.r) : nullptr, n0, ALN);
        if (XS) nl[0] = __shfl(l2, col), nl[1] = __shfl(l2, 32 + col);
        if (XD) nd[0] = -__shfl(dl, col), nd[1] = -__shfl(dl, 32 + col);
    }
    __syncthreads();
    init_pads<DQK, T, false, XS, XD>(g, smem, nt);
    commit<DQK, T, false, XS, XD, ALN, TINY>(rg, g, smem, 1.f, 1.f, g.N, nt, wave);
    commit<DQK, T, false, XS, XD, ALN, TINY>(rg1, g, smem + L::STAGE, 1.f, 1.f, ntiles > 1 ? g.N - T : g.N, nt, wave);
    request<DQK, T, false, ALN, TINY, BIG>(rg, g, win, ks, ntiles > 2 ? 2 : ntiles - 1, nt, wave);
    __syncthreads();

    f32x16 acc[2][L::RB];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int mb = 0; mb < L::RB; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[qb][mb][i] = 0.f;

    // (a group's first block of a tile: its rows are `g0` past the tile's)
    const int g0 = G == 1 ? 0 : grp * 32 * NB;
    const int tro = tr_lane_offset<L::XS>(lane) + g0 * L::XS, ako = (g0 + col) * L::XS + 8 * hf, avo = L::YR + (g0 + col) * L::YS + 8 * hf;
    bf16x8 Ak[L::KS], Av[L::VS], At[L::RB][2];
    f32x16 S[2], D[2];
    uint32_t P[2][8];
    read_rows<L::KS>(Ak, smem + ako);
    read_rows<L::VS>(Av, smem + avo);
    {
        const f32x16 z = {0};
        S[0] = mfma(Ak[0], Qb[0][0], z);
        D[0] = mfma(Av[0], Gb[0][0], z);
#pragma unroll
        for (int i = 1; i < L::KS; ++i) S[0] = mfma(Ak[i], Qb[0][i], S[0]);
        D[0] = mfma(Av[1], Gb[0][1], D[0]);
#pragma unroll
        for (int i = 0; i < 8; ++i) P[1][i] = 0u;         // (the first step's gradient products add zero)
#pragma unroll
        for (int mb = 0; mb < L::RB; ++mb)
#pragma unroll
            for (int i = 0; i < 2; ++i) At[mb][i] = as_bf16x8(0u, 0u, 0u, 0u);
    }
    int c0 = 0, c1 = L::STAGE, c2 = 2 * L::STAGE;        // this tile's, the next tile's and the free stage
    for (int tile = 0; tile < ntiles; ++tile) {
        const bf16_t *cur = smem + c0, *nxt = smem + c1;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int kb = s >> 1, qb = s & 1, cs = s & 1, ns = cs ^ 1, qn = qb ^ 1;
            const f32x16 z = {0};
            RIB_FENCE();
            // scores of block s + 1
            S[ns] = mfma(Ak[0], Qb[qn][0], z);
            D[ns] = mfma(Av[0], Gb[qn][0], z);
            if (!ALN && tile == ntiles - 1) mask_rows(S[cs], tile * T + g0 + kb * 32, g.N, hf);
            float p[16];
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(XS ? S[cs][i] + nl[qb] : S[cs][i]);
            RIB_FENCE();
            S[ns] = mfma(Ak[1], Qb[qn][1], S[ns]);
            D[ns] = mfma(Av[1], Gb[qn][1], D[ns]);
#pragma unroll
            for (int i = 4; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(XS ? S[cs][i] + nl[qb] : S[cs][i]);
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] *= XD ? D[cs][i] + nd[qb] : D[cs][i];
            if (s == 0) commit<DQK, T, false, XS, XD, ALN, TINY>(rg, g, smem + c2, 1.f, 1.f, rows_left<T>(g, tile + 2), nt, wave);
            RIB_FENCE();
#pragma unroll
            for (int i = 2; i < L::KS; ++i) S[ns] = mfma(Ak[i], Qb[qn][i], S[ns]);
#pragma unroll
            for (int i = 8; i < 12; ++i) p[i] = __builtin_amdgcn_exp2f(XS ? S[cs][i] + nl[qb] : S[cs][i]);
            P[cs][0] = pack_bf16(p[0], p[1]);
            P[cs][1] = pack_bf16(p[2], p[3]);
#pragma unroll
            for (int i = 4; i < 8; ++i) p[i] *= XD ? D[cs][i] + nd[qb] : D[cs][i];
            if (qb == 0) {      // operands of the next key block (behind this tile's last, of the next tile)
                read_rows<L::KS>(Ak, (kb + 1 < NB ? cur + (kb + 1) * 32 * L::XS : nxt) + ako);
                read_rows<L::VS>(Av, (kb + 1 < NB ? cur + (kb + 1) * 32 * L::YS : nxt) + avo);
            }
            RIB_FENCE();
            // gradient of block s - 1
            const bf16x8 B0 = as_bf16x8(P[ns][0], P[ns][1], P[ns][2], P[ns][3]), B1 = as_bf16x8(P[ns][4], P[ns][5], P[ns][6], P[ns][7]);
#pragma unroll
            for (int mb = 0; mb < L::RB; ++mb) acc[qn][mb] = mfma(At[mb][0], B0, acc[qn][mb]);
#pragma unroll
            for (int i = 12; i < 16; ++i) p[i] = __builtin_amdgcn_exp2f(XS ? S[cs][i] + nl[qb] : S[cs][i]);
            P[cs][2] = pack_bf16(p[4], p[5]);
            P[cs][3] = pack_bf16(p[6], p[7]);
#pragma unroll
            for (int i = 8; i < 12; ++i) p[i] *= XD ? D[cs][i] + nd[qb] : D[cs][i];
            RIB_FENCE();
#pragma unroll
            for (int mb = 0; mb < L::RB; ++mb) acc[qn][mb] = mfma(At[mb][1], B1, acc[qn][mb]);
            P[cs][4] = pack_bf16(p[8], p[9]);
            P[cs][5] = pack_bf16(p[10], p[11]);
#pragma unroll
            for (int i = 12; i < 16; ++i) p[i] *= XD ? D[cs][i] + nd[qb] : D[cs][i];
            P[cs][6] = pack_bf16(p[12], p[13]);
            P[cs][7] = pack_bf16(p[14], p[15]);
            RIB_FENCE();
            if (qb == 0) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int mb = 0; mb < L::RB; ++mb) At[mb][i] = read_tr<L::XS>(cur + (kb * 32 + 16 * i) * L::XS, tro, 32 * mb);
            }
            if (s == NS - 1) request<DQK, T, false, ALN, TINY, BIG>(rg, g, win, ks, tile + 3 < ntiles ? tile + 3 : ntiles - 1, nt, wave);
        }
        RIB_FENCE();
        __syncthreads();
        const int r0 = c0;
        c0 = c1, c1 = c2, c2 = r0;
    }
    {   // gradient of the last block
        const bf16x8 B0 = as_bf16x8(P[1][0], P[1][1], P[1][2], P[1][3]), B1 = as_bf16x8(P[1][4], P[1][5], P[1][6], P[1][7]);
#pragma unroll
        for (int mb = 0; mb < L::RB; ++mb) {
            acc[1][mb] = mfma(At[mb][0], B0, acc[1][mb]);
            acc[1][mb] = mfma(At[mb][1], B1, acc[1][mb]);
        }
    }

    if (G > 1) {
        float *const part = (float *)smem + lane;
        if (grp > 0) give_sums(acc, part + (wave - own) * sums_of<DQK, true>());
        __syncthreads();
        if (grp > 0) return;
#pragma unroll 1            // (several groups' sums in flight are spills: dkv 150 to 160 registers in four groups)
        for (int j = 0; j < G - 1; ++j) take_sums(acc, part + (wave + j * own) * sums_of<DQK, true>());
    }
    // Outputs straight from the accumulator layout: a lane holds, for one token, groups of four
    // consecutive columns (8-byte stores of the gradient, 16-byte stores of the partial).
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
        const int n = n0 + qb * 32 + col;
        if (n < g.N) {
            char *gd = (char *)(dq + (img + win.any(n)) * g.C + hd * g.d);
            char *pd = (char *)(dfq_part + (u * g.N + n) * g.r);
#pragma unroll
            for (int mb = 0; mb < L::RB; ++mb) store_block(acc[qb][mb], mb, hf, g, g.scale_c, g.scale_p, gd, pd);
        }
    }
}

// dK, dV (+ dF_k partial).  `fq` is, where has_table, the dq kernel's table of scaled RIB rows (they are the same for every window, and
// scaling them while they are staged cost a tenth of the loop's vector instructions).  Same walk with the roles exchanged.  There are no registers for a second
// pair of score blocks here, so the phases of a block alternate (the two waves of a SIMD fill each
// other's): gradient MFMAs of the block before and score MFMAs, then exponentials, products, packs.
template <int DQK, int T, bool XS, bool XD, bool ALN, int TINY, bool BIG, int NT, int G>
__global__ __launch_bounds__(T >= 64 ? NT : 192, 2) void dkv_kernel(Geo g, int nblk, const bf16_t *__restrict__ q, const bf16_t *__restrict__ k,
                                                       const bf16_t *__restrict__ v, const bf16_t *__restrict__ fq,
                                                       const bf16_t *__restrict__ fk, const bf16_t *__restrict__ dout,
                                                       const float *__restrict__ lse, const float *__restrict__ delta,
                                                       bf16_t *__restrict__ dk, bf16_t *__restrict__ dv,
                                                       float *__restrict__ dfk_part)
{
    RIB_BWD_SETUP
    constexpr int NB = T / 32 / G;          // query blocks of a tile: of this wave's group
    const float sp2 = g.scale_p * kLog2e;

    Regs<DQK, TINY> rg, rg1;
    bf16x8 Kb[2][L::KS], Vb[2][L::VS];
    {
        StatRegs<DQK, false, TINY> sr;
        stat_request<DQK, false, false, ALN, TINY, BIG>(sr, g, win, ks, n0, nullptr, false);
        request<DQK, T, true, ALN, TINY, BIG>(rg, g, win, qs, 0, nt, wave);
        request<DQK, T, true, ALN, TINY, BIG>(rg1, g, win, qs, ntiles > 1 ? 1 : 0, nt, wave);
        stat_stage<DQK, false, XS, XD, false, TINY>(sr, g, smem + wave * L::WAVE_STAT, 1.f, 1.f, 0.f, 0.f, Kb, Vb);
    }
    __syncthreads();
    init_pads<DQK, T, true, XS, XD>(g, smem, nt);
    commit<DQK, T, true, XS, XD, ALN, TINY>(rg, g, smem, sc2, sp2, g.N, nt, wave);
    commit<DQK, T, true, XS, XD, ALN, TINY>(rg1, g, smem + L::STAGE, sc2, sp2, ntiles > 1 ? g.N - T : g.N, nt, wave);
    request<DQK, T, true, ALN, TINY, BIG>(rg, g, win, qs, ntiles > 2 ? 2 : ntiles - 1, nt, wave);
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
    const int g0 = G == 1 ? 0 : grp * 32 * NB;

    const int trx = tr_lane_offset<L::XS>(lane) + g0 * L::XS, try_ = L::YR + tr_lane_offset<L::YS>(lane) + g0 * L::YS;
    const int aqo = (g0 + col) * L::XS + 8 * hf, ago = L::YR + (g0 + col) * L::YS + 8 * hf;
    bf16x8 Aq[L::KS], Ag[L::VS];
    read_rows<L::KS>(Aq, smem + aqo);
    read_rows<L::VS>(Ag, smem + ago);
    int c0 = 0, c1 = L::STAGE, c2 = 2 * L::STAGE;
    for (int tile = 0; tile < ntiles; ++tile) {
        const bf16_t *cur = smem + c0, *nxt = smem + c1;
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) {
            bf16x8 Aqt[L::RB][2], Agt[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                f32x16 S = {0}, D = {0};
                if (XS || XD) {
                    // accumulator row 8j + 4*hf + e is query qb*32 + that: four consecutive floats per j
                    const float *ex = (const float *)(cur + L::EX) + g0 + qb * 32 + 4 * hf;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (XS) {
                            const float4 a = *(const float4 *)(ex + 8 * j);
                            S[4 * j] = a.x, S[4 * j + 1] = a.y, S[4 * j + 2] = a.z, S[4 * j + 3] = a.w;
                        }
                        if (XD) {
                            const float4 a = *(const float4 *)(ex + T + 8 * j);
                            D[4 * j] = a.x, D[4 * j + 1] = a.y, D[4 * j + 2] = a.z, D[4 * j + 3] = a.w;
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
                        Agt[i] = read_tr<L::YS>(cur + (qb * 32 + 16 * i) * L::YS, try_, 0);
#pragma unroll
                        for (int mb = 0; mb < L::RB; ++mb)
                            Aqt[mb][i] = read_tr<L::XS>(cur + (qb * 32 + 16 * i) * L::XS, trx, 32 * mb);
                    }
                    if (qb == 0) commit<DQK, T, true, XS, XD, ALN, TINY>(rg, g, smem + c2, sc2, sp2, rows_left<T>(g, tile + 2), nt, wave);
                } else {
                    read_rows<L::KS>(Aq, (qb + 1 < NB ? cur + (qb + 1) * 32 * L::XS : nxt) + aqo);
                    read_rows<L::VS>(Ag, (qb + 1 < NB ? cur + (qb + 1) * 32 * L::YS : nxt) + ago);
                    if (qb == NB - 1)
                        request<DQK, T, true, ALN, TINY, BIG>(rg, g, win, qs, tile + 3 < ntiles ? tile + 3 : ntiles - 1, nt, wave);
                }
                RIB_FENCE();
                if (!ALN && tile == ntiles - 1) mask_rows(S, tile * T + g0 + qb * 32, g.N, hf);
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
                    RIB_FENCE();
                    const bf16x8 B = as_bf16x8(wds[4 * h], wds[4 * h + 1], wds[4 * h + 2], wds[4 * h + 3]);
                    accV[kb] = mfma(Agt[h], as_bf16x8(wp[4 * h], wp[4 * h + 1], wp[4 * h + 2], wp[4 * h + 3]), accV[kb]);
#pragma unroll
                    for (int mb = 0; mb < L::RB; ++mb) accK[kb][mb] = mfma(Aqt[mb][h], B, accK[kb][mb]);
                }
            }
        }
        RIB_FENCE();
        __syncthreads();
        const int r0 = c0;
        c0 = c1, c1 = c2, c2 = r0;
    }

    if (G > 1) {
        float *const part = (float *)smem + lane;
        if (grp > 0) {
            give_sums(accK, part + (wave - own) * sums_of<DQK, false>());
            give_sums(accV, part + (wave - own) * sums_of<DQK, false>() + 2 * L::RB * 1024);
        }
        __syncthreads();
        if (grp > 0) return;
#pragma unroll 1
        for (int j = 0; j < G - 1; ++j) {
            take_sums(accK, part + (wave + j * own) * sums_of<DQK, false>());
            take_sums(accV, part + (wave + j * own) * sums_of<DQK, false>() + 2 * L::RB * 1024);
        }
    }
    // (the streamed Q_aug rows carry scale * log2 e: undo the log2 e here)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const int n = n0 + kb * 32 + col;
        if (n < g.N) {
            const int64_t base = (img + win.any(n)) * g.C + hd * g.d;
            char *pd = (char *)(dfk_part + (u * g.N + n) * g.r);
#pragma unroll
            for (int mb = 0; mb < L::RB; ++mb) store_block(accK[kb][mb], mb, hf, g, kLn2, kLn2, (char *)(dk + base), pd);
            store_block(accV[kb], 0, hf, g, 1.f, 1.f, (char *)(dv + base), nullptr);
        }
    }
}

struct Args {
    const bf16_t *q, *k, *v, *fq, *fk, *out, *dout;
    const float *lse;
    float *delta;
    bf16_t *dq, *dk, *dv;
    float *pq, *pk;
    bf16_t *ftab;           // [heads][N][r]: scaled f_q rows, from the dq kernel (first window) to the dkv kernel
    hipStream_t st;
};

// Workgroups of `waves` waves, `nblk` of them per unit.
template <int DQK, int T, bool ALN, bool DQ, int G>
size_t lds_of(const Geo &g, int waves)
{
    const size_t tiles = Lay<DQK, T>::bytes(waves), sums = (size_t)(G - 1) * (waves / G) * sums_of<DQK, DQ>() * sizeof(float);
    return (tiles > sums ? tiles : sums) + (ALN ? 0 : (size_t)2 * g.M * sizeof(int));
}
template <int DQK, int T, bool XS, bool XD, bool ALN, int TINY, bool BIG, int NT = 256, int G = 1>
hipError_t launch_dkv(const Geo &g, int waves, int nblk, const Args &a)
{
    // (the map stands behind the tiles: sums that reach past them come after its last use)
    const size_t smem = lds_of<DQK, T, ALN, false, G>(g, waves);
    if (smem > (size_t)kMaxDynLds) return hipErrorInvalidValue;
    auto kern = dkv_kernel<DQK, T, XS, XD, ALN, TINY, BIG, NT, G>;
    const hipError_t e = prepare_kernel((const void *)kern, nullptr);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(g.units * nblk)), dim3(waves * 64), smem, a.st, g, nblk, a.q, a.k, a.v,
                       has_table(TINY) ? a.ftab : a.fq, a.fk, a.dout, a.lse,
                       a.delta, a.dk, a.dv, a.pk);
    return hipGetLastError();
}
template <int DQK, int T, bool XS, bool XD, bool ALN, int TINY, bool BIG, int NT = 256, int G = 1>
hipError_t launch_dq(const Geo &g, int waves, int nblk, const Args &a)
{
    const size_t smem = lds_of<DQK, T, ALN, true, G>(g, waves);
    if (smem > (size_t)kMaxDynLds) return hipErrorInvalidValue;
    auto kern = dq_kernel<DQK, T, XS, XD, ALN, TINY, BIG, NT, G>;
    const hipError_t e = prepare_kernel((const void *)kern, nullptr);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(g.units * nblk)), dim3(waves * 64), smem, a.st, g, nblk, a.q, a.k, a.v, a.fq, a.fk, a.out, a.dout,
                       a.lse, a.delta, a.dq, a.pq, a.ftab);
    return hipGetLastError();
}

// Whether the dkv kernel runs in workgroups of eight waves.  A lane then holds one 8-byte piece of each row instead of 16
// bytes, and it is the registers that count: with 64 columns the four-wave form spills 4 to 14 of them (us, four waves / eight,
// traced: 96 x 96 windows, r = 34 3089 / 2803, 64 x 64 2527 / 2282, 48 x 48, d = r = 32 537 / 512), with 48 and 32 none (64 x 64
// windows, r = 16 1067 / 1089, 32 x 32 410 / 435), and no second workgroup runs beside one's start and end.  So: 64 columns,
// grids of two rounds and more (fewer: a CU with four waves is faster than half the CUs with eight), and no more rounds
// than four waves take, which are counted one workgroup a CU: a last round of those that fills only one of a CU's two
// places costs about three quarters of one that fills both.  That is less than a round of eight waves, unless there are enough others
// to make up for it: four with the 7 % of aligned sides (five where the larger workgroups are not filled to nine tenths), eight with the 3 % of
// other sides.  (Backward, 6 heads, us, four / eight: 40 x 40, r = 34, 192 units, rounds of 6 and 3 451 / 442, 168 units, 5 and 3 387 / 406, 144 units, 4 and
// 3 327 / 376, 240 units, 7 and 4 552 / 566; 32 x 32, 288 units, 5 and 3 284 / 294; d = r = 32, 48 x 48, 192 units, 7 and 4 819 / 791, 56 x 56, 168 units, 9
// and 5 1356 / 1294; 45 x 45, r = 34, 216 units, 7 and 4 1049 / 1071.)
inline hipError_t eight_waves(const Geo &g, bool *yes)
{
    int cus = 0;
    const hipError_t e = compute_units(&cus);
    *yes = false;
    if (e != hipSuccess) return e;
    const int64_t nb = (g.N + 63) / 64, n8 = g.units * ((nb + 7) / 8), n4 = g.units * ((nb + 3) / 4);
    const int64_t r8 = (n8 + cus - 1) / cus, r4 = (n4 + cus - 1) / cus, enough = g.M % 8 != 0 ? 8 : (nb + 7) / 8 * 72 <= nb * 10 ? 4 : 5;
    *yes = n8 >= 2 * cus && 2 * r8 <= r4 + (r8 >= enough ? 1 : 0);
    return e;
}

// The pair: dq first, it writes the delta rows and the scaled RIB rows the dkv kernel streams.
template <int DQK, int T, bool XS, bool XD, bool ALN, int TINY, bool BIG>
hipError_t launch_pair(const Geo &g, int waves, int nblk, const Args &a)
{
    hipError_t e = launch_dq<DQK, T, XS, XD, ALN, TINY, BIG>(g, waves, nblk, a);
    if (e != hipSuccess) return e;
    if constexpr (DQK == 64 && T == 64 && (TINY == kLong || TINY == kLong8) && !BIG) {
        bool eight = false;
        if ((e = eight_waves(g, &eight)) != hipSuccess) return e;
        if (eight) return launch_dkv<DQK, 64, XS, XD, ALN, kLong8, false, 512>(g, 8, ((g.N + 63) / 64 + 7) / 8, a);
    }
    // With 64 columns and an aligned side dkv has fewer spills in 8-byte pieces (four waves 4 to 8 registers, with 16 bytes 8 to 12; three
    // waves with both extras in the C operand 13, 40) and is faster there (backward, 6 heads, d = r = 32, us, 8-byte / 16-byte: 40 x 40, 288 units 661 /
    // 675, 24 x 24, 672 units 327 / 353); three waves else spill alike and are slower (24 x 24, r = 34, 936 units 514 / 456), odd sides too (41 x 41, 264 units
    // 1013 / 993).
    constexpr bool less = DQK == 64 && ALN && TINY == kLong && (T == 64 || (XS && XD));
    return launch_dkv<DQK, T, XS, XD, ALN, less ? (int)kLong8 : TINY, BIG>(g, waves, nblk, a);
}

template <int DQK, bool XS, bool XD, int TINY>
hipError_t launch_rows(const Geo &g, bool aln, int waves, int nblk, const Args &a)
{
    if (aln)
        return waves == 4 ? launch_pair<DQK, 64, XS, XD, true, TINY, false>(g, waves, nblk, a)
                          : launch_pair<DQK, 32, XS, XD, true, TINY, false>(g, waves, nblk, a);
    return waves == 4 ? launch_pair<DQK, 64, XS, XD, false, TINY, false>(g, waves, nblk, a)
                      : launch_pair<DQK, 32, XS, XD, false, TINY, false>(g, waves, nblk, a);
}

// The pair on a small grid, whose workgroups of four waves would leave CUs empty or with a wave a SIMD: eight waves, G groups
// of which share the streamed side of 8 / G waves' stationary tokens; tiles of 32 G tokens, a block for each group.
template <int DQK, bool XS, bool XD, bool ALN, int G>
hipError_t launch_groups(const Geo &g, const Args &a)
{
    const int own = 8 / G, nblk = ((g.N + 63) / 64 + own - 1) / own;
    const hipError_t e = launch_dq<DQK, 32 * G, XS, XD, ALN, kLong8, false, 512, G>(g, 8, nblk, a);
    return e != hipSuccess ? e : launch_dkv<DQK, 32 * G, XS, XD, ALN, kLong8, false, 512, G>(g, 8, nblk, a);
}

// How many groups: where the grid is one round of the chip, four from 1024 tokens up, two else.  Backward, us, without / 2 / 4
// groups: one 96 x 96 window, d = 30, r = 16 367 / 318 / 205, one 63 x 63 of 6 heads, d = r = 32 386 / 308 / 203, one 48 x 48 102 / 92 / 66,
// one 32 x 32 53 / 52 / 41, 8 of 4 heads 57 / 55 / 46, one 24 x 24 45 / 37 / 40; but one 40 x 40, d = r = 32 (half a tile of 128 left over) 102 / 86 / 90,
// one 25 x 25 53 / 51 / 40: the line at 1024 was drawn while the sums of four groups spilled, and is not the best one without.
inline hipError_t groups_of(const Geo &g, int *groups)
{
    int cus = 0;
    const hipError_t e = compute_units(&cus);
    const int nb = (g.N + 63) / 64;
    *groups = g.N >= 1024 && g.units * ((nb + 1) / 2) <= cus ? 4 : g.units * ((nb + 3) / 4) <= cus ? 2 : 1;
    return e;
}

// Which widths and extras rows of a kind meet (short rows beside d = 32, and RIB rows of under 8 values, need few columns; those of
// more than 32 values take 64).
constexpr bool reached(int kind, int dqk, bool xs, bool xd)
{
    return kind == kAnyShort ? !xd && !(dqk == 48 && xs)
           : kind == kPairRib ? dqk == 32 || (dqk == 48 && !xs && xd)
           : kind == kNoRib   ? !xs && (dqk == 32 || (dqk == 48 && xd))
           : kind == kLong8   ? !(dqk == 48 && xs) && !(dqk == 64 && xd) : true;
}

// Workgroup shape: up to 4 waves of 64 stationary tokens, an equal number in every workgroup of a
// unit; workgroups under 4 waves stream tiles of 32 tokens (a lane stages at most two).  Images whose
// offsets need more than 32 bits run the four-wave form with 64-bit offsets at every size.
template <int DQK, bool XS, bool XD>
hipError_t launch_width(const Geo &g, const Args &a)
{
    const int nb = (g.N + 63) / 64, nblk = (nb + 3) / 4;
    int waves = (nb + nblk - 1) / nblk;
    if (waves < 2) waves = 2;
    const Short kind = short_rows(g);
    const bool aln = g.M % 8 == 0;
    if (!rows_supported(g)) {
        if (kind == kLong || kind == kLong8)
            return aln ? launch_pair<DQK, 64, XS, XD, true, kLong8, true>(g, 4, nblk, a)
                       : launch_pair<DQK, 64, XS, XD, false, kLong8, true>(g, 4, nblk, a);
        if constexpr (reached(kAnyShort, DQK, XS, XD) || reached(kPairRib, DQK, XS, XD) || reached(kNoRib, DQK, XS, XD))
            return launch_pair<DQK, 64, XS, XD, false, kAnyShort, true>(g, 4, nblk, a);
    }
    if constexpr (reached(kAnyShort, DQK, XS, XD)) {
        if (kind == kAnyShort)
            return waves == 4 ? launch_pair<DQK, 64, XS, XD, false, kAnyShort, false>(g, waves, nblk, a)
                              : launch_pair<DQK, 32, XS, XD, false, kAnyShort, false>(g, waves, nblk, a);
    }
    if constexpr (reached(kPairRib, DQK, XS, XD)) {
        if (kind == kPairRib) return launch_rows<DQK, XS, XD, kPairRib>(g, aln, waves, nblk, a);
    }
    if constexpr (reached(kNoRib, DQK, XS, XD)) {
        if (kind == kNoRib) return launch_rows<DQK, XS, XD, kNoRib>(g, aln, waves, nblk, a);
    }
    if (kind != kLong && kind != kLong8) return hipErrorInvalidValue;
    int groups = 1;
    const hipError_t e = groups_of(g, &groups);
    if (e != hipSuccess) return e;
    // (scalar token arithmetic needs whole tiles)
    if (groups == 4) return aln && g.N % 128 == 0 ? launch_groups<DQK, XS, XD, true, 4>(g, a) : launch_groups<DQK, XS, XD, false, 4>(g, a);
    if (groups == 2) return aln ? launch_groups<DQK, XS, XD, true, 2>(g, a) : launch_groups<DQK, XS, XD, false, 2>(g, a);
    if constexpr (reached(kLong8, DQK, XS, XD)) {
        if (kind == kLong8) return launch_rows<DQK, XS, XD, kLong8>(g, aln, waves, nblk, a);
    }
    return kind == kLong ? launch_rows<DQK, XS, XD, kLong>(g, aln, waves, nblk, a) : hipErrorInvalidValue;
}

// d + r within the padded width; columns carry LSE / delta wherever two are free.
hipError_t launch32(const Geo &g, const Args &a);
hipError_t launch48(const Geo &g, const Args &a);
hipError_t launch64(const Geo &g, const Args &a);
template <int DQK>
hipError_t launch_flags(const Geo &g, const Args &a)
{
    const bool xs = g.d + g.r + 2 > DQK, xd = g.d + 2 > 32;
    if constexpr (DQK == 32) {
        return xs ? launch_width<DQK, true, false>(g, a) : launch_width<DQK, false, false>(g, a);
    } else {
        if (xd) return xs ? launch_width<DQK, true, true>(g, a) : launch_width<DQK, false, true>(g, a);
        return xs ? launch_width<DQK, true, false>(g, a) : launch_width<DQK, false, false>(g, a);
    }
}

}  // namespace bwd
}  // namespace rib

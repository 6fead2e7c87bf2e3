// RIB window attention, forward, bf16 matrix cores: the kernel for windows of any size (64 tokens or
// more) and for grids too small to keep the streaming kernel of rib_mfma_fwd.hip busy.  Operator:
// include/rib_attn.h (paper Sec. 2.2; Sec. 3.1 Eq. 5-6).
//
// A wave owns QB * 32 queries (MFMA B operands in registers), a workgroup up to 256 queries of one
// (window, head) unit, and the unit's keys stream through LDS as token rows (rib_rows.h): transposed
// scores S^T = K_aug Q_aug^T (a lane owns a query column), packed probabilities as B operand of
// O^T += V^T P^T, V^T read transposed from the V rows.  Where the head dimension leaves two free
// columns of V (d <= 30) they hold ones and rows 30 and 31 of O^T are the softmax denominator;
// d = 32 (SUM) adds the probabilities up in fp32 (16 additions a block, 7 to 14 % of the forward; bf16
// dot products of the packed pairs cost half of that, but sum rounded values).  Probabilities are
// rounded to bf16 (v_cvt_pk_bf16_f32, which issues like the byte-permute a truncation takes).
//
// What bounds it: the vector issue beside the MFMAs (32 x 32 windows: 51 vector instructions a 32x32 block, of
// which exp2 and packs are 24, the vector ALU busy half of the cycles, the matrix pipe 32 %, and 41 % of a wave's
// time a wait on its previous instruction), under 600 tokens the start and end of a workgroup.  Three waves a SIMD
// (168 registers) where the width allows, so that one workgroup's ends lie under another's loop; that
// and whole-row staging took (us, with the kernels that served these windows before / with this one):
// 144 tokens, 2304 units 70.6 / 32.7; 576 tokens, 768 units 125.6 / 66.0; 256 tokens, 3456 units
// 74.9 / 70.7, 96 units 11.6 / 8.2; 2304 tokens, 192 units, d = r = 32 230 / 222; 2025 tokens, 96 units 122 / 80.
//
// The stabiliser is optimistic: no running maximum, a range check of every denominator afterwards,
// and a second walk with the running maximum where a workgroup has a failing row.
#pragma once

#include "rib_rows.h"

namespace rib {
namespace fwd_rows {

using namespace rows;

struct Args {
    const bf16_t *q, *k, *v, *fq, *fk;
    bf16_t *out;
    float *lse;
    int force_max;
    hipStream_t st;
};

// Raw words of a wave's QB * 32 query rows, 64 / LANES rows a pass.
template <int DQK, int QB, int TINY>
struct QRows {
    static constexpr int P = QB * 32 / Moved<TINY>::ROWS;
    Words<TINY> x[P], fa[P], fb[DQK == 64 ? P : 1];
};
template <int DQK, int QB, bool ALN, int TINY>
__device__ __forceinline__ void q_request(QRows<DQK, QB, TINY> &r, const Geo &g, const Win &win, const Stream &s, int n0)
{
    using M = Moved<TINY>;
    const int lane = threadIdx.x & 63, l = lane / M::LANES;
    const Piece pc = piece_of<TINY>(g, lane % M::LANES);
#pragma unroll
    for (int p = 0; p < QRows<DQK, QB, TINY>::P; ++p) {
        // (a wave past the window's end repeats its last rows)
        const int nf = n0 + p * M::ROWS, nb = ALN && nf > win.last - (M::ROWS - 1) ? win.last - (M::ROWS - 1) : nf, n = nb + l;
        r.x[p] = get<TINY>(s.xb, token_offset<false>(win.token<ALN, M::ROWS>(nb, l), s.xs) + 4u * pc.dc, pc.c1);
        if (!pc.fnone) {
            const uint32_t fr = __umul24((uint32_t)(n < win.last ? n : win.last), s.frow);
            r.fa[p] = get<TINY>(s.fb, fr + 4u * pc.f0, pc.f1d);
            if (DQK == 64) r.fb[p] = get<TINY>(s.fb, fr + 4u * pc.f1, pc.f1d);
        }
    }
}
// Scale (Eq. 5, times log2 e), round to bf16 and read back as B operands through the wave's own LDS area.
template <int DQK, int QB, int TINY>
__device__ __forceinline__ void q_stage(const QRows<DQK, QB, TINY> &r, const Geo &g, bf16_t *W, bf16x8 (&Q)[QB][DQK / 16])
{
    constexpr int STR = Lay<DQK, 64>::XS;
    using M = Moved<TINY>;
    const float sc = g.scale_c * kLog2e, sp = g.scale_p * kLog2e;
    const int lane = threadIdx.x & 63, l = lane / M::LANES, col = lane & 31, hf = lane >> 5;
    const Piece pc = piece_of<TINY>(g, lane % M::LANES);
    if (lane < 32 * QB) {       // padding columns of row `lane`
        bf16_t *xr = W + lane * STR;
        for (int c = g.d + g.r; c < DQK; c += 2) *(uint32_t *)(xr + c) = 0u;
    }
    bf16_t *xr = W + l * STR + 2 * pc.dc, *fr = W + l * STR + g.d + 2 * pc.f0, *fr1 = W + l * STR + g.d + 2 * pc.f1;
#pragma unroll
    for (int p = 0; p < QRows<DQK, QB, TINY>::P; ++p) {
        put<TINY>(xr + p * M::ROWS * STR, scaled<TINY>(r.x[p], sc), pc.c1);
        if (!pc.fnone) {
            put<TINY>(fr + p * M::ROWS * STR, scaled<TINY>(r.fa[p], sp), pc.f1d);
            if (DQK == 64) put<TINY>(fr1 + p * M::ROWS * STR, scaled<TINY>(r.fb[p], sp), pc.f1d);
        }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int b = 0; b < QB; ++b) read_rows<DQK / 16>(Q[b], W + (b * 32 + col) * STR + 8 * hf);
}

template <int DQK, int T, int QB>
constexpr size_t lds_bytes(int waves)
{
    using L = Lay<DQK, T>;
    const size_t tiles = (size_t)L::NSTAGE * L::STAGE, stat = (size_t)waves * QB * 32 * L::XS;
    return (tiles > stat ? tiles : stat) * sizeof(bf16_t);
}
// The sum of a lane's 16 probabilities of a block, in fp32.
template <class V>
__device__ __forceinline__ float sum16(const V &p)
{
    const float a = (p[0] + p[1]) + (p[2] + p[3]), b = (p[4] + p[5]) + (p[6] + p[7]);
    const float c = (p[8] + p[9]) + (p[10] + p[11]), d = (p[12] + p[13]) + (p[14] + p[15]);
    return (a + b) + (c + d);
}
constexpr int max_threads(int T, int QB, int G) { return QB == 1 || G > 1 ? 512 : T == 64 ? 256 : 192; }

// One step is one 32x32 block s = (key block, query block): the score MFMAs of block s + 1 and the two
// PV products of block s - 1 ride between the exponentials and packs of block s, in an order pinned
// with scheduling fences (as in the streaming kernel).
//
// G > 1: groups of waves share the streamed side of `waves / G` waves' queries (as in the backward pair): group `grp` takes its
// block of every tile, and the sums, which have no stabiliser, are added through LDS.  The second walk is every wave's own.
template <int DQK, int T, int QB, bool SUM, bool ALN, int TINY, int G>
__global__ __launch_bounds__(max_threads(T, QB, G), DQK <= 48 && TINY != kAnyShort && G == 1 ? 3 : 2) void rows_fwd_kernel(
    Geo g, int nblk, int force_max, const bf16_t *__restrict__ q, const bf16_t *__restrict__ k, const bf16_t *__restrict__ v,
    const bf16_t *__restrict__ fq, const bf16_t *__restrict__ fk, bf16_t *__restrict__ out, float *__restrict__ lse)
{
    using L = Lay<DQK, T>;
    constexpr int NB = T / 32 / G, NS = QB * NB;            // key blocks of a tile: of this wave's group
    static_assert(NS % 2 == 0, "two score blocks alternate");
    extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
    const int nt = G > 1 ? 512 : T == 64 && QB == 2 ? 256 : (int)blockDim.x, waves = nt >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, col = lane & 31, hf = lane >> 5;

    // workgroups are dealt round-robin to the 8 XCDs: an XCD works on a contiguous range of (unit, block)
    const int wgs = gridDim.x, per = wgs >> 3, rem = wgs & 7, xcd = blockIdx.x & 7;
    const int logical = xcd * per + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);
    const int u = logical / nblk, blk = logical - u * nblk;
    const int w = u / g.heads, hd = u - w * g.heads;
    int b;
    const Win win = window_of<ALN>(g, w, nt, (int *)((char *)smem + lds_bytes<DQK, T, QB>(waves)), b);
    const int64_t img = (int64_t)b * g.H * g.W;
    Stream ks, qs;
    ks.xb = (const char *)(k + img * g.tstride + hd * g.d);
    ks.yb = (const char *)(v + img * g.tstride + hd * g.d);
    ks.fb = (const char *)(fk + (int64_t)hd * g.N * g.r);
    ks.xs = ks.ys = qs.xs = qs.ys = g.tstride * 2;
    ks.frow = qs.frow = (uint32_t)g.r * 2u;
    qs.xb = qs.yb = (const char *)(q + img * g.tstride + hd * g.d);
    qs.fb = (const char *)(fq + (int64_t)hd * g.N * g.r);
    ks.lse = ks.delta = qs.lse = qs.delta = nullptr;
    const int own = waves / G, grp = G == 1 ? 0 : wave / own, n0 = (blk * own + (G == 1 ? wave : wave % own)) * (QB * 32);
    const int g0 = G == 1 ? 0 : grp * 32 * NB;              // the group's first row of a tile
    const int ntiles = (g.N + T - 1) / T;
    if (!ALN) __syncthreads();

    // one exposed memory latency: the wave's rows and the first two tiles are requested together
    Regs<DQK, TINY> rg, rg1;
    bf16x8 Qb[QB][L::KS];
    {
        QRows<DQK, QB, TINY> qr;
        q_request<DQK, QB, ALN, TINY>(qr, g, win, qs, n0);
        request<DQK, T, false, ALN, TINY, false>(rg, g, win, ks, 0, nt, wave);
        request<DQK, T, false, ALN, TINY, false>(rg1, g, win, ks, ntiles > 1 ? 1 : 0, nt, wave);
        q_stage<DQK, QB, TINY>(qr, g, smem + wave * (QB * 32 * L::XS), Qb);
    }
    __syncthreads();
    init_pads<DQK, T, false, true, SUM>(g, smem, nt);
    commit<DQK, T, false, true, SUM, ALN, TINY>(rg, g, smem, 1.f, 1.f, g.N, nt, wave);
    commit<DQK, T, false, true, SUM, ALN, TINY>(rg1, g, smem + L::STAGE, 1.f, 1.f, ntiles > 1 ? g.N - T : g.N, nt, wave);
    request<DQK, T, false, ALN, TINY, false>(rg, g, win, ks, ntiles > 2 ? 2 : ntiles - 1, nt, wave);
    __syncthreads();

    f32x16 O[QB];
    float lsum[QB], mrun[QB], den[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
        for (int i = 0; i < 16; ++i) O[qb][i] = 0.f;
        lsum[qb] = 0.f;
        mrun[qb] = 0.f;         // what LSE adds to the denominator's log2
    }
    const int tro = L::YR + tr_lane_offset<L::YS>(lane), ako = col * L::XS + 8 * hf, tro_g = tro + g0 * L::YS, ako_g = ako + g0 * L::XS;
    const f32x16 z = {0};
    // denominators: row 30 of O^T is register 14 of the upper lane half
    auto denominators = [&]() {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float mine = SUM ? lsum[qb] : O[qb][14], other = __shfl_xor(mine, 32);
            den[qb] = SUM ? mine + other : hf ? mine : other;
        }
    };
    bool bad = true;
    if (!force_max) {
        bf16x8 Ak[L::KS], At[2];
        f32x16 S[2];
        uint32_t P[2][8];
        read_rows<L::KS>(Ak, smem + ako_g);
        S[0] = mfma(Ak[0], Qb[0][0], z);
#pragma unroll
        for (int i = 1; i < L::KS; ++i) S[0] = mfma(Ak[i], Qb[0][i], S[0]);
        At[0] = At[1] = as_bf16x8(0u, 0u, 0u, 0u);      // (the first step's PV products add zero)
        if (QB == 1) read_rows<L::KS>(Ak, smem + 32 * L::XS + ako_g);
#pragma unroll
        for (int i = 0; i < 8; ++i) P[1][i] = 0u;
        int c0 = 0, c1 = L::STAGE, c2 = 2 * L::STAGE;    // this tile's, the next tile's and the free stage
        for (int tile = 0; tile < ntiles; ++tile) {
            const bf16_t *cur = smem + c0, *nxt = smem + c1;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int kb = s / QB, qb = s % QB, cs = s & 1, ns = cs ^ 1, qn = QB == 1 ? 0 : qb ^ 1;
                const bool turn = qb == 0;      // the step in which a key block's operands change hands
                float p[16];
                RIB_FENCE();
                S[ns] = mfma(Ak[0], Qb[qn][0], z);
                if (!ALN && tile == ntiles - 1) mask_rows(S[cs], tile * T + g0 + kb * 32, g.N, hf);
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(S[cs][i]);
                P[cs][0] = pack_bf16(p[0], p[1]);
                P[cs][1] = pack_bf16(p[2], p[3]);
                RIB_FENCE();
                S[ns] = mfma(Ak[1], Qb[qn][1], S[ns]);
#pragma unroll
                for (int i = 4; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(S[cs][i]);
                P[cs][2] = pack_bf16(p[4], p[5]);
                P[cs][3] = pack_bf16(p[6], p[7]);
                if (s == 0) commit<DQK, T, false, true, SUM, ALN, TINY>(rg, g, smem + c2, 1.f, 1.f, rows_left<T>(g, tile + 2), nt, wave);
                RIB_FENCE();
#pragma unroll
                for (int i = 2; i < L::KS; ++i) S[ns] = mfma(Ak[i], Qb[qn][i], S[ns]);
#pragma unroll
                for (int i = 8; i < 12; ++i) p[i] = __builtin_amdgcn_exp2f(S[cs][i]);
                P[cs][4] = pack_bf16(p[8], p[9]);
                P[cs][5] = pack_bf16(p[10], p[11]);
                if (turn) {     // K of the next key block (QB = 1: of the one after it)
                    const int kn = kb + (QB == 1 ? 2 : 1);
                    read_rows<L::KS>(Ak, (kn < NB ? cur + kn * 32 * L::XS : nxt + (kn - NB) * 32 * L::XS) + ako_g);
                }
                RIB_FENCE();
                O[qn] = mfma(At[0], as_bf16x8(P[ns][0], P[ns][1], P[ns][2], P[ns][3]), O[qn]);
#pragma unroll
                for (int i = 12; i < 16; ++i) p[i] = __builtin_amdgcn_exp2f(S[cs][i]);
                P[cs][6] = pack_bf16(p[12], p[13]);
                P[cs][7] = pack_bf16(p[14], p[15]);
                RIB_FENCE();
                O[qn] = mfma(At[1], as_bf16x8(P[ns][4], P[ns][5], P[ns][6], P[ns][7]), O[qn]);
                if (SUM) lsum[qb] += sum16(p);
                RIB_FENCE();
                if (turn) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) At[i] = read_tr<L::YS>(cur + (kb * 32 + 16 * i) * L::YS, tro_g, 0);
                }
                if (s == NS - 1) request<DQK, T, false, ALN, TINY, false>(rg, g, win, ks, tile + 3 < ntiles ? tile + 3 : ntiles - 1, nt, wave);
            }
            RIB_FENCE();
            __syncthreads();
            const int r0 = c0;
            c0 = c1, c1 = c2, c2 = r0;
        }
        O[QB - 1] = mfma(At[0], as_bf16x8(P[1][0], P[1][1], P[1][2], P[1][3]), O[QB - 1]);
        O[QB - 1] = mfma(At[1], as_bf16x8(P[1][4], P[1][5], P[1][6], P[1][7]), O[QB - 1]);
        if constexpr (G > 1) {
            // [wave][QB][17][64], behind the tiles and the map: a second walk needs the tiles' padding columns as they are
            float *const part = (float *)((char *)smem + lds_bytes<DQK, T, QB>(waves) + (ALN ? 0 : (size_t)8 * g.M)) + lane;
            if (grp > 0) {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    float *const p = part + ((wave - own) * QB + qb) * 17 * 64;
#pragma unroll
                    for (int i = 0; i < 16; ++i) p[i * 64] = O[qb][i];
                    if (SUM) p[16 * 64] = lsum[qb];
                }
            }
            __syncthreads();
            if (grp == 0) {
                for (int j = 0; j < G - 1; ++j)
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) {
                        const float *const p = part + ((wave + j * own) * QB + qb) * 17 * 64;
#pragma unroll
                        for (int i = 0; i < 16; ++i) O[qb][i] += p[i * 64];
                        if (SUM) lsum[qb] += p[16 * 64];
                    }
            }
        }
        denominators();
        bad = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
            if (grp == 0 && !((den[qb] >= 0x1p-60f) && (den[qb] <= 0x1p60f))) bad = true;
    }
    // Cold path: the walk again with a running maximum, one key block at a time.  (Rows past the
    // window's end repeat its last row, so they ask for it only if that row does.)
    if (__syncthreads_or(bad)) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
            for (int i = 0; i < 16; ++i) O[qb][i] = 0.f;
            lsum[qb] = 0.f;
            mrun[qb] = -INFINITY;
        }
        request<DQK, T, false, ALN, TINY, false>(rg, g, win, ks, 0, nt, wave);
#pragma unroll 1
        for (int tile = 0; tile < ntiles; ++tile) {     // two stages in turn, one barrier a tile
            bf16_t *cur = smem + (tile & 1) * L::STAGE;
            commit<DQK, T, false, true, SUM, ALN, TINY>(rg, g, cur, 1.f, 1.f, g.N - tile * T, nt, wave);
            request<DQK, T, false, ALN, TINY, false>(rg, g, win, ks, tile + 1 < ntiles ? tile + 1 : tile, nt, wave);
            __syncthreads();
#pragma unroll 1
            for (int kb = 0; kb < T / 32; ++kb) {
                const int key0 = tile * T + kb * 32;
                if (key0 >= g.N) break;
                bf16x8 Ak[L::KS], At[2];
                read_rows<L::KS>(Ak, cur + kb * 32 * L::XS + ako);
#pragma unroll
                for (int i = 0; i < 2; ++i) At[i] = read_tr<L::YS>(cur + (kb * 32 + 16 * i) * L::YS, tro, 0);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    f32x16 S = mfma(Ak[0], Qb[qb][0], z);
#pragma unroll
                    for (int i = 1; i < L::KS; ++i) S = mfma(Ak[i], Qb[qb][i], S);
                    if (!ALN) mask_rows(S, key0, g.N, hf);
                    float m = S[0];
#pragma unroll
                    for (int i = 1; i < 16; ++i) m = fmaxf(m, S[i]);
                    m = fmaxf(mrun[qb], fmaxf(m, __shfl_xor(m, 32)));
                    // (a row of minus infinities so far: any finite stabiliser does)
                    const float ms = m == -INFINITY ? 0.f : m, alpha = __builtin_amdgcn_exp2f(mrun[qb] - ms);
                    mrun[qb] = m;
                    uint32_t P[8];
                    lsum[qb] *= alpha;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        S[i] = __builtin_amdgcn_exp2f(S[i] - ms);
                        O[qb][i] *= alpha;
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) P[i] = pack_bf16(S[2 * i], S[2 * i + 1]);
                    if (SUM) lsum[qb] += sum16(S);
                    O[qb] = mfma(At[0], as_bf16x8(P[0], P[1], P[2], P[3]), O[qb]);
                    O[qb] = mfma(At[1], as_bf16x8(P[4], P[5], P[6], P[7]), O[qb]);
                }
            }
        }
        denominators();
    }

    if (G > 1 && grp > 0) return;
    // Normalise and store straight from the accumulator layout: a lane holds, for one token, four groups of
    // four consecutive channels.
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int n = n0 + qb * 32 + col;
        if (n >= g.N) continue;
        // byte offset of this lane's piece inside the image (fits 32 bits: checked on the host)
        const uint32_t obase = (win.any(n) * (uint32_t)g.C + (uint32_t)(hd * g.d + 4 * hf)) * 2u;
        char *ob = (char *)(out + img * g.C);
        const char *gb = (const char *)g.gate + img * g.C * 2;
        char *rb = g.out_raw ? (char *)g.out_raw + img * g.C * 2 : nullptr;
        const float inv = 1.f / den[qb];
        if (lse != nullptr && hf == 0)
            lse[(int64_t)u * g.N + n] = (mrun[qb] + __builtin_amdgcn_logf(den[qb])) * kLn2;
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) {
            const int left = g.d - (8 * c4 + 4 * hf);           // channels of this group inside the head
            const uint32_t off = obase + 16u * c4;
            dword2 w2;
            w2.x = pack_bf16(O[qb][4 * c4] * inv, O[qb][4 * c4 + 1] * inv);
            w2.y = pack_bf16(O[qb][4 * c4 + 2] * inv, O[qb][4 * c4 + 3] * inv);
            if (left < 2) continue;
            dword2 wo = w2;
            if (g.gate != nullptr) {    // CLA gate (Eq. 9) on the way out, the raw O beside it if asked for
                const dword2 gw = get8(gb, off, left < 4);
                wo.x = pack_bf16(lo_bf16(w2.x) * lo_bf16(gw.x), hi_bf16(w2.x) * hi_bf16(gw.x));
                wo.y = pack_bf16(lo_bf16(w2.y) * lo_bf16(gw.y), hi_bf16(w2.y) * hi_bf16(gw.y));
                if (rb) put8((bf16_t *)(rb + off), w2, left < 4);
            }
            put8((bf16_t *)(ob + off), wo, left < 4);
        }
    }
}

template <int DQK, int T, int QB, bool SUM, bool ALN, int TINY, int G = 1>
hipError_t launch_one(const Geo &g, int waves, int nblk, const Args &a)
{
    const size_t smem = lds_bytes<DQK, T, QB>(waves) + (ALN ? 0 : (size_t)2 * g.M * sizeof(int)) +
                        (size_t)(G - 1) * (waves / G) * QB * 17 * 64 * sizeof(float);
    if (smem > (size_t)kMaxDynLds) return hipErrorInvalidValue;
    auto kern = rows_fwd_kernel<DQK, T, QB, SUM, ALN, TINY, G>;
    const hipError_t e = prepare_kernel((const void *)kern, nullptr);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(g.units * nblk)), dim3(waves * 64), smem, a.st, g, nblk, a.force_max, a.q, a.k, a.v,
                       a.fq, a.fk, a.out, a.lse);
    return hipGetLastError();
}

template <int DQK, bool SUM, int TINY>
hipError_t launch_queries64(const Geo &g, bool aln, int waves, int nblk, const Args &a)
{
    if (aln)
        return waves == 4 ? launch_one<DQK, 64, 2, SUM, true, TINY>(g, waves, nblk, a)
                          : launch_one<DQK, 32, 2, SUM, true, TINY>(g, waves, nblk, a);
    return waves == 4 ? launch_one<DQK, 64, 2, SUM, false, TINY>(g, waves, nblk, a)
                      : launch_one<DQK, 32, 2, SUM, false, TINY>(g, waves, nblk, a);
}

// Workgroup shape.  64 queries a wave (half the operand reads per product): up to 4 waves, an equal
// number in every workgroup of a unit; workgroups under 4 waves stream tiles of 32 tokens (a lane
// stages at most two).  32 queries a wave, up to 8 waves, are for grids that leave SIMDs idle: half
// the work per wave and a second wave on each SIMD.
template <int DQK, bool SUM>
hipError_t launch_width(const Geo &g, int qb, const Args &a)
{
    const Short kind = short_rows(g);
    const bool aln = g.M % 8 == 0;
    constexpr bool short8 = !(DQK == 64 && SUM);    // (RIB rows of 4 or 6 values beside d = 32 fit 48 columns)
    if (g.N >= 1024 && (kind == kLong || kind == kLong8)) {
        int cus = 0;
        const hipError_t e = compute_units(&cus);
        if (e != hipSuccess) return e;
        // Four groups of two waves where that grid is one round of the chip and a wave's walk is long beside the sums at its end
        // (us, 32 queries a wave / groups: one 96 x 96 window, d = r = 32 136 / 81, of 2 heads, r = 34 115 / 82, one 64 x 64 of 6 heads 50 / 35, one
        // 48 x 48 of 4 heads 29.7 / 22.8, one 32 x 32 of 2 heads 15.9 / 14.3; one 24 x 24 of 2 heads 12.1 / 13.4, 128 units of 144 tokens 10.4 / 11.2).
        // (Scalar token arithmetic needs whole tiles.)
        const int nblk = (g.N + 127) / 128;
        if (g.units * nblk <= cus)
            return aln && g.N % 128 == 0 ? launch_one<DQK, 128, 2, SUM, true, kLong8, 4>(g, 8, nblk, a)
                                         : launch_one<DQK, 128, 2, SUM, false, kLong8, 4>(g, 8, nblk, a);
    }
    if (qb == 1 && (kind == kLong || kind == kLong8)) {
        const int nb = (g.N + 31) / 32, nblk = (nb + 7) / 8;
        int waves = (nb + nblk - 1) / nblk;
        if (waves < 4) waves = 4;
        if constexpr (short8) {
            if (kind == kLong8)
                return aln ? launch_one<DQK, 64, 1, SUM, true, kLong8>(g, waves, nblk, a)
                           : launch_one<DQK, 64, 1, SUM, false, kLong8>(g, waves, nblk, a);
        }
        return aln ? launch_one<DQK, 64, 1, SUM, true, kLong>(g, waves, nblk, a)
                   : launch_one<DQK, 64, 1, SUM, false, kLong>(g, waves, nblk, a);
    }
    const int nb = (g.N + 63) / 64, nblk = (nb + 3) / 4;
    int waves = (nb + nblk - 1) / nblk;
    if (waves < 2) waves = 2;
    if constexpr (!SUM) {       // (d = 2)
        if (kind == kAnyShort)
            return waves == 4 ? launch_one<DQK, 64, 2, SUM, false, kAnyShort>(g, waves, nblk, a)
                              : launch_one<DQK, 32, 2, SUM, false, kAnyShort>(g, waves, nblk, a);
    }
    // (short RIB rows beside d >= 4: d + r <= 32, or d = 32)
    if constexpr (DQK == 32 || (DQK == 48 && SUM)) {
        if (kind == kPairRib) return launch_queries64<DQK, SUM, kPairRib>(g, aln, waves, nblk, a);
        if (kind == kNoRib) return launch_queries64<DQK, SUM, kNoRib>(g, aln, waves, nblk, a);
    }
    if constexpr (short8) {
        if (kind == kLong8) return launch_queries64<DQK, SUM, kLong8>(g, aln, waves, nblk, a);
    }
    if (kind != kLong) return hipErrorInvalidValue;
    return launch_queries64<DQK, SUM, kLong>(g, aln, waves, nblk, a);
}

hipError_t launch32(const Geo &g, int qb, const Args &a);
hipError_t launch48(const Geo &g, int qb, const Args &a);
hipError_t launch64(const Geo &g, int qb, const Args &a);
template <int DQK>
hipError_t launch_flags(const Geo &g, int qb, const Args &a)
{
    if constexpr (DQK > 32) {
        if (g.d + 2 > 32) return launch_width<DQK, true>(g, qb, a);
    }
    return launch_width<DQK, false>(g, qb, a);
}

}  // namespace fwd_rows
}  // namespace rib

// What the bf16 matrix-core kernels that stream token rows share (both backward kernels and the
// forward kernel for windows of any size): operand types, the LDS image of a streamed tile, the
// window map, and the staging of a tile from the grid tensors into that image.
//
// A streamed tile lies in LDS as plain token rows, written as 16-byte pieces by 4 lanes a token (8 bytes, 8 lanes: rows of under 8 values, workgroups of
// eight waves in which all stage, kernels whose registers 16 bytes would spill); the
// operands of products that contract over tokens are read TRANSPOSED from the same rows
// (ds_read_b64_tr_b16).  A last partial tile repeats the window's last token, with zeros in place of its
// V / dO, and the kernels mask its rows of the scores.
#pragma once

#include "rib_common.h"

namespace rib {
namespace rows {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    bf16x2 v;
    v[0] = (__bf16)a;
    v[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t scale_pair(uint32_t w, float s) { return pack_bf16(lo_bf16(w) * s, hi_bf16(w) * s); }
// x as a bf16 pair (hi, lo) with hi + lo == x to ~2^-17 relative
__device__ __forceinline__ uint32_t split_bf16(float x)
{
    bf16x2 v;
    v[0] = (__bf16)x;
    v[1] = (__bf16)(x - (float)v[0]);
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint32_t trunc_pack(float lo, float hi)
{
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
__device__ __forceinline__ bf16x8 as_bf16x8(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    uint4 w = {a, b, c, d};
    return __builtin_bit_cast(bf16x8, w);
}
__device__ __forceinline__ f32x16 mfma(const bf16x8 &a, const bf16x8 &b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// The thread id as a value the optimiser cannot trace back: lane constants derived from it are
// recomputed where they are used instead of being held in registers across the MFMA blocks.
__device__ __forceinline__ int opaque_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Two dwords at a 4-byte aligned address.
struct __attribute__((packed, aligned(4))) dword2 {
    uint32_t x, y;
};
struct __attribute__((packed, aligned(4))) float2u {
    float x, y;
};
struct __attribute__((packed, aligned(4))) float4u {
    float x, y, z, w;
};

// A operand of a product that contracts over tokens: 32 columns starting at `c0` (a lane's row is
// column c0 + lane % 32) of 16 tokens starting at row image `rows`, in the order the 32x32
// accumulator layout hands its rows to the next MFMA (tokens 4*hf + 0..3, then 8 + 4*hf + 0..3).
// ds_read_b64_tr_b16 transposes 4 rows x 16 columns per group of 16 lanes: lane a of the group
// names row a / 4, columns 4 * (a % 4) .. + 3, and receives column a of the four rows.
// `lane_off` = tr_lane_offset<STRIDE>().
template <int STRIDE>
__device__ __forceinline__ int tr_lane_offset(int lane)
{
    const int a = lane & 15, chalf = (lane >> 4) & 1, hf = lane >> 5;
    return (4 * hf + (a >> 2)) * STRIDE + 16 * chalf + 4 * (a & 3);
}
typedef s16x4 __attribute__((address_space(3))) *lds_s16x4;
template <int STRIDE>
__device__ __forceinline__ bf16x8 read_tr(const bf16_t *rows, int lane_off, int c0)
{
    union {
        s16x4 h[2];
        bf16x8 v;
    } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(rows + lane_off + c0));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(rows + lane_off + c0 + 8 * STRIDE));
    return u.v;
}
template <int N>
__device__ __forceinline__ void read_rows(bf16x8 (&dst)[N], const bf16_t *base)
{
#pragma unroll
    for (int t = 0; t < N; ++t) dst[t] = *(const bf16x8 *)(base + 16 * t);
}

// LDS image of one streamed tile of T tokens: X = augmented rows (content | RIB | zero pad | two
// extra columns), Y = value-like rows (content | zero pad | two extra columns), then (XS / XD) the
// tile's -LSE*log2(e) and -delta as floats.  Strides are odd multiples of 16 bytes (conflict-free
// 16-byte reads).  Three stages rotate: while a tile is multiplied, the next one is complete (its
// first operands are read ahead of the barrier) and the one after it is being written.
template <int DQK, int T>
struct Lay {
    static constexpr int DVK = 32;
    static constexpr int XS = DQK + 8, YS = DVK + 8;
    static constexpr int YR = T * XS, EX = YR + T * YS;
    static constexpr int STAGE = EX + 4 * T;                        // bf16 elements
    static constexpr int KS = DQK / 16, VS = DVK / 16;
    static constexpr int RB = (DQK + 31) / 32;                      // 32-row blocks of dQ_aug^T / dK_aug^T
    static constexpr int NSTAGE = 3;
    static constexpr int WAVE_STAT = 64 * (XS + YS);                // one wave's stationary rows (before the first tile)
    static constexpr size_t bytes(int waves)
    {
        return (size_t)(NSTAGE * STAGE > waves * WAVE_STAT ? NSTAGE * STAGE : waves * WAVE_STAT) * sizeof(bf16_t);
    }
};

// A window of one image: where its tokens lie, relative to the image's first token.  ALN (window
// side a multiple of 8): eight consecutive tokens lie in one window row, so a wave's row is scalar
// arithmetic and a lane adds its column (wrapped once at the image edge).  Otherwise the separable
// map in LDS (row bases, then wrapped columns), with lookups clamped to the window's last token.
struct Win {
    const int *rowb, *colo;
    uint32_t inv_m;
    int M, last, y0, x0, H, W;
    // `n0`: the wave's first token (uniform), this lane's token is n0 + l; l < 8, or l < 16 (ROWS): two runs of eight
    template <bool ALN, int ROWS = 8>
    __device__ __forceinline__ uint32_t token(int n0, int l) const
    {
        if (ALN && ROWS == 16) {
            const int iy0 = (int)__umulhi((uint32_t)n0, inv_m), iy1 = (int)__umulhi((uint32_t)(n0 + 8), inv_m);
            const int ya = y0 + iy0 >= H ? y0 + iy0 - H : y0 + iy0, yb = y0 + iy1 >= H ? y0 + iy1 - H : y0 + iy1;
            const bool second = l >= 8;
            const uint32_t x = (uint32_t)(x0 + n0) - (uint32_t)(second ? iy1 * M : iy0 * M) + (uint32_t)l, xw = x - (uint32_t)W;
            return (x < xw ? x : xw) + (uint32_t)(second ? yb * W : ya * W);
        }
        if (ALN) {
            const int iy = (int)__umulhi((uint32_t)n0, inv_m);
            int y = y0 + iy;
            if (y >= H) y -= H;
            const uint32_t x = (uint32_t)(x0 + n0 - iy * M) + (uint32_t)l, xw = x - (uint32_t)W;
            return (x < xw ? x : xw) + (uint32_t)(y * W);
        }
        const int n = n0 + l, nc = n < last ? n : last;
        const int iy = (int)__umulhi((uint32_t)nc, inv_m);
        return (uint32_t)(rowb[iy] + colo[nc - __mul24(iy, M)]);
    }
    // any token (per lane)
    __device__ __forceinline__ uint32_t any(int n) const
    {
        const int iy = (int)__umulhi((uint32_t)n, inv_m);
        int y = y0 + iy;
        if (y >= H) y -= H;
        int x = x0 + n - __mul24(iy, M);
        if (x >= W) x -= W;
        return (uint32_t)(y * W + x);
    }
};
template <bool ALN>
__device__ __forceinline__ Win window_of(const Geo &g, int w, int nt, int *lds, int &b)
{
    const int wx = w % g.nwx, t = w / g.nwx, wy = t % g.nwy;
    b = t / g.nwy;
    Win m;
    m.y0 = wy * g.M + g.s, m.x0 = wx * g.M + g.s;
    m.rowb = lds, m.colo = lds + g.M;
    m.inv_m = g.inv_m, m.M = g.M, m.last = g.N - 1, m.H = g.H, m.W = g.W;
    if (!ALN) {
        for (int i = threadIdx.x; i < 2 * g.M; i += nt) {
            if (i < g.M) {
                const int y = m.y0 + i;
                lds[i] = (y >= g.H ? y - g.H : y) * g.W;
            } else {
                const int x = m.x0 + i - g.M;
                lds[i] = x >= g.W ? x - g.W : x;
            }
        }
    }
    return m;
}

// Workgroups are dealt round-robin to the 8 XCDs; renumber them so that each XCD works on a
// contiguous range of (unit, block) and its L2 sees all users of a window's lines.
__device__ __forceinline__ void block_coords(int nblk, int64_t &u, int &blk)
{
    const int G = gridDim.x, per = G >> 3, rem = G & 7, xcd = blockIdx.x & 7;
    const int logical = xcd * per + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);
    u = logical / nblk;
    blk = logical - (int)(u * nblk);
}

// What a lane moves: 4 lanes share a token, 16 bytes each: dwords 4j .. 4j+3 of the content row and of the RIB row (a second
// piece for RIB rows longer than 32 values).  Lanes past the end slide back onto the last four (they duplicate a
// neighbour).  Rows of less than 8 values are moved by 8 lanes, 8 bytes each; rows of a single dword (d = 2, r = 2)
// move alone.  Both widths fill L1 at the same rate (64 rows of 60 bytes: 114 and 118 ns a CU), but 16 bytes a lane halve the
// address arithmetic and the memory instructions, which ride on the vector issue beside the MFMAs (8 / 4 lanes, us: forward
// + backward of 8 images of 96 x 96, 24 x 24 windows, r = 18 361 / 335, 16 images, 32 x 32, r = 16 836 / 815; forward of 4 images of 96 x
// 144, 12 x 12 37 / 35).
// Which rows are that short is compiled in: a branch in the staging code splits the pinned order of the
// blocks it rides in (forward and backward of 8 images of 96 x 96, 6 heads, d = 30, r = 2, us with branches /
// without: 32 x 32 windows 601 / 369, 16 x 16 299 / 186, 24 x 24 594 / 337; r = 0, 32 x 32: 464 / 343).
enum Short { kLong = 0, kPairRib = 1, kNoRib = 2, kAnyShort = 3, kLong8 = 4 };  // d, r >= 8 | d >= 4: r = 2 | r = 0 | d = 2, any r (branches) | d, r >= 4
inline Short short_rows(const Geo &g)
{
    return g.d < 4 ? kAnyShort : g.r == 0 ? kNoRib : g.r < 4 ? kPairRib : g.d < 8 || g.r < 8 ? kLong8 : kLong;
}
template <int TINY>
struct Moved {
    static constexpr int LANES = TINY == kLong ? 4 : 8;         // lanes a token
    static constexpr int ROWS = 64 / LANES;                     // tokens an instruction
    static constexpr int WORDS = 16 / LANES;                    // dwords a lane
    static constexpr int SLOTS = LANES == 4 ? 1 : 2;            // tokens a lane moves of a streamed tile
    struct __attribute__((packed, aligned(4))) Words {
        uint32_t w[WORDS];
    };
};
template <int TINY>
using Words = typename Moved<TINY>::Words;
// Whether the backward's dq kernel writes the scaled RIB rows of Q_aug out for dkv to stream.  A row of one pair costs more to
// write and read back than to scale again (backward of 12 units of 9 x 9, d = 14, r = 2 19.3 us without / 20.0 with; d = 2, r = 34, 14 x 14 54.9 /
// 63.2, where the table is spilled registers too).
constexpr bool has_table(int tiny) { return tiny == kLong || tiny == kLong8; }
struct Piece {
    int dc, f0, f1;                 // first dword of the content / RIB pieces
    bool c1, f1d, fnone;            // single-dword content / RIB rows, no RIB at all (uniform)
};
template <int TINY>
__device__ __forceinline__ Piece piece_of(const Geo &g, int j)
{
    constexpr int WN = Moved<TINY>::WORDS;
    const int hp = g.d >> 1, rh = g.r >> 1;
    Piece p;
    p.c1 = TINY == kAnyShort && hp < 2;
    p.f1d = TINY == kPairRib || (TINY == kAnyShort && rh < 2);
    p.fnone = TINY == kNoRib || (TINY == kAnyShort && rh == 0);
    p.dc = p.c1 ? 0 : (WN * j < hp - WN ? WN * j : hp - WN);
    p.f0 = p.f1d ? 0 : (WN * j < rh - WN ? WN * j : rh - WN);
    p.f1 = p.f1d ? 0 : (16 + WN * j < rh - WN ? 16 + WN * j : rh - WN);
    return p;
}
template <class Off>
__device__ __forceinline__ dword2 get8(const char *base, Off off, bool one)
{
    dword2 v;
    if (one) v.x = *(const uint32_t *)(base + off), v.y = 0u;
    else v = *(const dword2 *)(base + off);
    return v;
}
__device__ __forceinline__ void put8(bf16_t *dst, const dword2 &v, bool one)
{
    if (one) *(uint32_t *)dst = v.x;
    else *(dword2 *)dst = v;
}
template <int TINY, class Off>
__device__ __forceinline__ Words<TINY> get(const char *base, Off off, bool one)
{
    Words<TINY> v;
    if constexpr (TINY == kAnyShort) {
        const dword2 x = get8(base, off, one);
        v.w[0] = x.x, v.w[1] = x.y;
    } else if (one) {
        v.w[0] = *(const uint32_t *)(base + off);
#pragma unroll
        for (int i = 1; i < Moved<TINY>::WORDS; ++i) v.w[i] = 0u;
    } else {
        v = *(const Words<TINY> *)(base + off);
    }
    return v;
}
template <int TINY>
__device__ __forceinline__ void put(bf16_t *dst, const Words<TINY> &v, bool one)
{
    if constexpr (TINY == kAnyShort) put8(dst, dword2{v.w[0], v.w[1]}, one);
    else if (one) *(uint32_t *)dst = v.w[0];
    else *(Words<TINY> *)dst = v;
}
template <int TINY>
__device__ __forceinline__ Words<TINY> scaled(Words<TINY> v, float s)
{
#pragma unroll
    for (int i = 0; i < Moved<TINY>::WORDS; ++i) v.w[i] = scale_pair(v.w[i], s);
    return v;
}

// Streamed operand pair of a unit.  QDO: X = q (strided; its RIB rows scaled already where there is a table), Y = dO (dense), extras = LSE, delta.
// Otherwise X = k, Y = v (both strided), extras = ones.
struct Stream {
    const char *xb, *yb, *fb;       // this image's and head's slices; this head's RIB table
    const float *lse, *delta;       // this unit's rows (QDO)
    int64_t xs, ys;                 // token strides in bytes
    uint32_t frow;                  // RIB row in bytes
};
// Byte offset of an image's token `t`: 32 bits and a 24-bit multiply (rows_supported), BIG in 64 bits.
template <bool BIG>
__device__ __forceinline__ auto token_offset(uint32_t t, int64_t stride)
{
    if constexpr (BIG) return (uint64_t)t * (uint64_t)stride;
    else return (uint32_t)__umul24(t, (uint32_t)stride);
}

// Whether pass `p` of a tile's staging has rows for the wave whose first slot is `slot`.  Where the number of lanes is a constant
// the pass is taken or left out as a whole, and no branch splits the blocks it rides in; elsewhere there is one comparison.
template <int TINY, int T>
__device__ __forceinline__ bool stages(int p, int nt, int slot)
{
    constexpr int slots = T * Moved<TINY>::LANES;
    if (__builtin_constant_p(nt) && nt * (p + 1) <= slots) return true;
    if (__builtin_constant_p(nt) && nt * p >= slots) return false;
    return slot < slots;
}

template <int DQK, int TINY>
struct Regs {
    static constexpr int S = Moved<TINY>::SLOTS;
    Words<TINY> x[S], y[S], fa[S], fb[DQK == 64 ? S : 1];
    float e0;
};

// Request tile `tile`: slots tid (and tid + NT) of the tile's T * LANES.
template <int DQK, int T, bool QDO, bool ALN, int TINY, bool BIG>
__device__ __forceinline__ void request(Regs<DQK, TINY> &rg, const Geo &g, const Win &win, const Stream &s, int tile, int nt, int wave)
{
    using M = Moved<TINY>;
    const int lane = opaque_tid() & 63, l = lane / M::LANES;
    const Piece pc = piece_of<TINY>(g, lane % M::LANES);
#pragma unroll
    for (int p = 0; p < M::SLOTS; ++p) {
        const int slot = p * nt + wave * 64;                // the wave's first slot
        if (stages<TINY, T>(p, nt, slot)) {
            const int n0 = tile * T + (int)((uint32_t)slot / M::LANES);
            const uint32_t t = win.token<ALN, M::ROWS>(n0, l);
            rg.x[p] = get<TINY>(s.xb, token_offset<BIG>(t, s.xs) + 4u * pc.dc, pc.c1);
            rg.y[p] = get<TINY>(s.yb, token_offset<BIG>(t, s.ys) + 4u * pc.dc, pc.c1);
            if (!pc.fnone) {
                const int n = n0 + l, nc = ALN ? n : (n < win.last ? n : win.last);
                const uint32_t fr = __umul24((uint32_t)nc, s.frow);
                rg.fa[p] = get<TINY>(s.fb, fr + 4u * pc.f0, pc.f1d);
                if (DQK == 64) rg.fb[p] = get<TINY>(s.fb, fr + 4u * pc.f1, pc.f1d);
            }
        }
    }
    if (QDO && wave < T / 32) {     // LSE by the lower, delta by the upper T of T / 32 waves' lanes
        const int tid = wave * 64 + lane, n = tile * T + (tid & (T - 1));
        rg.e0 = ((tid & T) ? s.delta : s.lse)[ALN ? n : (n < win.last ? n : win.last)];
    }
}

// Rows of tile `tile` (past the last one: of the last, which is staged in its place) inside the window.
template <int T>
__device__ __forceinline__ int rows_left(const Geo &g, int tile)
{
    const int left = g.N - tile * T;
    return left > 0 ? left : (g.N - 1) % T + 1;
}
// `sc`, `sp`: what Q content and, without a table of scaled rows, its RIB rows are multiplied by (QDO).  `left`: how many of the tile's rows lie inside the window.  The Y rows past it are zero, so that an
// infinity in the repeated last token does not meet the zero P of a masked row.
template <int DQK, int T, bool QDO, bool XS, bool XD, bool ALN, int TINY>
__device__ __forceinline__ void commit(const Regs<DQK, TINY> &rg, const Geo &g, bf16_t *S, float sc, float sp, int left, int nt, int wave)
{
    using L = Lay<DQK, T>;
    using M = Moved<TINY>;
    const int lane = opaque_tid() & 63, l = lane / M::LANES;
    const Piece pc = piece_of<TINY>(g, lane % M::LANES);
    bf16_t *xr = S + __mul24(l, L::XS) + 2 * pc.dc, *yr = S + L::YR + __mul24(l, L::YS) + 2 * pc.dc;
    bf16_t *fr = S + __mul24(l, L::XS) + g.d + 2 * pc.f0, *fr1 = S + __mul24(l, L::XS) + g.d + 2 * pc.f1;
    constexpr bool scale = QDO && !has_table(TINY);
#pragma unroll
    for (int p = 0; p < M::SLOTS; ++p) {
        const int slot = p * nt + wave * 64;
        if (stages<TINY, T>(p, nt, slot)) {
            const int r0 = (int)((uint32_t)slot / M::LANES);    // (uniform)
            Words<TINY> x = rg.x[p], y = rg.y[p], fa = rg.fa[p], fb = rg.fb[DQK == 64 ? p : 0];
            if (scale) {        // (ahead of the branches on short rows: behind them it is 30 spilled registers with 64 columns)
                x = scaled<TINY>(x, sc), fa = scaled<TINY>(fa, sp);
                if (DQK == 64) fb = scaled<TINY>(fb, sp);
            }
            if (!ALN && r0 + l >= left)
#pragma unroll
                for (int i = 0; i < M::WORDS; ++i) y.w[i] = 0u;
            put<TINY>(xr + r0 * L::XS, QDO && !scale ? scaled<TINY>(x, sc) : x, pc.c1);
            put<TINY>(yr + r0 * L::YS, y, pc.c1);
            if (!pc.fnone) {
                put<TINY>(fr + r0 * L::XS, fa, pc.f1d);
                if (DQK == 64) put<TINY>(fr1 + r0 * L::XS, fb, pc.f1d);
            }
        }
    }
    if (QDO && wave < T / 32) {
        const int tid = wave * 64 + lane, row = tid & (T - 1);
        const bool dl = (tid & T) != 0;
        const float v = dl ? -rg.e0 : -rg.e0 * kLog2e;
        const uint32_t pk = split_bf16(v);
        if (dl) {
            if (XD) ((float *)(S + L::EX))[T + row] = v;
            else *(uint32_t *)(S + L::YR + row * L::YS + L::DVK - 2) = pk;
        } else {
            if (XS) ((float *)(S + L::EX))[row] = v;
            else *(uint32_t *)(S + row * L::XS + DQK - 2) = pk;
        }
    }
}

// The columns no staging code writes, once for every row of every stage: zero padding (it meets
// the zero padding of the stationary operands, so it only has to be finite), and for K / V tiles
// the ones that LSE and delta meet.
template <int DQK, int T, bool QDO, bool XS, bool XD, int STAGES = Lay<DQK, T>::NSTAGE>
__device__ __forceinline__ void init_pads(const Geo &g, bf16_t *stages, int nt)
{
    using L = Lay<DQK, T>;
    for (int e = threadIdx.x; e < STAGES * T; e += nt) {
        bf16_t *xr = stages + (e / T) * L::STAGE + (e % T) * L::XS, *yr = stages + (e / T) * L::STAGE + L::YR + (e % T) * L::YS;
        for (int c = g.d + g.r; c < DQK; c += 2)
            if (c < DQK - 2 || XS) *(uint32_t *)(xr + c) = 0u;
            else if (!QDO) *(uint32_t *)(xr + c) = 0x3f803f80u;
        for (int c = g.d; c < L::DVK; c += 2)
            if (c < L::DVK - 2 || XD) *(uint32_t *)(yr + c) = 0u;
            else if (!QDO) *(uint32_t *)(yr + c) = 0x3f803f80u;
    }
}

// Rows of a score block whose streamed token lies past the window: minus infinity, so that P and
// dS vanish there.  (The staged rows repeat the last token's: what is not finite in one of them is
// not in the last token's own products either.)
__device__ __forceinline__ void mask_rows(f32x16 &S, int first, int N, int hf)
{
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (first + 8 * (i >> 2) + 4 * hf + (i & 3) >= N) S[i] = -INFINITY;
}

#define RIB_FENCE() __builtin_amdgcn_sched_barrier(0)

}  // namespace rows
}  // namespace rib

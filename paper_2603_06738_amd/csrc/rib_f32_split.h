// fp32 problems on the bf16 matrix cores, three bf16 parts to an fp32 value.
//
// x = x0 + x1 + x2 with x0 = bf16(x), x1 = bf16(x - x0), x2 = the rest: 8 + 8 + 8 bits and the signs
// hold all 24 of an fp32 significand.  A product of two such values is six bf16 products,
//   x0 y0 + (x0 y1 + x1 y0) + (x0 y2 + x1 y1 + x2 y0),
// exact in fp32 each.  What is left out (x1 y2 + x2 y1 + x2 y2) depends on how the parts are made.  Inputs
// have theirs rounded to nearest, so that the scores and dP lose at most 0.9 * 2^-24 of a product, as much
// as one fp32 multiplication.  P and dS are split by truncation: their products with V, dO, Q and K lose up
// to 2.5 * 2^-24, to either side.  (Truncated on both sides it would be 6.8 * 2^-24 and mostly to one;
// rounding P and dS too costs 3 %: 4 images of 32 x 32 windows, forward and backward, 1191 us / 1233.)
// The small ones are accumulated first.  v_mfma_f32_32x32x16_bf16 does 16 times
// the work of v_mfma_f32_32x32x2_f32 in half its time (32 clk against 64), so the six are 2.7 times
// faster than fp32 MFMAs, and unlike these they leave the vector ALU free.
//
// Everything else stays fp32: softmax state, P, dS, accumulators.  Inputs whose parts would leave
// the exponent range (2^32 and beyond, infinities; below 2^-100 the last part has fewer bits than it
// needs) are noticed while they are staged, and the workgroup then does its rows again with fp32 MFMAs
// (the *_body functions), whose arithmetic is defined for them.  P and dS are not checked: elements of
// theirs below 2^-110 go into their products with fewer than 24 bits.
//
// Layout: a wave owns 32 stationary tokens as B operands in registers, a workgroup of four to eight
// waves streams the other side through three LDS stages of 64 or 32 tokens: for each part the augmented rows
// [content, padded to even | RIB | zeros] and the value-like rows, which are also read transposed
// (rib_rows.h).  Splitting the streamed values is vector work that all waves of a workgroup share.
//
// What bounds them: the matrix pipe (31 / 55 / 67 MFMAs of 32 clk a 32x32 block in fwd / dq / dkv at 48
// columns: 37 / 43 / 40 % of the SIMD-cycles at 2.4 GHz by counters) and the vector ALU (301 / 371 / 499
// instructions a block, exponentials, splits and staging: 48 / 38 / 38 %), which hardly overlap; under 300
// tokens the start of a workgroup.  dkv spills (56 registers at 48 columns, 175 at 64).  Against the
// fp32-MFMA kernels (us, 96 x 96 images, 6 heads, d = 30, r = 16; before / after): 4 images of 32 x 32 windows
// forward 366 / 259, backward 1330 / 943; 8 images of 12 x 12 windows 266 / 169 and 1076 / 650.  Error against
// fp64 (2-norm, the 32 x 32 case): O 6.7e-7 / 2.8e-7, LSE 4.9e-8 / 2.5e-8, dQ 7.5e-7 / 4.0e-7, dK 7.6e-7 / 4.1e-7,
// dV 7.4e-7 / 4.0e-7.
// Measured and left out: the two waves of a SIMD half a block apart (no change), two LDS stages with two
// workgroups of four waves a CU (295 / 870 us when the three stages took 257 / 907), operands of the stationary
// side fetched element by element (ten microseconds more at a workgroup's start).
#pragma once

#include "rib_rows.h"

namespace rib {
namespace {
namespace split {

using rows::bf16x8;
using rows::as_bf16x8;
using rows::pack_bf16;
using rows::lo_bf16;
using rows::hi_bf16;
using rows::read_rows;
using rows::read_tr;
using rows::tr_lane_offset;
using rows::float2u;
using rows::float4u;

constexpr float kLimit = 0x1p32f;     // magnitudes the parts carry: below this,
constexpr int kSmallExp = 100;        // and 2^-kSmallExp or more (or zero)

// Offsets inside one image fit 32 bits and are built with a 24-bit multiply; both parts of an augmented row,
// padded to even lengths, fit its 64 columns and hold whole four-value pieces.
inline bool supported(const Geo &g)
{
    const int64_t pixels = (int64_t)g.H * g.W, stride = g.tstride > g.C ? g.tstride : (int64_t)g.C;
    return pixels < (1 << 24) && stride * 4 < (1 << 24) && pixels * stride * 4 < ((int64_t)1 << 32) &&
           g.N >= 64 && ((g.d + 1) & ~1) + ((g.r + 1) & ~1) <= 64 && g.d > 2 && (g.r == 0 || g.r > 2);
}
inline int width(const Geo &g)
{
    const int w = (((g.d + 1) & ~1) + ((g.r + 1) & ~1) + 15) / 16 * 16;
    return g.r > 32 ? 64 : w;               // (a second RIB slot per lane: 64 columns only)
}

template <int DA, int T>
struct Lay {
    static constexpr int XS = DA + 8, YS = 40, KS = DA / 16, RB = (DA + 31) / 32;
    static constexpr int XP = T * XS, YP = T * YS;        // one part of a stage
    static constexpr int YR = 3 * XP, EX = YR + 3 * YP;
    static constexpr int STAGE = EX + 4 * T;                // bf16 elements (LSE and delta rows as floats)
    static constexpr size_t BYTES = (size_t)3 * STAGE * sizeof(bf16_t);
};

// One wave's area for its stationary rows.
template <int DA>
constexpr int stat_elems() { return 3 * 32 * (DA + 8 > 40 ? DA + 8 : 40); }
// LDS ahead of the window map: the stages or, should it come to that, the fp32 body's tiles.
// (and, before the first tile, the waves' own areas)
template <int DA, int T, int XS>
constexpr size_t lds_tiles()
{
    constexpr size_t a = Lay<DA, T>::BYTES, b = sizeof(Smem<XS>), c = (size_t)(T == 32 ? 5 : 8) * stat_elems<DA>() * sizeof(bf16_t);
    return a > b ? (a > c ? a : c) : (b > c ? b : c);
}

// Three bf16 parts of a pair of values (each dword: low half the first).
struct Parts {
    uint32_t p[3];
};
__device__ __forceinline__ Parts split_pair(float a, float b)
{
    Parts r;
    r.p[0] = pack_bf16(a, b);
    const float a1 = a - lo_bf16(r.p[0]), b1 = b - hi_bf16(r.p[0]);
    r.p[1] = pack_bf16(a1, b1);
    r.p[2] = pack_bf16(a1 - lo_bf16(r.p[1]), b1 - hi_bf16(r.p[1]));
    return r;
}
// What a lane has staged so far: the largest magnitude, and the smallest first part that is not zero (of the
// low and the high halves of the dwords apart; twice the bits, minus one: without the sign, and zero the
// largest).  (A NaN is passed over: its first part is a NaN, which reaches what fp32 products would have
// reached.)
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
struct Range {
    float mx;
    u16x2 mn;
    __device__ __forceinline__ bool outside() const
    {
        constexpr unsigned short small = (unsigned short)((127 - kSmallExp) << 8) - 1;
        return mx >= kLimit || mn.x < small || mn.y < small;
    }
};
__device__ __forceinline__ void note_high(Range &rn, float a, float b) { rn.mx = fmaxf(fmaxf(rn.mx, fabsf(a)), fabsf(b)); }
__device__ __forceinline__ void note_low(Range &rn, const Parts &r)
{
    uint32_t key;       // (the compiler takes two instructions for 2 x - 1)
    asm("v_pk_mad_u16 %0, %1, 2, -1 op_sel_hi:[1,0,0]" : "=v"(key) : "v"(r.p[0]));
    rn.mn = __builtin_elementwise_min(rn.mn, __builtin_bit_cast(u16x2, key));
}

// The streamed pair of tensors of one (image, head), in bytes.
struct Stream {
    const char *xb, *yb, *fb;
    uint32_t xs, ys, frow;
};

// What a lane stages: 8 lanes share a token, lane j of them the values 4j .. 4j+3 of both content rows
// and of the RIB row (DA = 64: also 32 + 4j, ...).  Lanes past the end slide back onto the last four
// of the padded row (they duplicate a neighbour); its odd last value reads as zero.
struct Piece {
    int c, f0, f1;
    bool codd, fodd, fnone;         // (uniform) odd lengths / no RIB
};
__device__ __forceinline__ Piece piece_of(const Geo &g, int j)
{
    const int pd = (g.d + 1) & ~1, pr = (g.r + 1) & ~1;
    Piece p;
    p.c = 4 * j < pd - 4 ? 4 * j : pd - 4;
    p.f0 = 4 * j < pr - 4 ? 4 * j : pr - 4;
    p.f1 = 32 + 4 * j < pr - 4 ? 32 + 4 * j : pr - 4;
    p.codd = (g.d & 1) != 0, p.fodd = (g.r & 1) != 0, p.fnone = g.r == 0;
    return p;
}
__device__ __forceinline__ float4u get4(const char *base, uint32_t off, int c, int n, bool odd)
{
    const float *p = (const float *)(base + (off + 4u * c));
    if (!odd) return *(const float4u *)p;
    float4u v;
    v.x = p[0], v.y = p[1], v.z = p[2];
    v.w = c + 3 < n ? p[c + 3 < n ? 3 : 2] : 0.f;
    return v;
}
// (NT: the workgroup's lanes where they are a constant, 0: at least 256)
template <int DA, int T, int NT = 0>
struct Regs {
    static constexpr int SLOTS = NT ? T * 8 / NT : T / 32;
    float4u x[SLOTS], y[SLOTS], fa[SLOTS], fb[DA == 64 ? SLOTS : 1];
    float e0;
};
// Slots tid, tid + nt, ... of a tile's T * 8.
template <int DA, int T, bool EXTRA, int NT = 0>
__device__ __forceinline__ void request(Regs<DA, T, NT> &rg, const Geo &g, const rows::Win &win, const Stream &s, int tile, int wave,
                                        const float *lse, const float *delta)
{
    const int nt = NT ? NT : blockDim.x, lane = rows::opaque_tid() & 63, l = lane >> 3;
    const Piece pc = piece_of(g, lane & 7);
#pragma unroll
    for (int p = 0; p < Regs<DA, T, NT>::SLOTS; ++p) {
        const int slot = p * nt + wave * 64;
        if (slot < T * 8) {
            const int n = tile * T + (slot >> 3) + l, nc = n < win.last ? n : win.last;
            const uint32_t t = win.token<false>(n, 0);
            rg.x[p] = get4(s.xb, __umul24(t, s.xs), pc.c, g.d, pc.codd);
            rg.y[p] = get4(s.yb, __umul24(t, s.ys), pc.c, g.d, pc.codd);
            if (!pc.fnone) {
                const uint32_t fr = __umul24((uint32_t)nc, s.frow);
                rg.fa[p] = get4(s.fb, fr, pc.f0, g.r, pc.fodd);
                if (DA == 64) rg.fb[p] = get4(s.fb, fr, pc.f1, g.r, pc.fodd);
            }
        }
    }
    if (EXTRA && wave < T / 32) {   // LSE by the first T lanes, delta by the next
        const int e = wave * 64 + lane, n = tile * T + (e & (T - 1));
        rg.e0 = (e < T ? lse : delta)[n < win.last ? n : win.last];
    }
}
struct __attribute__((packed, aligned(4))) dwords2 {
    uint32_t x, y;
};
// LOW: whether a small value matters.  It does not in the operands of the scores (an error of 2^-100 in a logit).
template <bool LOW>
__device__ __forceinline__ void put4(bf16_t *dst, int part, const float4u &v, float s, Range &rn)
{
    const float a = v.x * s, b = v.y * s, c = v.z * s, d = v.w * s;
    note_high(rn, a, b);
    note_high(rn, c, d);
    const Parts lo = split_pair(a, b), hi = split_pair(c, d);
    if (LOW) {
        note_low(rn, lo);
        note_low(rn, hi);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) *(dwords2 *)(dst + i * part) = dwords2{lo.p[i], hi.p[i]};
}
// GRAD: the X rows are operands of gradients too.
template <int DA, int T, bool GRAD, bool EXTRA, int NT = 0>
__device__ __forceinline__ void commit(const Regs<DA, T, NT> &rg, const Geo &g, bf16_t *S, float sc, float sp, int wave, Range &rn)
{
    using L = Lay<DA, T>;
    const int nt = NT ? NT : blockDim.x, lane = rows::opaque_tid() & 63, l = lane >> 3, pd = (g.d + 1) & ~1;
    const Piece pc = piece_of(g, lane & 7);
#pragma unroll
    for (int p = 0; p < Regs<DA, T, NT>::SLOTS; ++p) {
        const int slot = p * nt + wave * 64;
        if (slot < T * 8) {
            bf16_t *xr = S + __mul24((slot >> 3) + l, L::XS), *yr = S + L::YR + __mul24((slot >> 3) + l, L::YS);
            put4<GRAD>(xr + pc.c, L::XP, rg.x[p], sc, rn);
            put4<true>(yr + pc.c, L::YP, rg.y[p], 1.f, rn);
            if (!pc.fnone) {
                put4<GRAD>(xr + pd + pc.f0, L::XP, rg.fa[p], sp, rn);
                if (DA == 64) put4<GRAD>(xr + pd + pc.f1, L::XP, rg.fb[p], sp, rn);
            }
        }
    }
    if (EXTRA && wave < T / 32) {
        const int e = wave * 64 + lane;
        const float v = e < T ? rg.e0 * kLog2e : rg.e0;
        note_high(rn, v, v);
        ((float *)(S + L::EX))[e] = v;
    }
}
// The columns no staging code writes (they meet zeros, so they only have to be finite).
template <int DA, int T, int STAGES = 3>
__device__ __forceinline__ void zero_pads(const Geo &g, bf16_t *stages)
{
    using L = Lay<DA, T>;
    const int pd = (g.d + 1) & ~1, pa = pd + ((g.r + 1) & ~1);
    for (int e = threadIdx.x; e < STAGES * 3 * T; e += (int)blockDim.x) {
        const int st = e / (3 * T), row = e - st * 3 * T;          // (the rows of the three parts follow one another)
        bf16_t *xr = stages + st * L::STAGE + row * L::XS, *yr = stages + st * L::STAGE + L::YR + row * L::YS;
        for (int c = pa; c < DA; c += 2) *(uint32_t *)(xr + c) = 0u;
        for (int c = pd; c < 32; c += 2) *(uint32_t *)(yr + c) = 0u;
    }
}

// A wave's 32 stationary rows between their request and their staging: 8 lanes a row, 8 rows a pass.
template <int DA, bool WITH_Y>
struct StatRegs {
    float4u x[4], y[WITH_Y ? 4 : 1], fa[4], fb[DA == 64 ? 4 : 1];
};
template <int DA, bool WITH_Y>
__device__ __forceinline__ void stat_request(StatRegs<DA, WITH_Y> &r, const Geo &g, const rows::Win &win, const Stream &s, int n0)
{
    const int lane = threadIdx.x & 63, l = lane >> 3;
    const Piece pc = piece_of(g, lane & 7);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int n = n0 + p * 8 + l, nc = n < win.last ? n : win.last;
        const uint32_t t = win.token<false>(n, 0);
        r.x[p] = get4(s.xb, __umul24(t, s.xs), pc.c, g.d, pc.codd);
        if (WITH_Y) r.y[p] = get4(s.yb, __umul24(t, s.ys), pc.c, g.d, pc.codd);
        if (!pc.fnone) {
            const uint32_t fr = __umul24((uint32_t)nc, s.frow);
            r.fa[p] = get4(s.fb, fr, pc.f0, g.r, pc.fodd);
            if (DA == 64) r.fb[p] = get4(s.fb, fr, pc.f1, g.r, pc.fodd);
        }
    }
}
// ... scaled, split and read back as B operands through the wave's own LDS area (three parts of 32 rows;
// the value-like rows follow in the same place).
template <int DA, bool WITH_Y>
__device__ __forceinline__ void stat_stage(const StatRegs<DA, WITH_Y> &r, const Geo &g, bf16_t *W, float sc, float sp, Range &rn,
                                           bf16x8 (&X)[3][DA / 16], bf16x8 (&Y)[3][2])
{
    constexpr int XS = DA + 8, YS = 40;
    const int lane = threadIdx.x & 63, l = lane >> 3, col = lane & 31, hf = lane >> 5;
    const int pd = (g.d + 1) & ~1, pa = pd + ((g.r + 1) & ~1);
    const Piece pc = piece_of(g, lane & 7);
    for (int e = lane; e < 96; e += 64)
        for (int c = pa; c < DA; c += 2) *(uint32_t *)(W + e * XS + c) = 0u;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        bf16_t *xr = W + (p * 8 + l) * XS;
        put4<false>(xr + pc.c, 32 * XS, r.x[p], sc, rn);
        if (!pc.fnone) {
            put4<false>(xr + pd + pc.f0, 32 * XS, r.fa[p], sp, rn);
            if (DA == 64) put4<false>(xr + pd + pc.f1, 32 * XS, r.fb[p], sp, rn);
        }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int p = 0; p < 3; ++p) read_rows<DA / 16>(X[p], W + p * 32 * XS + col * XS + 8 * hf);
    if (WITH_Y) {
        __builtin_amdgcn_wave_barrier();
        for (int e = lane; e < 96; e += 64)
            for (int c = pd; c < 32; c += 2) *(uint32_t *)(W + e * YS + c) = 0u;
#pragma unroll
        for (int p = 0; p < 4; ++p) put4<true>(W + (p * 8 + l) * YS + pc.c, 32 * YS, r.y[p], 1.f, rn);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < 3; ++p) read_rows<2>(Y[p], W + p * 32 * YS + col * YS + 8 * hf);
    }
}

// acc += A B over KS k-steps, six part products each, the small ones first.
template <int KS>
__device__ __forceinline__ void mul6(f32x16 &acc, const bf16x8 (&A)[3][KS], const bf16x8 (&B)[3][KS])
{
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int c = 0; c < 6; ++c)
#pragma unroll
        for (int t = 0; t < KS; ++t) acc = rows::mfma(A[pa[c]][t], B[pb[c]][t], acc);
}
// The same with the small products in an accumulator of their own, which the vector ALU adds: a matrix
// instruction drops the low bits of what it adds to larger values, always to one side.  In single
// elements that does not show, but dP, dS and the gradients are summed over many tokens with
// cancellation, where it does: the generator's weight gradients behind a layer of 20 windows of 625
// tokens were off by 6e-6 (2-norm, against fp64; fp32 products: 9e-7) until dP, the gradients and O
// were summed this way.  The scores need it not (measured).
template <int KS>
__device__ __forceinline__ void mul6_apart(f32x16 &acc, const bf16x8 (&A)[3][KS], const bf16x8 (&B)[3][KS])
{
    constexpr int pa[5] = {2, 0, 1, 1, 0}, pb[5] = {0, 2, 1, 0, 1};
    f32x16 t = {0};
#pragma unroll
    for (int c = 0; c < 5; ++c)
#pragma unroll
        for (int k = 0; k < KS; ++k) t = rows::mfma(A[pa[c]][k], B[pb[c]][k], t);
#pragma unroll
    for (int k = 0; k < KS; ++k) acc = rows::mfma(A[0][k], B[0][k], acc);
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] += t[i];
}
// A operands: 32 token rows at `row` of an image (natural order), or transposed (tokens contracted).
template <int N>
__device__ __forceinline__ void load_rows(bf16x8 (&A)[3][N], const bf16_t *base, int part)
{
#pragma unroll
    for (int p = 0; p < 3; ++p) read_rows<N>(A[p], base + p * part);
}
template <int STRIDE>
__device__ __forceinline__ void load_tr(bf16x8 (&A)[3][2], const bf16_t *rows0, int part, int off, int c0)
{
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int i = 0; i < 2; ++i) A[p][i] = read_tr<STRIDE>(rows0 + p * part + 16 * i * STRIDE, off, c0);
}
// The order of a region of MFMAs, the LDS reads of their operands and independent vector work:
// reads, then one MFMA and PER vector instructions in turn.
template <int MFMAS, int PER>
__device__ __forceinline__ void interleave()
{
    __builtin_amdgcn_sched_group_barrier(0x100, 32, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);
#pragma unroll
    for (int i = 0; i < MFMAS; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, PER, 0);
    }
}
// The same by truncation: cheaper, and the parts are exact all the same.
__device__ __forceinline__ float high_part(float a) { return __uint_as_float(__float_as_uint(a) & 0xffff0000u); }
__device__ __forceinline__ Parts split_pair_trunc(float a, float b)
{
    Parts r;
    r.p[0] = rows::trunc_pack(a, b);
    const float a1 = a - high_part(a), b1 = b - high_part(b);
    r.p[1] = rows::trunc_pack(a1, b1);
    r.p[2] = rows::trunc_pack(a1 - high_part(a1), b1 - high_part(b1));
    return r;
}
// A finished block of P or dS as B operands of the products over its rows.
__device__ __forceinline__ void split_block(bf16x8 (&B)[3][2], const f32x16 &S)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        Parts q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) q[i] = split_pair_trunc(S[8 * h + 2 * i], S[8 * h + 2 * i + 1]);
#pragma unroll
        for (int p = 0; p < 3; ++p) B[p][h] = as_bf16x8(q[0].p[p], q[1].p[p], q[2].p[p], q[3].p[p]);
    }
}

// Columns 32 mb .. of a token's gradient row: content (times sc) to the grid, RIB (times sp) to the partial.
__device__ __forceinline__ void store_cols(const f32x16 &acc, int mb, int hf, const Geo &g, float sc, float sp, float *grid_row,
                                           float *part_row)
{
    const int pd = (g.d + 1) & ~1;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int c = 32 * mb + 8 * a + 4 * hf;
        if (c + 4 <= g.d) {
            *(float4u *)(grid_row + c) = float4u{acc[4 * a] * sc, acc[4 * a + 1] * sc, acc[4 * a + 2] * sc, acc[4 * a + 3] * sc};
        } else if (part_row && c >= pd && c + 4 <= pd + g.r) {
            *(float4u *)(part_row + (c - pd)) = float4u{acc[4 * a] * sp, acc[4 * a + 1] * sp, acc[4 * a + 2] * sp, acc[4 * a + 3] * sp};
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (c + i < g.d) grid_row[c + i] = acc[4 * a + i] * sc;
                else if (part_row && c + i >= pd && c + i < pd + g.r) part_row[c + i - pd] = acc[4 * a + i] * sp;
            }
        }
    }
}

#define RIB_SPLIT_SETUP(MAP, ROW0, WAVE)                                                                         \
    using L = Lay<DA, T>;                                                                                         \
    extern __shared__ __attribute__((aligned(16))) bf16_t smem[];                                              \
    int64_t u;                                                                                                 \
    int blk, b;                                                                                                \
    unit_of_block(nblk, u, blk);                                                                               \
    const int w = (int)(u / g.heads), hd = (int)(u - (int64_t)w * g.heads);                                    \
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);                                         \
    const int lane = threadIdx.x & 63, col = lane & 31, hf = lane >> 5;                                        \
    const rows::Win win = rows::window_of<false>(g, w, (int)blockDim.x, (int *)((char *)smem + (MAP)), b);     \
    const int64_t img = (int64_t)b * g.H * g.W;                                                                \
    const int ntiles = (g.N + T - 1) / T;                                                                      \
    /* this lane's stationary token (past the window's end: its last, whose results are not stored) */         \
    const int row0 = ROW0, n = row0 + WAVE * 32 + col, nc = n < win.last ? n : win.last;                         \
    const int64_t tn = img + win.any(nc);                                                                      \
    Range rn = {0.f, {0xffff, 0xffff}};                                                                                  \
    __syncthreads();

// ln(2^m l) with one rounding of the sum: the integer part of log2 l joins m's product with ln 2, whose
// rounding error is carried along.
__device__ __forceinline__ float log_sum(float m, float l)
{
    constexpr float ln2 = 0.693147182464599609375f, ln2_lo = -1.904654299957e-9f;      // fp32(ln 2) and the rest
    int e;
    const float f = logf(frexpf(l, &e));
    const float a = m * ln2, b = (float)e * ln2, s = a + b, v = s - a;
    const float err = (a - (s - v)) + (b - v) + fmaf(m, ln2, -a) + fmaf((float)e, ln2, -b) + (m + (float)e) * ln2_lo;
    return s + (f + err);
}

// Normalised O of a lane's token, gated where asked for, and LSE.
__device__ __forceinline__ void store_out(const f32x16 &O, float l, float m, const Geo &g, int hf, int64_t tn, int hd, int64_t u, int n,
                                          float *out, float *lse)
{
    const float inv = 1.f / l;
    const int64_t base = tn * g.C + hd * g.d;
    if (g.gate) {           // CLA gate (Eq. 9) on the way out, the raw O beside it if asked for
        const float *gt = (const float *)g.gate + base;
        float *raw = g.out_raw ? (float *)g.out_raw + base : nullptr;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int c = acc_row(i) + 4 * hf;
            if (c >= g.d) continue;
            const float o = O[i] * inv;
            out[base + c] = o * gt[c];
            if (raw) raw[c] = o;
        }
    } else {
        store_cols(O, 0, hf, g, inv, 0.f, out + base, nullptr);
    }
    if (lse != nullptr && hf == 0) lse[u * g.N + n] = log_sum(m, l);
}

template <int DA, int T>
__global__ __launch_bounds__(512, 2) void fwd_kernel(Geo g, int nblk, uint32_t inv_r, const float *__restrict__ q,
                                                     const float *__restrict__ k, const float *__restrict__ v,
                                                     const float *__restrict__ fq, const float *__restrict__ fk,
                                                     float *__restrict__ out, float *__restrict__ lse)
{
    RIB_SPLIT_SETUP((lds_tiles<DA, T, DA + 1>()), blk * (int)(blockDim.x >> 1), wave)
    const int ax = col * L::XS + 8 * hf, tro_y = tr_lane_offset<L::YS>(lane);
    const Stream ks = {(const char *)(k + img * g.tstride + hd * g.d), (const char *)(v + img * g.tstride + hd * g.d),
                       (const char *)(fk + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.tstride * 4u,
                       (uint32_t)g.r * 4u};
    const Stream qs = {(const char *)(q + img * g.tstride + hd * g.d), nullptr,
                       (const char *)(fq + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.C * 4u,
                       (uint32_t)g.r * 4u};
    Regs<DA, T> rg, rg1;
    bf16x8 Q[3][L::KS], none[3][2];
    {
        // one exposed memory latency: the wave's rows and the first two tiles are requested together
        StatRegs<DA, false> sr;
        stat_request<DA, false>(sr, g, win, qs, row0 + wave * 32);
        request<DA, T, false>(rg, g, win, ks, 0, wave, nullptr, nullptr);
        request<DA, T, false>(rg1, g, win, ks, ntiles > 1 ? 1 : 0, wave, nullptr, nullptr);
        stat_stage<DA, false>(sr, g, smem + wave * stat_elems<DA>(), g.scale_c * kLog2e, g.scale_p * kLog2e, rn, Q, none);
    }
    __syncthreads();
    zero_pads<DA, T>(g, smem);
    commit<DA, T, false, false>(rg, g, smem, 1.f, 1.f, wave, rn);
    commit<DA, T, false, false>(rg1, g, smem + L::STAGE, 1.f, 1.f, wave, rn);
    request<DA, T, false>(rg, g, win, ks, ntiles > 2 ? 2 : ntiles - 1, wave, nullptr, nullptr);
    __syncthreads();

    f32x16 O = {0}, S, Sn;
    float m = -INFINITY, l = 0.f;
    auto scores = [&](f32x16 &S, const bf16_t *stage, int kb) {
        bf16x8 A[3][L::KS];
        load_rows<L::KS>(A, stage + kb * 32 * L::XS + ax, L::XP);
        S = f32x16{0};
        mul6<L::KS>(S, A, Q);
    };
    scores(S, smem, 0);
    int c0 = 0, c1 = L::STAGE, c2 = 2 * L::STAGE;
    for (int tile = 0; tile < ntiles; ++tile) {
        const bf16_t *cur = smem + c0, *nxt = smem + c1;
#pragma unroll
        for (int kb = 0; kb < T / 32; ++kb) {
            const int key0 = tile * T + kb * 32;
            if (kb == 0) __syncthreads();
            if (key0 + 32 > g.N) rows::mask_rows(S, key0, g.N, hf);
            float t = S[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) t = fmaxf(t, S[i]);
            t = fmaxf(t, __shfl_xor(t, 32));
            // the running maximum is raised only when exceeded by 2^8 (always by the first block)
            if (__any(t > m + 8.f)) {
                const float mn = fmaxf(m, t), alpha = __builtin_amdgcn_exp2f(m - mn);
                m = mn;
                l *= alpha;
#pragma unroll
                for (int i = 0; i < 16; ++i) O[i] *= alpha;
            }
            RIB_FENCE();
            // the next block's scores run beside this block's exponentials and splits
            scores(Sn, kb + 1 < T / 32 ? cur : nxt, kb + 1 < T / 32 ? kb + 1 : 0);
            float ps = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                S[i] = __builtin_amdgcn_exp2f(S[i] - m);
                ps += S[i];
            }
            l += ps;
            bf16x8 P[3][2], V[3][2];
            split_block(P, S);
            interleave<6 * L::KS, 150 / (6 * L::KS)>();
            RIB_FENCE();
            if (kb == 0) {
                commit<DA, T, false, false>(rg, g, smem + c2, 1.f, 1.f, wave, rn);
                request<DA, T, false>(rg, g, win, ks, tile + 3 < ntiles ? tile + 3 : ntiles - 1, wave, nullptr, nullptr);
            }
            load_tr<L::YS>(V, cur + L::YR + kb * 32 * L::YS, L::YP, tro_y, 0);
            mul6_apart<2>(O, V, P);
            S = Sn;
            RIB_FENCE();
        }
        const int r0 = c0;
        c0 = c1, c1 = c2, c2 = r0;
    }
    if (__syncthreads_or(rn.outside())) {
        fwd_body<DA>(g, *(Smem<DA + 1> *)smem, u, row0, g.N, inv_r, q, k, v, fq, fk, out, lse);
        return;
    }
    l += __shfl_xor(l, 32);
    if (n >= g.N) return;
    store_out(O, l, m, g, hf, tn, hd, u, n, out, lse);
}

// Small grids: a wave that walks the whole window takes all of the call's time while most of the chip is idle (one 48 x 48 image
// of 16 x 16 windows, 2 heads: 36 workgroups of four waves, 14 of the forward's 18 us in eight steps one after the other).
// So the streamed side is dealt out as well: workgroups of eight waves, QW = 8 / G of them with 32 stationary
// tokens each, in G groups; tiles of 32 G tokens, of which group `grp` takes the grp-th block; two stages, one barrier a
// tile.  The groups' sums are added through LDS in ascending order (the forward's with their own stabilisers).
// Us, before / with these kernels: that image's forward 18.5 / 14.0; forward + backward of one 32 x 32 window of 2 heads 204 /
// 123, one 64 x 64 window 722 / 378, 4 x 4 windows of 16 x 16, 2 heads 78 / 61.  Taken where they fit one round of the chip: in two
// they are slower (48 units of 256 tokens 18.7 / 25.7, 2 of 9216 402 / 441).
template <int DA>
struct Keys {
    static constexpr int G = DA == 64 ? 2 : 4, QW = 8 / G, T = 32 * G;        // (two stages of 128 tokens of 64 columns exceed a CU's LDS)
    using L = Lay<DA, T>;
    static constexpr size_t sums = (size_t)8 * (L::RB + 1) * 16 * 64 * sizeof(float);     // (dK_aug and dV of every wave)
    static constexpr size_t tiles = (size_t)2 * L::STAGE * sizeof(bf16_t), stat = (size_t)8 * stat_elems<DA>() * sizeof(bf16_t);
    template <int XS>
    static constexpr size_t lds()
    {
        constexpr size_t a = tiles > stat ? tiles : stat, b = sums > sizeof(Smem<XS>) ? sums : sizeof(Smem<XS>);
        return a > b ? a : b;
    }
};
template <int DA>
__global__ __launch_bounds__(512, 2) void fwd_keys_kernel(Geo g, int nblk, uint32_t inv_r, const float *__restrict__ q,
                                                          const float *__restrict__ k, const float *__restrict__ v,
                                                          const float *__restrict__ fq, const float *__restrict__ fk,
                                                          float *__restrict__ out, float *__restrict__ lse)
{
    using Z = Keys<DA>;
    constexpr int T = Z::T, NT = 512;
    RIB_SPLIT_SETUP((Z::template lds<DA + 1>()), blk * (32 * Z::QW), (wave % Z::QW))
    const int grp = wave / Z::QW;
    const int ax = col * L::XS + 8 * hf, tro_y = tr_lane_offset<L::YS>(lane);
    const Stream ks = {(const char *)(k + img * g.tstride + hd * g.d), (const char *)(v + img * g.tstride + hd * g.d),
                       (const char *)(fk + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.tstride * 4u,
                       (uint32_t)g.r * 4u};
    const Stream qs = {(const char *)(q + img * g.tstride + hd * g.d), nullptr,
                       (const char *)(fq + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.C * 4u,
                       (uint32_t)g.r * 4u};
    Regs<DA, T, NT> rg;
    bf16x8 Q[3][L::KS], none[3][2];
    {
        StatRegs<DA, false> sr;
        stat_request<DA, false>(sr, g, win, qs, row0 + (wave % Z::QW) * 32);
        request<DA, T, false, NT>(rg, g, win, ks, 0, wave, nullptr, nullptr);
        stat_stage<DA, false>(sr, g, smem + wave * stat_elems<DA>(), g.scale_c * kLog2e, g.scale_p * kLog2e, rn, Q, none);
    }
    __syncthreads();
    zero_pads<DA, T, 2>(g, smem);
    commit<DA, T, false, false, NT>(rg, g, smem, 1.f, 1.f, wave, rn);
    request<DA, T, false, NT>(rg, g, win, ks, ntiles > 1 ? 1 : 0, wave, nullptr, nullptr);

    f32x16 O = {0};
    float m = -INFINITY, l = 0.f;
#pragma unroll 1
    for (int tile = 0; tile < ntiles; ++tile) {
        const bf16_t *cur = smem + (tile & 1) * L::STAGE;
        const int key0 = tile * T + grp * 32;
        __syncthreads();
        if (tile + 1 < ntiles) {
            commit<DA, T, false, false, NT>(rg, g, smem + ((tile + 1) & 1) * L::STAGE, 1.f, 1.f, wave, rn);
            request<DA, T, false, NT>(rg, g, win, ks, tile + 2 < ntiles ? tile + 2 : ntiles - 1, wave, nullptr, nullptr);
        }
        if (key0 >= g.N) continue;
        f32x16 S = {0};
        {
            bf16x8 A[3][L::KS];
            load_rows<L::KS>(A, cur + grp * 32 * L::XS + ax, L::XP);
            mul6<L::KS>(S, A, Q);
        }
        if (key0 + 32 > g.N) rows::mask_rows(S, key0, g.N, hf);
        float t = S[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) t = fmaxf(t, S[i]);
        t = fmaxf(t, __shfl_xor(t, 32));
        if (__any(t > m + 8.f)) {
            const float mn = fmaxf(m, t), alpha = __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l *= alpha;
#pragma unroll
            for (int i = 0; i < 16; ++i) O[i] *= alpha;
        }
        float ps = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            S[i] = __builtin_amdgcn_exp2f(S[i] - m);
            ps += S[i];
        }
        l += ps;
        bf16x8 P[3][2], V[3][2];
        split_block(P, S);
        load_tr<L::YS>(V, cur + L::YR + grp * 32 * L::YS, L::YP, tro_y, 0);
        mul6_apart<2>(O, V, P);
    }
    if (__syncthreads_or(rn.outside())) {
        fwd_body<DA>(g, *(Smem<DA + 1> *)smem, u, row0, row0 + 32 * Z::QW, inv_r, q, k, v, fq, fk, out, lse);
        return;
    }
    float *const part = (float *)smem;          // [wave][18][64]
    if (grp > 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) part[(wave * 18 + i) * 64 + lane] = O[i];
        part[(wave * 18 + 16) * 64 + lane] = m;
        part[(wave * 18 + 17) * 64 + lane] = l;
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int j = 1; j < Z::G; ++j) {
        const float *pw = part + (wave + j * Z::QW) * 18 * 64 + lane;
        const float mj = pw[16 * 64], mn = fmaxf(m, mj);        // (no key of group j: minus infinity, and zeros)
        const float a = __builtin_amdgcn_exp2f(m - mn), b = __builtin_amdgcn_exp2f(mj - mn);
        m = mn;
        l = l * a + pw[17 * 64] * b;
#pragma unroll
        for (int i = 0; i < 16; ++i) O[i] = O[i] * a + pw[i * 64] * b;
    }
    l += __shfl_xor(l, 32);
    if (n >= g.N) return;
    store_out(O, l, m, g, hf, tn, hd, u, n, out, lse);
}

template <int DA, int T>
__global__ __launch_bounds__(512, 2) void dq_kernel(Geo g, int nblk, uint32_t inv_r, const float *__restrict__ q,
                                                    const float *__restrict__ k, const float *__restrict__ v,
                                                    const float *__restrict__ fq, const float *__restrict__ fk,
                                                    const float *__restrict__ dout, const float *__restrict__ lse,
                                                    const float *__restrict__ delta, float *__restrict__ dq,
                                                    float *__restrict__ dfq_part)
{
    RIB_SPLIT_SETUP((lds_tiles<DA, T, kXS>()), blk * (int)(blockDim.x >> 1), wave)
    const int ax = col * L::XS + 8 * hf, ay = L::YR + col * L::YS + 8 * hf, tro_x = tr_lane_offset<L::XS>(lane);
    const Stream ks = {(const char *)(k + img * g.tstride + hd * g.d), (const char *)(v + img * g.tstride + hd * g.d),
                       (const char *)(fk + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.tstride * 4u,
                       (uint32_t)g.r * 4u};
    const Stream qs = {(const char *)(q + img * g.tstride + hd * g.d), (const char *)(dout + img * g.C + hd * g.d),
                       (const char *)(fq + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.C * 4u,
                       (uint32_t)g.r * 4u};
    const float lse2 = lse[u * g.N + nc] * kLog2e, dl = delta[u * g.N + nc];
    note_high(rn, lse2, dl);
    Regs<DA, T> rg, rg1;
    bf16x8 Q[3][L::KS], G[3][2];
    {
        // one exposed memory latency: the wave's rows and the first two tiles are requested together
        StatRegs<DA, true> sr;
        stat_request<DA, true>(sr, g, win, qs, row0 + wave * 32);
        request<DA, T, false>(rg, g, win, ks, 0, wave, nullptr, nullptr);
        request<DA, T, false>(rg1, g, win, ks, ntiles > 1 ? 1 : 0, wave, nullptr, nullptr);
        stat_stage<DA, true>(sr, g, smem + wave * stat_elems<DA>(), g.scale_c * kLog2e, g.scale_p * kLog2e, rn, Q, G);
    }
    __syncthreads();
    zero_pads<DA, T>(g, smem);
    commit<DA, T, true, false>(rg, g, smem, 1.f, 1.f, wave, rn);
    commit<DA, T, true, false>(rg1, g, smem + L::STAGE, 1.f, 1.f, wave, rn);
    request<DA, T, false>(rg, g, win, ks, ntiles > 2 ? 2 : ntiles - 1, wave, nullptr, nullptr);
    __syncthreads();

    f32x16 acc[L::RB];
#pragma unroll
    for (int mb = 0; mb < L::RB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[mb][i] = 0.f;
    f32x16 S, D, Sn, Dn;
    auto scores = [&](f32x16 &S, f32x16 &D, const bf16_t *stage, int kb) {
        bf16x8 A[3][L::KS], V[3][2];
        load_rows<L::KS>(A, stage + kb * 32 * L::XS + ax, L::XP);
        load_rows<2>(V, stage + kb * 32 * L::YS + ay, L::YP);
        S = f32x16{0}, D = f32x16{0};
        mul6<L::KS>(S, A, Q);
        mul6_apart<2>(D, V, G);
    };
    scores(S, D, smem, 0);
    int c0 = 0, c1 = L::STAGE, c2 = 2 * L::STAGE;
    for (int tile = 0; tile < ntiles; ++tile) {
        const bf16_t *cur = smem + c0, *nxt = smem + c1;
#pragma unroll
        for (int kb = 0; kb < T / 32; ++kb) {
            const int key0 = tile * T + kb * 32;
            if (kb == 0) __syncthreads();
            if (key0 + 32 > g.N) rows::mask_rows(S, key0, g.N, hf);
            RIB_FENCE();
            // the next block's products run beside this block's exponentials and splits
            scores(Sn, Dn, kb + 1 < T / 32 ? cur : nxt, kb + 1 < T / 32 ? kb + 1 : 0);
#pragma unroll
            for (int i = 0; i < 16; ++i) S[i] = __builtin_amdgcn_exp2f(S[i] - lse2) * (D[i] - dl);
            bf16x8 B[3][2];
            split_block(B, S);
            interleave<6 * L::KS + 12, 160 / (6 * L::KS + 12)>();
            RIB_FENCE();
            if (kb == 0) {
                commit<DA, T, true, false>(rg, g, smem + c2, 1.f, 1.f, wave, rn);
                request<DA, T, false>(rg, g, win, ks, tile + 3 < ntiles ? tile + 3 : ntiles - 1, wave, nullptr, nullptr);
            }
#pragma unroll
            for (int mb = 0; mb < L::RB; ++mb) {
                bf16x8 A[3][2];
                load_tr<L::XS>(A, cur + kb * 32 * L::XS, L::XP, tro_x, 32 * mb);
                mul6_apart<2>(acc[mb], A, B);
            }
            S = Sn, D = Dn;
            RIB_FENCE();
        }
        const int r0 = c0;
        c0 = c1, c1 = c2, c2 = r0;
    }
    if (__syncthreads_or(rn.outside())) {
        dq_body<DA>(g, *(Smem<kXS> *)smem, u, row0, g.N, inv_r, q, k, v, fq, fk, dout, lse, delta, dq, dfq_part);
        return;
    }
    if (n >= g.N) return;
#pragma unroll
    for (int mb = 0; mb < L::RB; ++mb)
        store_cols(acc[mb], mb, hf, g, g.scale_c, g.scale_p, dq + tn * g.C + hd * g.d, dfq_part + (u * g.N + n) * g.r);
}

template <int DA, int T>
__global__ __launch_bounds__(512, 2) void dkv_kernel(Geo g, int nblk, uint32_t inv_r, const float *__restrict__ q,
                                                     const float *__restrict__ k, const float *__restrict__ v,
                                                     const float *__restrict__ fq, const float *__restrict__ fk,
                                                     const float *__restrict__ dout, const float *__restrict__ lse,
                                                     const float *__restrict__ delta, float *__restrict__ dk,
                                                     float *__restrict__ dv, float *__restrict__ dfk_part)
{
    RIB_SPLIT_SETUP((lds_tiles<DA, T, kXS>()), blk * (int)(blockDim.x >> 1), wave)
    const int ax = col * L::XS + 8 * hf, ay = L::YR + col * L::YS + 8 * hf, tro_x = tr_lane_offset<L::XS>(lane),
              tro_y = tr_lane_offset<L::YS>(lane);
    const Stream qs = {(const char *)(q + img * g.tstride + hd * g.d), (const char *)(dout + img * g.C + hd * g.d),
                       (const char *)(fq + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.C * 4u,
                       (uint32_t)g.r * 4u};
    const float *lu = lse + u * g.N, *du = delta + u * g.N;
    const Stream ks = {(const char *)(k + img * g.tstride + hd * g.d), (const char *)(v + img * g.tstride + hd * g.d),
                       (const char *)(fk + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.tstride * 4u,
                       (uint32_t)g.r * 4u};
    Regs<DA, T> rg, rg1;
    bf16x8 K[3][L::KS], V[3][2];
    {
        // one exposed memory latency: the wave's rows and the first two tiles are requested together
        StatRegs<DA, true> sr;
        stat_request<DA, true>(sr, g, win, ks, row0 + wave * 32);
        request<DA, T, true>(rg, g, win, qs, 0, wave, lu, du);
        request<DA, T, true>(rg1, g, win, qs, ntiles > 1 ? 1 : 0, wave, lu, du);
        stat_stage<DA, true>(sr, g, smem + wave * stat_elems<DA>(), 1.f, 1.f, rn, K, V);
    }
    __syncthreads();
    zero_pads<DA, T>(g, smem);
    commit<DA, T, true, true>(rg, g, smem, g.scale_c, g.scale_p, wave, rn);
    commit<DA, T, true, true>(rg1, g, smem + L::STAGE, g.scale_c, g.scale_p, wave, rn);
    request<DA, T, true>(rg, g, win, qs, ntiles > 2 ? 2 : ntiles - 1, wave, lu, du);
    __syncthreads();

    f32x16 accV = {0}, accK[L::RB];
#pragma unroll
    for (int mb = 0; mb < L::RB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) accK[mb][i] = 0.f;
    f32x16 S, D;
    auto scores = [&](const bf16_t *stage, int qb) {
        bf16x8 A[3][L::KS], G[3][2];
        load_rows<L::KS>(A, stage + qb * 32 * L::XS + ax, L::XP);
        load_rows<2>(G, stage + qb * 32 * L::YS + ay, L::YP);
        S = f32x16{0}, D = f32x16{0};
        mul6<L::KS>(S, A, K);
        mul6_apart<2>(D, G, V);
    };
    scores(smem, 0);
    int c0 = 0, c1 = L::STAGE, c2 = 2 * L::STAGE;
    for (int tile = 0; tile < ntiles; ++tile) {
        const bf16_t *cur = smem + c0, *nxt = smem + c1;
#pragma unroll
        for (int qb = 0; qb < T / 32; ++qb) {
            const int q0 = tile * T + qb * 32;
            if (qb == 0) __syncthreads();
            if (q0 + 32 > g.N) rows::mask_rows(S, q0, g.N, hf);
            // rows of S are queries: register 4j + i belongs to query 8j + 4hf + i of the block
            const float *ex = (const float *)(cur + L::EX) + qb * 32 + 4 * hf;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 le = *(const float4 *)(ex + 8 * j), de = *(const float4 *)(ex + T + 8 * j);
                const float ls[4] = {le.x, le.y, le.z, le.w}, ds[4] = {de.x, de.y, de.z, de.w};
#pragma unroll
                for (int i = 4 * j; i < 4 * j + 4; ++i) {
                    S[i] = __builtin_amdgcn_exp2f(fmaf(S[i], kLog2e, -ls[i & 3]));
                    D[i] = S[i] * (D[i] - ds[i & 3]);
                }
            }
            bf16x8 B[3][2], A[3][2];
            split_block(B, S);
            RIB_FENCE();
            if (qb == 0) {
                commit<DA, T, true, true>(rg, g, smem + c2, g.scale_c, g.scale_p, wave, rn);
                request<DA, T, true>(rg, g, win, qs, tile + 3 < ntiles ? tile + 3 : ntiles - 1, wave, lu, du);
            }
            load_tr<L::YS>(A, cur + L::YR + qb * 32 * L::YS, L::YP, tro_y, 0);
            mul6_apart<2>(accV, A, B);
            split_block(B, D);
#pragma unroll
            for (int mb = 0; mb < L::RB; ++mb) {
                load_tr<L::XS>(A, cur + qb * 32 * L::XS, L::XP, tro_x, 32 * mb);
                mul6_apart<2>(accK[mb], A, B);
            }
            scores(qb + 1 < T / 32 ? cur : nxt, qb + 1 < T / 32 ? qb + 1 : 0);
            RIB_FENCE();
        }
        const int r0 = c0;
        c0 = c1, c1 = c2, c2 = r0;
    }
    if (__syncthreads_or(rn.outside())) {
        dkv_body<DA>(g, *(Smem<kXS> *)smem, u, row0, g.N, inv_r, q, k, v, fq, fk, dout, lse, delta, dk, dv, dfk_part);
        return;
    }
    if (n >= g.N) return;
#pragma unroll
    for (int mb = 0; mb < L::RB; ++mb)
        store_cols(accK[mb], mb, hf, g, 1.f, 1.f, dk + tn * g.C + hd * g.d, dfk_part + (u * g.N + n) * g.r);
    store_cols(accV, 0, hf, g, 1.f, 0.f, dv + tn * g.C + hd * g.d, nullptr);
}

// The backward of small grids (see Keys).
template <int NB, int QW, int G>
__device__ __forceinline__ bool add_groups(f32x16 (&acc)[NB], float *part, int wave, int lane)
{
    const int grp = wave / QW;
    if (grp > 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) part[((wave * NB + b) * 16 + i) * 64 + lane] = acc[b][i];
    }
    __syncthreads();
    if (grp > 0) return false;
#pragma unroll
    for (int j = 1; j < G; ++j)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][i] += part[(((wave + j * QW) * NB + b) * 16 + i) * 64 + lane];
    return true;
}

template <int DA>
__global__ __launch_bounds__(512, 2) void dq_keys_kernel(Geo g, int nblk, uint32_t inv_r, const float *__restrict__ q,
                                                         const float *__restrict__ k, const float *__restrict__ v,
                                                         const float *__restrict__ fq, const float *__restrict__ fk,
                                                         const float *__restrict__ dout, const float *__restrict__ lse,
                                                         const float *__restrict__ delta, float *__restrict__ dq,
                                                         float *__restrict__ dfq_part)
{
    using Z = Keys<DA>;
    constexpr int T = Z::T, NT = 512;
    RIB_SPLIT_SETUP((Z::template lds<kXS>()), blk * (32 * Z::QW), (wave % Z::QW))
    const int grp = wave / Z::QW;
    const int ax = col * L::XS + 8 * hf, ay = L::YR + col * L::YS + 8 * hf, tro_x = tr_lane_offset<L::XS>(lane);
    const Stream ks = {(const char *)(k + img * g.tstride + hd * g.d), (const char *)(v + img * g.tstride + hd * g.d),
                       (const char *)(fk + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.tstride * 4u,
                       (uint32_t)g.r * 4u};
    const Stream qs = {(const char *)(q + img * g.tstride + hd * g.d), (const char *)(dout + img * g.C + hd * g.d),
                       (const char *)(fq + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.C * 4u,
                       (uint32_t)g.r * 4u};
    const float lse2 = lse[u * g.N + nc] * kLog2e, dl = delta[u * g.N + nc];
    note_high(rn, lse2, dl);
    Regs<DA, T, NT> rg;
    bf16x8 Q[3][L::KS], G[3][2];
    {
        StatRegs<DA, true> sr;
        stat_request<DA, true>(sr, g, win, qs, row0 + (wave % Z::QW) * 32);
        request<DA, T, false, NT>(rg, g, win, ks, 0, wave, nullptr, nullptr);
        stat_stage<DA, true>(sr, g, smem + wave * stat_elems<DA>(), g.scale_c * kLog2e, g.scale_p * kLog2e, rn, Q, G);
    }
    __syncthreads();
    zero_pads<DA, T, 2>(g, smem);
    commit<DA, T, true, false, NT>(rg, g, smem, 1.f, 1.f, wave, rn);
    request<DA, T, false, NT>(rg, g, win, ks, ntiles > 1 ? 1 : 0, wave, nullptr, nullptr);

    f32x16 acc[L::RB];
#pragma unroll
    for (int mb = 0; mb < L::RB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[mb][i] = 0.f;
#pragma unroll 1
    for (int tile = 0; tile < ntiles; ++tile) {
        const bf16_t *cur = smem + (tile & 1) * L::STAGE;
        const int key0 = tile * T + grp * 32;
        __syncthreads();
        if (tile + 1 < ntiles) {
            commit<DA, T, true, false, NT>(rg, g, smem + ((tile + 1) & 1) * L::STAGE, 1.f, 1.f, wave, rn);
            request<DA, T, false, NT>(rg, g, win, ks, tile + 2 < ntiles ? tile + 2 : ntiles - 1, wave, nullptr, nullptr);
        }
        if (key0 >= g.N) continue;
        f32x16 S = {0}, D = {0};
        {
            bf16x8 A[3][L::KS], V[3][2];
            load_rows<L::KS>(A, cur + grp * 32 * L::XS + ax, L::XP);
            load_rows<2>(V, cur + grp * 32 * L::YS + ay, L::YP);
            mul6<L::KS>(S, A, Q);
            mul6_apart<2>(D, V, G);
        }
        if (key0 + 32 > g.N) rows::mask_rows(S, key0, g.N, hf);
#pragma unroll
        for (int i = 0; i < 16; ++i) S[i] = __builtin_amdgcn_exp2f(S[i] - lse2) * (D[i] - dl);
        bf16x8 B[3][2];
        split_block(B, S);
#pragma unroll
        for (int mb = 0; mb < L::RB; ++mb) {
            bf16x8 A[3][2];
            load_tr<L::XS>(A, cur + grp * 32 * L::XS, L::XP, tro_x, 32 * mb);
            mul6_apart<2>(acc[mb], A, B);
        }
    }
    if (__syncthreads_or(rn.outside())) {
        dq_body<DA>(g, *(Smem<kXS> *)smem, u, row0, row0 + 32 * Z::QW, inv_r, q, k, v, fq, fk, dout, lse, delta, dq, dfq_part);
        return;
    }
    if (!add_groups<L::RB, Z::QW, Z::G>(acc, (float *)smem, wave, lane) || n >= g.N) return;
#pragma unroll
    for (int mb = 0; mb < L::RB; ++mb)
        store_cols(acc[mb], mb, hf, g, g.scale_c, g.scale_p, dq + tn * g.C + hd * g.d, dfq_part + (u * g.N + n) * g.r);
}

template <int DA>
__global__ __launch_bounds__(512, 2) void dkv_keys_kernel(Geo g, int nblk, uint32_t inv_r, const float *__restrict__ q,
                                                          const float *__restrict__ k, const float *__restrict__ v,
                                                          const float *__restrict__ fq, const float *__restrict__ fk,
                                                          const float *__restrict__ dout, const float *__restrict__ lse,
                                                          const float *__restrict__ delta, float *__restrict__ dk,
                                                          float *__restrict__ dv, float *__restrict__ dfk_part)
{
    using Z = Keys<DA>;
    constexpr int T = Z::T, NT = 512;
    RIB_SPLIT_SETUP((Z::template lds<kXS>()), blk * (32 * Z::QW), (wave % Z::QW))
    const int grp = wave / Z::QW;
    const int ax = col * L::XS + 8 * hf, ay = L::YR + col * L::YS + 8 * hf, tro_x = tr_lane_offset<L::XS>(lane),
              tro_y = tr_lane_offset<L::YS>(lane);
    const Stream qs = {(const char *)(q + img * g.tstride + hd * g.d), (const char *)(dout + img * g.C + hd * g.d),
                       (const char *)(fq + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.C * 4u,
                       (uint32_t)g.r * 4u};
    const float *lu = lse + u * g.N, *du = delta + u * g.N;
    const Stream ks = {(const char *)(k + img * g.tstride + hd * g.d), (const char *)(v + img * g.tstride + hd * g.d),
                       (const char *)(fk + (int64_t)hd * g.N * g.r), (uint32_t)g.tstride * 4u, (uint32_t)g.tstride * 4u,
                       (uint32_t)g.r * 4u};
    Regs<DA, T, NT> rg;
    bf16x8 K[3][L::KS], V[3][2];
    {
        StatRegs<DA, true> sr;
        stat_request<DA, true>(sr, g, win, ks, row0 + (wave % Z::QW) * 32);
        request<DA, T, true, NT>(rg, g, win, qs, 0, wave, lu, du);
        stat_stage<DA, true>(sr, g, smem + wave * stat_elems<DA>(), 1.f, 1.f, rn, K, V);
    }
    __syncthreads();
    zero_pads<DA, T, 2>(g, smem);
    commit<DA, T, true, true, NT>(rg, g, smem, g.scale_c, g.scale_p, wave, rn);
    request<DA, T, true, NT>(rg, g, win, qs, ntiles > 1 ? 1 : 0, wave, lu, du);

    f32x16 acc[L::RB + 1];          // dK_aug^T, then dV^T
#pragma unroll
    for (int mb = 0; mb <= L::RB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[mb][i] = 0.f;
#pragma unroll 1
    for (int tile = 0; tile < ntiles; ++tile) {
        const bf16_t *cur = smem + (tile & 1) * L::STAGE;
        const int q0 = tile * T + grp * 32;
        __syncthreads();
        if (tile + 1 < ntiles) {
            commit<DA, T, true, true, NT>(rg, g, smem + ((tile + 1) & 1) * L::STAGE, g.scale_c, g.scale_p, wave, rn);
            request<DA, T, true, NT>(rg, g, win, qs, tile + 2 < ntiles ? tile + 2 : ntiles - 1, wave, lu, du);
        }
        if (q0 >= g.N) continue;
        f32x16 S = {0}, D = {0};
        {
            bf16x8 A[3][L::KS], G[3][2];
            load_rows<L::KS>(A, cur + grp * 32 * L::XS + ax, L::XP);
            load_rows<2>(G, cur + grp * 32 * L::YS + ay, L::YP);
            mul6<L::KS>(S, A, K);
            mul6_apart<2>(D, G, V);
        }
        if (q0 + 32 > g.N) rows::mask_rows(S, q0, g.N, hf);
        // rows of S are queries: register 4j + i belongs to query 8j + 4hf + i of the block
        const float *ex = (const float *)(cur + L::EX) + grp * 32 + 4 * hf;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float4 le = *(const float4 *)(ex + 8 * j), de = *(const float4 *)(ex + T + 8 * j);
            const float ls[4] = {le.x, le.y, le.z, le.w}, ds[4] = {de.x, de.y, de.z, de.w};
#pragma unroll
            for (int i = 4 * j; i < 4 * j + 4; ++i) {
                S[i] = __builtin_amdgcn_exp2f(fmaf(S[i], kLog2e, -ls[i & 3]));
                D[i] = S[i] * (D[i] - ds[i & 3]);
            }
        }
        bf16x8 B[3][2], A[3][2];
        split_block(B, S);
        load_tr<L::YS>(A, cur + L::YR + grp * 32 * L::YS, L::YP, tro_y, 0);
        mul6_apart<2>(acc[L::RB], A, B);
        split_block(B, D);
#pragma unroll
        for (int mb = 0; mb < L::RB; ++mb) {
            load_tr<L::XS>(A, cur + grp * 32 * L::XS, L::XP, tro_x, 32 * mb);
            mul6_apart<2>(acc[mb], A, B);
        }
    }
    if (__syncthreads_or(rn.outside())) {
        dkv_body<DA>(g, *(Smem<kXS> *)smem, u, row0, row0 + 32 * Z::QW, inv_r, q, k, v, fq, fk, dout, lse, delta, dk, dv, dfk_part);
        return;
    }
    if (!add_groups<L::RB + 1, Z::QW, Z::G>(acc, (float *)smem, wave, lane) || n >= g.N) return;
#pragma unroll
    for (int mb = 0; mb < L::RB; ++mb)
        store_cols(acc[mb], mb, hf, g, 1.f, 1.f, dk + tn * g.C + hd * g.d, dfk_part + (u * g.N + n) * g.r);
    store_cols(acc[L::RB], 0, hf, g, 1.f, 0.f, dv + tn * g.C + hd * g.d, nullptr);
}

}  // namespace split
}  // namespace
}  // namespace rib

// RIB feature generator (paper Sec. 3.1 Eq. 1-3) and its backward.
//
// The work is tiny next to the attention it feeds (N <= 65536 tokens, 42 -> 32 -> heads*r
// features) and runs once per weight update: plain vector-ALU kernels with a fixed summation
// order.  What bounds them is latency -- a handful of workgroups, each a chain of fp64 sincos,
// dot products and loads -- so a workgroup takes only 16 tokens, every sincos and every hidden
// unit has a lane of its own, and operands are staged in bulk (48 x 48 window, 3 heads, r = 16:
// forward 31 -> 12 us, backward 120 -> 25 us; 64 tokens a workgroup and strided global reads before).
//
//   forward:  Fourier features (fp64 sines / cosines of the token's row and column coordinate,
//             rounded to fp32) into LDS, the shared hidden layer into LDS, then a lane per
//             (table, head, column) runs over the 16 tokens.
//   backward: (1) the same two stages, kept in the workspace (r_in, h) together with
//             dpre = ReLU'(pre) * sum over heads of dF W_p^T;
//             (2) per 256-token chunk, (table, head) and 8 to 32 hidden units, a workgroup sums its slice
//             of the weight gradients from LDS tiles, four lanes an element;
//             (3) chunks are added in ascending order.
#include <hip/hip_runtime.h>

#include "rib_common.h"

namespace rib {
namespace {

constexpr int kTok = 16;        // tokens per workgroup in the token-parallel kernels
constexpr int kChunk = 256;     // tokens per partial sum in the weight-gradient kernel
constexpr int kGenNT = 256;
constexpr int kStageFloats = 12 * 1024;     // LDS for the staged dF and W_p tiles of a group of heads

struct Gen {
    int M, N, heads, r, L, d_h, n_in;
};

// Fourier features of the workgroup's tokens -> rin[kTok][n_in] (LDS).  One lane per (token, axis,
// band): coordinate and sine / cosine in fp64.
__device__ __forceinline__ void stage_fourier(const Gen &g, int n0, float *rin)
{
    for (int e = threadIdx.x; e < kTok * 2 * (g.L + 1); e += kGenNT) {
        const int t = e & (kTok - 1), la = e / kTok, axis = la & 1, l = (la >> 1) - 1, n = n0 + t;
        if (n >= g.N) continue;
        const int iy = n / g.M, ix = n - iy * g.M;
        const int i = axis == 0 ? iy : ix;
        const double x = g.M > 1 ? -1.0 + 2.0 * (double)i / (double)(g.M - 1) : 0.0;
        float *row = rin + t * g.n_in;
        if (l < 0) {
            row[axis] = (float)x;
        } else {
            double s, c;
            sincos((double)(1 << l) * x, &s, &c);
            row[2 + 4 * l + axis] = (float)s;
            row[4 + 4 * l + axis] = (float)c;
        }
    }
}

// pre-activation of the shared hidden layer for (token t, unit c): r_in[t] . W_h[:, c] + b_h[c]
__device__ __forceinline__ float hidden_pre(const Gen &g, const float *rin_row, const float *__restrict__ W_h,
                                            const float *__restrict__ b_h, int c)
{
    float acc = b_h[c];
#pragma unroll 6
    for (int a = 0; a < g.n_in; ++a) acc = fmaf(rin_row[a], W_h[a * g.d_h + c], acc);
    return acc;
}

template <typename T>
__global__ __launch_bounds__(kGenNT) void features_fwd_kernel(Gen g, const float *__restrict__ W_h,
                                                              const float *__restrict__ b_h,
                                                              const float *__restrict__ W_pq,
                                                              const float *__restrict__ W_pk, T *__restrict__ f_q,
                                                              T *__restrict__ f_k)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float *hs = lds, *rin = lds + kTok * g.d_h;     // h transposed: [d_h][kTok]
    const int n0 = blockIdx.x * kTok;
    const int live = min(kTok, g.N - n0);
    stage_fourier(g, n0, rin);
    __syncthreads();
    for (int e = threadIdx.x; e < kTok * g.d_h; e += kGenNT) {
        const int t = e / g.d_h, c = e - t * g.d_h;
        hs[c * kTok + t] = t < live ? fmaxf(hidden_pre(g, rin + t * g.n_in, W_h, b_h, c), 0.f) : 0.f;
    }
    __syncthreads();
    const int cols = g.heads * g.r;
    for (int e = blockIdx.y * kGenNT + threadIdx.x; e < 2 * cols; e += gridDim.y * kGenNT) {
        const int which = e >= cols, ee = e - which * cols, hd = ee / g.r, j = ee - hd * g.r;
        const float *W = (which ? W_pk : W_pq) + (size_t)hd * g.d_h * g.r + j;
        float acc[kTok];
#pragma unroll
        for (int t = 0; t < kTok; ++t) acc[t] = 0.f;
#pragma unroll 4
        for (int c = 0; c < g.d_h; ++c) {
            const float w = W[c * g.r];
            const float4 *h = (const float4 *)(hs + c * kTok);
#pragma unroll
            for (int i = 0; i < kTok / 4; ++i) {
                const float4 v = h[i];
                acc[4 * i] = fmaf(v.x, w, acc[4 * i]);
                acc[4 * i + 1] = fmaf(v.y, w, acc[4 * i + 1]);
                acc[4 * i + 2] = fmaf(v.z, w, acc[4 * i + 2]);
                acc[4 * i + 3] = fmaf(v.w, w, acc[4 * i + 3]);
            }
        }
        T *dst = (which ? f_k : f_q) + ((size_t)hd * g.N + n0) * g.r + j;
#pragma unroll
        for (int t = 0; t < kTok; ++t)
            if (t < live) store_as(dst + t * g.r, acc[t]);
    }
}

// Backward stage 1: r_in, h and dpre of every token into the workspace.  The dF rows and W_p slices
// of as many heads as fit are staged in LDS at a time, with one round of loads in flight.
__global__ __launch_bounds__(kGenNT) void features_hidden_kernel(Gen g, int group, const float *__restrict__ W_h,
                                                                 const float *__restrict__ b_h,
                                                                 const float *__restrict__ W_pq,
                                                                 const float *__restrict__ W_pk,
                                                                 const float *__restrict__ df_q,
                                                                 const float *__restrict__ df_k, float *__restrict__ ws_rin,
                                                                 float *__restrict__ ws_h, float *__restrict__ ws_dpre)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int ws = g.r | 1;                             // odd row stride: the lanes of a read are consecutive units
    float *rin = lds, *gs = lds + kTok * g.n_in, *wl = gs + 2 * group * kTok * g.r;
    const int n0 = blockIdx.x * kTok;
    const int live = min(kTok, g.N - n0);
    stage_fourier(g, n0, rin);
    constexpr int kPer = kTok * 64 / kGenNT;            // (token, unit) pairs per lane, d_h <= 64
    float dh[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) dh[i] = 0.f;
    for (int h0 = 0; h0 < g.heads; h0 += group) {
        const int nh = min(group, g.heads - h0);
        __syncthreads();
        // gs[(2*head + which)][t][j], wl[(2*head + which)][c][j]
        const int grow = live * g.r;
        for (int s = 0; s < 2 * nh; ++s) {
            const float *src = ((s & 1) ? df_k : df_q) + ((size_t)(h0 + (s >> 1)) * g.N + n0) * g.r;
            for (int e = threadIdx.x; e < grow; e += kGenNT) gs[s * kTok * g.r + e] = src[e];
            const float *w = ((s & 1) ? W_pk : W_pq) + (size_t)(h0 + (s >> 1)) * g.d_h * g.r;
            for (int e = threadIdx.x; e < g.d_h * g.r; e += kGenNT) {
                const int c = e / g.r;
                wl[(s * g.d_h + c) * ws + (e - c * g.r)] = w[e];
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = i * kGenNT + threadIdx.x;
            if (e >= live * g.d_h) break;
            const int t = e / g.d_h, c = e - t * g.d_h;
            float acc = dh[i];
            for (int s = 0; s < 2 * nh; ++s) {
                const float *gr = gs + (s * kTok + t) * g.r, *wr = wl + (s * g.d_h + c) * ws;
#pragma unroll 8
                for (int j = 0; j < g.r; ++j) acc = fmaf(gr[j], wr[j], acc);
            }
            dh[i] = acc;
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < live * g.n_in; e += kGenNT) ws_rin[(size_t)n0 * g.n_in + e] = rin[e];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = i * kGenNT + threadIdx.x;
        if (e >= live * g.d_h) break;
        const int t = e / g.d_h, c = e - t * g.d_h;
        const float pre = hidden_pre(g, rin + t * g.n_in, W_h, b_h, c);
        ws_h[(size_t)n0 * g.d_h + e] = fmaxf(pre, 0.f);
        ws_dpre[(size_t)n0 * g.d_h + e] = pre > 0.f ? dh[i] : 0.f;
    }
}

// Gradient elements in one flat index space:
//   [0, P)            dW_pq[hd][c][j]   = sum_n h[n][c]    dF_q[hd][n][j]       P = heads*d_h*r
//   [P, 2P)           dW_pk
//   [2P, 2P + I)      dW_h[a][c]        = sum_n r_in[n][a] dpre[n][c]           I = n_in*d_h
//   [2P + I, .. + d_h) db_h[c]          = sum_n dpre[n][c]
__device__ __forceinline__ int n_grad_elems(const Gen &g) { return 2 * g.heads * g.d_h * g.r + g.n_in * g.d_h + g.d_h; }

// Backward stage 2: partial[chunk][e] = the sum over the chunk's tokens.  blockIdx.x names the slice:
// (table, head) and 8 * RPL hidden units -> those rows of its [d_h][r] block of dW_p, from h and dF;
// behind those, 8 * RPL input features -> rows of dW_h from r_in and dpre (the first one also db_h).
// The chunk's rows of both factors are staged in LDS with the tokens contiguous (zeros past the end).
// Four lanes share an element, 64 tokens each in ascending order, and their sums are added in ascending
// order, so that the scratch holds one partial per 256 tokens and the critical path is that of 64.
// What bounds it is the LDS bandwidth of a CU: small slices for few tokens, several rows a lane for many.
constexpr int kQuarter = kChunk / 4;
// Floats ahead of row `c` of a staged factor, and of its token `t`: the 16 lanes of a 16-byte read (four
// quarters of four rows) fall on different banks, and so do the writes of 16 rows.
__host__ __device__ inline int factor_row(int c) { return c * 4 * (kQuarter + 4) + (c >> 2) * 4; }
__device__ __forceinline__ int factor_token(int t) { return t + (t / kQuarter) * 4; }
__device__ __forceinline__ float add_quarters(float x)
{
    const int base = (int)(threadIdx.x & 63) & ~3;      // every lane of the four: ((s0 + s1) + s2) + s3
    return ((__shfl(x, base) + __shfl(x, base + 1)) + __shfl(x, base + 2)) + __shfl(x, base + 3);
}
// RPL: rows a lane sums at once, 8 * RPL rows a slice.
template <int RPL>
constexpr int grad_threads() { return RPL == 4 ? 1024 : 512; }
template <int RPL>
__global__ __launch_bounds__(grad_threads<RPL>()) void features_wgrad_kernel(Gen g, const float *__restrict__ df_q,
                                                                 const float *__restrict__ df_k,
                                                                 const float *__restrict__ ws_rin,
                                                                 const float *__restrict__ ws_h,
                                                                 const float *__restrict__ ws_dpre, float *__restrict__ partial)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    constexpr int rows = 8 * RPL, kGradNT = grad_threads<RPL>();
    const int total = n_grad_elems(g), P = g.heads * g.d_h * g.r, I = g.n_in * g.d_h;
    const int per = (g.d_h + rows - 1) / rows, np = 2 * g.heads * per;
    const bool wh = (int)blockIdx.x >= np;
    const int slice = blockIdx.x / per, which = slice >= g.heads, hd = slice - which * g.heads;
    const int row0 = (wh ? blockIdx.x - np : blockIdx.x - slice * per) * rows;
    const int wa = wh ? g.n_in : g.d_h, ra = min(rows, wa - row0), cb = wh ? g.d_h : g.r, count = min(ra, 8) * cb;
    const float *a = wh ? ws_rin : ws_h, *b = wh ? ws_dpre : (which ? df_k : df_q) + (size_t)hd * g.N * g.r;
    float *as = lds, *bs = lds + factor_row(rows);
    const int n0 = blockIdx.y * kChunk, nt = min(kChunk, g.N - n0);
    for (int e = threadIdx.x; e < kChunk * rows; e += kGradNT) {
        const int t = e / rows, c = e % rows;
        as[factor_row(c) + factor_token(t)] = t < nt && c < ra ? a[(size_t)(n0 + t) * wa + row0 + c] : 0.f;
    }
    for (int e = threadIdx.x; e < kChunk * cb; e += kGradNT) {
        const int t = e / cb;
        bs[factor_row(e - t * cb) + factor_token(t)] = t < nt ? b[(size_t)n0 * cb + e] : 0.f;
    }
    __syncthreads();
    float *dst = partial + (size_t)blockIdx.y * total + (wh ? 2 * P : which * P + hd * g.d_h * g.r) + row0 * cb;
    const int part = threadIdx.x & 3, first = threadIdx.x >> 2;
    // (a lane past the end sums the last element again: all lanes meet in add_quarters)
    for (int e0 = 0; e0 < count; e0 += kGradNT / 4) {
        const int e = min(e0 + first, count - 1), i = e / cb;
        const float *x = as + factor_row(i) + factor_token(part * kQuarter);
        const float4 *y = (const float4 *)(bs + factor_row(e - i * cb) + factor_token(part * kQuarter));
        float acc[RPL];
#pragma unroll
        for (int k = 0; k < RPL; ++k) acc[k] = 0.f;
#pragma unroll 8 / RPL
        for (int t = 0; t < kQuarter / 4; ++t) {
            const float4 v = y[t];
#pragma unroll
            for (int k = 0; k < RPL; ++k) {
                const float4 u = ((const float4 *)(x + factor_row(8 * k)))[t];
                acc[k] = fmaf(u.x, v.x, acc[k]);
                acc[k] = fmaf(u.y, v.y, acc[k]);
                acc[k] = fmaf(u.z, v.z, acc[k]);
                acc[k] = fmaf(u.w, v.w, acc[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            const float sum = add_quarters(acc[k]);
            if (part == 0 && e0 + first < count && i + 8 * k < ra) dst[e + 8 * k * cb] = sum;
        }
    }
    if (wh && row0 == 0) {
        const int c = min(first, g.d_h - 1);
        const float4 *y = (const float4 *)(bs + factor_row(c) + factor_token(part * kQuarter));
        float acc = 0.f;
#pragma unroll
        for (int t = 0; t < kQuarter / 4; ++t) {
            const float4 v = y[t];
            acc += v.x;
            acc += v.y;
            acc += v.z;
            acc += v.w;
        }
        acc = add_quarters(acc);
        if (part == 0 && first < g.d_h) dst[I + first] = acc;
    }
}

// Backward stage 3: chunks ascending, scattered to the four gradient tensors.
__global__ __launch_bounds__(kGenNT) void features_reduce_kernel(Gen g, int nchunks, const float *__restrict__ partial,
                                                                 float *__restrict__ dW_h, float *__restrict__ db_h,
                                                                 float *__restrict__ dW_pq, float *__restrict__ dW_pk)
{
    const int e = blockIdx.x * kGenNT + threadIdx.x, total = n_grad_elems(g);
    if (e >= total) return;
    float acc = 0.f;
#pragma unroll 8
    for (int ch = 0; ch < nchunks; ++ch) acc += partial[(size_t)ch * total + e];
    const int P = g.heads * g.d_h * g.r, I = g.n_in * g.d_h;
    if (e < P) dW_pq[e] = acc;
    else if (e < 2 * P) dW_pk[e - P] = acc;
    else if (e < 2 * P + I) dW_h[e - 2 * P] = acc;
    else db_h[e - 2 * P - I] = acc;
}

bool make_gen(const rib_gen_params *p, Gen *g, rib_status *st)
{
    if (p == nullptr) return *st = RIB_ERR_NULL, false;
    if (p->window < 1 || p->window > 256 || p->heads < 1 || p->heads > 64 || p->r < 1 || p->r > 64 || p->L < 0 ||
        p->L > 16 || p->d_h < 1 || p->d_h > 64)
        return *st = RIB_ERR_SHAPE, false;
    if (p->dtype != RIB_F32 && p->dtype != RIB_BF16) return *st = RIB_ERR_DTYPE, false;
    g->M = p->window, g->N = p->window * p->window, g->heads = p->heads, g->r = p->r, g->L = p->L, g->d_h = p->d_h;
    g->n_in = 2 + 4 * p->L;
    return *st = RIB_OK, true;
}

struct GenWs {
    size_t rin_off, h_off, dpre_off, partial_off, total;
    int nchunks;
};

GenWs gen_ws_layout(const Gen &g)
{
    auto up = [](size_t x) { return (x + 255) / 256 * 256; };
    GenWs l;
    l.nchunks = (g.N + kChunk - 1) / kChunk;
    const size_t elems = (size_t)2 * g.heads * g.d_h * g.r + (size_t)g.n_in * g.d_h + g.d_h;
    l.rin_off = 0;
    l.h_off = up((size_t)g.N * g.n_in * 4);
    l.dpre_off = l.h_off + up((size_t)g.N * g.d_h * 4);
    l.partial_off = l.dpre_off + up((size_t)g.N * g.d_h * 4);
    l.total = l.partial_off + up((size_t)l.nchunks * elems * 4);
    return l;
}

int grad_slices(const Gen &g, int rows) { return 2 * g.heads * ((g.d_h + rows - 1) / rows) + (g.n_in + rows - 1) / rows; }
template <int RPL>
hipError_t launch_wgrad(const Gen &g, int nchunks, const float *df_q, const float *df_k, const float *ws_rin, const float *ws_h,
                        const float *ws_dpre, float *partial, hipStream_t s)
{
    auto kern = features_wgrad_kernel<RPL>;
    const hipError_t e = prepare_kernel((const void *)kern, nullptr);
    if (e != hipSuccess) return e;
    const int cols = g.d_h > g.r ? g.d_h : g.r;
    const size_t lds = (size_t)(factor_row(8 * RPL) + factor_row((cols + 3) & ~3)) * sizeof(float);
    hipLaunchKernelGGL(kern, dim3((unsigned)grad_slices(g, 8 * RPL), (unsigned)nchunks), dim3(grad_threads<RPL>()), lds, s, g, df_q,
                       df_k, ws_rin, ws_h, ws_dpre, partial);
    return hipGetLastError();
}

}  // namespace
}  // namespace rib

using namespace rib;

extern "C" {

rib_status rib_features_fwd(const rib_gen_params *p, const float *W_h, const float *b_h, const float *W_pq,
                            const float *W_pk, void *f_q, void *f_k, void *stream)
{
    Gen g;
    rib_status st;
    if (!make_gen(p, &g, &st)) return st;
    if (!W_h || !b_h || !W_pq || !W_pk || !f_q || !f_k) return RIB_ERR_NULL;
    // a second grid dimension where a workgroup's columns would take several turns
    const dim3 grid((unsigned)((g.N + kTok - 1) / kTok), (unsigned)((2 * g.heads * g.r + kGenNT - 1) / kGenNT)), block(kGenNT);
    const size_t lds = (size_t)kTok * (g.n_in + g.d_h) * sizeof(float);
    hipStream_t s = (hipStream_t)stream;
    if (p->dtype == RIB_BF16)
        hipLaunchKernelGGL(features_fwd_kernel<bf16_t>, grid, block, lds, s, g, W_h, b_h, W_pq, W_pk, (bf16_t *)f_q,
                           (bf16_t *)f_k);
    else
        hipLaunchKernelGGL(features_fwd_kernel<float>, grid, block, lds, s, g, W_h, b_h, W_pq, W_pk, (float *)f_q,
                           (float *)f_k);
    return hipGetLastError() == hipSuccess ? RIB_OK : RIB_ERR_LAUNCH;
}

size_t rib_features_bwd_workspace_bytes(const rib_gen_params *p)
{
    Gen g;
    rib_status st;
    if (!make_gen(p, &g, &st)) return 0;
    return gen_ws_layout(g).total;
}

rib_status rib_features_bwd(const rib_gen_params *p, const float *W_h, const float *b_h, const float *W_pq,
                            const float *W_pk, const float *df_q, const float *df_k, float *dW_h, float *db_h,
                            float *dW_pq, float *dW_pk, void *workspace, size_t workspace_bytes, void *stream)
{
    Gen g;
    rib_status st;
    if (!make_gen(p, &g, &st)) return st;
    if (!W_h || !b_h || !W_pq || !W_pk || !df_q || !df_k || !dW_h || !db_h || !dW_pq || !dW_pk) return RIB_ERR_NULL;
    const GenWs l = gen_ws_layout(g);
    if (!workspace || ((uintptr_t)workspace & 255) != 0 || workspace_bytes < l.total) return RIB_ERR_WORKSPACE;
    char *ws = (char *)workspace;
    float *ws_rin = (float *)(ws + l.rin_off), *ws_h = (float *)(ws + l.h_off), *ws_dpre = (float *)(ws + l.dpre_off),
          *partial = (float *)(ws + l.partial_off);
    hipStream_t s = (hipStream_t)stream;
    const int total = 2 * g.heads * g.d_h * g.r + g.n_in * g.d_h + g.d_h;
    // heads staged at a time (at least one: 2 * (16 + 64) rows of up to 65 floats)
    const int per_head = 2 * (kTok * g.r + g.d_h * (g.r | 1));
    const int group = per_head * g.heads <= kStageFloats ? g.heads : per_head <= kStageFloats ? kStageFloats / per_head : 1;
    hipLaunchKernelGGL(features_hidden_kernel, dim3((unsigned)((g.N + kTok - 1) / kTok)), dim3(kGenNT),
                       ((size_t)kTok * g.n_in + (size_t)group * per_head) * sizeof(float), s, g, group, W_h, b_h, W_pq, W_pk,
                       df_q, df_k, ws_rin, ws_h, ws_dpre);
    if (hipGetLastError() != hipSuccess) return RIB_ERR_LAUNCH;
    const unsigned eb = (unsigned)((total + kGenNT - 1) / kGenNT);
    // Rows a lane: more of them read less LDS a product, but make fewer workgroups.  (Whole backward, us, with
    // 1 / 2 / 4, 6 heads, r = 16: 48 x 48 window, 3 heads, 270 slices of 8 rows 24.9 / 26.4 / 29.6; 64 x 64, 864
    // slices 34.4 / 32.6 / 34.9; 96 x 96, 1944 slices 54.7 / 50.5 / 45.5.)
    const int64_t slices = (int64_t)grad_slices(g, 8) * l.nchunks;
    const hipError_t e = slices <= 512    ? launch_wgrad<1>(g, l.nchunks, df_q, df_k, ws_rin, ws_h, ws_dpre, partial, s)
                         : slices <= 1024 ? launch_wgrad<2>(g, l.nchunks, df_q, df_k, ws_rin, ws_h, ws_dpre, partial, s)
                                          : launch_wgrad<4>(g, l.nchunks, df_q, df_k, ws_rin, ws_h, ws_dpre, partial, s);
    if (e != hipSuccess) return RIB_ERR_LAUNCH;
    hipLaunchKernelGGL(features_reduce_kernel, dim3(eb), dim3(kGenNT), 0, s, g, l.nchunks, partial, dW_h, db_h, dW_pq, dW_pk);
    return hipGetLastError() == hipSuccess ? RIB_OK : RIB_ERR_LAUNCH;
}

}  // extern "C"

// General-shape RIB window attention on the vector ALU (fp32 arithmetic).
//
// Serves fp32 problems and every bf16 problem the matrix-core kernels are not
// built for (odd head dims, tiny or non-power-of-two windows).  Same operator as
// include/rib_attn.h describes (paper Sec. 2.2; Sec. 3.1 Eq. 5-6): the augmented
// vectors Q_aug = [scale_c q || scale_p f_q], K_aug = [k || f_k] are assembled in
// registers / LDS while the window's tokens are gathered through the cyclic
// shift, logits are one dot product of the augmented vectors, and the softmax is
// computed online so no N x N matrix exists anywhere.
//
// Thread mapping: a workgroup of 256 lanes owns 64 consecutive window-local rows
// of one (window, head) unit; 4 neighbouring lanes share a row and split the
// key (or query) tile between them, merging their partial softmax states with
// lane shuffles at the end.  K_aug / V tiles of 64 tokens are staged in LDS.
#include "rib_common.h"

namespace rib {
namespace {

constexpr int kThreads = 256;
constexpr int kSplit = 4;                    // lanes per row
constexpr int kRows = kThreads / kSplit;     // rows per workgroup
constexpr int kTile = 64;                    // tokens staged per LDS tile
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Stage one tile of augmented vectors [kTile][DA] (content scaled by sc, RIB part
// by sp) and optionally a tile of a second grid tensor [kTile][DV] into LDS.
template <typename T, int DA, int DV>
__device__ __forceinline__ void stage_tile(const Geo &g, int w, int hd, int j0,
                                           const T *__restrict__ x, const T *__restrict__ f, float sc, float sp,
                                           int64_t xstride, const T *__restrict__ y, int64_t ystride,
                                           float (*A)[DA + 1], float (*Y)[DV + 1], int64_t *tok)
{
    const int tid = threadIdx.x;
    if (tid < kTile) {
        int j = j0 + tid;
        tok[tid] = j < g.N ? grid_token(g, w, j) : -1;
    }
    __syncthreads();
    for (int idx = tid; idx < kTile * DA; idx += kThreads) {
        int jj = idx / DA, t = idx - jj * DA;
        int64_t tk = tok[jj];
        float val = 0.f;
        if (tk >= 0) {
            if (t < g.d) val = widen(x[tk * xstride + hd * g.d + t]) * sc;
            else if (t < g.d + g.r) val = widen(f[((int64_t)hd * g.N + (j0 + jj)) * g.r + (t - g.d)]) * sp;
        }
        A[jj][t] = val;
    }
    if (y != nullptr) {
        for (int idx = tid; idx < kTile * DV; idx += kThreads) {
            int jj = idx / DV, t = idx - jj * DV;
            int64_t tk = tok[jj];
            float val = 0.f;
            if (tk >= 0 && t < g.d) val = widen(y[tk * ystride + hd * g.d + t]);
            Y[jj][t] = val;
        }
    }
}

// This lane's copy of a row's augmented vector.
template <typename T, int DA>
__device__ __forceinline__ void load_aug(const Geo &g, int hd, int n, int64_t tk, const T *__restrict__ x,
                                         const T *__restrict__ f, float sc, float sp, int64_t xstride, float *a)
{
#pragma unroll
    for (int t = 0; t < DA; ++t) {
        float val = 0.f;
        if (t < g.d) val = widen(x[tk * xstride + hd * g.d + t]) * sc;
        else if (t < g.d + g.r) val = widen(f[((int64_t)hd * g.N + n) * g.r + (t - g.d)]) * sp;
        a[t] = val;
    }
}

template <typename T, int DA, int DV>
__global__ __launch_bounds__(kThreads) void valu_fwd_kernel(Geo g, int nblk, const T *__restrict__ q,
                                                            const T *__restrict__ k, const T *__restrict__ v,
                                                            const T *__restrict__ fq, const T *__restrict__ fk,
                                                            T *__restrict__ out, float *__restrict__ lse)
{
    __shared__ float Ks[kTile][DA + 1];
    __shared__ float Vs[kTile][DV + 1];
    __shared__ int64_t tok[kTile];

    const int64_t u = blockIdx.x / nblk;
    const int blk = blockIdx.x - (int)(u * nblk);
    const int w = (int)(u / g.heads), hd = (int)(u - (int64_t)w * g.heads);
    const int tid = threadIdx.x, row = tid / kSplit, part = tid % kSplit;
    const int i = blk * kRows + row;
    const bool live = i < g.N;
    const int ic = live ? i : g.N - 1;
    const int64_t tq = grid_token(g, w, ic);

    float qa[DA];
    load_aug<T, DA>(g, hd, ic, tq, q, fq, g.scale_c * kLog2e, g.scale_p * kLog2e, g.tstride, qa);

    float m = -INFINITY, l = 0.f, o[DV];
#pragma unroll
    for (int t = 0; t < DV; ++t) o[t] = 0.f;

    constexpr int KC = 4;  // keys scored before one rescale
    for (int j0 = 0; j0 < g.N; j0 += kTile) {
        __syncthreads();
        stage_tile<T, DA, DV>(g, w, hd, j0, k, fk, 1.f, 1.f, g.tstride, v, g.tstride, Ks, Vs, tok);
        __syncthreads();
        for (int c = 0; c < kTile / (kSplit * KC); ++c) {
            float s[KC], mx = m;
#pragma unroll
            for (int e = 0; e < KC; ++e) {
                int jj = (c * KC + e) * kSplit + part;
                float acc = 0.f;
#pragma unroll
                for (int t = 0; t < DA; ++t) acc = fmaf(qa[t], Ks[jj][t], acc);
                s[e] = (j0 + jj < g.N) ? acc : -INFINITY;
                mx = fmaxf(mx, s[e]);
            }
            if (mx == -INFINITY) continue;
            float alpha = exp2f(m - mx);
            l *= alpha;
#pragma unroll
            for (int t = 0; t < DV; ++t) o[t] *= alpha;
#pragma unroll
            for (int e = 0; e < KC; ++e) {
                int jj = (c * KC + e) * kSplit + part;
                float p = exp2f(s[e] - mx);
                l += p;
#pragma unroll
                for (int t = 0; t < DV; ++t) o[t] = fmaf(p, Vs[jj][t], o[t]);
            }
            m = mx;
        }
    }
    // merge the kSplit partial states of this row
#pragma unroll
    for (int off = 1; off < kSplit; off <<= 1) {
        float m2 = __shfl_xor(m, off), l2 = __shfl_xor(l, off);
        float mx = fmaxf(m, m2);
        float a = (m == -INFINITY) ? 0.f : exp2f(m - mx);
        float a2 = (m2 == -INFINITY) ? 0.f : exp2f(m2 - mx);
        l = l * a + l2 * a2;
#pragma unroll
        for (int t = 0; t < DV; ++t) o[t] = o[t] * a + __shfl_xor(o[t], off) * a2;
        m = mx;
    }
    if (!live) return;
    const float inv = 1.f / l;
    T *dst = out + tq * g.C + hd * g.d;
    if (g.gate == nullptr) {
#pragma unroll
        for (int t = 0; t < DV; ++t)
            if (t % kSplit == part && t < g.d) store_as(dst + t, o[t] * inv);
    } else {    // CLA gate (Eq. 9) on the way out, the raw O beside it if asked for
        const T *gt = (const T *)g.gate + tq * g.C + hd * g.d;
        T *raw = g.out_raw ? (T *)g.out_raw + tq * g.C + hd * g.d : nullptr;
#pragma unroll
        for (int t = 0; t < DV; ++t)
            if (t % kSplit == part && t < g.d) {
                store_as(dst + t, o[t] * inv * widen(gt[t]));
                if (raw) store_as(raw + t, o[t] * inv);
            }
    }
    if (lse != nullptr && part == 0) lse[u * g.N + i] = (m + log2f(l)) * kLn2;
}

// delta[u][i] = dO[i] . O[i] over the head's channels.  Sixteen lanes share one
// (token, head): consecutive groups are the heads of one token, so a wave reads whole
// contiguous token rows of O and dO; each lane multiplies its share of the d channels
// (a pair per load where alignment allows) and the group adds up with lane shuffles.
template <typename T>
__device__ __forceinline__ float dot_share(const T *a, const T *b, int d, int sub)
{
    float acc = 0.f;
    for (int t = sub; t < d; t += 16) acc = fmaf(widen(a[t]), widen(b[t]), acc);
    return acc;
}
template <>
__device__ __forceinline__ float dot_share<bf16_t>(const bf16_t *a, const bf16_t *b, int d, int sub)
{
    float acc = 0.f;
    if (((d & 1) == 0) && ((((uintptr_t)a | (uintptr_t)b) & 3) == 0)) {      // dword pairs
        for (int t = 2 * sub; t < d; t += 32) {
            const uint32_t x = *(const uint32_t *)(a + t), y = *(const uint32_t *)(b + t);
            acc = fmaf(__uint_as_float(x << 16), __uint_as_float(y << 16), acc);
            acc = fmaf(__uint_as_float(x & 0xffff0000u), __uint_as_float(y & 0xffff0000u), acc);
        }
    } else {
        for (int t = sub; t < d; t += 16) acc = fmaf(widen(a[t]), widen(b[t]), acc);
    }
    return acc;
}

// One workgroup = 64 consecutive window-local tokens of one (window, head) unit: the grid
// tokens are computed once (one division per token) and kept in LDS; sixteen lanes share
// a token, and the four tokens of a lane group are loaded before any is reduced, so four
// memory round trips are in flight per lane.
template <typename T>
__global__ __launch_bounds__(kThreads) void valu_delta_kernel(Geo g, int nchunk, const T *__restrict__ out,
                                                              const T *__restrict__ dout, float *__restrict__ delta)
{
    __shared__ int64_t tok[64];
    const int64_t u = blockIdx.x / nchunk;
    const int n0 = (int)(blockIdx.x - u * nchunk) * 64;
    const int w = (int)(u / g.heads), hd = (int)(u - (int64_t)w * g.heads);
    const int tid = threadIdx.x, grp = tid >> 4, sub = tid & 15;
    if (tid < 64) tok[tid] = n0 + tid < g.N ? grid_token(g, w, n0 + tid) : -1;
    __syncthreads();
    float acc[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int64_t t = tok[it * 16 + grp];
        acc[it] = 0.f;
        if (t >= 0) {
            const int64_t base = t * g.C + hd * g.d;
            acc[it] = dot_share<T>(out + base, dout + base, g.d, sub);
        }
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) acc[it] += __shfl_xor(acc[it], off);
        const int nl = it * 16 + grp;
        if (sub == 0 && n0 + nl < g.N) delta[u * g.N + n0 + nl] = acc[it];
    }
}

// Gated variant (CLA, Eq. 9: O' = O * G): from the gradient dO' of the gated output,
//   dO = dO' * G (rounded to the storage type, written for the main kernels),
//   dG = dO' * O,      delta = dO . O   (with the rounded dO, as the main kernels see it; null where they make it themselves).
// Same mapping of lanes to (token, head) slices as above, so every element of the grid is
// written exactly once.
template <typename T>
__global__ __launch_bounds__(kThreads) void valu_delta_gated_kernel(Geo g, int nchunk, const T *__restrict__ out,
                                                                    const T *__restrict__ dout_g, const T *__restrict__ gate,
                                                                    float *__restrict__ delta, T *__restrict__ dout,
                                                                    T *__restrict__ dgate)
{
    __shared__ int64_t tok[64];
    const int64_t u = blockIdx.x / nchunk;
    const int n0 = (int)(blockIdx.x - u * nchunk) * 64;
    const int w = (int)(u / g.heads), hd = (int)(u - (int64_t)w * g.heads);
    const int tid = threadIdx.x, grp = tid >> 4, sub = tid & 15;
    if (tid < 64) tok[tid] = n0 + tid < g.N ? grid_token(g, w, n0 + tid) : -1;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int64_t t = tok[it * 16 + grp];
        float acc = 0.f;
        if (t >= 0) {
            const int64_t base = t * g.C + hd * g.d;
            for (int c = sub; c < g.d; c += 16) {
                const float o = widen(out[base + c]), gp = widen(dout_g[base + c]), gv = widen(gate[base + c]);
                T d_o;
                store_as(&d_o, gp * gv);
                dout[base + c] = d_o;
                store_as(dgate + base + c, gp * o);
                acc = fmaf(widen(d_o), o, acc);
            }
        }
        if (delta == nullptr) continue;
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
        const int nl = it * 16 + grp;
        if (sub == 0 && n0 + nl < g.N) delta[u * g.N + n0 + nl] = acc;
    }
}

// dQ and this unit's dF_q contribution: rows are queries, tiles are keys.
template <typename T, int DA, int DV>
__global__ __launch_bounds__(kThreads) void valu_bwd_dq_kernel(Geo g, int nblk, const T *__restrict__ q,
                                                               const T *__restrict__ k, const T *__restrict__ v,
                                                               const T *__restrict__ fq, const T *__restrict__ fk,
                                                               const T *__restrict__ dout, const float *__restrict__ lse,
                                                               const float *__restrict__ delta, T *__restrict__ dq,
                                                               float *__restrict__ dfq_part)
{
    __shared__ float Ks[kTile][DA + 1];
    __shared__ float Vs[kTile][DV + 1];
    __shared__ int64_t tok[kTile];

    const int64_t u = blockIdx.x / nblk;
    const int blk = blockIdx.x - (int)(u * nblk);
    const int w = (int)(u / g.heads), hd = (int)(u - (int64_t)w * g.heads);
    const int tid = threadIdx.x, row = tid / kSplit, part = tid % kSplit;
    const int i = blk * kRows + row;
    const bool live = i < g.N;
    const int ic = live ? i : g.N - 1;
    const int64_t tq = grid_token(g, w, ic);

    float qa[DA], go[DV], acc[DA];
    load_aug<T, DA>(g, hd, ic, tq, q, fq, g.scale_c * kLog2e, g.scale_p * kLog2e, g.tstride, qa);
#pragma unroll
    for (int t = 0; t < DV; ++t) go[t] = t < g.d ? widen(dout[tq * g.C + hd * g.d + t]) : 0.f;
#pragma unroll
    for (int t = 0; t < DA; ++t) acc[t] = 0.f;
    const float lse2 = lse[u * g.N + ic] * kLog2e;
    const float dl = delta[u * g.N + ic];

    for (int j0 = 0; j0 < g.N; j0 += kTile) {
        __syncthreads();
        stage_tile<T, DA, DV>(g, w, hd, j0, k, fk, 1.f, 1.f, g.tstride, v, g.tstride, Ks, Vs, tok);
        __syncthreads();
        for (int jj = part; jj < kTile; jj += kSplit) {
            if (j0 + jj >= g.N) break;
            float s = 0.f, dp = 0.f;
#pragma unroll
            for (int t = 0; t < DA; ++t) s = fmaf(qa[t], Ks[jj][t], s);
#pragma unroll
            for (int t = 0; t < DV; ++t) dp = fmaf(go[t], Vs[jj][t], dp);
            float ds = exp2f(s - lse2) * (dp - dl);
#pragma unroll
            for (int t = 0; t < DA; ++t) acc[t] = fmaf(ds, Ks[jj][t], acc[t]);
        }
    }
#pragma unroll
    for (int off = 1; off < kSplit; off <<= 1)
#pragma unroll
        for (int t = 0; t < DA; ++t) acc[t] += __shfl_xor(acc[t], off);
    if (!live) return;
    T *dst = dq + tq * g.C + hd * g.d;
    float *fdst = dfq_part + (u * g.N + i) * g.r;
#pragma unroll
    for (int t = 0; t < DA; ++t) {
        if (t % kSplit != part) continue;
        if (t < g.d) store_as(dst + t, acc[t] * g.scale_c);
        else if (t < g.d + g.r) fdst[t - g.d] = acc[t] * g.scale_p;
    }
}

// dK, dV and this unit's dF_k contribution: rows are keys, tiles are queries.
template <typename T, int DA, int DV>
__global__ __launch_bounds__(kThreads) void valu_bwd_dkv_kernel(Geo g, int nblk, const T *__restrict__ q,
                                                                const T *__restrict__ k, const T *__restrict__ v,
                                                                const T *__restrict__ fq, const T *__restrict__ fk,
                                                                const T *__restrict__ dout, const float *__restrict__ lse,
                                                                const float *__restrict__ delta, T *__restrict__ dk,
                                                                T *__restrict__ dv, float *__restrict__ dfk_part)
{
    __shared__ float Qs[kTile][DA + 1];
    __shared__ float Gs[kTile][DV + 1];
    __shared__ float lse2s[kTile], dls[kTile];
    __shared__ int64_t tok[kTile];

    const int64_t u = blockIdx.x / nblk;
    const int blk = blockIdx.x - (int)(u * nblk);
    const int w = (int)(u / g.heads), hd = (int)(u - (int64_t)w * g.heads);
    const int tid = threadIdx.x, row = tid / kSplit, part = tid % kSplit;
    const int j = blk * kRows + row;
    const bool live = j < g.N;
    const int jc = live ? j : g.N - 1;
    const int64_t tkv = grid_token(g, w, jc);

    float ka[DA], va[DV], dka[DA], dva[DV];
    load_aug<T, DA>(g, hd, jc, tkv, k, fk, 1.f, 1.f, g.tstride, ka);
#pragma unroll
    for (int t = 0; t < DV; ++t) va[t] = t < g.d ? widen(v[tkv * g.tstride + hd * g.d + t]) : 0.f;
#pragma unroll
    for (int t = 0; t < DA; ++t) dka[t] = 0.f;
#pragma unroll
    for (int t = 0; t < DV; ++t) dva[t] = 0.f;

    for (int i0 = 0; i0 < g.N; i0 += kTile) {
        __syncthreads();
        stage_tile<T, DA, DV>(g, w, hd, i0, q, fq, g.scale_c, g.scale_p, g.tstride, dout, (int64_t)g.C, Qs, Gs, tok);
        if (tid < kTile) {
            int i = i0 + tid;
            lse2s[tid] = i < g.N ? lse[u * g.N + i] * kLog2e : 0.f;
            dls[tid] = i < g.N ? delta[u * g.N + i] : 0.f;
        }
        __syncthreads();
        for (int ii = part; ii < kTile; ii += kSplit) {
            if (i0 + ii >= g.N) break;
            float s = 0.f, dp = 0.f;
#pragma unroll
            for (int t = 0; t < DA; ++t) s = fmaf(ka[t], Qs[ii][t], s);
#pragma unroll
            for (int t = 0; t < DV; ++t) dp = fmaf(va[t], Gs[ii][t], dp);
            float p = exp2f(s * kLog2e - lse2s[ii]);
            float ds = p * (dp - dls[ii]);
#pragma unroll
            for (int t = 0; t < DV; ++t) dva[t] = fmaf(p, Gs[ii][t], dva[t]);
#pragma unroll
            for (int t = 0; t < DA; ++t) dka[t] = fmaf(ds, Qs[ii][t], dka[t]);
        }
    }
#pragma unroll
    for (int off = 1; off < kSplit; off <<= 1) {
#pragma unroll
        for (int t = 0; t < DA; ++t) dka[t] += __shfl_xor(dka[t], off);
#pragma unroll
        for (int t = 0; t < DV; ++t) dva[t] += __shfl_xor(dva[t], off);
    }
    if (!live) return;
    T *kdst = dk + tkv * g.C + hd * g.d;
    T *vdst = dv + tkv * g.C + hd * g.d;
    float *fdst = dfk_part + (u * g.N + j) * g.r;
#pragma unroll
    for (int t = 0; t < DA; ++t) {
        if (t % kSplit != part) continue;
        if (t < g.d) store_as(kdst + t, dka[t]);
        else if (t < g.d + g.r) fdst[t - g.d] = dka[t];
    }
#pragma unroll
    for (int t = 0; t < DV; ++t)
        if (t % kSplit == part && t < g.d) store_as(vdst + t, dva[t]);
}

// dF[hd][e] = sum over windows w of part[(w*heads + hd)][e]; e over N*r, VEC of them a lane.  A workgroup's lanes are
// `slices` groups that each sum a run of windows (eight loads in flight), added through LDS in ascending order: the
// order is fixed by the sizes (VEC does not enter it).
template <int VEC>
__global__ __launch_bounds__(kThreads) void reduce_df_kernel(int64_t per_head, int heads, int blocks, int nwin, int slices, const float *__restrict__ part_q,
                                                             const float *__restrict__ part_k,
                                                             float *__restrict__ dfq, float *__restrict__ dfk)
{
    typedef float vec __attribute__((ext_vector_type(VEC)));
    __shared__ vec sums[kThreads];
    const int lanes = kThreads / slices, slice = threadIdx.x / lanes, lane = threadIdx.x - slice * lanes;
    const int hd = blockIdx.x / blocks, block = blockIdx.x - hd * blocks;
    const int64_t e = ((int64_t)block * lanes + lane) * VEC;
    const bool in = e < per_head;
    const int64_t step = (int64_t)heads * per_head;
    const float *p = (blockIdx.y == 0 ? part_q : part_k) + hd * per_head + (in ? e : 0);
    float *dst = (blockIdx.y == 0 ? dfq : dfk) + hd * per_head + e;
    const int run = (nwin + slices - 1) / slices;
    int w = slice * run;
    const int end = w + run < nwin ? w + run : nwin;
    vec acc = 0.f;
    for (; w + 8 <= end; w += 8) {
        vec t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = *(const vec *)(p + (w + i) * step);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += t[i];
    }
    // the rest of the run, requested together as well (its last window again where there are fewer): one after the other
    // they made a call of 24 windows, 12 a slice, 1 us longer than one slice of 24
    if (w < end) {
        vec t[7];
#pragma unroll
        for (int i = 0; i < 7; ++i) t[i] = *(const vec *)(p + (w + i < end ? w + i : end - 1) * step);
#pragma unroll
        for (int i = 0; i < 7; ++i)
            if (w + i < end) acc += t[i];
    }
    if (slices > 1) {
        sums[threadIdx.x] = acc;
        __syncthreads();
        if (slice != 0) return;
        for (int i = 1; i < slices; ++i) acc += sums[i * lanes + lane];
    }
    if (in) *(vec *)dst = acc;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
inline BwdWs ws_layout(const Geo &g) { return bwd_ws_layout(g); }

template <typename T, int DA, int DV>
hipError_t fwd_t(const Geo &g, const void *q, const void *k, const void *v, const void *fq, const void *fk,
                 void *out, float *lse, hipStream_t st)
{
    int nblk = (g.N + kRows - 1) / kRows;
    dim3 grid((unsigned)(g.units * nblk));
    hipLaunchKernelGGL((valu_fwd_kernel<T, DA, DV>), grid, dim3(kThreads), 0, st, g, nblk, (const T *)q,
                       (const T *)k, (const T *)v, (const T *)fq, (const T *)fk, (T *)out, lse);
    return hipGetLastError();
}

template <typename T, int DA, int DV>
hipError_t bwd_t(const Geo &g, const void *q, const void *k, const void *v, const void *fq, const void *fk,
                 const void *out, const void *dout, const float *lse, void *dq, void *dk, void *dv, float *dfq,
                 float *dfk, void *ws, hipStream_t st)
{
    BwdWs l = ws_layout(g);
    float *delta = (float *)((char *)ws + l.delta_off);
    float *pq = (float *)((char *)ws + l.dfq_off);
    float *pk = (float *)((char *)ws + l.dfk_off);
    int64_t rows = g.units * g.N;
    (void)rows;
    hipError_t e = g.gate ? hipSuccess : launch_delta(g, sizeof(T) == 2 ? RIB_BF16 : RIB_F32, out, dout, delta, st);
    if (e != hipSuccess) return e;
    int nblk = (g.N + kRows - 1) / kRows;
    dim3 grid((unsigned)(g.units * nblk));
    hipLaunchKernelGGL((valu_bwd_dq_kernel<T, DA, DV>), grid, dim3(kThreads), 0, st, g, nblk, (const T *)q,
                       (const T *)k, (const T *)v, (const T *)fq, (const T *)fk, (const T *)dout, lse, delta, (T *)dq,
                       pq);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((valu_bwd_dkv_kernel<T, DA, DV>), grid, dim3(kThreads), 0, st, g, nblk, (const T *)q,
                       (const T *)k, (const T *)v, (const T *)fq, (const T *)fk, (const T *)dout, lse, delta, (T *)dk,
                       (T *)dv, pk);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_reduce_df(g, pq, pk, dfq, dfk, st);
}

// Smallest compiled (DA, DV) bucket holding d + r and d.
inline int bucket(const Geo &g)
{
    int da = g.d + g.r;
    if (da <= 16 && g.d <= 8) return 0;
    if (da <= 48 && g.d <= 32) return 1;
    if (da <= 64 && g.d <= 32) return 2;
    return 3;  // da <= 128, d <= 64 (checked by the caller)
}

}  // namespace

size_t valu_bwd_workspace(const Geo &g) { return ws_layout(g).total; }

BwdWs bwd_ws_layout(const Geo &g)
{
    BwdWs l;
    size_t rows = (size_t)g.units * g.N;
    l.delta_off = 0;
    l.dfq_off = align256(rows * sizeof(float));
    l.dfk_off = l.dfq_off + align256(rows * g.r * sizeof(float));
    l.total = l.dfk_off + align256(rows * g.r * sizeof(float));
    return l;
}

hipError_t launch_delta(const Geo &g, int dtype, const void *out, const void *dout, float *delta, hipStream_t st)
{
    const int nchunk = (g.N + 63) / 64;
    dim3 grid((unsigned)(g.units * nchunk));
    if (dtype == RIB_BF16)
        hipLaunchKernelGGL((valu_delta_kernel<bf16_t>), grid, dim3(kThreads), 0, st, g, nchunk, (const bf16_t *)out,
                           (const bf16_t *)dout, delta);
    else
        hipLaunchKernelGGL((valu_delta_kernel<float>), grid, dim3(kThreads), 0, st, g, nchunk, (const float *)out,
                           (const float *)dout, delta);
    return hipGetLastError();
}

size_t gated_dout_bytes(const Geo &g, int dtype)
{
    const size_t n = (size_t)g.B * g.H * g.W * g.C * (dtype == RIB_BF16 ? 2 : 4);
    return (n + 255) / 256 * 256;
}

hipError_t launch_delta_gated(const Geo &g, int dtype, const void *out_raw, const void *dout_gated, const void *gate,
                              float *delta, void *dout, void *dgate, hipStream_t st)
{
    const int nchunk = (g.N + 63) / 64;
    dim3 grid((unsigned)(g.units * nchunk));
    if (dtype == RIB_BF16)
        hipLaunchKernelGGL((valu_delta_gated_kernel<bf16_t>), grid, dim3(kThreads), 0, st, g, nchunk,
                           (const bf16_t *)out_raw, (const bf16_t *)dout_gated, (const bf16_t *)gate, delta,
                           (bf16_t *)dout, (bf16_t *)dgate);
    else
        hipLaunchKernelGGL((valu_delta_gated_kernel<float>), grid, dim3(kThreads), 0, st, g, nchunk,
                           (const float *)out_raw, (const float *)dout_gated, (const float *)gate, delta,
                           (float *)dout, (float *)dgate);
    return hipGetLastError();
}

hipError_t launch_reduce_df(const Geo &g, const float *part_q, const float *part_k, float *dfq, float *dfk,
                            hipStream_t st)
{
    if (g.r == 0) return hipSuccess;
    const int64_t per_head = (int64_t)g.N * g.r;
    const int nwin = (int)(g.units / g.heads);
    // 16 bytes a lane where the rows of every window keep that alignment, and the caller's dF does.  The slices, and with them the
    // order of the sums, come from the sizes alone: the same call gives the same bits wherever dF lies.
    const uintptr_t at = (uintptr_t)dfq | (uintptr_t)dfk;
    const int whole = per_head % 4 == 0 ? 4 : per_head % 2 == 0 ? 2 : 1;
    const int vec = whole == 4 && at % 16 == 0 ? 4 : whole >= 2 && at % 8 == 0 ? 2 : 1;
    // Slices until the chip has two waves a SIMD: one slice / this rule / up to 16 until it has eight, us: 576 windows of 256
    // tokens, 6 heads, r = 18 50 / 25 / 25, 144 of 1024, r = 16 21 / 21 / 23, 128 of 576, r = 18 12.6 / 11.0 / 11.7 (the
    // partials of the first pass at 5 TB/s).  A slice of under eight windows has too few loads in flight.
    int slices = 1;
    while (slices < 16 && per_head * g.heads * 2 / whole * slices < 128 * 1024 && nwin / (2 * slices) >= 8) slices *= 2;
    const int64_t lanes = kThreads / slices * vec;
    const int blocks = (int)((per_head + lanes - 1) / lanes);
    const dim3 grid((unsigned)((int64_t)blocks * g.heads), 2);
    auto kern = vec == 4 ? reduce_df_kernel<4> : vec == 2 ? reduce_df_kernel<2> : reduce_df_kernel<1>;
    hipLaunchKernelGGL(kern, grid, dim3(kThreads), 0, st, per_head, g.heads, blocks, nwin, slices, part_q, part_k, dfq, dfk);
    return hipGetLastError();
}

#define RIB_VALU_DISPATCH(FN, ...)                                                         \
    switch (bucket(g) * 2 + (dtype == RIB_BF16 ? 1 : 0)) {                                 \
    case 0: return FN<float, 16, 8>(__VA_ARGS__);                                          \
    case 1: return FN<bf16_t, 16, 8>(__VA_ARGS__);                                         \
    case 2: return FN<float, 48, 32>(__VA_ARGS__);                                         \
    case 3: return FN<bf16_t, 48, 32>(__VA_ARGS__);                                        \
    case 4: return FN<float, 64, 32>(__VA_ARGS__);                                         \
    case 5: return FN<bf16_t, 64, 32>(__VA_ARGS__);                                        \
    case 6: return FN<float, 128, 64>(__VA_ARGS__);                                        \
    default: return FN<bf16_t, 128, 64>(__VA_ARGS__);                                      \
    }

hipError_t launch_valu_fwd(const Geo &g, int dtype, const void *q, const void *k, const void *v, const void *fq,
                           const void *fk, void *out, float *lse, hipStream_t st)
{
    RIB_VALU_DISPATCH(fwd_t, g, q, k, v, fq, fk, out, lse, st)
}

hipError_t launch_valu_bwd(const Geo &g, int dtype, const void *q, const void *k, const void *v, const void *fq,
                           const void *fk, const void *out, const void *dout, const float *lse, void *dq, void *dk,
                           void *dv, float *dfq, float *dfk, void *ws, hipStream_t st, void *gated_dout, void *dgate)
{
    if (g.gate) {
        float *delta = (float *)((char *)ws + bwd_ws_layout(g).delta_off);
        hipError_t e = launch_delta_gated(g, dtype, out, dout, g.gate, delta, gated_dout, dgate, st);
        if (e != hipSuccess) return e;
        dout = gated_dout;
    }
    RIB_VALU_DISPATCH(bwd_t, g, q, k, v, fq, fk, out, dout, lse, dq, dk, dv, dfq, dfk, ws, st)
}

}  // namespace rib

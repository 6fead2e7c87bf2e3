// Host side of the bf16 matrix-core backward: which problems it serves, by which kernels and in which padded width
// (rib_mfma_unit.h, rib_mfma_bwd.h; one translation unit per width keeps the build parallel).
#include "rib_mfma_bwd.h"
#include "rib_mfma_unit.h"

namespace rib {

bool mfma_bwd_supported(const Geo &g, int dtype)
{
    return dtype == RIB_BF16 && !(g.flags & RIB_FLAG_VECTOR_ONLY) && g.d <= 32 && (g.d & 1) == 0 && (g.r & 1) == 0 &&
           g.d + g.r <= 64 && g.N >= 64 && g.N <= 9216 && (g.tstride & 1) == 0;
}

hipError_t launch_mfma_bwd(const Geo &g, const void *q, const void *k, const void *v, const void *fq, const void *fk,
                           const void *out, const void *dout, const float *lse, void *dq, void *dk, void *dv,
                           float *dfq, float *dfk, void *ws, hipStream_t st, void *gated_dout, void *dgate)
{
    const BwdWs l = bwd_ws_layout(g);
    bwd::Args a;
    a.delta = (float *)((char *)ws + l.delta_off);
    a.pq = (float *)((char *)ws + l.dfq_off);
    a.pk = (float *)((char *)ws + l.dfk_off);
    // Units that one workgroup holds are done in one kernel (the figures stand in rib_mfma_unit.h), which makes delta of the
    // rows it stages; rows of a pair or less and 64-bit offsets have forms in the pair only.
    const bool one = g.N <= 512 && (rows::short_rows(g) == rows::kLong || rows::short_rows(g) == rows::kLong8) && rows_supported(g);
    if (g.gate) {
        const hipError_t e = launch_delta_gated(g, RIB_BF16, out, dout, g.gate, one ? nullptr : a.delta, gated_dout, dgate, st);
        if (e != hipSuccess) return e;
        dout = gated_dout;
    }
    a.q = (const bf16_t *)q, a.k = (const bf16_t *)k, a.v = (const bf16_t *)v;
    a.fq = (const bf16_t *)fq, a.fk = (const bf16_t *)fk;
    a.out = (const bf16_t *)out, a.dout = (const bf16_t *)dout, a.lse = lse;
    a.dq = (bf16_t *)dq, a.dk = (bf16_t *)dk, a.dv = (bf16_t *)dv;
    // the call's own dF_q output, which is written last, holds the scaled rows of f_q until then (2 of its 4 bytes a value)
    a.ftab = (bf16_t *)dfq;
    a.st = st;
    // (RIB rows of more than 32 values are staged by the 64-column kernels only)
    const int aug = g.d + g.r;
    const int width = aug <= 32 && g.d <= 30 ? 32 : aug <= 48 && g.r <= 32 ? 48 : 64;
    const hipError_t e = one ? (width == 32 ? unit::launch32(g, a) : width == 48 ? unit::launch48(g, a) : unit::launch64(g, a))
                             : (width == 32 ? bwd::launch32(g, a) : width == 48 ? bwd::launch48(g, a) : bwd::launch64(g, a));
    if (e != hipSuccess) return e;
    return launch_reduce_df(g, a.pq, a.pk, dfq, dfk, st);
}

}  // namespace rib

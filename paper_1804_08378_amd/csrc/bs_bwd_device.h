// Device helpers shared by the backward kernels: checked offsets (audit builds) and the
// average's divisor.
#pragma once
#include "bs_device.h"

namespace bs {

// Build with -DBS_BWD_AUDIT to check every element offset (32 or 64 bits) into the stage input, the upstream gradient and the
// input gradient, with the number of elements read or written there, against the extents the host passes (k.audit_lim[0..2],
// in elements) before it is used: an offset outside is counted in k.audit[site] and replaced by 0, so such a build cannot
// read or write outside those tensors.  Without the macro the checks compile to nothing.
#if defined(BS_BWD_AUDIT)
template <typename OFF>
BS_DEV OFF audited(const BwdK &k, int which, int site, OFF off, uint32_t n)
{
    if (k.audit && (off > k.audit_lim[which] || (uint64_t)off + n > k.audit_lim[which])) {
        atomicAdd(&k.audit[site], 1u);
        return 0u;
    }
    return off;
}
#else
template <typename OFF>
BS_DEV OFF audited(const BwdK &, int, int, OFF off, uint32_t) { return off; }
#endif

// float32 reciprocal of the divisor of the average pooling window (oh, ow): the forward
// kernels' rule (0: in-range cells, 1: kh * kw, 2: cells inside the padded plane).
BS_DEV float bwd_avg_inv(const PoolK &p, int32_t H, int32_t W, int32_t oh, int32_t ow)
{
    if (p.count_include_pad == 1) return p.inv_kk;
    const int32_t h0 = oh * p.sh - p.ph, w0 = ow * p.sw - p.pw;
    if (p.count_include_pad == 2) {
        const int32_t nr = min(h0 + p.kh, H + p.ph) - h0, nc = min(w0 + p.kw, W + p.pw) - w0;
        return 1.0f / (float)max(nr * nc, 1);
    }
    const int32_t nr = min(h0 + p.kh, H) - max(h0, 0), nc = min(w0 + p.kw, W) - max(w0, 0);
    return 1.0f / (float)max(nr * nc, 1);
}

}  // namespace bs

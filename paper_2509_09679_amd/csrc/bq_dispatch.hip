// Kernel selection: specialised kernels where one exists for the shape, generic kernels otherwise.
#include "bq_internal.h"

namespace bq {

hipError_t launch_transform(Mode mode, const void *in, void *out, const PlanView &pv, const Shape &s,
                            const QuantArgs *q, hipStream_t stream)
{
    if (k12_supported(mode, in, out, s, q)) return launch_k12(mode, in, out, pv, s, q, stream);
    if (small_supported(mode, in, out, s, q)) return launch_small(mode, in, out, pv, s, q, stream);
    return launch_generic(mode, in, out, pv, s, q, stream);
}

size_t bwd_workspace_bytes(const Shape &s)
{
    size_t need = bwd_workspace_bytes_generic(s);
    if (s.k >= 8 && s.k <= 13 && s.rows > 0 && (s.heads == 1 || (s.k < 12 && (int64_t)s.n * s.heads <= 4096))) {
        const size_t fast = bwd_fast_workspace_bytes(s);
        if (fast > need) need = fast;
    }
    if (s.k >= 3 && s.k <= 7 && s.rows > 0) {
        const size_t small = small_bwd_workspace_bytes(s);
        if (small > need) need = small;
    }
    return need;
}

hipError_t launch_bwd(const void *x, const void *dy, const PlanView &pv, void *dx, float *dtheta, void *ws,
                      const Shape &s, hipStream_t stream)
{
    if (!dtheta) {  // dx alone is the transposed transform of dy
        Shape t = s;
        return launch_transform(kInv, dy, dx, pv, t, nullptr, stream);
    }
    if (bwd_fast_supported(x, dy, dx, dtheta, s)) return launch_bwd_fast(x, dy, pv, dx, dtheta, ws, s, stream);
    if (small_bwd_supported(x, dy, dx, dtheta, s)) return launch_small_bwd(x, dy, pv, dx, dtheta, ws, s, stream);
    return launch_generic_bwd(x, dy, pv, dx, dtheta, ws, s, stream);
}

}  // namespace bq

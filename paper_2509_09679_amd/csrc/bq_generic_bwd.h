// The backward pass for any n in plain (cos, sin) rotations, as device code: the kernel for any n (bq_generic.hip) and, on plans
// that flag their scale-deferred tables, the specialised kernels of bq_bwd.hip and bq_bwd_small.hip run it.
#pragma once

#include "bq_device.h"

namespace bq {

template <bool kInverse>
__device__ __forceinline__ void rotate_pair(float &va, float &vb, float c, float s)
{
    const float xa = va, xb = vb;
    if (!kInverse) {  // G(theta):  [c -s; s c]
        va = __builtin_fmaf(c, xa, -(s * xb));
        vb = __builtin_fmaf(s, xa, c * xb);
    } else {  // G(theta)^T: [c s; -s c]
        va = __builtin_fmaf(c, xa, s * xb);
        vb = __builtin_fmaf(c, xb, -(s * xa));
    }
}

// ---------------------------------------------------------------------------------------------
// Backward.  A tile is U consecutive rows of ONE head, so that the thread owning pair p of a layer
// owns it for every row of the tile and for every tile its workgroup processes: the per-workgroup
// partial sums in `partial` are read-modify-written by one thread only, in a fixed order.
// dtheta_{i,p} += g_i[b] x_i[a] - g_i[a] x_i[b], evaluated on the layer's outputs (which follows from
// dG/dtheta = [[-s,-c],[c,-s]]: d y_a / d theta = -y_b, d y_b / d theta = y_a); then both x_i and g_i
// are taken back through the transposed layer (orthogonality makes stored activations unnecessary).
// ---------------------------------------------------------------------------------------------
struct BwdArgs {
    const void *x, *dy;
    void *dx;
    const float2 *cs;
    float *partial;  // [grid][heads*k*n/2]
    int64_t rows, ld_in, ld_out;
    int n, heads, k, rows_per_tile;
    int64_t n_tiles;
    PlanRef plan;
    int only_if_bad;  // != 0: run only when one of the plan's table sets is flagged unusable
};

// The share of workgroup `part` of `parts`; kThreads threads.  lds: 2 * rows_per_tile * n floats.  Acc: what a tile's rows are
// added up in, and its sum to the slice's.
template <typename T, int kThreads, typename Acc = float>
__device__ __forceinline__ void generic_bwd_rows(const BwdArgs &A, float *lds, int my_part, int parts)
{
    const int n = A.n, k = A.k, heads = A.heads, U = A.rows_per_tile;
    float *xb = lds;
    float *gb = lds + (size_t)U * n;
    const T *__restrict__ x = (const T *)A.x;
    const T *__restrict__ dy = (const T *)A.dy;
    T *__restrict__ dx = (T *)A.dx;
    const size_t n_angles = (size_t)heads * k * (n >> 1);
    float *__restrict__ part = A.partial + (size_t)my_part * n_angles;
    for (size_t q = threadIdx.x; q < n_angles; q += kThreads) part[q] = 0.0f;

    for (int64_t tile = my_part; tile < A.n_tiles; tile += parts) {
        const int head = (int)(tile % heads);
        const int64_t row0 = (tile / heads) * U;
        for (int e = threadIdx.x; e < U * n; e += kThreads) {
            const int64_t row = row0 + (e >> k);
            float vx = 0.0f, vg = 0.0f;
            if (row < A.rows) {
                const int64_t off = row * A.ld_in + (int64_t)head * n + (e & (n - 1));
                vx = to_float(x[off]);
                vg = to_float(dy[off]);
            }
            xb[e] = vx;
            gb[e] = vg;
        }
        __syncthreads();
        const float2 *__restrict__ csh = A.cs + (size_t)head * k * (n >> 1);
        for (int i = 1; i <= k; ++i) {  // recompute the layer outputs x_1 .. x_k
            const int h = 1 << (i - 1);
            for (int q = threadIdx.x; q < ((U * n) >> 1); q += kThreads) {
                const int ul = q >> (k - 1);
                const int p = q & ((n >> 1) - 1);
                const float2 w = csh[(size_t)(i - 1) * (n >> 1) + p];
                const int a = (ul << k) + (((p >> (i - 1)) << i) | (p & (h - 1)));
                rotate_pair<false>(xb[a], xb[a + h], w.x, w.y);
            }
            __syncthreads();
        }
        for (int i = k; i >= 1; --i) {
            const int h = 1 << (i - 1);
            for (int p = threadIdx.x; p < (n >> 1); p += kThreads) {
                const float2 w = csh[(size_t)(i - 1) * (n >> 1) + p];
                const int a0 = ((p >> (i - 1)) << i) | (p & (h - 1));
                Acc acc = 0;
                for (int ul = 0; ul < U; ++ul) {
                    const int a = (ul << k) + a0;
                    float xa = xb[a], xv = xb[a + h], ga = gb[a], gv = gb[a + h];
                    acc += (Acc)(gv * xa - ga * xv);
                    rotate_pair<true>(xa, xv, w.x, w.y);
                    rotate_pair<true>(ga, gv, w.x, w.y);
                    xb[a] = xa;
                    xb[a + h] = xv;
                    gb[a] = ga;
                    gb[a + h] = gv;
                }
                float &sum = part[((size_t)head * k + (i - 1)) * (size_t)(n >> 1) + p];
                sum = (float)((Acc)sum + acc);
            }
            __syncthreads();
        }
        if (dx) {
            for (int e = threadIdx.x; e < U * n; e += kThreads) {
                const int64_t row = row0 + (e >> k);
                if (row < A.rows)
                    dx[row * A.ld_out + (int64_t)head * n + (e & (n - 1))] = from_float<T>(gb[e]);
            }
        }
        __syncthreads();
    }
}

// Arguments of the whole batch; *parts: the slices of `ws` it may write, one per workgroup (host code)
BwdArgs generic_bwd_args(const void *x, const void *dy, const PlanView &pv, void *dx, void *ws, const Shape &s, int *parts);

}  // namespace bq

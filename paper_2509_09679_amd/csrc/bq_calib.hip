// What a calibration step on 16-bit rows needs between its dense products and the backward kernels: the error matrix
// split into 16-bit pieces, and the gradient through the fake quantiser.
//
// The gradients multiply the float32 error matrix E with 16-bit operands.  As float32 products they ran at 0.15 PFLOP/s and
// were 7.4 of the 16.8 ms of a step (16384 rows, n = m = 4096); with E as a sum of 16-bit pieces the same sums run on the
// 16-bit matrix instructions, which accumulate in float32.  binary16 rows: E times a power of two that puts its largest
// entry into [2^14, 2^15), in two pieces of 11 bits each, the second of them 2^12 times the remainder (exact, with a sign of
// its own, at most 2^15): E is piece 0 + 2^-12 piece 1 within 2^-23 |E| for entries down to 2^-28 of the largest and within
// 2^-51 of the largest below.  Unscaled, the remainder of a small entry fell on binary16's subnormal grid: tokens at 2^-20 of
// an outlier token had their gradient off by 2.1e-6, at 2^-24 by 3.3e-5.  Scaled it is 3.5e-7 for every token (median over
// tokens against 64 bits, 768 rows, n = 1024, m = 512), where float32 products leave 7.5e-7; a third piece changes nothing.
// bfloat16 rows: three pieces of 8 bits, no scales, their sum is E.
//
// The matrix instructions' products of binary16 operands below 2^-14 keep fewer bits: on a layer whose weights all lie there
// but for one output channel, those channels' gradients are off by 4e-6 (float32 products: 4e-7).
#include <cmath>

#include "bq_cascade.h"

namespace bq {

constexpr int kStatBlocks = 1024;
struct ResidualStats {
    double sum[kStatBlocks];
    float amax[kStatBlocks];
};
size_t residual_scratch_bytes() { return sizeof(ResidualStats); }

// Per workgroup: max |e| and the sum of squares (double).  One read of E: bound by HBM.
__global__ __launch_bounds__(256) void residual_stats_kernel(const float *__restrict__ e, int64_t count, ResidualStats *st)
{
    double sum = 0.0;
    float amax = 0.0f;
    const int64_t quads = count >> 2;
    const int64_t step = (int64_t)kStatBlocks * 256;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < quads; q += step) {
        const float4 v = *((const float4 *)e + q);
        amax = fmaxf(fmaxf(fmaxf(amax, fabsf(v.x)), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w)));
        sum += ((double)v.x * v.x + (double)v.y * v.y) + ((double)v.z * v.z + (double)v.w * v.w);
    }
    if (blockIdx.x == 0 && (int)threadIdx.x < (int)(count & 3)) {
        const float v = e[(quads << 2) + threadIdx.x];
        amax = fmaxf(amax, fabsf(v));
        sum += (double)v * v;
    }
    __shared__ double s_sum[256];
    __shared__ float s_max[256];
    s_sum[threadIdx.x] = sum;
    s_max[threadIdx.x] = amax;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) {
            s_sum[threadIdx.x] += s_sum[threadIdx.x + h];
            s_max[threadIdx.x] = fmaxf(s_max[threadIdx.x], s_max[threadIdx.x + h]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        st->sum[blockIdx.x] = s_sum[0];
        st->amax[blockIdx.x] = s_max[0];
    }
}

struct SplitArgs {
    const float *e;
    int64_t rows;
    int cols, ld;
    void *pieces;  // [2 or 3][rows][ld]
    const ResidualStats *st;
    float *result;  // [0] sum of squares of E, [1] factor that turns products with the pieces into products with 2 E
};

template <typename T>
__device__ __forceinline__ uint2 pack4(const float (&v)[4]);
template <>
__device__ __forceinline__ uint2 pack4<__half>(const float (&v)[4])
{
    return make_uint2(f32x2_to_f16x2_bits(v[0], v[1]), f32x2_to_f16x2_bits(v[2], v[3]));
}
template <>
__device__ __forceinline__ uint2 pack4<bf16_t>(const float (&v)[4])
{
    return make_uint2(f32x2_to_bf16x2_bits(v[0], v[1]), f32x2_to_bf16x2_bits(v[2], v[3]));
}
template <typename T>
__device__ __forceinline__ void unpack4(uint2 w, float (&v)[4]);
template <>
__device__ __forceinline__ void unpack4<__half>(uint2 w, float (&v)[4])
{
    const __half2 a = *(const __half2 *)&w.x, b = *(const __half2 *)&w.y;
    v[0] = __low2float(a); v[1] = __high2float(a); v[2] = __low2float(b); v[3] = __high2float(b);
}
template <>
__device__ __forceinline__ void unpack4<bf16_t>(uint2 w, float (&v)[4])
{
    v[0] = __uint_as_float(w.x << 16); v[1] = __uint_as_float(w.x & 0xFFFF0000u);
    v[2] = __uint_as_float(w.y << 16); v[3] = __uint_as_float(w.y & 0xFFFF0000u);
}

constexpr float kPieceStep = 4096.0f;  // binary16: every piece is this times what the pieces before it leave

// One read of E, one write of the pieces: bound by HBM.  Workgroups take whole rows; ld is a multiple of 8, so the pieces'
// rows are 16-byte aligned whatever the number of columns (the products' loads want that), with zeros behind the columns.
template <typename T>
__global__ __launch_bounds__(256) void residual_split_kernel(SplitArgs A)
{
    constexpr int kPieces = std::is_same<T, __half>::value ? 2 : 3;
    __shared__ float s_max[256];
    float amax = 0.0f;
#pragma unroll
    for (int j = 0; j < kStatBlocks / 256; ++j) amax = fmaxf(amax, A.st->amax[threadIdx.x + 256 * j]);
    s_max[threadIdx.x] = amax;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) s_max[threadIdx.x] = fmaxf(s_max[threadIdx.x], s_max[threadIdx.x + h]);
        __syncthreads();
    }
    float scale = 1.0f, factor = 2.0f;
    if (kPieces == 2) {
        int k = (int)((__float_as_uint(s_max[0]) >> 23) & 255u) - 127;  // floor(log2) of the largest entry, -127 if subnormal or 0
        k = k < -100 ? -100 : k;
        scale = __uint_as_float((uint32_t)(127 + 14 - k) << 23);
        factor = __uint_as_float((uint32_t)(127 + k - 13) << 23);
    }
    if (blockIdx.x == 0) {
        __shared__ double s_sum[256];
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < kStatBlocks / 256; ++j) t += A.st->sum[threadIdx.x + 256 * j];
        s_sum[threadIdx.x] = t;
        __syncthreads();
        for (int h = 128; h >= 1; h >>= 1) {
            if ((int)threadIdx.x < h) s_sum[threadIdx.x] += s_sum[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            A.result[0] = (float)s_sum[0];
            A.result[1] = factor;
        }
    }
    const bool quad_loads = (A.cols & 3) == 0;
    const size_t plane = (size_t)A.rows * A.ld;
    for (int64_t row = blockIdx.x; row < A.rows; row += gridDim.x) {
        const float *src = A.e + row * A.cols;
        T *dst = (T *)A.pieces + row * A.ld;
        for (int c = (int)threadIdx.x * 4; c < A.ld; c += 1024) {
            float v[4];
            if (quad_loads && c < A.cols) {
                const float4 q = *(const float4 *)(src + c);
                v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = c + r < A.cols ? src[c + r] : 0.0f;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] *= scale;
#pragma unroll
            for (int p = 0; p < kPieces; ++p) {
                const uint2 w = pack4<T>(v);
                *(uint2 *)(dst + p * plane + c) = w;
                float back[4];
                unpack4<T>(w, back);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] -= back[r];
                    if (kPieces == 2) v[r] *= kPieceStep;
                }
            }
        }
    }
}

// Gradient through Vq = s round(V / s), s = max |V| / qmax over a group, with a straight-through round: the incoming
// gradient g = factor * G passes unchanged, and the group's entry of largest magnitude (the first of equals) receives
// sign(v) / qmax * sum g (q - v / s) on top.  In place on G.  8 channels per thread; a group is `lanes` consecutive threads: the
// reductions are lane exchanges within a wave and, for groups of more than 512 channels, one value per wave through LDS.
// One read of V, Vq, G and one write of G: bound by HBM.  As torch operations it took 14 passes over float32 copies.
struct QuantGradArgs {
    const void *v, *vq;
    float *g;
    const float *factor;
    int64_t total;  // elements
    int lanes;      // threads of a group: 1 .. 1024
    float qmax;
};

template <typename T>
__global__ __launch_bounds__(1024) void quant_grad_kernel(QuantGradArgs A)
{
    __shared__ float s_max[16], s_sum[16];
    __shared__ int s_at[16];
    const int tid = threadIdx.x, wave = tid >> 6;
    const int in_wave = A.lanes < 64 ? A.lanes : 64, waves = A.lanes >> 6;  // waves of a group, 0 or 1: within one
    const float factor = A.factor[0];
    const int64_t at = ((int64_t)blockIdx.x * blockDim.x + tid) * 8;
    const bool live = at < A.total;  // whole groups are
    float v[8] = {}, q[8] = {}, g[8] = {};
    if (live) {
        unpack8(load8((const T *)A.v + at), v, (const T *)nullptr);
        unpack8(load8((const T *)A.vq + at), q, (const T *)nullptr);
        load_coef8(A.g + at, g);
    }
    float m = fabsf(v[0]);
    int first = tid * 8;  // position inside the workgroup: increasing inside a group
#pragma unroll
    for (int r = 1; r < 8; ++r)
        if (fabsf(v[r]) > m) {
            m = fabsf(v[r]);
            first = tid * 8 + r;
        }
    for (int d = 1; d < in_wave; d <<= 1) {
        const float om = __shfl_xor(m, d, 64);
        const int of = __shfl_xor(first, d, 64);
        if (om > m || (om == m && of < first)) {
            m = om;
            first = of;
        }
    }
    if (waves > 1) {
        if ((tid & 63) == 0) {
            s_max[wave] = m;
            s_at[wave] = first;
        }
        __syncthreads();
        const int w0 = wave & ~(waves - 1);
        m = s_max[w0];
        first = s_at[w0];
        for (int w = 1; w < waves; ++w)
            if (s_max[w0 + w] > m) {  // (the waves' positions increase)
                m = s_max[w0 + w];
                first = s_at[w0 + w];
            }
    }
    const float s = m / A.qmax;
    const float inv = s > 0.0f ? 1.0f / s : 0.0f;
    float sum = 0.0f;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        g[r] *= factor;
        sum = __builtin_fmaf(g[r], (q[r] - v[r]) * inv, sum);
    }
    for (int d = 1; d < in_wave; d <<= 1) sum += __shfl_xor(sum, d, 64);
    if (waves > 1) {
        if ((tid & 63) == 0) s_sum[wave] = sum;
        __syncthreads();
        const int w0 = wave & ~(waves - 1);
        sum = s_sum[w0];
        for (int w = 1; w < waves; ++w) sum += s_sum[w0 + w];
    }
    if (!live) return;
#pragma unroll
    for (int r = 0; r < 8; ++r)
        if (first == tid * 8 + r) {
            const float sign = v[r] > 0.0f ? 1.0f : v[r] < 0.0f ? -1.0f : 0.0f;
            g[r] += sum * sign / A.qmax;
        }
    store8(A.g + at, g);
}

// ---- host side -----------------------------------------------------------------------------------
hipError_t launch_residual_split(const float *e, int64_t rows, int cols, void *pieces, int ld, int dtype, float *result,
                                 void *scratch, hipStream_t stream)
{
    ResidualStats *st = (ResidualStats *)scratch;
    hipLaunchKernelGGL(residual_stats_kernel, dim3(kStatBlocks), dim3(256), 0, stream, e, rows * cols, st);
    SplitArgs A{e, rows, cols, ld, pieces, st, result};
    const unsigned grid = (unsigned)(rows < 2048 ? rows : 2048);
    if (dtype == BQ_F16)
        hipLaunchKernelGGL(residual_split_kernel<__half>, dim3(grid), dim3(256), 0, stream, A);
    else
        hipLaunchKernelGGL(residual_split_kernel<bf16_t>, dim3(grid), dim3(256), 0, stream, A);
    return hipGetLastError();
}

hipError_t launch_quant_grad(const void *v, const void *vq, float *g, const float *factor, const Shape &s, int bits, int group,
                             hipStream_t stream)
{
    QuantGradArgs A{};
    A.v = v;
    A.vq = vq;
    A.g = g;
    A.factor = factor;
    A.total = s.rows * s.n * s.heads;
    A.lanes = group / 8;
    A.qmax = (float)((1 << (bits - 1)) - 1);
    const int threads = A.lanes > 256 ? A.lanes : 256;
    const unsigned grid = (unsigned)((A.total + (int64_t)threads * 8 - 1) / ((int64_t)threads * 8));
    if (s.dtype == BQ_F16)
        hipLaunchKernelGGL(quant_grad_kernel<__half>, dim3(grid), dim3(threads), 0, stream, A);
    else
        hipLaunchKernelGGL(quant_grad_kernel<bf16_t>, dim3(grid), dim3(threads), 0, stream, A);
    return hipGetLastError();
}

}  // namespace bq

// Specialised kernels for small transforms, n = 8 .. 128 (k = 3 .. 7): forward, inverse and fused forward +
// quantisation, for any number of heads.
//
// A transform of n elements occupies n/8 consecutive lanes (at most one 16-lane row), 8 consecutive
// elements per lane, and never touches LDS: layers 1-3 pair registers, layers 4..k pair lanes through
// DPP (bq_cascade.h).  All k*8 scale-deferred coefficients and the 8 output scales of a thread stay
// in registers; a workgroup of up to 256 threads covers up to 2048 consecutive elements: a slice of a wide row
// (e.g. 32 heads x 128) or several narrow rows (e.g. 16 rows of 128, 2 rows of 12 x 64), see small_tiling, and loops
// over the batch with the same coefficients.  Two independent row groups are processed per iteration and the next two are
// prefetched meanwhile, so that four 16-byte loads per lane are in flight.
//
// If the plan flags the scale-deferred tables as unusable, rows go through plain (cos, sin) rotations (rare): the transforms
// hold them in registers, the quantisers, which are short of those, re-read them from the plan for every row.
#include "bq_cascade.h"

namespace bq {

constexpr int kSmallThreads = 256;

struct SmallArgs {
    const void *in;
    void *out;
    const float *fg, *fd;
    const float2 *cs;
    PlanRef plan;
    int64_t rows, ld_in, ld_out;
    int heads, width;    // width = heads * n
    int span, rows_per_block, slices;  // SmallTiling
    int64_t n_groups;    // row groups = ceil(rows / rows_per_block)
    uint8_t *codes;
    void *scales;
    unsigned long long *hist;  // kFwdFake: 2^bits counters or NULL
    int group, scale_f16;
};

// The cascade in plain (cos, sin) rotations held in registers.
// kOwn: rounded as slow_small() rounds them, an element's own product inside the fused operation:
//   y_a = fma(c, x_a, -(s x_b)),  y_b = fma(c, x_b, s x_a)   (transposed: the signs of s swap)
// i.e. fma(w1, own, w2 partner) in either lane of a pair.  Else (forward only) as the kernel for any n rounds them:
//   y_a = fma(c, x_a, -(s x_b)),  y_b = fma(s, x_a, c x_b)
// i.e. fma(w1, x_a, w2 x_b), with the lane's own (w1, w2).
template <int K, bool kInverse, bool kOwn>
struct PlainCascade {
    static_assert(kOwn || !kInverse, "");
    float rc[3][4], rs[3][4];        // layers 1..3: cos and (transposed: minus) sin of the thread's four pairs
    float w1[4][8], w2[4][8];        // layers 4..K
    bool upper[4];                   // this lane holds the upper elements of the layer's pairs
    __device__ __forceinline__ void load(const float2 *cs_head, int idx)
    {
        constexpr int half = 1 << (K - 1);
        auto entry = [&](int e, int i) {  // of the pair that element e belongs to in layer i
            const int h = 1 << (i - 1);
            return cs_head[(size_t)(i - 1) * half + (((e >> i) << (i - 1)) | (e & (h - 1)))];
        };
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            int q = 0;
#pragma unroll
            for (int r = 0; r < 8; ++r)
                if (!(r & (1 << j))) {
                    const float2 w = entry(idx + r, j + 1);
                    rc[j][q] = w.x;
                    rs[j][q] = kInverse ? -w.y : w.y;
                    ++q;
                }
        }
#pragma unroll
        for (int j = 0; j < K - 3; ++j) {
            upper[j] = ((idx >> (3 + j)) & 1) != 0;
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float2 w = entry(idx + r, 4 + j);
                w1[j][r] = !kOwn && upper[j] ? w.y : w.x;
                w2[j][r] = kOwn ? (upper[j] != kInverse ? w.y : -w.y) : (upper[j] ? w.x : -w.y);
            }
        }
    }
    template <int J>
    __device__ __forceinline__ void pairs(float (&u)[8]) const
    {
        int q = 0;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (!(r & (1 << J))) {
                const float xa = u[r], xb = u[r | (1 << J)];
                u[r] = __builtin_fmaf(rc[J][q], xa, -(rs[J][q] * xb));
                u[r | (1 << J)] = kOwn ? __builtin_fmaf(rc[J][q], xb, rs[J][q] * xa) : __builtin_fmaf(rs[J][q], xa, rc[J][q] * xb);
                ++q;
            }
    }
    template <int J, int CTRL>
    __device__ __forceinline__ void lanes(float (&u)[8]) const
    {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const float p = dpp_read<CTRL>(u[r]);
            const float xa = !kOwn && upper[J] ? p : u[r], xb = !kOwn && upper[J] ? u[r] : p;
            u[r] = __builtin_fmaf(w1[J][r], xa, w2[J][r] * xb);
        }
    }
    __device__ __forceinline__ void run(float (&u)[8]) const
    {
        if (!kInverse) {
            pairs<0>(u);
            pairs<1>(u);
            pairs<2>(u);
            if (K >= 4) lanes<0, 0xB1>(u);   // quad_perm [1,0,3,2]
            if (K >= 5) lanes<1, 0x4E>(u);   // quad_perm [2,3,0,1]
            if (K >= 6) lanes<2, 0x141>(u);  // row_half_mirror
            if (K >= 7) lanes<3, 0x128>(u);  // row_ror:8
        } else {
            if (K >= 7) lanes<3, 0x128>(u);
            if (K >= 6) lanes<2, 0x141>(u);
            if (K >= 5) lanes<1, 0x4E>(u);
            if (K >= 4) lanes<0, 0xB1>(u);
            pairs<2>(u);
            pairs<1>(u);
            pairs<0>(u);
        }
    }
};

template <typename T, int K, int kMode, int kBits, bool kPlain = false>
__global__ __launch_bounds__(kSmallThreads) void small_kernel(SmallArgs A)
{
    constexpr int n = 1 << K;
    constexpr bool kInverse = (kMode == kInv);
    const PlanHead ph = plan_head(A.plan);
    if (!ph.matches) return;
    const int tid = threadIdx.x;
    __shared__ unsigned long long wg_bins[16];  // kFwdFake: this workgroup's bin counts
    BinCount<kBits> bins;
    bins.clear();
    if (kMode == kFwdFake) {
        if (tid < 16) wg_bins[tid] = 0;
        __syncthreads();
    }
    auto flush_bins = [&]() {  // every thread gets here
        if (kMode == kFwdFake && A.hist) {
            bins.drain_wave(wg_bins);
            __syncthreads();
            if (tid < (1 << kBits) && wg_bins[tid]) atomicAdd(&A.hist[tid], wg_bins[tid]);
        }
    };
    const int chunk = (tid & ~15) | lane_chunk(tid & 15);  // chunk of 8 elements inside the workgroup's span
    const int e0 = chunk * 8;
    int col;
    int64_t row_in_block, grp_first, grp_step;
    if (A.slices > 1) {
        row_in_block = 0;
        col = (int)(blockIdx.x % A.slices) * A.span + e0;
        grp_first = blockIdx.x / A.slices;
        grp_step = gridDim.x / A.slices;
    } else {
        row_in_block = e0 / A.width;
        col = e0 - (int)row_in_block * A.width;
        grp_first = blockIdx.x;
        grp_step = gridDim.x;
    }
    if (e0 >= A.span || col >= A.width) {  // idle lane (whole transforms are): no row of the batch is its own
        row_in_block = (int64_t)1 << 60;
        col = 0;
    }
    const int head = col >> K;
    const int idx = col & (n - 1);
    const bool fast = (kInverse ? ph.bad_inv : ph.bad_fwd) == 0;

    const float2 *cs_head = A.cs + (size_t)head * K * (n >> 1);
    const T *in = (const T *)A.in;
    const uint32_t col_bytes = (uint32_t)col * (uint32_t)sizeof(T);

    auto row_of = [&](int64_t g) { return g * A.rows_per_block + row_in_block; };
    auto load_row = [&](int64_t g) {
        int64_t row = row_of(g);
        if (row >= A.rows) row = A.rows - 1;  // clamp: the value is not used
        uint32_t off = col_bytes;
        asm volatile("" : "+v"(off));
        return load8((const T *)((const char *)(in + row * A.ld_in) + off));
    };
    auto finish = [&](const float (&y)[8], int64_t g) {
        const int64_t row = row_of(g);
        if (kMode == kFwdFake) {
            const bool live = row < A.rows;  // lanes of a wave may hold different rows
            float f[8], s;
            bool ordinary;
            rounded8<kBits>(y, A.group >> 3, A.scale_f16 != 0, f, &s, &ordinary);
            if (A.hist) {
                if (live)
                    count8<kBits>(bins, f, ordinary);
                else
                    bins.skip();
                if (bins.full()) bins.drain(wg_bins);
            }
            if (A.out && live) {
                float yq[8];
                dequant8(f, s, yq);
                uint32_t off = col_bytes;
                asm volatile("" : "+v"(off));
                store8((T *)((char *)((T *)A.out + row * A.ld_out) + off), yq);
            }
            return;
        }
        if (row >= A.rows) return;
        if (kMode != kFwdQuant) {
            uint32_t off = col_bytes;
            asm volatile("" : "+v"(off));
            store8((T *)((char *)((T *)A.out + row * A.ld_out) + off), y);
        } else {
            const int lanes = A.group >> 3;
            float s;
            const uint32_t packed = quant8<kBits>(y, lanes, A.scale_f16 != 0, &s);
            uint8_t *codes_row = A.codes + row * (int64_t)(A.width * kBits / 8);
            const uint32_t coff = (uint32_t)col * kBits / 8;
            if (kBits == 2)
                *(uint16_t *)(codes_row + coff) = (uint16_t)packed;
            else
                *(uint32_t *)(codes_row + coff) = packed;
            const int64_t sidx = row * (int64_t)(A.width / A.group) + (uint32_t)col / (uint32_t)A.group;
            if (A.scale_f16)
                ((__half *)A.scales)[sidx] = __float2half_rn(s);
            else
                ((float *)A.scales)[sidx] = s;
        }
    };

    if (grp_first >= A.n_groups) return;
    constexpr bool kTransform = kMode == kFwd || kMode == kInv;
    auto plain_rows = [&](auto cascade) {
        cascade.load(cs_head, idx);
        Raw8 raw0 = load_row(grp_first);
        Raw8 raw1 = load_row(grp_first + grp_step);
        for (int64_t g = grp_first; g < A.n_groups; g += grp_step) {
            float u[8];
            unpack8(raw0, u, (const T *)nullptr);
            raw0 = raw1;
            raw1 = load_row(g + 2 * grp_step);
            cascade.run(u);
            finish(u, g);
        }
    };
    if constexpr (kPlain) {
        plain_rows(PlainCascade<K, false, false>());
        flush_bins();
        return;
    }
    if constexpr (kTransform) {
        // (re-read for every row, 20011 rows of 12 x 64 took 213 us, 2.5 times as long as in the LDS kernel these widths had)
        if (!fast) return plain_rows(PlainCascade<K, kInverse, true>());
    }
    if (!kTransform && !fast) {  // rare
        for (int64_t g = grp_first; g < A.n_groups; g += grp_step) {
            float u[8];
            unpack8(load_row(g), u, (const T *)nullptr);
            slow_small<K, kInverse>(u, cs_head, idx);
            finish(u, g);
        }
        flush_bins();
        return;
    }
    float c[7][8], d[8];
    {
        const float *fg = A.fg + (size_t)head * K * n;
#pragma unroll
        for (int j = 0; j < 7; ++j)
#pragma unroll
            for (int r = 0; r < 8; ++r) c[j][r] = (j < K) ? fg[j * n + idx + r] : 0.0f;
#pragma unroll
        for (int r = 0; r < 8; ++r) d[r] = A.fd[(size_t)head * n + idx + r];
    }
    Raw8 raw0 = load_row(grp_first);
    Raw8 raw1 = load_row(grp_first + grp_step);
    for (int64_t g = grp_first; g < A.n_groups; g += 2 * grp_step) {
        float u0[8], u1[8];
        unpack8(raw0, u0, (const T *)nullptr);
        unpack8(raw1, u1, (const T *)nullptr);
        raw0 = load_row(g + 2 * grp_step);
        raw1 = load_row(g + 3 * grp_step);
        fast_small<K, kInverse>(u0, c, d);
        fast_small<K, kInverse>(u1, c, d);
        finish(u0, g);
        if (g + grp_step < A.n_groups) finish(u1, g + grp_step);
    }
    flush_bins();
}

template <typename T, int K>
static void (*pick_small(Mode mode, int bits, bool plain))(SmallArgs)
{
    if (mode == kFwd) return small_kernel<T, K, kFwd, 4>;
    if (mode == kInv) return small_kernel<T, K, kInv, 4>;
    if (plain) {
        if (mode == kFwdFake) return bits == 2 ? small_kernel<T, K, kFwdFake, 2, true> : small_kernel<T, K, kFwdFake, 4, true>;
        return bits == 2 ? small_kernel<T, K, kFwdQuant, 2, true> : small_kernel<T, K, kFwdQuant, 4, true>;
    }
    if (mode == kFwdFake) return bits == 2 ? small_kernel<T, K, kFwdFake, 2> : small_kernel<T, K, kFwdFake, 4>;
    return bits == 2 ? small_kernel<T, K, kFwdQuant, 2> : small_kernel<T, K, kFwdQuant, 4>;
}

template <typename T>
static void (*pick_small_k(int k, Mode mode, int bits, bool plain))(SmallArgs)
{
    switch (k) {
        case 3: return pick_small<T, 3>(mode, bits, plain);
        case 4: return pick_small<T, 4>(mode, bits, plain);
        case 5: return pick_small<T, 5>(mode, bits, plain);
        case 6: return pick_small<T, 6>(mode, bits, plain);
        default: return pick_small<T, 7>(mode, bits, plain);
    }
}

// Workgroups of one to four waves.  Rows of up to 2048 elements: as many whole rows as fit; wider rows: slices of whole
// heads.  The number of waves is the one that leaves the fewest lanes idle (none for widths that divide 2048, for multiples
// of 512, and for 2 rows of 768 or 16 rows of 96 elements; 6 % for 3 rows of 640), the larger at equal shares.  Widths with
// idle lanes went to the LDS kernel for any n before: 20011 fp16 rows of 12 x 64, forward, 81 -> 13 us, and
// 574 -> 40 us backward.  The backward kernel holds eight waves per compute unit, of which three-wave workgroups fill six:
// they count as four there (10000 rows of 12 x 128: 80 us in three-wave workgroups, 62 us in single-wave ones).
//
// At equal shares three waves come last unless few_workgroups: 2048 waves are 682 workgroups of three, of which a compute unit
// gets two or three (87382 rows of 12 x 128: float32 forward 226 us in workgroups of three waves, 211 us in slices of one;
// fp16 INT4 83 and 75).  A call that counts bins ends with one atomic per bin and workgroup and wants few of them (2731
// rows, fp16 INT4 43 and 108 us, float32 19 and 35), float32 rows up to 2^26 elements (87382 rows 239 and 225).
SmallTiling small_tiling(int n, int heads, bool backward, bool few_workgroups)
{
    const int64_t width = (int64_t)n * heads;
    SmallTiling best{};
    int64_t best_lanes = 0, best_used = 0;  // lanes spent on so many elements
    for (const int waves : {4, few_workgroups ? 3 : 2, few_workgroups ? 2 : 1, few_workgroups ? 1 : 3}) {
        SmallTiling t{};
        t.threads = waves * 64;
        const int room = t.threads * 8;
        const int cost = backward && waves == 3 ? 256 : t.threads;
        int64_t used, lanes;
        if (width <= room) {
            t.rows_per_block = (int)(room / width);
            t.slices = 1;
            t.span = (int)(t.rows_per_block * width);
            used = t.span;
            lanes = cost;
        } else {
            const int most = room / n;  // heads per slice
            t.rows_per_block = 1;
            t.slices = (heads + most - 1) / most;
            t.span = (heads + t.slices - 1) / t.slices * n;
            used = width;
            lanes = (int64_t)t.slices * cost;
        }
        if (best_lanes == 0 || used * best_lanes > best_used * lanes) {
            best = t;
            best_lanes = lanes;
            best_used = used;
        }
    }
    return best;
}

bool small_supported(Mode mode, const void *in, const void *out, const Shape &s, const QuantArgs *q)
{
    if (s.k < 3 || s.k > 7) return false;
    const int isz = s.dtype == BQ_F32 ? 4 : 2;
    const int vec = 16 / isz;
    if (((uintptr_t)in & 15) || (s.ld_x % vec)) return false;
    if (mode != kFwdQuant && out && (((uintptr_t)out & 15) || (s.ld_y % vec))) return false;
    if (mode == kFwdQuant || mode == kFwdFake) {
        if (q->group > s.n) return false;
        if (mode == kFwdQuant && ((uintptr_t)q->codes & 3)) return false;
    }
    return true;
}

hipError_t launch_small(Mode mode, const void *in, void *out, const PlanView &pv, const Shape &s,
                        const QuantArgs *q, hipStream_t stream)
{
    SmallArgs A{};
    A.in = in;
    A.out = out;
    A.fg = mode == kInv ? pv.fg_inv : pv.fg_fwd;
    A.fd = mode == kInv ? pv.fd_inv : pv.fd_fwd;
    A.cs = pv.cs;
    A.plan = pv.ref;
    A.rows = s.rows;
    A.ld_in = s.ld_x;
    A.ld_out = s.ld_y;
    A.heads = s.heads;
    A.width = s.n * s.heads;
    const bool counts = mode == kFwdFake && q->hist != nullptr;
    SmallTiling t = small_tiling(s.n, s.heads, false, counts && (s.dtype != BQ_F32 || s.rows * A.width < (int64_t)1 << 26));
    // the plain transforms of 16-bit rows stream fastest from single-wave workgroups (measured: up to 20 % over
    // four-wave ones at the same number of waves; float32 rows and the quantisers prefer the wider ones)
    if ((mode == kFwd || mode == kInv) && s.dtype != BQ_F32 && (A.width % 512 == 0 || 512 % A.width == 0))
        t = SmallTiling{64, 512, A.width < 512 ? 512 / A.width : 1, A.width < 512 ? 1 : A.width / 512};
    A.span = t.span;
    A.rows_per_block = t.rows_per_block;
    A.slices = t.slices;
    A.n_groups = (s.rows + A.rows_per_block - 1) / A.rows_per_block;
    int bits = 4;
    if (q) {
        A.codes = q->codes;
        A.scales = q->scales;
        A.hist = q->hist;
        A.group = q->group;
        A.scale_f16 = q->scale_f16;
        bits = q->bits;
    }
    // Persistent workgroups, a multiple of the slice count.  How many waves stream best was measured per mode
    // (262144 rows of 32 x 128): the plain transforms and everything on float32 rows with 2048 waves (8 per
    // compute unit: 5.5 TB/s against 4.4 TB/s with four times as many), the 16-bit quantisers, which need the
    // occupancy to hide their arithmetic, with 8192.
    const bool few = mode == kFwd || mode == kInv || s.dtype == BQ_F32;
    const int64_t wgs = (few ? 2048 : 8192) / (t.threads / 64);
    int64_t per_slice = wgs / A.slices > 0 ? wgs / A.slices : 1;
    if (per_slice > A.n_groups) per_slice = A.n_groups;
    const unsigned grid = (unsigned)(per_slice * A.slices);
    // The quantisers of widths that went to the LDS kernel before (all but divisors of 2048 and multiples of 512) keep its plain
    // rotations, bit for bit, in every row of a batch: the deferred form's last bit would move a few codes in 10^6 across a
    // rounding boundary, each of them by a whole step.  20011 fp16 rows of 12 x 64, INT4: 96 us there, 24 us here (14.5 in the
    // deferred form: the plain one takes two operations per element and layer, five where a pair sits in two lanes).
    const bool plain = 2048 % A.width != 0 && A.width % 512 != 0;
    void (*kern)(SmallArgs) = s.dtype == BQ_F32   ? pick_small_k<float>(s.k, mode, bits, plain)
                              : s.dtype == BQ_F16 ? pick_small_k<__half>(s.k, mode, bits, plain)
                                                  : pick_small_k<bf16_t>(s.k, mode, bits, plain);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(t.threads), 0, stream, A);
    return hipGetLastError();
}

}  // namespace bq

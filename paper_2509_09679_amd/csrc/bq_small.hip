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
// If the plan flags the scale-deferred tables as unusable, rows go through plain (cos, sin) rotations (rare).
#include "bq_cascade.h"

namespace bq {

constexpr int kSmallThreads = 256;

struct SmallArgs {
    const void *in;
    void *out;
    const float *fg, *fd;
    const float2 *cs;
    PlanRef plan;
    int64_t group_in, group_out;  // bytes from one row group to the next
    uint32_t row_in, row_out;     // ... and from row to row of a group
    int heads, width;    // width = heads * n
    int span, rows_per_block, slices;  // SmallTiling
    int n_groups;        // row groups = ceil(rows / rows_per_block); < 2^31: each is about a kilobyte or more
    int last_rows;       // rows of the last group
    uint8_t *codes;
    void *scales;
    unsigned long long *hist;  // kFwdFake: 2^bits counters or NULL
    int group, scale_f16;
};

// kWhole: quantiser groups of n channels (else any that divide n)
template <typename T, int K, int kMode, int kBits, bool kPlain = false, bool kWhole = false>
// (four waves per SIMD: the quantisers fill them; without the bound some end up a few registers above 128)
__global__ __launch_bounds__(kSmallThreads, kMode == kFwd || kMode == kInv || (kPlain && kMode == kFwdFake && sizeof(T) == 4) ? 1 : 4) void small_kernel(SmallArgs A)
{
    constexpr int n = 1 << K;
    constexpr bool kInverse = (kMode == kInv);
    const PlanHead ph = plan_head(A.plan);  // (looked at below: the scalar arithmetic up to there passes in its latency)
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
            bins.template drain_wave<long long>(wg_bins);
            __syncthreads();
            if (tid < (1 << kBits) && wg_bins[tid]) atomicAdd(&A.hist[tid], wg_bins[tid]);
        }
    };
    const int chunk = (tid & ~15) | lane_chunk(tid & 15);  // chunk of 8 elements inside the workgroup's span
    const int e0 = chunk * 8;
    // Everything about a row but the lane's place in its group is uniform: rows are addressed as a scalar base per group, which moves
    // on by a constant, and a 32-bit offset per lane.  (With a 64-bit row number per lane, the four 64-bit products and comparisons
    // of a row were a tenth of its vector cycles; with a product per group, transforms of 2^22 elements took 4 to 9 % longer.)
    int col, row_in_group = 0, grp_first, grp_step;
    if (A.slices > 1) {
        col = (int)(blockIdx.x % A.slices) * A.span + e0;
        grp_first = (int)blockIdx.x / A.slices;
        grp_step = (int)gridDim.x / A.slices;
    } else {
        row_in_group = e0 / A.width;
        col = e0 - row_in_group * A.width;
        grp_first = (int)blockIdx.x;
        grp_step = (int)gridDim.x;
    }
    const bool idle = e0 >= A.span || col >= A.width;  // idle lane (whole transforms are): no row of the batch is its own
    if (idle) row_in_group = col = 0;
    const bool in_last = !idle && row_in_group < A.last_rows;  // its row exists in the last group, too
    const int last = A.n_groups - 1;
    const uint32_t col_bytes = (uint32_t)col * (uint32_t)sizeof(T);
    const uint32_t off_in = (uint32_t)row_in_group * A.row_in + col_bytes, off_out = (uint32_t)row_in_group * A.row_out + col_bytes;

    const int groups = kMode == kFwdQuant ? A.width / A.group : 0;  // quantiser groups of a row
    const uint32_t off_code = (uint32_t)(row_in_group * (A.width * kBits / 8) + col * kBits / 8);
    const uint32_t off_scale = kMode == kFwdQuant ? (uint32_t)(row_in_group * groups + col / A.group) : 0u;
    struct Place {  // of a row group: byte offsets of its rows and outputs
        int64_t in, out, code, scale;
    };
    const int64_t code_bytes = (int64_t)A.rows_per_block * (A.width * kBits / 8), scale_bytes = (int64_t)A.rows_per_block * groups * (A.scale_f16 ? 2 : 4);
    Place at = {grp_first * A.group_in, grp_first * A.group_out, grp_first * code_bytes, grp_first * scale_bytes};
    const Place step = {grp_step * A.group_in, grp_step * A.group_out, grp_step * code_bytes, grp_step * scale_bytes};
    auto load_row = [&](int g, int64_t in) {
        uint32_t off = off_in;
        if (g == last && !in_last) off = col_bytes;  // no such row: the group's first (the value is not used)
        if (g > last) in = off = 0;                  // past the end: one cache line (not used either)
        asm volatile("" : "+v"(off));
        return load8((const T *)((const char *)A.in + in + off));
    };
    if (grp_first >= A.n_groups || !ph.matches) return;
    const int head = col >> K;
    const int idx = col & (n - 1);
    const bool fast = (kInverse ? ph.bad_inv : ph.bad_fwd) == 0;

    const float2 *cs_head = A.cs + (size_t)head * K * (n >> 1);
    auto finish = [&](const float (&y)[8], int g, const Place &p) {
        const bool live = g == last ? in_last : !idle;  // lanes of a wave may hold different rows
        const int lanes = kWhole ? n / 8 : A.group >> 3;
        if (kMode == kFwdFake) {
            float f[8], s;
            bool ordinary;
            rounded8<kBits>(y, lanes, A.scale_f16 != 0, f, &s, &ordinary);
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
                uint32_t off = off_out;
                asm volatile("" : "+v"(off));
                store8((T *)((char *)A.out + p.out + off), yq);
            }
            return;
        }
        if (!live) return;
        if (kMode != kFwdQuant) {
            uint32_t off = off_out;
            asm volatile("" : "+v"(off));
            store8((T *)((char *)A.out + p.out + off), y);
        } else {
            float s;
            const uint32_t packed = quant8<kBits>(y, lanes, A.scale_f16 != 0, &s);
            uint32_t coff = off_code;
            asm volatile("" : "+v"(coff));
            uint8_t *codes = A.codes + p.code + coff;
            if (kBits == 2)
                *(uint16_t *)codes = (uint16_t)packed;
            else
                *(uint32_t *)codes = packed;
            uint32_t soff = off_scale;
            asm volatile("" : "+v"(soff));
            char *scales = (char *)A.scales + p.scale;
            if (A.scale_f16)
                *((__half *)scales + soff) = __float2half_rn(s);
            else
                *((float *)scales + soff) = s;
        }
    };
    auto advance = [&](int64_t groups_on) {
        at.in += groups_on * step.in;
        if (kMode != kFwdQuant) at.out += groups_on * step.out;
        if (kMode == kFwdQuant) {
            at.code += groups_on * step.code;
            at.scale += groups_on * step.scale;
        }
    };

    auto plain_rows = [&](auto cascade) {
        cascade.load(cs_head, idx);
        Raw8 raw0 = load_row(grp_first, at.in);
        Raw8 raw1 = load_row(grp_first + grp_step, at.in + step.in);
        for (int g = grp_first; g < A.n_groups; g += grp_step) {
            float u[8];
            unpack8(raw0, u, (const T *)nullptr);
            raw0 = raw1;
            raw1 = load_row(g + 2 * grp_step, at.in + 2 * step.in);
            cascade.run(u);
            finish(u, g, at);
            advance(1);
        }
    };
    if constexpr (kPlain) {
        plain_rows(PlainCascade<K, false, false>());
        flush_bins();
        return;
    }
    // rare: a flagged plan.  (Re-read for every row, 20011 rows of 12 x 64, forward, took 213 us, 8192 rows of 32 x 128, fp16 INT4, 402;
    // held in registers 18 and 30.5.)
    if (!fast) {
        plain_rows(PlainCascade<K, kInverse, true>());
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
    Raw8 raw0 = load_row(grp_first, at.in);
    Raw8 raw1 = load_row(grp_first + grp_step, at.in + step.in);
    for (int g = grp_first; g < A.n_groups; g += 2 * grp_step) {
        float u0[8], u1[8];
        unpack8(raw0, u0, (const T *)nullptr);
        unpack8(raw1, u1, (const T *)nullptr);
        raw0 = load_row(g + 2 * grp_step, at.in + 2 * step.in);
        raw1 = load_row(g + 3 * grp_step, at.in + 3 * step.in);
        fast_small<K, kInverse>(u0, c, d);
        fast_small<K, kInverse>(u1, c, d);
        finish(u0, g, at);
        advance(1);
        if (g + grp_step < A.n_groups) finish(u1, g + grp_step, at);
        advance(1);
    }
    flush_bins();
}

template <typename T, int K>
static void (*pick_small(Mode mode, int bits, bool plain, bool whole))(SmallArgs)
{
    if (mode == kFwd) return small_kernel<T, K, kFwd, 4>;
    if (mode == kInv) return small_kernel<T, K, kInv, 4>;
    if (plain) {
        if (mode == kFwdFake) return bits == 2 ? small_kernel<T, K, kFwdFake, 2, true> : small_kernel<T, K, kFwdFake, 4, true>;
        if (whole) return bits == 2 ? small_kernel<T, K, kFwdQuant, 2, true, true> : small_kernel<T, K, kFwdQuant, 4, true, true>;
        return bits == 2 ? small_kernel<T, K, kFwdQuant, 2, true> : small_kernel<T, K, kFwdQuant, 4, true>;
    }
    if (mode == kFwdFake) return bits == 2 ? small_kernel<T, K, kFwdFake, 2> : small_kernel<T, K, kFwdFake, 4>;
    if (whole) return bits == 2 ? small_kernel<T, K, kFwdQuant, 2, false, true> : small_kernel<T, K, kFwdQuant, 4, false, true>;
    return bits == 2 ? small_kernel<T, K, kFwdQuant, 2> : small_kernel<T, K, kFwdQuant, 4>;
}

template <typename T>
static void (*pick_small_k(int k, Mode mode, int bits, bool plain, bool whole))(SmallArgs)
{
    switch (k) {
        case 3: return pick_small<T, 3>(mode, bits, plain, whole);
        case 4: return pick_small<T, 4>(mode, bits, plain, whole);
        case 5: return pick_small<T, 5>(mode, bits, plain, whole);
        case 6: return pick_small<T, 6>(mode, bits, plain, whole);
        default: return pick_small<T, 7>(mode, bits, plain, whole);
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
    A.heads = s.heads;
    A.width = s.n * s.heads;
    const bool counts = mode == kFwdFake && q->hist != nullptr;
    SmallTiling t = small_tiling(s.n, s.heads, false, counts && (s.dtype != BQ_F32 || s.rows * A.width < (int64_t)1 << 26));
    // the plain transforms of 16-bit rows stream fastest from single-wave workgroups (measured: up to 20 % over
    // four-wave ones at the same number of waves; float32 rows and the quantisers prefer the wider ones)
    if ((mode == kFwd || mode == kInv) && s.dtype != BQ_F32 && (A.width % 512 == 0 || 512 % A.width == 0))
        t = SmallTiling{64, 512, A.width < 512 ? 512 / A.width : 1, A.width < 512 ? 1 : A.width / 512};
    // a lane's offset inside a row group has 32 bits: rows further apart than that are groups of their own
    const int64_t isz = s.dtype == BQ_F32 ? 4 : 2;
    if (t.slices == 1 && t.rows_per_block * (s.ld_x > s.ld_y ? s.ld_x : s.ld_y) * isz >= (int64_t)1 << 32) {
        t.rows_per_block = 1;
        t.span = A.width;
    }
    A.span = t.span;
    A.rows_per_block = t.rows_per_block;
    A.slices = t.slices;
    A.n_groups = (int)((s.rows + A.rows_per_block - 1) / A.rows_per_block);
    A.last_rows = (int)(s.rows - (int64_t)(A.n_groups - 1) * A.rows_per_block);
    A.row_in = (uint32_t)(s.ld_x * isz);
    A.row_out = (uint32_t)(s.ld_y * isz);
    A.group_in = A.rows_per_block * s.ld_x * isz;
    A.group_out = A.rows_per_block * s.ld_y * isz;
    int bits = 4;
    if (q) {
        A.codes = q->codes;
        A.scales = q->scales;
        A.hist = q->hist;
        A.group = q->group;
        A.scale_f16 = q->scale_f16;
        bits = q->bits;
    }
    // The quantisers of widths that went to the LDS kernel before (all but divisors of 2048 and multiples of 512) keep its plain
    // rotations, bit for bit, in every row of a batch: the deferred form's last bit would move a few codes in 10^6 across a
    // rounding boundary, each of them by a whole step.  20011 fp16 rows of 12 x 64, INT4: 96 us there, 24 us here (14.5 in the
    // deferred form: the plain one takes two operations per element and layer, five where a pair sits in two lanes).
    const bool plain = 2048 % A.width != 0 && A.width % 512 != 0;
    // Persistent workgroups, a multiple of the slice count.  How many waves run best was measured, in us at 2^22, 2^24, 2^25 and 2^27
    // elements of 32 x 128 (plain rotations: 12 x 64):
    //   transforms      2048 (8 per compute unit: 5.5 TB/s, 4.4 with four times as many)
    //   bf16 INT4       8192 8.7 14.4 21.2 74.2 | 4096 6.1 13.2 20.5 75.0 | 3072 5.7 12.8 20.6 78.4 | 2048 5.6 13.4 22.3 93.5
    //   plain rotations 8192 13.6 21.8 32.5 115 | 4096 9.8 21.1 35.2 128 | 3072 8.6 19.0 31.3 118 | 2048 9.1 24.0 42.5 161
    //   float32 INT4    4096 7.8 16.2 32.9 126 | 3072 7.4 16.0 32.3 118 | 2048 7.4 16.2 31.1 115 | 1024 7.8 19.7 40.0 135
    //   plain rotations 4096 10.6 21.7 44.9 180 | 3072 9.0 19.5 35.4 129 | 2048 9.8 24.0 45.1 164
    //   bf16 values     8192 10.1 17.6 33.6 115 | 4096 7.5 16.7 32.0 115 | 3072 7.1 15.3 30.4 109 | 2048 7.1 16.2 32.0 111
    //   ... and counts  8192 35.0 38.7 47.1 124 | 4096 21.2 28.8 37.8 121 | 3072 19.1 25.2 36.8 115 | 2048 16.2 24.5 41.4 132
    //   float32 values  3072 9.6 31.3 56.9 213 | 2048 10.0 29.8 55.3 211 | 1024 9.8 28.1 50.9 187
    const int64_t elements = s.rows * A.width;
    int waves = 2048;
    if (mode == kFwdQuant || mode == kFwdFake) {
        if (s.dtype == BQ_F32)
            waves = plain ? (elements < (int64_t)1 << (counts ? 25 : 22) ? 2048 : 3072) : mode == kFwdFake && !counts ? 1024 : 2048;
        else if (elements >= (int64_t)1 << 23)
            waves = mode == kFwdFake || elements < (int64_t)3 << 23 ? 3072 : !plain ? 4096 : elements < (int64_t)1 << 26 ? 3072 : 8192;
    }
    int64_t per_slice = waves / (t.threads / 64) / A.slices;
    // A workgroup takes two row groups at a time (in plain rotations one, but counts make it want fewer): as many workgroups as groups leave it half empty (2^20 elements, forward 3.8 us, with
    // half as many 3.2; INT4 4.2 and 3.7), which they may where there are compute units to spare.
    if (per_slice * 2 > A.n_groups && (counts || !plain || mode == kFwd || mode == kInv)) per_slice = (A.n_groups + 1) / 2;
    if (per_slice < 256 / A.slices) per_slice = 256 / A.slices;
    if (per_slice < 1) per_slice = 1;
    if (per_slice > A.n_groups) per_slice = A.n_groups;
    const unsigned grid = (unsigned)(per_slice * A.slices);
    const bool whole = q && q->group == s.n;
    void (*kern)(SmallArgs) = s.dtype == BQ_F32   ? pick_small_k<float>(s.k, mode, bits, plain, whole)
                              : s.dtype == BQ_F16 ? pick_small_k<__half>(s.k, mode, bits, plain, whole)
                                                  : pick_small_k<bf16_t>(s.k, mode, bits, plain, whole);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(t.threads), 0, stream, A);
    return hipGetLastError();
}

}  // namespace bq

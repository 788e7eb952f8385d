// Backward pass for small transforms, n = 8 .. 128 (k = 3 .. 7), for any number of heads: dx = B^T dy and dtheta (paper, "Gradient Flow Through Butterfly Layers").
//
// Geometry of the small forward kernels (bq_small.hip): a transform occupies n/8 consecutive lanes, 8
// consecutive elements per lane, no LDS and no barrier; a workgroup of up to 256 threads covers up to 2048 consecutive
// elements (a slice of a wide row or several narrow rows, small_tiling) and loops over the batch.  Per row a thread
// recomputes the forward state of its 8 elements (layers 1..k), then runs the transposed cascade on the
// state and the gradient together with the deferred sums of bq_bwd_blocks.h.  Everything a thread needs
// for that (both directions' coefficients, 44 sums) stays in registers: about 230 of them, so two waves
// share a SIMD; the loop has no dependence on LDS or barriers to hide.
//
// Partial sums: every (workgroup, row position inside its span) pair owns one slot of `partial` holding all
// angles; an entry is written by exactly one thread.  A second kernel adds the slots in double in a fixed
// order: no atomics, the result does not depend on scheduling.
//
// When the plan flags the scale-deferred tables as unusable, workgroups of 256 threads run the backward pass for any n instead
// (bq_generic_bwd.h); narrower ones exit and leave it to a launch of its own (2 us of every call on other plans; in 64 threads that
// pass would take longer).  The second kernel adds those sums.
#include "bq_bwd_blocks.h"
#include "bq_generic_bwd.h"
#include "bq_internal.h"

namespace bq {

constexpr int kSbThreads = 256;
constexpr int kSbMaxSlots = 4096;  // (8192: 200000 rows of 128 unchanged at 60 us, 8192 rows 26 -> 39 us)

// With no more slices than this a launch has at most 2048 waves, so the slots hold at most 2048 x 512 elements' angles
// (14 MiB at n = 128): below the 32 MiB of the entry point that brings its own workspace.
constexpr int kSbMaxSlices = 512;

struct SmallBwdArgs {
    const void *x, *dy;
    void *dx;
    float *partial;  // [slots][n_angles]
    const float *fg_fwd, *fd_fwd, *fg_inv, *fd_inv, *fw_inv;
    PlanRef plan;
    int64_t rows, ld_in, ld_out;
    int heads, width;    // width = heads * n
    int span, rows_per_block, slices;  // SmallTiling
    int64_t n_groups;    // row groups = ceil(rows / rows_per_block)
    int64_t n_angles;    // heads * k * n / 2
    int grid;            // workgroups; a launch may have more, which only help on flagged plans
    int plain_parts;     // flagged plans: the workgroups that take part, each with a slice of its own; 0: a launch of its own does
};
constexpr int kSbPlainTile = 1024;  // elements of a tile of that pass at n <= 128

template <typename T, int K, bool kDx>
__global__ __launch_bounds__(kSbThreads) void small_bwd_kernel(SmallBwdArgs A, BwdArgs P)
{
    constexpr int n = 1 << K;
    __shared__ float plain_tile[2 * kSbPlainTile];
    const PlanUse use = plan_use(A.plan);
    if (use == kPlanForeign) return;
    if (use == kPlanPlain) {
        if ((int)blockIdx.x < A.plain_parts) generic_bwd_rows<T, kSbThreads>(P, plain_tile, (int)blockIdx.x, A.plain_parts);
        return;
    }
    if ((int)blockIdx.x >= A.grid) return;
    const int tid = threadIdx.x;
    const int chunk = (tid & ~15) | lane_chunk(tid & 15);  // chunk of 8 elements inside the workgroup's span
    const int e0 = chunk * 8;
    int col;
    int64_t row_in_block, grp_first, grp_step, slot;
    if (A.slices > 1) {
        row_in_block = 0;
        col = (int)(blockIdx.x % A.slices) * A.span + e0;
        grp_first = blockIdx.x / A.slices;
        grp_step = A.grid / A.slices;
        slot = grp_first;
    } else {
        row_in_block = e0 / A.width;
        col = e0 - (int)row_in_block * A.width;
        grp_first = blockIdx.x;
        grp_step = A.grid;
        slot = (int64_t)blockIdx.x * A.rows_per_block + row_in_block;
    }
    const bool idle = e0 >= A.span || col >= A.width;  // no row of the batch and no slot is this lane's own
    if (idle) {
        row_in_block = (int64_t)1 << 60;
        col = 0;
    }
    const int head = col >> K;
    const int idx = col & (n - 1);
    const uint32_t col_bytes = (uint32_t)col * (uint32_t)sizeof(T);

    float cf[7][8], df[8], di[8];
    CoefRegs ci;
    {
        const float *ff = A.fg_fwd + (size_t)head * K * n, *fi = A.fg_inv + (size_t)head * K * n;
#pragma unroll
        for (int j = 0; j < 7; ++j)
#pragma unroll
            for (int r = 0; r < 8; ++r) {  // layers above k do not exist: weight zero leaves the element as it is
                cf[j][r] = (j < K) ? ff[j * n + idx + r] : 0.0f;
                ci.c[j][r] = (j < K) ? fi[j * n + idx + r] : 0.0f;
            }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            df[r] = A.fd_fwd[(size_t)head * n + idx + r];
            di[r] = A.fd_inv[(size_t)head * n + idx + r];
        }
    }
    NAcc acc;
    acc.clear();

    auto row_of = [&](int64_t g) { return g * A.rows_per_block + row_in_block; };
    auto load_row = [&](const void *base, int64_t g) {
        int64_t row = row_of(g);
        if (row >= A.rows) row = A.rows - 1;  // clamp (in bounds); such a row gets a zero gradient below
        uint32_t off = col_bytes;
        asm volatile("" : "+v"(off));
        return load8((const T *)((const char *)((const T *)base + row * A.ld_in) + off));
    };
    if (grp_first < A.n_groups) {
        Raw8 rx = load_row(A.x, grp_first), rg = load_row(A.dy, grp_first);
        for (int64_t g = grp_first; g < A.n_groups; g += grp_step) {
            float vx[8], vg[8];
            unpack8(rx, vx, (const T *)nullptr);
            unpack8(rg, vg, (const T *)nullptr);
            const int64_t nxt = g + grp_step < A.n_groups ? g + grp_step : g;
            rx = load_row(A.x, nxt);
            rg = load_row(A.dy, nxt);
            const int64_t row = row_of(g);
            const bool live = row < A.rows;  // lanes of a wave may hold different rows
            if (!live) {
#pragma unroll
                for (int r = 0; r < 8; ++r) vg[r] = 0.0f;
            }
            fast_small<K, false>(vx, cf, df);  // x_k
            n_phase(vx, vg, ci, acc);
            if (kDx && live) {
#pragma unroll
                for (int r = 0; r < 8; ++r) vg[r] *= di[r];
                uint32_t off = col_bytes;
                asm volatile("" : "+v"(off));
                store8((T *)((char *)((T *)A.dx + row * A.ld_out) + off), vg);
            }
        }
    }
    // deferred sums -> this slot's entries (workgroups without rows write zeros)
    if (idle) return;  // (whole transforms are idle, so no partner is missing below)
    float *part = A.partial + slot * A.n_angles + (size_t)head * K * (n / 2);
#pragma unroll
    for (int J = 0; J < 3; ++J) {  // layers 1..3: pairs of registers
        const int i = J + 1;
        int q = 0;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (!(r & (1 << J))) {
                const int a = idx + r;
                part[(i - 1) * (n / 2) + pair_index(a, i)] = acc.r[J][q];
                ++q;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // layers 4..7: pairs of lanes (masks 1, 2, 7, 8)
        const int i = 4 + j;
        if (i > K) continue;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const float mine = acc.d[j][r];
            const float other = lane_partner(mine, j);
            const int e = idx + r;
            if (!(e & (1 << (i - 1)))) {  // the lane holding the lower element writes
                part[(i - 1) * (n / 2) + pair_index(e, i)] = mine - other;
            }
        }
    }
}

// dtheta[q] = sum over slots of partial[slot][q], in double, times the angle's scale: a workgroup takes 16 angles (64 bytes of a slot), its 64 groups
// of 16 threads take every 64th slot each and their sums are added in group order.  A serial chain of loads per thread: with
// 32 angles and 8 groups of 256 threads, 4096 slots of n = 128 ran 14 workgroups of 512
// loads each (whole backward pass of 8192 fp16 rows of 128: 156 -> 26 us).  Flagged
// plans: the same over the generic kernel's plain_slots slices.
constexpr int kSbReduceAngles = 16, kSbReduceGroups = 64;
__global__ __launch_bounds__(kSbReduceAngles * kSbReduceGroups) void small_bwd_reduce_kernel(
    const float *__restrict__ partial, float *__restrict__ dtheta, int64_t n_angles, int64_t slots, PlanRef plan, int64_t plain_slots,
    const float *__restrict__ fw_inv, int k)
{
    const PlanUse use = plan_use(plan);
    if (use == kPlanForeign) return;
    if (use == kPlanPlain) slots = plain_slots;
    __shared__ double sums[kSbReduceGroups][kSbReduceAngles];
    const int lane = threadIdx.x % kSbReduceAngles, grp = threadIdx.x / kSbReduceAngles;
    const int64_t q = (int64_t)blockIdx.x * kSbReduceAngles + lane;
    double acc = 0.0, scale = 1.0;
    if (grp == 0 && q < n_angles && use == kPlanFast) {
        const int layer = (int)(q >> (k - 1));  // counted through the heads
        scale = sum_scale(fw_inv, k, layer / k, layer % k + 1, (int)q & ((1 << (k - 1)) - 1), false);
    }
    if (q < n_angles) {
#pragma unroll 8
        for (int64_t s = grp; s < slots; s += kSbReduceGroups) acc += (double)partial[s * n_angles + q];
    }
    sums[grp][lane] = acc;
    __syncthreads();
    if (grp == 0 && q < n_angles) {
        double t = sums[0][lane];
        for (int g = 1; g < kSbReduceGroups; ++g) t += sums[g][lane];
        dtheta[q] = (float)(t * scale);
    }
}

// ---- host side -----------------------------------------------------------------------------------
struct SmallBwdGrid {
    SmallTiling t;
    int64_t n_groups, slots;
    unsigned grid;
};

static SmallBwdGrid small_bwd_grid(const Shape &s)
{
    SmallBwdGrid g;
    g.t = small_tiling(s.n, s.heads, true, true);
    g.n_groups = (s.rows + g.t.rows_per_block - 1) / g.t.rows_per_block;
    // 2048 waves, eight per compute unit (all that fit with these kernels' registers), whatever the workgroup width;
    // the slot count (partial sums to write and to add) stays bounded
    const int64_t wgs = 2048 / (g.t.threads / 64);
    int64_t per_slice = wgs / g.t.slices > 0 ? wgs / g.t.slices : 1;
    if (per_slice * g.t.rows_per_block > kSbMaxSlots) per_slice = kSbMaxSlots / g.t.rows_per_block;
    if (per_slice > g.n_groups) per_slice = g.n_groups;
    g.grid = (unsigned)(per_slice * g.t.slices);
    g.slots = per_slice * g.t.rows_per_block;
    return g;
}

bool small_bwd_supported(const void *x, const void *dy, const void *dx, const float *dtheta, const Shape &s)
{
    if (s.k < 3 || s.k > 7 || dtheta == nullptr || s.rows == 0) return false;
    if (small_tiling(s.n, s.heads, true, true).slices > kSbMaxSlices) return false;
    const int vec = s.dtype == BQ_F32 ? 4 : 8;
    if (((uintptr_t)x & 15) || ((uintptr_t)dy & 15) || (dx && ((uintptr_t)dx & 15))) return false;
    if ((s.ld_x % vec) || (s.ld_y % vec)) return false;
    return true;
}

size_t small_bwd_workspace_bytes(const Shape &s)
{
    const SmallBwdGrid g = small_bwd_grid(s);
    if (g.t.slices > kSbMaxSlices) return 0;  // not a shape of these kernels
    return align256((size_t)g.slots * s.heads * s.k * (s.n / 2) * sizeof(float));
}

template <typename T, int K>
static void launch_small_bwd_k(const SmallBwdArgs &A, const BwdArgs &P, unsigned grid, int threads, hipStream_t stream)
{
    if (A.dx)
        hipLaunchKernelGGL((small_bwd_kernel<T, K, true>), dim3(grid), dim3(threads), 0, stream, A, P);
    else
        hipLaunchKernelGGL((small_bwd_kernel<T, K, false>), dim3(grid), dim3(threads), 0, stream, A, P);
}

template <typename T>
static void launch_small_bwd_t(const SmallBwdArgs &A, const BwdArgs &P, int k, unsigned grid, int threads, hipStream_t stream)
{
    switch (k) {
        case 3: return launch_small_bwd_k<T, 3>(A, P, grid, threads, stream);
        case 4: return launch_small_bwd_k<T, 4>(A, P, grid, threads, stream);
        case 5: return launch_small_bwd_k<T, 5>(A, P, grid, threads, stream);
        case 6: return launch_small_bwd_k<T, 6>(A, P, grid, threads, stream);
        default: return launch_small_bwd_k<T, 7>(A, P, grid, threads, stream);
    }
}

hipError_t launch_small_bwd(const void *x, const void *dy, const PlanView &pv, void *dx, float *dtheta, void *ws,
                            const Shape &s, hipStream_t stream)
{
    const SmallBwdGrid g = small_bwd_grid(s);
    SmallBwdArgs A{};
    A.x = x;
    A.dy = dy;
    A.dx = dx;
    A.partial = (float *)ws;
    A.fg_fwd = pv.fg_fwd;
    A.fd_fwd = pv.fd_fwd;
    A.fg_inv = pv.fg_inv;
    A.fd_inv = pv.fd_inv;
    A.fw_inv = pv.fw_inv;
    A.plan = pv.ref;
    A.rows = s.rows;
    A.ld_in = s.ld_x;
    A.ld_out = s.ld_y;
    A.heads = s.heads;
    A.width = s.n * s.heads;
    A.span = g.t.span;
    A.rows_per_block = g.t.rows_per_block;
    A.slices = g.t.slices;
    A.n_groups = g.n_groups;
    A.n_angles = (int64_t)s.heads * s.k * (s.n / 2);
    int plain_parts;
    const BwdArgs P = generic_bwd_args(x, dy, pv, dx, ws, s, &plain_parts);
    const bool inside = g.t.threads == kSbThreads && P.rows_per_tile * s.n <= kSbPlainTile;
    A.grid = (int)g.grid;
    const unsigned grid = inside && plain_parts > A.grid ? (unsigned)plain_parts : g.grid;
    if (inside) A.plain_parts = plain_parts;
    switch (s.dtype) {
        case BQ_F32: launch_small_bwd_t<float>(A, P, s.k, grid, g.t.threads, stream); break;
        case BQ_F16: launch_small_bwd_t<__half>(A, P, s.k, grid, g.t.threads, stream); break;
        default: launch_small_bwd_t<bf16_t>(A, P, s.k, grid, g.t.threads, stream); break;
    }
    if (!inside) {
        const hipError_t e = launch_generic_bwd_if_bad(x, dy, pv, dx, ws, s, stream, &plain_parts);
        if (e != hipSuccess) return e;
    }
    const unsigned blocks = (unsigned)((A.n_angles + kSbReduceAngles - 1) / kSbReduceAngles);
    hipLaunchKernelGGL(small_bwd_reduce_kernel, dim3(blocks), dim3(kSbReduceAngles * kSbReduceGroups), 0, stream, (const float *)ws,
                       dtheta, A.n_angles, g.slots, A.plan, (int64_t)plain_parts, A.fw_inv, s.k);
    return hipGetLastError();
}

}  // namespace bq

// Specialised kernels for n = 4096 (k = 12) and n = 8192 (k = 13): forward, inverse and fused forward +
// quantisation.  Included by one translation unit per width.
//
// One workgroup of 512 threads owns one transform at a time; thread t holds 8 elements.  All
// n*k scale-deferred coefficients (bq_internal.h) of the workgroup's head stay in registers (96 + 8
// per thread) while the workgroup loops over its rows, so a row costs one coalesced 16-byte load per
// thread, 12 FMAs per element, two LDS transposes and one store.
//
//   layout N ("natural"): thread (wave w, lane l) holds idx = 8*chunk + r, chunk = 64 w + e(l),
//                         r = 0..7.  Layers 1-3 pair registers, layers 4-7 pair lanes of a 16-lane
//                         row through DPP (bq_cascade.h).
//   layout P            : thread holds idx = baseP + b0 + 1024 r1 + 2048 r2 (register r' = b0 + 2 r1 +
//                         4 r2): idx bit 0 and idx bits 10, 11 are register bits, idx bits 7, 8, 9 are
//                         the chunk bits of lane bits 0..2 (DPP masks 1, 2, 7), idx bit 2 is lane
//                         bit 3, the remaining idx bits are lane bits 4, 5 and the wave index.
//                         Layers 8, 9, 10 use DPP, layers 11, 12 pair registers.
//   forward : A: load N, layers 1..7, write LDS1 | B: read P, layers 8..12, write LDS2 |
//             C: read N, output scale, quantise or store
//   inverse : A: load N, write LDS1 | B: read P, layers 12..8, write LDS2 | C: read N, layers 7..1,
//             output scale, store
//
// The three phases of consecutive rows are software-pipelined: iteration `it` of a workgroup runs
// C(row it-2), B(row it-1), A(row it) and then ONE barrier; three row buffers rotate through the roles,
// so every read of a buffer is separated from the next write to it by a barrier.  (Some variants use two
// buffers: A then overwrites what C has just read, each thread at the very addresses it read itself.)
//
// LDS accesses are 64-bit (two adjacent floats per lane), which is what reaches the full LDS rate.
// LDS float address of idx is idx + 2 (idx >> 5) + 2 (idx >> 9).  For a group of 16 lanes the N-side
// accesses vary idx bits 3..6 and the P-side accesses idx bits 2, 7, 8, 9; in both cases the four
// bits move the address by 2, 4, 8 and 16 words modulo 32, so the 16 lanes hit 16 different bank
// pairs (the padding terms supply what the plain index lacks).
//
// n = 8192 (kWide): layers 1..12 act inside each half of a row and only layer 13 couples element e with e + 4096.  A
// thread holds the same 8 positions of both halves (16 elements, up to 256 registers, one workgroup of 512 threads per
// compute unit) and runs the scheme above on both, each half in row buffers of its own; layer 13 pairs registers, forward in
// phase C (layout N), inverse at the start of phase B (layout P).  One workgroup of 1024 threads with a half each, which
// this replaces, had 128 registers for the same 120 values per thread: 4 to 20 of them were reloaded from scratch memory in
// every row (each reload waiting for everything in flight), layer 13 went through LDS and cost a second barrier.  32768 rows:
// bf16 forward 209 -> 198 us, inverse 259 -> 218, INT4 271 -> 219, fake-quantised INT4 with counts 617 -> 385; float32 forward
// 396 -> 381, inverse 400 -> 382, INT2 276 -> 238.
//
// If the plan flags the scale-deferred tables as unusable (a cosine too close to zero), the cascade
// of a row runs through LDS with plain (cos, sin) rotations instead; everything else is unchanged.
#pragma once

#include <type_traits>

#include "bq_cascade.h"

namespace bq {

constexpr int kN = 4096, kK = 12, kThreads = 512;
constexpr int kLdsRow = 4368;  // floats: 4095 + 2*127 + 2*7 + 1, rounded up to a multiple of 4
// Dynamic LDS of a workgroup, n <= 4096: the input ring (three slots of 8 KB or, two-buffer variants, two slots of a row) and
// behind it as many row buffers; the two-buffer variants keep per-thread constants in the rest ("parked": float4 q of
// thread t at park[512 q + t]).  Two workgroups fit on a compute unit.  The kernel asserts that its variant fits.
constexpr size_t kParkQuadBytes = 16 * kThreads;
constexpr size_t kLdsBytes = (3 * kN * 2 / 4 + 3 * kLdsRow) * sizeof(float);
// n = 8192: one workgroup; largest with 32-bit rows, two slots and two buffers per half and three quads
constexpr size_t kLdsBytesWide = 2 * (2 * kN + 2 * kLdsRow) * sizeof(float) + 3 * kParkQuadBytes;
static_assert(kLdsBytes + 512 <= 80 * 1024 && kLdsBytesWide + 512 <= 160 * 1024, "LDS of a compute unit");

struct K12Args {
    const void *in;
    void *out;
    const float *fg;   // [heads][k][n] coefficients of the direction
    const float *fd;   // [heads][n] output scales
    const float2 *cs;  // [heads][k][n/2]
    PlanRef plan;  // not read by the fixed transform (its coefficients come from the element index)
    int64_t rows, ld_in, ld_out;
    int heads;
    // The gridDim.x / heads workgroups of a head take its rows in turn: each has rows_each of them (< 2^31), the first
    // rows_extra one more.  Divided on the host: a 64-bit division takes the kernel a hundred instructions.
    int rows_each, rows_extra;
    // quantiser
    uint8_t *codes;
    void *scales;
    unsigned long long *hist;  // kFwdFake: 2^bits counters or NULL
    int group, scale_f16;
    // the batch is larger than the memory-side cache (input and output are touched once): the launcher then picks
    // the kNt variants of the plain transforms
    int streaming;
    // transforms of n = 2^n_log < 4096 points (kVirt): a "row" of the kernel is a block of 4096 consecutive
    // elements of the caller's [rows][heads * n] array.  Rows of up to 4096 elements: 2^(12 - row_log) whole rows
    // (row_log = log2 of the row width; ld_in / ld_out are the strides between blocks, sub_ld_* the caller's
    // strides, heads = 1).  Wider rows: block `head` of the heads = width / 4096 blocks of a row (row_log = 12).
    // tail_rows != 0: the last of the `rows` blocks has only so many of the caller's rows.  Its missing rows are read as
    // copies of its first one and not stored; the rows it has are rotated like those of whole blocks, so that a row's result does
    // not depend on how many rows come with it (in the kernel for any n, which they went through before, plain rotations rounded
    // them: a few codes in 10^6 of theirs differ from those).  (kTail variants; large batches take them for the last block alone,
    // short_block_apart().  The rows of a short block went through the kernel for any n, a launch of 10 to
    // 95 us behind this one: 2001 rows of 2048, float32 inverse 34 -> 11 us, fp16 INT4 36 -> 14 us, one scale per row
    // 112 -> 15 us.)
    int n, n_log, row_log, tail_rows;
    int64_t sub_ld_in, sub_ld_out;
};

// Element offset, inside a kernel row, of the element with index e (a multiple of 8) of the 4096-point block.
template <bool kVirt, bool kWide = false>
__device__ __forceinline__ uint32_t elem_off(const K12Args &A, int head, int e, int64_t sub_ld)
{
    if (!kVirt) return (uint32_t)(head * (kWide ? 2 * kN : kN) + e);
    return (uint32_t)((e >> A.row_log) * (int)sub_ld + head * kN + (e & ((1 << A.row_log) - 1)));
}
// kVirt: element e of the short last block lies in a row that the block does not have
__device__ __forceinline__ bool in_tail_gap(const K12Args &A, int e) { return (e >> A.row_log) >= A.tail_rows; }
// Byte offset, inside a kernel row, of the 16 bytes at element e: `off` (elem_off of e) except in the short block
// (a uniform branch, so that the offsets of the short block occupy no registers in the row loop).
template <bool kTail, typename T>
__device__ __forceinline__ uint32_t tail_off(const K12Args &A, uint32_t off, int e, bool short_block)
{
    if (kTail && short_block) {
        asm volatile("" : "+v"(e));
        if (in_tail_gap(A, e)) off = (uint32_t)(e & ((1 << A.row_log) - 1)) * (uint32_t)sizeof(T);
    }
    return off;
}
// kVirt: the transform (head of the caller's row) that element e of block `head` belongs to
__device__ __forceinline__ int virt_head(const K12Args &A, int head, int e)
{
    return (head * kN + (e & ((1 << A.row_log) - 1))) >> A.n_log;
}

__device__ __forceinline__ int lds_addr(int idx) { return idx + 2 * (idx >> 5) + 2 * (idx >> 9); }
constexpr int kPStepR1 = 1024 + 2 * 32 + 2 * 2;  // address step of register bit r1 (idx + 1024)
constexpr int kPStepR2 = 2 * kPStepR1;           // register bit r2 (idx + 2048)

// thread's base index in layout P
__device__ __forceinline__ int base_p(int wave, int lane)
{
    const int c3 = lane_chunk(lane & 15) & 7;
    return (c3 << 7) | (((lane >> 3) & 1) << 2) | (((lane >> 4) & 1) << 1) | (((lane >> 5) & 1) << 3) | (wave << 4);
}
__device__ __forceinline__ int p_reg_idx(int r) { return (r & 1) + 1024 * ((r >> 1) & 1) + 2048 * (r >> 2); }

__device__ __forceinline__ void lds_write_n(float *buf, int an, const float (&u)[8])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) *(float2 *)&buf[an + 2 * j] = make_float2(u[2 * j], u[2 * j + 1]);
}
__device__ __forceinline__ void lds_read_n(const float *buf, int an, float (&u)[8])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float2 v = *(const float2 *)&buf[an + 2 * j];
        u[2 * j] = v.x;
        u[2 * j + 1] = v.y;
    }
}
__device__ __forceinline__ void lds_write_p(float *buf, int ap, const float (&u)[8])
{
#pragma unroll
    for (int j = 0; j < 4; ++j)
        *(float2 *)&buf[ap + (j & 1) * kPStepR1 + (j >> 1) * kPStepR2] = make_float2(u[2 * j], u[2 * j + 1]);
}
__device__ __forceinline__ void lds_read_p(const float *buf, int ap, float (&u)[8])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float2 v = *(const float2 *)&buf[ap + (j & 1) * kPStepR1 + (j >> 1) * kPStepR2];
        u[2 * j] = v.x;
        u[2 * j + 1] = v.y;
    }
}

// Rows of a plan table in layout P.  They are read from memory in 16-byte pieces and turned around in LDS: read straight from
// memory in layout P, neighbouring lanes are 512 bytes apart and every lane becomes an access of its own, 20 eight-byte loads for
// the five rows (one fp16 row of 4096, INT4: 8.3 us).
//
// A wave's elements in layout P are the runs of 16 with idx bits 4..6 = wave, 32 of them 128 apart.  The wave loads its runs
// with two loads per lane and row and turns them around in a piece of LDS of its own; a wave's LDS instructions complete in
// order, so there is no barrier and no wait but those for the data.  One row, back to back inside a graph, against two barriers
// per two rows through the whole workgroup's row buffers (turn_together): fp16 INT4 n = 4096 4.96 -> 4.68 us, inverse 4.81 -> 4.62,
// float32 4.74 -> 4.44, n = 8192 forward 7.79 -> 7.45, inverse 7.73 -> 7.12.  Of these 1.7 us are the launch and 0.8 (n = 8192:
// 2.1) the tables.
constexpr int kPieceFloats = 512;  // a wave's part of a table row
// first of the four elements that a lane loads, part 0 or 1
__device__ __forceinline__ int piece_idx(int wave, int lane, int part) { return ((lane >> 2) + 16 * part) * 128 + wave * 16 + (lane & 3) * 4; }
// place of element o of run `run`; every other pair of runs has its two halves swapped, so that the runs that lane bits 0..2 walk
// over in layout P lie in different banks
__device__ __forceinline__ int piece_addr(int run, int o) { return run * 16 + (o ^ ((run & 2) << 2)); }
// kRows rows: v[j][part] -> c[j], through `own`, kRows * kPieceFloats floats of LDS that only this wave uses
template <int kRows>
__device__ __forceinline__ void turn_own(float *own, int lane, int idx_p, const float4 (*v)[2], float (*c)[8])
{
    const int at = piece_addr(lane >> 2, (lane & 3) * 4), from = piece_addr(idx_p >> 7, idx_p & 15);
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        *(float4 *)&own[j * kPieceFloats + at] = v[j][0];
        *(float4 *)&own[j * kPieceFloats + at + 256] = v[j][1];  // 16 runs further on
    }
    asm volatile("" ::: "memory");  // (other lanes' pieces: the compiler must not move the reads up)
#pragma unroll
    for (int j = 0; j < kRows; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // idx bits 10 and 11: 8 and 16 runs
            const float2 w = *(const float2 *)&own[j * kPieceFloats + from + (q & 1) * 128 + (q >> 1) * 256];
            c[j][2 * q] = w.x;
            c[j][2 * q + 1] = w.y;
        }
    asm volatile("" ::: "memory");
}
// The same through two row buffers of the workgroup, from the thread's 8 consecutive entries (its own place in layout N).
// Every thread of the workgroup must call it.
__device__ __forceinline__ void turn_together(float *b0, float *b1, int an, int ap, const float (&s0)[8], const float (&s1)[8],
                                              float (&c0)[8], float (&c1)[8])
{
    lds_write_n(b0, an, s0);
    lds_write_n(b1, an, s1);
    __syncthreads();
    lds_read_p(b0, ap, c0);
    lds_read_p(b1, ap, c1);
    __syncthreads();
}

// Layer 13 of an 8192-point transform on the two halves of a thread's elements.  kFirst: it opens the cascade, every scale
// is still 1 and the lower element's coefficient is minus the upper one's.
template <bool kFirst>
__device__ __forceinline__ void half_layer(float (&u)[2][8], const float (&lo)[8], const float (&up)[8])
{
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const float ua = u[0][r], ub = u[1][r];
        u[0][r] = __builtin_fmaf(kFirst ? -up[r] : lo[r], ub, ua);
        u[1][r] = __builtin_fmaf(up[r], ua, ub);
    }
}

// slow cascade through LDS with (cos, sin); in: u[] in layout N, out: y[] in layout N (true values)
// n_log < 12: the block holds 4096 >> n_log independent transforms of 2^n_log points (same angles).
// kHalves = 2: one 8192-point transform, u[h] the thread's elements of half h.
// row_mask, head0: several transforms with their own angles side by side in the block (see K12Args): element a
// belongs to transform (head0 + (a & row_mask)) >> n_log.
template <bool kInverse, int kHalves>
__device__ __forceinline__ void slow_cascade(float (&u)[kHalves][8], float *buf, const float2 *__restrict__ cs, int idx_n,
                                             int n_log, int row_mask = 0, int head0 = 0)
{
    constexpr int kPoints = kHalves * kN;
    // n = 8192: the loads of four pairs in front of the first store.  Pair by pair a flagged plan's call took 40 % longer than
    // with the 1024 threads this width had before (one row 17.2 us, 512 rows 34.8), this way 12.9 and 26.0.  All eight pairs
    // at once 13.8 and 27.1; at n <= 4096 two pairs already cost 38 spilled registers.
    constexpr int kBatch = kHalves == 2 ? 4 : 1;
    __syncthreads();
#pragma unroll
    for (int h = 0; h < kHalves; ++h)
#pragma unroll
        for (int r = 0; r < 8; ++r) buf[h * kN + idx_n + r] = u[h][r];
    __syncthreads();
    const int half_n = 1 << (n_log - 1);
    for (int step = 0; step < n_log; ++step) {
        const int i = kInverse ? (n_log - step) : (step + 1);
        const int h = 1 << (i - 1);
        for (int p0 = threadIdx.x; p0 < kPoints / 2; p0 += kBatch * kThreads) {
            float2 w[kBatch];
            float xa[kBatch], xb[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int p = p0 + j * kThreads;
                const int a = ((p >> (i - 1)) << i) | (p & (h - 1));
                const int hd = (head0 + (a & row_mask)) >> n_log;
                w[j] = cs[((size_t)hd * n_log + (i - 1)) * half_n + (p & (half_n - 1))];
                xa[j] = buf[a];
                xb[j] = buf[a + h];
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int p = p0 + j * kThreads;
                const int a = ((p >> (i - 1)) << i) | (p & (h - 1));
                if (!kInverse) {
                    buf[a] = __builtin_fmaf(w[j].x, xa[j], -(w[j].y * xb[j]));
                    buf[a + h] = __builtin_fmaf(w[j].y, xa[j], w[j].x * xb[j]);
                } else {
                    buf[a] = __builtin_fmaf(w[j].x, xa[j], w[j].y * xb[j]);
                    buf[a + h] = __builtin_fmaf(w[j].x, xb[j], -(w[j].y * xa[j]));
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int h = 0; h < kHalves; ++h)
#pragma unroll
        for (int r = 0; r < 8; ++r) u[h][r] = buf[h * kN + idx_n + r];
    __syncthreads();
}

// max |y| over a group of 256 .. 8192 consecutive channels (up to the whole row): 16-lane rows by DPP, the
// wave by two lane shuffles, several waves through `wg_max` (one float per wave) and one workgroup barrier.
// Every thread of the workgroup must call it; successive calls must be separated by a barrier of their own
// (the row loop's is).
template <int kHalves>
__device__ __forceinline__ void big_group_max(const float (&y)[kHalves][8], int group, int wave, float *wg_max, float (&m)[kHalves])
{
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
        m[h] = row16_max(amax8(y[h]));
        m[h] = fmaxf(m[h], __shfl_xor(m[h], 16));
        if (group >= 512) m[h] = fmaxf(m[h], __shfl_xor(m[h], 32));
    }
    if (group > 512) {
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int h = 0; h < kHalves; ++h) wg_max[h * 8 + wave] = m[h];
        __syncthreads();
        const int waves = group >> 9;
#pragma unroll
        for (int h = 0; h < kHalves; ++h) {
            const int first = (h * 8 + wave) & ~(waves - 1);
            float g = wg_max[first];
            for (int w = 1; w < waves; ++w) g = fmaxf(g, wg_max[first + w]);
            m[h] = g;
        }
    }
}

// Epilogue shared by the fast and the slow loop: y[] holds the rotated values in layout N.
// kLanes > 0 fixes the group size (8 * kLanes) and kScale fixes the scale type (0 = float32,
// 1 = binary16) at compile time; kLanes == 0 reads both from the arguments.
// Addresses are a uniform row base plus a 32-bit per-thread offset.
constexpr int kScaleF16 = 2, kScaleF32 = 3;
template <int kLanes, int kScale>
__device__ __forceinline__ bool scale_is_f16(const K12Args &A)
{
    return kLanes > 0 ? kScale != 0 : kScale == kScaleF16 || (kScale != kScaleF32 && A.scale_f16 != 0);
}
struct NoCount {};
template <int kMode, int kBits>
struct CountOf {
    typedef NoCount type;
};
template <int kBits>
struct CountOf<kFwdFake, kBits> {
    typedef BinCount<kBits> type;
};

// kFwdFake only: kYq = the dequantised row is stored, kHist = the bins are counted.
// y[h]: half h of the row (n = 8192), else the row; chunk: the thread's group of 8 elements inside its half.
// kBig: quantiser groups of more than 128 channels (the maximum then comes from big_group_max()).
// live (kVirt): the thread's row exists; else nothing is stored or counted.
template <typename T, int kMode, int kBits, int kLanes, int kScale, bool kYq, bool kHist, bool kVirt, int kHalves, bool kBig,
          bool kNt = false>
__device__ __forceinline__ void finish_row(const K12Args &A, const float (&y)[kHalves][8], int64_t row, int head, int chunk,
                                           typename CountOf<kMode, kBits>::type &bins, unsigned long long *wg_bins,
                                           float *wg_max, bool live = true)
{
    constexpr bool kWide = kHalves == 2;
    float group_max[kHalves] = {};
    if (kBig) big_group_max<kHalves>(y, A.group, chunk >> 6, wg_max, group_max);
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
        const int chunk_row = h * (kN / 8) + chunk;
        if (kMode == kFwdFake) {
            const int lanes = A.group >> 3;  // lanes per group
            float f[8], s;
            bool ordinary;
            // (rows with float32 scales apart: three registers spilled with the short quotient and reciprocal, none with the divisions)
            rounded8<kBits, kBig, kScale == kScaleF32>(y[h], lanes, scale_is_f16<kLanes, kScale>(A), f, &s, &ordinary, group_max[h]);
            if (kHist) {
                auto &bc = (BinCount<kBits> &)bins;
                if (!kVirt || live)
                    count8<kBits>(bc, f, ordinary);
                else
                    bc.skip();
                if (bc.full()) bc.drain(wg_bins);
            }
            if (kYq && (!kVirt || live)) {
                float yq[8];
                dequant8(f, s, yq);
                T *out_row = (T *)A.out + row * A.ld_out + h * kN;
                uint32_t off = elem_off<kVirt, kWide>(A, head, chunk * 8, A.sub_ld_out) * (uint32_t)sizeof(T);
                asm volatile("" : "+v"(off));
                store8((T *)((char *)out_row + off), yq);
            }
        } else if (kMode != kFwdQuant) {
            if (kVirt && !live) continue;
            T *out_row = (T *)A.out + row * A.ld_out + h * kN;
            uint32_t off = elem_off<kVirt, kWide>(A, head, chunk * 8, A.sub_ld_out) * (uint32_t)sizeof(T);
            asm volatile("" : "+v"(off));
            if (kNt)
                store8_nt((T *)((char *)out_row + off), y[h]);
            else
                store8((T *)((char *)out_row + off), y[h]);
        } else {
            const int lanes = kLanes > 0 ? kLanes : (A.group >> 3);  // lanes per group
            const bool f16 = scale_is_f16<kLanes, kScale>(A);
            float s;
            const uint32_t packed = quant8<kBits, kBig>(y[h], lanes, f16, &s, group_max[h]);
            if (kVirt && !live) continue;
            const int64_t unit = row * A.heads + head;
            uint8_t *codes_row = A.codes + unit * (kHalves * kN * kBits / 8) + h * (kN * kBits / 8);
            uint32_t coff = (uint32_t)(chunk * kBits);
            asm volatile("" : "+v"(coff));
            if (kBits == 2)
                *(uint16_t *)(codes_row + coff) = (uint16_t)packed;
            else
                *(uint32_t *)(codes_row + coff) = packed;
            // every lane of a group stores the group's scale (same value, same address): no divergence
            const int groups = (kHalves * kN / 8) / lanes;
            uint32_t goff = ((uint32_t)chunk_row / (uint32_t)lanes) * (f16 ? 2u : 4u);
            asm volatile("" : "+v"(goff));
            if (f16)
                *(__half *)((char *)((__half *)A.scales + unit * groups) + goff) = __float2half_rn(s);
            else
                *(float *)((char *)((float *)A.scales + unit * groups) + goff) = s;
        }
    }
}

template <typename T, int kMode, int kBits, int kLanes, int kScale, bool kYq = true, bool kHist = false, bool kVirt = false,
          bool kWide = false, bool kBig = false, bool kNt = false, bool kTail = false>
__global__ __launch_bounds__(kThreads, kWide ? 2 : 4) void k12_kernel(K12Args A)
{
    static_assert(!kTail || kVirt, "short blocks of several rows");
    static_assert(!(kWide && kVirt), "blocks of small transforms are a 4096-point scheme");
    // kNt: rows are loaded and stored with the non-temporal hint.  262144 fp16 rows of n = 4096: forward 0.796 ->
    // 0.778 ms on every box tried.  Not used where it did not hold up: the inverse gained 3.5 % on some boxes and
    // lost as much on others, float32 rows lost 15 - 19 % (0.78 -> 0.93 ms), the fused quantiser stores too little.
    static_assert(!kNt || ((kMode == kFwd || kMode == kHadamard) && sizeof(T) == 2), "16-bit forward transforms only");
    // (the two-phase inverse of 16-bit rows, bq_k12_inv.h, has a variant of its own that does gain)
    static_assert(!kBig || ((kMode == kFwdQuant || kMode == kFwdFake) && kLanes == 0), "large groups: general quantiser variants");
    constexpr int kHalves = kWide ? 2 : 1;
    constexpr int kPoints = kHalves * kN;  // n
    constexpr int kLayers = kWide ? kK + 1 : kK;
    __shared__ unsigned long long wg_bins[16];  // kFwdFake: this workgroup's bin counts
    __shared__ float wg_max[16];                // quantiser groups that span several waves: one maximum per wave
    typename CountOf<kMode, kBits>::type bins;
    if (kMode == kFwdFake && kHist) {
        ((BinCount<kBits> &)bins).clear();
        if (threadIdx.x < 16) wg_bins[threadIdx.x] = 0;
        __syncthreads();
    }
    // kFwdFake: per-thread counts -> workgroup counts -> the caller's counters (every thread gets here).  kTight: what ends the
    // kernel decides how many registers the row loop spills (float32 rows, INT2: 10 with both outputs, 22 with 64-bit sums of the
    // wave; 6 with counts only and lanes adding for themselves, 13 with sums of the wave).  INT2, groups of 256, 64-bit sums of the
    // wave / as it is: 40001 rows of 4096, float32 both 420 / 298 us, float32 counts 248 / 171, fp16 both 296 / 226; 700 rows 19.5 /
    // 16.7, 16.6 / 13.5, 17.9 / 15.5.
    constexpr bool kTight = kBig && !kVirt && !kWide;
    constexpr int kSpread = kTight && !kYq && sizeof(T) == 4 && kBits == 2 ? 3 : 0;  // lane by lane: four words per bin, less one
    auto flush_bins = [&]() {
        if (kMode == kFwdFake && kHist) {
            auto &bc = (BinCount<kBits> &)bins;
            if constexpr (!kTight)
                bc.template drain_wave<long long>(wg_bins);
            else if constexpr (kYq || sizeof(T) == 2)
                bc.template drain_wave<int>(wg_bins);
            else
                bc.drain(wg_bins + 4 * (threadIdx.x & kSpread));
            __syncthreads();
            if (threadIdx.x < (1 << kBits)) {
                unsigned long long count = wg_bins[threadIdx.x];
#pragma unroll
                for (int c = 1; c <= kSpread; ++c) count += wg_bins[threadIdx.x + 4 * c];
                if (count) atomicAdd(&A.hist[threadIdx.x], count);
            }
        }
    };
    constexpr bool kRing32 = sizeof(T) == 4;
    // kTwoBuf: two row buffers and two ring slots instead of three.  Phase A of row `it` writes the buffer that
    // phase C of row it-2 has just read (there each thread reads and writes the same addresses, and C comes
    // first), and the load of row it+2 refills the slot that A has just read.  What is saved holds per-thread constants
    // (kPark*, below).  Used
    //  - for 32-bit rows (slots twice as large: three of them plus three buffers would not leave room for two
    //    workgroups per compute unit; before, such rows were prefetched in registers, at the price of a dozen
    //    spilled ones: 131072 rows of n = 4096 went from 1.20 / 0.92 / 0.84 ms to 0.81 / 0.80 / 0.53 ms);
    //  - for n = 8192, which needs the registers;
    //  - for the fake-quantising variants that count bins, where they are short as well: INT4 with both outputs (65536 fp16
    //    rows of n = 4096: 1.14 -> 1.00 ms for four times as many), INT2 that only counts (0.82 -> 0.77 ms), and blocks of
    //    smaller transforms (65536 fp16 rows of n = 1024: INT2 109 -> 84 us, INT4 100 -> 75).  On the other 16-bit variants
    //    of n <= 4096 it measured equal or slower.
    constexpr bool kTwoBuf = kRing32 || kWide || (kMode == kFwdFake && kHist && (kVirt || (kYq && kBits == 4) || (!kYq && kBits == 2)));
    // What the two-buffer variants park in the LDS that is left, in quads of four floats per thread: output scales (all of
    // them for 16-bit rows; for 32-bit rows, in the modes that are short of registers, what fits) and, where the bins are
    // counted, the first layer's four coefficients per half.
    constexpr bool kShort = kMode == kFwdQuant || kMode == kFwdFake;
    constexpr int kParkScales = !kTwoBuf ? 0 : !kRing32 ? 2 * kHalves : !kShort ? 0 : kWide ? 3 : 1;
    constexpr bool kParkFirst = kTwoBuf && !kRing32 && kMode == kFwdFake;
    // LDS: the input ring first (low addresses), then the row buffers, then what is parked
    constexpr int kSlots = kTwoBuf ? 2 : 3;
    constexpr int kRingFloats = kSlots * kPoints * (int)sizeof(T) / 4;
    static_assert((kRingFloats + kSlots * kHalves * kLdsRow) * sizeof(float) + (kParkScales + (kParkFirst ? kHalves : 0)) * kParkQuadBytes <=
                      (kWide ? kLdsBytesWide : kLdsBytes), "dynamic LDS of the launch");
    // How the tables get into layout P.  The variants that are shortest of registers come out of the compiler with more spilled
    // ones in the row loop where the waves turn their own pieces (40001 float32 rows of 2048, fake-quantised INT4 with counts, 173
    // -> 220 us; 32768 bf16 rows of 8192, INT4 with one group per row, 344 -> 355): they keep the turn through the row buffers.
    constexpr bool kTurnOwn = kMode != kFwdFake && !(kWide && kBig);
    // a wave's share of the row buffers, before they hold rows
    constexpr int kOwnFloats = kSlots * kHalves * kLdsRow / 8 & ~3, kOwnRows = kOwnFloats / kPieceFloats;
    static_assert(kOwnRows >= 2, "five rows in three turns");
    extern __shared__ float lds_raw[];
    float *lds = lds_raw + kRingFloats;
    constexpr bool kInverse = (kMode == kInv);
    // kHadamard: the same cascade with every coefficient +1 (lower element of a pair) or -1 (upper element), i.e.
    // additions and subtractions; nothing is read from a plan.  A layer then maps (a, b) to (a + b, b - a), which
    // is the Sylvester butterfly (a + b, a - b) up to the sign of its second output; over all layers the signs
    // collect to (-1)^popcount(index) per output element, which the single scale 1 / sqrt(n) takes along.
    constexpr bool kHad = (kMode == kHadamard);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;  // kWide: chunk and idx_n count inside a half
    const int chunk = wave * 64 + lane_chunk(lane);
    const int idx_n = chunk * 8;
    const int head = blockIdx.x % A.heads;
    const int64_t row_first = blockIdx.x / A.heads;
    const int64_t row_step = gridDim.x / A.heads;
    const uint32_t off_n = elem_off<kVirt, kWide>(A, head, idx_n, A.sub_ld_in);  // element offset of the thread inside a row
    // tables: rows of n entries, indexed inside the transform the element belongs to
    const int tn = kVirt ? A.n : kPoints;
    const int nk = kVirt ? A.n_log : kLayers;
    const int tmask = tn - 1;
    const T *in = (const T *)A.in;
    if (row_first >= A.rows) return;
    PlanHead ph = {true, 0, 0};
    if (!kHad) ph = plan_head(A.plan);
    if (!ph.matches) return;

    if ((kInverse ? ph.bad_inv : ph.bad_fwd) != 0) {  // rare: plain rotations through LDS
        const float2 *cs = A.cs + (kVirt ? 0 : (size_t)head * kLayers * (kPoints / 2));
        for (int64_t row = row_first; row < A.rows; row += row_step) {
            float u[kHalves][8];
            const bool short_block = kTail && row == A.rows - 1;
            const uint32_t off = kTail ? tail_off<kTail, T>(A, off_n * (uint32_t)sizeof(T), idx_n, short_block) / (uint32_t)sizeof(T) : off_n;
#pragma unroll
            for (int h = 0; h < kHalves; ++h) unpack8(load8(in + row * A.ld_in + off + h * kN), u[h], (const T *)nullptr);
            slow_cascade<kInverse, kHalves>(u, lds, cs, idx_n, nk, kVirt ? (1 << A.row_log) - 1 : 0, kVirt ? head * kN : 0);
            finish_row<T, kMode, kBits, kLanes, kScale, kYq, kHist, kVirt, kHalves, kBig, kNt>(A, u, row, head, chunk, bins, wg_bins, wg_max,
                                                                                                       !(short_block && in_tail_gap(A, idx_n)));
        }
        flush_bins();
        return;
    }
    // coefficients: cn[h][j][r] for layer j+1 (layout N), cp[h][j][r'] for layer 8+j (layout P), d[h][r] (layout N)
    const int idx_p = base_p(wave, lane);
    const int an = lds_addr(idx_n);
    const int ap = lds_addr(idx_p);
    float cn[kHalves][7][8], cp[kHalves][5][8];
    float cw[2][8];  // kWide: layer 13, in layout N (forward, phase C) or layout P (inverse, phase B; the upper half's only)
    if (kHad) {
#pragma unroll
        for (int h = 0; h < kHalves; ++h)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
#pragma unroll
                for (int j = 0; j < 7; ++j) cn[h][j][r] = (((idx_n + r) >> j) & 1) ? -1.0f : 1.0f;
#pragma unroll
                for (int j = 0; j < 5; ++j) cp[h][j][r] = (((idx_p + p_reg_idx(r)) >> (7 + j)) & 1) ? -1.0f : 1.0f;
                cw[h][r] = h ? -1.0f : 1.0f;
            }
    } else {
        // tables are [head][layer][n]; kVirt: the head is the element's own (virt_head)
        auto table = [&](int e) {
            return A.fg + (kVirt ? (size_t)virt_head(A, head, e) * nk * tn : (size_t)head * kLayers * kPoints) + (e & tmask);
        };
        const float *fg0 = table(idx_n);
        auto load_n = [&](int h) {  // layers 1..7 and, where it is applied in layout N, layer 13
#pragma unroll
            for (int j = 0; j < 7; ++j) load_coef8(fg0 + h * kN + (size_t)j * tn, cn[h][j]);
            if (kWide && !kInverse) load_coef8(fg0 + h * kN + (size_t)kK * tn, cw[h]);
        };
        if constexpr (kTurnOwn) {
            const float *pp[2] = {table(piece_idx(wave, lane, 0)), table(piece_idx(wave, lane, 1))};
            float *own = lds + wave * kOwnFloats;
#pragma unroll
            for (int h = 0; h < kHalves; ++h) {
                // layers 8..12 and, where it is applied in layout P, layer 13 (the upper half's coefficients)
                constexpr int kRowsP = kWide && kInverse ? 6 : 5;
                float4 st[kRowsP][2];
#pragma unroll
                for (int j = 0; j < kRowsP; ++j)  // layers above log2 n do not exist: weight zero leaves the element as it is
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        st[j][q] = j < 5 + h && (!kVirt || 8 + j <= nk) ? *(const float4 *)(pp[q] + (size_t)(7 + j) * tn + h * kN)
                                                                        : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                load_n(h);
                // as many rows at a time as the wave's piece holds
                constexpr int kFirst = kOwnRows < 5 ? kOwnRows : 5, kSecond = 5 - kFirst < kFirst ? 5 - kFirst : kFirst;
                turn_own<kFirst>(own, lane, idx_p, st, cp[h]);
                turn_own<kSecond>(own, lane, idx_p, st + kFirst, cp[h] + kFirst);
                turn_own<5 - kFirst - kSecond>(own, lane, idx_p, st + kFirst + kSecond, cp[h] + kFirst + kSecond);
                if constexpr (kWide && kInverse)
                    if (h == 1) turn_own<1>(own, lane, idx_p, st + 5, cw + 1);
            }
            __syncthreads();  // the pieces are row buffers from here on
            // The empty statements keep the compiler from dropping the lower elements' coefficients of layer 1, which the forward
            // cascade does without: it would read the others with four strided 4-byte loads instead of two of 16 bytes (one fp16
            // row of 4096, INT4: 4.81 -> 4.50 us, 37 rows of 8192 8.13 -> 7.47, 1777 rows 11.6 -> 11.2).
#pragma unroll
            for (int h = 0; h < kHalves; ++h)
#pragma unroll
                for (int r = 0; r < 8; r += 2) asm volatile("" ::"v"(cn[h][0][r]));
        } else {
            static_assert(!(kWide && kInverse), "layer 13 in layout P");
#pragma unroll
            for (int h = 0; h < kHalves; ++h) {
                float st[5][8], unused[8];
#pragma unroll
                for (int j = 0; j < 5; ++j) {
#pragma unroll
                    for (int r = 0; r < 8; ++r) st[j][r] = 0.0f;
                    if (!kVirt || 8 + j <= nk) load_coef8(fg0 + h * kN + (size_t)(7 + j) * tn, st[j]);
                }
                load_n(h);
                float *b0 = lds + h * kLdsRow, *b1 = lds + (kHalves + h) * kLdsRow;
                turn_together(b0, b1, an, ap, st[0], st[1], cp[h][0], cp[h][1]);
                turn_together(b0, b1, an, ap, st[2], st[3], cp[h][2], cp[h][3]);
                turn_together(b0, b1, an, ap, st[4], st[4], cp[h][4], unused);
            }
        }
    }

    // rows of this workgroup: below 2^28 for every batch the library accepts, so the loop counters are 32-bit
    // (64-bit comparisons of uniform values would be done on the vector unit)
    // (The fake quantisers divide here: with the host's figures the compiler keeps other values in registers and the float32
    // variants spill in the row loop, 40000 rows of 2048 with one group per row 193 -> 273 us.)
    const int n_my = kMode == kFwdFake ? (int)((A.rows - row_first + row_step - 1) / row_step)
                                       : A.rows_each + ((int)row_first < A.rows_extra ? 1 : 0);
    // the short last block, if it is this workgroup's, is the last of its rows
    const int tail_j = kTail && row_first + (n_my - 1) * row_step == A.rows - 1 ? n_my - 1 : -1;

    // Phase B of one row: layers 8..12 (or 12..8) on layout P, in place in its LDS buffer (one per half).
    auto phase_b = [&](float *lb) {
        float u[kHalves][8];
#pragma unroll
        for (int h = 0; h < kHalves; ++h) lds_read_p(lb + h * kLdsRow, ap, u[h]);
        if constexpr (kWide && kInverse) half_layer<true>(u, cw[0], cw[1]);
#pragma unroll
        for (int h = 0; h < kHalves; ++h) {
            if (!kInverse) {
                dpp_layer_xor1(u[h], cp[h][0]);
                dpp_layer_xor2(u[h], cp[h][1]);
                dpp_layer_xor7(u[h], cp[h][2]);
                reg_layer<1>(u[h], cp[h][3]);
                reg_layer<2>(u[h], cp[h][4]);
            } else {
                if (kWide)
                    reg_layer<2>(u[h], cp[h][4]);
                else
                    reg_layer_first<2>(u[h], cp[h][4]);
                reg_layer<1>(u[h], cp[h][3]);
                dpp_layer_xor7(u[h], cp[h][2]);
                dpp_layer_xor2(u[h], cp[h][1]);
                dpp_layer_xor1(u[h], cp[h][0]);
            }
            lds_write_p(lb + h * kLdsRow, ap, u[h]);
        }
    };
    // Layers of phase A after the first one / layers of phase C before the output scale.
    auto layers_a = [&](float (&u)[8], const float (&c)[7][8]) {
        if (!kInverse) {
            reg_layer<1>(u, c[1]);
            reg_layer<2>(u, c[2]);
            dpp_layer_xor1(u, c[3]);
            dpp_layer_xor2(u, c[4]);
            dpp_layer_xor7(u, c[5]);
            dpp_layer_xor8(u, c[6]);
        }
    };
    auto layers_c = [&](float (&u)[8], const float (&c)[7][8]) {
        if (kInverse) {
            dpp_layer_xor8(u, c[6]);
            dpp_layer_xor7(u, c[5]);
            dpp_layer_xor2(u, c[4]);
            dpp_layer_xor1(u, c[3]);
            reg_layer<2>(u, c[2]);
            reg_layer<1>(u, c[1]);
            reg_layer<0>(u, c[0]);
        }
    };
    // ---- input staged through an LDS ring filled by direct global->LDS loads -------------------
    // Two rows per workgroup have to be in flight from HBM to cover its latency, and there are
    // no registers left to hold them.  global_load_lds_dwordx4 moves 16 bytes per lane straight
    // into LDS (16-bit rows: wave w, lane l -> bytes [1024 w + 16 l, +16) of the ring slot, row order), the
    // thread later reads its own chunk back with ds_read_b128.  A wave only reads what it loaded
    // itself, so s_waitcnt vmcnt is the only synchronisation.  These loads and waits are inline
    // assembly: the compiler would otherwise wait for ALL outstanding loads before any LDS read.
    // Memory operations of a wave complete in issue order, and per iteration a wave issues one
    // ring load (in A) and at least kStores stores (in C); row `it` was requested two iterations
    // earlier, followed by stores, the load of row it+1 and stores again, so at most
    // 2 kStores + 1 younger operations may still be pending when row `it` is consumed.  The
    // first four iterations (pipeline fill, fewer stores issued) wait for everything.
    // 32-bit rows: two such loads per lane and row (kHalfLoads), two stores per lane for a row of output; n = 8192: as many
    // for each half.
    constexpr int kHalfLoads = (int)sizeof(T) / 2, kLoads = kHalves * kHalfLoads;
    constexpr int kStores = (kMode == kFwdQuant) ? 2 * kHalves : (kMode == kFwdFake && !kYq) ? 0 : kLoads;
    constexpr int kPending = 2 * kStores + kLoads;  // operations younger than the last load of the awaited row
    constexpr uint32_t kSlotBytes = kPoints * sizeof(T);
    float d[kHalves][8];
    float4 *park = (float4 *)(lds + 2 * kHalves * kLdsRow) + tid;  // quad q: park[q * kThreads], read back by the same thread only
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
        if (kHad) {
            const float scale = kWide ? 0.011048543456039806f : 0.015625f;  // 1 / sqrt(8192), 1 / sqrt(4096)
#pragma unroll
            for (int r = 0; r < 8; ++r) d[h][r] = (__builtin_popcount(h * kN + idx_n + r) & 1) ? -scale : scale;
        } else {
            const float *fd = A.fd + (kVirt ? (size_t)virt_head(A, head, idx_n) * tn : (size_t)head * kPoints) + h * kN;
            load_coef8(fd + (idx_n & tmask), d[h]);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (2 * h + q < kParkScales) park[(2 * h + q) * kThreads] = make_float4(d[h][4 * q], d[h][4 * q + 1], d[h][4 * q + 2], d[h][4 * q + 3]);
        if (kParkFirst) park[(kParkScales + h) * kThreads] = make_float4(cn[h][0][1], cn[h][0][3], cn[h][0][5], cn[h][0][7]);
    }
    constexpr int kPer = 16 / (int)sizeof(T);  // elements per lane and load
    constexpr uint32_t kHalfSlot = kN * sizeof(T);  // bytes of a half in a slot
    const uint32_t ring0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_raw;
    const uint32_t slice = ring0 + (uint32_t)wave * (1024u * kHalfLoads);             // this wave's piece of a slot's first half
    const uint32_t rd_addr = slice + (uint32_t)lane_chunk(lane) * (16u * kHalfLoads);  // this thread's chunk
    // lane's bytes in a row, first and (32-bit rows) second load
    const uint32_t voff = elem_off<kVirt, kWide>(A, head, wave * 512 + lane * kPer, A.sub_ld_in) * (uint32_t)sizeof(T);
    const uint32_t voff1 = kHalfLoads == 2 ? elem_off<kVirt, kWide>(A, head, wave * 512 + (64 + lane) * kPer, A.sub_ld_in) * (uint32_t)sizeof(T) : 0u;
    const uint32_t slice_s = __builtin_amdgcn_readfirstlane(slice);  // uniform over the wave
    auto ring_load = [&](int j, int slot) {
        const int jj = j < n_my ? j : n_my - 1;  // past the end: re-read the last row (unused)
        const uint32_t vo = tail_off<kTail, T>(A, voff, wave * 512 + lane * kPer, jj == tail_j);
        const uint32_t vo1 = kHalfLoads == 2 ? tail_off<kTail, T>(A, voff1, wave * 512 + (64 + lane) * kPer, jj == tail_j) : 0u;
#pragma unroll
        for (int h = 0; h < kHalves; ++h) {
            const char *rowp = (const char *)(in + (row_first + jj * row_step) * A.ld_in + h * kN);
            const uint32_t m0v = slice_s + (uint32_t)slot * kSlotBytes + (uint32_t)h * kHalfSlot;
            if (kNt) {
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2 nt" : : "v"(vo), "s"(m0v), "s"(rowp) : "memory");
            } else {
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2" : : "v"(vo), "s"(m0v), "s"(rowp) : "memory");
                if (kHalfLoads == 2)
                    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %2" : : "v"(vo1), "s"(m0v + 1024u), "s"(rowp) : "memory");
            }
        }
    };
    ring_load(0, 0);
    ring_load(1, 1);
    // One pipeline step with the roles of the three buffers fixed at compile time (BA: phase A of row it,
    // BB: phase B of row it-1, BC: phase C of row it-2), so that buffer offsets become immediates of the
    // LDS instructions instead of per-lane address arithmetic.  Three such steps make one turn.
    auto step = [&](auto BA, auto BB, auto BC, int it) {
        constexpr int ba = decltype(BA)::value, bb = decltype(BB)::value, bc = decltype(BC)::value;
        float *la = lds + ba * kHalves * kLdsRow, *lb = lds + bb * kHalves * kLdsRow;  // (n = 8192: one buffer per half)
        float *lc = lds + bc * kHalves * kLdsRow;
        auto phase_a = [&]() {  // A(it)
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            u32x4 v[4];  // 16 bytes of half h at h * kHalfLoads (32-bit rows: and the next)
            constexpr int ro = ba * (int)kSlotBytes;
            constexpr int o1 = ro + (kHalfLoads == 2 ? 16 : (int)kHalfSlot), o2 = ro + (int)kHalfSlot, o3 = o2 + 16;
            if (it >= 4)
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPending) : "memory");
            else
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (kLoads == 1)
                asm volatile("ds_read_b128 %0, %1 offset:%2\n\ts_waitcnt lgkmcnt(0)" : "=v"(v[0]) : "v"(rd_addr), "n"(ro) : "memory");
            else if (kLoads == 2)
                asm volatile("ds_read_b128 %0, %2 offset:%3\n\tds_read_b128 %1, %2 offset:%4\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(v[0]), "=&v"(v[1]) : "v"(rd_addr), "n"(ro), "n"(o1) : "memory");
            else
                asm volatile("ds_read_b128 %0, %4 offset:%5\n\tds_read_b128 %1, %4 offset:%6\n\tds_read_b128 %2, %4 offset:%7\n\t"
                             "ds_read_b128 %3, %4 offset:%8\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                             : "v"(rd_addr), "n"(ro), "n"(o1), "n"(o2), "n"(o3) : "memory");
            // refills the slot of row it-1, consumed in the previous iteration (kTwoBuf: the slot just read)
            ring_load(it + 2, kTwoBuf ? ba : bb);
#pragma unroll
            for (int h = 0; h < kHalves; ++h) {
                Raw8 raw;
                const u32x4 v0 = v[h * kHalfLoads], v1 = v[h * kHalfLoads + (kHalfLoads - 1)];
                raw.lo = make_uint4(v0.x, v0.y, v0.z, v0.w);
                if (kHalfLoads == 2) raw.hi = make_uint4(v1.x, v1.y, v1.z, v1.w);
                float u[8];
                unpack8(raw, u, (const T *)nullptr);
                if (kParkFirst) {
                    const float4 c = park[(kParkScales + h) * kThreads];
                    const float c0[8] = {0.0f, c.x, 0.0f, c.y, 0.0f, c.z, 0.0f, c.w};
                    reg_layer_first<0>(u, c0);
                } else if (!kInverse) {
                    reg_layer_first<0>(u, cn[h][0]);
                }
                layers_a(u, cn[h]);
                lds_write_n(la + h * kLdsRow, an, u);
            }
        };
        auto phase_c = [&]() {  // C(it-2)
            float u[kHalves][8];
#pragma unroll
            for (int h = 0; h < kHalves; ++h) lds_read_n(lc + h * kLdsRow, an, u[h]);
            if constexpr (kWide && !kInverse) half_layer<false>(u, cw[0], cw[1]);  // layer 13
#pragma unroll
            for (int h = 0; h < kHalves; ++h) {
                layers_c(u[h], cn[h]);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (2 * h + q < kParkScales) {
                        const float4 p = park[(2 * h + q) * kThreads];
                        u[h][4 * q] *= p.x;
                        u[h][4 * q + 1] *= p.y;
                        u[h][4 * q + 2] *= p.z;
                        u[h][4 * q + 3] *= p.w;
                    } else {
#pragma unroll
                        for (int r = 4 * q; r < 4 * q + 4; ++r) u[h][r] *= d[h][r];
                    }
                }
            }
            finish_row<T, kMode, kBits, kLanes, kScale, kYq, kHist, kVirt, kHalves, kBig, kNt>(A, u, row_first + (it - 2) * row_step, head, chunk, bins, wg_bins, wg_max,
                                                                                               !(kTail && it - 2 == tail_j && in_tail_gap(A, idx_n)));
        };
        // The phases touch different buffers, so any order is correct as long as C precedes A where the two
        // share a buffer.  n = 4096: C, B, A measured 1-2 % faster than the other orders on all modes.
        if (it >= 2) phase_c();
        if (it >= 1 && it <= n_my) phase_b(lb);  // B(it-1)
        // (ahead of the other waves' arithmetic: it is this phase that sends for the next row.  131072 fp16 rows, forward, 356 ->
        // 348 us; the quantisers within 1 %; with a second barrier in the iteration 1 % slower)
        if (!kBig) __builtin_amdgcn_s_setprio(1);
        if (it < n_my) phase_a();
        if (!kBig) __builtin_amdgcn_s_setprio(0);
        __syncthreads();
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;
    const int end = n_my + 2;
    if (kTwoBuf) {
        for (int it = 0; it < end; it += 2) {  // (A, B, C) buffers: (0, 1, 0) -> (1, 0, 1) -> ...
            step(I0{}, I1{}, I0{}, it);
            if (it + 1 < end) step(I1{}, I0{}, I1{}, it + 1);
        }
    } else {
        for (int it = 0; it < end; it += 3) {  // (A, B, C) buffers: (0, 2, 1) -> (1, 0, 2) -> (2, 1, 0) -> ...
            step(I0{}, I2{}, I1{}, it);
            if (it + 1 < end) step(I1{}, I0{}, I2{}, it + 1);
            if (it + 2 < end) step(I2{}, I1{}, I0{}, it + 2);
        }
    }
    flush_bins();
}

template <typename T, bool kVirt, bool kWide, bool kBig, bool kTail>
static hipError_t launch_k12_t(Mode mode, const K12Args &A, int bits, unsigned grid, hipStream_t stream)
{
    constexpr bool V = kVirt, W = kWide, G = kBig;
    // Where the row loop is slower for the code of the other scale type beside it, the types are apart (us together / apart): 40001 and
    // 131072 fp16 rows of 4096, INT2 rows with groups of 4096, binary16 scales 174 / 154 and 534 / 471, float32 scales 172 / 153 and
    // 533 / 478, bf16 173 / 152 and 536 / 479; 32768 bf16 rows of 8192, INT4 codes, groups of 8192 351 / 335 and 349 / 337, of 256 249 /
    // 230 and 245 / 232.
    constexpr int kFakeF16 = kBig && !kVirt && !kWide && sizeof(T) == 2 ? kScaleF16 : 0, kFakeF32 = kFakeF16 ? kScaleF32 : 0;
    constexpr int kCodesF16 = kBig && kWide ? kScaleF16 : 0, kCodesF32 = kCodesF16 ? kScaleF32 : 0;
    void (*kern)(K12Args) = nullptr;
    if (mode == kFwdFake) {
        if (A.out && A.hist)
            kern = bits == 2 ? k12_kernel<T, kFwdFake, 2, 0, 0, true, true, V, W, G, false, kTail> : k12_kernel<T, kFwdFake, 4, 0, 0, true, true, V, W, G, false, kTail>;
        else if (A.out)
            kern = bits == 2 ? (A.scale_f16 ? k12_kernel<T, kFwdFake, 2, 0, kFakeF16, true, false, V, W, G, false, kTail>
                                            : k12_kernel<T, kFwdFake, 2, 0, kFakeF32, true, false, V, W, G, false, kTail>)
                             : k12_kernel<T, kFwdFake, 4, 0, 0, true, false, V, W, G, false, kTail>;
        else
            kern = bits == 2 ? k12_kernel<T, kFwdFake, 2, 0, 0, false, true, V, W, G, false, kTail> : k12_kernel<T, kFwdFake, 4, 0, 0, false, true, V, W, G, false, kTail>;
    } else if (mode == kFwdQuant && (kBig || kVirt || A.group != 128 || !A.scale_f16)) {
        if (A.scale_f16)
            kern = bits == 2 ? k12_kernel<T, kFwdQuant, 2, 0, kCodesF16, true, false, V, W, G, false, kTail> : k12_kernel<T, kFwdQuant, 4, 0, kCodesF16, true, false, V, W, G, false, kTail>;
        else
            kern = bits == 2 ? k12_kernel<T, kFwdQuant, 2, 0, kCodesF32, true, false, V, W, G, false, kTail> : k12_kernel<T, kFwdQuant, 4, 0, kCodesF32, true, false, V, W, G, false, kTail>;
    } else if constexpr (!kBig) {
        if constexpr (!kVirt) {
            if (mode == kHadamard)
                kern = k12_kernel<T, kHadamard, 4, 0, 0, true, false, false, W>;
        }
        if (kern) {
        } else if (mode == kFwd)
            kern = k12_kernel<T, kFwd, 4, 0, 0, true, false, V, W, false, false, kTail>;
        else if (mode == kInv)
            kern = k12_kernel<T, kInv, 4, 0, 0, true, false, V, W, false, false, kTail>;
        else  // the common activation format: group 128, binary16 scales
            kern = bits == 2 ? k12_kernel<T, kFwdQuant, 2, 16, 1, true, false, false, W> : k12_kernel<T, kFwdQuant, 4, 16, 1, true, false, false, W>;
    }
    if constexpr (!kBig && sizeof(T) == 2) {  // large batches of 16-bit rows: the non-temporal variants
        if (A.streaming && mode == kFwd) kern = k12_kernel<T, kFwd, 4, 0, 0, true, false, V, W, false, true, kTail>;
        if constexpr (!kVirt) {
            if (A.streaming && mode == kHadamard) kern = k12_kernel<T, kHadamard, 4, 0, 0, true, false, false, W, false, true>;
        }
    }
    if (!kern) return hipErrorInvalidValue;
    constexpr size_t lds_bytes = kWide ? kLdsBytesWide : kLdsBytes;
    // one record per kernel of this instantiation of the launcher (the modes, bit widths, output choices, scale types)
    static LdsLimitOnce once[5][2][3][2];
    const int variant = mode != kFwdFake ? 0 : (A.out && A.hist) ? 0 : A.out ? 1 : 2;
    const int general = (mode == kFwdQuant && (kBig || kVirt || A.group != 128 || !A.scale_f16)) ? 1 : 0;
    const bool quantises = mode == kFwdQuant || mode == kFwdFake;
    const int last = quantises ? A.scale_f16 != 0 : A.streaming && sizeof(T) == 2 && (mode == kFwd || mode == kHadamard);
    hipError_t e = once[mode][bits == 2 ? 0 : 1][mode == kFwdQuant ? general : variant][last].set((const void *)kern, lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds_bytes, stream, A);
    return hipGetLastError();
}

template <bool kVirt, bool kWide, bool kBig = false, bool kTail = false>
static hipError_t launch_k12_dtype(Mode mode, const K12Args &A, int bits, unsigned grid, int dtype, hipStream_t stream)
{
    switch (dtype) {
        case BQ_F32: return launch_k12_t<float, kVirt, kWide, kBig, kTail>(mode, A, bits, grid, stream);
        case BQ_F16: return launch_k12_t<__half, kVirt, kWide, kBig, kTail>(mode, A, bits, grid, stream);
        default: return launch_k12_t<bf16_t, kVirt, kWide, kBig, kTail>(mode, A, bits, grid, stream);
    }
}

// the n = 8192 instantiations live in a translation unit of their own
hipError_t launch_k13_dtype(Mode mode, const K12Args &A, int bits, unsigned grid, int dtype, hipStream_t stream);
// ... and so do those for quantiser groups of more than 128 channels (virt: n < 4096, wide: n = 8192)
hipError_t launch_k12_big_dtype(Mode mode, const K12Args &A, int bits, unsigned grid, int dtype, bool virt, bool wide,
                                hipStream_t stream);
// ... and the variants for a short last block (n < 4096)
hipError_t launch_k12_tail_dtype(Mode mode, const K12Args &A, int bits, unsigned grid, int dtype, bool big, hipStream_t stream);

}  // namespace bq

// n = 256 .. 4096 instantiations of the specialised transform kernels, and the choice between them.
#include "bq_k12_grid.h"
#include "bq_k12_kernel.h"
#include "bq_k12_inv.h"

namespace bq {

// n = 4096 or 8192 with any number of heads, or n = 256 .. 2048 where 4096 consecutive elements of the
// [rows][heads * n] array form one block of the kernel: several whole rows (k12_block_rows of them; the last block may have
// fewer) or a 4096-element piece of a wider row.
bool k12_supported(Mode mode, const void *in, const void *out, const Shape &s, const QuantArgs *q)
{
    if (s.n > 2 * kN || s.n < 256) return false;
    const int64_t width = (int64_t)s.n * s.heads;
    if (s.n < kN) {
        const bool rows_per_block = width <= kN && kN % width == 0;
        const bool blocks_per_row = width % kN == 0 && width / kN <= 512;
        if (!rows_per_block && !blocks_per_row) return false;
    }
    const int isz = s.dtype == BQ_F32 ? 4 : 2;
    const int vec = 16 / isz;  // elements per 16 bytes
    if (((uintptr_t)in & 15) || (s.ld_x % vec)) return false;
    if (mode != kFwdQuant && out && (((uintptr_t)out & 15) || (s.ld_y % vec))) return false;
    if (s.n < kN && ((int64_t)k12_block_rows(s) * (s.ld_x > s.ld_y ? s.ld_x : s.ld_y) * isz >= ((int64_t)1 << 31))) return false;
    if (s.n >= kN && s.heads > 512) return false;
    if (mode == kFwdQuant || mode == kFwdFake) {
        if (mode == kFwdQuant && ((uintptr_t)q->codes & 3)) return false;
    }
    return true;
}

bool hadamard_supported(const void *in, const void *out, const Shape &s)
{
    if (s.n != kN && s.n != 2 * kN) return false;
    if (s.heads > 512) return false;
    const int vec = s.dtype == BQ_F32 ? 4 : 8;  // elements per 16 bytes
    if (((uintptr_t)in & 15) || ((uintptr_t)out & 15) || (s.ld_x % vec) || (s.ld_y % vec)) return false;
    return true;
}

// per_head workgroups take the rows of every head in turn; returns the grid
static unsigned split_rows(K12Args &A, int64_t per_head)
{
    A.rows_each = (int)(A.rows / per_head);
    A.rows_extra = (int)(A.rows % per_head);
    return (unsigned)(per_head * A.heads);
}

hipError_t launch_hadamard(const void *in, void *out, const Shape &s, hipStream_t stream)
{
    K12Args A{};
    A.in = in;
    A.out = out;
    A.rows = s.rows;
    A.ld_in = A.sub_ld_in = s.ld_x;
    A.ld_out = A.sub_ld_out = s.ld_y;
    A.n = s.n;
    A.n_log = s.k;
    // beyond the 256 MB of the memory-side cache neither input nor output is found in a cache again
    A.streaming = (int64_t)s.rows * s.n * s.heads * (s.dtype == BQ_F32 ? 4 : 2) >= ((int64_t)256 << 20) ? 1 : 0;
    A.heads = s.heads;
    const bool wide = s.n > kN;
    int64_t per_head = 256 / A.heads > 0 ? 256 / A.heads : 1;  // as for the forward transform: one workgroup per compute unit
    if (per_head > A.rows) per_head = A.rows;
    const unsigned grid = split_rows(A, per_head);
    if (wide) return launch_k13_dtype(kHadamard, A, 4, grid, s.dtype, stream);
    return launch_k12_dtype<false, false>(kHadamard, A, 4, grid, s.dtype, stream);
}

int k12_block_rows(const Shape &s)
{
    const int64_t width = (int64_t)s.n * s.heads;
    return s.n < kN && width < kN ? (int)(kN / width) : 1;
}

// Elements of a batch from which its short last block is a launch of its own behind the whole blocks, which then run in the
// kernels without the check: the second launch costs 5 to 6 us, the check a share of the batch.  Measured at n = 256, 1024 and
// 2048, 2^18 to 2^30 elements, as one launch / as two:
//   INT2 codes of float32 rows, groups up to 128  2^25 43 / 43 us, 2^26 74 / 67, 2^28 293 / 237  (INT4: 2^28 286 / 290)
//   transforms of 16-bit rows                     2^26 52 / 56, 2^28 202 / 194 (forward), 191 / 190 (inverse), 2^30 789 / 752, 752 / 740
//   quantisers of 16-bit rows, groups above 128   2^26 65 / 67, 2^28 242 / 220, 2^30 939 / 820
//   everything else                               2^28 -2 to +6 %, 2^30 -4 to +1 %
static int64_t short_block_apart(Mode mode, int dtype, int bits, bool big)
{
    if (dtype == BQ_F32) return mode == kFwdQuant && bits == 2 && !big ? (int64_t)1 << 26 : (int64_t)1 << 29;
    return mode == kFwd || mode == kInv || big ? (int64_t)1 << 28 : (int64_t)1 << 29;
}

hipError_t launch_k12(Mode mode, const void *in, void *out, const PlanView &pv, const Shape &s,
                      const QuantArgs *q, hipStream_t stream)
{
    const bool virt = s.n < kN, wide = s.n > kN;
    const bool big = (mode == kFwdQuant || mode == kFwdFake) && q->group > 128;
    const int64_t width = (int64_t)s.n * s.heads;
    const int block_rows = k12_block_rows(s);  // rows of the caller per kernel row
    if (s.rows > block_rows && s.rows % block_rows != 0 && s.rows * width >= short_block_apart(mode, s.dtype, q ? q->bits : 0, big)) {
        const size_t isz = s.dtype == BQ_F32 ? 4 : 2;
        Shape whole = s, rest = s;
        rest.rows = s.rows % block_rows;
        whole.rows = s.rows - rest.rows;
        hipError_t e = launch_k12(mode, in, out, pv, whole, q, stream);
        if (e != hipSuccess) return e;
        QuantArgs qr = q ? *q : QuantArgs{};
        if (mode == kFwdQuant) {
            qr.codes += (size_t)whole.rows * (width * q->bits / 8);
            qr.scales = (char *)q->scales + (size_t)whole.rows * (width / q->group) * (q->scale_f16 ? 2 : 4);
        }
        return launch_k12(mode, (const char *)in + (size_t)whole.rows * s.ld_x * isz, out ? (char *)out + (size_t)whole.rows * s.ld_y * isz : nullptr,
                          pv, rest, q ? &qr : nullptr, stream);
    }
    K12Args A{};
    A.in = in;
    A.out = out;
    A.fg = mode == kInv ? pv.fg_inv : pv.fg_fwd;
    A.fd = mode == kInv ? pv.fd_inv : pv.fd_fwd;
    A.cs = pv.cs;
    A.plan = pv.ref;
    A.rows = (s.rows + block_rows - 1) / block_rows;
    A.tail_rows = (int)(s.rows % block_rows);
    A.ld_in = s.ld_x * block_rows;
    A.ld_out = s.ld_y * block_rows;
    A.sub_ld_in = s.ld_x;
    A.sub_ld_out = s.ld_y;
    A.n = s.n;
    A.n_log = s.k;
    // beyond the 256 MB of the memory-side cache neither input nor output is found in a cache again
    A.streaming = (int64_t)s.rows * s.n * s.heads * (s.dtype == BQ_F32 ? 4 : 2) >= ((int64_t)256 << 20) ? 1 : 0;
    A.heads = virt ? (width > kN ? (int)(width / kN) : 1) : s.heads;  // virt: 4096-element blocks per row
    A.row_log = virt ? (width >= kN ? kK : ilog2_exact((int)width)) : 0;
    int bits = 4;
    if (q) {
        A.codes = q->codes;
        A.scales = q->scales;
        A.hist = q->hist;
        A.group = q->group;
        A.scale_f16 = q->scale_f16;
        bits = q->bits;
    }
    // Persistent workgroups, a multiple of the head count: each pays for its tables (213 KB from L2 at n = 4096) once.
    // Transforms: one per compute unit (2^30 16-bit elements at every n from 256 to 4096: forward 0.79 ms, 0.84 with three, five or
    // seven per unit, 6 to 18 % more at other counts; two-phase inverse of 16-bit rows 0.78 ms, 512 workgroups 0.86, 768 0.85,
    // 1024 0.99; float32 rows forward 0.776, inverse 0.779 ms; small batches too).  n = 8192: one fits.
    const bool inv_ring = mode == kInv && !wide && s.dtype != BQ_F32;
    int64_t per_head = 256 / A.heads > 0 ? 256 / A.heads : 1;
    if ((mode == kFwdQuant || mode == kFwdFake) && !wide)
        per_head = quantiser_workgroups_per_head(A.rows, A.heads,
                                                 {mode == kFwdFake && out != nullptr, mode == kFwdFake && A.hist != nullptr, big, s.dtype == BQ_F32});
    if (per_head > A.rows) per_head = A.rows;
    const unsigned grid = split_rows(A, per_head);
    if (A.tail_rows) return launch_k12_tail_dtype(mode, A, bits, grid, s.dtype, big, stream);
    if (big)
        return launch_k12_big_dtype(mode, A, bits, grid, s.dtype, virt, wide, stream);
    if (wide) return launch_k13_dtype(mode, A, bits, grid, s.dtype, stream);
    if (inv_ring)  // 16-bit rows: the two-phase inverse
        return virt ? launch_k12_inv_ring<true>(A, grid, s.dtype, stream) : launch_k12_inv_ring<false>(A, grid, s.dtype, stream);
    if (virt) return launch_k12_dtype<true, false>(mode, A, bits, grid, s.dtype, stream);
    return launch_k12_dtype<false, false>(mode, A, bits, grid, s.dtype, stream);
}

}  // namespace bq

// n = 256 .. 2048 instantiations for batches whose last block of 4096 elements is short (K12Args::tail_rows).
#include "bq_k12_kernel.h"
#include "bq_k12_inv.h"

namespace bq {

hipError_t launch_k12_tail_dtype(Mode mode, const K12Args &A, int bits, unsigned grid, int dtype, bool big, hipStream_t stream)
{
    if (big) return launch_k12_dtype<true, false, true, true>(mode, A, bits, grid, dtype, stream);
    if (mode == kInv && dtype != BQ_F32) return launch_k12_inv_ring<true, true>(A, grid, dtype, stream);
    return launch_k12_dtype<true, false, false, true>(mode, A, bits, grid, dtype, stream);
}

}  // namespace bq

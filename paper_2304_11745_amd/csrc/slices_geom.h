// K positions of slices_kernel's requests (host and device code).
#pragma once
#include <hip/hip_runtime.h>

namespace gacer {

// K range [k_lo, k_end) of wave or workgroup slice `slice`, of `per` elements each
struct SlicesRange { int k_lo, k_end; };
__host__ __device__ inline SlicesRange slices_range(int K, int per, int slice)
{
    const int lo = slice * per, k_lo = K < lo ? K : lo, hi = k_lo + per;
    return {k_lo, K < hi ? K : hi};
}

// Scalar offset of the loads of the batch at element kb: its K position in bytes.  A batch beyond the slice (a wave requests two batches
// whatever it has; the fused affine form two past the last) is masked by its vector offsets, which stand for "out of range" only as
// long as the scalar offset lies in the descriptor's range.  With a single row that range ends with K, so no offset passes `last`, K's
// last vector.
__host__ __device__ inline int slices_offset(int kb, int last, int esz) { return kb * esz < last ? kb * esz : last; }
inline int slices_last(int K, int esz) { return K * esz - 16; }

}  // namespace gacer

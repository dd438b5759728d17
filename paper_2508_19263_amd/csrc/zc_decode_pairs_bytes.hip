// Builds of k_decode_pairs for FP8 in byte symbols.
#include "zc_decode_pairs_kernel.h"

namespace zc {

int launch_pairs_bytes(bool two, bool xor_delta, uint32_t chunks, bool long_rings, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work,
                       const TensorDev &s, int use_single, uint32_t first_slot, hipStream_t st)
{
    if (!long_rings) return launch_pairs_x<ZC_FMT_FP8_E4M3_BYTES, kMany>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st);
    // (a whole table is for calls that leave a workgroup a compute unit: see pairs_shape in zc_decompress.cpp)
    if (two || n_work > 256) return launch_pairs_x<ZC_FMT_FP8_E4M3_BYTES, kFewTwo>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st);
    return launch_pairs_x<ZC_FMT_FP8_E4M3_BYTES, kFew>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st);
}

}  // namespace zc

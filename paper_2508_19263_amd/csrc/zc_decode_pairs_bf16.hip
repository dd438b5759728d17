// Builds of k_decode_pairs for BF16.
#include "zc_decode_pairs_kernel.h"

namespace zc {

int launch_pairs_bf16(bool two, bool xor_delta, uint32_t chunks, bool long_rings, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work,
                      const TensorDev &s, int use_single, uint32_t first_slot, hipStream_t st)
{
    // (a workgroup per compute unit: the loop that waits for no word is ahead; with several wavefronts per SIMD the one of fewer instructions.
    // 1,526 chunks of a delta 314 | 303 us, but 3,052, three wavefronts per SIMD, 436 | 454)
    if (!long_rings && two && n_work <= 256) return launch_pairs_x<ZC_FMT_BF16, kManyTwo>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st);
    if (!long_rings) return launch_pairs_x<ZC_FMT_BF16, kMany>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st);
    if (two) return launch_pairs_x<ZC_FMT_BF16, kFewTwo>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st);
    return launch_pairs_x<ZC_FMT_BF16, kFew>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st);
}

}  // namespace zc

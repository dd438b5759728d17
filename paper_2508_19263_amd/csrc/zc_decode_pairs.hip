// Builds of k_decode_pairs for FP8 E4M3 and E5M2, and the choice among all of them.
#include "zc_decode_pairs_kernel.h"

namespace zc {

// two: some tensor's sign+mantissa field is table decoded too; chunks: per work item, 4 with long rings, else 1, 2, 4 or 8; first_slot:
// where a single tensor's first work item starts
int launch_decode_pairs(uint32_t fmt, bool two, bool xor_delta, uint32_t chunks, bool long_rings, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work,
                        const TensorDev *single, uint32_t first_slot, void *stream)
{
    if (n_work == 0) return 0;
    if (long_rings ? chunks != 4 : chunks != 1 && chunks != 2 && chunks != 4 && chunks != 8) return 1;
    hipStream_t st = (hipStream_t)stream;
    const TensorDev s = single ? *single : TensorDev{};
    const int use_single = single ? 1 : 0;
    switch (fmt) {
    case ZC_FMT_BF16: return launch_pairs_bf16(two, xor_delta, chunks, long_rings, d_descs, d_work, n_work, s, use_single, first_slot, st);
    case ZC_FMT_FP8_E4M3_BYTES: return launch_pairs_bytes(two, xor_delta, chunks, long_rings, d_descs, d_work, n_work, s, use_single, first_slot, st);
    case ZC_FMT_FP8_E4M3: return long_rings ? launch_pairs_x<ZC_FMT_FP8_E4M3, kFew>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st) : 1;       // (only calls of few chunks come here)
    case ZC_FMT_FP8_E5M2:
        if (!long_rings) return launch_pairs_x<ZC_FMT_FP8_E5M2, kMany>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st);
        return launch_pairs_x<ZC_FMT_FP8_E5M2, kFew>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st);
    default: return 1;
    }
}

}  // namespace zc

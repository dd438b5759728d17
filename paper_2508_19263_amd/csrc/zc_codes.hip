// Code construction on the device: from the histograms that k_hist left in the workspace to everything the
// size pass and the encoder read (encode tables, field modes and refill periods in the descriptors, the
// code-length tables in the header blobs), without a round trip to the host.  One workgroup per (tensor,
// field).  The result is bit for bit what the host construction in zc_codebook.cpp gives: the same optimal
// length-limited code (package-merge) with the same tie rules
//   * leaves ordered by (frequency, symbol value), ascending;
//   * in a merged row a leaf goes before a package of equal weight;
//   * canonical codes handed out in (length, symbol value) order,
// the same choice between a coded, a raw and a constant field (Sec. 3.1: a field that does not compress is
// stored as is), and the same histogram marginals per format.
//
// Package-merge in the form used here keeps, per row, only the weights (two rows at a time) and one bit
// per item that says whether it is a leaf: the code length of the i-th cheapest leaf is the number of rows
// in which it lies inside the item budget that is walked down from the top row (2n-2 items there; every
// package inside the budget stands for two items of the row below).  A row is the merge of the sorted
// leaves with the sorted packages of the row below, so every item finds its place with one binary search.
#include <hip/hip_runtime.h>

#include "zc_internal.h"

namespace zc {

namespace {

constexpr int kCodeThreads = 256;          // >= the largest alphabet: one thread per symbol, leaf and package
constexpr int kMaxRow = 512;               // a row holds at most 2n-1 items

__device__ __forceinline__ uint32_t reverse_code(uint32_t code, uint32_t len) { return len ? __brev(code) >> (32 - len) : 0u; }

// sums and maxima over the workgroup: shuffles inside a wavefront, then one LDS atomic per wavefront (all lanes
// of a workgroup hitting one LDS address with atomics take their turns one by one)
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64); return v; }
__device__ __forceinline__ uint32_t wave_max(uint32_t v) { for (int o = 32; o > 0; o >>= 1) { const uint32_t w = __shfl_xor(v, o, 64); v = w > v ? w : v; } return v; }
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v)
{
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)v, o, 64), hi = __shfl_xor((uint32_t)(v >> 32), o, 64);
        v += ((unsigned long long)hi << 32) | lo;
    }
    return v;
}

// Rows limit-1 .. 1 of the package-merge (the row `limit` is the leaves themselves, lw[0..n) ascending): fills
// leaf_bits and row_size.  W: the weight type; 32 bits are enough when 16 times the sum of all weights fits (an
// item of any row holds a leaf at most once per row below it), and halve the LDS traffic of the searches.
// Called by the whole workgroup.
template <typename W>
__device__ void build_rows(const W *lw, W *pw, W *row0, W *row1, uint32_t n, int limit, uint32_t (*leaf_bits)[kMaxRow / 32], uint32_t *row_size)
{
    const uint32_t tid = threadIdx.x;
    if (tid == 0) row_size[limit] = n;
    uint32_t m = n;                                       // items of the row below
    const W *below = lw;
    W *out = row0, *other = row1;
    for (int d = limit - 1; d >= 1; d--) {
        const uint32_t n_pk = m / 2;
        if (tid < n_pk) pw[tid] = below[2 * tid] + below[2 * tid + 1];
        __syncthreads();
        // Both searches of a thread advance together, in halving steps from the largest power of two that either list
        // reaches (an LDS round trip each: nine for 256 leaves, five for 16): the packages strictly cheaper than leaf `tid`
        // go before it, the leaves that cost no more than package `tid` go before that.
        const W wl = tid < n ? lw[tid] : (W)0, wp = tid < n_pk ? pw[tid] : (W)0;
        uint32_t below_leaf = 0, below_pack = 0;
#pragma unroll 1
        for (uint32_t step = 1u << (31 - __clz((int)(n > n_pk ? n : n_pk))); step > 0; step >>= 1) {
            const uint32_t a = below_leaf + step, b = below_pack + step;
            const W pa = pw[(a <= n_pk ? a : 1u) - 1], lb = lw[(b <= n ? b : 1u) - 1];
            if (a <= n_pk && pa < wl) below_leaf = a;
            if (b <= n && lb <= wp) below_pack = b;
        }
        if (tid < n) {
            const uint32_t pos = tid + below_leaf;
            out[pos] = wl;
            atomicOr(&leaf_bits[d][pos / 32], 1u << (pos % 32));
        }
        if (tid < n_pk) out[tid + below_pack] = wp;
        m = n + n_pk;
        if (tid == 0) row_size[d] = m;
        __syncthreads();
        // A row whose weights are those of the row below has nothing but copies of itself above it (a code that the limit does
        // not bind: 256 nearly equally likely symbols are through after nine of sixteen rows).  Not looked for in the first rows.
        if (limit - d >= 7 && d > 1 && row_size[d + 1] == m) {
            bool same = true;
            for (uint32_t i = tid; i < m; i += kCodeThreads) same = same && out[i] == below[i];
            if (__syncthreads_and(same ? 1 : 0)) {
                for (uint32_t i = tid; i < (uint32_t)(d - 1) * (kMaxRow / 32); i += kCodeThreads) leaf_bits[1 + i / (kMaxRow / 32)][i % (kMaxRow / 32)] = leaf_bits[d][i % (kMaxRow / 32)];
                if (tid >= 1 && tid < (uint32_t)d) row_size[tid] = m;
                __syncthreads();
                return;
            }
        }
        below = out;
        W *const swap = out; out = other; other = swap;
    }
}

}  // namespace

__global__ __launch_bounds__(kCodeThreads) void k_codes(TensorDev *descs, const uint64_t *hist, CodeParams cp, uint8_t *blobs, uint32_t *enc_tables)
{
    __shared__ unsigned long long h[256];              // the field's histogram by symbol
    __shared__ unsigned long long lw[256];             // leaf weights, cheapest first
    __shared__ unsigned long long row[2][kMaxRow];     // the row below and the row being merged
    __shared__ __attribute__((aligned(16))) unsigned long long pw[256];      // package weights of the row below
    __shared__ uint32_t leaf_bits[17][kMaxRow / 32];   // per row: which items are leaves
    __shared__ uint32_t leaves_before[17][kMaxRow / 32];
    __shared__ uint32_t row_size[17], leaves_in[17];
    __shared__ uint32_t wave_count[kCodeThreads / 64][17], next[17];
    __shared__ uint8_t order[256], len[256];
    __shared__ unsigned long long pay_s, sum_s;
    __shared__ uint32_t n_s, konst_s, flat_s, lmax_s;

    const uint32_t t = blockIdx.x, f = blockIdx.y, tid = threadIdx.x;
    const uint32_t fmt = cp.fmt;
    const uint32_t grouped = (fmt == ZC_FMT_FP8_E4M3_BYTES || fmt == ZC_FMT_FP4_E2M1_MX_BYTES) ? 1u : 0u;
    const uint32_t sb = (f == 2 || grouped || fmt == ZC_FMT_FP8_E5M2 || fmt == ZC_FMT_BF16) ? 8u : fmt == ZC_FMT_FP8_E4M3 ? 4u : 2u;
    const uint32_t A = 1u << sb;
    const int limit = cp.limit[f];
    const uint64_t *hist3 = hist + (uint64_t)t * 768;

    // ---- the field's histogram
    h[tid] = 0; len[tid] = 0;
    if (tid < 17) { row_size[tid] = 0; leaves_in[tid] = 0; next[tid] = 0; }
    for (uint32_t i = tid; i < 17 * (kMaxRow / 32); i += kCodeThreads) (&leaf_bits[0][0])[i] = 0;
    if (tid == 0) { pay_s = 0; sum_s = 0; n_s = 0; konst_s = 0; flat_s = 0; lmax_s = 0; }
    __syncthreads();
    if (f == 2) h[tid] = hist3[512 + tid];
    else if (fmt == ZC_FMT_BF16 || grouped) h[tid] = hist3[256 * f + tid];
    else {
        // copies of the two fields' bins, one behind the other
        const uint32_t stride = hist_copy_stride(fmt), second = hist_second_field(fmt);
        for (uint32_t i = tid; i < 512; i += kCodeThreads) {
            const uint32_t at = i % stride, v = f ? at - second : at;
            if (at >= second == (f == 1) && v < A) atomicAdd(&h[v], hist3[i]);
        }
    }
    __syncthreads();

    // ---- leaves in (frequency, symbol) order
    const unsigned long long hv = tid < A ? h[tid] : 0ull;
    const bool present = hv != 0;
    {
        const uint32_t wn = wave_sum(present ? 1u : 0u), wk = wave_max(present ? tid : 0u);
        const unsigned long long ws = wave_sum(hv);
        if ((tid & 63) == 0) { atomicAdd(&n_s, wn); atomicMax(&konst_s, wk); atomicAdd(&sum_s, ws); }
    }
    __syncthreads();
    const uint32_t n = n_s;
    const bool narrow = 16ull * sum_s < (1ull << 32);         // every weight of every row fits 32 bits
    uint32_t rank = 0;
    if (narrow) {
        // absent symbols get the largest key, so they rank behind every present one and need no test of their own
        uint32_t *h32 = reinterpret_cast<uint32_t *>(pw);
        h32[tid] = present ? (uint32_t)hv : 0xFFFFFFFFu;
        __syncthreads();
        const uint32_t mine = h32[tid];
        const uint4 *h4 = reinterpret_cast<const uint4 *>(h32);
#pragma unroll 8
        for (uint32_t u = 0; u < A; u += 4) {
            const uint4 q = h4[u / 4];
            rank += (q.x < mine || (q.x == mine && u < tid)) ? 1u : 0u;
            rank += (q.y < mine || (q.y == mine && u + 1 < tid)) ? 1u : 0u;
            rank += (q.z < mine || (q.z == mine && u + 2 < tid)) ? 1u : 0u;
            rank += (q.w < mine || (q.w == mine && u + 3 < tid)) ? 1u : 0u;
        }
    } else {
#pragma unroll 8
        for (uint32_t u = 0; u < A; u++) {
            const unsigned long long hu = h[u];
            rank += (hu != 0 && (hu < hv || (hu == hv && u < tid))) ? 1u : 0u;
        }
    }
    if (present) { lw[rank] = hv; order[rank] = (uint8_t)tid; }
    __syncthreads();

    uint32_t mode = ZC_MODE_EMPTY, konst = 0, lmax = 0;
    if (n == 1) { mode = ZC_MODE_CONST; konst = konst_s; }
    else if (n > 1) {
        mode = ZC_MODE_HUFF;
        // ---- rows limit-1 .. 1
        if (narrow) {
            uint32_t *lw32 = reinterpret_cast<uint32_t *>(h);      // the histogram by symbol is not needed any more
            const uint32_t mine = tid < n ? (uint32_t)lw[tid] : 0u;
            __syncthreads();
            if (tid < n) lw32[tid] = mine;
            __syncthreads();
            build_rows<uint32_t>(lw32, reinterpret_cast<uint32_t *>(pw), reinterpret_cast<uint32_t *>(row[0]), reinterpret_cast<uint32_t *>(row[1]),
                                 n, limit, leaf_bits, row_size);
        } else build_rows<unsigned long long>(lw, pw, row[0], row[1], n, limit, leaf_bits, row_size);
        // ---- walk the budget down from the top row.  leaves_before[d][w]: leaves in the first 32 * w items of row d, so that a
        // row costs the walk one LDS round trip
        for (uint32_t i = tid; i < 17 * (kMaxRow / 32); i += kCodeThreads) {
            const uint32_t d = i / (kMaxRow / 32), w = i % (kMaxRow / 32);
            uint32_t c = 0;
            for (uint32_t v = 0; v < w; v++) c += (uint32_t)__popc(leaf_bits[d][v]);
            leaves_before[d][w] = c;
        }
        __syncthreads();
        if (tid < 64) {
            uint32_t budget = 2 * n - 2;
            for (int d = 1; d <= limit && budget > 0; d++) {
                const uint32_t b = budget < row_size[d] ? budget : row_size[d];
                // (b is below 512: a row holds at most 2n - 1 items)
                const uint32_t leaves = d == limit ? b : leaves_before[d][b / 32] + (uint32_t)__popc(leaf_bits[d][b / 32] & ((1u << (b % 32)) - 1));
                if (tid == 0) leaves_in[d] = leaves;
                budget = 2 * (b - leaves);
            }
        }
        __syncthreads();
        {
            uint32_t l = 0;
            if (tid < n) {
                for (int d = 1; d <= limit; d++) l += leaves_in[d] > tid ? 1u : 0u;
                len[order[tid]] = (uint8_t)l;
            }
            const unsigned long long wp = wave_sum(tid < n ? lw[tid] * l : 0ull);
            const uint32_t wl = wave_max(l);
            if ((tid & 63) == 0) { atomicAdd(&pay_s, wp); atomicMax(&lmax_s, wl); }
        }
        __syncthreads();
        lmax = lmax_s;
        // Sec. 3.1: a field that does not compress is stored as is
        if (cp.policy == ZC_POLICY_AUTO && 16ull * pay_s > 15ull * sum_s * sb) { mode = ZC_MODE_RAW; lmax = 0; }
    }
    __syncthreads();
    if (mode != ZC_MODE_HUFF) len[tid] = 0;
    __syncthreads();

    // ---- canonical codes in (length, symbol) order
    const uint32_t my_len = tid < A ? len[tid] : 0u;
    uint32_t before = 0;                               // symbols below this one with the same length: first those of the wavefront
#pragma unroll
    for (uint32_t l = 1; l <= 16; l++) {
        const uint64_t m = __ballot(my_len == l);
        const uint32_t c = (uint32_t)__popcll(m);
        if (my_len == l) before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        if ((tid & 63) == 0) wave_count[tid >> 6][l] = c;
    }
    {
        const uint32_t c = (uint32_t)__popcll(__ballot(tid < A && my_len == sb));
        if ((tid & 63) == 0 && c) atomicAdd(&flat_s, c);
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t code = 0, below = 0;
        for (int l = 1; l <= 16; l++) {
            code = (code + below) << 1;
            below = wave_count[0][l] + wave_count[1][l] + wave_count[2][l] + wave_count[3][l];
            next[l] = code;
        }
    }
    __syncthreads();
    uint32_t code = 0;
    if (my_len) {
        for (uint32_t w = 0; w < tid >> 6; w++) before += wave_count[w][my_len];
        code = next[my_len] + before;
    }

    // ---- what the other kernels read
    enc_tables[(uint64_t)t * 768 + f * 256 + tid] = tid < A ? (my_len << 16) | reverse_code(code, my_len) : 0u;
    uint8_t *blob = blobs + (uint64_t)t * cp.blob_bytes;
    TensorDev &d = descs[t];
    if (tid < A) blob[d.table_off[f] + tid] = (uint8_t)my_len;
    if (tid == 0) {
        const uint32_t kind = mode == ZC_MODE_RAW ? 2u : mode != ZC_MODE_HUFF ? 3u : flat_s == A ? 1u : 0u;
        // symbols between two refill steps of the field's stream: the largest power of two r with r * lmax <= 32,
        // at most a run
        const uint32_t G = f == 2 ? 16u : cp.run_len;
        uint32_t r = 1;
        const uint32_t lm = lmax < 1 ? 1u : lmax;
        while (2 * r * lm <= 32) r *= 2;
        if (r > G) r = G;
        blob[32 + 4 * f] = (uint8_t)mode; blob[33 + 4 * f] = (uint8_t)sb; blob[34 + 4 * f] = (uint8_t)lmax; blob[35 + 4 * f] = (uint8_t)konst;
        d.mode[f] = (uint8_t)mode; d.lmax[f] = (uint8_t)lmax; d.konst[f] = (uint8_t)konst; d.period[f] = (uint8_t)r; d.kind[f] = (uint8_t)kind;
    }
}

// After k_codes: which kernels take the tensor's whole chunks, and the exponent-pair table of the FP8
// kernels (two codes concatenated, for a pair of exponents: the table slot of the third field, which FP8
// does not have).  The FP8 kernels are written for a refill period of 4 on the exponents (longest code 5..8
// bits) and a sign+mantissa field that is flat coded or raw.
__global__ __launch_bounds__(256) void k_codes_finish(TensorDev *descs, CodeParams cp, uint32_t *enc_tables)
{
    TensorDev &d = descs[blockIdx.x];
    const bool fast = cp.fmt == ZC_FMT_FP8_E4M3 && d.fast_shape && d.mode[0] == ZC_MODE_HUFF && d.period[0] == 4 && (d.kind[1] == 1 || d.kind[1] == 2);
    uint32_t *enc = enc_tables + (uint64_t)blockIdx.x * 768;
    if (fast) {
        const uint32_t u = threadIdx.x, e0 = enc[u & 15], e1 = enc[u >> 4];
        const uint32_t l0 = e0 >> 16, l1 = e1 >> 16;
        enc[512 + u] = ((l0 + l1) << 16) | (e0 & 0xFFFFu) | ((e1 & 0xFFFFu) << l0);
    }
    // BF16, and FP8 in byte symbols: the 64-lane encoder takes a table-coded exponent field next to a sign+mantissa field
    // that is flat, raw, or table coded with a refill period of 2 or 4; the BF16 page kernels (fewer lanes) want the latter flat or raw and, with
    // two exponents per refill step, no 1-bit code (the bound on their staging ring needs 4 bits per step)
    __shared__ uint32_t lmin_s;
    if (threadIdx.x == 0) lmin_s = 16;
    __syncthreads();
    const uint32_t my_len = enc[threadIdx.x] >> 16;
    if (my_len) atomicMin(&lmin_s, my_len);
    __syncthreads();
    const bool plain_sm = d.kind[1] == 1 || d.kind[1] == 2;
    // (FP8 E5M2, 16 symbols per run: both fields table coded, refill periods of at most 8)
    const bool e5m2 = cp.fmt == ZC_FMT_FP8_E5M2 && d.streams == 64 && d.kind[1] == 0 && d.period[0] <= 8 && d.period[1] >= 2 && d.period[1] <= 8;
    const bool bf16 = d.fast_shape && d.kind[0] == 0 &&
                      (d.streams == 64 ? (e5m2 || ((cp.fmt == ZC_FMT_BF16 || cp.fmt == ZC_FMT_FP8_E4M3_BYTES) &&
                                                   (plain_sm || (d.kind[1] == 0 && (d.period[1] == 2 || d.period[1] == 4)))))
                                       : (cp.fmt == ZC_FMT_BF16 && plain_sm && (d.period[0] != 2 || lmin_s >= 2)));
    if (threadIdx.x == 0) d.route = fast ? 1 : bf16 ? 2 : 0;
}

int launch_codes(TensorDev *d_descs, uint32_t n_tensors, const uint64_t *d_hist, const CodeParams &cp, uint8_t *d_blobs, uint32_t *d_enc, bool routes, void *stream)
{
    if (n_tensors == 0) return 0;
    hipLaunchKernelGGL(k_codes, dim3(n_tensors, cp.nf), dim3(kCodeThreads), 0, (hipStream_t)stream, d_descs, d_hist, cp, d_blobs, d_enc);
    if (routes) hipLaunchKernelGGL(k_codes_finish, dim3(n_tensors), dim3(256), 0, (hipStream_t)stream, d_descs, cp, d_enc);
    return (int)hipGetLastError();
}

}  // namespace zc

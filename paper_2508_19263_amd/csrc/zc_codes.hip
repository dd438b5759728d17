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
// Package-merge in the form used here keeps, per row, only the weights (two rows at a time) and every leaf's place: the code length of the
// i-th cheapest leaf is the number of rows in which its place lies inside the item budget that is walked down from the top row (2n-2
// items there; every package inside the budget stands for two items of the row below).  A row is the merge of the sorted leaves with
// the sorted packages of the row below, so every item finds its place with one binary search.
//
// Bound by latency: every step is a round trip to LDS.  So the steps of the searches are unrolled (the lists are padded, so that a step is a read at
// a constant distance, a compare and an addition: 100 cycles for both of a thread's, where a loop with its bounds checks took 360), up to 64 leaves
// are one wavefront's and need no barriers, a row whose packages are those of the row below is not merged at all, and leaves are ranked by keys of weight and
// symbol in one.  MI355X, two fields of 256 symbols, limit 16: 30.9 -> 17.0 us (38.4 -> 17.1 with weights of 64 bits); of its cycles the rows took 37,000 and take
// 22,000, the ranks 18,000 and 7,500 (a key is compared in one instruction; two compares of 32 bits, for weight and symbol, take 10,000), the walk 8,300 and 3,800, the
// canonical codes 6,000 and 3,300.
#include <hip/hip_runtime.h>

#include "zc_internal.h"

namespace zc {

namespace {

constexpr int kCodeThreads = 256;          // >= the largest alphabet: one thread per symbol, leaf and package
constexpr int kMaxRow = 512;               // a row holds at most 2n-1 items

__device__ __forceinline__ uint32_t reverse_code(uint32_t code, uint32_t len) { return len ? __brev(code) >> (32 - len) : 0u; }

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v)
{
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)v, o, 64), hi = __shfl_xor((uint32_t)(v >> 32), o, 64);
        v += ((unsigned long long)hi << 32) | lo;
    }
    return v;
}

// ONE: the caller is one wavefront, whose LDS accesses are served in order
template <bool ONE>
__device__ __forceinline__ void sync_rows()
{
    if (ONE) { asm volatile("" ::: "memory"); __builtin_amdgcn_wave_barrier(); }         // (for the compiler; no wait)
    else __syncthreads();
}
// a barrier, and whether v holds for all threads; said: a word per wavefront, not the one of the last call
template <bool ONE>
__device__ __forceinline__ bool all_and_sync(bool v, uint32_t *said)
{
    if (ONE) { sync_rows<true>(); return __all(v); }
    const uint32_t mine = __all(v) ? 1u : 0u;
    if ((threadIdx.x & 63) == 0) said[threadIdx.x >> 6] = mine;
    __syncthreads();
    return (said[0] & said[1] & said[2] & said[3]) != 0;
}

// Rows limit-1 .. 1 of the package-merge (the row `limit` is the leaves themselves, lw[0..n) ascending, n < 2 * TOP): fills place[d][i], where leaf i
// lies in row d, and row_size.  lw and pw hold 2 * TOP entries, those beyond the lists the largest value of W, the weight type; 32 bits are
// enough when 16 times the sum of all weights fits (an item of any row holds a leaf at most once per row below it), and halve the LDS traffic of
// the searches.  Called by the whole workgroup, or (ONE) by its first wavefront for up to 64 leaves.
template <typename W, int TOP, bool ONE>
__device__ void build_rows(const W *lw, W *pw, W *row0, W *row1, uint32_t n, int limit, uint16_t (*place)[kCodeThreads], uint32_t *row_size)
{
    __shared__ uint32_t said[2][kCodeThreads / 64];
    const uint32_t tid = threadIdx.x;
    if (tid == 0) row_size[limit] = n;
    uint32_t m = n, n_pk_below = 0xFFFFFFFFu;             // items of the row below
    const W *below = lw;
    W *out = row0, *other = row1;
    const W none = ~(W)0, wl = tid < n ? lw[tid] : (W)0;
    W wp_below = none;
    for (int d = limit - 1; d >= 1; d--) {
        const uint32_t n_pk = m / 2;
        const W wp = tid < n_pk ? below[2 * tid] + below[2 * tid + 1] : none;
        pw[tid] = wp;
        // A row with the packages of the row below is that row, and so are all above it (a code that the limit does not bind: 256 nearly
        // equally likely symbols are through after nine of sixteen rows).
        if (all_and_sync<ONE>(wp == wp_below && n_pk == n_pk_below, said[d & 1])) {
            if (tid < n) {
                const uint16_t at = place[d + 1][tid];
                for (int i = d; i >= 1; i--) place[i][tid] = at;
            }
            if (tid >= 1 && tid <= (uint32_t)d) row_size[tid] = n + n_pk;
            break;
        }
        wp_below = wp; n_pk_below = n_pk;
        // Both searches of a thread advance together, in halving steps: the packages strictly cheaper than leaf `tid` go before it, the
        // leaves that cost no more than package `tid` go before that.
        uint32_t below_leaf = 0, below_pack = 0;
#pragma unroll
        for (int step = TOP; step > 0; step >>= 1) {
            const W pa = pw[below_leaf + step - 1], lb = lw[below_pack + step - 1];
            below_leaf += pa < wl ? step : 0;
            below_pack += lb <= wp ? step : 0;
        }
        if (tid < n) {
            out[tid + below_leaf] = wl;
            place[d][tid] = (uint16_t)(tid + below_leaf);
        }
        if (tid < n_pk) out[tid + below_pack] = wp;
        m = n + n_pk;
        if (tid == 0) row_size[d] = m;
        sync_rows<ONE>();
        below = out;
        W *const swap = out; out = other; other = swap;
    }
}
template <typename W>
__device__ __forceinline__ void build_rows_of(const W *lw, W *pw, W *row0, W *row1, uint32_t n, int limit, uint16_t (*place)[kCodeThreads], uint32_t *row_size)
{
    if (n <= 64) {
        if (threadIdx.x < 64) {
            if (n < 32) build_rows<W, 16, true>(lw, pw, row0, row1, n, limit, place, row_size);
            else build_rows<W, 64, true>(lw, pw, row0, row1, n, limit, place, row_size);
        }
    } else build_rows<W, 256, false>(lw, pw, row0, row1, n, limit, place, row_size);
    __syncthreads();
}

// By one wavefront, K * 64 leaves at most, a lane has the leaves lane, lane + 64, ..: 2n-2 items of the top row are taken, and of every further
// row two for each package taken of the row above it.  A leaf's code is as long as there are rows in which it is taken, the cheapest leaf's the longest.
template <int K>
__device__ __forceinline__ void walk_rows(uint32_t n, int limit, const uint16_t (*place)[kCodeThreads], const uint32_t *row_size, const uint8_t *order, uint8_t *len, uint32_t &longest)
{
    const uint32_t tid = threadIdx.x, sizes = row_size[tid];
    uint32_t p[16][K], l[K];
#pragma unroll
    for (int k = 0; k < K; k++) l[k] = 0;
#pragma unroll
    for (int d = 1; d <= 16; d++)                                // (all rows at once; those beyond the limit hold nothing that is looked at)
#pragma unroll
        for (int k = 0; k < K; k++) p[d - 1][k] = (uint32_t)place[d][k * 64 + tid];
    uint32_t budget = 2 * n - 2;
#pragma unroll
    for (int d = 1; d <= 16; d++) {
        if (d > limit || budget == 0) break;
        const uint32_t size = (uint32_t)__builtin_amdgcn_readlane((int)sizes, d), b = budget < size ? budget : size;
        uint32_t leaves = 0;
#pragma unroll
        for (int k = 0; k < K; k++) {
            const uint32_t i = (uint32_t)k * 64 + tid;
            const bool in = i < n && (d == limit ? i : p[d - 1][k]) < b;
            l[k] += in ? 1u : 0u;
            leaves += (uint32_t)__popcll(__ballot(in));
        }
        budget = 2 * (b - leaves);
    }
#pragma unroll
    for (int k = 0; k < K; k++)
        if (k * 64 + tid < n) len[order[k * 64 + tid]] = (uint8_t)l[k];
    if (tid == 0) longest = l[0];
}

}  // namespace

__global__ __launch_bounds__(kCodeThreads) void k_codes(TensorDev *descs, const uint64_t *hist, CodeParams cp, uint8_t *blobs, uint32_t *enc_tables)
{
    __shared__ __attribute__((aligned(16))) unsigned long long h[256];       // the field's histogram by symbol, then keys
    __shared__ unsigned long long lw[2 * kCodeThreads];         // leaf weights, cheapest first
    __shared__ unsigned long long row[2][kMaxRow];     // the row below and the row being merged
    __shared__ unsigned long long pw[2 * kCodeThreads];         // package weights of the row below
    __shared__ uint16_t place[17][kCodeThreads];       // per row: where every leaf lies
    __shared__ uint32_t row_size[64];
    __shared__ uint32_t wave_count[kCodeThreads / 64][17], next[17], present_in[kCodeThreads / 64];
    __shared__ uint8_t order[256], len[256];
    __shared__ unsigned long long pay_s;
    __shared__ uint32_t konst_s, lmax_s;

    const uint32_t t = blockIdx.x, f = blockIdx.y, tid = threadIdx.x;
    const uint32_t fmt = cp.fmt;
    const uint32_t grouped = (fmt == ZC_FMT_FP8_E4M3_BYTES || fmt == ZC_FMT_FP4_E2M1_MX_BYTES) ? 1u : 0u;
    const uint32_t sb = (f == 2 || grouped || fmt == ZC_FMT_FP8_E5M2 || fmt == ZC_FMT_BF16) ? 8u : fmt == ZC_FMT_FP8_E4M3 ? 4u : 2u;
    const uint32_t A = 1u << sb;
    const int limit = cp.limit[f];
    const uint64_t *hist3 = hist + (uint64_t)t * 768;

    // ---- the field's histogram
    h[tid] = 0; len[tid] = 0;
    if (tid < 64) row_size[tid] = 0;
    if (tid == 0) { pay_s = 0; konst_s = 0; lmax_s = 0; }
    lw[tid] = lw[kCodeThreads + tid] = pw[tid] = pw[kCodeThreads + tid] = ~0ull;
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
    // (every symbol is counted once; 56 bits of weight and 8 of the symbol make a key, and symbols that do not occur come last)
    const uint32_t pack = grouped ? (fmt == ZC_FMT_FP8_E4M3_BYTES ? 1u : 2u) : 0u, per_scale = fmt == ZC_FMT_FP4_E2M1_NV ? 4u : 5u;      // (as shifts)
    const uint64_t n_elems = descs[t].n_elems;
    const unsigned long long sum = f == 2 ? n_elems >> per_scale : (n_elems + (1u << pack) - 1) >> pack;
    const bool narrow = 16ull * sum < (1ull << 32);           // every weight of every row fits 32 bits
    const unsigned long long key = present ? hv << 8 | tid : ~0ull;
    {
        const uint64_t there = __ballot(present);
        if ((tid & 63) == 0) present_in[tid >> 6] = (uint32_t)__popcll(there);
    }
    __syncthreads();                                      // (h has been read)
    h[tid] = key;
    if (present) konst_s = tid;                           // (one symbol: that one)
    __syncthreads();
    const uint32_t n = present_in[0] + present_in[1] + present_in[2] + present_in[3];
    uint32_t rank = 0;
    {
        const ulonglong2 *k2 = reinterpret_cast<const ulonglong2 *>(h);
#pragma unroll 16
        for (uint32_t u = 0; u < A; u += 2) {
            const ulonglong2 q = k2[u / 2];
            rank += (q.x < key ? 1u : 0u) + (q.y < key ? 1u : 0u);
        }
    }
    // weights of 32 bits lie in the first half of lw and pw, whose other half stays the padding
    uint32_t *const lw32 = reinterpret_cast<uint32_t *>(lw), *const pw32 = reinterpret_cast<uint32_t *>(pw);
    if (present) {
        if (narrow) lw32[rank] = (uint32_t)hv;
        else lw[rank] = hv;
        order[rank] = (uint8_t)tid;
    }
    __syncthreads();

    uint32_t mode = ZC_MODE_EMPTY, konst = 0, lmax = 0;
    if (n == 1) { mode = ZC_MODE_CONST; konst = konst_s; }
    else if (n > 1) {
        mode = ZC_MODE_HUFF;
        // ---- rows limit-1 .. 1
        if (narrow) build_rows_of<uint32_t>(lw32, pw32, reinterpret_cast<uint32_t *>(row[0]), reinterpret_cast<uint32_t *>(row[1]), n, limit, place, row_size);
        else build_rows_of<unsigned long long>(lw, pw, row[0], row[1], n, limit, place, row_size);
        // ---- walk the budget down from the top row, by one wavefront
        if (tid < 64) {
            if (n <= 64) walk_rows<1>(n, limit, place, row_size, order, len, lmax_s);
            else walk_rows<4>(n, limit, place, row_size, order, len, lmax_s);
            if (cp.policy == ZC_POLICY_AUTO) {
                unsigned long long pay = 0;
                for (uint32_t i = tid; i < n; i += 64) pay += (narrow ? (unsigned long long)lw32[i] : lw[i]) * len[order[i]];
                pay = wave_sum(pay);
                if (tid == 0) pay_s = pay;
            }
        }
        __syncthreads();
        lmax = lmax_s;
        // Sec. 3.1: a field that does not compress is stored as is
        if (cp.policy == ZC_POLICY_AUTO && 16ull * pay_s > 15ull * sum * sb) { mode = ZC_MODE_RAW; lmax = 0; }
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
    __syncthreads();
    if (tid < 64) {
        // the first code of length l is the sum over the shorter lengths j of count(j) * 2^(l - j): a scan of count(j) * 2^(16 - j)
        const uint32_t l = tid;
        uint32_t x = 0;
        if (l >= 1 && l <= 16) x = (wave_count[0][l] + wave_count[1][l] + wave_count[2][l] + wave_count[3][l]) << (16 - l);
        const uint32_t own = x;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (tid >= (uint32_t)o) x += y;
        }
        if (l >= 1 && l <= 16) next[l] = (x - own) >> (16 - l);
    }
    __syncthreads();
    const uint32_t flat = wave_count[0][sb] + wave_count[1][sb] + wave_count[2][sb] + wave_count[3][sb];       // symbols with a code of the plain length
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
        const uint32_t kind = mode == ZC_MODE_RAW ? 2u : mode != ZC_MODE_HUFF ? 3u : flat == A ? 1u : 0u;
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

// Histograms of fields of few values (FP8 E4M3: 16 and 16, E5M2: 32 and 8, FP4: 4 and 4), counted in bit planes instead of by
// additions to LDS (a3), and for 64 lanes and chunks of one histogram block the counts per chunk lane from which
// k_sizes_fp8_counts and k_sizes_e5m2_counts work.
//
// A byte histogram in LDS takes one atomic addition per byte and wavefront, eight cycles of the compute unit's LDS each, whatever the data:
// 5.0 TB/s for the whole card, which is what bounded these passes.  Here a thread takes eight words (32 bytes) at a time, turns them
// into their eight bit planes (48 instructions: three rounds of exchanging halves between pairs of words; a plane's bit is one
// byte's bit), and counts, for every set of a field's planes, in how many bytes all of them are set (one AND and one
// v_bcnt_u32_b32 per set, which adds to its count: 26 instructions for four planes).  The counts of the values follow from those of
// the sets once, at the end: a value's own count is what its set has minus what sets with more planes have.  100 instructions per 32 bytes
// (E5M2 116, FP4 64) are 12 TB/s for the card, so these passes stand at the speed of their reads; zeros count nothing, so that what
// lies beyond the end of a tensor needs no test.
//
// The counts go to the tensor's bins by atomic additions, which take their turns per cache line at the memory side: workgroups
// are spread over several copies of the bins (hist_copies), which whoever reads them adds up.
#include <hip/hip_runtime.h>

#include "zc_internal.h"
#include "zc_device.h"
#include "zc_encode_device.h"

namespace zc {

namespace {

constexpr int kNt = 2;                     // cache policy of loads: non-temporal

// planes of the exponent and the sign+mantissa field, lowest bit of the symbol first; BYTE: one element per byte (else two)
template <int FMT> struct Planes;
template <> struct Planes<ZC_FMT_FP8_E4M3> { static constexpr int PE = 4, PM = 4; static constexpr bool BYTE = true; static constexpr int E[4] = {3, 4, 5, 6}, M[4] = {0, 1, 2, 7}; };
template <> struct Planes<ZC_FMT_FP8_E5M2> { static constexpr int PE = 5, PM = 3; static constexpr bool BYTE = true; static constexpr int E[5] = {2, 3, 4, 5, 6}, M[3] = {0, 1, 7}; };
template <> struct Planes<ZC_FMT_FP4_E2M1_MX> { static constexpr int PE = 2, PM = 2; static constexpr bool BYTE = false; static constexpr int E[2] = {1, 2}, M[2] = {0, 3}; };

// (mask & x) | (~mask & y) in one instruction (the compiler makes two of most of these)
__device__ __forceinline__ uint32_t pick(uint32_t mask, uint32_t x, uint32_t y)
{
    uint32_t r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "s"(mask), "v"(x), "v"(y));
    return r;
}

// eight words -> eight bit planes
template <int S>
__device__ __forceinline__ void exchange_bits(uint32_t (&w)[8])
{
    constexpr uint32_t m = S == 4 ? 0x0F0F0F0Fu : S == 2 ? 0x33333333u : 0x55555555u;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int i = k % S + k / S * 2 * S;                     // the four words whose number lacks the bit S
        const uint32_t a = w[i], b = w[i + S];
        w[i] = pick(m, a, b << S);
        w[i + S] = pick(m, a >> S, b);
    }
}
__device__ __forceinline__ void to_planes(uint32_t (&w)[8]) { exchange_bits<4>(w); exchange_bits<2>(w); exchange_bits<1>(w); }

// c[s] += bits set in all the planes of the set s, for every set but the empty one
template <int P>
__device__ __forceinline__ void count_sets(const uint32_t (&p)[P], uint32_t (&c)[1 << P])
{
    uint32_t all[1 << P];
#pragma unroll
    for (int s = 1; s < 1 << P; s++) {
        const int low = __builtin_ctz(s), rest = s & (s - 1);
        all[s] = rest ? all[rest] & p[low] : p[low];
        c[s] += (uint32_t)__popc(all[s]);
    }
}

// counts of sets -> counts of values; c[0] is the number of symbols on the way in
template <int P>
__device__ __forceinline__ void sets_to_values(uint32_t (&c)[1 << P])
{
#pragma unroll
    for (int i = 0; i < P << (P - 1); i++) {
        const int b = i >> (P - 1), k = i & ((1 << (P - 1)) - 1), v = (k >> b << (b + 1)) | (k & ((1 << b) - 1));       // the values without bit b
        c[v] -= c[v | 1 << b];
    }
}

template <int FMT>
struct FieldCounts {
    using P = Planes<FMT>;
    static constexpr int NE = 1 << P::PE, NM = 1 << P::PM;
    uint32_t e[NE], m[NM];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < NE; i++) e[i] = 0;
#pragma unroll
        for (int i = 0; i < NM; i++) m[i] = 0;
    }
    __device__ __forceinline__ void add(const u32x4 &x, const u32x4 &y)
    {
        uint32_t w[8] = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
        to_planes(w);
#pragma unroll
        for (int h = 0; h < (P::BYTE ? 1 : 2); h++) {
            uint32_t pe[P::PE], pm[P::PM];
#pragma unroll
            for (int i = 0; i < P::PE; i++) pe[i] = w[P::E[i] + 4 * h];
#pragma unroll
            for (int i = 0; i < P::PM; i++) pm[i] = w[P::M[i] + 4 * h];
            count_sets<P::PE>(pe, e);
            count_sets<P::PM>(pm, m);
        }
        __builtin_amdgcn_sched_barrier(0);                       // (side by side two of these would take the registers of a wavefront or two)
    }
    // symbols: how many this thread has counted (modulo 2^32, as the counts then are)
    __device__ __forceinline__ void finish(uint32_t symbols)
    {
        e[0] = symbols; m[0] = symbols;
        sets_to_values<P::PE>(e);
        sets_to_values<P::PM>(m);
    }
};

// Sums of c[0..N) over the wavefront, in a butterfly that halves what a lane carries at every step: lane j < N ends with (and returns) the
// sum of c[value_of_lane<N>(j)]; the others with copies.
template <int N, int STEP = 0>
__device__ __forceinline__ uint32_t sum_over_wave(uint32_t (&c)[N])
{
    constexpr int n = N >> (STEP + 1);
    if constexpr (n > 0) {
        const uint32_t upper = 0u - ((threadIdx.x >> STEP) & 1u);        // all ones in the lanes that keep the upper half
#pragma unroll
        for (int i = 0; i < n; i++) {
            // (bitwise, so that the counts stay in registers)
            const uint32_t a = c[i], b = c[n + i], d = (a ^ b) & upper;
            c[i] = (a ^ d) + (uint32_t)__shfl_xor((int)(b ^ d), 1 << STEP, 64);          // keeps b, gives a where upper
        }
        return sum_over_wave<N, STEP + 1>(c);
    } else {
#pragma unroll
        for (int o = N; o < 64; o <<= 1) c[0] += (uint32_t)__shfl_xor((int)c[0], o, 64);
        return c[0];
    }
}
template <int N>
__device__ __forceinline__ uint32_t value_of_lane(uint32_t lane) { return __brev(lane & (N - 1)) >> (32 - __builtin_ctz(N)); }

// The workgroup's counts into a copy of the tensor's bins.  sums: 4 * (NE + NM) words of LDS.  symbols: what value 0 has besides (the threads
// finished with none).
template <int FMT>
__device__ __forceinline__ void add_to_bins(FieldCounts<FMT> &c, uint32_t *sums, uint32_t symbols, uint64_t *bins)
{
    constexpr int NE = FieldCounts<FMT>::NE, NM = FieldCounts<FMT>::NM, N = NE + NM;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t se = sum_over_wave<NE>(c.e), sm = sum_over_wave<NM>(c.m);
    if (lane < NE) sums[wave * N + value_of_lane<NE>(lane)] = se;
    if (lane < NM) sums[wave * N + NE + value_of_lane<NM>(lane)] = sm;
    __syncthreads();
    if (tid < N) {
        const uint32_t v = tid < NE ? tid : tid - NE;
        const uint32_t n = sums[tid] + sums[N + tid] + sums[2 * N + tid] + sums[3 * N + tid] + (v == 0 ? symbols : 0u);
        if (n) atomicAdd(reinterpret_cast<unsigned long long *>(bins + (tid < NE ? tid : hist_second_field(FMT) + v)), (unsigned long long)n);
    }
}

// The copy of a tensor's bins that this workgroup adds to
template <int FMT>
__device__ __forceinline__ uint64_t *bins_of(uint64_t *hist, uint32_t tensor) { return hist + (uint64_t)tensor * 768 + (blockIdx.x % hist_copies(FMT)) * hist_copy_stride(FMT); }

}  // namespace

// One workgroup per part of a histogram block of one tensor: rounds of four 4 KiB rows, the next round's loads in flight while one is
// counted.  FP4: the first scale_groups workgroups count the scale bytes (256 values: LDS, one copy of the bins per bank as in k_hist)
// of the other list, in the same launch.
template <int FMT, bool DELTA, int NT>
__global__ __launch_bounds__(256) void k_hist_planes(const TensorDev *descs, const WorkItem *work, uint32_t split, uint64_t *hist, const WorkItem *scale_work,
                                                     uint32_t scale_groups, uint32_t scale_split, uint32_t per_scale)
{
    using C = FieldCounts<FMT>;
    constexpr bool SCALES = !Planes<FMT>::BYTE;
    __shared__ uint32_t lds[SCALES ? 256 * 32 : 4 * (C::NE + C::NM)];
    const uint32_t tid = threadIdx.x;
    if (SCALES && blockIdx.x < scale_groups) {
        const WorkItem it = scale_work[blockIdx.x / scale_split];
        const TensorDev &d = descs[it.tensor];
        const uint32_t part = kHistBlockBytes / scale_split;
        const uint64_t n = d.n_elems / per_scale, start = (uint64_t)it.first * kHistBlockBytes + (uint64_t)(blockIdx.x % scale_split) * part;
        if (start >= n) return;
        const uint64_t end = start + part < n ? start + part : n;
        for (uint32_t i = tid; i < 256 * 32; i += 256) lds[i] = 0;
        __syncthreads();
        uint32_t *const mine = lds + (tid & 31);
        for (uint64_t off = start + tid * 16; off < end; off += 256 * 16) {
            const uint32_t valid = end - off >= 16 ? 16u : (uint32_t)(end - off);
            const uint4 v = load_run(d.scales + off, valid);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 16; i++)
                if ((uint32_t)i < valid) atomicAdd(mine + ((w[i >> 2] >> (8 * (i & 3))) & 0xFFu) * 32, 1u);
        }
        __syncthreads();
        uint32_t sum = 0;
#pragma unroll 8
        for (uint32_t r = 0; r < 32; r++) sum += lds[tid * 32 + ((r + tid) & 31)];
        if (sum) atomicAdd(reinterpret_cast<unsigned long long *>(&hist[(uint64_t)it.tensor * 768 + 512 + tid]), (unsigned long long)sum);
        return;
    }
    const uint32_t group = blockIdx.x - (SCALES ? scale_groups : 0);
    const WorkItem it = work[group / split];
    const TensorDev &d = descs[it.tensor];
    const uint32_t part = kHistBlockBytes / split;
    const uint64_t nbytes = Planes<FMT>::BYTE ? d.n_elems : (d.n_elems + 1) / 2, start = (uint64_t)it.first * kHistBlockBytes + (uint64_t)(group % split) * part;
    if (start >= nbytes) return;                                 // whole workgroup: the block ends before this part
    const uint32_t len = nbytes - start < part ? (uint32_t)(nbytes - start) : part, whole = len & ~15u;
    const uint8_t *src_at = reinterpret_cast<const uint8_t *>(uni64((uint64_t)(d.src + start)));
    const uint8_t *base_at = DELTA ? reinterpret_cast<const uint8_t *>(uni64((uint64_t)(d.base ? d.base + start : nullptr))) : nullptr;
    const __amdgpu_buffer_rsrc_t src = rsrc_of(src_at, uni32(whole)), bas = rsrc_of(base_at, DELTA && base_at ? uni32(whole) : 0u);
    constexpr int K = 4;
    struct Round { u32x4 x[K], y[DELTA ? K : 1]; } a, b;
    auto fetch = [&](uint32_t round, Round &r) {                 // (zeros beyond the end)
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int at = (int)((round * K + k) * 4096 + tid * 16);
            r.x[k] = __builtin_amdgcn_raw_buffer_load_b128(src, at, 0, NT);
            if (DELTA) r.y[k] = __builtin_amdgcn_raw_buffer_load_b128(bas, at, 0, NT);
        }
    };
    C c;
    c.clear();
    auto count = [&](const Round &r) {
#pragma unroll
        for (int k = 0; k < K; k += 2) {
            if (DELTA) c.add(r.x[k] ^ r.y[k], r.x[k + 1] ^ r.y[k + 1]);
            else c.add(r.x[k], r.x[k + 1]);
        }
    };
    const uint32_t rounds = (whole + K * 4096 - 1) / (K * 4096);
    fetch(0, a);
    for (uint32_t i = 0; i < rounds; i += 2) {
        fetch(i + 1, b);
        count(a);
        fetch(i + 2, a);
        count(b);
    }
    if (len != whole && tid == 0) {                              // the last, partial run
        uint4 v = load_run(src_at + whole, len - whole);
        if (DELTA && base_at) v = xor4(v, load_run(base_at + whole, len - whole));
        c.add(u32x4{v.x, v.y, v.z, v.w}, u32x4{0, 0, 0, 0});
    }
    c.finish(0);
    add_to_bins<FMT>(c, lds, Planes<FMT>::BYTE ? len : 2 * len, bins_of<FMT>(hist, it.tensor));
}

// The same for 64 lanes and chunks of kHistBlockBytes, one workgroup per whole chunk (the host uses this kernel for no other): thread t
// takes the runs t, t + 256, ...: all of chunk lane t % 64, which it shares with three threads of the other wavefronts.  The four
// threads' counts, added up in LDS two to a word (a lane holds 4,096 bytes), are the lane's: E4M3 16 exponent counts of 16 bits (2 KiB per
// chunk), E5M2 32 exponent and 8 sign+mantissa counts (5 KiB).  1.96 GB of FP8: 402 us
// with the counts in LDS, 386 here, 310 = 6.3 TB/s with non-temporal loads and the chunks in their natural order (the XCDs' order keeps eight times as
// many DRAM pages open: a bare read of 2 GiB in parts of 256 KiB goes at 5.7 - 5.9 TB/s in that order, at 6.5 with the hint, at 7.0 with the hint in natural order).
template <int FMT, bool DELTA>
__global__ __launch_bounds__(256) void k_hist_fp8_lanes(const TensorDev *descs, const WorkItem *work, uint64_t *hist, uint16_t *lane_counts)
{
    using C = FieldCounts<FMT>;
    constexpr bool E5M2 = FMT == ZC_FMT_FP8_E5M2;
    constexpr uint32_t kWords = E5M2 ? 20 : 8, kMine = kWords / 4;       // words per lane, and per thread on the way out
    static_assert(kHistBlockBytes / 64 < 65536, "a lane's count of one value fits 16 bits");
    __shared__ uint32_t sums[4 * (C::NE + C::NM)];
    __shared__ uint32_t part[4 * kWords * 64];
    const WorkItem it = work[blockIdx.x];
    const TensorDev &d = descs[it.tensor];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t start = (uint64_t)it.first * kHistBlockBytes;
    if (d.chunk_bytes != kHistBlockBytes || start + kHistBlockBytes > d.n_elems) return;      // whole workgroup; the host never asks for this
    const __amdgpu_buffer_rsrc_t src = rsrc_of(reinterpret_cast<const uint8_t *>(uni64((uint64_t)(d.src + start))), kHistBlockBytes);
    const bool has_base = DELTA && d.base;
    const __amdgpu_buffer_rsrc_t bas = rsrc_of(reinterpret_cast<const uint8_t *>(uni64((uint64_t)(has_base ? d.base + start : nullptr))), has_base ? kHistBlockBytes : 0u);
    constexpr int K = 4;
    struct Round { u32x4 x[K], y[DELTA ? K : 1]; } a, b;
    auto fetch = [&](uint32_t round, Round &r) {                 // (zeros beyond the end)
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int at = (int)((round * K + k) * 4096 + tid * 16);
            r.x[k] = __builtin_amdgcn_raw_buffer_load_b128(src, at, 0, kNt);
            if (DELTA) r.y[k] = __builtin_amdgcn_raw_buffer_load_b128(bas, at, 0, kNt);
        }
    };
    C c;
    c.clear();
    auto count = [&](const Round &r) {
#pragma unroll
        for (int k = 0; k < K; k += 2) {
            if (DELTA) c.add(r.x[k] ^ r.y[k], r.x[k + 1] ^ r.y[k + 1]);
            else c.add(r.x[k], r.x[k + 1]);
        }
    };
    constexpr uint32_t kRounds = kHistBlockBytes / (K * 4096);
    static_assert(kRounds % 2 == 0, "rounds in pairs");
    fetch(0, a);
    for (uint32_t i = 0; i < kRounds; i += 2) {
        fetch(i + 1, b);
        count(a);
        fetch(i + 2, a);
        count(b);
    }
    c.finish(kHistBlockBytes / 256);
#pragma unroll
    for (int j = 0; j < C::NE / 2; j++) part[(wave * kWords + j) * 64 + lane] = c.e[2 * j] | (c.e[2 * j + 1] << 16);
    if (E5M2)
#pragma unroll
        for (int j = 0; j < 4; j++) part[(wave * kWords + 16 + j) * 64 + lane] = c.m[2 * j] | (c.m[2 * j + 1] << 16);
    add_to_bins<FMT>(c, sums, 0, bins_of<FMT>(hist, it.tensor));         // (its barrier is that of `part` too)
    const uint64_t chunk_global = (uint64_t)(d.units_off / 2) + it.first;      // two fields: units_off counts two entries per chunk
    uint32_t *out = reinterpret_cast<uint32_t *>(lane_counts + (chunk_global * 64 + lane) * (2 * kWords)) + wave * kMine;
    uint32_t w[kMine];
#pragma unroll
    for (uint32_t j = 0; j < kMine; j++) {
        const uint32_t *p = part + (wave * kMine + j) * 64 + lane;
        w[j] = p[0] + p[kWords * 64] + p[2 * kWords * 64] + p[3 * kWords * 64];
    }
    if (!E5M2) *reinterpret_cast<uint2 *>(out) = make_uint2(w[0], w[1]);
    else
#pragma unroll
        for (uint32_t j = 0; j < kMine; j++) out[j] = w[j];
}

// FP8 E4M3 pages (fewer than 64 lanes per chunk, page_counts_shape): a thread takes a whole (page, lane) pair at a time, so that its counts are
// the pair's: 16 counts of 8 bits (255 stands for 256, all a pair can hold, as no other pair of counts adds up to one less than it should) and the
// exponents of its last four symbols, from which k_sizes_pages works in place of a second read of the source: 18 bytes where the size pass
// read 256.  2.15 GB of pages of 2 KiB: 407 us against 319 without the pairs' counts (the loads of a wavefront lie in eight pages), and 33 us for the sizes
// against 366 - 419 for a pass over the source.
template <bool DELTA, int NT>
__global__ __launch_bounds__(256) void k_hist_pages(const TensorDev *descs, const WorkItem *work, uint32_t split, uint64_t *hist, u32x4 *counts, uint16_t *lasts)
{
    constexpr int FMT = ZC_FMT_FP8_E4M3;
    using C = FieldCounts<FMT>;
    __shared__ uint32_t sums[4 * (C::NE + C::NM)];
    const uint32_t tid = threadIdx.x;
    const WorkItem it = work[blockIdx.x / split];
    const TensorDev &d = descs[it.tensor];
    const uint32_t cb = uni32(d.chunk_bytes), S = uni32(d.streams), rows = cb / (16 * S), part = kHistBlockBytes / split;
    const uint64_t n = d.n_elems, n_pages = n / cb, paged = n_pages * cb, start = (uint64_t)it.first * kHistBlockBytes + (uint64_t)(blockIdx.x % split) * part;
    if (start >= n) return;                                      // whole workgroup: the block ends before this part
    const uint32_t whole = start >= paged ? 0u : paged - start < part ? (uint32_t)(paged - start) : part;      // (whole pages: a part is whole passes)
    const uint8_t *src_at = reinterpret_cast<const uint8_t *>(uni64((uint64_t)(d.src + start)));
    const uint8_t *base_at = DELTA ? reinterpret_cast<const uint8_t *>(uni64((uint64_t)(d.base ? d.base + start : nullptr))) : nullptr;
    const __amdgpu_buffer_rsrc_t src = rsrc_of(src_at, uni32(whole)), bas = rsrc_of(base_at, DELTA && base_at ? uni32(whole) : 0u);
    const uint32_t lane = tid & (S - 1), page = tid / S;         // (S is a power of two)
    const uint32_t pass_bytes = 4096 * rows, per_pass = (rows + 3) / 4;       // of 256 pairs; rounds of four rows
    constexpr int K = 4;
    struct Round { u32x4 x[K], y[DELTA ? K : 1]; } a, b;
    uint32_t f_at = page * cb + lane * 16, f_row = 0;            // where the next round is fetched from
    auto fetch = [&](Round &r) {                                 // (zeros beyond the end)
#pragma unroll
        for (int k = 0; k < K; k++) {
            const int at = (int)(f_row + k < rows ? f_at + (f_row + k) * 16 * S : 0xFFFFFFF0u);
            r.x[k] = __builtin_amdgcn_raw_buffer_load_b128(src, at, 0, NT);
            if (DELTA) r.y[k] = __builtin_amdgcn_raw_buffer_load_b128(bas, at, 0, NT);
        }
        f_row += K;
        if (f_row >= rows) { f_row = 0; f_at += pass_bytes; }
    };
    C c;
    c.clear();
    uint32_t all[C::NE];                                         // the exponents' counts (by sets) over all pages so far
#pragma unroll
    for (int i = 0; i < C::NE; i++) all[i] = 0;
    const uint64_t first_pair = ((uint64_t)(d.units_off / 2) + start / cb) * S;      // two fields: units_off counts two entries per chunk
    uint32_t row = 0, pair = tid;
    auto count = [&](const Round &r) {
        u32x4 x[K];
#pragma unroll
        for (int k = 0; k < K; k++) x[k] = DELTA ? r.x[k] ^ r.y[k] : r.x[k];
#pragma unroll
        for (int k = 0; k < K; k += 2) c.add(x[k], x[k + 1]);
        row += K;
        if (row < rows) return;
        // the pair is through: its counts, and the last word of its last row
        uint32_t v[C::NE];
#pragma unroll
        for (int i = 1; i < C::NE; i++) { v[i] = c.e[i]; all[i] += c.e[i]; c.e[i] = 0; }
        v[0] = rows * 16;
        sets_to_values<Planes<FMT>::PE>(v);
        const uint32_t left = rows + K - row, w = left == 1 ? x[0][3] : left == 2 ? x[1][3] : left == 3 ? x[2][3] : x[3][3];
        if (pair * 16 * rows < whole) {
            u32x4 packed;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                uint32_t q[4];
#pragma unroll
                for (int j = 0; j < 4; j++) q[j] = v[4 * i + j] > 255 ? 255u : v[4 * i + j];
                packed[i] = q[0] | q[1] << 8 | q[2] << 16 | q[3] << 24;
            }
            counts[first_pair + pair] = packed;
            const uint32_t e = (w >> 3) & 0x0F0F0F0Fu, t = e | e >> 4;
            lasts[first_pair + pair] = (uint16_t)((t & 0xFFu) | (t >> 8 & 0xFF00u));
        }
        row = 0;
        pair += 256;
    };
    const uint32_t rounds = (whole + pass_bytes - 1) / pass_bytes * per_pass;
    fetch(a);
    for (uint32_t i = 0; i < rounds; i += 2) {
        fetch(b);
        count(a);
        fetch(a);
        if (i + 1 < rounds) count(b);
    }
#pragma unroll
    for (int i = 1; i < C::NE; i++) c.e[i] = all[i];
    // what is left of the tensor behind its whole pages: less than a page, at most 8 KiB
    uint32_t rest = 0;
    if (paged >= start && paged < start + part && paged < n) {
        rest = (uint32_t)(n - paged);
        for (uint32_t at = tid * 32; at < rest; at += 256 * 32) {
            uint4 v[2] = {make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0)};
#pragma unroll
            for (uint32_t k = 0; k < 2; k++)
                if (at + 16 * k < rest) {
                    v[k] = load_run(src_at + whole + at + 16 * k, rest - at - 16 * k);
                    if (DELTA && base_at) v[k] = xor4(v[k], load_run(base_at + whole + at + 16 * k, rest - at - 16 * k));
                }
            c.add(u32x4{v[0].x, v[0].y, v[0].z, v[0].w}, u32x4{v[1].x, v[1].y, v[1].z, v[1].w});
        }
    }
    c.finish(0);
    add_to_bins<FMT>(c, sums, whole + rest, bins_of<FMT>(hist, it.tensor));
}

// Stream sizes of whole FP8 pages from those counts, for tensors the page kernels take (route 1): a lane's words are min(steps,
// floor((bits - bits of its last four codes) / 32) + 2) as in k_sizes_fp8_counts, its bits the counts times the code lengths, four products to an
// instruction.  Work items of the page kernels.
__global__ __launch_bounds__(256) void k_sizes_pages(const TensorDev *descs, const WorkItem *work, const uint32_t *enc_tables, const u32x4 *counts, const uint16_t *lasts,
                                                     uint32_t *units, uint32_t slots_per_group)
{
    __shared__ uint32_t len16[16];
    const WorkItem it = work[blockIdx.x];
    const TensorDev *dp = descs + it.tensor;
    if (dp->route != 1) return;                                  // whole workgroup: not the page kernels' tensor
    if (threadIdx.x < 16) len16[threadIdx.x] = enc_tables[(uint64_t)it.tensor * 768 + threadIdx.x] >> 16;
    __syncthreads();
    const uint32_t cb = uni32(dp->chunk_bytes), S = uni32(dp->streams), symbols = cb / S, steps = symbols / 4, nc = uni32(dp->n_chunks);
    const uint32_t n_full = (uint32_t)(uni64(dp->n_elems) / cb), first = it.first;
    uint32_t lens[4];
    uint64_t nibbles = 0;                                        // (lengths of at most 8)
#pragma unroll
    for (int i = 0; i < 4; i++) {
        lens[i] = len16[4 * i] | len16[4 * i + 1] << 8 | len16[4 * i + 2] << 16 | len16[4 * i + 3] << 24;
#pragma unroll
        for (int j = 0; j < 4; j++) nibbles |= (uint64_t)len16[4 * i + j] << (4 * (4 * i + j));
    }
    const uint64_t pair0 = ((uint64_t)(uni32(dp->units_off) / 2) + first) * S;
    uint32_t *my = units + uni32(dp->units_off);
    for (uint32_t i = threadIdx.x; i < slots_per_group * S; i += 256) {        // (whole wavefronts: slots come in multiples of 64 / S)
        const uint32_t chunk = first + i / S;
        const bool alive = chunk < n_full;
        uint32_t q = 0;
        if (alive) {
            const u32x4 c = counts[pair0 + i];
            const uint32_t last = lasts[pair0 + i];
            uint32_t sum = 0, bits = 0;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                sum = __builtin_amdgcn_udot4(c[j], 0x01010101u, sum, false);
                bits = __builtin_amdgcn_udot4(c[j], lens[j], bits, false);
            }
            if (sum != symbols) bits += bits / 255;              // one value in all 256 places
            uint32_t tail = 0;
#pragma unroll
            for (int j = 0; j < 4; j++) tail += (uint32_t)(nibbles >> (4 * ((last >> (4 * j)) & 15u))) & 15u;
            q = ((bits - tail) >> 5) + 2;
            q = q < steps ? q : steps;
        }
        for (uint32_t o = S / 2; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
        if (alive && (i & (S - 1)) == 0) {
            my[chunk] = (q + 3) / 4;
            my[nc + chunk] = cb / 32;                            // 4 bits per element, 16-byte units (flat code and raw alike)
        }
    }
}

int launch_hist_fp8_lanes(bool e5m2, bool delta, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work, uint64_t *d_hist, uint16_t *d_lane_counts, void *stream)
{
    if (n_work == 0) return 0;
    hipStream_t st = (hipStream_t)stream;
#define ZC_LANES(F, D) hipLaunchKernelGGL((k_hist_fp8_lanes<F, D>), dim3(n_work), dim3(256), 0, st, d_descs, d_work, d_hist, d_lane_counts)
    if (e5m2) { if (delta) ZC_LANES(ZC_FMT_FP8_E5M2, true); else ZC_LANES(ZC_FMT_FP8_E5M2, false); }
    else { if (delta) ZC_LANES(ZC_FMT_FP8_E4M3, true); else ZC_LANES(ZC_FMT_FP8_E4M3, false); }
#undef ZC_LANES
    return (int)hipGetLastError();
}

// Parts per block: as many as it takes for some two thousand workgroups (a compute unit holds five or so), rounds permitting.
static uint32_t parts_of(uint32_t n_work, uint32_t most)
{
    uint32_t split = 1;
    while (split < most && (uint64_t)n_work * split < 1536) split *= 2;
    return split;
}

int launch_hist_pages(bool delta, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work, uint32_t pass_bytes, uint64_t *d_hist, uint8_t *d_counts, uint8_t *d_lasts,
                      void *stream)
{
    if (n_work == 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    const uint32_t split = parts_of(n_work, kHistBlockBytes / pass_bytes);
    // Non-temporal loads as in launch_hist_planes.  Whole calls over pages of 2 KiB, 8 lanes, without | with the hint, us: 512 blocks 136 | 145, 900 256 | 255,
    // 1,100 315 | 312, 2,000 586 | 568, 6,000 1,695 | 1,654; of 4 KiB, 16 lanes: 512 126 | 135, 1,024 236 | 241, 1,300 317 | 309, 3,000 723 | 696.
    const bool once = n_work > 1024;
#define ZC_PAGES(D, N) hipLaunchKernelGGL((k_hist_pages<D, N>), dim3(n_work * split), dim3(256), 0, st, d_descs, d_work, split, d_hist, (u32x4 *)d_counts, (uint16_t *)d_lasts)
    if (delta) { if (once) ZC_PAGES(true, kNt); else ZC_PAGES(true, 0); }
    else { if (once) ZC_PAGES(false, kNt); else ZC_PAGES(false, 0); }
#undef ZC_PAGES
    return (int)hipGetLastError();
}

int launch_sizes_pages(const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work, const uint32_t *d_enc, const uint8_t *d_counts, const uint8_t *d_lasts,
                       uint32_t *d_units, uint32_t slots_per_group, void *stream)
{
    if (n_work == 0) return 0;
    hipLaunchKernelGGL(k_sizes_pages, dim3(n_work), dim3(256), 0, (hipStream_t)stream, d_descs, d_work, d_enc, (const u32x4 *)d_counts, (const uint16_t *)d_lasts, d_units, slots_per_group);
    return (int)hipGetLastError();
}

int launch_hist_planes(uint32_t fmt, bool delta, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work, const WorkItem *d_scale_work, uint32_t n_scale,
                       uint64_t *d_hist, void *stream)
{
    if (n_work == 0 && n_scale == 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    const uint32_t split = parts_of(n_work, kHistBlockBytes / 16384), scale_split = parts_of(n_scale, 8), scale_groups = n_scale * scale_split;
    const dim3 grid(n_work * split + scale_groups);
    // Non-temporal loads where the elements are more than the 256 MB that the memory-side cache holds: 2.15 GB of pages 411 -> 319 us.  Fewer are
    // partly found in the caches by the size pass and the encoder (seven FP8 tensors of 135 MB, whole call: 186 us with the hint, 181 without).
    const bool once = n_work > 1024;
    const uint32_t per_scale = scale_block(fmt) ? scale_block(fmt) : 1;
#define ZC_PLANES(F, D) \
    if (once) hipLaunchKernelGGL((k_hist_planes<F, D, kNt>), grid, dim3(256), 0, st, d_descs, d_work, split, d_hist, d_scale_work, scale_groups, scale_split, per_scale); \
    else hipLaunchKernelGGL((k_hist_planes<F, D, 0>), grid, dim3(256), 0, st, d_descs, d_work, split, d_hist, d_scale_work, scale_groups, scale_split, per_scale)
#define ZC_PLANES2(F) if (delta) { ZC_PLANES(F, true); } else { ZC_PLANES(F, false); } break
    switch (fmt) {
    case ZC_FMT_FP8_E4M3: ZC_PLANES2(ZC_FMT_FP8_E4M3);
    case ZC_FMT_FP8_E5M2: ZC_PLANES2(ZC_FMT_FP8_E5M2);
    case ZC_FMT_FP4_E2M1_MX:
    case ZC_FMT_FP4_E2M1_NV: ZC_PLANES2(ZC_FMT_FP4_E2M1_MX);     // the same elements
    default: return 1;
    }
#undef ZC_PLANES2
#undef ZC_PLANES
    return (int)hipGetLastError();
}

}  // namespace zc

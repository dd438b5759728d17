// 64-lane decoders with large lookup tables (a8, a9): BF16, FP8 (E4M3, E5M2, byte symbols); any chunks, a short last one and
// lists of chunk ids included; exponent field table decoded with a refill period of 2, 4 or 8, sign+mantissa field table decoded
// on the same period or stored plainly (flat code, raw, constant; E5M2: its flat 3-bit code).  The kernel, for zc_decode_pairs*.hip, which
// have its builds by format (each takes minutes to compile).
//
// A chunk is one wavefront's serial chain: window, lookups, refill (whose word depends on how many lanes take one), window; a call of
// few chunks takes as long as one chunk's chain.  A wavefront alone on its SIMD issues an instruction every 4 cycles and waits 55 for an
// LDS read, 16 where a scalar instruction reads a mask just written by a vector one, 30 for a branch taken: what a period takes is
// its instructions, with the waits beside them.  So
//   - calls of one round of workgroups have tables by 16 bits, in 128 of a compute unit's 160 KiB of LDS: every code fits, no
//     lookup has to be checked, and FP8 E4M3 exponents (codes of at most 8 bits) come in pairs; or pairs by 15 bits, for other exponents with
//     such codes.  In the others the tables are small: exponents in pairs by 12 or 13 bits, which halves the lookups, other symbols by 12
//     bits, and what does not resolve sends the wavefront through the period once more.
//   - in calls of one round a period does not wait for the words asked for before it (late_run), and a row is put together and stored
//     while the next one's entries are looked up.
//   - two table-decoded fields go through the chain side by side.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "zc_internal.h"
#include "zc_device.h"
#include "zc_decode_device.h"

namespace zc {

// What a launch is for: calls of one round of workgroups (kFew; kFewTwo: some tensor's sign+mantissa field is table decoded too), whose
// workgroups have a compute unit to themselves, with tables of up to 136 KiB; all others; of those, two fields and up to 256 workgroups (a
// kernel of its own: it takes 20 registers more).
enum Launch { kFew, kFewTwo, kMany, kManyTwo };

// builds by format: zc_decode_pairs_bf16.hip, zc_decode_pairs_bytes.hip
int launch_pairs_bf16(bool two, bool xor_delta, uint32_t chunks, bool long_rings, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work,
                      const TensorDev &s, int use_single, uint32_t first_slot, hipStream_t st);
int launch_pairs_bytes(bool two, bool xor_delta, uint32_t chunks, bool long_rings, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work,
                       const TensorDev &s, int use_single, uint32_t first_slot, hipStream_t st);

namespace {

// canonical code of a field: limit[l] = left-aligned (16 bits) exclusive upper bound of the codes of length <= l, rebase[l] =
// rank of the first code of length l minus that code, sorted = symbols in (length, symbol) order
struct PairCanon { uint32_t limit[17], rebase[17]; uint8_t sorted[256]; };

template <int B> __device__ __forceinline__ uint32_t add_byte(uint32_t a, uint32_t b)       // a + byte B of b
{
    uint32_t r;
    if (B == 0) asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(a), "v"(b));
    else if (B == 1) asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(a), "v"(b));
    else asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
template <int B> __device__ __forceinline__ uint32_t shr_byte(uint32_t v, uint32_t by)       // v >> the low 5 bits of byte B of by
{
    uint32_t r;
    if (B == 0) r = v >> (by & 31u);
    else if (B == 1) asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD" : "=v"(r) : "v"(by), "v"(v));
    else asm("v_lshrrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_2 src1_sel:DWORD" : "=v"(r) : "v"(by), "v"(v));
    return r;
}

// A field's table, by the stream bits a lookup goes by: whole ones by 16, which every code (kWholePairs: every pair of codes of at most
// eight bits) fits, so that nothing is ever unresolved; pairs by 11 - 15 bits; singles by 12 (kShort12: of codes no longer than that).
enum Table { kNone = 32, kPairs11 = 11, kPairs12 = 12, kPairs13 = 13, kPairs15 = 15, kSingles12 = 32 + 12, kWhole = 64 + 16, kWholePairs = 96 + 16, kShort12 = 128 + 12 };
constexpr bool in_pairs(Table t) { return t < 32 || t == kWholePairs; }
constexpr bool is_whole(Table t) { return t == kWhole || t == kWholePairs; }
constexpr bool is_sure(Table t) { return is_whole(t) || t == kShort12; }
constexpr uint32_t index_bits(Table t) { return t % 32; }
constexpr uint32_t entry_bytes(Table t) { return t < 32 ? 4 : 2; }

// When the words that a period's lanes ask for at its end come in: before the next one begins; behind the next one's first entry; or at
// the next one's end (where a period is one lookup: another one later), while that goes well, then behind the first entry; or always
// there (codes too short to be late: a second loop in the kernel costs such calls 1 - 2 %).  See late_run.
enum Loop { kWait, kInside, kLate, kSteady };

// How a chunk is decoded: words of a stream's ring, tables of the two fields
template <uint32_t RING, Loop LOOP, Table T0, Table T1 = kNone> struct Build {
    static constexpr uint32_t kRing = RING;
    static constexpr Loop kLoop = LOOP;
    static constexpr bool kInFours = RING >= 1024 && LOOP != kWait;      // see fours_service
    template <int F> static constexpr Table kTable = F == 0 ? T0 : T1;
};

// How the table entries of field F of format FMT are laid out.  put: a symbol at its place in an output word (kFirst: the bits it can
// take).  The length (a pair's, or a single's) lies in bits the output's two fields leave to each other; it is added by the byte it
// lies in where it has one: a symbol's bit above it leaves the low 7 bits of a sum alone (kNoise).
// Whole tables: 16-bit entries with the length less one (kLow: the length, in the low bits).  Else an entry that does not resolve has
// length 0, so that the lookups after it in the period do not resolve either and the last one tells:
// kPairs*: 32-bit entries of two symbols, the second kSecond bits above the first; kUnresolved (the sign bit) where the pair does
// not fit the index, which has the first symbol alone, its length at kLen1 (0 there: longer than the index).
// kSingles12: 16-bit entries, 0 for a code longer than the index.
//
// Chance that one of 64 lanes finds a pair unresolved, for weights of the kinds the codec is meant for: BF16 exponents 16 % by 12
// bits, E5M2 (a wide spread of exponents) 22 % by 13; singles by 12 bits 19 % (deltas' sign+mantissa) to 42 % (byte symbols).  Each
// sends its wavefront through the period again; hence the whole tables where there is the LDS for them.
constexpr uint32_t kUnresolved = 0x80000000u;
template <int FMT, int F, Table T> struct Layout;
template <Table T> struct Layout<ZC_FMT_BF16, 0, T> {            // pairs
    static constexpr bool kNoise = true, kLow = false;
    static constexpr uint32_t kFirst = 0x7F80u;
    static constexpr int kSecond = 16, kLen = 0, kLen1 = 16;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return s << 7; }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return add_byte<0>(c, e); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return shr_byte<0>(x, e); }
};
template <Table T> struct Layout<ZC_FMT_BF16, 1, T> {            // singles and whole
    static constexpr bool kNoise = true, kLow = false;
    static constexpr uint32_t kFirst = 0x807Fu;
    static constexpr int kSecond = 16, kLen = 8, kLen1 = 0;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return ((s & 0x80u) << 8) | (s & 0x7Fu); }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return add_byte<1>(c, e); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return shr_byte<1>(x, e); }
};
// one value per byte: the pair in bytes 0 and 1, its length in byte 2, the first symbol's in byte 3
template <Table T> struct Layout<ZC_FMT_FP8_E5M2, 0, T> {
    static constexpr bool kNoise = false, kLow = false;
    static constexpr uint32_t kFirst = 0xFFu;
    static constexpr int kSecond = 8, kLen = 16, kLen1 = 24;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return (s << 2) & 0x7Cu; }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return add_byte<2>(c, e); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return shr_byte<2>(x, e); }
};
template <Table T> struct Layout<ZC_FMT_FP8_E4M3, 1, T> : Layout<ZC_FMT_BF16, 1, T> {};      // (never table decoded here)
template <Table T> struct Layout<ZC_FMT_FP8_E5M2, 1, T> : Layout<ZC_FMT_BF16, 1, T> {};
// byte symbols: a symbol is two values, half an output word (exponent bits 0x78 of every byte, sign+mantissa bits 0x87)
template <Table T> struct Layout<ZC_FMT_FP8_E4M3_BYTES, 0, T> {
    static constexpr bool kNoise = false, kLow = false;
    static constexpr uint32_t kFirst = 0x7878u;
    static constexpr int kSecond = 16, kLen = 7, kLen1 = 0;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return ((s & 15u) << 3) | ((s & 0xF0u) << 7); }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return c + ((e >> 7) & 15u); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return x >> ((e >> 7) & 15u); }
};
template <Table T> struct Layout<ZC_FMT_FP8_E4M3_BYTES, 1, T> {
    static constexpr bool kNoise = false, kLow = false;
    static constexpr uint32_t kFirst = 0x8787u;
    static constexpr int kSecond = 16, kLen = 3, kLen1 = 0;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return (s & 7u) | ((s & 8u) << 4) | ((s & 0x70u) << 4) | ((s & 0x80u) << 8); }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return c + ((e >> 3) & 15u); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return x >> ((e >> 3) & 15u); }
};
// FP8 exponents in whole pairs, in bytes 0 and 1 of half an output word
template <> struct Layout<ZC_FMT_FP8_E4M3, 0, kWholePairs> {
    static constexpr bool kNoise = false, kLow = false;
    static constexpr uint32_t kFirst = 0x78u;
    static constexpr int kSecond = 8, kLen = 7, kLen1 = 0;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return (s << 3) & 0x78u; }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return c + ((e >> 7) & 15u); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return x >> ((e >> 7) & 15u); }
};
// the length in the low bits, above which a symbol's in a sum of entries are left alone
struct LengthLow {
    static constexpr bool kNoise = true, kLow = true;
    static constexpr int kLen = 0, kLen1 = 0;
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return c + e; }
    static __device__ __forceinline__ uint64_t shift(uint64_t x, uint32_t e) { return x >> (e & 63u); }
};
template <int FMT> struct OneByte : LengthLow {                  // a symbol in byte 1
    static constexpr uint32_t kFirst = 0xFF00u;
    static constexpr int kSecond = 8;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return (FMT == ZC_FMT_FP8_E4M3 ? (s << 3) & 0x78u : (s << 2) & 0x7Cu) << 8; }
};
template <> struct Layout<ZC_FMT_FP8_E4M3, 0, kWhole> : OneByte<ZC_FMT_FP8_E4M3> {};
template <> struct Layout<ZC_FMT_FP8_E5M2, 0, kWhole> : OneByte<ZC_FMT_FP8_E5M2> {};
template <> struct Layout<ZC_FMT_BF16, 0, kWhole> : LengthLow {
    static constexpr uint32_t kFirst = 0x7F80u;
    static constexpr int kSecond = 16;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return s << 7; }
};
template <int FMT, int F, class W> struct Entries : Layout<FMT, F, W::template kTable<F>> {
    static constexpr Table kTable = W::template kTable<F>;
    static constexpr bool kPair = in_pairs(kTable), kWhole = is_whole(kTable), kSure = is_sure(kTable);
    static constexpr uint32_t kBits = index_bits(kTable), kBytes = entry_bytes(kTable);
};
__device__ __forceinline__ uint32_t first_len(uint32_t e, int shift) { return (e >> shift) & 15u; }
// lookups of a period of R symbols
template <int FMT, int F, int R, class W> constexpr int kLookups = Entries<FMT, F, W>::kPair ? R / 2 : R;
// bits of an output word that come from the exponent entries
template <int FMT> constexpr uint32_t kExponentBits = FMT == ZC_FMT_BF16 ? 0x7F807F80u : FMT == ZC_FMT_FP8_E5M2 ? 0x7C7C7C7Cu : 0x78787878u;
// bytes of a field's table
template <int F, class W> constexpr uint32_t kTableBytes = entry_bytes(W::template kTable<F>) << index_bits(W::template kTable<F>);
// where the rings start: every ring at a multiple of its size, so that a place in it is or-ed to its start
template <class W> constexpr uint32_t rings_at(bool two)
{
    constexpr uint32_t ring = W::kRing * 4;
    return (kTableBytes<0, W> + (two ? kTableBytes<1, W> : 0u) + ring - 1) / ring * ring;
}

// all threads of the workgroup (at least 256)
__device__ __forceinline__ void build_canon(PairCanon &C, uint32_t (*wave_count)[17], const uint8_t *lengths, uint32_t alphabet)
{
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t len = 0, rank = 0;
    if (tid < 256) {
        len = tid < alphabet ? lengths[tid] : 0u;
        if (len > 16) len = 0;
        uint32_t count = 0;
#pragma unroll
        for (uint32_t l = 1; l <= 16; l++) {
            const uint64_t m = __ballot(len == l);
            if (len == l) rank = prefix_count64(m);
            if (lane == l) count = (uint32_t)__popcll(m);
        }
        if (lane < 17) wave_count[wave][lane] = count;
    }
    __syncthreads();
    // lane l of every wavefront: the codes of length l; scans over the lanes give limits and ranks
    const uint32_t l = lane < 17 ? lane : 16u;
    const uint32_t n = lane >= 1 && lane < 17 ? wave_count[0][l] + wave_count[1][l] + wave_count[2][l] + wave_count[3][l] : 0u;
    uint32_t limit = lane < 17 ? n << (16 - l) : 0u, start = n;
    const uint32_t own = limit;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
        const uint32_t a = (uint32_t)__shfl_up((int)limit, o, 64), b = (uint32_t)__shfl_up((int)start, o, 64);
        if (lane >= (uint32_t)o) { limit += a; start += b; }
    }
    start -= n;
    if (wave == 0 && lane < 17) { C.limit[lane] = limit; C.rebase[lane] = start - ((limit - own) >> (16 - l)); }
    if (tid < 256) {
        uint32_t at = (uint32_t)__shfl((int)start, (int)len, 64) + rank;
        for (uint32_t w = 0; w < wave; w++) at += wave_count[w][len];
        if (len) C.sorted[at & 255u] = (uint8_t)tid;
    }
    __syncthreads();
}

// the code at the start of bits w (in code order, left aligned), by limits 1 .. K: its length, K + 1 where it is longer
template <uint32_t K>
__device__ __forceinline__ uint32_t code_length(uint32_t w, const uint32_t (&limit)[K + 1])
{
    uint32_t len = 1;
#pragma unroll
    for (uint32_t l = 1; l <= K; l++) len += w >= limit[l];
    return len;
}
__device__ __forceinline__ uint32_t code_symbol(const PairCanon &C, uint32_t w, uint32_t len) { return C.sorted[(C.rebase[len] + (w >> (16 - len))) & 255u]; }

// A whole table, by 1,024 threads: thread t has the entries whose low ten bits are t, for which a code of at most ten bits is looked up
// once (a pair's first code has at most eight: then only the second one differs); the few indices with longer codes are dealt out
// to all threads.
struct LongCodes { uint32_t n; uint16_t at[1024]; };
template <int FMT, int F, class W>
__device__ __forceinline__ void build_whole(uint16_t *table, const PairCanon &C, const uint32_t (&limit)[17], LongCodes &longs)
{
    typedef Entries<FMT, F, W> P;
    const uint32_t tid = threadIdx.x;
    constexpr uint32_t less = P::kLow ? 0 : 1;
    if (tid == 0) longs.n = 0;
    __syncthreads();
    if (tid < 1024) {
        const uint32_t w = __brev(tid) >> 16, len = code_length<16>(w, limit);
        if (P::kPair) {
            if (tid < 256) longs.at[tid] = (uint16_t)(P::put(code_symbol(C, w, len < 16 ? len : 16u)) | ((len < 16 ? len : 16u) - 1) << P::kLen);
        } else if (len <= 10) {
            const uint16_t e = (uint16_t)(P::put(code_symbol(C, w, len)) | (len - less) << P::kLen);
#pragma unroll 8
            for (uint32_t j = 0; j < 64; j++) table[tid + j * 1024] = e;
        } else longs.at[atomicAdd(&longs.n, 1u)] = (uint16_t)tid;
    }
    __syncthreads();
    if (P::kPair) {
        if (tid < 1024) {
            const uint32_t a = longs.at[tid & 255u], l1 = first_len(a, P::kLen) + 1;
#pragma unroll 8
            for (uint32_t j = 0; j < 64; j++) {
                const uint32_t i = tid + j * 1024, b = longs.at[(i >> l1) & 255u];
                table[i] = (uint16_t)((a & P::kFirst) | ((b & P::kFirst) << P::kSecond) | ((l1 + first_len(b, P::kLen)) & 15u) << P::kLen);
            }
        }
    } else {
        for (uint32_t q = tid, n = longs.n * 64; q < n; q += blockDim.x) {
            const uint32_t i = longs.at[q >> 6] + (q & 63u) * 1024, w = __brev(i) >> 16;
            uint32_t len = code_length<16>(w, limit);
            if (len > 16) len = 16;
            table[i] = (uint16_t)(P::put(code_symbol(C, w, len)) | (len - less) << P::kLen);
        }
    }
    __syncthreads();
}

// Pairs by 15 bits of codes of at most eight, by 1,024 threads: only two of eight bits each do not fit
template <int FMT, int F, class W>
__device__ __forceinline__ void build_pairs(uint32_t *table, const PairCanon &C, const uint32_t (&limit)[16], LongCodes &longs)
{
    typedef Entries<FMT, F, W> P;
    const uint32_t tid = threadIdx.x;
    if (tid < 256) {
        const uint32_t w = __brev(tid) >> 16, len = code_length<15>(w, limit);
        longs.at[tid] = (uint16_t)(code_symbol(C, w, len) | (len < 9 ? len : 8u) << 8);
    }
    __syncthreads();
    const uint32_t a = longs.at[tid & 255u], l1 = a >> 8;
#pragma unroll 8
    for (uint32_t j = 0; j < 32; j++) {
        const uint32_t i = tid + j * 1024, b = longs.at[(i >> l1) & 255u], l2 = b >> 8;
        table[i] = P::put(a & 255u) | l1 << P::kLen1 | (l1 + l2 < 16 ? P::put(b & 255u) << P::kSecond | (l1 + l2) << P::kLen : kUnresolved);
    }
    __syncthreads();
}

template <int FMT, int F, class W>
__device__ __forceinline__ void build_entries(char *table, const PairCanon &C, LongCodes &longs)
{
    typedef Entries<FMT, F, W> P;
    constexpr uint32_t K = P::kBits, entries = 1u << K;
    const uint32_t lane = threadIdx.x & 63, mine = lane < 17 ? C.limit[lane] : 0u;
    uint32_t limit[K + 1];
#pragma unroll
    for (uint32_t l = 1; l <= K; l++) limit[l] = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)l);
    uint32_t *const pairs = reinterpret_cast<uint32_t *>(table);
    uint16_t *const singles = reinterpret_cast<uint16_t *>(table);
    if constexpr (P::kWhole) { build_whole<FMT, F, W>(singles, C, limit, longs); return; }
    if constexpr (P::kTable == kPairs15) { build_pairs<FMT, F, W>(pairs, C, limit, longs); return; }
    // A thread's entries have the low eight bits of their index in common, so a code of at most eight bits can be looked up once for
    // all of them: 1,000 E5M2 tensors of 2 KB 24.5 -> 21.5 us.  The other formats have longer codes in some lane of nearly every
    // wavefront, which would make it 3 - 5 % slower for small chunks.
    constexpr bool kOnce = FMT == ZC_FMT_FP8_E5M2;
    uint32_t len = 0, e = 0;
    for (uint32_t i = threadIdx.x; i < entries; i += blockDim.x) {
        if (!kOnce || len == 0 || len > 8) {
            const uint32_t w = __brev(i) >> 16;                  // the stream bits in code order, left aligned
            len = code_length<K>(w, limit);
            e = P::kPair ? kUnresolved : 0u;
            if (len <= K) e |= P::put(code_symbol(C, w, len)) | (len << (P::kPair ? P::kLen1 : P::kLen));
        }
        if (P::kPair) pairs[i] = e; else singles[i] = (uint16_t)e;
    }
    __syncthreads();
    if (!P::kPair) return;
    for (uint32_t i = threadIdx.x; i < entries; i += blockDim.x) {
        // (an entry read here may already hold its second symbol: its first one and that one's length never change)
        const uint32_t e = pairs[i], l1 = first_len(e, P::kLen1);
        if (!l1) continue;
        const uint32_t e2 = pairs[i >> l1], l2 = first_len(e2, P::kLen1);
        if (l2 && l1 + l2 <= K) pairs[i] = (e & ~kUnresolved) | ((e2 & P::kFirst) << P::kSecond) | ((l1 + l2) << P::kLen);
    }
    __syncthreads();
}

// The kernel has no LDS of fixed size, so what it is launched with starts at LDS address 0, and tables and rings are reached by
// plain addresses: a table index is an address as soon as it is masked.
typedef uint32_t __attribute__((address_space(3))) LdsWord;
typedef uint16_t __attribute__((address_space(3))) LdsHalf;
__device__ __forceinline__ uint32_t lds_word(uint32_t at) { return *reinterpret_cast<const LdsWord *>(at); }
// (not to be moved behind a branch)
__device__ __forceinline__ uint32_t lds_word_now(uint32_t at) { return *reinterpret_cast<const volatile LdsWord *>(at); }

// One table-decoded stream of a lane: 64 bits in (hi, lo), c of them used.  After a refill c is below 32, but for a lane whose
// every period so far took exactly 32 bits (as at the start): c is 32 then and lo and hi are both the word that comes next,
// so that a funnel shift by c's low five bits gives the window either way.
struct PairStream {
    uint32_t lo, hi, c;
    uint32_t wpos, wbase, pslot;             // as in HuffStream
    bool pending;
    uint32_t on;
    u32x4 pv[4];                             // the newest segment, on its way into the ring
    uint32_t ring;                           // LDS address
    uint32_t limit[4];                       // limits of the lengths from the index's on (uniform), see long_symbol
    __amdgpu_buffer_rsrc_t rs;
};

// Ring of W words per wavefront and field, refilled SEG = W / 4 words at a time; see ring_service in zc_decode_s64.hip
template <uint32_t B>
__device__ __forceinline__ void ring_write(uint32_t at, const u32x4 &v)
{
    typedef u32x4 __attribute__((address_space(3))) LdsX4;
    typedef u32x2 __attribute__((address_space(3))) LdsX2;
    if (B == 4) *reinterpret_cast<LdsX4 *>(at) = v;
    else if (B == 2) *reinterpret_cast<LdsX2 *>(at) = u32x2{v.x, v.y};
    else *reinterpret_cast<LdsWord *>(at) = v.x;
}
template <uint32_t B>
__device__ __forceinline__ u32x4 segment_load(__amdgpu_buffer_rsrc_t rs, uint32_t at)
{
    u32x4 v = {0, 0, 0, 0};
    if (B == 4) v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)at, 0, 0);
    else if (B == 2) { const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)at, 0, 0); v.x = w.x; v.y = w.y; }
    else v.x = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)at, 0, 0);
    return v;
}

// A segment of SEG words: pieces of 64 * B words, B of them per lane and load
template <class W> struct Segment {
    static constexpr uint32_t kWords = W::kRing / 4, B = kWords >= 256 ? 4 : kWords / 64, kPieces = kWords / (64 * B);
    static_assert((B == 1 || B == 2 || B == 4) && kPieces >= 1 && kPieces <= 4, "whole loads");
};

template <class W>
__device__ __forceinline__ void pair_open(PairStream &S, uint32_t lane, bool owner)
{
    constexpr uint32_t B = Segment<W>::B;
    constexpr uint32_t kLoads = W::kRing / (64 * B), kAtOnce = kLoads < 8 ? kLoads : 8;
#pragma unroll 1
    for (uint32_t q = 0; q < kLoads; q += kAtOnce) {
        u32x4 v[kAtOnce];
#pragma unroll
        for (uint32_t i = 0; i < kAtOnce; i++) v[i] = segment_load<B>(S.rs, ((q + i) * 64 + lane) * B * 4);
        __builtin_amdgcn_sched_barrier(0);                       // (all of them in flight, then the writes)
#pragma unroll
        for (uint32_t i = 0; i < kAtOnce; i++) ring_write<B>(S.ring + ((q + i) * 64 + lane) * B * 4, v[i]);
    }
    const uint64_t takers = __ballot(owner);
    S.hi = lds_word(S.ring + prefix_count64(takers) * 4);
    S.lo = S.hi;
    S.c = 32; S.wpos = (uint32_t)__popcll(takers); S.wbase = 0; S.pslot = 0; S.pending = false; S.on = 0;
    if (W::kInFours) S.wbase = S.pslot = W::kRing;
#pragma unroll
    for (int i = 0; i < 4; i++) S.pv[i] = u32x4{0, 0, 0, 0};
}

// the segment on its way, when there is one, into its place
template <class W>
__device__ __forceinline__ void pair_settle(PairStream &S, uint32_t lane)
{
    constexpr uint32_t B = Segment<W>::B;
    if (S.pending) {
#pragma unroll
        for (uint32_t q = 0; q < Segment<W>::kPieces; q++) ring_write<B>(S.ring + (S.pslot + (q * 64 + lane) * B) * 4, S.pv[q]);
    }
}

template <class W>
__device__ __forceinline__ void pair_service(PairStream &S, uint32_t lane)
{
    constexpr uint32_t SEG = Segment<W>::kWords, B = Segment<W>::B;
    if (S.wpos - S.wbase >= SEG) {
        pair_settle<W>(S, lane);
#pragma unroll
        for (uint32_t q = 0; q < Segment<W>::kPieces; q++) S.pv[q] = segment_load<B>(S.rs, (S.wbase + W::kRing + (q * 64 + lane) * B) * 4);
        S.pslot = S.wbase & (W::kRing - 1);
        S.wbase += SEG;
        S.pending = true;
    }
}

// The same for the long rings, whose wavefronts are alone on their SIMDs and have nobody to hide a wait: a row asks for a piece of an
// eighth of the ring (128 words; FP8 and E5M2 weights take 83 per row) and writes the one that was asked for four rows ago into the
// ring, each of the four into registers of its own.  (With one segment at a time a wait for it is a wait for what the row before
// has asked for.)
// wbase: words that are in the ring, pslot: words asked for, pv[i], on: the pieces on their way
template <class W> constexpr uint32_t kPiece = W::kRing / 8;
constexpr uint32_t kGuard = 256;                                 // (a period takes 64 words at most, and four are what a guard is for)
template <class W>
__device__ __forceinline__ void fours_write(PairStream &S, uint32_t i, uint32_t lane)
{
    constexpr uint32_t B = kPiece<W> / 64;
    if (S.on & (1u << i)) {
        ring_write<B>(S.ring + ((S.wbase & (W::kRing - 1)) + lane * B) * 4, S.pv[i]);
        S.wbase += kPiece<W>;
    }
}
template <class W, uint32_t ROW>
__device__ __forceinline__ void fours_service(PairStream &S, uint32_t lane)
{
    constexpr uint32_t B = kPiece<W> / 64;
    fours_write<W>(S, ROW, lane);
    S.on &= ~(1u << ROW);
    if (S.pslot + kPiece<W> - S.wpos <= W::kRing) {
        S.pv[ROW] = segment_load<B>(S.rs, (S.pslot + lane * B) * 4);
        S.pslot += kPiece<W>;
        S.on |= 1u << ROW;
    }
}
// what is on its way (the oldest of it after row ROW's) into the ring, then as much as it holds: there has to be a guard's worth
template <class W, uint32_t ROW>
__device__ __forceinline__ void fours_guard(PairStream &S, uint32_t lane)
{
    constexpr uint32_t B = kPiece<W> / 64;
    if (__builtin_expect(S.wbase - S.wpos >= kGuard, 1)) return;
#pragma unroll
    for (uint32_t k = 1; k <= 4; k++) fours_write<W>(S, (ROW + k) & 3u, lane);
    S.on = 0;
    while (S.wbase + kPiece<W> - S.wpos <= W::kRing) {
        ring_write<B>(S.ring + ((S.wbase & (W::kRing - 1)) + lane * B) * 4, segment_load<B>(S.rs, (S.wbase + lane * B) * 4));
        S.wbase += kPiece<W>;
    }
    S.pslot = S.wbase;
}

// A code longer than the K index bits, K = 12 .. 14: the left-aligned codes of length <= l all lie below limit[l], so its length is
// K + 1 plus the number of those limits that the next 16 bits reach.
template <uint32_t K>
__device__ __forceinline__ uint32_t long_symbol(const PairStream &S, const PairCanon &C, uint32_t x, uint32_t &len)
{
    const uint32_t w = __brev(x) >> 16;
    len = K + 1;
#pragma unroll
    for (uint32_t i = 0; i < 15 - K; i++) len += w >= S.limit[i];
    return C.sorted[(C.rebase[len] + (w >> (16 - len))) & 255u];
}

// The entry at the window x, which lies SCALE bits up (where it is scaled by an entry's size, masked it is an address)
template <int FMT, int F, int SCALE, class W>
__device__ __forceinline__ uint32_t entry_at(uint32_t x)
{
    typedef Entries<FMT, F, W> P;
    constexpr int size = P::kBytes == 4 ? 2 : 1;
    constexpr uint32_t mask = ((1u << P::kBits) - 1) << size, table = F == 0 ? 0u : kTableBytes<0, W>;
    const uint32_t at = ((x << (size - SCALE)) & mask) + table;
    if (P::kBytes == 4) return lds_word(at);
    return *reinterpret_cast<const LdsHalf *>(at);
}
// Bits a period's window is scaled by: where the bits this costs at its top are no lookup's.  (In a whole table's period, with its
// lengths less one, the shift past a code leaves the window scaled by one; kLow: a window of 64 bits.)
template <int FMT, int F, int N, class W>
constexpr int kScale = Entries<FMT, F, W>::kLow ? 1 : Entries<FMT, F, W>::kWhole || N * (int)Entries<FMT, F, W>::kBits + (Entries<FMT, F, W>::kPair ? 2 : 1) > 32 ? 0 : Entries<FMT, F, W>::kPair ? 2 : 1;

// the entries of a period from FROM on, where the one before it was found at the window (scaled)
template <int FMT, int F, int N, class W, int FROM>
__device__ __forceinline__ void look_on(uint64_t window, uint32_t e[N])
{
    typedef Entries<FMT, F, W> P;
    uint32_t x = (uint32_t)window;
#pragma unroll
    for (int i = FROM; i < N; i++) {
        if constexpr (P::kLow) {
            window = P::shift(window, e[i - 1]);
            e[i] = entry_at<FMT, F, 1, W>((uint32_t)window);
            continue;
        }
        const uint32_t y = (uint32_t)P::shift(x, e[i - 1]);
        e[i] = entry_at<FMT, F, P::kWhole ? 1 : kScale<FMT, F, N, W>, W>(y);
        x = P::kWhole ? y >> 1 : y;
    }
}
// c: bits used before a period's entries, returns them after it (in the low 7 bits)
template <int FMT, int F, int N, class W>
__device__ __forceinline__ uint32_t add_up(uint32_t c, const uint32_t e[N])
{
    if (Entries<FMT, F, W>::kWhole && !Entries<FMT, F, W>::kLow) c += N;
#pragma unroll
    for (int i = 0; i < N; i++) c = Entries<FMT, F, W>::add(c, e[i]);
    return c;
}
// a period's entries, N of them, from window x
template <int FMT, int F, int N, class W>
__device__ __forceinline__ uint32_t look_up(uint32_t c, uint32_t x, uint32_t e[N])
{
    const uint64_t window = (uint64_t)x << kScale<FMT, F, N, W>;
    e[0] = entry_at<FMT, F, kScale<FMT, F, N, W>, W>((uint32_t)window);
    look_on<FMT, F, N, W, 1>(window, e);
    return add_up<FMT, F, N, W>(c, e);
}
template <int FMT, int F, class W>
__device__ __forceinline__ bool unresolved(uint32_t e) { return !Entries<FMT, F, W>::kSure && (Entries<FMT, F, W>::kPair ? (int)e < 0 : e == 0); }

// The same where an entry does not resolve in some lane; e[0]: as look_up found it (in every lane the right one); FOUND: and the others,
// which are right in the lanes where those before them resolved
template <int FMT, int F, int N, class W, bool FOUND>
__device__ __forceinline__ uint32_t look_up_slowly(const PairStream &S, const PairCanon &C, uint32_t c, uint32_t x, uint32_t e[N])
{
    typedef Entries<FMT, F, W> P;
    constexpr uint32_t K = P::kBits;
    if constexpr (P::kWhole) return look_up<FMT, F, N, W>(c, x, e);
    else {
#pragma unroll
    for (int i = 0; i < N; i++) {
        uint32_t a = e[i], len;
        if (P::kPair) {
            if (i > 0) a = entry_at<FMT, F, 0, W>(x);
            // both symbols one after the other in every lane
            uint32_t l1 = first_len(a, P::kLen1), s1 = a & P::kFirst;
            uint32_t b = entry_at<FMT, F, 0, W>(x >> l1);
            uint32_t l2 = first_len(b, P::kLen1), s2 = b & P::kFirst;
            if (__builtin_expect(__ballot(l1 == 0 || l2 == 0) != 0, 0)) {
                if (l1 == 0) {
                    s1 = P::put(long_symbol<K>(S, C, x, l1)) & P::kFirst;
                    b = entry_at<FMT, F, 0, W>(x >> l1);
                    l2 = first_len(b, P::kLen1); s2 = b & P::kFirst;
                }
                if (l2 == 0) s2 = P::put(long_symbol<K>(S, C, x >> l1, l2)) & P::kFirst;
            }
            a = s1 | (s2 << P::kSecond);
            len = l1 + l2;
        } else {
            if (i > 0 && !FOUND) a = entry_at<FMT, F, 0, W>(x);
            len = first_len(a, P::kLen);
            a &= P::kFirst;
            if (len == 0) {
                a = P::put(long_symbol<K>(S, C, x, len)) & P::kFirst;
                if (FOUND && i + 1 < N) e[i + 1] = entry_at<FMT, F, 0, W>(x >> len);
            }
        }
        e[i] = a;
        c += len;
        x = len < 32 ? x >> len : 0u;
    }
    return c;
    }
}

// The refill step that follows a period: lanes that hold 32 bits or less take the next word of the stream, in lane order.
// t: bits used so far, in its low 7 bits.  CAREFUL: owner says which lanes own a symbol at the step the words are for, and
// lanes whose every period took 32 bits are looked after.
struct Refill { bool need; uint32_t t, w, taken; };
template <class W, bool CAREFUL, bool NOISE>
__device__ __forceinline__ Refill ask(const PairStream &S, uint32_t t, bool owner)
{
    Refill r;
    r.t = CAREFUL ? t & 127u : NOISE ? t & 63u : t;
    r.need = r.t > 31u && (!CAREFUL || owner);
    const uint64_t bm = __ballot(r.need);
    const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(bm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bm, S.wpos));
    r.w = lds_word_now(S.ring + (pos & (W::kRing - 1)) * 4);          // (its latency covers the check of the entries)
    r.taken = (uint32_t)__popcll(bm);
    return r;
}
template <bool CAREFUL>
__device__ __forceinline__ void take(PairStream &S, const Refill &r)
{
    S.lo = r.need ? ((CAREFUL && r.t == 64u) ? r.w : S.hi) : S.lo;
    S.hi = r.need ? r.w : S.hi;
    S.c = CAREFUL ? (r.need ? r.t - 32u : r.t) : r.t & 31u;
    S.wpos += r.taken;
}

// One run of G symbols of the exponent field (A) and, when TWO, of the sign+mantissa field (B): their entries in ea, eb.  CAREFUL: nsym is
// what this lane owns of its symbols, nsym_next of the one's after it
template <int FMT, int R, bool TWO, class W, bool CAREFUL, bool SERVICE>
__device__ __forceinline__ void pair_run(PairStream &A, PairStream &B, const PairCanon *C, uint32_t lane, uint32_t ea[], uint32_t eb[],
                                            uint32_t nsym, uint32_t nsym_next)
{
    constexpr int G = Fmt<FMT>::G, NA = kLookups<FMT, 0, R, W>, NB = kLookups<FMT, 1, R, W>;
    constexpr uint32_t kPerService = W::kRing / 4 / 64;                // refill steps between two looks at the ring
#pragma unroll
    for (int g = 0; g < G / R; g++) {
        if (W::kInFours) {
            if (g % 4 == 0) { fours_guard<W, 3>(A, lane); if (TWO) fours_guard<W, 3>(B, lane); }
        } else if (SERVICE && (uint32_t)g % kPerService == 0) {
            pair_service<W>(A, lane);
            if (TWO) pair_service<W>(B, lane);
        }
        const uint32_t xa = __builtin_amdgcn_alignbit(A.hi, A.lo, A.c), xb = TWO ? __builtin_amdgcn_alignbit(B.hi, B.lo, B.c) : 0u;
        const bool owner = !CAREFUL || (g + 1 < G / R ? (uint32_t)((g + 1) * R) < nsym : nsym_next > 0);
        uint32_t *const a = ea + g * NA, *const b = eb + g * NB;
        uint32_t ta = look_up<FMT, 0, NA, W>(A.c, xa, a), tb = TWO ? look_up<FMT, 1, NB, W>(B.c, xb, b) : 0u;
        Refill ra = ask<W, CAREFUL, Entries<FMT, 0, W>::kNoise>(A, ta, owner), rb;
        if (TWO) rb = ask<W, CAREFUL, Entries<FMT, 1, W>::kNoise>(B, tb, owner);
        if (__builtin_expect(__any(unresolved<FMT, 0, W>(a[NA - 1])), 0)) {
            ta = look_up_slowly<FMT, 0, NA, W, true>(A, C[0], A.c, xa, a);
            ra = ask<W, CAREFUL, Entries<FMT, 0, W>::kNoise>(A, ta, owner);
        }
        if (TWO && __builtin_expect(__any(unresolved<FMT, 1, W>(b[NB - 1])), 0)) {
            tb = look_up_slowly<FMT, 1, NB, W, true>(B, C[1], B.c, xb, b);
            rb = ask<W, CAREFUL, Entries<FMT, 1, W>::kNoise>(B, tb, owner);
        }
        take<CAREFUL>(A, ra);
        if (TWO) take<CAREFUL>(B, rb);
    }
}

// Whole rows in which every lane owns every symbol and has left the state of the start: a period does not wait for the words asked
// for before it.  It goes by what (hi, lo) still hold: where a period is one lookup, the words asked for at the end of the period
// before the last one come in during it, else those asked for at the end of the last one.  So the chain of a period is its lookups
// alone, and the refill (the count of the lanes that take a word, an address, an LDS read) runs beside them.  Zeros come into a
// window that runs out of bits; an entry found there is still the right one as long as its codes' bits were there, so a period
// has gone wrong only in lanes that wait for a word and are already past the next 32 bits (3.6 % of the periods of FP8 E4M3 weights,
// 2.1 % of byte symbols, 1.0 % of deltas, hardly any where a period is one lookup), and is done once more.  Where
// codes are so long that two periods often take more than 32 bits (wide) that would be nearly every period.  There the word comes in
// behind the period's first entry (kInside), which costs two to three more instructions and goes wrong only where one code is that long.
// What is not the chain stands where LDS reads are waited for anyway, masks are read late, and there is one branch per period.
// x: the window, scaled for a lookup; e: the entry found there; c: bits used of (hi, lo) once what is owed has come in; need, w: lanes
// that asked at the end of the last period, and the words; owed, v: at the end of the one before it (kTwice only).
// (Copied member by member: as a whole, the padding would go through scratch memory.)
struct Late {
    uint64_t x;
    uint32_t lo, hi, c, e, w, v, wpos, wrap, taken;
    uint64_t asked, asked_before;            // the lanes with need, with owed
    bool need, owed;
    __device__ __forceinline__ Late() {}
    __device__ __forceinline__ Late(const Late &o) { *this = o; }
    __device__ __forceinline__ Late &operator=(const Late &o)
    {
        lo = o.lo; hi = o.hi; c = o.c; x = o.x; e = o.e; w = o.w; v = o.v; wpos = o.wpos; wrap = o.wrap; taken = o.taken;
        asked = o.asked; asked_before = o.asked_before; need = o.need; owed = o.owed;
        return *this;
    }
};
// one pair per period: no lane asks twice within two periods (31 bits, a pair of at most 15, again one: no 64)
template <int FMT, int F, int N, class W> constexpr bool kTwice = N == 1 && Entries<FMT, F, W>::kPair && !Entries<FMT, F, W>::kWhole;
__device__ __forceinline__ void in_order() { __builtin_amdgcn_sched_barrier(0); }

// what the lanes look up next at bit t of (hi, lo)
template <int FMT, int F, int N, class W>
__device__ __forceinline__ void late_window(Late &S, uint32_t t)
{
    const uint64_t w = ((uint64_t)S.hi << 32 | S.lo) >> (t & 63u);
    S.x = Entries<FMT, F, W>::kLow ? w << 1 : (uint32_t)w << kScale<FMT, F, N, W>;
    S.e = entry_at<FMT, F, kScale<FMT, F, N, W>, W>((uint32_t)S.x);
}
// the word they ask for
template <class W>
__device__ __forceinline__ void late_ask(Late &S, uint32_t ring)
{
    S.need = S.c > 31u;
    const uint64_t bm = S.asked = __ballot(S.need);
    const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(bm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bm, S.wpos));
    uint32_t at;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(at) : "v"(pos << 2), "v"(S.wrap), "s"(ring));        // ring + pos % kRing * 4
    S.w = lds_word_now(at);
    in_order();                                                  // (what reads the mask in scalar registers: not right behind the comparison)
    const uint32_t n = (uint32_t)__popcll(bm);
    S.wpos += n;
    S.taken += n;
    asm("" : "+v"(S.wpos));                                      // (stays in a vector register, where it is counted on from; taken: the same in a scalar one)
}
__device__ __forceinline__ void late_take(Late &S, bool lanes, uint32_t word)
{
    S.lo = lanes ? S.hi : S.lo;
    S.hi = lanes ? word : S.hi;
}
// The period's entries; INSIDE: the word that is out comes in (into next) behind the first of them
template <int FMT, int F, int N, class W, bool INSIDE>
__device__ __forceinline__ void late_look(Late &next, const Late &L, uint32_t e[N])
{
    typedef Entries<FMT, F, W> P;
    e[0] = L.e;
    if constexpr (INSIDE) {
        static_assert(N > 1, "a second lookup");
        next = L;
        late_take(next, L.need, L.w);
        const uint32_t second = P::add((L.c & 31u) + (P::kWhole && !P::kLow ? 1u : 0u), e[0]) & 63u;
        const uint64_t w = ((uint64_t)next.hi << 32 | next.lo) >> second, x = P::kLow ? w << 1 : (uint32_t)w << kScale<FMT, F, N, W>;
        e[1] = entry_at<FMT, F, kScale<FMT, F, N, W>, W>((uint32_t)x);
        look_on<FMT, F, N, W, 2>(x, e);
    } else look_on<FMT, F, N, W, 1>(L.x, e);
}
// everything asked for comes in
template <bool TWICE>
__device__ __forceinline__ void late_settle(Late &S)
{
    if (TWICE) late_take(S, S.owed, S.v);
    late_take(S, S.need, S.w);
    S.c &= 31u;
    S.need = S.owed = false; S.asked = S.asked_before = 0;
}
template <int FMT, int F, int N, class W>
__device__ __forceinline__ void late_open(Late &L, const PairStream &S)
{
    L.lo = S.lo; L.hi = S.hi; L.c = S.c; L.wpos = L.taken = S.wpos;
    L.need = L.owed = false; L.asked = L.asked_before = 0; L.w = L.v = 0;
    L.wrap = (W::kRing - 1) * 4;
    asm("" : "+v"(L.wpos), "+v"(L.wrap));
    late_window<FMT, F, N, W>(L, L.c);
}
template <bool TWICE>
__device__ __forceinline__ void late_close(Late &L, PairStream &S)
{
    late_settle<TWICE>(L);
    S.lo = L.lo; S.hi = L.hi; S.c = L.c; S.wpos = L.taken;
}
// The rest of the period: what was out comes in, the next window is looked up, the next word asked for.  t: the bit the next window
// starts at, c: bits used as they are counted for the next word (at t, less 32 in the lanes whose word is not in yet)
template <int FMT, int F, int N, class W, bool INSIDE>
__device__ __forceinline__ void late_go_on(Late &next, const Late &L, const PairStream &S, uint32_t t, uint32_t c)
{
    if (kTwice<FMT, F, N, W>) {
        late_take(next, L.owed, L.v);
        late_window<FMT, F, N, W>(next, t);
        next.owed = L.need; next.asked_before = L.asked; next.v = L.w;
    } else {
        if (!INSIDE) late_take(next, L.need, L.w);
        late_window<FMT, F, N, W>(next, t);
    }
    in_order();                                                  // (the chain goes through the entry: its read first)
    next.c = Entries<FMT, F, W>::kNoise ? c & 63u : c;
    late_ask<W>(next, S.ring);
}
// the period from L on as it should go; returns the lanes in which it did not.  c: bits used after its entries
template <int FMT, int F, int N, class W, bool INSIDE>
__device__ __forceinline__ uint64_t late_period(Late &next, const Late &L, const PairStream &S, const uint32_t e[N], uint32_t c)
{
    constexpr bool TWICE = kTwice<FMT, F, N, W>;
    if constexpr (INSIDE) {
        // (an entry that did not resolve because its bits were not there: the ones after it may.  All in one sign.)
        int sign = 64 - (int)(Entries<FMT, F, W>::add(L.c + (Entries<FMT, F, W>::kWhole && !Entries<FMT, F, W>::kLow ? 1u : 0u), e[0]) & 127u);
        if (!Entries<FMT, F, W>::kSure) sign |= Entries<FMT, F, W>::kPair ? (int)(e[0] | e[N - 1]) : ((int)e[0] - 1) | ((int)e[N - 1] - 1);
        const uint64_t amiss = __ballot(sign < 0);
        late_go_on<FMT, F, N, W, true>(next, L, S, c, c);
        return amiss;
    }
    const uint64_t open = __ballot(unresolved<FMT, F, W>(e[N - 1]));
    next = L;
    late_go_on<FMT, F, N, W, false>(next, L, S, TWICE ? Entries<FMT, F, W>::add(L.c, e[0]) : c, c);
    return open | (next.asked & (TWICE ? L.asked_before : L.asked));
}
// The period once more, where it went wrong in some lane
template <int FMT, int F, int N, class W>
__device__ __forceinline__ void late_again(Late &next, const Late &L, const PairStream &S, const PairCanon &C, uint32_t e[N])
{
    typedef Entries<FMT, F, W> P;
    constexpr bool TWICE = kTwice<FMT, F, N, W>;
    constexpr uint32_t K = P::kBits;
    uint64_t amiss = 1;
    uint32_t l1 = 0, l2 = 0, b = 0;
    if (TWICE) {
        // some lanes' second symbols have to be looked up by themselves: that is all, unless a code is longer than the index, a
        // lane's words are late, or it takes so many bits that the next period's index might not be there
        l1 = first_len(e[0], P::kLen1);
        b = entry_at<FMT, F, kScale<FMT, F, N, W>, W>((uint32_t)L.x >> l1);
        l2 = first_len(b, P::kLen1);
        const int room = (int)((L.owed ? 32u : 63u - K) - (L.c + l1 + l2)), shorter = (int)(l1 < l2 ? l1 : l2) - 1;
        amiss = __ballot((room | shorter) < 0) | (next.asked & L.asked_before);
    }
    next = L;
    if (TWICE && amiss == 0) {
        e[0] = (e[0] & P::kFirst) | ((b & P::kFirst) << P::kSecond);
        late_go_on<FMT, F, N, W, false>(next, L, S, L.c + l1 + l2, (L.c & 31u) + l1 + l2);
        return;
    }
    late_settle<TWICE>(next);
    const uint32_t x = __builtin_amdgcn_alignbit(next.hi, next.lo, next.c);
    e[0] = entry_at<FMT, F, 0, W>(x);
    next.c = look_up_slowly<FMT, F, N, W, false>(S, C, next.c, x, e) & 63u;
    if (TWICE) {
        // (nothing is owed after it: its codes may be longer than the index)
        late_ask<W>(next, S.ring);
        late_settle<TWICE>(next);
        late_window<FMT, F, N, W>(next, next.c);
        asm volatile("" : "+v"(next.e));                         // (waited for here, or the way on would wait for all that is out)
    } else {
        late_window<FMT, F, N, W>(next, next.c);
        in_order();
        late_ask<W>(next, S.ring);
    }
}

// Periods there have been, less kAgain times those in which a word came too late; rows up to which words come in late (none if that was often)
struct LateRoom { static constexpr int kAgain = 12; int room; uint32_t end; };

// fill(g): what there is to do while the entries of period g are on their way
template <int FMT, int R, bool TWO, class W, bool SERVICE, uint32_t ROW, bool INSIDE, class Fill>
__device__ __forceinline__ void late_run(Late &LA, Late &LB, PairStream &A, PairStream &B, const PairCanon *C, uint32_t lane, uint32_t ea[], uint32_t eb[], LateRoom &late, Fill fill)
{
    constexpr int G = Fmt<FMT>::G, NA = kLookups<FMT, 0, R, W>, NB = kLookups<FMT, 1, R, W>;
    constexpr bool inside_a = INSIDE && NA > 1, inside_b = INSIDE && NB > 1;
    constexpr uint32_t kPerService = W::kRing / 4 / 64;         // refill steps between two looks at the ring
#pragma unroll
    for (int g = 0; g < G / R; g++) {
        if (W::kInFours) {
            A.wpos = LA.taken;
            if (TWO) B.wpos = LB.taken;
            if (g == 0) { fours_service<W, ROW>(A, lane); if (TWO) fours_service<W, ROW>(B, lane); }
            if (g % 4 == 0) { fours_guard<W, ROW>(A, lane); if (TWO) fours_guard<W, ROW>(B, lane); }
        } else if (SERVICE && (uint32_t)g % kPerService == 0) {
            A.wpos = LA.taken; pair_service<W>(A, lane);
            if (TWO) { B.wpos = LB.taken; pair_service<W>(B, lane); }
        }
        uint32_t *const a = ea + g * NA, *const b = eb + g * NB;
        Late nextA, nextB;
        late_look<FMT, 0, NA, W, inside_a>(nextA, LA, a);
        if (TWO) late_look<FMT, 1, NB, W, inside_b>(nextB, LB, b);
        in_order();                                              // (nothing that waits for the words before this)
        fill(g, G / R);
        in_order();
        const uint32_t ca = add_up<FMT, 0, NA, W>(LA.c & 31u, a), cb = TWO ? add_up<FMT, 1, NB, W>(LB.c & 31u, b) : 0u;
        const uint64_t wrong_a = late_period<FMT, 0, NA, W, inside_a>(nextA, LA, A, a, ca);
        const uint64_t wrong_b = TWO ? late_period<FMT, 1, NB, W, inside_b>(nextB, LB, B, b, cb) : 0u;
        if (__builtin_expect((wrong_a | wrong_b) != 0, 0)) {
            const bool late_a = !kTwice<FMT, 0, NA, W> && (nextA.asked & LA.asked) != 0, late_b = TWO && !kTwice<FMT, 1, NB, W> && (nextB.asked & LB.asked) != 0;
            if (!INSIDE && W::kLoop == kLate && (late_a || late_b)) {
                late.room -= LateRoom::kAgain;
                if (late.room < 0) late.end = 0;
            }
            if (!TWO || wrong_a != 0) late_again<FMT, 0, NA, W>(nextA, LA, A, C[0], a);
            if (TWO && wrong_b != 0) late_again<FMT, 1, NB, W>(nextB, LB, B, C[1], b);
        }
        LA = nextA;
        if (TWO) LB = nextB;
    }
}

// output word i of a run from its entries of field F
template <int FMT, int F, class W>
__device__ __forceinline__ uint32_t entry_word(const uint32_t e[], int i)
{
    // a word is one pair, two singles or two pairs that take half of it each (the low halves of both), or four singles of a byte
    typedef Entries<FMT, F, W> P;
    constexpr bool one = P::kPair && P::kSecond == 16, four = !P::kPair && P::kSecond == 8;
    if (one) return e[i];
    if (four)
        return __builtin_amdgcn_perm(__builtin_amdgcn_perm(e[4 * i + 3], e[4 * i + 2], 0x0C0C0501u), __builtin_amdgcn_perm(e[4 * i + 1], e[4 * i], 0x0C0C0501u), 0x05040100u);
    return __builtin_amdgcn_perm(e[2 * i + 1], e[2 * i], 0x05040100u);
}

// word i of a plainly stored sign+mantissa run (two packed words, symbols in order) as it lies in the output
template <int FMT>
__device__ __forceinline__ uint32_t plain_word(uint32_t p0, uint32_t p1, int i)
{
    const uint32_t p = i < 2 ? p0 : p1;
    if (FMT == ZC_FMT_BF16) {
        const uint32_t t = __builtin_amdgcn_perm(0, p, (i & 1) ? 0x0C030C02u : 0x0C010C00u);      // bytes 2i, 2i+1 into bytes 0 and 2
        return t | (t << 8);
    }
    // four nibbles s m m m into four bytes s 0000 mmm
    const uint32_t h = p >> (16 * (i & 1));
    const uint32_t b = __builtin_amdgcn_perm(0, h, 0x0C010C00u), n = b | (b << 4);        // (the nibbles at bits 0, 8, 16, 24; above them others)
    return ((n << 4) & 0x80808080u) | (n & 0x07070707u);
}

// 32-bit word whose bytes are the next four 3-bit codes of v (first code in bits 2..0): a code is s, m1, m0 with the
// sign first in stream order, a byte of the result is s << 7 | m1 << 1 | m0
__device__ __forceinline__ uint32_t flat3_bytes(uint32_t v)
{
    const uint32_t a = (v & 0x7u) | ((v & 0x38u) << 5) | ((v & 0x1C0u) << 10) | ((v & 0xE00u) << 15);      // one code per byte
    return ((a << 7) & 0x80808080u) | (a & 0x02020202u) | ((a >> 2) & 0x01010101u);
}

// how the sign+mantissa field comes: table decoded with the exponents, by a flat code, raw, constant, or by E5M2's flat 3-bit
// code.  (Builds of their own: with a choice at run time the compiler waits for everything in flight before a row's words, the
// ones asked for two rows ahead included.)
constexpr int kSmTable = KIND_HUFF, kSmFlat = KIND_FLAT, kSmRaw = KIND_RAW, kSmConst = KIND_CONST, kSmFlat3 = 4;

// what a row takes from global memory besides its stream words
struct RowAhead { uint32_t m[4]; u32x4 base; };

struct ChunkOut {
    uint32_t nbytes, whole_rows, tail_bytes, tail_sym;       // tail_*: what this lane owns in the row after the whole ones
    uint8_t *dst;
    const uint8_t *base;
    __amdgpu_buffer_rsrc_t r1, ds, bs;
    uint32_t konst1;                                         // the constant symbol in every place of a word
};

template <int FMT, int R, int SM, bool XOR, class W>
__device__ __forceinline__ void pair_rows(PairStream &A, PairStream &B, const PairCanon *C, const ChunkOut &o, uint32_t lane)
{
    constexpr int NP = Fmt<FMT>::G;                              // entries of a run, at most
    constexpr bool TWO = SM == kSmTable;
    // (With several wavefronts per SIMD it is the number of instructions alone: 2,048 BF16 chunks 200 | 257 us.  Two fields and two
    // wavefronts: 1,526 chunks of a delta 314 | 303, but 3,052, three of them, 436 | 454.)
    constexpr bool kAhead = W::kLoop != kWait;
    constexpr int NA = kLookups<FMT, 0, R, W>, NB = kLookups<FMT, 1, R, W>;
    constexpr uint32_t EX = kExponentBits<FMT>;
    const uint32_t rows = o.whole_rows;
    Late LA, LB;
    // sign+mantissa words of a row (flat: one per 32 bits of symbols, rows of 64 words; raw: a lane's eight bytes) and the base
    // of a delta.  Row offsets go into the scalar operand, which is not range checked, so they never leave the whole rows.
    // E5M2's flat code: a lane's word q is word 64 * q + lane, two rows take three; past the stream's end zeros come back.
    auto fetch_flat3 = [&](uint32_t pair, RowAhead &f) {
#pragma unroll
        for (int k = 0; k < 3; k++) f.m[k] = __builtin_amdgcn_raw_buffer_load_b32(o.r1, (int)(lane * 4 + (pair * 3 + k) * 256), 0, 0);
    };
    auto fetch = [&](uint32_t row, RowAhead &f) {
        row = row < rows ? row : rows - 1;
        if (SM == kSmFlat) {
#pragma unroll
            for (int h = 0; h < 2; h++) f.m[h] = __builtin_amdgcn_raw_buffer_load_b32(o.r1, (int)(lane * 4), (int)((row * 2 + h) * 256), 0);
        }
        if (SM == kSmRaw) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(o.r1, (int)(lane * 8), (int)(row * 512), 0);
            f.m[0] = v.x; f.m[1] = v.y;
        }
        if (SM == kSmConst) { f.m[0] = o.konst1; f.m[1] = o.konst1; }
        if (XOR) f.base = __builtin_amdgcn_raw_buffer_load_b128(o.bs, (int)(lane * 16), (int)(row * 1024), 0);
    };
    // word i of a row's output, without the base; m: its sign+mantissa words (E5M2: its pair of rows' three)
    auto out_word = [&](uint32_t row, const uint32_t m[4], const uint32_t ea[], const uint32_t eb[], int i) {
        uint32_t mw;
        if (SM == kSmTable) mw = entry_word<FMT, 1, W>(eb, i);
        else if (SM == kSmFlat3) {
            // an even row's 48 bits start at bit 0 of the three words, an odd one's at bit 48
            const uint32_t lo = (row & 1) ? __builtin_amdgcn_alignbit(m[2], m[1], 16) : m[0];
            const uint32_t hi = (row & 1) ? m[2] >> 16 : m[1];
            mw = flat3_bytes(i == 0 ? lo : i == 1 ? lo >> 12 : i == 2 ? __builtin_amdgcn_alignbit(hi, lo, 24) : hi >> 4);
        } else {
            constexpr bool flat = SM == kSmFlat;
            constexpr int SB = Fmt<FMT>::SB == 8 ? 8 : 4;
            // (byte symbols are coded as bytes, most significant bit first, and their nibbles are in order then)
            mw = plain_word<FMT>(flat ? reverse_in_groups<SB>(m[0]) : m[0], flat ? reverse_in_groups<SB>(m[1]) : m[1], i);
        }
        return (entry_word<FMT, 0, W>(ea, i) & EX) | (mw & ~EX);
    };
    auto put_row = [&](uint32_t row, const uint32_t m[4], const uint32_t ea[], const uint32_t eb[], const u32x4 &base) {
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = out_word(row, m, ea, eb, i);
        if (XOR) v ^= base;
        store_row<2>(v, o.ds, lane, row);
    };
    // entries of a row and of the one before it, which is put together and stored while the next one's entries are looked up
    uint32_t ea[2][NP], eb[2][NP];
    RowAhead f[4];
    const bool ragged = o.nbytes % 1024 != 0;
    // ---- rows that need care: the first, until no lane is in the state of the start; the last before an incomplete one
    auto careful_row = [&](uint32_t row) {
        fetch(row, f[3]);
        if (SM == kSmFlat3) fetch_flat3(row / 2, f[2]);
        pair_run<FMT, R, TWO, W, true, true>(A, B, C, lane, ea[1], eb[1], (uint32_t)Fmt<FMT>::G, (ragged && row + 1 == rows) ? o.tail_sym : 1u);
        put_row(row, SM == kSmFlat3 ? f[2].m : f[3].m, ea[1], eb[1], f[3].base);
    };
    uint32_t row = 0;
    const uint32_t fast_end = ragged && rows ? rows - 1 : rows;
    // (an even number of rows: the fast loop starts at a pair of E5M2's flat code)
#pragma unroll 1
    while (row < rows && (row >= fast_end || row < 2 || (row & 1) || __any(A.c == 32 || (TWO && B.c == 32)))) {
        careful_row(row);
        row++;
    }
    // Four rows at a time, each row's words asked for four rows ahead (when the registers are free again: a copy of them would wait
    // for what is in flight).  The rings are looked at every kRows rows.  A segment's words go into the ring only when the next one
    // is asked for, and what waits for them waits for everything that was asked for before them: the rows in between are what
    // they have to arrive.
    constexpr uint32_t kRows = W::kRing / 4 / 64 / (Fmt<FMT>::G / R) >= 4 ? 4 : W::kRing / 4 / 64 / (Fmt<FMT>::G / R) >= 2 ? 2 : 1;
    if (row + 4 <= fast_end) {
        if (!W::kInFours) { pair_settle<W>(A, lane); A.pending = false; }
        if (TWO) { pair_settle<W>(B, lane); B.pending = false; }
        if (kAhead) {
            late_open<FMT, 0, NA, W>(LA, A);
            if (TWO) late_open<FMT, 1, NB, W>(LB, B);
        }
        // (kAhead: the row before the first is stored once more, from the same registers: it is what the first one's waits are filled with)
#pragma unroll
        for (uint32_t i = 0; i < (kAhead ? 3 : 4); i++) {
            fetch(row + i, f[i]);
            if (SM == kSmFlat3 && i % 2 == 0 && (i == 0 || !kAhead)) fetch_flat3((row + i) / 2, f[i]);
        }
        LateRoom late = {4 * LateRoom::kAgain, fast_end};
        auto block_row = [&](auto index, auto inside) {
            constexpr uint32_t i = decltype(index)::value, last = (i + 3) & 3;
            if (!kAhead) {
                pair_run<FMT, R, TWO, W, false, i % kRows == 0>(A, B, C, lane, ea[0], eb[0], 0, 0);
                put_row(row + i, SM == kSmFlat3 ? f[i & 2].m : f[i].m, ea[0], eb[0], f[i].base);
                if (SM == kSmFlat3 && i % 2 == 1) fetch_flat3((row + i + 3) / 2, f[i & 2]);
                fetch(row + i + 4, f[i]);
                return;
            }
            const uint32_t prev = row + i - 1;
            u32x4 v;
            late_run<FMT, R, TWO, W, i % kRows == 0, i, decltype(inside)::value>(LA, LB, A, B, C, lane, ea[i & 1], eb[i & 1], late, [&](int g, int periods) {
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    if (k * periods / 4 != g) continue;
                    v[k] = out_word(last, SM == kSmFlat3 ? f[last & 2].m : f[last].m, ea[last & 1], eb[last & 1], k);
                    asm volatile("" : "+v"(v[k]));               // (here, not at the store)
                    if (k < 3) continue;
                    if (XOR) v ^= f[last].base;
                    store_row<2>(v, o.ds, lane, prev);
                }
            });
            if (SM == kSmFlat3 && last % 2 == 1) fetch_flat3((prev + 3) / 2, f[last & 2]);
            fetch(prev + 4, f[last]);
        };
        auto block = [&](auto inside) {
            block_row(std::integral_constant<uint32_t, 0>(), inside);
            block_row(std::integral_constant<uint32_t, 1>(), inside);
            block_row(std::integral_constant<uint32_t, 2>(), inside);
            block_row(std::integral_constant<uint32_t, 3>(), inside);
            row += 4;
        };
        if constexpr (W::kLoop == kSteady) {
#pragma unroll 1
            while (row + 4 <= fast_end) block(std::false_type());
        } else if constexpr (W::kLoop == kLate) {
            // as long as one period in twelve goes wrong at most, but for a few at first
#pragma unroll 1
            while (row + 4 <= late.end) {
                block(std::false_type());
                late.room = late.room + 4 * Fmt<FMT>::G / R < 8 * LateRoom::kAgain ? late.room + 4 * Fmt<FMT>::G / R : 8 * LateRoom::kAgain;
            }
        }
        if constexpr (W::kLoop != kSteady) {
#pragma unroll 1
            while (row + 4 <= fast_end) block(std::true_type());
        }
        if (kAhead) {
            put_row(row - 1, SM == kSmFlat3 ? f[2].m : f[3].m, ea[1], eb[1], f[3].base);
            late_close<kTwice<FMT, 0, NA, W>>(LA, A);
            if (TWO) late_close<kTwice<FMT, 1, NB, W>>(LB, B);
        }
    }
#pragma unroll 1
    for (; row < rows; row++) careful_row(row);
    if (!ragged) return;
    // ---- the incomplete last row: a lane owns a whole run, part of one or nothing
    uint32_t m[4] = {o.konst1, o.konst1, 0, 0};
    pair_run<FMT, R, TWO, W, true, true>(A, B, C, lane, ea[0], eb[0], o.tail_sym, 0u);
    if (SM == kSmFlat3) {
        // Steps of eight codes, 24 bits, two per row.  Lanes in step ask for words 0 .. 4 at steps 0 .. 4 and then at all but
        // every fourth step, so of the two words a row's 48 bits lie in, the first has been asked for by every lane before the
        // row's first step (the chunk's first row: at it) and the second at that step (there: at the next), by the lanes that
        // own a symbol then.
        const uint64_t own0 = __ballot(o.tail_sym > 0), own1 = __ballot(o.tail_sym > 8);
        const uint32_t word = rows / 2 * 3 + (rows & 1);
        uint32_t at0 = word * 64 + lane, at1 = (word + 1) * 64 + prefix_count64(own0);
        bool has0 = true, has1 = o.tail_sym > 0;
        if (rows == 0) { at0 = prefix_count64(own0); at1 = (uint32_t)__popcll(own0) + prefix_count64(own1); has0 = o.tail_sym > 0; has1 = o.tail_sym > 8; }
        const uint32_t w0 = __builtin_amdgcn_raw_buffer_load_b32(o.r1, (int)(has0 ? at0 * 4 : 0xFFFFFFF0u), 0, 0);
        const uint32_t w1 = __builtin_amdgcn_raw_buffer_load_b32(o.r1, (int)(has1 ? at1 * 4 : 0xFFFFFFF0u), 0, 0);
        m[0] = w0; m[1] = (rows & 1) ? w0 : w1; m[2] = w1;
    } else {
        uint32_t at = rows * 2 * 64;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            if (SM == kSmFlat) {
                const bool owner = (uint32_t)(h * (32 / Fmt<FMT>::SB)) < o.tail_sym;
                const uint64_t bm = __ballot(owner);
                m[h] = __builtin_amdgcn_raw_buffer_load_b32(o.r1, (int)(owner ? (at + prefix_count64(bm)) * 4 : 0xFFFFFFF0u), 0, 0);
                at += (uint32_t)__popcll(bm);
            } else if (SM == kSmRaw) m[h] = __builtin_amdgcn_raw_buffer_load_b32(o.r1, (int)(((rows * 64 + lane) * 2 + h) * 4), 0, 0);
        }
    }
    if (o.tail_bytes) {
        uint4 v = make_uint4(out_word(rows, m, ea[0], eb[0], 0), out_word(rows, m, ea[0], eb[0], 1), out_word(rows, m, ea[0], eb[0], 2), out_word(rows, m, ea[0], eb[0], 3));
        const uint32_t at = rows * 1024 + lane * 16;
        if (XOR) v = xor4(v, load_run(o.base + at, o.tail_bytes));
        store_run(o.dst + at, v, o.tail_bytes);
    }
}

template <class... W> struct Choice {};
template <int FMT, Launch L> struct Builds;
// FP8 E4M3: codes of at most eight bits, longer ones
template <> struct Builds<ZC_FMT_FP8_E4M3, kFew> { typedef Choice<Build<1024, kLate, kWholePairs>, Build<1024, kSteady, kWhole>> All; };
// E5M2, BF16: codes of more than eight bits, all others.  (Two of E5M2's 32 symbols take ten bits at most in the mean, two of FP8's sixteen eight.)
template <> struct Builds<ZC_FMT_FP8_E5M2, kFew> { typedef Choice<Build<1024, kSteady, kWhole>, Build<1024, kInside, kPairs15>> All; };
template <> struct Builds<ZC_FMT_FP8_E5M2, kMany> { typedef Choice<Build<512, kWait, kPairs13>> All; };
template <> struct Builds<ZC_FMT_BF16, kFew> { typedef Choice<Build<1024, kLate, kWhole>, Build<1024, kInside, kPairs15>> All; };
// BF16 with two fields: see choose_build; the last two are for a tensor with one among others with two
template <> struct Builds<ZC_FMT_BF16, kFewTwo> {
    typedef Choice<Build<512, kLate, kPairs11, kWhole>, Build<512, kLate, kWhole, kShort12>, Build<512, kLate, kWhole, kSingles12>, Build<512, kInside, kPairs15, kShort12>,
                   Build<1024, kLate, kWhole>, Build<1024, kInside, kPairs15>> All;
};
template <> struct Builds<ZC_FMT_BF16, kMany> { typedef Choice<Build<512, kWait, kPairs12, kSingles12>> All; };
template <> struct Builds<ZC_FMT_BF16, kManyTwo> { typedef Choice<Build<512, kLate, kPairs12, kSingles12>> All; };
template <> struct Builds<ZC_FMT_FP8_E4M3_BYTES, kFew> { typedef Choice<Build<1024, kLate, kWhole>> All; };
template <> struct Builds<ZC_FMT_FP8_E4M3_BYTES, kFewTwo> { typedef Choice<Build<2048, kWait, kSingles12, kSingles12>> All; };
template <> struct Builds<ZC_FMT_FP8_E4M3_BYTES, kMany> { typedef Choice<Build<512, kWait, kSingles12, kSingles12>> All; };

// Refill periods and sign+mantissa fields that a launch's build I is for
template <int FMT, Launch L> constexpr bool is_for(uint32_t I, int R, int SM)
{
    if (FMT == ZC_FMT_FP8_E5M2) return SM == kSmFlat3 && (L == kMany || (I == 0) == (R == 2));
    if (FMT == ZC_FMT_FP8_E4M3) return (SM == kSmFlat || SM == kSmRaw) && R == (I == 0 ? 4 : 2);
    if (SM == kSmFlat3 || (L == kFew && SM == kSmTable)) return false;
    if (FMT == ZC_FMT_FP8_E4M3_BYTES || L == kMany || L == kManyTwo) return true;
    if (L == kFew) return (I == 0) == (R == 2);
    return (I < 4) == (SM == kSmTable) && (I == 3 || I == 5) == (R != 2);
}
template <int FMT, Launch L>
__device__ __forceinline__ uint32_t choose_build(const PairCanon *C, uint32_t R, bool two)
{
    if (FMT == ZC_FMT_FP8_E4M3) return R == 2;
    if (FMT == ZC_FMT_FP8_E5M2 || (FMT == ZC_FMT_BF16 && L == kFew)) return L == kFew && R != 2;
    if (FMT == ZC_FMT_BF16 && L == kFewTwo) {
        if (!two) return R != 2 ? 5 : 4;
        if (R != 2) return 3;
        // The exponents have the whole table, but where the other field has codes of more than 12 bits and they have one of a single bit
        // (deltas): then they take so few bits that pairs by 11 are unresolved in 1.5 % of the periods (weights: 39 %), and leave the LDS to
        // the other field.  Eight chunks of 128 KiB, exponents in pairs by 11 or 13 bits | the whole table, us: weights, whose sign+mantissa
        // codes have nine bits, 64 KiB 70 | 58, 200 tensors of 256 KiB 205 | 201; exponents spread with scale 8, signs+mantissas with scale 60:
        // 264 | 107, with scale 2, codes of 16 bits: 268 | 114.  A tensor with one such field beside those: pairs by 11 bits | as on its own:
        // 8 MiB 173 | 117.
        if (uniform32(C[1].limit[12]) >= 65536u) return 1;
        return uniform32(C[0].limit[1]) != 0 ? 0 : 2;
    }
    return 0;
}

}  // namespace

// (longs: only where there are whole tables)
struct PairShared { TensorDev d; PairCanon canon[2]; uint32_t wave_count[4][17], flat3; };
struct FewShared : PairShared { LongCodes longs; };
template <Launch L> constexpr uint32_t kSharedBytes = L == kFew || L == kFewTwo ? sizeof(FewShared) : sizeof(PairShared);

// Build I of a launch's and its number, for f
template <int FMT, Launch L, uint32_t I, class F, class W, class... Rest>
__device__ __forceinline__ void with_build(Choice<W, Rest...>, uint32_t which, const F &f)
{
    if constexpr (sizeof...(Rest) == 0) f(W(), std::integral_constant<uint32_t, I>());
    else if (which == I) f(W(), std::integral_constant<uint32_t, I>());
    else with_build<FMT, L, I + 1>(Choice<Rest...>(), which, f);
}
// One wavefront per chunk, `chunks` of them per workgroup (whose wavefronts build the tables together) around one copy of the tables.
// Bound by the instructions of a chunk's chain up to about a thousand chunks (one wavefront per SIMD), then by all instructions, and
// from BF16's eight thousand on by HBM.  MI355X, GPU time, us, 200 chunks of 256 KiB, with tables by 12 - 14 bits and every period's word
// waited for | now: FP8 182 | 134 (201 instructions per row of 1 KiB, the table's construction included), BF16 129 | 118, E5M2 296 | 232 (307
// instructions), byte symbols 232 | 128, BF16 deltas 267 | 194; chunks of 16 KiB: E5M2 38 | 24, deltas 38 | 26, byte symbols 25 | 17; a single
// chunk of BF16 weights whose sign+mantissa codes differ in length: 64 KiB: 66 | 58, 256 KiB: 197 | 192.
template <int FMT, bool XOR, Launch L>
__global__ __launch_bounds__(1024) void k_decode_pairs(const TensorDev *descs, const WorkItem *work, TensorDev single, int use_single, uint32_t first_slot,
                                                       uint32_t chunks, uint32_t lds_tables_and_rings)
{
    using F_ = Fmt<FMT>;
    // all LDS in one piece, sized by the host, with field 0's table at its start (so that its entries need no base address);
    // then field 1's table where it has one, the rings, and what the workgroup shares besides
    extern __shared__ __attribute__((aligned(16))) char lds[];
    FewShared &sh = *reinterpret_cast<FewShared *>(lds + lds_tables_and_rings);              // (kMany, kManyTwo: a PairShared)
    PairCanon *const canon = sh.canon;
    uint32_t(*const wave_count)[17] = sh.wave_count;
    WorkItem it;
    if (use_single) { it.tensor = 0; it.first = first_slot + blockIdx.x * chunks; }
    else it = work[blockIdx.x];
    if (threadIdx.x == 0) { sh.d = use_single ? single : descs[it.tensor]; sh.flat3 = 1; }
    __syncthreads();
    const TensorDev &d = sh.d;
    constexpr uint32_t kAlphabet = 1u << F_::SB;
    const uint32_t p0 = uniform32(d.period[0]), p1 = uniform32(d.period[1]), kind1 = uniform32(d.kind[1]);
    if (FMT == ZC_FMT_FP8_E5M2) {
        // the sign+mantissa table must be the flat 3-bit code over the values 0..7
        if (threadIdx.x < 256 && d.comp[d.table_off[1] + threadIdx.x] != (threadIdx.x < 8 ? 3 : 0)) sh.flat3 = 0;
        __syncthreads();
    }
    const bool two = FMT != ZC_FMT_FP8_E5M2 && kind1 == KIND_HUFF;
    // whole workgroup; the host never asks for these
    if (uniform32(d.kind[0]) != KIND_HUFF || (p0 != 2 && p0 != 4 && p0 != 8) || (two && (p1 != p0 || L == kFew))) return;
    if (FMT == ZC_FMT_FP8_E5M2 && (uniform32(d.mode[1]) != ZC_MODE_HUFF || !sh.flat3)) return;
    if (FMT == ZC_FMT_FP8_E4M3 && ((kind1 != KIND_FLAT && kind1 != KIND_RAW) || p0 == 8)) return;
    build_canon(canon[0], wave_count, d.comp + d.table_off[0], kAlphabet);
    if (two) build_canon(canon[1], wave_count, d.comp + d.table_off[1], kAlphabet);
    const uint32_t which = choose_build<FMT, L>(canon, p0, two);
    typedef typename Builds<FMT, L>::All All;
    with_build<FMT, L, 0>(All(), which, [&](auto build, auto) __attribute__((always_inline)) {
        typedef decltype(build) W;
        build_entries<FMT, 0, W>(lds, canon[0], sh.longs);
        if (FMT != ZC_FMT_FP8_E5M2 && FMT != ZC_FMT_FP8_E4M3 && L != kFew && two) build_entries<FMT, 1, W>(lds + kTableBytes<0, W>, canon[1], sh.longs);
    });

    const uint32_t lane = threadIdx.x & 63, wave = uniform32(threadIdx.x >> 6);
    if (wave >= chunks) return;
    const uint32_t slot = uniform32(it.first + wave);
    uint32_t chunk = slot;
    const uint32_t *ids = reinterpret_cast<const uint32_t *>(uniform64((uint64_t)d.ids));
    if (ids) {
        // a list of chunk ids: slot i of the output takes chunk ids[i]; an id out of range leaves its slot alone
        if (slot >= uniform32(d.n_ids)) return;
        chunk = uniform32(ids[slot]);
    }
    if (chunk >= uniform32(d.n_chunks)) return;
    const uint32_t cb = uniform32(d.chunk_bytes);
    const uint64_t E = (uint64_t)cb * 8 / F_::EB, before = (uint64_t)chunk * E, n_elems = uniform64(d.n_elems);
    if (n_elems <= before) return;
    const uint32_t n = (uint32_t)(n_elems - before < E ? n_elems - before : E);
    ChunkOut o;
    o.nbytes = (uint32_t)((uint64_t)n * F_::EB / 8);         // (n * EB passes 32 bits from chunks of 512 MiB on)
    o.whole_rows = o.nbytes / 1024;
    const uint32_t tail_at = o.whole_rows * 1024 + lane * 16;
    o.tail_bytes = o.nbytes > tail_at ? (o.nbytes - tail_at < 16u ? o.nbytes - tail_at : 16u) : 0u;
    o.tail_sym = (o.tail_bytes * 8 / F_::EB + F_::GRP - 1) / F_::GRP;          // a last partial group of values is one symbol
    const uint8_t *comp = reinterpret_cast<const uint8_t *>(uniform64((uint64_t)d.comp));
    const uint64_t payload = uniform64(d.payload_off), total = uniform64(d.total_bytes);
    const uint8_t *sp[2];
    uint32_t sb[2];
#pragma unroll
    for (int f = 0; f < 2; f++)
        if (!stream_range(d, comp, f, chunk, payload, total, sp[f], sb[f])) return;      // damaged index: leave the chunk alone
    // a plainly stored sign+mantissa field takes 512 bytes per row (E5M2's three bits per value 384): a shorter stream (a damaged
    // index) leaves the chunk alone.  It must not be read either: but for E5M2's, rows are addressed through the scalar offset,
    // which is not range checked
    if ((kind1 == KIND_FLAT || kind1 == KIND_RAW || FMT == ZC_FMT_FP8_E5M2) && sb[1] < o.whole_rows * (FMT == ZC_FMT_FP8_E5M2 ? 384u : 512u)) return;
    o.dst = reinterpret_cast<uint8_t *>(uniform64((uint64_t)d.dst)) + (uint64_t)slot * cb;
    o.base = XOR ? reinterpret_cast<const uint8_t *>(uniform64((uint64_t)d.base)) + (uint64_t)chunk * cb : comp;
    o.r1 = make_rsrc(sp[1], sb[1]);
    o.ds = make_rsrc(o.dst, o.nbytes);
    o.bs = make_rsrc(o.base, XOR ? o.nbytes : 0);
    o.konst1 = (uint32_t)splat(uniform32(d.konst[1]), F_::SB);
    const bool first = o.whole_rows > 0 || o.tail_sym > 0;       // does this lane own a symbol at step 0?
    with_build<FMT, L, 0>(All(), which, [&](auto build, auto number) __attribute__((always_inline)) {
        typedef decltype(build) W;
        PairStream A, B;
        const uint32_t rings = rings_at<W>(two) + wave * (two ? 2 : 1) * W::kRing * 4;               // (two: there is a second table)
        A.ring = rings; A.rs = make_rsrc(sp[0], sb[0]);
        B.ring = rings + W::kRing * 4; B.rs = o.r1;
        constexpr uint32_t KA = Entries<FMT, 0, W>::kBits, KB = Entries<FMT, 1, W>::kBits;
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) {
            A.limit[i] = i + KA < 15 ? uniform32(canon[0].limit[i + KA + 1]) : 0u;
            B.limit[i] = two && i + KB < 15 ? uniform32(canon[1].limit[i + KB + 1]) : 0u;
        }
        pair_open<W>(A, lane, first);
        if (two) pair_open<W>(B, lane, first);
        const uint32_t sm = FMT == ZC_FMT_FP8_E5M2 ? (uint32_t)kSmFlat3 : kind1;
#define ZC_ROWS(R, SM) case (R) * 8 + (SM): if constexpr (is_for<FMT, L>(decltype(number)::value, R, SM)) pair_rows<FMT, R, SM, XOR, W>(A, B, canon, o, lane); break
        switch (p0 * 8 + sm) {
            ZC_ROWS(2, kSmTable); ZC_ROWS(4, kSmTable); ZC_ROWS(8, kSmTable);
            ZC_ROWS(2, kSmFlat); ZC_ROWS(4, kSmFlat); ZC_ROWS(8, kSmFlat);
            ZC_ROWS(2, kSmRaw); ZC_ROWS(4, kSmRaw); ZC_ROWS(8, kSmRaw);
            ZC_ROWS(2, kSmConst); ZC_ROWS(4, kSmConst); ZC_ROWS(8, kSmConst);
            ZC_ROWS(2, kSmFlat3); ZC_ROWS(4, kSmFlat3); ZC_ROWS(8, kSmFlat3);
        }
#undef ZC_ROWS
    });
}

// LDS that a launch's tables and rings take: its largest build's
template <class... W> constexpr uint32_t most_lds(Choice<W...>, bool two, uint32_t chunks)
{
    uint32_t most = 0;
    for (const uint32_t n : {(two && W::template kTable<1> != kNone ? rings_at<W>(true) + chunks * 2 * W::kRing * 4 : rings_at<W>(false) + chunks * W::kRing * 4) ...}) most = n > most ? n : most;
    return most;
}
template <int FMT, Launch L>
static int launch_pairs_x(bool two, bool xor_delta, uint32_t chunks, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work, const TensorDev &s, int use_single,
                          uint32_t first_slot, hipStream_t st)
{
    typedef typename Builds<FMT, L>::All All;
    const uint32_t lds = most_lds(All(), two, chunks), all = lds + kSharedBytes<L>;
    static_assert(L == kMany || L == kManyTwo || most_lds(All(), L == kFewTwo, 4) + kSharedBytes<L> <= 160 * 1024, "a compute unit's LDS");
    // (whole tables by 1,024 threads; small ones by eight wavefronts, four where a call has more workgroups than the compute units hold
    // of eight: 1,500 BF16 tensors of one chunk of 100,000 bytes: 255 | 213 us)
    const uint32_t few = FMT == ZC_FMT_FP8_E4M3_BYTES && L == kFewTwo ? 256 : 1024;
    const dim3 grid(n_work), block(L == kFew || L == kFewTwo ? few : chunks > 4 || n_work <= 4 * 256 ? 512 : 256);
    if (xor_delta) hipLaunchKernelGGL((k_decode_pairs<FMT, true, L>), grid, block, all, st, d_descs, d_work, s, use_single, first_slot, chunks, lds);
    else hipLaunchKernelGGL((k_decode_pairs<FMT, false, L>), grid, block, all, st, d_descs, d_work, s, use_single, first_slot, chunks, lds);
    return (int)hipGetLastError();
}

}  // namespace zc

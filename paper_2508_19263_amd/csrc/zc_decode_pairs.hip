// 64-lane decoders with large lookup tables (a8, a9): BF16, FP8 (E4M3, E5M2, byte symbols); any chunks, a short last one and
// lists of chunk ids included; exponent field table decoded with a refill period of 2, 4 or 8, sign+mantissa field table decoded
// on the same period or stored plainly (flat code, raw, constant; E5M2: its flat 3-bit code).
//
// A chunk is one wavefront's serial chain: window, lookups, refill (whose word depends on how many lanes take one), window.
// Every link is an LDS round trip with the arithmetic that gives its address, about 140 cycles, and a call of few chunks takes as long
// as one chunk's chain.  So
//   - exponents are looked up in pairs: the next 13 stream bits give the next TWO symbols, which halves the lookups and their
//     address and shift instructions.  An entry already is the pair's part of an output word.  (Sign+mantissa codes and byte
//     symbols are too long for pairs: singles, by 12 bits.)
//   - the refill word is asked for before the lookups' entries are checked: an entry that did not resolve (a pair longer than
//     13 bits, a code longer than the index) sends the wavefront through the period once more.
//   - two table-decoded fields go through the chain side by side.
#include <hip/hip_runtime.h>

#include "zc_internal.h"
#include "zc_device.h"
#include "zc_decode_device.h"

namespace zc {

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

// How the table entries of field F of format FMT are laid out.  put: a symbol at its place in an output word (kFirst: the bits
// it can take).  The length (a pair's, or a single's) lies in bits the output's two fields leave to each other, at kLen; it is
// added by the byte it lies in where it has one: a symbol's bit above it leaves the low 7 bits of a sum alone.  An entry that
// does not resolve has length 0, so that the lookups after it in the period do not resolve either and the last one tells.
// kPair: 32-bit entries of two symbols, the second kSecond bits above the first; kUnresolved (the sign bit) where the pair does
// not fit the index, which has the first symbol alone, its length at kLen1 (0 there: longer than the index).
// Else 16-bit entries, 0 for a code longer than the index.
template <int FMT, int F> struct Entries;
template <> struct Entries<ZC_FMT_BF16, 0> {
    static constexpr bool kPair = true;
    static constexpr uint32_t kFirst = 0x7F80u;
    static constexpr int kSecond = 16, kLen = 0, kLen1 = 16;
    static constexpr bool kNoise = true;                      // a symbol's bit shares the length's byte
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return s << 7; }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return add_byte<0>(c, e); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return shr_byte<0>(x, e); }
};
template <> struct Entries<ZC_FMT_BF16, 1> {
    static constexpr bool kPair = false;
    static constexpr uint32_t kFirst = 0x807Fu;
    static constexpr int kSecond = 16, kLen = 8, kLen1 = 0;
    static constexpr bool kNoise = true;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return ((s & 0x80u) << 8) | (s & 0x7Fu); }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return add_byte<1>(c, e); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return shr_byte<1>(x, e); }
};
// one value per byte: the pair in bytes 0 and 1, its length in byte 2, the first symbol's in byte 3
template <int FMT> struct PairPerHalf {
    static constexpr bool kPair = true;
    static constexpr uint32_t kFirst = 0xFFu;
    static constexpr int kSecond = 8, kLen = 16, kLen1 = 24;
    static constexpr bool kNoise = false;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return FMT == ZC_FMT_FP8_E4M3 ? (s << 3) & 0x78u : (s << 2) & 0x7Cu; }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return add_byte<2>(c, e); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return shr_byte<2>(x, e); }
};
template <> struct Entries<ZC_FMT_FP8_E4M3, 0> : PairPerHalf<ZC_FMT_FP8_E4M3> {};
template <> struct Entries<ZC_FMT_FP8_E5M2, 0> : PairPerHalf<ZC_FMT_FP8_E5M2> {};
template <> struct Entries<ZC_FMT_FP8_E4M3, 1> : Entries<ZC_FMT_BF16, 1> {};     // (never table decoded here)
template <> struct Entries<ZC_FMT_FP8_E5M2, 1> : Entries<ZC_FMT_BF16, 1> {};
// byte symbols: a symbol is two values, half an output word (exponent bits 0x78 of every byte, sign+mantissa bits 0x87)
template <> struct Entries<ZC_FMT_FP8_E4M3_BYTES, 0> {
    static constexpr bool kPair = false;
    static constexpr uint32_t kFirst = 0x7878u;
    static constexpr int kSecond = 16, kLen = 7, kLen1 = 0;
    static constexpr bool kNoise = false;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return ((s & 15u) << 3) | ((s & 0xF0u) << 7); }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return c + ((e >> 7) & 15u); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return x >> ((e >> 7) & 15u); }
};
template <> struct Entries<ZC_FMT_FP8_E4M3_BYTES, 1> {
    static constexpr bool kPair = false;
    static constexpr uint32_t kFirst = 0x8787u;
    static constexpr int kSecond = 16, kLen = 3, kLen1 = 0;
    static constexpr bool kNoise = false;
    static __device__ __forceinline__ uint32_t put(uint32_t s) { return (s & 7u) | ((s & 8u) << 4) | ((s & 0x70u) << 4) | ((s & 0x80u) << 8); }
    static __device__ __forceinline__ uint32_t add(uint32_t c, uint32_t e) { return c + ((e >> 3) & 15u); }
    static __device__ __forceinline__ uint32_t shift(uint32_t x, uint32_t e) { return x >> ((e >> 3) & 15u); }
};
constexpr uint32_t kUnresolved = 0x80000000u;
__device__ __forceinline__ uint32_t first_len(uint32_t e, int shift) { return (e >> shift) & 15u; }
// bits of an output word that come from the exponent entries
template <int FMT> constexpr uint32_t kExponentBits = FMT == ZC_FMT_BF16 ? 0x7F807F80u : FMT == ZC_FMT_FP8_E5M2 ? 0x7C7C7C7Cu : 0x78787878u;
// Words of a stream's ring: long where a workgroup of four wavefronts has a compute unit to itself (half of that where two
// fields share it), short with eight wavefronts per workgroup and several workgroups per compute unit
constexpr uint32_t kLongRing = 4096, kLongRingTwo = 2048, kShortRing = 512;

// Stream bits a lookup goes by.  Chance that one of 64 lanes finds a pair unresolved, for weights of the kinds the codec is meant
// for: BF16 exponents 17 % with 12 bits and 9 % with 13, FP8 E4M3 5 % with 13 and 1.4 % with 14, E5M2 (a wide spread of exponents)
// 31 % with 13; BF16 deltas' sign+mantissa pairs and byte symbols' would be unresolved nearly always.  Singles by 12 bits: 5 - 25 %.
// FP8 E4M3 comes here only in calls of few chunks, which have the LDS for 64 KiB of table; BF16 saves half the table for more
// workgroups per compute unit in the others (8,192 chunks: 787 against 829 us; 1,000 chunks with the long ring: 152 against 141).
template <int FMT, int F, uint32_t RW> constexpr uint32_t kIndexBits = !Entries<FMT, F>::kPair ? 12u : FMT == ZC_FMT_FP8_E4M3 ? 14u : FMT == ZC_FMT_BF16 && RW == kShortRing ? 12u : 13u;
// bytes of a field's table
template <int FMT, int F, uint32_t RW> constexpr uint32_t kTableBytes = (Entries<FMT, F>::kPair ? 4u : 2u) << kIndexBits<FMT, F, RW>;

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

template <int FMT, int F, uint32_t RW>
__device__ __forceinline__ void build_entries(char *table, const PairCanon &C)
{
    typedef Entries<FMT, F> P;
    constexpr uint32_t K = kIndexBits<FMT, F, RW>, entries = 1u << K;
    const uint32_t lane = threadIdx.x & 63, mine = lane < 17 ? C.limit[lane] : 0u;
    uint32_t limit[K + 1];
#pragma unroll
    for (uint32_t l = 1; l <= K; l++) limit[l] = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)l);
    uint32_t *const pairs = reinterpret_cast<uint32_t *>(table);
    uint16_t *const singles = reinterpret_cast<uint16_t *>(table);
    // A thread's entries have the low eight bits of their index in common, so a code of at most eight bits can be looked up once for
    // all of them: FP8 E4M3, 64 KiB of table, chunks of 32 KiB 52 -> 45 us, 1,000 E5M2 tensors of 2 KB 24.5 -> 21.5.  The other formats have
    // longer codes in some lane of nearly every wavefront, which would make it 3 - 5 % slower for small chunks.
    constexpr bool kOnce = FMT == ZC_FMT_FP8_E4M3 || FMT == ZC_FMT_FP8_E5M2;
    uint32_t len = 0, e = 0;
    for (uint32_t i = threadIdx.x; i < entries; i += blockDim.x) {
        if (!kOnce || len == 0 || len > 8) {
            const uint32_t w = __brev(i) >> 16;                  // the stream bits in code order, left aligned
            len = 1;
#pragma unroll
            for (uint32_t l = 1; l <= K; l++) len += w >= limit[l];
            e = P::kPair ? kUnresolved : 0u;
            if (len <= K) e |= P::put(C.sorted[(C.rebase[len] + (w >> (16 - len))) & 255u]) | (len << (P::kPair ? P::kLen1 : P::kLen));
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
    u32x4 pv[4];                             // the newest segment, on its way into the ring
    uint32_t ring;                           // LDS address
    uint32_t limit[4];                       // limits of the lengths from the index's on (uniform), see long_symbol
    __amdgpu_buffer_rsrc_t rs;
};

// Ring of RW words per wavefront and field, refilled SEG = RW / 4 words at a time; see ring_service in zc_decode_s64.hip
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
template <uint32_t RW> struct Segment {
    static constexpr uint32_t kWords = RW / 4, B = kWords >= 256 ? 4 : kWords / 64, kPieces = kWords / (64 * B);
    static_assert((B == 1 || B == 2 || B == 4) && kPieces >= 1 && kPieces <= 4, "whole loads");
};

template <uint32_t RW>
__device__ __forceinline__ void pair_open(PairStream &S, uint32_t lane, bool owner)
{
    constexpr uint32_t B = Segment<RW>::B;
    constexpr uint32_t kLoads = RW / (64 * B), kAtOnce = kLoads < 8 ? kLoads : 8;
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
    S.c = 32; S.wpos = (uint32_t)__popcll(takers); S.wbase = 0; S.pslot = 0; S.pending = false;
#pragma unroll
    for (int i = 0; i < 4; i++) S.pv[i] = u32x4{0, 0, 0, 0};
}

// the segment on its way, when there is one, into its place
template <uint32_t RW>
__device__ __forceinline__ void pair_settle(PairStream &S, uint32_t lane)
{
    constexpr uint32_t B = Segment<RW>::B;
    if (S.pending) {
#pragma unroll
        for (uint32_t q = 0; q < Segment<RW>::kPieces; q++) ring_write<B>(S.ring + (S.pslot + (q * 64 + lane) * B) * 4, S.pv[q]);
    }
}

template <uint32_t RW>
__device__ __forceinline__ void pair_service(PairStream &S, uint32_t lane)
{
    constexpr uint32_t SEG = Segment<RW>::kWords, B = Segment<RW>::B;
    if (S.wpos - S.wbase >= SEG) {
        pair_settle<RW>(S, lane);
#pragma unroll
        for (uint32_t q = 0; q < Segment<RW>::kPieces; q++) S.pv[q] = segment_load<B>(S.rs, (S.wbase + RW + (q * 64 + lane) * B) * 4);
        S.pslot = S.wbase & (RW - 1);
        S.wbase += SEG;
        S.pending = true;
    }
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

template <int FMT, int F, uint32_t RW>
__device__ __forceinline__ uint32_t entry_at(uint32_t x)
{
    constexpr uint32_t mask = (1u << kIndexBits<FMT, F, RW>) - 1, table = F == 0 ? 0u : kTableBytes<FMT, 0, RW>;
    if (Entries<FMT, F>::kPair) return lds_word(((x << 2) & (mask << 2)) + table);
    return *reinterpret_cast<const LdsHalf *>(((x << 1) & (mask << 1)) + table);
}

// a period's entries, N of them; c: bits used before it, returns them after it (in the low 7 bits)
template <int FMT, int F, int N, uint32_t RW>
__device__ __forceinline__ uint32_t look_up(uint32_t c, uint32_t x, uint32_t e[N])
{
#pragma unroll
    for (int i = 0; i < N; i++) {
        e[i] = entry_at<FMT, F, RW>(x);
        c = Entries<FMT, F>::add(c, e[i]);
        if (i + 1 < N) x = Entries<FMT, F>::shift(x, e[i]);
    }
    return c;
}
template <int FMT, int F>
__device__ __forceinline__ bool unresolved(uint32_t e) { return Entries<FMT, F>::kPair ? (int)e < 0 : e == 0; }

// The same where an entry does not resolve in some lane.
template <int FMT, int F, int N, uint32_t RW>
__device__ __forceinline__ uint32_t look_up_slowly(const PairStream &S, const PairCanon &C, uint32_t x, uint32_t e[N])
{
    typedef Entries<FMT, F> P;
    constexpr uint32_t K = kIndexBits<FMT, F, RW>;
    uint32_t c = S.c;
#pragma unroll
    for (int i = 0; i < N; i++) {
        uint32_t a = entry_at<FMT, F, RW>(x), len;
        if (P::kPair) {
            // both symbols one after the other in every lane
            uint32_t l1 = first_len(a, P::kLen1), s1 = a & P::kFirst;
            if (__any(l1 == 0)) { if (l1 == 0) s1 = P::put(long_symbol<K>(S, C, x, l1)) & P::kFirst; }
            const uint32_t y = x >> l1, b = entry_at<FMT, F, RW>(y);
            uint32_t l2 = first_len(b, P::kLen1), s2 = b & P::kFirst;
            if (__any(l2 == 0)) { if (l2 == 0) s2 = P::put(long_symbol<K>(S, C, y, l2)) & P::kFirst; }
            a = s1 | (s2 << P::kSecond);
            len = l1 + l2;
        } else {
            len = first_len(a, P::kLen);
            a &= P::kFirst;
            if (__any(len == 0)) { if (len == 0) a = P::put(long_symbol<K>(S, C, x, len)) & P::kFirst; }
        }
        e[i] = a;
        c += len;
        x = len < 32 ? x >> len : 0u;
    }
    return c;
}

// The refill step that follows a period: lanes that hold 32 bits or less take the next word of the stream, in lane order.
// t: bits used so far, in its low 7 bits.  CAREFUL: owner says which lanes own a symbol at the step the words are for, and
// lanes whose every period took 32 bits are looked after.
struct Refill { bool need; uint32_t t, w, taken; };
template <uint32_t RW, bool CAREFUL, bool NOISE>
__device__ __forceinline__ Refill ask(const PairStream &S, uint32_t t, bool owner)
{
    Refill r;
    r.t = CAREFUL ? t & 127u : NOISE ? t & 63u : t;
    r.need = r.t > 31u && (!CAREFUL || owner);
    const uint64_t bm = __ballot(r.need);
    const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(bm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bm, S.wpos));
    r.w = lds_word_now(S.ring + (pos & (RW - 1)) * 4);          // (its latency covers the check of the entries)
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

// One run of G symbols of the exponent field (A) and, when TWO, of the sign+mantissa field (B): their entries in ea, eb
template <int FMT, int R, bool TWO, uint32_t RW, bool CAREFUL, bool SERVICE>
__device__ __forceinline__ void pair_run(PairStream &A, PairStream &B, const PairCanon *C, uint32_t lane, uint32_t ea[], uint32_t eb[],
                                         uint32_t nsym, uint32_t nsym_next)
{
    constexpr int G = Fmt<FMT>::G, NA = Entries<FMT, 0>::kPair ? R / 2 : R, NB = Entries<FMT, 1>::kPair ? R / 2 : R;
    constexpr uint32_t kPerService = RW / 4 / 64;                // refill steps between two looks at the ring
#pragma unroll
    for (int g = 0; g < G / R; g++) {
        if (SERVICE && (uint32_t)g % kPerService == 0) { pair_service<RW>(A, lane); if (TWO) pair_service<RW>(B, lane); }
        const uint32_t xa = __builtin_amdgcn_alignbit(A.hi, A.lo, A.c), xb = TWO ? __builtin_amdgcn_alignbit(B.hi, B.lo, B.c) : 0u;
        const bool owner = !CAREFUL || (g + 1 < G / R ? (uint32_t)((g + 1) * R) < nsym : nsym_next > 0);
        uint32_t *const a = ea + g * NA, *const b = eb + g * NB;
        uint32_t ta = look_up<FMT, 0, NA, RW>(A.c, xa, a), tb = TWO ? look_up<FMT, 1, NB, RW>(B.c, xb, b) : 0u;
        Refill ra = ask<RW, CAREFUL, Entries<FMT, 0>::kNoise>(A, ta, owner), rb;
        if (TWO) rb = ask<RW, CAREFUL, Entries<FMT, 1>::kNoise>(B, tb, owner);
        if (__builtin_expect(__any(unresolved<FMT, 0>(a[NA - 1])), 0)) {
            ta = look_up_slowly<FMT, 0, NA, RW>(A, C[0], xa, a);
            ra = ask<RW, CAREFUL, Entries<FMT, 0>::kNoise>(A, ta, owner);
        }
        if (TWO && __builtin_expect(__any(unresolved<FMT, 1>(b[NB - 1])), 0)) {
            tb = look_up_slowly<FMT, 1, NB, RW>(B, C[1], xb, b);
            rb = ask<RW, CAREFUL, Entries<FMT, 1>::kNoise>(B, tb, owner);
        }
        take<CAREFUL>(A, ra);
        if (TWO) take<CAREFUL>(B, rb);
    }
}

// the output words of a run from its entries of field F
template <int FMT, int F>
__device__ __forceinline__ void entry_words(const uint32_t e[], uint32_t w[4])
{
    // a word is one pair, two singles, or two pairs that take half of it each: the low halves of both
    constexpr bool kWhole = Entries<FMT, F>::kPair && Entries<FMT, F>::kSecond == 16;
#pragma unroll
    for (int i = 0; i < 4; i++) w[i] = kWhole ? e[i] : __builtin_amdgcn_perm(e[2 * i + 1], e[2 * i], 0x05040100u);
}

// a plainly stored sign+mantissa run (two packed words, symbols in order) as it lies in the output words
template <int FMT>
__device__ __forceinline__ void plain_words(uint32_t p0, uint32_t p1, uint32_t w[4])
{
    const uint32_t p[2] = {p0, p1};
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if (FMT == ZC_FMT_BF16) {
            const uint32_t t = __builtin_amdgcn_perm(0, p[i / 2], (i & 1) ? 0x0C030C02u : 0x0C010C00u);      // bytes 2i, 2i+1 into bytes 0 and 2
            w[i] = t | (t << 8);
        } else {
            // four nibbles s m m m into four bytes s 0000 mmm
            const uint32_t h = p[i / 2] >> (16 * (i & 1));
            const uint32_t b = __builtin_amdgcn_perm(0, h, 0x0C010C00u), n = b | (b << 4);        // (the nibbles at bits 0, 8, 16, 24; above them others)
            w[i] = ((n << 4) & 0x80808080u) | (n & 0x07070707u);
        }
    }
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

template <int FMT, int R, int SM, bool XOR, uint32_t RW>
__device__ __forceinline__ void pair_rows(PairStream &A, PairStream &B, const PairCanon *C, const ChunkOut &o, uint32_t lane)
{
    constexpr int NP = Fmt<FMT>::G;                              // entries of a run, at most
    constexpr bool TWO = SM == kSmTable;
    constexpr uint32_t EX = kExponentBits<FMT>;
    const uint32_t rows = o.whole_rows;
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
    // the sign+mantissa output words of a row; m: its words (E5M2: its pair of rows' three)
    auto sm_words = [&](uint32_t row, const uint32_t m[4], const uint32_t eb[], uint32_t mw[4]) {
        if (SM == kSmTable) entry_words<FMT, 1>(eb, mw);
        else if (SM == kSmFlat3) {
            // an even row's 48 bits start at bit 0 of the three words, an odd one's at bit 48
            const uint32_t lo = (row & 1) ? __builtin_amdgcn_alignbit(m[2], m[1], 16) : m[0];
            const uint32_t hi = (row & 1) ? m[2] >> 16 : m[1];
            mw[0] = flat3_bytes(lo); mw[1] = flat3_bytes(lo >> 12);
            mw[2] = flat3_bytes(__builtin_amdgcn_alignbit(hi, lo, 24)); mw[3] = flat3_bytes(hi >> 4);
        } else {
            constexpr bool flat = SM == kSmFlat;
            constexpr int SB = Fmt<FMT>::SB == 8 ? 8 : 4;
            // (byte symbols are coded as bytes, most significant bit first, and their nibbles are in order then)
            plain_words<FMT>(flat ? reverse_in_groups<SB>(m[0]) : m[0], flat ? reverse_in_groups<SB>(m[1]) : m[1], mw);
        }
    };
    auto merge = [&](const uint32_t ea[], const uint32_t mw[4]) {
        uint32_t ew[4];
        entry_words<FMT, 0>(ea, ew);
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = (ew[i] & EX) | (mw[i] & ~EX);
        return v;
    };
    auto fast_row = [&](auto service, uint32_t row, const RowAhead &f, const RowAhead &even) {      // even: the pair of rows' three words (E5M2)
        uint32_t ea[NP], eb[NP], mw[4];
        pair_run<FMT, R, TWO, RW, false, decltype(service)::value>(A, B, C, lane, ea, eb, 0, 0);
        sm_words(row, SM == kSmFlat3 ? even.m : f.m, eb, mw);
        u32x4 v = merge(ea, mw);
        if (XOR) v ^= f.base;
        store_row<2>(v, o.ds, lane, row);
    };
    const bool ragged = o.nbytes % 1024 != 0;
    // ---- rows that need care: the first, until no lane is in the state of the start; the last before an incomplete one
    auto careful_row = [&](uint32_t row) {
        uint32_t ea[NP], eb[NP], mw[4];
        RowAhead f;
        fetch(row, f);
        if (SM == kSmFlat3) fetch_flat3(row / 2, f);
        pair_run<FMT, R, TWO, RW, true, true>(A, B, C, lane, ea, eb, (uint32_t)Fmt<FMT>::G, (ragged && row + 1 == rows) ? o.tail_sym : 1u);
        sm_words(row, f.m, eb, mw);
        u32x4 v = merge(ea, mw);
        if (XOR) v ^= f.base;
        store_row<2>(v, o.ds, lane, row);
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
    constexpr uint32_t kRows = RW / 4 / 64 / (Fmt<FMT>::G / R) >= 4 ? 4 : RW / 4 / 64 / (Fmt<FMT>::G / R) >= 2 ? 2 : 1;
    if (row + 4 <= fast_end) {
        pair_settle<RW>(A, lane);
        A.pending = false;
        if (TWO) { pair_settle<RW>(B, lane); B.pending = false; }
        RowAhead f[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) {
            fetch(row + i, f[i]);
            if (SM == kSmFlat3 && i % 2 == 0) fetch_flat3((row + i) / 2, f[i]);
        }
        auto block_row = [&](auto index) {
            constexpr uint32_t i = decltype(index)::value;
            fast_row(std::integral_constant<bool, i % kRows == 0>(), row + i, f[i], f[i & 2]);
            if (SM == kSmFlat3 && i % 2 == 1) fetch_flat3((row + i + 3) / 2, f[i & 2]);
            fetch(row + i + 4, f[i]);
        };
#pragma unroll 1
        for (; row + 4 <= fast_end; row += 4) {
            block_row(std::integral_constant<uint32_t, 0>());
            block_row(std::integral_constant<uint32_t, 1>());
            block_row(std::integral_constant<uint32_t, 2>());
            block_row(std::integral_constant<uint32_t, 3>());
        }
    }
#pragma unroll 1
    for (; row < rows; row++) careful_row(row);
    if (!ragged) return;
    // ---- the incomplete last row: a lane owns a whole run, part of one or nothing
    uint32_t ea[NP], eb[NP], mw[4], m[4] = {o.konst1, o.konst1, 0, 0};
    pair_run<FMT, R, TWO, RW, true, true>(A, B, C, lane, ea, eb, o.tail_sym, 0u);
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
        sm_words(rows, m, eb, mw);
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
        sm_words(rows, m, eb, mw);
    }
    if (o.tail_bytes) {
        const u32x4 t = merge(ea, mw);
        uint4 v = make_uint4(t.x, t.y, t.z, t.w);
        const uint32_t at = rows * 1024 + lane * 16;
        if (XOR) v = xor4(v, load_run(o.base + at, o.tail_bytes));
        store_run(o.dst + at, v, o.tail_bytes);
    }
}

}  // namespace

struct PairShared { TensorDev d; PairCanon canon[2]; uint32_t wave_count[4][17], flat3; };

// One wavefront per chunk, `chunks` of them per workgroup (of four or eight wavefronts, which build the tables together) around one
// copy of the tables; RW: words of a stream's ring.
// Bound by the latency of a chunk's chain up to about a thousand chunks (one wavefront per SIMD), then by the instructions, and
// from BF16's eight thousand on by HBM.  MI355X, whole calls, chunks of 256 KiB and a short one, against the kernels with single
// lookups of 11 bits and a launch of their own for the short chunk (before | now, us): 512 chunks: FP8 263 | 199, BF16 343 | 138,
// E5M2 497 | 281, byte symbols 423 | 237, BF16 deltas 600 | 277; 8,192: BF16 804 | 787, E5M2 1,084 | 1,058, byte symbols 1,082 | 900.
template <int FMT, bool XOR, uint32_t RW>
__global__ __launch_bounds__(1024) void k_decode_pairs(const TensorDev *descs, const WorkItem *work, TensorDev single, int use_single, uint32_t first_slot,
                                                       uint32_t chunks, uint32_t lds_tables_and_rings)
{
    using F_ = Fmt<FMT>;
    // all LDS in one piece, sized by the host, with field 0's table at its start (so that its entries need no base address);
    // then field 1's table where it has one, the rings, and what the workgroup shares besides
    extern __shared__ __attribute__((aligned(16))) char lds[];
    PairShared &sh = *reinterpret_cast<PairShared *>(lds + lds_tables_and_rings);
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
    if (uniform32(d.kind[0]) != KIND_HUFF || (p0 != 2 && p0 != 4 && p0 != 8) || (two && (p1 != p0 || RW == kLongRing))) return;
    if (FMT == ZC_FMT_FP8_E5M2 && (uniform32(d.mode[1]) != ZC_MODE_HUFF || !sh.flat3)) return;
    if (FMT == ZC_FMT_FP8_E4M3 && ((kind1 != KIND_FLAT && kind1 != KIND_RAW) || p0 == 8)) return;
    char *const table1 = lds + kTableBytes<FMT, 0, RW>;
    build_canon(canon[0], wave_count, d.comp + d.table_off[0], kAlphabet);
    build_entries<FMT, 0, RW>(lds, canon[0]);
    if (two) {
        build_canon(canon[1], wave_count, d.comp + d.table_off[1], kAlphabet);
        build_entries<FMT, 1, RW>(table1, canon[1]);
    }

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
    PairStream A, B;
    const uint32_t rings = kTableBytes<FMT, 0, RW> + (two ? kTableBytes<FMT, 1, RW> : 0u) + wave * (two ? 2 * RW : RW) * 4;
    const bool first = o.whole_rows > 0 || o.tail_sym > 0;       // does this lane own a symbol at step 0?
    A.ring = rings; A.rs = make_rsrc(sp[0], sb[0]);
    B.ring = rings + RW * 4; B.rs = o.r1;
#pragma unroll
    for (uint32_t i = 0; i < 4; i++) {
        A.limit[i] = i + kIndexBits<FMT, 0, RW> < 15 ? uniform32(canon[0].limit[i + kIndexBits<FMT, 0, RW> + 1]) : 0u;
        B.limit[i] = two && i + kIndexBits<FMT, 1, RW> < 15 ? uniform32(canon[1].limit[i + kIndexBits<FMT, 1, RW> + 1]) : 0u;
    }
    pair_open<RW>(A, lane, first);
    if (two) pair_open<RW>(B, lane, first);
#define ZC_ROWS(R, SM) case (R) * 8 + (SM): pair_rows<FMT, R, SM, XOR, RW>(A, B, canon, o, lane); break
    if constexpr (FMT == ZC_FMT_FP8_E5M2) {
        switch (p0 * 8 + kSmFlat3) { ZC_ROWS(2, kSmFlat3); ZC_ROWS(4, kSmFlat3); ZC_ROWS(8, kSmFlat3); }
    } else if constexpr (FMT == ZC_FMT_FP8_E4M3) {
        switch (p0 * 8 + kind1) { ZC_ROWS(2, kSmFlat); ZC_ROWS(4, kSmFlat); ZC_ROWS(2, kSmRaw); ZC_ROWS(4, kSmRaw); }
    } else {
        switch (p0 * 8 + kind1) {
            ZC_ROWS(2, kSmFlat); ZC_ROWS(4, kSmFlat); ZC_ROWS(8, kSmFlat);
            ZC_ROWS(2, kSmRaw); ZC_ROWS(4, kSmRaw); ZC_ROWS(8, kSmRaw);
            ZC_ROWS(2, kSmConst); ZC_ROWS(4, kSmConst); ZC_ROWS(8, kSmConst);
        }
        if constexpr (RW != kLongRing) switch (p0 * 8 + kind1) { ZC_ROWS(2, kSmTable); ZC_ROWS(4, kSmTable); ZC_ROWS(8, kSmTable); }
    }
#undef ZC_ROWS
}

template <int FMT, uint32_t RW>
static int launch_pairs_x(bool two, bool xor_delta, uint32_t chunks, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work, const TensorDev &s, int use_single,
                          uint32_t first_slot, hipStream_t st)
{
    const uint32_t lds = kTableBytes<FMT, 0, RW> + (two ? kTableBytes<FMT, 1, RW> : 0u) + chunks * (two ? 2u : 1u) * RW * 4, all = lds + (uint32_t)sizeof(PairShared);
    // (with short rings eight wavefronts build the tables, four where a call has more workgroups than the compute units hold of eight:
    // 1,500 BF16 tensors of one chunk of 100,000 bytes: 255 | 213 us)
    const dim3 grid(n_work), block(RW == kShortRing && (chunks > 4 || n_work <= 4 * 256) ? 512 : 256);
    if (xor_delta) hipLaunchKernelGGL((k_decode_pairs<FMT, true, RW>), grid, block, all, st, d_descs, d_work, s, use_single, first_slot, chunks, lds);
    else hipLaunchKernelGGL((k_decode_pairs<FMT, false, RW>), grid, block, all, st, d_descs, d_work, s, use_single, first_slot, chunks, lds);
    return (int)hipGetLastError();
}

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
#define ZC_PAIRS(F, RW) return launch_pairs_x<F, RW>(two, xor_delta, chunks, d_descs, d_work, n_work, s, use_single, first_slot, st)
    case ZC_FMT_BF16: if (!long_rings) ZC_PAIRS(ZC_FMT_BF16, kShortRing); if (two) ZC_PAIRS(ZC_FMT_BF16, kLongRingTwo); ZC_PAIRS(ZC_FMT_BF16, kLongRing);
    case ZC_FMT_FP8_E4M3_BYTES:
        if (!long_rings) ZC_PAIRS(ZC_FMT_FP8_E4M3_BYTES, kShortRing);
        if (two) ZC_PAIRS(ZC_FMT_FP8_E4M3_BYTES, kLongRingTwo);
        ZC_PAIRS(ZC_FMT_FP8_E4M3_BYTES, kLongRing);
    case ZC_FMT_FP8_E4M3: if (!long_rings) return 1; ZC_PAIRS(ZC_FMT_FP8_E4M3, kLongRing);       // (only calls of few chunks come here)
    case ZC_FMT_FP8_E5M2: if (!long_rings) ZC_PAIRS(ZC_FMT_FP8_E5M2, kShortRing); ZC_PAIRS(ZC_FMT_FP8_E5M2, kLongRing);
#undef ZC_PAIRS
    default: return 1;
    }
}

}  // namespace zc

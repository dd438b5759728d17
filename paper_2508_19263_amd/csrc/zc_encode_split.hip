// Stream sizes and encoder of 64-lane chunks that are walked by sixteen wavefronts (or eight, see split_waves) at once instead of one (a5, a7 for the
// two-field formats): a tensor's short last chunk, chunks that are not whole rows, and every chunk of a call that has too
// few of them to fill the GPU with one wavefront each.
//
// A chunk's stream is one sequence of words, but where a lane stands in it follows from bit totals alone.  With B(g) the
// bits of a lane's symbols before refill step g, the words the lane has asked for up to and including step g are
// min(g + 1, floor(B(g) / 32) + 2): a request needs k <= 32 unread bits, and a step takes at most 32 bits.  So a wavefront
// that starts at any row knows, from the bit totals of the rows before it, how many words every lane has asked for (their
// sum is the place of the next word), how many bits the lock-step decoder holds there and how far the lane's word in
// progress is filled.  What it cannot know is where the words lie that were asked for before its first row and are not
// complete there, at most two per lane: it keeps their contents in LDS, and once all wavefronts are through, one of them
// walks along the seams and puts those words together with what the wavefront before had of them.
#include <hip/hip_runtime.h>

#include "zc_internal.h"
#include "zc_device.h"
#include "zc_encode_device.h"

namespace zc {

namespace {

// Wavefronts per chunk: sixteen, of which a compute unit holds two workgroups, 512 chunks in all; eight in launches of more, which would
// leave the last round nearly empty.  Whole calls over chunks of 256 KiB, sixteen | eight, us: FP8 520: 223 | 202, 600: 234 | 215,
// 768: 238 | 231; BF16 520: 235 | 216, 768: 246 | 235; not E5M2 (520: 292 | 299) and byte symbols (600: 280 | 289), whose chunks are worth
// more instructions.  Short last chunks, however many, are ahead with eight throughout (both kernels' GPU time; chunks of 5,000, 40,000 and
// 200,000 bytes): 513 tensors of FP8 25 | 15, 39 | 30, 113 | 93, of BF16 27 | 15, 52 | 40, 163 | 139, of deltas 27 | 16, 51 | 39, 169 | 146; 1,100:
// FP8 42 | 24, 67 | 49, 185 | 148, deltas 48 | 27, 86 | 63, 280 | 229; 3,000: FP8 94 | 45, 152 | 97, 433 | 323, BF16 106 | 56, 195 | 130, 625 | 481,
// deltas 109 | 57, 196 | 131, 666 | 506.
inline uint32_t split_waves(uint32_t fmt, uint32_t n_work) { return n_work > 512 && (fmt == ZC_FMT_FP8_E4M3 || fmt == ZC_FMT_BF16) ? 8 : 16; }
// places of the (up to two) words a wavefront finds asked for and not complete at its first row; as byte offsets they lie
// beyond every stream, so the range check of the buffer store drops them
constexpr uint32_t kSeam0 = 0xFFFFFFFEu, kSeam1 = 0xFFFFFFFFu;

// 16 bytes from p of which the first `valid` may be read, every load in flight at once
__device__ __forceinline__ u32x4 load_ragged(const uint8_t *p, uint32_t valid)
{
    if (valid >= 16) return *reinterpret_cast<const u32x4 *>(p);
    const uint32_t words = valid >> 2;
    u32x4 v = {0, 0, 0, 0};
    const uint32_t a = words > 0 ? reinterpret_cast<const uint32_t *>(p)[0] : 0u;
    const uint32_t b = words > 1 ? reinterpret_cast<const uint32_t *>(p)[1] : 0u;
    const uint32_t c = words > 2 ? reinterpret_cast<const uint32_t *>(p)[2] : 0u;
    const uint32_t rest = valid & 3;
    const uint8_t *q = p + words * 4;
    uint32_t t = rest > 0 ? q[0] : 0u;
    t |= (rest > 1 ? (uint32_t)q[1] : 0u) << 8;
    t |= (rest > 2 ? (uint32_t)q[2] : 0u) << 16;
    v.x = words > 0 ? a : t;
    v.y = words > 1 ? b : words == 1 ? t : 0u;
    v.z = words > 2 ? c : words == 2 ? t : 0u;
    v.w = words == 3 ? t : 0u;
    return v;
}

// what every wavefront of the workgroup knows about its chunk
template <int FMT>
struct ChunkView {
    uint32_t n, nbytes, runs, rows;          // elements, bytes, 16-byte runs, rows of 64 runs (the last may be incomplete)
    const uint8_t *src, *base;
    __device__ __forceinline__ bool set(const TensorDev *dp, uint32_t chunk)
    {
        using F_ = Fmt<FMT>;
        const uint32_t cb = uni32(dp->chunk_bytes);
        const uint64_t E = (uint64_t)cb * 8 / F_::EB, first = (uint64_t)chunk * E, n_elems = uni64(dp->n_elems);
        if (uni32(dp->streams) != 64 || chunk >= uni32(dp->n_chunks) || first >= n_elems) return false;
        n = (uint32_t)(n_elems - first < E ? n_elems - first : E);
        nbytes = (uint32_t)(((uint64_t)n * F_::EB + 7) / 8);
        runs = (nbytes + 15) / 16;
        rows = (runs + 63) / 64;
        src = reinterpret_cast<const uint8_t *>(uni64((uint64_t)dp->src)) + (uint64_t)chunk * cb;
        const uint64_t b = uni64((uint64_t)dp->base);
        base = b ? reinterpret_cast<const uint8_t *>(b) + (uint64_t)chunk * cb : nullptr;
        return true;
    }
    // the run of a lane in a row (zeros where it has none)
    __device__ __forceinline__ u32x4 run_of(uint32_t row, uint32_t lane) const
    {
        const uint32_t at = (row * 64 + lane) * 16;
        u32x4 v = {0, 0, 0, 0};
        if (at < nbytes) {
            v = load_ragged(src + at, nbytes - at);
            if (base) v ^= load_ragged(base + at, nbytes - at);
        }
        return v;
    }
    // elements and symbols the lane owns in a row
    __device__ __forceinline__ uint32_t symbols_of(uint32_t row, uint32_t lane) const
    {
        using F_ = Fmt<FMT>;
        const uint32_t done = (row * 64 + lane) * F_::EPR;
        const uint32_t nel = n > done ? (n - done < (uint32_t)F_::EPR ? n - done : (uint32_t)F_::EPR) : 0u;
        return (nel + F_::GRP - 1) / F_::GRP;                    // a last partial group is filled with zeros
    }
};

// The symbols of a run as the words w[] they are packed in.  A field's table in LDS: 256 entries (code in bits 15..0, first
// bit lowest, length in bits 20..16) of the symbols themselves where they have 8 bits, and where they have 4 bits of the
// pairs a byte holds when a refill period is four symbols or more (two codes of at most 8 bits), else of the 16 symbols.
template <int FMT>
__device__ __forceinline__ void split_words(const u32x4 &v, uint32_t w[2][4])
{
    uint64_t P0, Q0, P1, Q1;
    split_run4<FMT>(make_uint4(v.x, v.y, v.z, v.w), P0, Q0, P1, Q1);
    w[0][0] = (uint32_t)P0; w[0][1] = (uint32_t)(P0 >> 32); w[0][2] = (uint32_t)Q0; w[0][3] = (uint32_t)(Q0 >> 32);
    w[1][0] = (uint32_t)P1; w[1][1] = (uint32_t)(P1 >> 32); w[1][2] = (uint32_t)Q1; w[1][3] = (uint32_t)(Q1 >> 32);
}

__device__ __forceinline__ uint32_t table_entry(const char *lut, uint32_t w, int byte) { return *reinterpret_cast<const uint32_t *>(lut + byte_times4(w, byte, 2u)); }

// the codes of the refill period of R symbols that starts at symbol j0 of a whole run, joined, and their length
template <int SB, int R>
__device__ __forceinline__ void period_code(const uint32_t w[4], int j0, const char *lut, uint32_t &code_out, uint32_t &len_out)
{
    if constexpr (SB == 4 && R == 2) {
        const uint32_t b = w[j0 / 8] >> (4 * (j0 % 8));
        const uint32_t x = *reinterpret_cast<const uint32_t *>(lut + ((b & 15u) << 2)), y = *reinterpret_cast<const uint32_t *>(lut + (((b >> 4) & 15u) << 2));
        join_codes(x, y, code_out, len_out);
    } else {
        constexpr int kUnits = R * SB / 8;                           // table bytes of a period: at least 2
        static_assert((SB == 8 || SB == 4) && (SB == 8 || R >= 4), "a period is two table entries or more");
        uint32_t code[kUnits / 2], len[kUnits / 2];
#pragma unroll
        for (int u = 0; u < kUnits / 2; u++) {
            const int b = j0 * SB / 8 + 2 * u;
            join_codes(table_entry(lut, w[b / 4], b % 4), table_entry(lut, w[(b + 1) / 4], (b + 1) % 4), code[u], len[u]);
        }
#pragma unroll
        for (int m = kUnits / 2; m > 1; m /= 2)
#pragma unroll
            for (int u = 0; u < m / 2; u++) {
                code[u] = code[2 * u] | (code[2 * u + 1] << len[2 * u]);
                len[u] = len[2 * u] + len[2 * u + 1];
            }
        code_out = code[0]; len_out = len[0];
    }
}

// bits of a whole run, and of its last refill period
template <int SB, int G, int R>
__device__ __forceinline__ void run_bits_r(const uint32_t w[4], const char *lut, uint32_t &bits, uint32_t &last)
{
#pragma unroll
    for (int j0 = 0; j0 < G; j0 += R) {
        uint32_t code, len;
        period_code<SB, R>(w, j0, lut, code, len);
        bits += len;
        last = len;
    }
}
template <int SB, int G>
__device__ __forceinline__ void run_bits(uint32_t period, const uint32_t w[4], const char *lut, uint32_t &bits, uint32_t &last)
{
    switch (period) {
    case 2: run_bits_r<SB, G, 2>(w, lut, bits, last); break;
    case 4: run_bits_r<SB, G, 4>(w, lut, bits, last); break;
    case 8: run_bits_r<SB, G, 8>(w, lut, bits, last); break;
    default: run_bits_r<SB, G, (G >= 16 ? 16 : 8)>(w, lut, bits, last); break;
    }
}

// What a lane keeps of a stream, see k_encode_fp8; seam[]: contents of the words found open at the first row.
struct SplitStream {
    uint32_t lo, nacc;
    int32_t k;
    uint32_t p0, p1, wpos;
    uint32_t n_seam;                         // of those words, how many are complete
};

// one refill step, then `len` bits of `code`
__device__ __forceinline__ void put_period(SplitStream &S, bool active, uint32_t code, uint32_t len, __amdgpu_buffer_rsrc_t out, uint32_t *seam)
{
    const bool req = active && S.k <= 32;
    const uint64_t bm = __ballot(req);
    const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(bm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bm, S.wpos));
    S.p0 = S.k == 0 ? pos : S.p0;
    S.p1 = req ? pos : S.p1;
    S.k += req ? 32 : 0;
    S.wpos += (uint32_t)__popcll(bm);
    const uint64_t placed = (uint64_t)code << S.nacc;            // nothing is left above bit nacc
    S.lo |= (uint32_t)placed;
    S.nacc += len;
    S.k -= (int32_t)len;
    if (S.nacc >= 32) {
        __builtin_amdgcn_raw_buffer_store_b32(S.lo, out, (int)(S.p0 * 4), 0, 0);
        if (S.p0 >= kSeam0) { seam[(S.p0 - kSeam0) * 64] = S.lo; S.n_seam++; }
        S.lo = (uint32_t)(placed >> 32); S.nacc -= 32; S.p0 = S.p1;
    }
}

template <int SB, int G, int R>
__device__ __forceinline__ void put_run_r(SplitStream &S, const uint32_t w[4], const char *lut, __amdgpu_buffer_rsrc_t out, uint32_t *seam)
{
#pragma unroll
    for (int j0 = 0; j0 < G; j0 += R) {
        uint32_t code, len;
        period_code<SB, R>(w, j0, lut, code, len);
        put_period(S, true, code, len, out, seam);
    }
}
template <int SB, int G>
__device__ __forceinline__ void put_run(SplitStream &S, uint32_t period, const uint32_t w[4], const char *lut, __amdgpu_buffer_rsrc_t out, uint32_t *seam)
{
    switch (period) {
    case 2: put_run_r<SB, G, 2>(S, w, lut, out, seam); break;
    case 4: put_run_r<SB, G, 4>(S, w, lut, out, seam); break;
    case 8: put_run_r<SB, G, 8>(S, w, lut, out, seam); break;
    default: put_run_r<SB, G, (G >= 16 ? 16 : 8)>(S, w, lut, out, seam); break;
    }
}

// symbol j of a run, j known only at run time
template <int SB>
__device__ __forceinline__ uint32_t symbol_at(const uint32_t w[4], uint32_t j)
{
    const uint32_t bit = j * SB, a = w[0], b = w[1], c = w[2], d = w[3];      // (copies: a choice among the elements would put the array in memory)
    const uint32_t x = bit < 32 ? a : bit < 64 ? b : bit < 96 ? c : d;
    return (x >> (bit & 31)) & ((1u << SB) - 1);
}

// the last row of a chunk, in which a lane owns nsym <= G symbols: steps and codes of what it owns
template <int SB, int G>
__device__ void put_last_run(SplitStream &S, uint32_t period, const uint32_t w[4], uint32_t nsym, const uint32_t *enc, __amdgpu_buffer_rsrc_t out, uint32_t *seam)
{
#pragma unroll 1
    for (uint32_t j0 = 0; j0 < (uint32_t)G; j0 += period) {
        uint32_t code = 0, len = 0;
#pragma unroll 1
        for (uint32_t j = j0; j < j0 + period && j < (uint32_t)G; j++) {
            const uint32_t e = j < nsym ? enc[symbol_at<SB>(w, j)] : 0u;
            code |= len < 32 ? (e & 0xFFFFu) << len : 0u;
            len += e >> 16;
        }
        put_period(S, j0 < nsym, code, len, out, seam);
    }
}

// the encode tables of the workgroup's tensor: singles as they come, `tab` as split_words' comment says
template <int FMT>
__device__ __forceinline__ void load_tables(const TensorDev *dp, const uint32_t *enc_of_tensor, uint32_t enc[2][256], uint32_t tab[2][256])
{
    using F_ = Fmt<FMT>;
    const uint32_t tid = threadIdx.x;
    if (tid < 512) enc[tid >> 8][tid & 255] = enc_of_tensor[tid];
    __syncthreads();
    if (tid < 512) {
        const uint32_t f = tid >> 8, u = tid & 255;
        uint32_t e = enc[f][u];
        if (F_::SB == 4 && uni32(dp->period[f]) >= 4) {
            const uint32_t a = enc[f][u & 15], b = enc[f][u >> 4];
            e = (a & 0xFFFFu) | ((b & 0xFFFFu) << (a >> 16)) | (((a >> 16) + (b >> 16)) << 16);
        }
        tab[f][u] = e;
    }
    __syncthreads();
}

}  // namespace

// A segment's rows: the chunk's, dealt out to W wavefronts in pieces
template <uint32_t W>
struct Segment {
    uint32_t per_wave, begin, end;
    __device__ __forceinline__ Segment(uint32_t rows, uint32_t wave)
    {
        per_wave = (rows + W - 1) / W;
        begin = wave * per_wave < rows ? wave * per_wave : rows;
        end = begin + per_wave < rows ? begin + per_wave : rows;
    }
};

// Does a field's number of bits follow from its data?  (A flat code's is the symbols' plain length, a field that is not coded has none.)  What k_sizes_split
// leaves for the encoder it leaves for these fields.
__device__ __forceinline__ bool bits_vary(uint32_t mode, uint32_t kind) { return mode == ZC_MODE_HUFF && kind != 1; }

// Bits of rows [begin, end) of a chunk, whole runs in every lane, per field that `walk` names, and of their last refill period
template <int FMT>
__device__ __forceinline__ void bits_of_rows(const ChunkView<FMT> &C, uint32_t begin, uint32_t end, uint32_t lane, const bool walk[2], const uint32_t period[2], const char *const lut[2],
                                             uint32_t bits[2], uint32_t last[2])
{
    using F_ = Fmt<FMT>;
    for (uint32_t r0 = begin; r0 < end; r0 += 4) {
        u32x4 v[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) {
            const uint64_t at = (uint64_t)((r0 + i < end ? r0 + i : end - 1) * 64 + lane) * 16;
            v[i] = *reinterpret_cast<const u32x4 *>(C.src + at);
            if (C.base) v[i] ^= *reinterpret_cast<const u32x4 *>(C.base + at);
        }
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) {
            if (r0 + i >= end) break;
            uint32_t w[2][4];
            split_words<FMT>(v[i], w);
#pragma unroll
            for (int f = 0; f < 2; f++)
                if (walk[f]) run_bits<F_::SB, F_::G>(period[f], w[f], lut[f], bits[f], last[f]);
        }
    }
}

// Stream sizes of the chunks of a work list, one chunk per item.  W wavefronts add up the code lengths of a segment of the rows
// each; the closed form above, taken at a lane's last step, gives the lane's words.  seg: where the segments' bits and those of their last periods
// (bits << 6 | last; W * 2 * 64 words per item) are left for the encoder where a field's bits_vary, or null.
template <int FMT, uint32_t W>
__global__ __launch_bounds__(64 * W) void k_sizes_split(const TensorDev *descs, const WorkItem *work, const uint32_t *enc_tables, uint32_t *units, uint32_t *seg)
{
    using F_ = Fmt<FMT>;
    static_assert(F_::NF == 2 && (F_::SB == 4 || F_::SB == 8) && F_::G * F_::SB <= 128, "two fields of 4- or 8-bit symbols, at most two 64-bit words per run");
    __shared__ uint32_t enc[2][256], tab[2][256];
    __shared__ uint32_t part[W][2][64], part_last[2][64];
    const WorkItem it = work[blockIdx.x];
    const TensorDev *dp = descs + it.tensor;
    const uint32_t lane = threadIdx.x & 63, wave = uni32(threadIdx.x >> 6);
    const uint32_t chunk = uni32(it.first);
    ChunkView<FMT> C;
    if (!C.set(dp, chunk)) return;                               // whole workgroup; the host never asks for this
    const uint32_t mode[2] = {uni32(dp->mode[0]), uni32(dp->mode[1])}, kind[2] = {uni32(dp->kind[0]), uni32(dp->kind[1])};
    const uint32_t period[2] = {uni32(dp->period[0]), uni32(dp->period[1])};
    load_tables<FMT>(dp, enc_tables + (uint64_t)it.tensor * 768, enc, tab);
    // the last row is taken apart from the others, whose runs are whole in every lane
    const bool walk[2] = {bits_vary(mode[0], kind[0]), bits_vary(mode[1], kind[1])};
    const char *const lut[2] = {reinterpret_cast<const char *>(tab[0]), reinterpret_cast<const char *>(tab[1])};
    const Segment<W> R_(C.rows, wave);
    uint32_t bits[2] = {0, 0}, last[2] = {0, 0};
    const uint32_t end = R_.end < C.rows ? R_.end : C.rows - 1;  // (rows >= 1)
    if ((walk[0] || walk[1]) && R_.begin < end) bits_of_rows<FMT>(C, R_.begin, end, lane, walk, period, lut, bits, last);
#pragma unroll
    for (int f = 0; f < 2; f++) {
        part[wave][f][lane] = bits[f];
        if (R_.begin < end && end == C.rows - 1) part_last[f][lane] = last[f];      // of the row before the last one
        if (seg && walk[f]) seg[(uint64_t)blockIdx.x * (W * 128) + (wave * 2 + f) * 64 + lane] = bits[f] << 6 | last[f];
    }
    __syncthreads();
    if (wave >= 2) return;
    const uint32_t f = wave;                                     // wavefront f finishes field f
    const uint32_t nsyms = (C.n + F_::GRP - 1) / F_::GRP;
    const uint32_t fmode = f ? mode[1] : mode[0], fkind = f ? kind[1] : kind[0], R = f ? period[1] : period[0];
    uint32_t u = 0;
    if (fmode == ZC_MODE_HUFF) {
        uint32_t q = 0;
        if (lane < C.runs) {
            const uint32_t row = (C.runs - 1 - lane) / 64;       // the lane's last row
            const uint32_t nsym = C.symbols_of(row, lane);
            const uint32_t total = row * F_::G + nsym, steps = (total + R - 1) / R;
            uint32_t before = 0;                                 // bits before the lane's last step
            if (fkind == 1) before = (steps - 1) * R * F_::SB;
            else {
#pragma unroll
                for (uint32_t wv = 0; wv < W; wv++) before += part[wv][f][lane];
                if (row + 1 < C.rows) before -= part_last[f][lane];          // a whole run, in the row before the last one
                else {
                    uint32_t w[2][4], x[4];
                    split_words<FMT>(C.run_of(row, lane), w);
#pragma unroll
                    for (int i = 0; i < 4; i++) x[i] = f ? w[1][i] : w[0][i];
                    const uint32_t in_last = nsym - (steps - 1 - row * F_::G / R) * R;        // symbols of the last step (R divides G)
#pragma unroll 1
                    for (uint32_t j = 0; j < nsym - in_last; j++) before += enc[f][symbol_at<F_::SB>(x, j)] >> 16;
                }
            }
            q = before / 32 + 2;
            q = q < steps ? q : steps;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
        u = (q + 3) / 4;
    } else if (fmode == ZC_MODE_RAW) u = (uint32_t)((((uint64_t)nsyms * F_::SB + 7) / 8 + 15) / 16);
    if (lane == 0) units[uni32(dp->units_off) + f * uni32(dp->n_chunks) + chunk] = u;
}

// The encoder, one chunk per work item.  Bound by its vector instructions on the one compute unit that has the chunk (256 rows
// of about 270, bit totals included); the source is read a second time, from the L2.  MI355X, chunks of 256 KiB: 36 us for 16
// FP8 chunks where one wavefront each takes 157 us, 54 us for BF16 deltas (both fields table coded), and 36 us for a set's
// short last chunks instead of 435 - 500 us in the generic encoder.  Its size pass: 11 - 17 us (15 - 52 us before it asked for
// four rows at a time).
// seg: the segments' bits as k_sizes_split left them, or null: they are added up here, which reads the source once more.  (Seven FP8 tensors, 517 chunks and
// their short last ones: 91 -> 71 us; 32 chunks of BF16 19 -> 16.)
template <int FMT, uint32_t W>
__global__ __launch_bounds__(64 * W) void k_encode_split(const TensorDev *descs, const WorkItem *work, const uint32_t *enc_tables, const uint32_t *seg)
{
    using F_ = Fmt<FMT>;
    constexpr int SB = F_::SB, G = F_::G, WPR = G * SB / 32;     // WPR: words of a plainly stored field per run
    static_assert(F_::NF == 2 && (SB == 4 || SB == 8) && (WPR == 2 || WPR == 4), "two fields of 4- or 8-bit symbols, at most two 64-bit words per run");
    __shared__ uint32_t enc[2][256], tab[2][256];
    __shared__ uint32_t seg_bits[W][2][64], seg_last[W][2][64];     // a segment's bits and those of its last period
    __shared__ uint32_t seam[2][W][2][64];             // see SplitStream
    __shared__ uint32_t end_lo[2][W][64], end_p0[2][W][64], end_p1[2][W][64];
    __shared__ uint8_t n_seam[2][W][64], end_owed[2][64];
    __shared__ uint32_t end_words[2];
    const WorkItem it = work[blockIdx.x];
    const TensorDev *dp = descs + it.tensor;
    const uint32_t lane = threadIdx.x & 63, wave = uni32(threadIdx.x >> 6);
    const uint32_t chunk = uni32(it.first);
    ChunkView<FMT> C;
    if (!C.set(dp, chunk)) return;                               // whole workgroup; the host never asks for this
    const uint32_t mode[2] = {uni32(dp->mode[0]), uni32(dp->mode[1])}, kind[2] = {uni32(dp->kind[0]), uni32(dp->kind[1])};
    const uint32_t period[2] = {uni32(dp->period[0]), uni32(dp->period[1])};
    uint8_t *comp = reinterpret_cast<uint8_t *>(uni64((uint64_t)dp->comp));
    const uint64_t payload = uni64(dp->payload_off);
    __amdgpu_buffer_rsrc_t out[2];
#pragma unroll
    for (int f = 0; f < 2; f++) {
        const uint32_t *index = reinterpret_cast<const uint32_t *>(comp + uni32(dp->index_off[f]));
        const uint64_t a = uni32(index[chunk]), b = uni32(index[chunk + 1]);
        if (a > b || (b - a) * 16 > 0x7FFFFFFFull) return;       // whole workgroup: index not as the size pass left it
        out[f] = rsrc_of(comp + payload + 16 * a, (uint32_t)((b - a) * 16));
    }
    load_tables<FMT>(dp, enc_tables + (uint64_t)it.tensor * 768, enc, tab);
    // table-coded fields have a state that runs through the rows; flat, raw and constant ones do not (16 symbols of 8 bits to a run: a flat code's words are
    // written like those of any other)
    const bool table[2] = {mode[0] == ZC_MODE_HUFF && (WPR == 4 || kind[0] != 1), mode[1] == ZC_MODE_HUFF && (WPR == 4 || kind[1] != 1)};
    const bool flat[2] = {mode[0] == ZC_MODE_HUFF && !table[0], mode[1] == ZC_MODE_HUFF && !table[1]};
    const char *const lut[2] = {reinterpret_cast<const char *>(tab[0]), reinterpret_cast<const char *>(tab[1])};

    const Segment<W> R_(C.rows, wave);
    const uint32_t segments = (C.rows + R_.per_wave - 1) / R_.per_wave, row_begin = R_.begin, row_end = R_.end;
    const uint32_t whole = C.nbytes / 1024 < row_end ? C.nbytes / 1024 : row_end;         // rows of this segment in which every lane holds a whole run end here
    // two rows are asked for ahead of the one that is coded
    auto fetch = [&](uint32_t row) {
        u32x4 v = {0, 0, 0, 0};
        if (row < whole) {
            const uint64_t at = (uint64_t)(row * 64 + lane) * 16;
            v = *reinterpret_cast<const u32x4 *>(C.src + at);
            if (C.base) v ^= *reinterpret_cast<const u32x4 *>(C.base + at);
        } else if (row < row_end) v = C.run_of(row, lane);
        return v;
    };
    u32x4 next = fetch(row_begin), after = fetch(row_begin + 1);
    // ---- bits of every segment but the last (whose rows may be incomplete, and whose bits nobody asks for)
    if ((table[0] || table[1]) && wave + 1 < segments) {
        const bool vary[2] = {bits_vary(mode[0], kind[0]), bits_vary(mode[1], kind[1])};
        uint32_t bits[2] = {0, 0}, last[2] = {0, 0};
        if (!seg && (vary[0] || vary[1])) bits_of_rows<FMT>(C, row_begin, row_end, lane, vary, period, lut, bits, last);
#pragma unroll
        for (int f = 0; f < 2; f++) {
            if (!vary[f]) { bits[f] = (row_end - row_begin) * (G * SB); last[f] = period[f] * SB; }
            else if (seg) {
                const uint32_t x = seg[(uint64_t)blockIdx.x * (W * 128) + (wave * 2 + f) * 64 + lane];
                bits[f] = x >> 6; last[f] = x & 63u;
            }
        }
#pragma unroll
        for (int f = 0; f < 2; f++) { seg_bits[wave][f][lane] = bits[f]; seg_last[wave][f][lane] = last[f]; }
    }
    __syncthreads();
    // ---- where this wavefront's lanes stand
    SplitStream S[2];
#pragma unroll
    for (int f = 0; f < 2; f++) {
        uint32_t B = 0, q = 0;
        if (table[f] && row_begin > 0 && row_begin < C.rows) {
            for (uint32_t w = 0; w < wave; w++) B += seg_bits[w][f][lane];
            const uint32_t steps = row_begin * (G / period[f]);
            q = ((B - seg_last[wave - 1][f][lane]) >> 5) + 2;
            q = q < steps ? q : steps;
        }
        S[f].lo = 0; S[f].nacc = B & 31; S[f].k = (int32_t)(32 * q - B);
        S[f].p0 = kSeam0; S[f].p1 = kSeam1; S[f].n_seam = 0;
        uint32_t sum = q;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        S[f].wpos = uni32(sum);
    }
    // ---- its rows
    auto plain_row = [&](int f, const uint32_t w[4], uint32_t row) {
        // every lane holds a whole run here
        if (flat[f]) {
#pragma unroll
            for (int h = 0; h < 2; h++) __builtin_amdgcn_raw_buffer_store_b32(reverse_in_groups<SB>(w[h]), out[f], (int)(((row * 2 + h) * 64 + lane) * 4), 0, 0);
        } else if (mode[f] == ZC_MODE_RAW) {
            if (WPR == 2) __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[0], w[1]}, out[f], (int)((row * 64 + lane) * 8), 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b128(u32x4{w[0], w[1], w[2], w[3]}, out[f], (int)((row * 64 + lane) * 16), 0, 0);
        }
    };
    for (uint32_t row = row_begin; row < whole; row++) {
        const u32x4 v = next;
        next = after;
        after = fetch(row + 2);
        uint32_t w[2][4];
        split_words<FMT>(v, w);
#pragma unroll
        for (int f = 0; f < 2; f++) {
            if (table[f]) put_run<SB, G>(S[f], period[f], w[f], lut[f], out[f], &seam[f][wave][0][lane]);
            else plain_row(f, w[f], row);
        }
    }
    if (whole < row_end && row_begin < row_end) {                // the chunk's incomplete last row (next holds its runs)
        const uint32_t row = row_end - 1, run = row * 64 + lane, nsym = C.symbols_of(row, lane);
        uint32_t w[2][4];
        split_words<FMT>(next, w);
#pragma unroll
        for (int f = 0; f < 2; f++) {
            if (table[f]) put_last_run<SB, G>(S[f], period[f], w[f], nsym, enc[f], out[f], &seam[f][wave][0][lane]);
            else if (flat[f]) {
                // one word per 32 / SB symbols to each lane that owns one of them, then zeros up to a whole 16-byte unit
                uint32_t at = row * 2 * 64;
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    const bool owner = (uint32_t)(h * (32 / SB)) < nsym;
                    const uint64_t bm = __ballot(owner);
                    __builtin_amdgcn_raw_buffer_store_b32(reverse_in_groups<SB>(w[f][h]), out[f], (int)(owner ? (at + prefix_count(bm)) * 4 : 0xFFFFFFF0u), 0, 0);
                    at += (uint32_t)__popcll(bm);
                }
                if (lane < ((4 - (at & 3)) & 3)) __builtin_amdgcn_raw_buffer_store_b32(0u, out[f], (int)((at + lane) * 4), 0, 0);
            } else if (mode[f] == ZC_MODE_RAW && nsym) {
                if (WPR == 2) {
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[f][0], w[f][1]}, out[f], (int)(run * 8), 0, 0);
                    if ((run & 1) == 0 && run + 1 >= C.runs) __builtin_amdgcn_raw_buffer_store_b64(u32x2{0, 0}, out[f], (int)((run + 1) * 8), 0, 0);
                } else __builtin_amdgcn_raw_buffer_store_b128(u32x4{w[f][0], w[f][1], w[f][2], w[f][3]}, out[f], (int)(run * 16), 0, 0);
            }
        }
    }
#pragma unroll
    for (int f = 0; f < 2; f++) {
        if (!table[f] || row_begin >= row_end) continue;
        end_lo[f][wave][lane] = S[f].lo; end_p0[f][wave][lane] = S[f].p0; end_p1[f][wave][lane] = S[f].p1;
        n_seam[f][wave][lane] = (uint8_t)S[f].n_seam;
        if (row_end == C.rows) {
            end_owed[f][lane] = (uint8_t)(((uint32_t)S[f].k + S[f].nacc) >> 5);
            if (lane == 0) end_words[f] = S[f].wpos;
        }
    }
    __syncthreads();
    // ---- the seams: wavefront f walks along those of field f
    if (wave >= 2) return;
    const uint32_t f = wave;
    if (!(f == 0 ? table[0] : table[1])) return;
    const __amdgpu_buffer_rsrc_t o = f == 0 ? out[0] : out[1];
    uint32_t lo = end_lo[f][0][lane], p0 = end_p0[f][0][lane], p1 = end_p1[f][0][lane];
    for (uint32_t s = 1; s < segments; s++) {
        const uint32_t done = n_seam[f][s][lane], e0 = end_p0[f][s][lane], e1 = end_p1[f][s][lane];
        if (done > 0) __builtin_amdgcn_raw_buffer_store_b32(lo | seam[f][s][0][lane], o, (int)(p0 * 4), 0, 0);
        if (done > 1) __builtin_amdgcn_raw_buffer_store_b32(seam[f][s][1][lane], o, (int)(p1 * 4), 0, 0);
        lo = end_lo[f][s][lane] | (done > 0 ? 0u : lo);
        const uint32_t c0 = e0 == kSeam0 ? p0 : e0 == kSeam1 ? p1 : e0, c1 = e1 == kSeam0 ? p0 : e1 == kSeam1 ? p1 : e1;
        p0 = c0; p1 = c1;
    }
    // the words still owed to the decoder (a partial word and a look-ahead word), then zeros up to a whole 16-byte unit
    const uint32_t owed = end_owed[f][lane], words = end_words[f];
    if (owed > 0) __builtin_amdgcn_raw_buffer_store_b32(lo, o, (int)(p0 * 4), 0, 0);
    if (owed > 1) __builtin_amdgcn_raw_buffer_store_b32(0u, o, (int)(p1 * 4), 0, 0);
    if (lane < ((4 - (words & 3)) & 3)) __builtin_amdgcn_raw_buffer_store_b32(0u, o, (int)((words + lane) * 4), 0, 0);
}

int launch_sizes_split(uint32_t fmt, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work, const uint32_t *d_enc, uint32_t *d_units, uint32_t *d_seg, void *stream)
{
    if (n_work == 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    const uint32_t waves = split_waves(fmt, n_work);
    const dim3 grid(n_work), block(64 * waves);
    switch (fmt) {
    case ZC_FMT_BF16:
        if (waves == 8) hipLaunchKernelGGL((k_sizes_split<ZC_FMT_BF16, 8>), grid, block, 0, st, d_descs, d_work, d_enc, d_units, d_seg);
        else hipLaunchKernelGGL((k_sizes_split<ZC_FMT_BF16, 16>), grid, block, 0, st, d_descs, d_work, d_enc, d_units, d_seg);
        break;
    case ZC_FMT_FP8_E4M3:
        if (waves == 8) hipLaunchKernelGGL((k_sizes_split<ZC_FMT_FP8_E4M3, 8>), grid, block, 0, st, d_descs, d_work, d_enc, d_units, d_seg);
        else hipLaunchKernelGGL((k_sizes_split<ZC_FMT_FP8_E4M3, 16>), grid, block, 0, st, d_descs, d_work, d_enc, d_units, d_seg);
        break;
    case ZC_FMT_FP8_E4M3_BYTES: hipLaunchKernelGGL((k_sizes_split<ZC_FMT_FP8_E4M3_BYTES, 16>), grid, block, 0, st, d_descs, d_work, d_enc, d_units, d_seg); break;
    case ZC_FMT_FP8_E5M2: hipLaunchKernelGGL((k_sizes_split<ZC_FMT_FP8_E5M2, 16>), grid, block, 0, st, d_descs, d_work, d_enc, d_units, d_seg); break;
    default: return 1;
    }
    return (int)hipGetLastError();
}

int launch_encode_split(uint32_t fmt, const TensorDev *d_descs, const WorkItem *d_work, uint32_t n_work, const uint32_t *d_enc, const uint32_t *d_seg, void *stream)
{
    if (n_work == 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    const uint32_t waves = split_waves(fmt, n_work);
    const dim3 grid(n_work), block(64 * waves);
    switch (fmt) {
    case ZC_FMT_BF16:
        if (waves == 8) hipLaunchKernelGGL((k_encode_split<ZC_FMT_BF16, 8>), grid, block, 0, st, d_descs, d_work, d_enc, d_seg);
        else hipLaunchKernelGGL((k_encode_split<ZC_FMT_BF16, 16>), grid, block, 0, st, d_descs, d_work, d_enc, d_seg);
        break;
    case ZC_FMT_FP8_E4M3:
        if (waves == 8) hipLaunchKernelGGL((k_encode_split<ZC_FMT_FP8_E4M3, 8>), grid, block, 0, st, d_descs, d_work, d_enc, d_seg);
        else hipLaunchKernelGGL((k_encode_split<ZC_FMT_FP8_E4M3, 16>), grid, block, 0, st, d_descs, d_work, d_enc, d_seg);
        break;
    case ZC_FMT_FP8_E4M3_BYTES: hipLaunchKernelGGL((k_encode_split<ZC_FMT_FP8_E4M3_BYTES, 16>), grid, block, 0, st, d_descs, d_work, d_enc, d_seg); break;
    case ZC_FMT_FP8_E5M2: hipLaunchKernelGGL((k_encode_split<ZC_FMT_FP8_E5M2, 16>), grid, block, 0, st, d_descs, d_work, d_enc, d_seg); break;
    default: return 1;
    }
    return (int)hipGetLastError();
}

}  // namespace zc

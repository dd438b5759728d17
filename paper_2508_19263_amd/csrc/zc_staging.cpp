// Page-locked host memory of the library: what the host sends to a workspace (descriptors, work lists, tables)
// and what it reads back between kernels (histograms, stream sizes, headers).  A copy to or from pageable
// memory is staged by the runtime in pieces and makes the caller wait; from page-locked memory it is one
// asynchronous transfer, or for small ones a kernel that reads the buffer; and what a kernel leaves in such memory the host can wait for by
// looking at it, where an event would hold up the next kernel.  The buffers are allocated on first use and kept until zc_release_host_buffers() or
// the end of the process.
#include <hip/hip_runtime.h>

#include <chrono>
#include <cstring>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

#include "zc_host.h"

namespace zc {

namespace {

// Bytes up to which the GPU fetches by itself (k_hand_over); a larger transfer is worth the runtime's copy, whose launch it
// hides.  (Decode plans, that kernel | the runtime's copy, us: 1 FP8 tensor of 16 KiB 21.2 | 21.3, 64 of them 23.4 | 23.1, from 100 on, more than 16
// KiB to send, 23.4 | 39.0.)
constexpr uint64_t kHandOver = 256 * 1024;

// words of page-locked memory that a kernel sets when it is through with what the host waits for
bool told(const uint32_t *flags, uint32_t n)
{
    for (uint32_t i = 0; i < n; i++) if (__atomic_load_n(flags + i, __ATOMIC_ACQUIRE) != kTold) return false;
    return true;
}
// Waits until all are set.  Looks without a pause for a while, as the runtime's own waits do, then lets other threads run between looks;
// once a second idle(), which does not wait, says whether the work has ended without them (an error): hipSuccess and not yet set then means they never will be.
template <typename Idle>
zc_status wait_until_told(const uint32_t *flags, uint32_t n, const Idle &idle)
{
    using clock = std::chrono::steady_clock;
    clock::time_point start = clock::now(), asked = start;
    for (uint32_t i = 0; i < n;) {
        if (__atomic_load_n(flags + i, __ATOMIC_ACQUIRE) == kTold) { i++; continue; }
        for (int k = 0; k < 64 && __atomic_load_n(flags + i, __ATOMIC_ACQUIRE) != kTold; k++) __builtin_ia32_pause();
        const clock::time_point now = clock::now();
        if (now - start > std::chrono::milliseconds(2)) std::this_thread::yield();
        if (now - asked > std::chrono::seconds(1)) {
            const hipError_t e = idle();
            if (e == hipSuccess) return told(flags, n) ? ZC_OK : ZC_ERR_DEVICE;
            if (e != hipErrorNotReady) return ZC_ERR_DEVICE;
            asked = now;
        }
    }
    return ZC_OK;
}

zc_status host_alloc(uint8_t **p, uint64_t bytes)
{
    // coherent: the GPU's words are seen while its kernel still runs
    return hipHostMalloc((void **)p, bytes, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess ? ZC_OK : ZC_ERR_DEVICE;
}

// ---- uploads -----------------------------------------------------------------------------------
// A few buffers used in turn: the pieces of an upload are packed into one at their workspace offsets and leave in
// a single asynchronous transfer (k_hand_over, or above kHandOver a copy).  A buffer's next user waits until the transfer that
// last left it is through (the words k_hand_over sets, or the event behind a copy), so calls queued back to back block only when more than kSlots uploads are still
// ahead of the device.  Every buffer has a lock of its own, held while its user waits, fills the buffer and queues the transfer: callers on
// other threads wait for each other only when they are dealt the same buffer.
class HostStage {
public:
    zc_status upload(uint8_t *d_ws, uint64_t lo, uint64_t hi, const Piece *pieces, int n, hipStream_t hs, uint64_t *d_zero, uint64_t n_zero)
    {
        if (hi <= lo) { LAUNCH_TRY(launch_zero(d_zero, n_zero, hs)); return ZC_OK; }
        int mine;
        {
            std::lock_guard<std::mutex> deal(m_);
            mine = next_;
            next_ = (next_ + 1) % kSlots;
        }
        Slot &k = slot_[mine];
        std::lock_guard<std::mutex> lock(k.m);
        const zc_status free_again = k.wait();
        if (free_again) return free_again;
        const uint64_t need = hi - lo;
        if (need > k.cap) {
            if (k.mem) (void)hipHostFree(k.mem);
            k.mem = nullptr; k.cap = 0;
            const uint64_t want = need + need / 2 + 4096;
            if (host_alloc(&k.mem, kFlagBytes + want)) { k.mem = nullptr; return ZC_ERR_DEVICE; }
            k.cap = want;
        }
        uint8_t *const buf = k.mem + kFlagBytes;
        for (int i = 0; i < n; i++)
            if (pieces[i].bytes) std::memcpy(buf + (pieces[i].off - lo), pieces[i].src, pieces[i].bytes);
        if (need <= kHandOver && (uintptr_t)(d_ws + lo) % 16 == 0) {
            const uint32_t groups = hand_over_groups((uint32_t)need);
            std::memset(k.flags(), 0, groups * sizeof(uint32_t));
            hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;         // (the null stream is never captured)
            if (hs && hipStreamIsCapturing(hs, &capture) != hipSuccess) return ZC_ERR_DEVICE;
            LAUNCH_TRY(launch_hand_over(buf, d_ws + lo, need, false, d_zero, n_zero, k.flags(), hs));
            k.groups = groups;
            k.captured = capture != hipStreamCaptureStatusNone;
        } else {
            if (!k.ev && hipEventCreateWithFlags(&k.ev, hipEventDisableTiming) != hipSuccess) return ZC_ERR_DEVICE;
            HIP_TRY(hipMemcpyAsync(d_ws + lo, buf, need, hipMemcpyHostToDevice, hs));
            LAUNCH_TRY(launch_zero(d_zero, n_zero, hs));
            HIP_TRY(hipEventRecord(k.ev, hs));
            k.copying = true;
        }
        return ZC_OK;
    }
    // waits for the transfers still in flight, then frees every buffer
    zc_status release()
    {
        zc_status st = ZC_OK;
        for (Slot &k : slot_) {
            std::lock_guard<std::mutex> lock(k.m);
            if (k.wait()) st = ZC_ERR_DEVICE;
            k.copying = k.captured = false; k.groups = 0;
            if (k.mem && hipHostFree(k.mem) != hipSuccess) st = ZC_ERR_DEVICE;
            k.mem = nullptr; k.cap = 0;
            if (k.ev) (void)hipEventDestroy(k.ev);
            k.ev = nullptr;
        }
        return st;
    }
private:
    static constexpr int kSlots = 4;
    static constexpr uint64_t kFlagBytes = 512;                  // in front of a buffer: the words k_hand_over sets
    static_assert(kHandOver / 4096 * sizeof(uint32_t) <= kFlagBytes, "a word per workgroup that reads");
    struct Slot {
        std::mutex m;
        uint8_t *mem = nullptr;
        uint64_t cap = 0;
        hipEvent_t ev = nullptr;
        bool copying = false;               // a copy with the event behind it is in flight
        uint32_t groups = 0;                // words that the kernel in flight has still to set
        bool captured = false;              // that kernel went into a graph: nobody knows when it reads the buffer
        uint32_t *flags() const { return reinterpret_cast<uint32_t *>(mem); }
        // For the words as long as it takes: the stream may be gone by now, so there is nothing to ask but the device, and that would be to wait for every
        // stream's work, among it what this thread would have to do first, and would spoil another thread's capture.
        zc_status wait()
        {
            if (captured || (copying && hipEventSynchronize(ev) != hipSuccess)) return ZC_ERR_DEVICE;
            copying = false;
            const zc_status st = groups ? wait_until_told(flags(), groups, [] { return hipErrorNotReady; }) : ZC_OK;
            groups = 0;
            return st;
        }
    };
    std::mutex m_;              // guards next_ only
    Slot slot_[kSlots];
    int next_ = 0;
};

HostStage &host_stage() { static HostStage s; return s; }

// ---- read-backs --------------------------------------------------------------------------------
// Buffers are handed out one per call in flight and come back when the call returns.
class HostLanding {
public:
    uint8_t *acquire(uint64_t bytes, uint64_t *cap)
    {
        std::lock_guard<std::mutex> lock(m_);
        for (size_t i = 0; i < free_.size(); i++)
            if (free_[i].second >= bytes) {
                uint8_t *b = free_[i].first; *cap = free_[i].second;
                free_.erase(free_.begin() + (long)i);
                return b;
            }
        if (!free_.empty()) { (void)hipHostFree(free_.back().first); free_.pop_back(); }     // too small: replace it
        uint8_t *b = nullptr;
        const uint64_t want = bytes + bytes / 2 + 4096;
        if (host_alloc(&b, want)) return nullptr;
        *cap = want;
        return b;
    }
    void give_back(uint8_t *b, uint64_t cap)
    {
        std::lock_guard<std::mutex> lock(m_);
        free_.push_back({b, cap});
    }
    // frees the buffers no call holds (a call in flight returns its buffer afterwards, to be freed by the next release)
    zc_status release()
    {
        std::lock_guard<std::mutex> lock(m_);
        zc_status st = ZC_OK;
        for (auto &f : free_) if (hipHostFree(f.first) != hipSuccess) st = ZC_ERR_DEVICE;
        free_.clear();
        return st;
    }
private:
    std::mutex m_;
    std::vector<std::pair<uint8_t *, uint64_t>> free_;
};

HostLanding &host_landing() { static HostLanding s; return s; }

}  // namespace

zc_status stage_upload(uint8_t *d_ws, uint64_t lo, uint64_t hi, const Piece *pieces, int n, void *stream, uint64_t *d_zero, uint64_t n_zero)
{
    return host_stage().upload(d_ws, lo, hi, pieces, n, (hipStream_t)stream, d_zero, n_zero);
}

zc_status wait_for_records(const HostRecords &to, uint32_t n, void *stream)
{
    return wait_until_told(to.flags, n, [stream] { return hipStreamQuery((hipStream_t)stream); });
}

HostRecords LandingLease::records(uint32_t n, bool blobs)
{
    const uint64_t bytes = (uint64_t)n * (blobs ? kBlobBytes : sizeof(ScanOut));
    HostRecords to = {ptr, reinterpret_cast<uint32_t *>(ptr + bytes), blobs ? 1u : 0u};
    std::memset(to.flags, 0, (uint64_t)n * sizeof(uint32_t));
    return to;
}

LandingLease::LandingLease(uint64_t bytes) { if (bytes) ptr = host_landing().acquire(bytes, &cap); }
LandingLease::~LandingLease() { if (ptr) host_landing().give_back(ptr, cap); }

}  // namespace zc

extern "C" zc_status zc_release_host_buffers(void)
{
    const zc_status a = zc::host_stage().release(), b = zc::host_landing().release();
    return a ? a : b;
}

// Large device arrays to the caller's (pageable) host memory.
//
// A plain copy to pageable memory moves at 10 GB/s: one host thread empties the
// runtime's staging buffer and, for an array that the caller has just allocated, takes
// all of its page faults.  Here the DMA engine fills a ring of pinned slots and several
// threads empty it, sharing the faults.  Four arrays of 134 MB (16.8 million particles):
// 53 ms plain, 17 ms this way (31 GB/s); three arrays of 134 MB: 39 ms and 13 ms.  Arrays
// under 32 MB go in smaller pieces, so that several threads take part: four of 4 MB 3.5 and
// 1.9 ms, of 8 MB 4.2 (in pieces of 2 MiB) and 2.5 ms; four of 2 MB are as fast plain.
#pragma once

#include <hip/hip_runtime.h>
#include <sched.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <thread>
#include <vector>

namespace ecpic {

// The pinned ring of one context (allocated with its first large readout, freed with it).
class HostCopy {
public:
    HostCopy() = default;
    HostCopy(const HostCopy &) = delete;
    HostCopy &operator=(const HostCopy &) = delete;
    ~HostCopy() { release(); }

    void release() {
        for (hipEvent_t &e : ev_)
            if (e) { (void)hipEventDestroy(e); e = nullptr; }
        if (ring_) (void)hipHostFree(ring_);
        ring_ = nullptr;
    }

    // dst[0, bytes) = src, after the work queued on s; returns when dst holds it.
    hipError_t to_host(void *dst, const void *src, size_t bytes, hipStream_t s, int device) {
        if (bytes < MIN_BYTES || !pageable(dst) || !ready()) return plain(dst, src, bytes, s);
        const size_t piece = std::min(SLOT, std::max(MIN_PIECE, bytes / 16 / MIN_PIECE * MIN_PIECE));
        const size_t chunks = (bytes + piece - 1) / piece;
        const int threads = (int)std::min<size_t>(std::min(THREADS, processors()), chunks / 2);
        auto size_of = [&](size_t k) { return std::min(piece, bytes - k * piece); };
        // Thread t moves the chunks k = t mod threads.  filled counts the chunks whose
        // DMA is queued (its event recorded), moved[slot] those a slot has passed on.
        std::atomic<size_t> filled{0};
        std::atomic<size_t> moved[SLOTS];
        for (auto &m : moved) m.store(0, std::memory_order_relaxed);
        std::atomic<int> err{(int)hipSuccess};
        auto mover = [&](int t) {
            if (hipSetDevice(device) != hipSuccess) err = (int)hipErrorInvalidDevice;
            for (size_t k = t; k < chunks; k += threads) {
                while (filled.load(std::memory_order_acquire) <= k) {
                    if (err != (int)hipSuccess) return;
                    std::this_thread::yield();
                }
                const int slot = (int)(k % SLOTS);
                const hipError_t e = hipEventSynchronize(ev_[slot]);
                if (e != hipSuccess) { err = (int)e; return; }
                std::memcpy((char *)dst + k * piece, ring_ + (size_t)slot * SLOT, size_of(k));
                moved[slot].fetch_add(1, std::memory_order_release);
            }
        };
        std::vector<std::thread> pool;
        try {
            for (int t = 0; t < threads; ++t) pool.emplace_back(mover, t);
        } catch (...) {   // no threads to be had
            err = (int)hipErrorOutOfMemory;
            for (std::thread &t : pool) t.join();
            return plain(dst, src, bytes, s);
        }
        for (size_t k = 0; k < chunks && err == (int)hipSuccess; ++k) {
            const int slot = (int)(k % SLOTS);
            while (moved[slot].load(std::memory_order_acquire) < k / SLOTS && err == (int)hipSuccess)
                std::this_thread::yield();
            if (err != (int)hipSuccess) break;
            hipError_t e = hipMemcpyAsync(ring_ + (size_t)slot * SLOT, (const char *)src + k * piece, size_of(k),
                                          hipMemcpyDeviceToHost, s);
            if (e == hipSuccess) e = hipEventRecord(ev_[slot], s);
            if (e != hipSuccess) { err = (int)e; break; }
            filled.store(k + 1, std::memory_order_release);
        }
        for (std::thread &t : pool) t.join();
        return (hipError_t)err.load();
    }

    // A small array from pinned memory to dst.  (Not a blocking copy where the runtime makes
    // it: that one would wait for the work of other streams.)
    static hipError_t from_pinned(void *dst, const void *src, size_t bytes, hipStream_t s) {
        if (!pageable(dst)) return plain(dst, src, bytes, s, hipMemcpyDefault);
        std::memcpy(dst, src, bytes);
        return hipSuccess;
    }

private:
    static constexpr size_t SLOT = (size_t)2 << 20, MIN_PIECE = (size_t)512 << 10, MIN_BYTES = (size_t)3 << 20;
    static constexpr int SLOTS = 16, THREADS = 8;

    static hipError_t plain(void *dst, const void *src, size_t bytes, hipStream_t s,
                            hipMemcpyKind kind = hipMemcpyDeviceToHost) {
        const hipError_t e = hipMemcpyAsync(dst, src, bytes, kind, s);
        return e != hipSuccess ? e : hipStreamSynchronize(s);
    }

    // Processors the calling thread may run on (the threads it starts inherit them).
    static int processors() {
        cpu_set_t set;
        return sched_getaffinity(0, sizeof(set), &set) == 0 ? std::max(1, CPU_COUNT(&set)) : THREADS;
    }

    // Memory the runtime knows (pinned by the caller, or on a device) needs no ring.
    static bool pageable(const void *dst) {
        hipPointerAttribute_t at{};
        const bool clean = hipPeekAtLastError() == hipSuccess;   // else the error is a launch's, and stays
        if (hipPointerGetAttributes(&at, dst) != hipSuccess) {
            if (clean) (void)hipGetLastError();
            return dst != nullptr;
        }
        return dst && at.type == hipMemoryTypeUnregistered;
    }

    bool ready() {
        if (ring_) return true;
        if (hipHostMalloc((void **)&ring_, SLOT * SLOTS, 0) != hipSuccess) {
            ring_ = nullptr;
            (void)hipGetLastError();
            return false;
        }
        for (hipEvent_t &e : ev_)
            if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                e = nullptr;
                (void)hipGetLastError();
                release();
                return false;
            }
        return true;
    }

    char *ring_ = nullptr;
    hipEvent_t ev_[SLOTS] = {};
};

}  // namespace ecpic

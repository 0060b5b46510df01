// Copies of large device arrays into the caller's ordinary host memory.
//
// hipMemcpy into pageable memory goes through the runtime's staging on one
// thread, and into arrays that were just allocated that thread also takes
// every page fault: 448 MB (the fields of 200 x 200 x 280 nodes) came in 45 ms,
// 26 ms when the pages were there, 8.2 ms into pinned memory.  Here the copy
// goes through a few pinned slots in chunks, and several threads move the
// chunks on (and take the faults) while the next ones arrive.  Memory that HIP
// knows (pinned, managed or device memory of the caller) is copied to directly:
// into pinned arrays that is the faster way (537 MB 9.9 ms against 13.6 through
// the slots), and the threads could not write device memory.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstddef>
#include <cstring>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

namespace lbm_host {

// Owned by a context (its calls are not concurrent) and freed with it.
class HostCopier {
  public:
    // below this the direct copy is as fast as starting the threads and, the
    // first time, pinning the slots (about 2 ms)
    static constexpr size_t MIN_BYTES = size_t(24) << 20;

    HostCopier() = default;
    HostCopier(const HostCopier &) = delete;
    HostCopier &operator=(const HostCopier &) = delete;
    ~HostCopier()
    {
        for (hipEvent_t e : ev_)
            if (e) (void)hipEventDestroy(e);
        if (pin_) (void)hipHostFree(pin_);
    }

    // dst[i] <- src[i], bytes each, for i < n (null dst: skipped), after the
    // stream's work so far; returns when the data are there.  `device` is the
    // stream's; any other may be current.
    hipError_t copy(int device, hipStream_t st, void *const *dst, const void *const *src, size_t bytes, int n)
    {
        size_t total = 0;
        for (int i = 0; i < n; ++i) total += dst[i] ? bytes : 0;
        if (total >= MIN_BYTES && ordinary(dst, n) && ready(device)) {
            if (staged(device, st, dst, src, bytes, n) == hipSuccess) return hipSuccess;
            (void)hipGetLastError();  // the direct copy says whether the stream has failed
        }
        for (int i = 0; i < n; ++i)
            if (dst[i]) {
                const hipError_t e = hipMemcpyAsync(dst[i], src[i], bytes, hipMemcpyDeviceToHost, st);
                if (e != hipSuccess) return e;
            }
        return hipStreamSynchronize(st);
    }

  private:
    static constexpr int SLOTS = 8, THREADS = 6;
    static constexpr size_t CHUNK = size_t(2) << 20;
    char *pin_ = nullptr;
    hipEvent_t ev_[SLOTS] = {};
    bool failed_ = false;

    // Memory that HIP does not know.
    static bool ordinary(void *const *dst, int n)
    {
        for (int i = 0; i < n; ++i) {
            hipPointerAttribute_t at;
            if (!dst[i]) continue;
            if (hipPointerGetAttributes(&at, dst[i]) != hipSuccess)
                (void)hipGetLastError();  // (older runtimes: an error for such memory)
            else if (at.type != hipMemoryTypeUnregistered)
                return false;
        }
        return true;
    }

    // The slots and their events, which belong to the stream's device.
    bool ready(int device)
    {
        if (pin_ || failed_) return pin_ != nullptr;
        int current = device;
        // a capture that is under way, here or on another thread, goes on
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        bool ok = hipGetDevice(&current) == hipSuccess && hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        if (ok) {
            if (current != device) ok = hipSetDevice(device) == hipSuccess;
            ok = ok && hipHostMalloc((void **)&pin_, SLOTS * CHUNK, hipHostMallocDefault) == hipSuccess;
            for (hipEvent_t &e : ev_) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
            if (current != device) (void)hipSetDevice(current);
            (void)hipThreadExchangeStreamCaptureMode(&mode);
        }
        if (!ok) {
            (void)hipGetLastError();
            if (pin_) (void)hipHostFree(pin_);
            pin_ = nullptr;
            failed_ = true;  // copy directly from now on
        }
        return ok;
    }

    struct Piece {
        char *dst;
        const char *src;
        size_t bytes;
    };

    // (an error: the data may not be there)
    hipError_t staged(int device, hipStream_t st, void *const *dst, const void *const *src, size_t bytes, int n)
    {
        std::vector<Piece> pieces;
        std::vector<std::thread> pool;
        std::mutex mu;
        std::condition_variable cv;
        long issued = 0, taken = 0;             // pieces on the stream; pieces workers have taken
        long freed[SLOTS];                      // last piece moved out of each slot, -1: none
        bool stop = false;
        hipError_t bad = hipSuccess;
        for (long &f : freed) f = -1;
        auto work = [&]() {
            (void)hipSetDevice(device);
            std::unique_lock<std::mutex> lk(mu);
            for (;;) {
                cv.wait(lk, [&] { return taken < issued || stop; });
                if (taken >= issued) return;
                const long k = taken++;
                lk.unlock();
                const int s = (int)(k % SLOTS);
                const hipError_t e = hipEventSynchronize(ev_[s]);
                if (e == hipSuccess) std::memcpy(pieces[(size_t)k].dst, pin_ + (size_t)s * CHUNK, pieces[(size_t)k].bytes);
                lk.lock();
                if (e != hipSuccess && bad == hipSuccess) bad = e;
                freed[s] = k;
                cv.notify_all();
            }
        };
        try {
            for (int i = 0; i < n; ++i)
                for (size_t o = 0; dst[i] && o < bytes; o += CHUNK)
                    pieces.push_back({(char *)dst[i] + o, (const char *)src[i] + o, std::min(CHUNK, bytes - o)});
            pool.reserve(THREADS);
            for (int t = 0; t < THREADS; ++t) pool.emplace_back(work);
        } catch (const std::exception &) {
            if (pool.empty()) return hipErrorOutOfMemory;  // no thread
        }
        for (long k = 0; k < (long)pieces.size(); ++k) {
            const int s = (int)(k % SLOTS);
            {
                std::unique_lock<std::mutex> lk(mu);
                cv.wait(lk, [&] { return k < SLOTS || freed[s] == k - SLOTS; });
                if (bad != hipSuccess) break;
            }
            const Piece &p = pieces[(size_t)k];
            hipError_t e = hipMemcpyAsync(pin_ + (size_t)s * CHUNK, p.src, p.bytes, hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipEventRecord(ev_[s], st);
            std::lock_guard<std::mutex> lk(mu);
            if (e != hipSuccess) {
                bad = e;
                break;
            }
            issued = k + 1;
            cv.notify_one();
        }
        {
            std::lock_guard<std::mutex> lk(mu);
            stop = true;
        }
        cv.notify_all();
        for (std::thread &t : pool) t.join();
        const hipError_t e = hipStreamSynchronize(st);
        return bad != hipSuccess ? bad : e;
    }
};

}  // namespace lbm_host

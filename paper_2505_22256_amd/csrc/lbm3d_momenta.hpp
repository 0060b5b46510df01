// The device memory of the momenta that the 3-D steps of relaxation time 1 keep
// between their two passes.  A step is faster with it and runs without it.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace lbm3_host {

class Momenta {
  public:
    Momenta() = default;
    Momenta(const Momenta &) = delete;
    Momenta &operator=(const Momenta &) = delete;
    ~Momenta()
    {
        if (p_) (void)hipFree(p_);
    }
    void *get() const { return p_; }

    // Allocate them on `device`, whichever is current, if there is room.  (Here and
    // not in a step, which a caller may capture; a capture that is under way, here or
    // on another thread, goes on.)
    void want(int device, size_t bytes)
    {
        if (p_) return;
        int current = device;
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (hipGetDevice(&current) != hipSuccess || hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return;
        if ((current != device && hipSetDevice(device) != hipSuccess) || hipMalloc(&p_, bytes) != hipSuccess) {
            p_ = nullptr;
            (void)hipGetLastError();
        }
        if (current != device) (void)hipSetDevice(current);
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    }

    // A step on `st` is about to use them.
    void used(hipStream_t st)
    {
        hipStreamCaptureStatus status = hipStreamCaptureStatusActive;
        if (!p_ || captured_) return;
        if (hipStreamIsCapturing(st, &status) != hipSuccess) (void)hipGetLastError();
        captured_ = status != hipStreamCaptureStatusNone;
    }

    // Free them after the work on `st`; false where there are none, or a captured
    // step may use them again.
    bool give_back(hipStream_t st)
    {
        if (!p_ || captured_ || hipStreamSynchronize(st) != hipSuccess) return false;
        (void)hipFree(p_);
        p_ = nullptr;
        return true;
    }

  private:
    void *p_ = nullptr;
    bool captured_ = false;
};

// Allocate scratch that a call cannot do without: where the room is gone the
// momenta, which only save time, make place for it.
template <class T> hipError_t alloc_scratch(T **p, size_t bytes, Momenta &mom, hipStream_t st)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipSuccess) return e;
    if (mom.give_back(st)) {
        (void)hipGetLastError();
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) *p = nullptr;
    return e;
}

}  // namespace lbm3_host

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

  private:
    void *p_ = nullptr;
};

}  // namespace lbm3_host

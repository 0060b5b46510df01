"""HostCopier (csrc/lbm_hostcopy.hpp) on the host, against a small stand-in for
the HIP runtime that keeps each call's rules: an event records only on a stream of
its own device, a chunk's memory is what the runtime says it is.  What a GPU test
cannot set up: another device current than the stream's, a runtime that fails
half-way, a capture under way."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++") or shutil.which("c++")

HIP = r"""
#pragma once
#include <cstddef>
#include <cstdlib>
#include <cstring>
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2, hipErrorInvalidHandle = 400 };
enum hipMemoryType { hipMemoryTypeUnregistered = 0, hipMemoryTypeHost = 1, hipMemoryTypeDevice = 2, hipMemoryTypeManaged = 3 };
enum hipMemcpyKind { hipMemcpyDeviceToHost = 2 };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal, hipStreamCaptureModeRelaxed };
enum { hipHostMallocDefault = 0, hipEventDisableTiming = 2 };
struct Stream { int device; };
struct Event { int device; bool recorded; };
typedef Stream *hipStream_t;
typedef Event *hipEvent_t;
struct hipPointerAttribute_t { hipMemoryType type; int device; };

struct Runtime {
    int events = 0, copies = 0, fail_record = -1, records = 0;
    bool attr_error = false, no_pin = false, strict_alloc = false;
    const void *known = nullptr;  // an address that is not ordinary memory
    hipMemoryType known_type = hipMemoryTypeHost;
};
extern Runtime rt;
extern thread_local int current;
extern thread_local hipStreamCaptureMode capture_mode;

inline hipError_t hipGetDevice(int *d) { *d = current; return hipSuccess; }
inline hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m)
{
    const hipStreamCaptureMode old = capture_mode;
    capture_mode = *m;
    *m = old;
    return hipSuccess;
}
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t *at, const void *p)
{
    if (p == rt.known) { at->type = rt.known_type; at->device = 0; return hipSuccess; }
    if (rt.attr_error) return hipErrorInvalidValue;
    at->type = hipMemoryTypeUnregistered;
    at->device = -1;
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    if (rt.no_pin || (rt.strict_alloc && capture_mode != hipStreamCaptureModeRelaxed)) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    return hipSuccess;
}
inline hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = new Event{current, false}; ++rt.events; return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { delete e; --rt.events; return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    if (e->device != s->device) return hipErrorInvalidHandle;
    if (rt.records++ == rt.fail_record) return hipErrorInvalidValue;
    e->recorded = true;
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    ++rt.copies;
    std::memcpy(d, s, n);
    return hipSuccess;
}
"""

MAIN = r"""
#include "lbm_hostcopy.hpp"
#include <cstdio>
Runtime rt;
thread_local int current = 0;
thread_local hipStreamCaptureMode capture_mode = hipStreamCaptureModeGlobal;

int main(int, char **argv)
{
    const std::string what = argv[1];
    const size_t bytes = (size_t(20) << 20) + 8;  // two arrays of a ragged number of chunks
    std::vector<char> a(bytes), b(bytes), x(bytes), y(bytes);
    for (size_t i = 0; i < bytes; ++i) a[i] = char(i * 7 + i / 4096), b[i] = char(i * 5 + i / 1000);
    void *dst[3] = {x.data(), nullptr, y.data()};
    const void *src[3] = {a.data(), a.data(), b.data()};
    Stream st{0};
    bool direct = true;
    if (what == "plain" || what == "attr-error") direct = false, rt.attr_error = what == "attr-error";
    if (what == "other-device") st.device = 1, direct = false;
    if (what == "pinned") rt.known = x.data();
    if (what == "device") rt.known = y.data(), rt.known_type = hipMemoryTypeDevice;
    if (what == "no-pin") rt.no_pin = true;
    if (what == "half-way") rt.fail_record = 5;
    if (what == "capture") rt.strict_alloc = true, direct = false;
    int rc = 0;
    {
        lbm_host::HostCopier c;
        for (int k = 0; k < 2; ++k) {
            rt.copies = 0;
            std::fill(x.begin(), x.end(), 0);
            std::fill(y.begin(), y.end(), 0);
            const hipError_t e = c.copy(st.device, &st, dst, src, bytes, 3);
            if (e != hipSuccess) std::printf("error %d\n", (int)e), rc = 1;
            if (x != a || y != b) std::printf("wrong bytes\n"), rc = 1;
            if (what != "half-way" && (rt.copies == 2) != direct) std::printf("%d copies\n", rt.copies), rc = 1;
        }
        if (current != 0) std::printf("device %d left current\n", current), rc = 1;
        if (capture_mode != hipStreamCaptureModeGlobal) std::printf("capture mode changed\n"), rc = 1;
    }
    if (rt.events) std::printf("%d events left\n", rt.events), rc = 1;
    return rc;
}
"""


@pytest.mark.skipif(CXX is None, reason="no host compiler")
@pytest.mark.parametrize("what", ["plain", "attr-error", "other-device", "pinned", "device", "no-pin", "half-way", "capture"])
def test_copies(tmp_path, what):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    (tmp_path / "main.cpp").write_text("#include <string>\n" + MAIN)
    exe = tmp_path / "main"
    subprocess.run([CXX, "-O1", "-std=c++17", "-pthread", "-I", str(tmp_path), "-I",
                    os.path.join(ROOT, "paper_2505_22256_amd", "csrc"), str(tmp_path / "main.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout)

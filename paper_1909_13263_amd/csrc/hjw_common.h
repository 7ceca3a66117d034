// hjw_common.h - constants and error reporting shared by the library's sources.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <string>

#include "hjw.h"

namespace hjw {

// Thread-local text of the last error (defined in hjw.hip).
std::string& last_error();

inline hjw_status fail(hjw_status code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    last_error() = buf;
    return code;
}

// The device of a stream's launches (the current one's for the default stream).
inline int stream_device(hipStream_t stream) {
    int dev = 0;
    if (stream && hipStreamGetDevice(stream, &dev) == hipSuccess) return dev;
    (void)hipGetLastError();
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    return dev;
}

constexpr int kMaxDevices = 64;

// What the calls of this process that are stepping on a device could hold of it at once, in
// thousandths, summed over them (defined in hjw.hip).
std::atomic<int>& stepping_share(int device);

// A call that is stepping on a device, for its duration.
class Stepping {
    std::atomic<int>& sum_;
    const int share_;

public:
    Stepping(int device, int share) : sum_(stepping_share(device)), share_(share) { sum_ += share_; }
    ~Stepping() { sum_ -= share_; }
    Stepping(const Stepping&) = delete;
    Stepping& operator=(const Stepping&) = delete;
    int others() const { return sum_.load() - share_; }
};

constexpr size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

}  // namespace hjw

#define HIP_TRY(expr)                                                                     \
    do {                                                                                  \
        hipError_t e_ = (expr);                                                           \
        if (e_ != hipSuccess)                                                             \
            return ::hjw::fail(HJW_EHIP, "%s failed: %s (%d)", #expr, hipGetErrorString(e_), \
                               int(e_));                                                  \
    } while (0)

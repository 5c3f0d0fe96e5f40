// Launches of one call side by side on streams of their own.
#pragma once

#include "wl_internal.h"

namespace wl {

// Up to kMax side streams on the current device, with the events that tie them
// to a caller's stream.  Plain data: whoever makes them releases them.
struct SideStreams {
    static constexpr int kMax = 4;
    int n = 0;  // streams that exist
    hipStream_t s[kMax] = {};
    hipEvent_t done[kMax] = {};
    hipEvent_t start = nullptr;

    // As many of `want` as the runtime gives (none is no error: the launches
    // then follow each other on the caller's stream).
    void make(int want) {
        if (want > kMax) want = kMax;
        if (want <= n) return;
        if (!start && hipEventCreateWithFlags(&start, hipEventDisableTiming) != hipSuccess) {
            start = nullptr;
            (void)hipGetLastError();
            return;
        }
        while (n < want) {
            if (hipStreamCreateWithFlags(&s[n], hipStreamNonBlocking) != hipSuccess) break;
            if (hipEventCreateWithFlags(&done[n], hipEventDisableTiming) != hipSuccess) {
                (void)hipStreamDestroy(s[n]);
                break;
            }
            ++n;
        }
        if (n < want) (void)hipGetLastError();
    }
    void release() {
        while (n > 0) {
            --n;
            (void)hipEventDestroy(done[n]);
            (void)hipStreamDestroy(s[n]);
        }
        if (start) (void)hipEventDestroy(start);
        start = nullptr;
    }
};

// One fork: the first launch goes to the caller's stream, each later one to a
// side stream that waits for what the caller's stream held at open(); after
// join() the caller's stream waits for all of them.  Left without a join (an
// error), it waits on the host, so that nothing of the call is still running
// when the caller gets its buffers back.
class Fork {
  public:
    Fork(SideStreams& side, hipStream_t caller) : side_(side), caller_(caller) {}
    Fork(const Fork&) = delete;
    Fork& operator=(const Fork&) = delete;
    ~Fork() {
        for (int k = 0; k < used_; ++k) (void)hipStreamSynchronize(side_.s[k]);
    }
    wl_status open() {
        if (side_.n > 0) WL_CHECK_HIP(hipEventRecord(side_.start, caller_));
        return WL_OK;
    }
    wl_status next(hipStream_t* out) {
        *out = caller_;
        const int k = launches_++ - 1;
        if (k < 0 || side_.n == 0) return WL_OK;
        *out = side_.s[k % side_.n];
        if (k < side_.n) {
            WL_CHECK_HIP(hipStreamWaitEvent(*out, side_.start, 0));
            used_ = k + 1;
        }
        return WL_OK;
    }
    wl_status join() {
        for (int k = 0; k < used_; ++k) {
            WL_CHECK_HIP(hipEventRecord(side_.done[k], side_.s[k]));
            WL_CHECK_HIP(hipStreamWaitEvent(caller_, side_.done[k], 0));
        }
        used_ = 0;
        return WL_OK;
    }

  private:
    SideStreams& side_;
    hipStream_t caller_;
    int launches_ = 0;
    int used_ = 0;  // side streams with work that the caller's stream does not wait for yet
};

}  // namespace wl

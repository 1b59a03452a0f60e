// Host side of the reports that kernels make in pinned memory (kernels.h,
// Report): a spin on the word instead of an event.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <immintrin.h>
#include <thread>

namespace cgmi {

// Waits until the word has reached `first` and then either `want` or a payload
// other than 0, which is returned in *payload.  The stream is asked for errors
// now and then only (a failed launch never reports), and the time slice given
// away once the wait is longer than a short kernel.
inline hipError_t wait_report(const unsigned long long *word, uint32_t first, uint32_t want, hipStream_t s,
                              uint32_t *payload)
{
    bool idle = false;
    for (uint64_t spin = 1;; ++spin) {
        const unsigned long long v = __atomic_load_n(word, __ATOMIC_ACQUIRE);
        const uint32_t tick = (uint32_t)(v >> 32);
        if ((int32_t)(tick - first) >= 0 && ((int32_t)(tick - want) >= 0 || (uint32_t)v != 0)) {
            *payload = (uint32_t)v;
            return hipSuccess;
        }
        if (idle) // all work of the stream is done, and no report
            return hipErrorUnknown;
        if (spin == 4096) { // (in a capture nothing runs, so nothing reports)
            hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
            if (s != nullptr && hipStreamIsCapturing(s, &capture) == hipSuccess && capture != hipStreamCaptureStatusNone)
                return hipErrorStreamCaptureUnsupported;
        }
        if (spin < 4096)
            _mm_pause();
        else
            std::this_thread::yield();
        if ((spin & 0xfffff) == 0) {
            const hipError_t e = hipStreamQuery(s);
            if (e == hipErrorNotReady)
                (void)hipGetLastError(); // (not an error of the caller's)
            if (e != hipSuccess && e != hipErrorNotReady)
                return e;
            idle = e == hipSuccess;
        }
    }
}

} // namespace cgmi

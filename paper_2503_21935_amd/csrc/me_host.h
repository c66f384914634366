// me_host.h -- host-side rules that need no device.
#pragma once
#include <cstdint>

// HIP takes launches of fewer than 2^32 threads, which at several threads per event is
// less than a call may hold (2^29 events at 8 lanes each, momenta of 86 GB and more).
// f(first, blocks) for each launch: `blocks` blocks of `threads` threads with `per`
// events each, from event `first`.
template <class F>
static inline void me_each_launch(int64_t nevt, int per, int threads, F&& f) {
    const int64_t most = (int64_t(1) << 31) / threads;  // blocks of a launch: 2^31 threads
    for (int64_t first = 0; first < nevt; first += most * per) {
        const int64_t blocks = (nevt - first + per - 1) / per;
        f(first, (unsigned)(blocks < most ? blocks : most));
    }
}

// me_host.h -- host-side rules that need no device.
#pragma once
#include <cstddef>
#include <cstdint>
#include <initializer_list>

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

// Lanes per event (2^k) of a call that asks for single helicities: as many as keep it
// within `turn` lanes, one turn of the chip (at most 64, at most one per helicity).  Such
// a call takes the time of one lane's helicities, however few its events are (64 events of
// g g -> t tbar g g 2.8 ms at one lane each, 0.06 at 64).  A call of half a turn or more
// gains nothing: the VALU is busy with one wave per SIMD.
static inline int me_turn_lanes_lg(int64_t nevt, int nhel, int64_t turn) {
    int lg = 0;
    while (lg < 6 && nevt <= (turn >> (lg + 1)) && (2 << lg) <= nhel) ++lg;
    return lg;
}

// Mixed form, one event per lane: helicities per block where their values are added by a
// kernel of their own (nh: not done).  One wave takes 45 us per helicity of g g -> t tbar g g and the
// chip holds 1024 of these waves, so a call of up to 65,536 events took the 2.9 ms
// of 64 helicities in turn (64 events now 72 us, 16,384 0.81 ms, with the
// rerun), and one of a few more than a multiple of it a whole turn more (70,000
// events 3.3 ms against 5.8).  Where the last turn is not nearly full the list is
// parted until there are 8 turns of blocks, whose setup is a tenth of a
// helicity's work; where it is full that costs 2 % (131,072 events 6.0 ms against 5.9).
static inline int mixed_per_block(int64_t nevt, int nh) {
    const int64_t tiles = (nevt + 63) / 64, turns = (tiles + 1023) / 1024;
    int per = nh;
    if (10 * 1024 * turns <= 11 * tiles) return per;
    while (per > 1 && tiles * ((nh + per - 1) / per) < 8 * 1024) per = (per + 1) / 2;
    return per;
}

// Buffers that grow together: their pointers and new sizes in bytes, `cap` the number of
// elements they hold.  Frees the old ones and allocates new ones for n elements.  After
// a failure cap is 0 and every pointer is null or a live buffer, so that the next
// call grows them again and none is used or freed after its release.
struct me_buffer {
    void** p;
    size_t bytes;
};
template <class Alloc, class Free>
static inline auto me_regrow(int64_t n, int64_t& cap, std::initializer_list<me_buffer> bufs, Alloc&& alloc,
                             Free&& release) -> decltype(release((void*)nullptr)) {
    typedef decltype(release((void*)nullptr)) status;
    cap = 0;
    for (const me_buffer& b : bufs) {
        void* old = *b.p;
        *b.p = nullptr;
        const status e = old ? release(old) : status(0);
        if (e != status(0)) return e;
    }
    for (const me_buffer& b : bufs) {
        const status e = alloc(b.p, b.bytes);
        if (e != status(0)) {
            *b.p = nullptr;
            return e;
        }
    }
    cap = n;
    return status(0);
}

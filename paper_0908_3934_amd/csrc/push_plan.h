// Shape of a network in the push ensemble kernel and the numbering of its
// words of spike bits: plain C++, shared by the planner and the kernel.
#pragma once

#include <cstddef>
#include <cstdint>

#ifdef __HIPCC__
#define GEONET_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define GEONET_HOST_DEVICE inline
#endif

namespace geonet {

// A step's words of a network are numbered window * groups + group.  The window
// of word k is (k * inv) >> kWordShift with inv = ceil(2^kWordShift / groups):
// exact where k * (groups * inv - 2^kWordShift) < 2^kWordShift, whose left side
// is below 255 * 128 * 128 for the most windows and groups there are, and
// k * inv < 255 * (2^kWordShift + groups) fits 32 bits.  (20 bits were too few:
// 123 groups with 80 windows took word 8,609 for one of window 70.)
constexpr int kWordShift = 24, kWordMaxGroups = 128, kWordMaxWindows = 255;

GEONET_HOST_DEVICE uint32_t word_inverse(uint32_t groups) { return ((1u << kWordShift) + groups - 1u) / groups; }
GEONET_HOST_DEVICE uint32_t word_window(uint32_t k, uint32_t inv) { return k * inv >> kWordShift; }

// The widest window of delays that `room` bytes of LDS and the bits of an edge
// word (`tbits` of them a target) have space for: each further window is one
// more visit per spike.  0: none has.
struct PushShape {
    int tbits = 1, window = 0, n_win = 0;
    size_t ring = 0, lds = 0;                  // bytes of the input slots, of all
};

inline PushShape push_shape(int64_t n, int max_delay, size_t room) {
    PushShape s;
    const size_t groups = static_cast<size_t>((n + 63) / 64);
    while ((int64_t(1) << s.tbits) < n) ++s.tbits;
    for (int w = max_delay < 1 << (16 - s.tbits) ? max_delay : 1 << (16 - s.tbits); w >= 1; --w) {
        const size_t n_win = static_cast<size_t>((max_delay + w - 1) / w);
        s.ring = static_cast<size_t>(w + 1) * groups * 64 * sizeof(float);
        s.lds = s.ring + ((n_win - 1) * static_cast<size_t>(w) + 2) * groups * 8 + 2 * 33 * sizeof(double);
        s.n_win = static_cast<int>(n_win);
        s.window = w;
        if (s.lds <= room) return s;
    }
    s.window = 0;
    return s;
}

}  // namespace geonet

// Values that a kernel hands to a polling host, each with the tag of the hand-over beside it.
//
// A tag after the values, however fenced, does not do: the stores leave the device in order but
// need not become visible in order across the cache lines of host memory.  With one tag in the
// third line, 7 of 5.4M reads found the line before it still holding the last iteration's
// values, which put the host a block width off the device (a solve in some thousands stopped
// with a rank-0 Delta or did not converge).  A value and its tag are one 16-byte store to one
// line, so a tag that has arrived vouches for its value.
#pragma once

#include <atomic>

namespace ba {

struct alignas(16) Tagged {
    double value, tag;
};

// The n values to out, once all of them bear `tag`; false (out unspecified) while one does not.
inline bool tagged_read(const volatile Tagged *v, int n, double tag, double *out) {
    for (int i = 0; i < n; ++i) {
        if (v[i].tag != tag) return false;
        std::atomic_thread_fence(std::memory_order_acquire);
        out[i] = v[i].value;
    }
    return true;
}

}  // namespace ba

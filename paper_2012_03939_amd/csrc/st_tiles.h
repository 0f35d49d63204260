// How the waves of a traversal launch share its tiles of 64 consecutive rays.  Plain
// C++, so that the hand-out can be run, and every tile counted, on the CPU as well.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define ST_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define ST_HOST_DEVICE inline
#endif

namespace st {

constexpr int TAKE_NC = 16;     // counters of a launch

// Calls fn(tile) for the tiles, of `tiles`, that fall to wave w of `waves`.  The first
// is the wave's own number; of the others, counter c hands out every nc-th, and take(c)
// returns how many it has given out before.  A wave takes from one counter alone, so no
// more counters are in use than there are waves: with all 16, the tiles of the counters
// from `waves` on would be nobody's in a launch of fewer (one of at most 768 paths, whose
// shadow rays, several a path, are more tiles than its waves).
template <class Take, class Fn>
ST_HOST_DEVICE void hand_out_tiles(uint32_t w, uint32_t waves, uint32_t tiles, Take take, Fn fn) {
    const uint32_t nc = waves < (uint32_t)TAKE_NC ? waves : (uint32_t)TAKE_NC;
    const uint32_t c = waves < (uint32_t)TAKE_NC ? w : w % (uint32_t)TAKE_NC;
    for (uint32_t t = w; t < tiles;) {
        uint32_t next = tiles;
        if (tiles > waves) next = waves + take(c) * nc + c;
        fn(t);
        t = next;
    }
}

} // namespace st

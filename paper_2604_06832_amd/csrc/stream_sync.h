// Words through which the wavefronts of a workgroup of the streaming forward kernel talk (stream_fwd.h), and the counters of its
// barriers (host and device).
#pragma once
#include <hip/hip_runtime.h>

namespace bd {

// words of the LDS synchronisation block
enum { SY_LANDED = 0, SY_CONSUMED = 4, SY_DEAD = 8, SY_CBAR = 9, SY_ARRIVE = 10, SY_EPOCH = 11, SY_XEPOCH = 12, SY_PACE = 13, SY_WORDS = 16 };

// Has a counter that only grows, and wraps, reached `target`?  (Good while the two are less than 2^31 apart.)
__host__ __device__ inline bool counter_reached(unsigned v, unsigned target) { return (int)(v - target) >= 0; }

// Value of word i when a launch starts: the barriers' words hold the last barriers of the launches before (the epochs number all
// barriers of a context; from zero they would count as reached once the context has run 2^31 of them, 15 million forwards of 36 layers).
__host__ __device__ inline unsigned sync_word_at_start(int i, unsigned pace, unsigned bar_epoch, unsigned xbar_epoch) {
  return i == SY_PACE ? pace : i == SY_EPOCH ? bar_epoch : i == SY_XEPOCH ? xbar_epoch : 0u;
}

}  // namespace bd

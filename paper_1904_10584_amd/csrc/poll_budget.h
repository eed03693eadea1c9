// How long a kernel polls for another workgroup before it gives up.
#pragma once

#ifdef __HIPCC__
#define AM_POLL_FN __host__ __device__ __forceinline__
#else
#define AM_POLL_FN inline
#endif

namespace am {

// Bounds the failed polls of each wait by itself (a pass may take any number of
// steps, each with a few of them); once one wait has run out, no later one waits.
template <unsigned LIMIT> struct PollBudget {
  unsigned failed = 0;  // of this wait, or beyond the limit for good
  AM_POLL_FN void begin() {
    if (failed <= LIMIT) failed = 0;
  }
  // Another poll has failed: whether to give up.
  AM_POLL_FN bool spent() { return ++failed > LIMIT; }
};

}  // namespace am

// The wait of a redo launch's items for those of the pass before (scan.hip, ivf.hip), which always ends.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define DCPQ_BOTH __host__ __device__
#else
#define DCPQ_BOTH
#endif

namespace dcpq {

// Looks before a wait is given up.  What is waited for is in the hands of running workgroups, and takes milliseconds at most over a flat array, a second over the
// longest lists; a look takes a microsecond or more, so that this many are some twenty seconds.  A wait comes to that only where another call overwrites the counters, that is where
// two calls share a workspace at the same time, which is not allowed; the launch then ends and its results are wrong.
constexpr uint32_t kRedoPatience = 1u << 24;

// In the counter that hands out the items: set by who gives up a wait, and the items handed out from then on are not worked on.
constexpr unsigned long long kRedoGivenUp = 1ull << 63;

// load() once it is n or more (true), or after `patience` looks (false).
template <typename Load, typename Pause>
DCPQ_BOTH inline bool wait_until(Load load, Pause pause, uint32_t n, uint32_t patience)
{
    for (uint32_t looks = 0; load() < n; ++looks) {
        if (looks == patience) return false;
        pause();
    }
    return true;
}

}  // namespace dcpq

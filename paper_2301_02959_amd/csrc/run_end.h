// How far a run of equal rows goes on over the chunks of a list, for the kernel that folds the runs' carries (bwd.hip).
#pragma once

#include "fs_common.h"

namespace fs {

// The last chunk that the run at the end of chunk `chunk` goes on into; it does go on into the next one.
//   far_too            whether it goes on into chunk `chunk` + 2
//   goes_on_into(c)    whether it goes on into chunk c < chunks
// Most runs end in the very next chunk, so the search gallops from there (1, 2, 4 .. chunks ahead) and then bisects: no
// further load for a short run instead of log2(m) dependent ones.
template <typename GoesOnInto>
__host__ __device__ inline int64_t last_chunk_of_run(int64_t chunk, int64_t chunks, bool far_too, GoesOnInto goes_on_into)
{
    int64_t lo = chunk + 1, step = 1;                                // it goes on into chunk lo
    bool go_on = far_too;
    while (go_on) {
        lo += step;
        step <<= 1;
        go_on = lo + step < chunks && goes_on_into(lo + step);
    }
    int64_t hi = lo + step < chunks ? lo + step : chunks;            // not into chunk hi (or there is none)
    while (hi - lo > 1) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (goes_on_into(mid)) lo = mid; else hi = mid;
    }
    return lo;
}

}  // namespace fs

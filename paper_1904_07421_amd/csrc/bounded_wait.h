// The wait of a block for words that other blocks of its launch write.
#pragma once

#include <climits>

namespace jitdb {

// Looks until look(need) holds, look(n) being whether every word is at least n, with rest() before every look; false when `looks` of them
// were not enough.  What is left of `looks` is the next wait's: a string of waits ends as well.  (Words that never come are given
// up by asking for less, so that the loop has one way out and nothing behind it: it is on the way of h from one block to the next.)
template <typename Look, typename Rest>
#ifdef __HIPCC__
__device__ __forceinline__
#else
inline
#endif
bool wait_bounded(int need, int &looks, Look &&look, Rest &&rest) {
    int least;
    bool seen;
    do {
        least = looks > 0 ? need : INT_MIN;
        rest();
        seen = look(least);
        --looks;
    } while (!seen);
    return least == need;
}

}  // namespace jitdb

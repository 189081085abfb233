// When a context's particle pool grows.  Host code without a device call.
#pragma once
#include <cstdint>

namespace ugk {

enum : unsigned long long { POOL_REFUSED = 1 };     // bit of the error word: a step found no room

// The slots that a step which found no room needs, or 0 when it was not refused for that or
// the capacity does not hold them.  What else the refused step raised means nothing: its
// sweeps ran without its particles.
inline int64_t pool_need(unsigned long long err, int64_t have, int64_t capacity, int64_t slots, int64_t births)
{
    if (!(err & POOL_REFUSED) || have >= capacity || births > capacity - slots) return 0;
    return slots + births;
}

}  // namespace ugk

// A context's particle pool: when it grows, to what size, and its move to another
// allocation.  Host code without a device call of its own.
#pragma once
#include <algorithm>
#include <array>
#include <cstddef>
#include <cstdint>
#include <memory>
#include <new>
#include <vector>

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

// The sizes a pool of `have` slots tries when it needs `need`, in this order: four times the
// pool, so that copies stay few, a quarter more than needed, and what is needed.
inline std::array<int64_t, 3> pool_sizes(int64_t need, int64_t have, int64_t capacity)
{
    const int64_t roomy = std::min(need + need / 4, capacity);
    return {std::min(std::max(roomy, 4 * have), capacity), roomy, need};
}

// An array of the pool: bytes per slot, and whether it holds the committed particles
// (the other half of each pair is scratch between steps).
struct PoolArray {
    int per;
    bool live;
};

inline size_t pool_bytes(int64_t cap, int per) { return ((size_t)cap * per + 255) / 256 * 256; }

inline size_t pool_total(const std::vector<PoolArray>& arrays, int64_t cap)
{
    size_t t = 0;
    for (const PoolArray& a : arrays) t += pool_bytes(cap, a.per);
    return t;
}

enum class PoolMove { done, no_memory, failed, lost };

// The allocation *mem of *cap slots with n committed particles exchanged for one of the first
// of `sizes` that can be had.  Where the device does not hold both, the particles wait in
// host memory while the old allocation makes room, so that a pool reaches any size that
// fits by itself.  no_memory, failed (a copy): the pool is as it was; lost (somebody else took
// the memory in between): there is none.  Mem:
//   void* alloc(size_t)                      device memory or nullptr
//   void release(void*)
//   size_t room()                            free device memory
//   void within / down / up(to, from, bytes) copies on the context's stream
//   bool wait()                              for them; false: one failed
template <class Mem>
PoolMove pool_move(Mem& m, const std::vector<PoolArray>& arrays, void** mem, int64_t* cap, int64_t n,
                   const std::array<int64_t, 3>& sizes)
{
    // every committed array: its place in a pool of c slots, in the old one, and one after another
    auto each = [&](int64_t c, auto&& copy) {
        size_t to = 0, from = 0, packed = 0;
        for (const PoolArray& a : arrays) {
            const size_t bytes = (size_t)n * a.per;
            if (a.live && n > 0) copy(to, from, packed, bytes);
            if (a.live) packed += bytes;
            to += pool_bytes(c, a.per);
            from += pool_bytes(*cap, a.per);
        }
        return packed;
    };
    char* const old = (char*)*mem;
    for (int64_t c : sizes) {
        char* p = (char*)m.alloc(pool_total(arrays, c));
        if (!p) continue;
        each(c, [&](size_t to, size_t from, size_t, size_t bytes) { m.within(p + to, old + from, bytes); });
        if (!m.wait()) {
            m.release(p);
            return PoolMove::failed;
        }
        if (old) m.release(old);
        *mem = p;
        *cap = c;
        return PoolMove::done;
    }
    if (!old || m.room() + pool_total(arrays, *cap) < pool_total(arrays, sizes.back())) return PoolMove::no_memory;
    const size_t packed = each(*cap, [](size_t, size_t, size_t, size_t) {});
    std::unique_ptr<char[]> host(new (std::nothrow) char[packed + 1]);
    if (!host) return PoolMove::no_memory;
    each(*cap, [&](size_t, size_t from, size_t at, size_t bytes) { m.down(host.get() + at, old + from, bytes); });
    if (!m.wait()) return PoolMove::failed;
    m.release(old);
    *mem = nullptr;
    for (int64_t c : {sizes[0], sizes[1], sizes[2], *cap}) {
        char* p = (char*)m.alloc(pool_total(arrays, c));
        if (!p) continue;
        each(c, [&](size_t to, size_t, size_t at, size_t bytes) { m.up(p + to, host.get() + at, bytes); });
        if (!m.wait()) {
            m.release(p);
            return PoolMove::lost;
        }
        *mem = p;
        const bool grown = c >= sizes[2];
        *cap = c;
        return grown ? PoolMove::done : PoolMove::no_memory;
    }
    return PoolMove::lost;
}

}  // namespace ugk

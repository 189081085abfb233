// Moves a pool of `have` slots with n particles to `need` slots on a device of `budget`
// bytes, of which `taken` are taken by somebody else as soon as the old pool is released;
// copy number `bad` fails (0: none).  Prints the outcome, the slots, whether every committed
// byte is in its place, the copies through the host, and the bytes still allocated.
#include "../../paper_2312_16981_amd/csrc/pool.hpp"
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

using namespace ugk;

struct Fake {
    size_t budget, taken;
    int bad, copies = 0, host = 0;
    std::map<void*, size_t> live;
    size_t used() const
    {
        size_t s = 0;
        for (auto& q : live) s += q.second;
        return s;
    }
    size_t room() { return budget - used(); }
    void* alloc(size_t n)
    {
        if (n > room()) return nullptr;
        void* p = std::malloc(n);
        live[p] = n;
        return p;
    }
    void release(void* p)
    {
        std::free(p);
        live.erase(p);
        budget -= taken;
        taken = 0;
    }
    void copy(void* to, const void* from, size_t n)
    {
        if (++copies != bad) std::memcpy(to, from, n);
    }
    void within(void* to, const void* from, size_t n) { copy(to, from, n); }
    void down(void* to, const void* from, size_t n) { ++host; copy(to, from, n); }
    void up(void* to, const void* from, size_t n) { ++host; copy(to, from, n); }
    bool wait() { return bad == 0 || copies < bad; }
};

int main(int, char** a)
{
    const long long have = std::atoll(a[1]), n = std::atoll(a[2]), need = std::atoll(a[3]), cap = std::atoll(a[4]);
    // the moving pair x, cell and the stable nu, with the committed half first or second
    const std::vector<PoolArray> A = {{8, true}, {4, true}, {8, false}, {8, false}, {4, false}, {8, true}};
    Fake m{(size_t)std::atoll(a[5]), (size_t)std::atoll(a[6]), std::atoi(a[7])};
    void* mem = m.alloc(pool_total(A, have));
    int64_t slots = have;
    auto fill = [&](char* p, int64_t c, bool check) {
        size_t at = 0;
        bool same = true;
        for (size_t q = 0; q < A.size(); ++q) {
            for (size_t b = 0; A[q].live && b < (size_t)n * A[q].per; ++b) {
                const char v = (char)(31 * q + b * 7 + b / 256);
                if (check) same = same && p[at + b] == v;
                else p[at + b] = v;
            }
            at += pool_bytes(c, A[q].per);
        }
        return same;
    };
    fill((char*)mem, have, false);
    const PoolMove r = pool_move(m, A, &mem, &slots, n, pool_sizes(need, have, cap));
    std::printf("%d %lld %d %d %zu\n", (int)r, (long long)slots, mem ? (int)fill((char*)mem, slots, true) : -1, m.host,
                m.used());
    if (mem) std::free(mem);
}

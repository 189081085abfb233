// Prints what a refused step's pool grows to, one line per line of
// "error have capacity slots births".
#include "../../paper_2312_16981_amd/csrc/pool.hpp"
#include <cstdio>

int main()
{
    unsigned long long err;
    long long have, cap, slots, births;
    while (std::scanf("%llu %lld %lld %lld %lld", &err, &have, &cap, &slots, &births) == 5)
        std::printf("%lld\n", (long long)ugk::pool_need(err, have, cap, slots, births));
}

// CPU check of map_builders (test infrastructure): over sides and numbers of maps
// up to the largest that the interface takes, the maps built at once fit LDS and
// the block's waves, and take the fewest rounds.
#include "../../paper_2301_11735_amd/csrc/kernels.h"

#include <cstdio>

int main()
{
    const uint32_t counts[] = {1, 2, 3, 8, 9, 14, 15, 16, 17, 20, 33, 1000, 1u << 31, 0xFFFFFFF0u, 0xFFFFFFF1u, 0xFFFFFFF9u, 0xFFFFFFFFu};
    for (int L = 4; L <= lat::kMapMaxL; L += 4) {
        uint64_t most = lat::kMapThreads / 64;
        while (most > 1 && lat::map_lds_bytes(L, (int)most) > lat::kMapLdsMax) --most;
        for (uint32_t n : counts) {
            const uint64_t g = (uint64_t)lat::map_builders(L, n), rounds = (n + most - 1) / most;
            if (g < 1 || g > most || g > n || (n + g - 1) / g != rounds) {
                std::printf("L = %d, %u maps: %llu builders, at most %llu\n", L, n, (unsigned long long)g, (unsigned long long)most);
                return 1;
            }
        }
    }
    std::printf("OK\n");
    return 0;
}

// Prints the tuner's keys of the problems given on the command line, one line each: "t batched n runs P S runout" or
// "s kind n cap P S velocity"; and the velocity rule of
// "v slots P 0 0 0 0" as 0 (table), 1 (straight first if chosen) or 2 (straight).
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "../../paper_2506_23364_amd/csrc/tuning.h"

int main(int argc, char** argv) {
    for (int i = 1; i < argc;) {
        const bool smooth = std::strcmp(argv[i], "s") == 0;
        long long v[6] = {};
        const int n = 6;
        if (i + 6 >= argc) return 1;
        for (int k = 0; k < 6; ++k) v[k] = std::atoll(argv[i + 1 + k]);
        if (argv[i][0] == 'v') {
            const auto slots = (unsigned long long)v[0];
            const auto P = (uint32_t)v[1];
            std::printf("%d\n", avl::velocity_straight(slots, P) ? 2 : avl::velocity_straight_first(slots, P) ? 1 : 0);
            i += 7;
            continue;
        }
        i += 7;
        const auto key = smooth ? avl::smooth_key(0, (int)v[0], v[1], v[2], (uint32_t)v[3], (uint32_t)v[4], v[5] != 0)
                                : avl::tune_key(0, v[0] != 0, v[1], v[2], (uint32_t)v[3], (uint32_t)v[4], v[5] != 0);
        for (auto k : key) std::printf("%lld ", (long long)k);
        std::printf("\n");
    }
    return 0;
}

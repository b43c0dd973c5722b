// What the autotuner keeps a choice for, and a rule that its choice enters: plain code without HIP, so that it can be tested by
// itself. A key separates the
// problems that run different kernels or sizes far apart (each size by its power of two); key[1] is the kind: 0 single run,
// 1 batch, 2 smooth forward, 3 adjoint.
#pragma once

#include <cstdint>
#include <vector>

namespace avl {

inline int ilog2(uint64_t v) {
    int r = 0;
    while (v > 1) {
        v >>= 1;
        ++r;
    }
    return r;
}

// runout: a single run with the runout-angle stop runs an instantiation of its own (a batch always has the stop compiled in).
// With one choice for both, a 1001 x 1203 pass of 32 particles a texel without the stop took 394 us after one with it, 356 with
// a shape of its own.
inline std::vector<int64_t> tune_key(int dev, bool batched, int64_t n, int64_t n_runs, uint32_t P, uint32_t S, bool runout) {
    return {dev, batched ? 1 : 0, ilog2((uint64_t)n), ilog2((uint64_t)n_runs), ilog2(P), ilog2((uint64_t)S + 1),
            runout && !batched ? 1 : 0};
}

// velocity: the forward with the velocity raster is a kernel of its own (other tables, a barrier every few steps), so a
// shape found for the deposit alone says nothing about it. With one choice for both, a velocity pass after a deposit of its
// size took the deposit's shape: 40,000 particles of 4 a cell 233 us, with its own 216; 640,000 of 128 a cell 639 and 612.
inline std::vector<int64_t> smooth_key(int dev, int kind, int64_t n, int64_t cap, uint32_t P, uint32_t S, bool velocity) {
    return {dev, kind, ilog2((uint64_t)n), ilog2((uint64_t)cap + 1), ilog2(P), ilog2((uint64_t)S + 1), velocity ? 1 : 0};
}

// How the smooth forward adds its velocity splats, for `slots` particles of P a release cell: straight to the raster or through
// a table in LDS. Few particles stay below the rate of the memory side's adds, which nothing waits for, while the table's round
// trips and barriers lengthen each step; and the fewer particles share a release cell, the fewer splats the table can merge.
// Straight for sure up to kDirectSlots particles, and with up to eight a cell up to 128 kDirectSlots / P^2.
constexpr unsigned long long kDirectSlots = 3072;
constexpr bool velocity_straight(unsigned long long slots, uint32_t P) {
    return slots <= kDirectSlots || (P <= 8u && slots * P * P <= 128u * kDirectSlots);
}
// Past that the length of the paths decides, which no size shows: paths of some 12 steps, us through the table and straight for
// their first 32 pairs of steps: 40,000 particles of 4 a cell 247 and 175, 80,000 of 4 250 and 211, 40,000 of 8 183 and 157,
// 10,000 of 8 136 and 111; paths of 100 steps and more: 1959 and 2018, 3026 and 3388, 1865 and 2077, 231 and 330. So up to
// 1024 kDirectSlots / P^2 the tuner times both and the chosen form may start straight; with the table taking over, a choice
// made on short paths costs long ones of its size class 1.03 to 1.5 times their time (straight to the end: up to 1.8). Beyond,
// the table wins on both (320,000 of 4 376 and 479). With more than eight a cell starting straight would win a tenth at most
// (6000 of 10 82 and 77, 15,000 of 10 140 and 122) and a wrong choice cost 1.4 to 1.8 times, so there the table it is.
constexpr uint32_t kStraightReplicas = 8;
constexpr bool velocity_straight_first(unsigned long long slots, uint32_t P) {
    return P <= kStraightReplicas && slots * P * P <= 1024u * kDirectSlots;
}

}  // namespace avl

// What the autotuner keeps a choice for: plain host code without HIP, so that it can be tested by itself. A key separates the
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

}  // namespace avl

// Run tables on the device: the checks of a run's parameters and its derived constants.
#pragma once

#include "particle.h"

namespace avl {

// Why a run releases nothing: 1 an index out of range, 2 invalid parameters, 3 more release cells than cap_cells (< 0:
// no limit); 0 if it runs.
__device__ __forceinline__ int32_t param_status(const ::avl_params& p) {
    const bool ok = __builtin_isfinite(p.mu) && p.mu >= 0.0f && !__builtin_isnan(p.xi) && p.xi > 0.0f &&
                    __builtin_isfinite(p.flow_height) && p.flow_height > 0.0f && p.persistence >= 0.0f &&
                    p.persistence <= 1.0f && __builtin_isfinite(p.randomness) && p.randomness >= 0.0f &&
                    __builtin_isfinite(p.step_cells) && p.step_cells > 0.0f && p.step_cells <= 16.0f &&
                    __builtin_isfinite(p.tan_alpha) && p.flags == 0u;
    return ok ? 0 : 2;
}

// Derived constants of a run, binary32, in this order. raster_off, n_slots and use_rec are the caller's.
__device__ __forceinline__ RunConst run_const(const RunSpec& sp, const ::avl_params& p, int32_t H, int32_t W, float cs,
                                              uint32_t P) {
    const uint64_t HW = (uint64_t)H * W;
    RunConst c{};
    const float g = 9.81f;
    const float g2 = g + g;
    c.per = p.persistence;
    c.Q = 1.0f - c.per;
    c.rnd = p.randomness;
    c.L = p.step_cells;
    const float dl = c.L * cs;
    c.dl2 = dl * dl;
    c.mdl = p.mu * dl;
    c.cd = g2 / (p.xi * p.flow_height);
    c.use_alpha = p.tan_alpha >= 0.0f ? 1u : 0u;
    c.tca = p.tan_alpha * cs;
    c.key0 = (uint32_t)sp.seed;
    c.key1 = (uint32_t)(sp.seed >> 32);
    c.run = sp.run_id;
    c.dem_off = (uint32_t)(sp.tile * HW);
    c.pad_off = (uint32_t)(sp.tile * (uint64_t)padded_cells(H, W));
    c.cells_off = (uint32_t)(sp.scenario * HW);
    c.P = P;
    return c;
}

// The run table of a single run with n release cells.
__device__ __forceinline__ void setup_one(const SetupOne& u, int32_t H, int32_t W, int64_t n) {
    const RunSpec sp = u.spec_dev ? *u.spec_dev : u.spec;
    const ::avl_params p = u.p_dev ? *u.p_dev : u.p;
    int32_t bad = (sp.tile != 0u || sp.scenario != 0u || sp.param != 0u) ? 1 : param_status(p);
    if (!bad && u.cap_cells >= 0 && n > u.cap_cells) bad = 3;
    RunConst c = run_const(sp, p, H, W, u.cs, u.P);
    c.n_slots = bad ? 0ull : (unsigned long long)(uint32_t)n * u.P;
    *u.run = c;
    u.run_off[0] = 0ull;
    u.run_off[1] = (c.n_slots + dev::kChunk - 1) / dev::kChunk * dev::kChunk;
    if (u.status) *u.status = bad;
}

}  // namespace avl

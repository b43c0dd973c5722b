// Device helpers shared by the particle kernels (plain, batched, smooth forward and adjoint): the
// random stream, the bilinear height patch and the wave-level queue utilities. Internal header.
#pragma once

#include "avl_internal.h"

namespace avl {
namespace dev {

constexpr uint32_t kChunk = 64;  // particle slots taken from a queue per reservoir refill

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of the 4x32 multiply-xor bijection with a Weyl key
// schedule.
__device__ __forceinline__ uint4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                               uint32_t k1) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        // each 32 x 32 -> 64-bit product as one v_mad_u64_u32 (both halves at the cost of one quarter-rate
        // multiply; a low and a high multiply written apart are two)
        const uint64_t p0 = (uint64_t)c0 * 0xD2511F53u, p1 = (uint64_t)c2 * 0xCD9E8D57u;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        // three-way XORs as single gfx950 three-input bit operations (truth table 0x96)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c3, k1, 0x96);
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return make_uint4(c0, c1, c2, c3);
}

// Square root and reciprocal square root from one hardware estimate y of 1 / sqrt(x) (1 ulp), one quarter-rate
// instruction for both where an estimate each for the root and for the division by it would be two.
//
// Root: s0 = x y, then one residual step s = s0 + (x - s0 s0) (y / 2) (Goldschmidt's iteration closed by Markstein's
// residual correction, both through fma). Equal to the correctly rounded sqrtf(x) for every one of the binary32
// numbers in [2^-96, max]: checked for all 2.0e9 of them on gfx950 (a GPU test repeats it). +inf gives NaN.
struct RootEst {
    float s, y;  // sqrt(x) correctly rounded; the estimate of 1 / s
};
__device__ __forceinline__ RootEst sqrt_est(float x) {
    RootEst r;
    r.y = __builtin_amdgcn_rsqf(x);
    const float s0 = x * r.y;
    r.s = __builtin_fmaf(__builtin_fmaf(-s0, s0, x), 0.5f * r.y, s0);
    return r;
}

// 1 / s correctly rounded, s = sqrt(x): two Newton steps on the estimate moved up by one ulp. From below, the
// iteration misses the s whose significand is all ones, the one case Markstein's theorem leaves out; from above it
// reaches that one too. Equal to 1 / sqrtf(x) for every binary32 x in [2^-96, max] (the same check).
__device__ __forceinline__ float recip_root(const RootEst& e) {
    const float y = __uint_as_float(__float_as_uint(e.y) + 1u);
    const float r = __builtin_fmaf(__builtin_fmaf(-e.s, y, 1.0f), y, y);
    return __builtin_fmaf(__builtin_fmaf(-e.s, r, 1.0f), r, r);
}

// q / s correctly rounded for q = 0 or |q| in [2^-40, 2^40] and s in [2^-40, 2^40]: with r = 1 / s correctly rounded
// and q r within an ulp of the quotient, one residual step rounds it correctly (Markstein, IBM J. Res. Dev. 34, 1990).
__device__ __forceinline__ float div_root(float q, const RootEst& e) {
    const float r = recip_root(e);
    const float q0 = q * r;
    return __builtin_fmaf(__builtin_fmaf(-e.s, q0, q), r, q0);
}

// sqrtf(x) for x >= 0 or NaN: sqrt_est, unless a lane of the wave holds a value whose bits are below `lo` (those of 2^-96,
// or 0 where no lane can hold a smaller number than 2^-96), an infinity or a NaN, when the whole wave takes sqrtf (a
// wave-uniform branch, so the common case pays one compare).
constexpr uint32_t kRootLo = 0x0F800000u;  // 2^-96
__device__ __forceinline__ float sqrt_rn(float x, uint32_t lo) {
    if (__builtin_expect(__ballot(__float_as_uint(x) - lo > 0x7F7FFFFFu - lo) != 0ull, 0)) return sqrtf(x);
    return sqrt_est(x).s;
}

// x in [2^-80, 2^80] (one unsigned compare of the bits; 0, NaN and negative x fall outside), so that sqrt(x) lies in
// [2^-40, 2^40], for every active lane of the wave: a wave-uniform value, so that the direction's two quotients by a
// root run without a branch per lane.
__device__ __forceinline__ bool all_mid_range(float x) {
    return __builtin_expect(__ballot(__float_as_uint(x) - 0x17800000u > 0x67800000u - 0x17800000u) == 0ull, 1);
}

// the same with 0 and NaN allowed, whose quotients are selected away: lakes, clamped and masked heights are exactly flat, and the
// lanes beside a flat one keep the short form
__device__ __forceinline__ bool all_mid_range_or_unused(float x) {
    return __ballot(x > 0.0f && __float_as_uint(x) - 0x17800000u > 0x67800000u - 0x17800000u) == 0ull;
}

// The step's new direction in place: w = (per d - t g) + rnd r with t = Q / |g| (0 on flat ground), d = w / |w| (kept
// where w = 0). Q = 1 - persistence is 0 or in [2^-24, 1]. Both roots and quotients are correctly rounded.
// The step is bound by VALU issue when the chip is full and by its own dependent chain when it is not: against an
// estimate each for root, root correction by its neighbours and reciprocal, this form issues about 19 slots less a step
// (8192^2 pass of 1.2e9 steps 8.72 -> 8.51 ms, 30,000-particle overlay 210 -> 203 us).
// A wave with a flat lane keeps the short form (2048^2 tile, heights clamped at their 0.8 quantile, 2.3e8 steps: 1755 -> 1695 us;
// at 0.5, 6.1e8 steps: 4030 -> 3980).
__device__ __forceinline__ void steer(float& dx, float& dy, float gx, float gy, float per, float Q, float rnd, float rx,
                                      float ry) {
    const float gg = gx * gx + gy * gy;
    float t = div_root(Q, sqrt_est(gg));
    if (!all_mid_range(gg)) {
        if (!all_mid_range_or_unused(gg)) t = Q / sqrtf(gg);
        t = gg > 0.0f ? t : 0.0f;
    }
    const float wx = (per * dx - t * gx) + rnd * rx;
    const float wy = (per * dy - t * gy) + rnd * ry;
    const float ww = wx * wx + wy * wy;
    float inv = recip_root(sqrt_est(ww));
    if (all_mid_range(ww)) {
        dx = wx * inv;
        dy = wy * inv;
    } else {
        if (!all_mid_range_or_unused(ww)) inv = 1.0f / sqrtf(ww);
        dx = ww > 0.0f ? wx * inv : dx;
        dy = ww > 0.0f ? wy * inv : dy;
    }
}

// inclusive sum over the wave's lanes
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        uint32_t t = __shfl_up(v, d, kWave);
        if (lane >= d) v += t;
    }
    return v;
}

// 24 random bits m -> 2 (m 2^-24) - 1, uniform in [-1, 1). Both products are exact and so is the difference
// ((m - 2^23) 2^-23 needs at most 24 significant bits), so one fma gives the same bits.
__device__ __forceinline__ float signed_unit(uint32_t u) {
    return __builtin_fmaf((float)(u >> 8), 0x1p-23f, -1.0f);
}

struct Sample {
    float z, gx, gy;
};

// Bilinear patch through the four texel centres around (x, y), indices clamped to the grid.
__device__ __forceinline__ Sample bilinear(const float* __restrict__ dem, int H, int W, float x, float y) {
    const float sx = x - 0.5f, sy = y - 0.5f;
    const float fc = floorf(sx), fr = floorf(sy);
    const float fx = sx - fc, fy = sy - fr;
    const int c0 = (int)fc, r0 = (int)fr;
    const int ca = min(max(c0, 0), W - 1), cb = min(max(c0 + 1, 0), W - 1);
    const int ra = min(max(r0, 0), H - 1), rb = min(max(r0 + 1, 0), H - 1);
    const float* rowa = dem + (size_t)ra * W;
    const float* rowb = dem + (size_t)rb * W;
    const float a = rowa[ca], b = rowa[cb], c = rowb[ca], d = rowb[cb];
    const float top = a + fx * (b - a);
    const float bot = c + fx * (d - c);
    Sample s;
    s.z = top + fy * (bot - top);
    s.gx = (b - a) + fy * ((d - c) - (b - a));
    s.gy = bot - top;
    return s;
}

// The same patch read from the DEM with a one-texel replicated border (row length Wp = W + 2 texels,
// row_bytes = 4 Wp) through a buffer resource: for (x, y) inside the grid the corner (floor(x - 1/2),
// floor(y - 1/2)) lies in [-1, W - 1] x [-1, H - 1], i.e. inside the padded grid, and the border holds
// exactly the clamped texels, so the four values and the arithmetic are those of bilinear().
// In two parts, so that work that does not need the heights can run while they are on their way.
struct PatchLoad {
    float a, b, c, d, fx, fy;
};
__device__ __forceinline__ PatchLoad bilinear_pad_load(__amdgpu_buffer_rsrc_t rs, uint32_t Wp, uint32_t row_bytes, float x,
                                                       float y) {
    const float sx = x - 0.5f, sy = y - 0.5f;
    const float fc = floorf(sx), fr = floorf(sy);
    const uint32_t off = (__umul24((uint32_t)((int)fr + 1), Wp) + (uint32_t)((int)fc + 1)) * 4u;
    // two 8-byte loads (the raw words of a, b and of c, d), both issued before either is used
    const auto ab = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
    const auto cd = __builtin_amdgcn_raw_buffer_load_b64(rs, off, row_bytes, 0);
    __builtin_amdgcn_sched_barrier(0);  // keep both loads ahead of their uses (one memory latency, not two)
    return PatchLoad{__uint_as_float(ab[0]), __uint_as_float(ab[1]), __uint_as_float(cd[0]), __uint_as_float(cd[1]),
                     sx - fc, sy - fr};
}
__device__ __forceinline__ Sample bilinear_pad_value(const PatchLoad& p) {
    const float top = p.a + p.fx * (p.b - p.a);
    const float bot = p.c + p.fx * (p.d - p.c);
    Sample s;
    s.z = top + p.fy * (bot - top);
    s.gx = (p.b - p.a) + p.fy * ((p.d - p.c) - (p.b - p.a));
    s.gy = bot - top;
    return s;
}
__device__ __forceinline__ Sample bilinear_pad(__amdgpu_buffer_rsrc_t rs, uint32_t Wp, uint32_t row_bytes, float x,
                                               float y) {
    return bilinear_pad_value(bilinear_pad_load(rs, Wp, row_bytes, x, y));
}

// buffer resource over `bytes` bytes at p (gfx9 descriptor word 3: 32-bit data format)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// Corners and fractions of the bilinear patch (or splat) at (x, y), indices clamped to the grid.
struct Corners {
    int ca, cb, ra, rb;
    float fx, fy;
};
__device__ __forceinline__ Corners corners(int H, int W, float x, float y) {
    const float sx = x - 0.5f, sy = y - 0.5f;
    const float fc = floorf(sx), fr = floorf(sy);
    Corners k;
    k.fx = sx - fc;
    k.fy = sy - fr;
    const int c0 = (int)fc, r0 = (int)fr;
    k.ca = min(max(c0, 0), W - 1);
    k.cb = min(max(c0 + 1, 0), W - 1);
    k.ra = min(max(r0, 0), H - 1);
    k.rb = min(max(r0 + 1, 0), H - 1);
    return k;
}

// Start state of release texel `texel` of a release texture with mult x mult texels per DEM cell (row-major,
// W * mult wide): its centre ((c + 1/2) / mult, (r + 1/2) / mult) in DEM cell units (mult = 1: the centre of
// DEM cell `texel`), the bilinear sample there and the unit direction of steepest descent (zero on flat
// ground). `cell` keeps the texel index, which keys the particle's random stream.
__device__ __forceinline__ StartRec start_state(const float* __restrict__ dem, int H, int W, uint32_t mult,
                                                uint32_t texel) {
    StartRec st;
    const uint32_t Wf = (uint32_t)W * mult;
    const uint32_t r = texel / Wf;
    const uint32_t c = texel - r * Wf;
    const float fm = (float)mult;
    st.x = ((float)c + 0.5f) / fm;
    st.y = ((float)r + 0.5f) / fm;
    const Sample s0 = bilinear(dem, H, W, st.x, st.y);
    st.z = s0.z;
    st.gx = s0.gx;
    st.gy = s0.gy;
    const float gg = s0.gx * s0.gx + s0.gy * s0.gy;
    if (gg > 0.0f) {
        const float t = 1.0f / sqrtf(gg);
        st.dx = -(s0.gx * t);
        st.dy = -(s0.gy * t);
    } else {
        st.dx = 0.0f;
        st.dy = 0.0f;
    }
    st.cell = texel;
    return st;
}

// start state at the centre of DEM cell `cell`, with the patch read from the padded DEM (the same values, so the same result)
__device__ __forceinline__ StartRec start_state_pad(__amdgpu_buffer_rsrc_t rs, uint32_t Wp, uint32_t row_bytes, int W,
                                                    uint32_t cell) {
    StartRec st;
    const int r = (int)(cell / (uint32_t)W);
    const int c = (int)(cell - (uint32_t)r * (uint32_t)W);
    st.x = (float)c + 0.5f;
    st.y = (float)r + 0.5f;
    const Sample s0 = bilinear_pad(rs, Wp, row_bytes, st.x, st.y);
    st.z = s0.z;
    st.gx = s0.gx;
    st.gy = s0.gy;
    const float gg = s0.gx * s0.gx + s0.gy * s0.gy;
    if (gg > 0.0f) {
        const float t = 1.0f / sqrtf(gg);
        st.dx = -(s0.gx * t);
        st.dy = -(s0.gy * t);
    } else {
        st.dx = 0.0f;
        st.dy = 0.0f;
    }
    st.cell = cell;
    return st;
}

__device__ __forceinline__ uint32_t udiv(uint32_t n, const DivU32& d) {
    const uint32_t t = __umulhi(d.mul, n);
    return (t + ((n - t) >> d.sh1)) >> d.sh2;
}

__device__ __forceinline__ uint64_t wave_bcast64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t wave_sum64(uint64_t v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

__device__ __forceinline__ uint32_t xcd_id() {
    // HW_REG_XCC_ID bits [3:0]: the XCD this wave runs on
    return __builtin_amdgcn_s_getreg((3 << 11) | 20) & (uint32_t)(kXcds - 1);
}

__device__ __forceinline__ float uniform_f(float v) {
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}
__device__ __forceinline__ uint32_t uniform_u(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// The run constants held in scalar registers (every lane has the same run).
__device__ __forceinline__ RunConst uniform_run(const RunConst& r) {
    RunConst u = r;
    u.per = uniform_f(r.per);
    u.Q = uniform_f(r.Q);
    u.rnd = uniform_f(r.rnd);
    u.L = uniform_f(r.L);
    u.dl2 = uniform_f(r.dl2);
    u.mdl = uniform_f(r.mdl);
    u.cd = uniform_f(r.cd);
    u.tca = uniform_f(r.tca);
    u.key0 = uniform_u(r.key0);
    u.key1 = uniform_u(r.key1);
    u.run = uniform_u(r.run);
    u.use_alpha = uniform_u(r.use_alpha);
    u.dem_off = uniform_u(r.dem_off);
    u.cells_off = uniform_u(r.cells_off);
    u.raster_off = uniform_u(r.raster_off);
    u.P = uniform_u(r.P);
    u.n_slots = ((unsigned long long)uniform_u((uint32_t)(r.n_slots >> 32)) << 32) | uniform_u((uint32_t)r.n_slots);
    // the DEM tile's offset builds the buffer resource of every gather: a value the compiler cannot prove
    // uniform there makes each buffer load a loop over the distinct resources of the wave's lanes
    u.pad_off = uniform_u(r.pad_off);
    u.use_rec = uniform_u(r.use_rec);
    return u;
}

// Run holding padded slot `slot`: the r with run_off[r] <= slot < run_off[r + 1]. Wave-uniform input.
__device__ __forceinline__ uint32_t find_run(const unsigned long long* __restrict__ off, uint32_t n_runs,
                                             uint64_t slot) {
    uint32_t lo = 0, hi = n_runs;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (off[mid] <= slot)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// start of XCD partition p of the padded slot range [0, total): a multiple of kChunk
__device__ __forceinline__ uint64_t part_begin(uint64_t total, uint32_t p) {
    if (p >= (uint32_t)kXcds) return total;
    return (total / kChunk * p / kXcds) * kChunk;
}

// Blocks of a persistent grid that take part for `total` slots: enough for about `spl` slots per lane, at least one per XCD. A
// problem that does not fill the chip is over soonest with one slot per lane (30,000 paths of 11 steps 0.13 ms, 0.31 with
// eight); eight, kSlotsPerLane, is what the shapes made for large problems and the recording kernel take.
constexpr uint64_t kSlotsPerLane = 8;
__device__ __forceinline__ uint64_t active_blocks(uint64_t total, int block_threads, uint32_t spl) {
    const uint64_t per_block = (uint64_t)block_threads * (spl ? spl : 1u);
    const uint64_t want = (total + per_block - 1) / per_block;
    return want > (uint64_t)kXcds ? want : (uint64_t)kXcds;
}

// Partitions of the slot queues that have nothing left, as bits, from one look at all the counters (the wave's first
// kXcds lanes read one each, past the caches): one round trip to the memory side, where finding it out with an atomic on
// each counter in turn took eight (a wave or block that ran out of slots stalled 4 to 10 us for it). The counters only
// grow, so a partition seen empty stays empty; one seen with slots left may be empty by the time they are taken.
// Called by whole waves.
__device__ __forceinline__ uint32_t empty_partitions(const unsigned long long* queues, uint64_t total, int lane) {
    // the larger of the two sizes partitions have: one that is a chunk smaller and just ran out costs one failed take
    const uint64_t size = (total / kChunk + kXcds - 1) / kXcds * kChunk;
    uint32_t q = (uint32_t)lane * kQueueStride;
    asm volatile("" : "+v"(q));  // no register held for the address outside this rare path
    bool none = false;
    if (lane < kXcds) none = __hip_atomic_load(queues + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= size;
    return (uint32_t)__ballot(none) & ((1u << kXcds) - 1u);
}

// the first partition after `part`, cyclically, that `gone` does not mark (some partition is unmarked)
__device__ __forceinline__ uint32_t next_partition(uint32_t part, uint32_t gone) {
    const uint32_t left = ~gone & ((1u << kXcds) - 1u);
    const uint32_t turned = ((left << kXcds | left) >> (part + 1u)) & ((1u << kXcds) - 1u);  // bit i: part + 1 + i
    return (part + 1u + (uint32_t)__builtin_ctz(turned)) % (uint32_t)kXcds;
}
constexpr uint32_t kAllGone = (1u << kXcds) - 1u;

// Wave-uniform slot dispenser of the smooth kernels. The first chunks of 64 slots are dealt out without
// atomics, round-robin over the grid's waves (kStaticShare of the chunks, a whole number of rounds); the
// rest come from per-XCD queues, the wave starting on its own XCD's partition of the remainder and moving
// on when it is empty. Device-scope atomics on one counter are serialised at the memory side: taking
// every chunk from the queues cost each wave 4.5-10 us per take (up to ~150 waves per counter). The
// counters sit kQueueStride words apart, each in a memory line of its own.
// A problem of at most two chunks per wave is dealt out whole.
constexpr uint32_t kStaticShareNum = 3, kStaticShareDen = 4;
struct Dispenser {
    uint64_t total;      // padded slot count (a multiple of kChunk)
    uint64_t dyn_begin;  // slots below it are dealt out statically
    uint64_t st_next;    // the wave's next static chunk (>= dyn_begin: none left)
    uint64_t st_stride;  // kChunk x the grid's waves
    uint32_t part, gone;  // the partition taken from; those known to be empty
    bool queue_empty;
    uint64_t res_next, res_end;

    // `wave`: the wave's index among the `waves` waves of the grid that take part
    __device__ __forceinline__ void init(uint64_t total_slots, uint32_t xcd, uint64_t wave, uint64_t waves) {
        total = total_slots;
        const uint64_t chunks = total / kChunk;
        const uint64_t rounds = chunks <= 2 * waves ? 2 : chunks * kStaticShareNum / kStaticShareDen / waves;
        dyn_begin = min(rounds * waves * kChunk, total);
        st_stride = waves * kChunk;
        st_next = wave * kChunk;
        part = xcd;
        gone = 0;
        queue_empty = dyn_begin >= total;
        res_next = res_end = 0;
    }
    __device__ __forceinline__ bool drained() const {
        return queue_empty && st_next >= dyn_begin && res_next >= res_end;
    }

    // Hands slots to the idle lanes (ballot `idle`) in lane order; returns this lane's slot or ~0.
    __device__ __forceinline__ uint64_t take(unsigned long long* __restrict__ queues, uint64_t idle, int lane,
                                             uint64_t below) {
        const int nidle = __popcll(idle);
        const uint64_t avail = res_end - res_next;
        const int rank = __popcll(idle & below);
        uint64_t slot = ~0ull;
        if (avail >= (uint64_t)nidle) {
            slot = res_next + rank;
            res_next += nidle;
            return slot;
        }
        uint64_t base = 0, cend = 0;
        if (st_next < dyn_begin) {
            base = st_next;
            cend = base + kChunk;
            st_next += st_stride;
        } else {
            const int leader = __ffsll((long long)idle) - 1;
            const uint64_t rem = total - dyn_begin;
            while (!queue_empty) {
                const uint64_t pb = dyn_begin + part_begin(rem, part), pe = dyn_begin + part_begin(rem, part + 1);
                uint64_t got = 0;
                if (lane == leader) got = atomicAdd(queues + part * kQueueStride, (unsigned long long)kChunk);
                got = wave_bcast64(__shfl(got, leader, kWave));
                if (pb + got < pe) {
                    base = pb + got;
                    cend = (base + kChunk < pe) ? base + kChunk : pe;
                    break;
                }
                if (gone == 0u) gone = empty_partitions(queues, rem, lane);  // one look; later failures are races
                gone |= 1u << part;
                if (gone == kAllGone)
                    queue_empty = true;
                else
                    part = next_partition(part, gone);
            }
        }
        if ((uint64_t)rank < avail)
            slot = res_next + rank;
        else if (base + (rank - avail) < cend)
            slot = base + (rank - avail);
        const uint64_t next = base + ((uint64_t)nidle - avail);
        res_next = next < cend ? next : cend;
        res_end = cend;
        return slot;
    }
};

}  // namespace dev
}  // namespace avl

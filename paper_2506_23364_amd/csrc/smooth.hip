// Smooth variant of the trajectory pass and its adjoint (arXiv 2506.23364, section 5.2: the particles
// spread the released mass along the flow; here the mass each particle carries is deposited where it
// comes to rest, so the deposit raster is a differentiable function of the friction parameters).
//
// Forward: every particle of release cell c carries mp = mass[c] / P. An energy stop during a step puts
// it at the zero of the step's (linear) energy numerator, the fraction t* = v^2 / (v^2 - num) of the
// step; a runout-angle stop or the step limit leaves it where it is; leaving the grid loses the mass.
// The mass is splatted bilinearly (the height patch's corners and weights) into an int64 fixed-point
// raster (2^-24 units): order-independent, so reproducible bit for bit. Optionally every accepted step
// splats mp * v at the new position (velocity raster). Every kCkpt steps the particle's state
// (x, y, dx, dy, v^2) is checkpointed, and its end (steps done, reason) is recorded.
//
// Adjoint, per particle: the paths do not depend on (mu, xi, h, mass), so only v^2 along the path and
// the fractional last step do. Given gD = dL/dD, the kernel recomputes the last segment from its
// checkpoint, takes dL/dp* through the splat weights and dL/dt* = dL/dp* . (p1 - p), then runs the
// reverse sweep of the v^2 recursion segment by segment (each segment recomputed forward from its
// checkpoint into a per-lane scratch of (a_k, v^2_{k+1}), then swept backward). Per-particle
// results are reduced in a fixed order (deterministic).
#include <algorithm>

#include "particle.h"
#include "setup.h"
#include "tuning.h"

namespace avl {

using namespace dev;

namespace {

constexpr uint32_t kCkpt = 64;        // steps between checkpoints (even: segments start on even steps)
constexpr int kBackwardBlock = 256, kBackwardGrid = 1536;  // the adjoint kernel (its scratch is sized for this)
static_assert(kBackwardGrid % kXcds == 0, "each XCD has the same number of blocks");
constexpr int kReduceChunk = 4096;    // particles per block of the gradient reduction
static_assert(kCkpt % 2 == 0, "segments must start on even steps (one Philox block serves two steps)");

enum : uint32_t { kEndLimit = 0, kEndExit = 1, kEndStop = 2, kEndAngle = 3 };
enum : int { kAccept = 0, kExit = 1, kStop = 2, kAngle = 3 };

struct State {
    float x, y, z, gx, gy, dx, dy, v2, x0, y0, zr;
};

struct StepOut {
    int outcome;
    float x1, y1, num;  // target of the step and its energy numerator
    float a;            // drag term a = 2g ds / (xi h) of an accepted step
};

// The DEM with its replicated border, read through a buffer resource (no clamps, 32-bit offsets, both
// rows of the patch in flight), as in the plain pass; the same values as the clamped patch.
struct PadDem {
    __amdgpu_buffer_rsrc_t rs;
    uint32_t Wp, row_bytes;
};

__device__ __forceinline__ PadDem pad_dem(const SmoothArgs& a) {
    PadDem d;
    d.rs = buffer_rsrc(a.dem_pad, a.pad_bytes);
    d.Wp = (uint32_t)a.W + 2u;
    d.row_bytes = 4u * d.Wp;
    return d;
}

__device__ __forceinline__ Sample sample(const PadDem& d, float x, float y) {
    return bilinear_pad(d.rs, d.Wp, d.row_bytes, x, y);
}

// A step of the model (the same binary32 operations as the plain pass) in two parts, so that work that does not need the
// heights can run while they are on their way: the new direction, the target and the patch's loads; then the outcome,
// which updates s when the step is accepted. Every lane runs the whole step and the outcome selects what it keeps: a
// target off the grid is read through the buffer's bounds check, which cannot fault; its values are discarded.
struct Target {
    float x1, y1;
    PatchLoad pl;
};
__device__ __forceinline__ Target step_begin(State& s, uint32_t ux, uint32_t uy, const RunConst& rc, const PadDem& dem) {
    const float rx = signed_unit(ux), ry = signed_unit(uy);
    steer(s.dx, s.dy, s.gx, s.gy, rc.per, rc.Q, rc.rnd, rx, ry);
    Target t;
    t.x1 = s.x + rc.L * s.dx;
    t.y1 = s.y + rc.L * s.dy;
    t.pl = bilinear_pad_load(dem.rs, dem.Wp, dem.row_bytes, t.x1, t.y1);
    return t;
}

__device__ __forceinline__ StepOut step_end(State& s, const Target& t, const RunConst& rc, int H, int W, float g2) {
    StepOut o;
    o.x1 = t.x1;
    o.y1 = t.y1;
    const float fc1 = floorf(o.x1), fr1 = floorf(o.y1);
    const bool inb = fc1 >= 0.0f && fc1 < (float)W && fr1 >= 0.0f && fr1 < (float)H;
    const Sample s1 = bilinear_pad_value(t.pl);
    const float dz = s.z - s1.z;
    // dl2 + dz^2 >= dl2: with dl2 >= 2^-96 (a run constant) no lane is below the short form's range
    const float ds = sqrt_rn(rc.dl2 + dz * dz, rc.dl2 >= 0x1p-96f ? 0u : kRootLo);
    const float num = s.v2 + g2 * (dz - rc.mdl);
    const bool pos = num > 0.0f;
    const float aa = rc.cd * ds;
    const float v2n = num / (1.0f + aa);
    bool angle = false;
    if (rc.use_alpha) {
        const float hx = o.x1 - s.x0, hy = o.y1 - s.y0;
        angle = (s.zr - s1.z) < rc.tca * sqrtf(hx * hx + hy * hy);
    }
    o.num = inb ? num : 0.0f;
    o.a = (inb && pos) ? aa : 0.0f;
    o.outcome = !inb ? kExit : (!pos ? kStop : (angle ? kAngle : kAccept));
    const bool acc = inb && pos && !angle;
    s.x = acc ? o.x1 : s.x;
    s.y = acc ? o.y1 : s.y;
    s.z = acc ? s1.z : s.z;
    s.gx = acc ? s1.gx : s.gx;
    s.gy = acc ? s1.gy : s.gy;
    s.v2 = acc ? v2n : s.v2;
    return o;
}

__device__ __forceinline__ StepOut step(State& s, uint32_t ux, uint32_t uy, const RunConst& rc, const PadDem& dem, int H, int W,
                                        float g2) {
    const Target t = step_begin(s, ux, uy, rc, dem);
    return step_end(s, t, rc, H, W, g2);
}

// Philox words of steps n and n + 1 (n even)
__device__ __forceinline__ uint4 step_words(uint32_t n, uint32_t rep, uint32_t cell_id, const RunConst& rc) {
    // the key is wave-uniform: pinned to scalar registers, the round keys are scalar adds inside the block
    uint32_t k0 = __builtin_amdgcn_readfirstlane(rc.key0);
    uint32_t k1 = __builtin_amdgcn_readfirstlane(rc.key1);
    asm volatile("" : "+s"(k0), "+s"(k1));
    return philox4x32_10(n >> 1, rep, cell_id, rc.run, k0, k1);
}

// Workgroup table of splats: the particles of a block come from neighbouring release cells, so their paths and resting
// points share cells, and their splats are summed in LDS (int64, order-independent like the raster) before they reach
// the raster: the deposit once when the block ends, the velocity at each epoch boundary. Device-scope adds straight to
// the raster are performed at the memory side, at some 30e9 a second: the velocity raster of 9.3e6 steps (four 64-bit
// adds each) took 1.3 ms. A cell's candidates are the four slots of its bucket, seen in one 16-byte read; a cell that
// finds them taken goes to the raster directly.
constexpr uint32_t kDepEmpty = 0xFFFFFFFFu;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int kSlots>
struct SumTable {
    alignas(16) uint32_t tag[kSlots];
    unsigned long long val[kSlots];
};

// The tables' adds name the LDS address space: the compiler would otherwise merge them with the raster's
// fallback add into one generic (flat) atomic through a selected pointer, which every later LDS wait and
// every vector-memory wait then has to wait for.
typedef __attribute__((address_space(3))) unsigned long long lds_u64;
__device__ __forceinline__ void lds_add_u64(unsigned long long* p, unsigned long long v) {
    __hip_atomic_fetch_add((lds_u64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ u32x4 lds_ld4(const uint32_t* p) {
    return *(const volatile __attribute__((address_space(3))) u32x4*)(const __attribute__((address_space(3))) uint32_t*)p;
}

template <int kSlots>
__device__ __forceinline__ uint32_t sum_home(uint32_t cell) {
    return (__umul24((__umul24(cell, 0x9E3779u) >> 8) & 0xFFFFu, (uint32_t)kSlots / 4u) >> 16) * 4u;
}

// Adds v to the slot of `cell`, claimed if a candidate is empty, else to the raster; t: the tags at `at`, its bucket, read
// before (slots only go from empty to a tag between two flushes, so an old read is right or shows an empty slot, which
// the compare-and-swap settles).
template <int kSlots>
__device__ __forceinline__ void sum_add(SumTable<kSlots>& tb, unsigned long long* __restrict__ q, uint32_t cell, uint32_t at,
                                        const u32x4& t, unsigned long long v) {
    if (v == 0ull) return;
    int i = -1;
#pragma unroll
    for (int k = 3; k >= 0; --k) i = t[k] == cell ? k : i;
    if (i < 0) {
#pragma unroll 1
        for (int k = 0; k < 4 && i < 0; ++k) {
            if (tb.tag[at + k] == kDepEmpty || tb.tag[at + k] == cell) {
                const uint32_t old = atomicCAS(&tb.tag[at + k], kDepEmpty, cell);
                if (old == kDepEmpty || old == cell) i = k;
            }
        }
    }
    if (i >= 0)
        lds_add_u64(&tb.val[at + i], v);
    else
        atomicAdd(q + cell, v);
}

// fixed point of one splat weight: rint(w * 2^24); `small`: every lane's total is below 2^31, so that the rounded value
// converts through 32 bits (the 64-bit conversion is some ten instructions)
__device__ __forceinline__ unsigned long long splat_fixed(float w, bool small) {
    const float r = rintf(w * 16777216.0f);
    return small ? (unsigned long long)(long long)(int)r : (unsigned long long)(long long)r;
}

// bilinear splat of val at (x, y) through a table (the height patch's corners and weights, clamped corners merging)
template <int kSlots>
__device__ __forceinline__ void splat(SumTable<kSlots>& tb, unsigned long long* __restrict__ q, int H, int W, float x, float y,
                                      float val) {
    const Corners k = corners(H, W, x, y);
    const float w00 = (1.0f - k.fx) * (1.0f - k.fy), w01 = k.fx * (1.0f - k.fy);
    const float w10 = (1.0f - k.fx) * k.fy, w11 = k.fx * k.fy;
    const uint32_t c00 = (uint32_t)(k.ra * W + k.ca), c01 = (uint32_t)(k.ra * W + k.cb);
    const uint32_t c10 = (uint32_t)(k.rb * W + k.ca), c11 = (uint32_t)(k.rb * W + k.cb);
    const uint32_t a00 = sum_home<kSlots>(c00), a01 = sum_home<kSlots>(c01);
    const uint32_t a10 = sum_home<kSlots>(c10), a11 = sum_home<kSlots>(c11);
    const u32x4 t00 = lds_ld4(tb.tag + a00), t01 = lds_ld4(tb.tag + a01);
    const u32x4 t10 = lds_ld4(tb.tag + a10), t11 = lds_ld4(tb.tag + a11);
    const bool small = __ballot(!(fabsf(val) < 127.0f)) == 0ull;  // 127 x 2^24 < 2^31
    sum_add(tb, q, c00, a00, t00, splat_fixed(val * w00, small));
    sum_add(tb, q, c01, a01, t01, splat_fixed(val * w01, small));
    sum_add(tb, q, c10, a10, t10, splat_fixed(val * w10, small));
    sum_add(tb, q, c11, a11, t11, splat_fixed(val * w11, small));
}

// the same splat straight to the raster
__device__ __forceinline__ void splat_direct(unsigned long long* __restrict__ q, int H, int W, float x, float y, float val) {
    const Corners k = corners(H, W, x, y);
    const float w00 = (1.0f - k.fx) * (1.0f - k.fy), w01 = k.fx * (1.0f - k.fy);
    const float w10 = (1.0f - k.fx) * k.fy, w11 = k.fx * k.fy;
    const bool small = __ballot(!(fabsf(val) < 127.0f)) == 0ull;
    atomicAdd(q + (uint32_t)(k.ra * W + k.ca), splat_fixed(val * w00, small));
    atomicAdd(q + (uint32_t)(k.ra * W + k.cb), splat_fixed(val * w01, small));
    atomicAdd(q + (uint32_t)(k.rb * W + k.ca), splat_fixed(val * w10, small));
    atomicAdd(q + (uint32_t)(k.rb * W + k.cb), splat_fixed(val * w11, small));
}

// release cell of particle slot `slot`, and the particle's replica index within it
__device__ __forceinline__ uint64_t cell_of_slot(uint64_t slot, const SmoothArgs& a, uint32_t P, uint32_t* rep) {
    const uint64_t i = (slot >> 32) == 0 ? (uint64_t)udiv((uint32_t)slot, a.pdiv) : slot / P;
    *rep = (uint32_t)(slot - i * P);
    return i;
}

}  // namespace

// kBlk threads per block share the tables; a.spl particle slots per lane size the grid of a small problem. With kVel every
// accepted step also splats the velocity raster, through a table that the block flushes every kVelPairs pairs of steps, or
// straight, or straight for the first kStraightPairs pairs where the tuner chose that (tuning.h).
constexpr int kVelPairs = 16, kStraightPairs = 32, kAllPairs = 0x7FFFFFFF;
template <int kBlk, bool kVel>
__global__ __launch_bounds__(kBlk) void k_smooth_forward(SmoothArgs a) {
    if ((uint64_t)blockIdx.x >= active_blocks(a.run_off[1], kBlk, a.spl)) return;  // small problems: fewer blocks
    constexpr int kDepSlots = kVel ? 1024 : 4096;  // 12 or 48 KB
    constexpr int kVelSlots = kVel ? 3072 : 4;     // 36 KB
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    const RunConst rc = uniform_run(a.runs[0]);
    const int H = a.H, W = a.W;
    const PadDem dd = pad_dem(a);
    Dispenser disp;
    {
        const uint64_t total = wave_bcast64(a.run_off[1]);
        const uint64_t nb = min((uint64_t)gridDim.x, active_blocks(total, blockDim.x, a.spl));
        const uint32_t wpb = blockDim.x / kWave;
        disp.init(total, xcd_id(), (uint64_t)blockIdx.x * wpb + threadIdx.x / kWave, nb * wpb);
    }
    const size_t cplane = (size_t)a.C * a.cap;
    __shared__ SumTable<kDepSlots> dep;
    __shared__ SumTable<kVelSlots> vel;
    for (int k = threadIdx.x; k < kDepSlots; k += kBlk) {
        dep.tag[k] = kDepEmpty;
        dep.val[k] = 0ull;
    }
    if constexpr (kVel) {
        for (int k = threadIdx.x; k < kVelSlots; k += kBlk) {
            vel.tag[k] = kDepEmpty;
            vel.val[k] = 0ull;
        }
    }
    __syncthreads();
    bool direct = false;
    int pairs = kAllPairs;  // until the table's next flush
    if constexpr (kVel) {
        const bool always = velocity_straight(rc.n_slots, rc.P);
        direct = always || (a.direct != 0u && velocity_straight_first(rc.n_slots, rc.P));
        if (!always) pairs = direct ? kStraightPairs : kVelPairs;
    }

    bool alive = false;
    State s{};
    s.gx = s.dx = 1.0f;  // a lane without a particle runs the steps too and discards them
    uint32_t n = 0, rep = 0, cell_id = 0;
    uint64_t slot_id = 0;
    float mp = 0.0f;
    uint64_t st_acc = 0;
    uint32_t st_exit = 0, st_stop = 0, st_limit = 0;
    // the particle that ended in the lane's previous step: its record and its deposit wait for the next step's gather
    bool ended = false, rests = false;
    uint64_t end_slot = 0;
    uint32_t end_val = 0;
    float end_x = 0, end_y = 0, end_mp = 0;
    auto finish_ends = [&]() {
        if (__ballot(ended) == 0ull) return;
        if (ended) {
            if (rests) splat(dep, a.dep_q, H, W, end_x, end_y, end_mp);
            a.end_rec[end_slot] = end_val;
            ended = false;
        }
    };

    // one step of every live particle; checkpoints only before even steps
    auto advance = [&](uint32_t ux, uint32_t uy, bool even) {
        const bool lim = n >= a.S;
        if (even) {
            const bool ck = alive && !lim && n != 0 && n % kCkpt == 0;  // checkpoint 0 is the release cell's start record
            if (__ballot(ck) != 0ull && ck) {
                const size_t at = (size_t)(n / kCkpt) * a.cap + slot_id;
                a.ck[at] = s.x;
                a.ck[cplane + at] = s.y;
                a.ck[2 * cplane + at] = s.dx;
                a.ck[3 * cplane + at] = s.dy;
                a.ck[4 * cplane + at] = s.v2;
            }
        }
        const float xp = s.x, yp = s.y, v2p = s.v2;
        const Target tg = step_begin(s, ux, uy, rc, dd);
        finish_ends();
        const StepOut o = step_end(s, tg, rc, H, W, a.g2);
        const bool acc = alive && !lim && o.outcome == kAccept;
        const bool over = alive && !acc;
        if (__ballot(over) != 0ull && over) {
            const bool stop = !lim && o.outcome == kStop;
            const float t = stop && v2p > 0.0f ? v2p / (v2p - o.num) : 0.0f;
            ended = true;
            rests = lim || o.outcome != kExit;
            end_x = stop ? xp + t * (o.x1 - xp) : xp;
            end_y = stop ? yp + t * (o.y1 - yp) : yp;
            end_mp = mp;
            end_slot = slot_id;
            end_val = (n << 2) | (lim ? kEndLimit : o.outcome == kExit ? kEndExit : stop ? kEndStop : kEndAngle);
            st_limit += lim ? 1u : 0u;
            st_exit += rests ? 0u : 1u;
            st_stop += rests && !lim ? 1u : 0u;
            s.gx = 1.0f;
            s.gy = 0.0f;
        }
        n += acc ? 1u : 0u;
        if constexpr (kVel) {
            if (acc) {
                const float v = mp * sqrtf(s.v2);
                if (direct)
                    splat_direct(a.vel_q, H, W, s.x, s.y, v);
                else
                    splat(vel, a.vel_q, H, W, s.x, s.y, v);
            }
        }
        alive = acc;
    };

    // Particles start between pairs of steps only, so that one Philox block (two steps) serves every lane of a pair. A
    // particle starts from its release cell's start record (one load, the mass per particle beside it).
    for (;;) {
        bool finished = false;
        for (int pair = 0; !kVel || pair < pairs; ++pair) {
            const uint64_t idle = __ballot(!alive);
            const bool drained = disp.drained();
            if (__popcll(idle) == kWave && drained) {
                finished = true;
                break;
            }
            if (idle && !drained) {
                const uint64_t slot = disp.take(a.queues, idle, lane, below);
                if (!alive && slot < rc.n_slots) {
                    const uint64_t i = cell_of_slot(slot, a, rc.P, &rep);
                    const StartRec st = a.starts[i];
                    mp = a.mpc[i];
                    s.x = st.x;
                    s.y = st.y;
                    s.z = st.z;
                    s.gx = st.gx;
                    s.gy = st.gy;
                    s.dx = st.dx;
                    s.dy = st.dy;
                    s.x0 = st.x;
                    s.y0 = st.y;
                    s.zr = st.z;
                    s.v2 = 0.0f;
                    cell_id = st.cell;
                    slot_id = slot;
                    st_acc += n;  // the lane's previous particle
                    n = 0;
                    alive = true;
                }
            }
            const uint4 o = step_words(n, rep, cell_id, rc);
            advance(o.x, o.y, true);
            advance(o.z, o.w, false);
        }
        if (!kVel || pairs == kAllPairs) break;
        direct = false;
        pairs = kVelPairs;
        __syncthreads();
        for (int k = threadIdx.x; k < kVelSlots; k += kBlk) {
            if (vel.tag[k] != kDepEmpty) {
                if (vel.val[k] != 0ull) atomicAdd(a.vel_q + vel.tag[k], vel.val[k]);
                vel.tag[k] = kDepEmpty;
                vel.val[k] = 0ull;
            }
        }
        if (!__syncthreads_or(finished ? 0 : 1)) break;
    }
    finish_ends();
    // every wave of the block is done: the table's sums go to the raster, and the statistics, summed over
    // the block in LDS, go to the four counters with one atomic each per block (the counters share a
    // memory line, where device-scope atomics serialise). Steps: the accepted ones, the exits and the stops.
    __shared__ unsigned long long bst[4];
    if (threadIdx.x < 4) bst[threadIdx.x] = 0ull;
    __syncthreads();
    const uint64_t s1 = wave_sum64(st_exit), s2 = wave_sum64(st_stop);
    const uint64_t s0 = wave_sum64(st_acc + n) + s1 + s2, s3 = wave_sum64(st_limit);
    if (lane == 0) {
        lds_add_u64(&bst[0], s0);
        lds_add_u64(&bst[1], s1);
        lds_add_u64(&bst[2], s2);
        lds_add_u64(&bst[3], s3);
    }
    for (int k = threadIdx.x; k < kDepSlots; k += kBlk)
        if (dep.tag[k] != kDepEmpty && dep.val[k] != 0ull) atomicAdd(a.dep_q + dep.tag[k], dep.val[k]);
    __syncthreads();
    if (threadIdx.x < 4 && bst[threadIdx.x]) atomicAdd(a.stats + threadIdx.x, bst[threadIdx.x]);
}

// The adjoint takes as many steps forward and back as the particle took, which the forward has recorded. Of 64 consecutive
// particles all lanes wait for the longest, 15 steps where the mean is 9 on a 1024^2 scene: so a block takes a window of
// consecutive particles, sorts them by length in LDS (a counting sort), and its waves take 64 at a time, the longest
// first. What is left is the chain of the longest paths, at some 0.8 us a step forward and back: the forward steps run in
// pairs with the next pair's random words computed behind a gather, and a segment's first steps are kept in LDS.
// Long paths lie together: where each block has one window, the windows are dealt out in scattered pieces of 64 particles,
// so that each has its share of them; where blocks take several in turn, a window is consecutive, each XCD's blocks have
// one stretch of the particles, for its L2, and blocks with long paths take fewer windows.
// 640,000 particles of up to 78 steps: adjoint and its sums 205 -> 160 us (191 with consecutive windows). Larger blocks, wave
// priorities for the long groups and more or fewer steps in LDS gave nothing or cost up to 15 %.
constexpr int kLenBins = 128;
constexpr uint32_t kMaxWindow = 2048;
constexpr uint32_t kLdsSteps = 8;  // a lane's first (a_k, v^2_{k+1}) of a segment are in LDS, the rest in a.scratch

__device__ __forceinline__ uint32_t length_bin(uint32_t rec) {
    const uint32_t n = (rec & 3u) == kEndExit ? 0u : rec >> 2;
    return n < 64u ? n : min(63u + n / 64u, (uint32_t)kLenBins - 1u);
}

__global__ __launch_bounds__(kBackwardBlock) void k_smooth_backward(SmoothArgs a) {
    __shared__ uint16_t order[kMaxWindow];
    __shared__ uint8_t len[kMaxWindow];
    __shared__ uint32_t bins[kLenBins];
    __shared__ uint32_t next_group, next_win, count;
    __shared__ float2 near[kLdsSteps * kBackwardBlock];
    const int lane = threadIdx.x & (kWave - 1);
    const RunConst rc = uniform_run(a.runs[0]);
    const uint32_t windows = (uint32_t)((rc.n_slots + a.window - 1) / a.window);
    const uint32_t per = (windows + kXcds - 1) / kXcds;  // windows of an XCD's stretch
    const uint32_t each = gridDim.x / kXcds;             // blocks of an XCD, a window each to begin with
    uint32_t part = blockIdx.x % kXcds;
    uint32_t win = blockIdx.x / kXcds < per ? part * per + blockIdx.x / kXcds : windows;
    if (win >= windows && per <= each) return;
    const int H = a.H, W = a.W;
    const PadDem dd = pad_dem(a);
    const size_t T = (size_t)gridDim.x * blockDim.x;
    const size_t gtid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t cplane = (size_t)a.C * a.cap;
    const float g2dl = a.g2dl;
    const float xi = a.pdev ? a.pdev->xi : a.xi;  // a device-side loop keeps the parameters on the device

    auto particle = [&](uint64_t slot) {
        uint32_t rep = 0;
        const uint64_t i = cell_of_slot(slot, a, rc.P, &rep);
        const StartRec st = a.starts[i];  // the release state, as the forward started the particle
        const uint32_t cell_id = st.cell;
        const float mp = a.mpc[i];
        const uint32_t rec = a.end_rec[slot];
        const uint32_t n_end = rec >> 2, reason = rec & 3u;
        float dmu = 0.0f, dxi = 0.0f, dh = 0.0f, gw = 0.0f;
        if (reason != kEndExit) {
            // last segment: from its checkpoint (or the release) up to the end
            State s{};
            int32_t c_last = -1;
            if (a.C > 0) c_last = (int32_t)min(n_end / kCkpt, a.C - 1);
            auto load = [&](int32_t c) {
                s.x0 = st.x;
                s.y0 = st.y;
                s.zr = st.z;
                if (c <= 0) {  // the release (checkpoint 0 is the start record, v^2 = 0)
                    s.x = st.x;
                    s.y = st.y;
                    s.z = st.z;
                    s.gx = st.gx;
                    s.gy = st.gy;
                    s.dx = st.dx;
                    s.dy = st.dy;
                    s.v2 = 0.0f;
                    return;
                }
                const size_t at = (size_t)c * a.cap + slot;
                s.x = a.ck[at];
                s.y = a.ck[cplane + at];
                s.dx = a.ck[2 * cplane + at];
                s.dy = a.ck[3 * cplane + at];
                s.v2 = a.ck[4 * cplane + at];
                const Sample sm = sample(dd, s.x, s.y);
                s.z = sm.z;
                s.gx = sm.gx;
                s.gy = sm.gy;
            };
            load(c_last);
            const uint32_t n0 = c_last < 0 ? 0u : (uint32_t)c_last * kCkpt;
            // Steps c0 .. c0 + m - 1 from s, m <= kCkpt, in pairs, the next pair's words computed while the second
            // step's patch is on its way. c0 is a checkpoint and so even: afterwards `words` are those of the pair
            // that step c0 + m belongs to.
            uint4 words{};
            auto recompute = [&](uint32_t c0, uint32_t m) {
                auto keep = [&](uint32_t t, float aa) {
                    if (t < kLdsSteps)
                        near[t * kBackwardBlock + threadIdx.x] = make_float2(aa, s.v2);
                    else
                        a.scratch[(size_t)t * T + gtid] = make_float2(aa, s.v2);
                };
                words = step_words(c0, rep, cell_id, rc);
                for (uint32_t t = 0; t < m; t += 2) {
                    keep(t, step(s, words.x, words.y, rc, dd, H, W, a.g2).a);
                    if (t + 1 >= m) break;
                    const Target tg = step_begin(s, words.z, words.w, rc, dd);
                    words = step_words(c0 + t + 2, rep, cell_id, rc);
                    keep(t + 1, step_end(s, tg, rc, H, W, a.g2).a);
                }
            };
            recompute(n0, n_end > n0 ? n_end - n0 : 0u);
            float px = s.x, py = s.y;
            float lam = 0.0f;
            const bool stop = reason == kEndStop;
            float sx = 0.0f, sy = 0.0f, v2p = 0.0f, num = 0.0f;
            if (stop) {
                const float xp = s.x, yp = s.y;
                v2p = s.v2;
                const StepOut o = step(s, (n_end & 1u) ? words.z : words.x, (n_end & 1u) ? words.w : words.y, rc, dd, H, W, a.g2);
                num = o.num;
                const float t = v2p > 0.0f ? v2p / (v2p - num) : 0.0f;
                sx = o.x1 - xp;
                sy = o.y1 - yp;
                px = xp + t * sx;
                py = yp + t * sy;
            }
            // dL/dp* through the splat weights, dL/dt*
            const Corners k = corners(H, W, px, py);
            const float g00 = a.gD[(size_t)k.ra * W + k.ca], g01 = a.gD[(size_t)k.ra * W + k.cb];
            const float g10 = a.gD[(size_t)k.rb * W + k.ca], g11 = a.gD[(size_t)k.rb * W + k.cb];
            const float w00 = (1.0f - k.fx) * (1.0f - k.fy), w01 = k.fx * (1.0f - k.fy);
            const float w10 = (1.0f - k.fx) * k.fy, w11 = k.fx * k.fy;
            gw = ((g00 * w00) + (g01 * w01)) + ((g10 * w10) + (g11 * w11));
            if (stop) {
                const float gpx = ((g01 - g00) * (1.0f - k.fy)) + ((g11 - g10) * k.fy);
                const float gpy = ((g10 - g00) * (1.0f - k.fx)) + ((g11 - g01) * k.fx);
                const float gt = mp * ((gpx * sx) + (gpy * sy));
                const float Dn = v2p - num;
                if (Dn > 0.0f) {
                    lam = gt / Dn;
                    dmu = -((gt * (v2p / Dn)) * (g2dl / Dn));
                }
                // reverse sweep: the last segment from the scratch, then earlier segments recomputed
                // an energy stop needs a step, so step_limit >= 1 and checkpoint 0 exists: c_last >= 0
                for (int32_t c = c_last; c >= 0; --c) {
                    const uint32_t c0 = (uint32_t)c * kCkpt;
                    uint32_t m = n_end - c0;
                    if (c != c_last) {
                        load(c);
                        m = kCkpt;
                        recompute(c0, m);
                    }
                    auto back = [&](const float2 e) {
                        const float aa = e.x, v2n = e.y;
                        const float op = 1.0f + aa;
                        dmu = dmu - lam * (g2dl / op);
                        dxi = dxi + lam * ((v2n * aa) / (xi * op));
                        dh = dh + lam * ((v2n * aa) / (a.h * op));
                        lam = lam / op;
                    };
                    if (m > kLdsSteps) {
                        float2 e = a.scratch[(size_t)(m - 1u) * T + gtid];
                        for (uint32_t t = m - 1u; t > kLdsSteps; --t) {
                            const float2 f = a.scratch[(size_t)(t - 1u) * T + gtid];  // on its way during the divisions
                            back(e);
                            e = f;
                        }
                        back(e);
                    }
                    for (uint32_t t = min(m, kLdsSteps); t-- > 0;) back(near[t * kBackwardBlock + threadIdx.x]);
                }
            }
        }
        a.pp[slot] = dmu;
        a.pp[a.cap + slot] = dxi;
        a.pp[2 * a.cap + slot] = dh;
        a.pp[3 * a.cap + slot] = gw;
    };

    const bool spread = per <= each;  // a window a block
    for (;;) {
        if (win < windows) {
            auto slot_of = [&](uint32_t k) {
                return spread ? ((uint64_t)(k / kWave) * windows + win) * kWave + k % kWave : (uint64_t)win * a.window + k;
            };
            for (uint32_t k = threadIdx.x; k < kLenBins; k += kBackwardBlock) bins[k] = 0u;
            if (threadIdx.x == 0) next_group = 0u;
            __syncthreads();
            for (uint32_t k = threadIdx.x; k < a.window; k += kBackwardBlock) {
                const uint64_t slot = slot_of(k);
                if (slot < rc.n_slots) {
                    const uint32_t b = length_bin(a.end_rec[slot]);
                    len[k] = (uint8_t)b;
                    atomicAdd(&bins[b], 1u);
                }
            }
            __syncthreads();
            if (threadIdx.x < kWave) {  // where each length's particles begin, the longest first
                const int hi = kLenBins - 1 - 2 * lane;
                const uint32_t n0 = bins[hi], n1 = bins[hi - 1];
                const uint32_t upto = wave_incl_scan(n0 + n1);
                bins[hi] = upto - n0 - n1;
                bins[hi - 1] = upto - n1;
                if (lane == kWave - 1) count = upto;
            }
            __syncthreads();
            for (uint32_t k = threadIdx.x; k < a.window; k += kBackwardBlock)
                if (slot_of(k) < rc.n_slots) order[atomicAdd(&bins[len[k]], 1u)] = (uint16_t)k;
            __syncthreads();
            for (;;) {
                uint32_t g = 0;
                if (lane == 0) g = atomicAdd(&next_group, 1u);
                g = __builtin_amdgcn_readfirstlane(g) * kWave;
                if (g >= count) break;
                if (g + lane < count) particle(slot_of(order[g + lane]));
            }
        }
        if (per <= each) break;
        __syncthreads();
        if (threadIdx.x == 0) {
            next_win = windows;
            for (int k = 0; k < kXcds; ++k, part = (part + 1) % kXcds) {
                const uint32_t at = each + (uint32_t)atomicAdd(a.queues + part * kQueueStride, 1ull);
                if (at < per && part * per + at < windows) {
                    next_win = part * per + at;
                    break;
                }
            }
        }
        __syncthreads();
        win = next_win;
        if (win >= windows) break;
    }
}

// ------------------------------------------------------------------------------------------ reductions

// After the adjoint kernel, one launch: its first a.nb blocks sum the particles' (dmu, dxi, dh), the others the cells'
// dL/dmass. All sums are binary64 in a fixed order, so the results do not depend on timing. A pass is over in some
// 200 us, and these sums are bound by the latency of their loads and by their launches: three kernels with one 4-byte load
// in flight per thread took 33 us for 640,000 particles of 5000 cells, this one takes 10.
//
// dL/dparams: a block sums kReduceChunk particles (16 per thread in order, then a fixed tree) into part[block]; the last
// block to finish sums the blocks that held particles, each thread every 256th in order, then the same tree.
// dL/dmass of release cell i: (sum over its P particles of sum gD w, in order) / P. A wave takes kMassRows cells and reads
// them kWave particles at a time, each cell one contiguous stretch, and turns them through LDS so that a lane sums a
// cell's particles in order; below kMassCols particles a cell, where most lanes of such a load would have no particle, a
// thread reads its own cell's particles.
constexpr int kReduceThreads = 256;
constexpr int kMassRows = 16;
constexpr uint32_t kMassCols = 16;
constexpr uint32_t kTicket = 16;  // the word of the queue counters' memory that counts finished blocks; zero at launch
static_assert(kReduceChunk == 16 * kReduceThreads && kTicket < kQueueStride, "");
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

struct ReduceArgs {
    const float* pp;
    unsigned long long cap;
    const RunConst* runs;
    const unsigned long long* n_slots;  // particles; nothing writes it while the sums run
    double* part;  // 3 a.nb
    double* out;   // 3, nullable
    unsigned long long* queues;
    uint32_t nb;
    const int32_t* cells;  // dmass: cells, their number, the raster
    const int32_t* n_cells;
    float* dmass;
};

__device__ __forceinline__ void tree_sum3(double (&sh)[3][kReduceThreads], const double (&acc)[3]) {
    for (int q = 0; q < 3; ++q) sh[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int d = kReduceThreads / 2; d >= 1; d >>= 1) {
        if ((int)threadIdx.x < d)
            for (int q = 0; q < 3; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + d];
        __syncthreads();
    }
}

// The block's part of dL/dparams; true in the block that finished last, which has the sums in sh[q][0] and has written
// them to a.out (unless null).
__device__ __forceinline__ bool reduce_params(const ReduceArgs& a, double (&sh)[3][kReduceThreads]) {
    __shared__ uint32_t rank;
    const unsigned long long n = *a.n_slots;
    const uint32_t used = max(1u, (uint32_t)((n + kReduceChunk - 1) / kReduceChunk));  // blocks that hold particles
    if (blockIdx.x >= used) return false;
    const unsigned long long base = (unsigned long long)blockIdx.x * kReduceChunk + threadIdx.x * 16ull;
    double acc[3] = {0.0, 0.0, 0.0};
    if (base + 16 <= n) {
        f32x4_any v[3][4];
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int k = 0; k < 4; ++k) v[q][k] = *reinterpret_cast<const f32x4_any*>(a.pp + q * a.cap + base + 4 * k);
#pragma unroll
        for (int k = 0; k < 16; ++k)
#pragma unroll
            for (int q = 0; q < 3; ++q) acc[q] += (double)v[q][k / 4][k % 4];
    } else {
        for (unsigned long long i = base; i < n; ++i)
            for (int q = 0; q < 3; ++q) acc[q] += (double)a.pp[q * a.cap + i];
    }
    tree_sum3(sh, acc);
    if (threadIdx.x == 0) {
        for (int q = 0; q < 3; ++q) a.part[3 * (size_t)blockIdx.x + q] = sh[q][0];
        __threadfence();
        rank = (uint32_t)atomicAdd(a.queues + kTicket, 1ull);
    }
    __syncthreads();
    if (rank != used - 1u) return false;
    __threadfence();
    for (int q = 0; q < 3; ++q) acc[q] = 0.0;
    for (uint32_t b = threadIdx.x; b < used; b += kReduceThreads)
        for (int q = 0; q < 3; ++q) acc[q] += a.part[3 * (size_t)b + q];
    tree_sum3(sh, acc);
    if (threadIdx.x == 0 && a.out)
        for (int q = 0; q < 3; ++q) a.out[q] = sh[q][0];
    return true;
}

__device__ __forceinline__ void reduce_mass(const ReduceArgs& a, float* lds) {
    const uint32_t P = a.runs[0].P;
    const int64_t n = *a.n_cells;
    if (a.runs[0].n_slots == 0) return;
    const float* const gw = a.pp + 3 * a.cap;
    const int64_t block = blockIdx.x - a.nb, blocks = gridDim.x - a.nb;
    if (P < kMassCols) {
        for (int64_t i = block * kReduceThreads + threadIdx.x; i < n; i += blocks * kReduceThreads) {
            double s = 0.0;
            for (uint32_t j = 0; j < P; ++j) s += (double)gw[(size_t)i * P + j];
            a.dmass[a.cells[i]] = (float)(s / (double)P);
        }
        return;
    }
    constexpr int kWaves = kReduceThreads / kWave, kPitch = kWave + 1;
    const int lane = threadIdx.x & (kWave - 1);
    float* const tile = lds + (threadIdx.x / kWave) * kMassRows * kPitch;
    for (int64_t i0 = (block * kWaves + threadIdx.x / kWave) * kMassRows; i0 < n; i0 += blocks * kWaves * kMassRows) {
        double s = 0.0;
        for (uint32_t j0 = 0; j0 < P; j0 += kWave) {
            const uint32_t cols = min(P - j0, (uint32_t)kWave);
            float v[kMassRows];
#pragma unroll
            for (int r = 0; r < kMassRows; ++r)
                v[r] = i0 + r < n && (uint32_t)lane < cols ? gw[(size_t)(i0 + r) * P + j0 + lane] : 0.0f;
#pragma unroll
            for (int r = 0; r < kMassRows; ++r) tile[r * kPitch + lane] = v[r];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the tile is the wave's own
            if (lane < kMassRows)
                for (uint32_t j = 0; j < cols; ++j) s += (double)tile[lane * kPitch + j];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        if (lane < kMassRows && i0 + lane < n) a.dmass[a.cells[i0 + lane]] = (float)(s / (double)P);
    }
}

__global__ __launch_bounds__(kReduceThreads) void k_smooth_reduce(ReduceArgs a) {
    __shared__ union {
        double sum[3][kReduceThreads];
        float tile[kReduceThreads / kWave * kMassRows * (kWave + 1)];
    } sh;
    if (blockIdx.x < a.nb)
        reduce_params(a, sh.sum);
    else
        reduce_mass(a, sh.tile);
}

// fixed point (2^-24) -> float, the deposit and (grid y = 1) the velocity raster; four values a thread, by 16-byte
// accesses where both arrays are aligned for them
__device__ __forceinline__ float q_value(unsigned long long q) { return (float)((double)(long long)q * 0x1p-24); }

__global__ __launch_bounds__(256) void k_q_to_float(const unsigned long long* __restrict__ q0, float* __restrict__ out0,
                                                    const unsigned long long* __restrict__ q1, float* __restrict__ out1,
                                                    int64_t n) {
    const unsigned long long* const q = blockIdx.y ? q1 : q0;
    float* const out = blockIdx.y ? out1 : out0;
    if (!q || !out) return;
    const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i0 + 4 <= n && ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(out)) & 15) == 0) {
        const ulonglong2 a = *reinterpret_cast<const ulonglong2*>(q + i0), b = *reinterpret_cast<const ulonglong2*>(q + i0 + 2);
        *reinterpret_cast<float4*>(out + i0) = make_float4(q_value(a.x), q_value(a.y), q_value(b.x), q_value(b.y));
    } else {
        for (int64_t i = i0; i < n && i < i0 + 4; ++i) out[i] = q_value(q[i]);
    }
}

// ------------------------------------------------------------------------------------------ calibration loop
// An iteration of the loop is four launches: forward, loss, adjoint, and the adjoint's sums with the step. On a tile of
// 501 x 640 the passes take 85 us and the gap behind each launch some 5, so what the parts between the passes need
// cleared, converted or set up is done by the kernel before (ten launches, the deposit written as floats and read back,
// dL/dmass that no one asks for: 20 iterations of a 1,500-cell, 96,000-particle release 3.09 -> 2.30 ms).

// L = sum (D - T)^2 / N and dL/dD = c (D - T), c = 2/N rounded to binary32. The differences are binary32;
// their squares are exact in binary64 and summed in a fixed order (per thread over a fixed grid stride,
// then over the wave, the block, and the kMseBlocks block sums), so L does not depend on timing.
constexpr int kMseBlocks = 1024;
constexpr int kMseThreads = 256;

__device__ __forceinline__ double block_sum_f64(double v, double* lds) {
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    if (lane == 0) lds[wid] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < (int)(blockDim.x / kWave); ++k) t += lds[k];
    return t;  // valid in thread 0
}

constexpr int kQueueWords = kXcds * (int)kQueueStride;
__device__ __forceinline__ void clear_queues(unsigned long long* queues) {
    for (int i = threadIdx.x; i < kQueueWords; i += blockDim.x) queues[i] = 0ull;
}

__global__ __launch_bounds__(kMseThreads) void k_calib_loss(unsigned long long* __restrict__ dep_q,
                                                            const float* __restrict__ tgt, int64_t n, float c,
                                                            float* __restrict__ gD, double* __restrict__ part,
                                                            unsigned long long* __restrict__ queues,
                                                            const RunConst* __restrict__ runs,
                                                            unsigned long long* __restrict__ slots) {
    __shared__ double lds[kMseThreads / kWave];
    if (blockIdx.x == 0) {
        clear_queues(queues);
        if (threadIdx.x == 0) *slots = runs[0].n_slots;
    }
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kMseThreads + threadIdx.x; i < n; i += (int64_t)kMseBlocks * kMseThreads) {
        const float d = q_value(dep_q[i]) - tgt[i];
        dep_q[i] = 0ull;
        gD[i] = c * d;
        acc += (double)d * (double)d;
    }
    const double t = block_sum_f64(acc, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
}

hipError_t launch_calib_loss(unsigned long long* dep_q, const float* target, int64_t n, float c, float* gD, double* part,
                             unsigned long long* queues, const RunConst* runs, unsigned long long* slots, hipStream_t s) {
    hipLaunchKernelGGL(k_calib_loss, dim3(kMseBlocks), dim3(kMseThreads), 0, s, dep_q, target, n, c, gD, part, queues, runs,
                       slots);
    return hipGetLastError();
}

size_t mse_partials() { return kMseBlocks; }

// Adam (Kingma and Ba 2015, algorithm 1) on (mu, xi) in binary64, one thread: the host loop's arithmetic in
// its order (bias corrections from running products of the rates, the step clamped at the lower bounds), so
// a loop that stays on the device takes the same steps.
__global__ void k_calib_init(RunSpec spec, ::avl_params start, RunSpec* __restrict__ spec_dev,
                             ::avl_params* __restrict__ p_dev, double* __restrict__ st, int32_t* __restrict__ err) {
    *spec_dev = spec;
    *p_dev = start;
    st[0] = (double)start.mu;
    st[1] = (double)start.xi;
    st[2] = st[3] = st[4] = st[5] = 0.0;
    st[6] = st[7] = 1.0;
    err[0] = err[1] = 0;
}

__device__ void adam_step(const CalibStep& a, double loss, const double* g3) {
    double* const st = a.state;
    const int32_t status = *a.next.status;
    if (status != 0 && a.err[0] == 0) {
        a.err[0] = status;
        a.err[1] = a.t;
    }
    a.row[0] = loss;
    a.row[1] = st[0];
    a.row[2] = st[1];
    a.row[3] = g3[0];
    a.row[4] = g3[1];
    st[6] *= a.c.b1;
    st[7] *= a.c.b2;
    for (int k = 0; k < 2; ++k) {
        const double g = g3[k];
        st[2 + k] = a.c.b1 * st[2 + k] + (1.0 - a.c.b1) * g;
        st[4 + k] = a.c.b2 * st[4 + k] + (1.0 - a.c.b2) * (g * g);
        const double mh = st[2 + k] / (1.0 - st[6]);
        const double vh = st[4 + k] / (1.0 - st[7]);
        double th = st[k] - a.c.lr[k] * mh / (sqrt(vh) + a.c.eps);
        if (th < a.c.lo[k]) th = a.c.lo[k];
        st[k] = th;
    }
    a.p->mu = (float)st[0];
    a.p->xi = (float)st[1];
}

// The block that finishes last writes the next iteration's run table and clears the ticket, while blocks that hold no
// particles may not have started yet: they read the number of particles from c.slots, which the loss kernel wrote, and leave.
__global__ __launch_bounds__(kReduceThreads) void k_calib_step(ReduceArgs a, CalibStep c, int32_t H, int32_t W) {
    static_assert(kReduceThreads == kMseThreads, "the loss sums in this order");
    __shared__ double sum[3][kReduceThreads];
    __shared__ double lds[kMseThreads / kWave];
    if (!reduce_params(a, sum)) return;
    double acc = 0.0;
    for (int k = threadIdx.x; k < kMseBlocks; k += kMseThreads) acc += c.loss_part[k];
    const double t = block_sum_f64(acc, lds);
    clear_queues(a.queues);
    if (threadIdx.x < 4) c.stats[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) {
        const double g3[3] = {sum[0][0], sum[1][0], sum[2][0]};
        adam_step(c, t / c.n, g3);
        setup_one(c.next, H, W, (int64_t)*c.n_cells);
    }
}

hipError_t launch_calib_init(RunSpec spec, ::avl_params start, RunSpec* spec_dev, ::avl_params* p_dev, double* state,
                             int32_t* err, hipStream_t s) {
    hipLaunchKernelGGL(k_calib_init, dim3(1), dim3(1), 0, s, spec, start, spec_dev, p_dev, state, err);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ launchers

size_t smooth_checkpoints(uint32_t S) { return S == 0 ? 0 : (S + kCkpt - 1) / kCkpt; }
size_t smooth_scratch_bytes() { return (size_t)kCkpt * kBackwardGrid * kBackwardBlock * sizeof(float2); }
size_t smooth_reduce_blocks(unsigned long long cap) { return (size_t)((cap + kReduceChunk - 1) / kReduceChunk) + 1; }

namespace {

struct SmoothVariant {
    int block;
    uint32_t spl;
};
// Forward candidates: (threads per block, slots per lane). Small blocks with a slot per lane serve problems that leave SIMDs
// idle otherwise (96,000 particles: 52 us with 1024 threads or two slots, 47 so). The first is kept unless another is
// faster, and holds for the larger problems of its size class too, since it leaves no lane a second round. With the velocity
// raster and few particles a cell each shape is a candidate twice, the second time starting straight where it may.
constexpr SmoothVariant kFwdVariants[] = {{256, 1}, {1024, 2}, {512, 2}, {1024, 1}, {256, 8}, {512, 1}};
// adjoint candidates: particles of a window
constexpr uint32_t kBwdWindows[] = {1024, 512, 256, 2048};

template <int kBlk, bool kVel>
void launch_fwd(const SmoothArgs& a, hipStream_t s) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(&k_smooth_forward<kBlk, kVel>),
                                                     kBlk, 0) != hipSuccess ||
        per_cu <= 0)
        per_cu = 1;
    hipLaunchKernelGGL((k_smooth_forward<kBlk, kVel>), dim3(cus * per_cu), dim3(kBlk), 0, s, a);
}

}  // namespace

constexpr int kFwdShapes = (int)(sizeof(kFwdVariants) / sizeof(kFwdVariants[0]));
int smooth_forward_variants(bool velocity, uint32_t P) {
    return velocity && P <= kStraightReplicas ? 2 * kFwdShapes : kFwdShapes;
}
int smooth_backward_variants() { return (int)(sizeof(kBwdWindows) / sizeof(kBwdWindows[0])); }

hipError_t launch_smooth_forward(const SmoothArgs& a, int variant, hipStream_t s) {
    if (variant < 0 || variant >= 2 * kFwdShapes) variant = 0;
    SmoothArgs b = a;
    b.direct = variant >= kFwdShapes ? 1u : 0u;
    variant %= kFwdShapes;
    b.spl = kFwdVariants[variant].spl;
    switch (kFwdVariants[variant].block) {
        case 1024: b.vel_q ? launch_fwd<1024, true>(b, s) : launch_fwd<1024, false>(b, s); break;
        case 512: b.vel_q ? launch_fwd<512, true>(b, s) : launch_fwd<512, false>(b, s); break;
        default: b.vel_q ? launch_fwd<256, true>(b, s) : launch_fwd<256, false>(b, s); break;
    }
    return hipGetLastError();
}

hipError_t launch_smooth_backward_kernel(const SmoothArgs& a, int variant, hipStream_t s) {
    if (variant < 0 || variant >= smooth_backward_variants()) variant = 0;
    SmoothArgs b = a;
    b.window = kBwdWindows[variant];
    hipLaunchKernelGGL(k_smooth_backward, dim3(kBackwardGrid), dim3(kBackwardBlock), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_smooth_reductions(const SmoothArgs& a, const int32_t* n_cells, float* dmass, int64_t max_cells,
                                    double* part, double* dparams, hipStream_t s) {
    ReduceArgs r{a.pp, a.cap, a.runs, &a.runs->n_slots, part, dparams, a.queues, (uint32_t)smooth_reduce_blocks(a.cap), a.cells, n_cells, dmass};
    const int64_t mass = std::min<int64_t>((max_cells + 63) / 64, 4096);  // 16 cells a wave, then the next ones
    hipLaunchKernelGGL(k_smooth_reduce, dim3(r.nb + (uint32_t)mass), dim3(kReduceThreads), 0, s, r);
    return hipGetLastError();
}

hipError_t launch_calib_step(const SmoothArgs& a, double* part, const CalibStep& c, hipStream_t s) {
    ReduceArgs r{a.pp, a.cap, a.runs, c.slots, part, nullptr, a.queues, (uint32_t)smooth_reduce_blocks(a.cap), a.cells, nullptr, nullptr};
    hipLaunchKernelGGL(k_calib_step, dim3(r.nb), dim3(kReduceThreads), 0, s, r, c, a.H, a.W);
    return hipGetLastError();
}

hipError_t launch_q_to_float(const unsigned long long* q0, float* out0, const unsigned long long* q1, float* out1, int64_t n,
                             hipStream_t s) {
    const bool one = q0 && out0, two = q1 && out1;
    if (n <= 0 || (!one && !two)) return hipSuccess;
    hipLaunchKernelGGL(k_q_to_float, dim3((unsigned)((n + 1023) / 1024), two ? 2 : 1), dim3(256), 0, s, q0, out0, q1, out1, n);
    return hipGetLastError();
}

}  // namespace avl

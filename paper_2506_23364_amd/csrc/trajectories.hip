// Particle trajectories of the avalanche overlay (section 5.2 of arXiv 2506.23364, the trajectory node):
// particles released per coded texel, steered by persistence and a random deviation from the optimal
// (downslope) path, slowed by Coulomb/Voellmy friction, stopped by the energy line or a runout angle;
// accumulated into a hit-count raster and a max-velocity raster. One kernel serves a single run and a
// batch of runs (parameter sets x DEM tiles x release scenarios) in one persistent launch.
//
// Design for gfx950 (measured choices; the alternatives are recorded in the design notes):
//  - One persistent grid sized to the chip's occupancy; one lane carries one particle at a time and its
//    whole state stays in VGPRs. A lane whose particle ended takes the next particle slot before the next
//    pair of steps: a single run's waves take exactly what their idle lanes need from the block's window, a
//    batch's from a per-wave reservoir refilled 64 slots at a time (a chunk belongs to one run).
//  - Slots are ordered replica-major within a release cell and run-major across runs; every run starts
//    at a multiple of 64, so a 64-slot chunk belongs to one run. Release cells are in row-major order,
//    so consecutive slots start at the same or neighbouring cells and their paths share most cells.
//  - Device-scope atomics on the rasters are performed beyond L2 (at the memory side), so they are the
//    cost to cut. Entry counts and per-cell max v^2 go first into a table in LDS shared by the whole
//    workgroup (tag, count, max; two buckets of four slots per cell), flushed to the rasters at epoch boundaries
//    (a pair of barriers every kFlush iterations per wave on average). A cell whose candidate slots are all
//    held by other cells goes straight to the raster. A visit that ended is accumulated in the next iteration,
//    while that iteration's heights are on their way, so the table's LDS round trips are hidden behind the
//    gather (3 % of the large passes).
//  - An epoch is a budget of kFlush x (waves per block) wave-iterations that the block's waves claim two
//    at a time from an LDS counter, so a wave that runs faster than its neighbours does more of them and
//    every wave reaches the boundary within about one iteration of the others (a fixed count per wave
//    left the fast waves waiting at the first barrier for 15-25 % of their time).
//  - The waves of a workgroup share a window of consecutive slots (two ranges, topped up at epoch
//    boundaries), so the table sees the paths of neighbouring release cells together. Top-ups are guided:
//    up to kWindow x kBlock slots, but at most half the partition's remainder over the blocks of an XCD,
//    so windows shrink as the queues drain and the blocks finish together. A wave that runs the window
//    dry mid-epoch takes slots from the queues directly.
//  - The slot range is split into one partition per XCD; windows and chunks come from the XCD's own
//    partition first and from the others only when it is empty. Each XCD's L2 then holds its own band
//    of the DEM (or its own runs).
//  - Every run writes the caller's rasters directly (a single run v^2 bits, turned into speeds by a finalize
//    pass, a batch's runs the speeds). Per-XCD private copies bought nothing once the table had cut the
//    atomics: the atomics are performed at the memory side either way, and zeroing and merging the copies
//    cost 9 % at 8192^2.
//  - Accumulation is integer only (u32 add; u32 max on the bits of v^2 >= 0, whose order is the value
//    order), so every raster is independent of scheduling and of the kernel variant: bit-reproducible.
//  - Philox4x32-10 gives four words per block; one block serves two consecutive steps.
#include "particle.h"

namespace avl {

namespace {

constexpr uint32_t kEmpty = 0xFFFFFFFFu;
using dev::kChunk;

// Bits of sqrt(v^2), for the flush of a batch: the correctly rounded root is monotone, so the largest root is the root of
// the largest v^2. A pass over the rasters that takes the root at the end reads and writes 8 bytes a texel for every run
// (256 runs of 1024^2: 222 of 2560 us); a single run has few texels for its steps, and there the pass is the cheaper one
// (8192^2 and 1.2e9 steps: 62 us of 8 ms, against 2 % of the kernel).
__device__ __forceinline__ uint32_t root_bits(uint32_t v2) {
    const bool odd = v2 != 0u && v2 - dev::kRootLo > 0x7F7FFFFFu - dev::kRootLo;
    if (__builtin_expect(__ballot(odd) != 0ull, 0)) return __float_as_uint(sqrtf(__uint_as_float(v2)));
    return v2 ? __float_as_uint(dev::sqrt_est(__uint_as_float(v2)).s) : 0u;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// four consecutive words of a table in LDS, 16-byte aligned, in one read
__device__ __forceinline__ u32x4 lds_ld4(const uint32_t* p) {
    return *(const volatile __attribute__((address_space(3))) u32x4*)(const __attribute__((address_space(3))) uint32_t*)p;
}

// A raster cell's v^2 bits as this CU's caches hold them: a workgroup-scope read, served by L1 or the XCD's
// L2 when they hold the line. The raster's maxima are performed at the memory side, so the cached value can
// be older than the memory's, but every value the cell takes during the pass is at least the one before
// it (it is zeroed before the launch, and the kernel's start discards lines cached before that), so a
// read that is already >= v proves a max with v unnecessary. A read from the memory side (nontemporal)
// took 1.27x as long over the 8192^2 pass: each epoch boundary waits for these reads.
__device__ __forceinline__ uint32_t cached_bits(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Max into a global raster cell, skipped when a cached read already shows a value >= bits.
__device__ __forceinline__ void global_max(uint32_t* __restrict__ p, uint32_t bits) {
    if (cached_bits(p) < bits) atomicMax(p, bits);
}

}  // namespace

using namespace dev;

// Workgroup-shared accumulation table: kTbl slots of (cell key, entry count, max v^2 bits) in LDS,
// eight candidate slots per cell. A particle's visit to a cell (from its entry, or its release,
// to the step that leaves the cell or ends the path) goes into the table once, when it ends: one entry
// and the visit's largest v^2 (the counts are the same as counting each entry when it happens, and one
// table operation per visit replaces a claim at the entry plus a max at the exit). Slots are emptied only
// at epoch boundaries: each boundary flushes a slot to the rasters and empties it, except (with retention
// on) a slot whose cell saw enough visits end in the epoch that ended, which keeps its key, count and
// maximum into the next epoch. With retention the count word holds two 16-bit halves: the entries so far
// (low) and their number at the last boundary (high).
template <int kTbl>
struct Table {
    // a bucket is four consecutive slots: one 16-byte read shows a key's four candidates
    alignas(16) uint32_t tag[kTbl];
    uint32_t cnt[kTbl], vmx[kTbl];
};

// Workgroup control block in LDS. The window is a range of consecutive slots that the workgroup's waves
// share; it changes only between the barriers of an epoch boundary.
struct Control {
    unsigned long long base[2];   // the window: two ranges of consecutive slots, taken in order
    uint32_t len[2];              // their lengths (multiples of 64 in a batch)
    uint32_t take;                // window slots handed out this epoch
    uint32_t busy[2];             // waves with work left, per epoch parity
    uint32_t part, gone, empty;   // the window's own walk over the XCD partitions, those known to be empty
    uint32_t dry;                 // the tail probe has seen the block run out of slots
    uint32_t iters;               // pairs of wave-iterations of the epoch's budget claimed so far
    unsigned long long left;      // slots left in the partition after the window's last top-up
    unsigned long long st[4];     // single run: the block's statistics, summed when its waves are done
};

// kAlpha: the runout-angle stop is compiled in; a single run without it takes the instantiation without.
// A single run with it keeps the release point and height in registers; a batch re-derives them from the
// release cell when a run uses the stop, so its kernel carries no registers for them.
// kKeep: table retention, 0 off; else a slot whose cell saw at least kKeep visits end in the epoch that
// ended stays in the table (its count and maximum reach the rasters at a later boundary).
// kWpe: waves per SIMD the register budget is sized for (8: 64 VGPRs; 6: 80).
// kRec: the recording instantiation (single run): the particles of the recorded range also write their
// points and end records (a diagnostic; the other instantiations compile none of it).
template <bool kBatch, bool kAlpha, int kBlock, int kFlush, int kTbl, int kWindow, int kKeep, int kWpe = 8,
          bool kRec = false>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kWpe)))
void k_trajectories(TrajArgs a) {
    static_assert(!(kRec && kBatch), "recording is for single runs");
    // a lane ends at most one visit per iteration and a block runs at most kFlush x (waves per block)
    // wave-iterations per epoch, so a slot gains at most kBlock * kFlush entries per epoch; a
    // retained count stays below kKeepCap, so the low half never carries
    static_assert(kKeep == 0 || kBlock * kFlush <= 32768, "retention needs 16-bit counts per epoch");
    constexpr uint32_t kKeepCap = 65536u - (uint32_t)(kBlock * kFlush);
    constexpr uint32_t kSuper = (uint32_t)kWindow * kBlock;  // slots per window top-up
    static_assert(kTbl % kBlock == 0, "every thread flushes the same number of table slots");
    constexpr int kPer = kTbl / kBlock;
    constexpr uint32_t kBuckets = (uint32_t)kTbl / 4u;
    __shared__ Table<kTbl> tb;
    __shared__ Control ctl;
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    const uint64_t total = wave_bcast64(a.run_off[a.n_runs]);
    // A small problem runs on fewer blocks: those past what gives each lane about the variant's slots per lane leave at
    // once.
    const uint64_t active = min((uint64_t)gridDim.x, active_blocks(total, kBlock, a.slots_per_lane));
    if ((uint64_t)blockIdx.x >= active) return;
    const int W = a.W, H = a.H;
    const float fW = (float)W, fH = (float)H;
    const uint32_t xcd = xcd_id();
    uint32_t* const counts = a.counts;
    uint32_t* const vmax2 = a.vmax2;
    const uint32_t Wp = (uint32_t)W + 2u, row_bytes = 4u * Wp;  // rows of the padded DEM tiles

    for (int k = threadIdx.x; k < kTbl; k += kBlock) {
        tb.tag[k] = kEmpty;
        tb.cnt[k] = 0u;
        tb.vmx[k] = 0u;
    }

    // A problem of at most a slot per lane runs out of slots at once, and the look at all the counters saves its waves a
    // walk over them (sweep of 94,000 paths 140 -> 132 us); in a larger one, where slots run out late and unevenly, the
    // walk measured faster (3.8e6 paths 413 us with the look, 376 without).
    const bool look = total <= (uint64_t)gridDim.x * kBlock;

    // Takes up to `len` consecutive slots from the XCD queues, starting with this XCD's partition and moving on to one
    // that has slots left when it is empty; [base, end) is empty once every partition is. A whole wave calls it, with
    // wave-uniform arguments. `left` receives what remained of the partition after the take.
    auto take_global = [&](uint32_t& part, uint32_t& gone, uint32_t& empty, uint32_t len, uint64_t& base,
                           uint64_t& end, uint64_t& left) {
        base = end = left = 0;
        while (!empty) {
            const uint64_t pb = part_begin(total, part), pe = part_begin(total, part + 1);
            uint64_t got = 0;
            if (lane == 0) got = atomicAdd(a.queues + part * kQueueStride, (unsigned long long)len);
            got = wave_bcast64(got);
            if (pb + got < pe) {
                base = pb + got;
                end = (base + len < pe) ? base + len : pe;
                left = pe - end;
                return;
            }
            if (look && gone == 0u) gone = empty_partitions(a.queues, total, lane);  // later failures are races
            gone |= 1u << part;
            if (gone == kAllGone)
                empty = 1u;
            else
                part = next_partition(part, gone);
        }
    };

    // Table slot of `key`, claimed if a candidate is empty; -1 if all of them are held by other cells. The candidates are
    // the four slots of the key's bucket, then those of a second bucket. A bucket's tags come in one 16-byte read: one
    // that shows the key is final within the epoch (only the key's own claim writes it, and slots are emptied only at a
    // boundary), and an empty one is settled by the compare-and-swap. (A kept slot behind a newly emptied one can give
    // a cell a second slot: both are flushed, the sums and maxima unchanged.) Two buckets of four overflow less than
    // eight slots in a row, and all candidates of a bucket are seen in one LDS round trip (8192^2 pass 9.2 -> 8.7 ms).
    auto bucket = [&](uint32_t key, uint32_t mul) -> uint32_t {
        // multiplicative hash modulo 2^24 with full-rate 24-bit products; the key's low 24 bits spread one block's cells
        return (__umul24((__umul24(key, mul) >> 8) & 0xFFFFu, kBuckets) >> 16) * 4u;
    };
    auto first_of = [&](const u32x4& t, uint32_t v) -> int {
        int e = -1;
#pragma unroll
        for (int i = 3; i >= 0; --i) e = t[i] == v ? i : e;
        return e;
    };
    // The claim past the first try: the key's two buckets, a compare-and-swap per empty candidate. Each failed one means
    // that the slot was filled meanwhile, so eight rounds see every candidate.
    auto claim_slow = [&](uint32_t key) -> int {
        const uint32_t first = bucket(key, 0x9E3779u);
        uint32_t at = first;
#pragma unroll 1
        for (int tries = 0; tries < 8; ++tries) {
            const u32x4 t = lds_ld4(tb.tag + at);
            int i = first_of(t, key);
            if (i >= 0) return (int)at + i;
            i = first_of(t, kEmpty);
            if (i >= 0) {
                const uint32_t old = atomicCAS(tb.tag + at + i, kEmpty, key);
                if (old == kEmpty || old == key) return (int)at + i;
            } else if (at == first) {
                at = bucket(key, 0xC2B2AEu) ^ 4u;
            } else {
                break;
            }
        }
        return -1;
    };
    // The visit that ended in the lane's previous iteration: its cell (kEmpty: none) and largest v^2. All lanes run the
    // bucket read and its compares; a branch is taken by the whole wave, for the lanes that claim and that overflow.
    uint32_t leave_key = kEmpty, leave_bits = 0;
    auto accumulate = [&]() {
        const bool has = leave_key != kEmpty;
        if (__ballot(has) == 0ull) return;
        const uint32_t at = bucket(leave_key, 0x9E3779u);
        const u32x4 t = lds_ld4(tb.tag + at);
        const int m = first_of(t, leave_key);
        int sl = m < 0 ? -1 : (int)at + m;
        if (__ballot(has && m < 0) != 0ull) {
            if (has && m < 0) {
                // the common claim: the bucket's first empty slot, taken by this key
                const int e = first_of(t, kEmpty);
                if (e >= 0) {
                    const uint32_t old = atomicCAS(tb.tag + at + e, kEmpty, leave_key);
                    if (old == kEmpty || old == leave_key) sl = (int)at + e;
                }
            }
            if (__ballot(has && sl < 0) != 0ull) {
                if (has && sl < 0) {
                    sl = claim_slow(leave_key);
                    if (sl < 0) {
                        atomicAdd(counts + leave_key, 1u);
                        if (leave_bits) global_max(vmax2 + leave_key, kBatch ? root_bits(leave_bits) : leave_bits);
                    }
                }
            }
        }
        if (has && sl >= 0) {
            atomicAdd(tb.cnt + sl, 1u);
            atomicMax(tb.vmx + sl, leave_bits);
        }
        leave_key = kEmpty;
    };

    // Shifts the window past the slots handed out in the epoch that ended and tops it up with a new
    // range when the second range has been reached. The block's first wave, between the barriers of a boundary.
    // The first range is at most half of the block's fair share of its partition (rounded up to a chunk): the blocks that
    // come first otherwise take kSuper slots each, and of a problem of one slot per lane they took four times their
    // share while the blocks after them found none (314,576 paths of 130 steps in 512-thread blocks: 1.4 ms, with the half share 0.60 ms).
    const uint64_t first_div = 2ull * max(1ull, (unsigned long long)active / kXcds);
    const uint64_t guide_div = 2ull * max(1u, gridDim.x / (uint32_t)kXcds);  // 2 x blocks per XCD
    auto refill_window = [&](bool first) {
        uint64_t b0 = 0, b1 = 0, left = 0;
        uint32_t l0 = 0, l1 = 0, t = 0, part = xcd, gone = 0, empty = total == 0 ? 1u : 0u;
        if (first) {
            left = part_begin(total, xcd + 1) - part_begin(total, xcd);
        } else {
            b0 = wave_bcast64(ctl.base[0]);
            b1 = wave_bcast64(ctl.base[1]);
            l0 = uniform_u(ctl.len[0]);
            l1 = uniform_u(ctl.len[1]);
            t = min(uniform_u(ctl.take), l0 + l1);
            part = uniform_u(ctl.part);
            gone = uniform_u(ctl.gone);
            empty = uniform_u(ctl.empty);
            left = wave_bcast64(ctl.left);
        }
        if (t >= l0) {
            b0 = b1 + (t - l0);
            l0 = l1 - (t - l0);
            l1 = 0;
        } else {
            b0 += t;
            l0 -= t;
        }
        if (l1 == 0u) {
            // guided top-up: a share of what the partition had left, so windows shrink as the queues
            // drain and every block runs out of work at about the same time
            const uint64_t share = left / (first ? first_div : guide_div);
            const uint32_t want = share >= kSuper ? kSuper : ((uint32_t)share / kChunk + 1u) * kChunk;
            uint64_t we = 0;
            take_global(part, gone, empty, want, b1, we, left);
            l1 = (uint32_t)(we - b1);
        }
        if (lane == 0) {
            ctl.base[0] = b0;
            ctl.base[1] = b1;
            ctl.len[0] = l0;
            ctl.len[1] = l1;
            ctl.take = 0;
            ctl.part = part;
            ctl.gone = gone;
            ctl.empty = empty;
            ctl.left = left;
            ctl.iters = 0u;
            if (first) {
                ctl.busy[0] = ctl.busy[1] = 0;
                ctl.dry = 0u;
            }
        }
    };
    // tail probe (diagnostics): per block the real-time clock at its start, when it first finds no slot left
    // in its window nor in any queue, and at its end
    unsigned long long* const probe = a.probe ? a.probe + 3 * (size_t)blockIdx.x : nullptr;
    if (probe && threadIdx.x == 0) probe[0] = __builtin_amdgcn_s_memrealtime();
    if (threadIdx.x < kWave) refill_window(true);
    __syncthreads();

    // The wave's run: its constants in scalar registers and its padded DEM tile through a buffer
    // resource (32-bit offsets, no clamps). A single run keeps run 0; in a batch a wave works on one run
    // at a time, and slots of the next run wait in its reservoir until the wave has no particle left.
    uint32_t wrun = 0;
    RunConst rc = uniform_run(a.runs[0]);
    __amdgpu_buffer_rsrc_t dem_rs = buffer_rsrc(a.dem_pad + rc.pad_off, a.pad_bytes);

    // per-lane statistics of run wrun, added to the run's counters when the wave changes run or ends. A
    // step is a move that does not hit the step limit: it is accepted, leaves the grid or stops, so the
    // steps are the accepted ones (each particle's final n, added when its lane takes the next particle or
    // the statistics are flushed) plus the exits and stops, and no counter moves per step for them.
    uint64_t st_acc = 0;
    uint32_t st_exit = 0, st_stop = 0, st_limit = 0;
    uint32_t n = 0;  // the lane's particle: accepted steps so far (not yet in st_acc)
    auto flush_stats = [&]() {
        st_acc += n;
        n = 0;
        const uint64_t s1 = wave_sum64(st_exit), s2 = wave_sum64(st_stop);
        const uint64_t s0 = wave_sum64(st_acc) + s1 + s2, s3 = wave_sum64(st_limit);
        if (lane == 0) {
            unsigned long long* st = a.stats + 4 * (size_t)wrun;
            if (s0) atomicAdd(st + 0, (unsigned long long)s0);
            if (s1) atomicAdd(st + 1, (unsigned long long)s1);
            if (s2) atomicAdd(st + 2, (unsigned long long)s2);
            if (s3) atomicAdd(st + 3, (unsigned long long)s3);
        }
        st_acc = 0;
        st_exit = st_stop = st_limit = 0;
    };

    // wave-uniform slot state: this wave's own walk over the XCD partitions (once the window is spent),
    // and a reservoir of up to 64 slots with the run they belong to
    uint32_t part = xcd, gone = 0, queue_empty = (total == 0) ? 1u : 0u;
    uint64_t res_next = 0, res_end = 0;
    uint32_t res_run = 0;

    // lane state
    bool alive = false;
    // (a lane without a particle keeps a unit gradient and direction: it runs the steps too, see below)
    float x = 0, y = 0, z = 0, gx = 1, gy = 0, dx = 1, dy = 0, v2 = 0, x0 = 0, y0 = 0, zr = 0, cmax2 = 0;
    uint32_t rep = 0, cell_id = 0, cur = 0;
    uint32_t rk = ~0u;  // recording: index of the lane's particle in the recorded range, ~0 if outside it
    auto rec_point = [&](uint32_t m, float px, float py, float pv2) {
        if constexpr (kRec) {
            if (rk == ~0u || !a.rec_xy) return;
            unsigned long long at;
            if (a.rec_off) {
                at = a.rec_off[rk] + m;
            } else {
                if (m >= a.rec_stride) return;
                at = (unsigned long long)rk * a.rec_stride + m;
            }
            a.rec_xy[at] = make_float2(px, py);
            if (a.rec_v2) a.rec_v2[at] = pv2;
        }
    };
    auto rec_end = [&](uint32_t why) {
        if constexpr (kRec) {
            if (rk != ~0u) a.rec_end[rk] = (n << 2) | why;
        }
    };


    // One step of every live particle, n the parity of `odd`. Every lane runs the whole step and the outcome selects what
    // it keeps: a lane at the step limit, leaving the grid or stopping discards its target (an off-grid target's gather
    // reads through the buffer's bounds check, so it cannot fault), and a lane without a particle discards everything.
    // Without a branch around the step or per outcome the compiler copies no particle state at joins, and a wave with
    // few lanes left, which decides when a pass ends, has no branch to wait for.
    auto step = [&](uint32_t ux, uint32_t uy) {
        const RunConst& R = rc;
        const float rx = signed_unit(ux), ry = signed_unit(uy);
        steer(dx, dy, gx, gy, R.per, R.Q, R.rnd, rx, ry);
        const float x1 = x + R.L * dx;
        const float y1 = y + R.L * dy;
        const PatchLoad pl = bilinear_pad_load(dem_rs, Wp, row_bytes, x1, y1);
        accumulate();  // the previous step's visit, while the heights are on their way
        const float fc1 = floorf(x1), fr1 = floorf(y1);
        const bool lim = n >= a.S;
        const bool inside = fc1 >= 0.0f && fc1 < fW && fr1 >= 0.0f && fr1 < fH;
        const bool go = alive && !lim, inb = go && inside;
        const Sample s1 = bilinear_pad_value(pl);
        const float dz = z - s1.z;
        // dl2 + dz^2 >= dl2: with dl2 >= 2^-96 (a run constant) no lane is below the short form's range
        const float ds = sqrt_rn(R.dl2 + dz * dz, R.dl2 >= 0x1p-96f ? 0u : kRootLo);
        const float num = v2 + a.g2 * (dz - R.mdl);
        bool stop = !(num > 0.0f);
        const float v2n = num / (1.0f + R.cd * ds);
        if (kAlpha && R.use_alpha) {
            float ax0 = x0, ay0 = y0, azr = zr;
            if (kBatch) {  // the release cell's centre and the height sampled there
                const uint32_t rr = udiv(cell_id, a.wdiv), cc = cell_id - rr * (uint32_t)W;
                ax0 = (float)cc + 0.5f;
                ay0 = (float)rr + 0.5f;
                azr = bilinear_pad(dem_rs, Wp, row_bytes, ax0, ay0).z;
            }
            const float hx = x1 - ax0, hy = y1 - ay0;
            stop = stop || (azr - s1.z) < R.tca * sqrtf(hx * hx + hy * hy);
        }
        const bool acc = inb && !stop;
        st_limit += (alive && lim) ? 1u : 0u;
        st_exit += (go && !inside) ? 1u : 0u;
        st_stop += (inb && stop) ? 1u : 0u;
        if constexpr (kRec) {
            if (alive) {
                if (lim)
                    rec_end(0u);
                else if (!inside)
                    rec_end(1u);
                else if (stop) {
                    rec_point(n + 1u, x1, y1, 0.0f);
                    rec_end(2u);
                }
            }
        }
        x = acc ? x1 : x;
        y = acc ? y1 : y;
        z = acc ? s1.z : z;
        gx = acc ? s1.gx : 1.0f;
        gy = acc ? s1.gy : 0.0f;
        v2 = acc ? v2n : v2;
        n += acc ? 1u : 0u;
        if constexpr (kRec) {
            if (acc) rec_point(n, x, y, v2);
        }
        // row x W as a 24-bit multiply (full rate; a 32-bit one is quarter rate): both factors are below
        // 2^23 on an accepted grid and nc is used only for a step inside it
        const uint32_t nc = R.raster_off + __umul24((uint32_t)(int)fr1, (uint32_t)W) + (uint32_t)(int)fc1;
        const bool change = acc && nc != cur;
        leave_key = (alive && (change || !acc)) ? cur : kEmpty;
        leave_bits = __float_as_uint(cmax2);
        cur = change ? nc : cur;
        cmax2 = change ? v2 : ((acc && v2 > cmax2) ? v2 : cmax2);
        alive = acc;
    };

    // pairs of wave-iterations per epoch: the wave claims two steps at a time, from an even step on
    constexpr uint32_t kBudget = (uint32_t)(kFlush / 2) * (uint32_t)(kBlock / kWave);
    static_assert(kFlush % 2 == 0, "an epoch is a whole number of step pairs");
    for (uint32_t epoch = 0;; ++epoch) {
        // the window of this epoch
        const uint64_t wb0 = wave_bcast64(ctl.base[0]), wb1 = wave_bcast64(ctl.base[1]);
        const uint32_t wl0 = uniform_u(ctl.len[0]), wl1 = uniform_u(ctl.len[1]);
        bool win_out = wl0 + wl1 == 0u;
        // few slots left: a single run's wave then takes no more from the queues than it has idle lanes, for what it held
        // in reserve would wait for its own lanes while other waves run out
        const bool scarce = uniform_u(ctl.empty) != 0u || wave_bcast64(ctl.left) < guide_div * kChunk;
        bool finished = false;

        // the wave claims each pair of the epoch's budget one pair ahead, so the LDS round trip overlaps the pair
        // before it
        uint32_t ticket = 0;
        if (lane == 0) ticket = atomicAdd(&ctl.iters, 1u);
        for (;;) {
            const uint64_t idle = __ballot(!alive);
            const int nidle = __popcll(idle);
            const bool drained = win_out && queue_empty && res_next >= res_end;
            if (nidle == kWave && drained) {
                finished = true;
                break;
            }
            if (__builtin_amdgcn_readfirstlane(ticket) >= kBudget) break;
            if (lane == 0) ticket = atomicAdd(&ctl.iters, 1u);

            // ---- hand slots to idle lanes in lane order. Between pairs of steps only, so that one
            // Philox block (two steps) serves every lane of the pair.
            bool fresh = false;
            if (nidle > 0 && !drained) {
                const int rank = __popcll(idle & below);
                uint64_t slot = ~0ull;
                if constexpr (!kBatch) {
                    // one run: the reservoir's remainder, then as many slots as lanes are idle from the window (which
                    // may end in its second range), else from the queues
                    const uint32_t avail = (uint32_t)(res_end - res_next);
                    if (avail >= (uint32_t)nidle) {
                        slot = res_next + rank;
                        res_next += nidle;
                    } else {
                        const uint32_t need = (uint32_t)nidle - avail;
                        uint64_t b1 = 0, b2 = 0;
                        uint32_t n1 = 0, n2 = 0;
                        if (!win_out) {
                            uint32_t v = 0;
                            if (lane == 0) v = atomicAdd(&ctl.take, need);
                            v = __builtin_amdgcn_readfirstlane(v);
                            if (v < wl0) {
                                b1 = wb0 + v;
                                n1 = min(need, wl0 - v);
                                b2 = wb1;
                                n2 = min(need - n1, wl1);
                            } else if (v - wl0 < wl1) {
                                b1 = wb1 + (v - wl0);
                                n1 = min(need, wl1 - (v - wl0));
                            } else {
                                win_out = true;
                            }
                        }
                        if (n1 == 0u && !queue_empty) {
                            uint64_t e, left;
                            take_global(part, gone, queue_empty, scarce ? need : max(need, kChunk), b1, e, left);
                            n1 = (uint32_t)(e - b1);
                        }
                        const uint32_t r = (uint32_t)rank - avail;
                        if ((uint32_t)rank < avail)
                            slot = res_next + rank;
                        else if (r < n1)
                            slot = b1 + r;
                        else if (r - n1 < n2)
                            slot = b2 + (r - n1);
                        res_next = b1 + min(n1, need);
                        res_end = b1 + n1;
                    }
                } else {
                    // a batch: the reservoir, refilled with the next 64-slot chunk of the window (else of the queues) when
                    // it runs dry; empty when neither has any left. A chunk of another run waits in the reservoir
                    // until the wave has no particle of its current run left
                    auto next_chunk = [&](uint64_t& base, uint64_t& cend) {
                        base = cend = 0;
                        if (!win_out) {
                            uint32_t v = 0;
                            if (lane == 0) v = atomicAdd(&ctl.take, kChunk);
                            v = __builtin_amdgcn_readfirstlane(v);
                            // the ranges are multiples of 64 long, so a chunk never straddles them
                            if (v < wl0) {
                                base = wb0 + v;
                                cend = base + min(wl0 - v, kChunk);
                            } else if (v - wl0 < wl1) {
                                base = wb1 + (v - wl0);
                                cend = base + min(wl1 - (v - wl0), kChunk);
                            } else {
                                win_out = true;
                            }
                        }
                        if (cend == base && !queue_empty) {
                            uint64_t left;
                            take_global(part, gone, queue_empty, kChunk, base, cend, left);
                        }
                    };
                    uint64_t want = idle;  // idle lanes not yet served
#pragma unroll 1
                    for (int round = 0; round < 2 && want != 0ull; ++round) {
                        if (res_next >= res_end) {
                            uint64_t base, cend;
                            next_chunk(base, cend);
                            if (cend == base) break;  // nothing left for this wave
                            res_next = base;
                            res_end = cend;
                            res_run = find_run(a.run_off, a.n_runs, base);
                        }
                        if (res_run != wrun) {
                            if (want != idle || __ballot(alive) != 0ull) break;
                            flush_stats();
                            wrun = res_run;
                            rc = uniform_run(a.runs[wrun]);
                            dem_rs = buffer_rsrc(a.dem_pad + rc.pad_off, a.pad_bytes);
                        }
                        const uint64_t avail = res_end - res_next;
                        const bool mine = ((want >> lane) & 1ull) != 0ull;
                        const int r = __popcll(want & below);
                        const bool served = mine && (uint64_t)r < avail;
                        if (served) slot = res_next + (uint64_t)r;
                        const uint64_t n_want = (uint64_t)__popcll(want);
                        res_next += avail < n_want ? avail : n_want;
                        want &= ~__ballot(served);
                    }
                }
                uint64_t i = 0;  // release-cell index of the new particle within its run
                if (!alive && slot < total) {
                    const uint64_t local = slot - (kBatch ? a.run_off[wrun] : 0ull);
                    if (local < rc.n_slots) {  // past n_slots: padding up to the next multiple of 64
                        i = (local >> 32) == 0 ? (uint64_t)udiv((uint32_t)local, a.pdiv) : local / rc.P;
                        rep = (uint32_t)local - (uint32_t)i * rc.P;
                        fresh = true;
                    }
                }
                if (fresh) {
                    // a single run reads the start state from its per-cell records, and so does a batch run
                    // whose scenario's records were made on its tile (a uniform branch); any other batch run
                    // computes it from the same padded tile the steps read
                    const StartRec st = !kBatch     ? a.starts[i]
                                        : rc.use_rec ? a.starts[rc.cells_off + i]
                                                     : start_state_pad(dem_rs, Wp, row_bytes, W,
                                                                       (uint32_t)a.cells[rc.cells_off + i]);
                    cell_id = st.cell;
                    x = st.x;
                    y = st.y;
                    z = st.z;
                    gx = st.gx;
                    gy = st.gy;
                    dx = st.dx;
                    dy = st.dy;
                    if (kAlpha && !kBatch) {
                        x0 = x;
                        y0 = y;
                        zr = z;
                    }
                    v2 = 0.0f;
                    cmax2 = 0.0f;
                    st_acc += n;  // the lane's previous particle
                    n = 0;
                    // the raster cell of the release point: the release texel's index keys the random
                    // stream, the DEM cell under its centre takes the counts (the same cell at one texel per
                    // DEM cell)
                    cur = rc.raster_off +
                          (kBatch ? cell_id : (uint32_t)(int)floorf(y) * (uint32_t)W + (uint32_t)(int)floorf(x));
                    alive = true;
                    if constexpr (kRec) {
                        const uint64_t k = (uint64_t)i * rc.P + rep;  // the particle's index in the run
                        rk = (k >= a.rec_first && k - a.rec_first < a.rec_n) ? (uint32_t)(k - a.rec_first) : ~0u;
                        rec_point(0u, x, y, 0.0f);
                    }
                }
            }

            // ---- two steps of every live particle: particles start here only, so their step count is even and one
            // Philox block serves both
            {
                // the key is wave-uniform: pinning it to scalar registers here makes the round keys
                // scalar adds inside the block instead of 20 loop-invariant values hoisted out of the
                // loop, spilled to vector lanes and read back by VALU instructions
                uint32_t k0 = __builtin_amdgcn_readfirstlane(rc.key0);
                uint32_t k1 = __builtin_amdgcn_readfirstlane(rc.key1);
                asm volatile("" : "+s"(k0), "+s"(k1));
                const uint4 o = philox4x32_10(n >> 1, rep, cell_id, rc.run, k0, k1);
                step(o.x, o.y);
                step(o.z, o.w);
            }
        }
        accumulate();

        // ---- epoch boundary: count the waves with work left, flush the table, refill the window
        if (lane == 0 && !finished) atomicAdd(&ctl.busy[epoch & 1u], 1u);
        __syncthreads();
        if (threadIdx.x < kWave) refill_window(false);
        if (threadIdx.x == 0) {
            ctl.busy[(epoch + 1) & 1u] = 0u;
            if (probe && !ctl.dry && ctl.empty && ctl.len[0] == 0u) {
                ctl.dry = 1u;
                probe[1] = __builtin_amdgcn_s_memrealtime();
            }
        }
        // flush this thread's kPer slots: all raster reads of the max check are issued before any is
        // used, so the flush costs one memory round trip rather than one per slot. The last boundary
        // (no wave has work left) flushes every slot.
        const bool last = ctl.busy[epoch & 1u] == 0u;
        uint32_t ft[kPer], fc[kPer], fv[kPer], fg[kPer];
        bool keep[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int k = threadIdx.x + j * kBlock;
            ft[j] = tb.tag[k];
            fc[j] = tb.cnt[k];
            fv[j] = tb.vmx[k];
            if constexpr (kKeep > 0) {
                const uint32_t c = fc[j] & 0xFFFFu, seen = fc[j] >> 16;
                keep[j] = !last && ft[j] != kEmpty && c - seen >= (uint32_t)kKeep && c < kKeepCap;
                fc[j] = c;
            } else {
                keep[j] = false;
            }
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j)  // an empty slot reads cell 0: no branch between the loads
            fg[j] = keep[j] ? 0u : cached_bits(vmax2 + (ft[j] != kEmpty ? ft[j] : 0u));
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int k = threadIdx.x + j * kBlock;
            if (keep[j]) {
                tb.cnt[k] = fc[j] | (fc[j] << 16);
            } else if (ft[j] != kEmpty) {
                if (fc[j]) atomicAdd(counts + ft[j], fc[j]);
                if constexpr (kBatch) fv[j] = root_bits(fv[j]);
                tb.tag[k] = kEmpty;
                tb.cnt[k] = 0u;
                tb.vmx[k] = 0u;
            }
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j)  // a stale read >= v suffices
            if (!keep[j] && ft[j] != kEmpty && fg[j] < fv[j]) atomicMax(vmax2 + ft[j], fv[j]);
        __syncthreads();
        if (ctl.busy[epoch & 1u] == 0u) break;
    }
    if constexpr (kBatch) {
        flush_stats();
    } else {
        // every wave leaves the loop at the same boundary: the block's statistics are summed in LDS and
        // reach the four counters with one atomic each per block, not per wave (the counters share a
        // memory line, where device-scope atomics serialise)
        unsigned long long* const bst = ctl.st;
        if (threadIdx.x < 4) bst[threadIdx.x] = 0ull;
        __syncthreads();
        st_acc += n;
        const uint64_t s1 = wave_sum64(st_exit), s2 = wave_sum64(st_stop);
        const uint64_t s0 = wave_sum64(st_acc) + s1 + s2, s3 = wave_sum64(st_limit);
        if (lane == 0) {
            if (s0) atomicAdd(bst + 0, (unsigned long long)s0);
            if (s1) atomicAdd(bst + 1, (unsigned long long)s1);
            if (s2) atomicAdd(bst + 2, (unsigned long long)s2);
            if (s3) atomicAdd(bst + 3, (unsigned long long)s3);
        }
        __syncthreads();
        if (threadIdx.x < 4 && bst[threadIdx.x]) atomicAdd(a.stats + threadIdx.x, bst[threadIdx.x]);
    }
    if (probe && threadIdx.x == 0) probe[2] = __builtin_amdgcn_s_memrealtime();
}

// ------------------------------------------------------------------------------------------ variants

namespace {

constexpr int kCandidates = 8;  // table slots a key may take: two buckets of four

struct Variant {
    const void* single;
    const void* batch;
    int block;
    uint32_t spl;  // particle slots per lane that size the grid of a small problem
    int shape[7];  // block, iterations per epoch, table slots, candidate slots, window, retention, waves per SIMD
    void (*launch_single)(dim3, dim3, hipStream_t, const TrajArgs&);        // runout-angle stop compiled in
    void (*launch_single_plain)(dim3, dim3, hipStream_t, const TrajArgs&);  // without it
    void (*launch_batch)(dim3, dim3, hipStream_t, const TrajArgs&);
};

template <bool B, bool A, int Blk, int F, int T, int M, int K, int Wpe>
void launch_t(dim3 g, dim3 t, hipStream_t s, const TrajArgs& a) {
    hipLaunchKernelGGL((k_trajectories<B, A, Blk, F, T, M, K, Wpe>), g, t, 0, s, a);
}

template <int Blk, int F, int T, int M, int K, int Wpe = 8>
constexpr Variant make_variant(uint32_t spl = (uint32_t)kSlotsPerLane) {
    return Variant{reinterpret_cast<const void*>(&k_trajectories<false, true, Blk, F, T, M, K, Wpe>),
                   reinterpret_cast<const void*>(&k_trajectories<true, true, Blk, F, T, M, K, Wpe>), Blk, spl,
                   {Blk, F, T, kCandidates, M, K, Wpe},
                   &launch_t<false, true, Blk, F, T, M, K, Wpe>, &launch_t<false, false, Blk, F, T, M, K, Wpe>,
                   &launch_t<true, true, Blk, F, T, M, K, Wpe>};
}

// candidates of the autotuner: (threads per block, iterations per epoch, table slots per block,
// window top-up in blocks of slots, retention threshold[, waves per SIMD of the register budget]) and the
// slots per lane that size a small problem's grid. 1024-thread blocks run two per CU at eight waves per SIMD
// (64 VGPRs; 6144 slots of 12 bytes are 72 KiB of LDS per block); the 768- and 512-thread shapes run at six
// (80 VGPRs), two and three blocks per CU, and the 384-thread shape at six with four blocks per CU. The fifth
// keeps no slot across epochs. The 1024-thread shapes spill up to 24 bytes a lane since the steps run in pairs, and lose where the
// chip is full (8192^2 13.9 to 18.4 ms against 12.7 to 13.0 of the best six-wave shapes, 2048^2 tile 2.85 to 3.15 against 2.69,
// 1024-run ensemble 26.7 to 30.8 against 24.6); in between one of them is kept now and then (release texture of 2 x 2 texels, 1001 x 1203).
// A problem that does not fill the chip lasts as long as a lane's paths, so one slot per lane is best for it (first
// shape: 314,576 paths of 130 steps 0.60 ms, at two slots per lane 1.04, at eight 2.4; 30,000 paths of 11 steps 0.13,
// 0.19 and 0.31 ms), and one that fills it does not see the difference. The first shape is the fastest, or within a
// few percent of it, on every workload from 10^5 to 2 10^9 steps, so it is also what a call takes that may not time.
const Variant kVariants[] = {
    make_variant<512, 16, 4096, 4, 1, 6>(1u),   make_variant<1024, 32, 6144, 4, 2>(),
    make_variant<1024, 16, 6144, 4, 1>(1u),     make_variant<1024, 16, 6144, 4, 2>(),
    make_variant<1024, 32, 4096, 4, 0>(),       make_variant<768, 16, 6144, 4, 1, 6>(1u),
    make_variant<768, 16, 6144, 4, 2, 6>(),     make_variant<512, 16, 4096, 4, 2, 6>(),
    make_variant<1024, 16, 6144, 4, 1>(2u),     make_variant<1024, 16, 6144, 4, 1>(4u),
    make_variant<512, 16, 4096, 4, 1, 6>(2u),   make_variant<512, 32, 4096, 4, 2, 6>(),
    make_variant<512, 16, 4096, 4, 1, 6>(),     make_variant<768, 16, 6144, 4, 1, 6>(),
    make_variant<384, 16, 3072, 4, 2, 6>(1u),
};

}  // namespace

int trajectory_variants() { return (int)(sizeof(kVariants) / sizeof(kVariants[0])); }

bool trajectory_variant_info(int variant, int32_t* info) {
    if (variant < 0 || variant >= trajectory_variants()) return false;
    const Variant& v = kVariants[variant];
    for (int i = 0; i < 7; ++i) info[i] = v.shape[i];
    info[7] = (int32_t)v.spl;
    return true;
}

LaunchShape trajectory_shape(bool batched, int variant) {
    if (variant < 0 || variant >= trajectory_variants()) variant = 0;
    const Variant& v = kVariants[variant];
    LaunchShape sh{v.block, 2048, variant};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return sh;
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return sh;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, batched ? v.batch : v.single, v.block, 0) !=
            hipSuccess ||
        per_cu <= 0)
        per_cu = 1;
    sh.grid = cus * per_cu;
    return sh;
}

hipError_t launch_trajectories_record(const TrajArgs& a, hipStream_t s) {
    auto* k = &k_trajectories<false, true, 1024, 16, 6144, 4, 1, 8, true>;
    int dev = 0, cus = 256, per_cu = 1;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0 &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(k), 1024, 0) ==
            hipSuccess &&
        per_cu > 0) {
    } else {
        cus = 256;
        per_cu = 1;
    }
    TrajArgs b = a;
    b.slots_per_lane = (uint32_t)kSlotsPerLane;
    hipLaunchKernelGGL(k, dim3(cus * per_cu), dim3(1024), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_trajectories(const TrajArgs& a, bool batched, const LaunchShape& shape, hipStream_t s) {
    const int vi = (shape.variant >= 0 && shape.variant < trajectory_variants()) ? shape.variant : 0;
    const Variant& v = kVariants[vi];
    TrajArgs b = a;
    b.slots_per_lane = v.spl;
    if (batched)
        v.launch_batch(dim3(shape.grid), dim3(v.block), s, b);
    else if (a.runout_angle)
        v.launch_single(dim3(shape.grid), dim3(v.block), s, b);
    else
        v.launch_single_plain(dim3(shape.grid), dim3(v.block), s, b);
    return hipGetLastError();
}

}  // namespace avl

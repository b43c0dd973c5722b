// What a trajectory pass needs before its particles start: cleared rasters, counters and queues, the DEM with a
// replicated border, the row-major list of release texels (section 5.2 of arXiv 2506.23364: particles are released
// per coded texel) with the start state of each, and the run table.
//
// A small pass is over in some 150 us, so launches count: these parts were ten kernels of 3 to 5 us each. They are
// three, or two where the masks are small (kDirectScan): one for everything that depends on the call's inputs alone (its
// blocks take one of three roles), a scan of the mask counts where there are many, and one that writes the cells and
// their records and, for a single run, the run table. All of them are streaming passes.
#include <algorithm>

#include "particle.h"
#include "setup.h"

namespace avl {

using namespace dev;

// ------------------------------------------------------------------------------------------ first kernel
// Roles by block: counts of nonzero mask bytes per kScanChunk texels; 4096 texels of a padded DEM; 8192 words of a
// fill (kernels and not memset nodes, so that the sequence can be captured into a graph).
namespace {
constexpr int kPrepThreads = 256;
constexpr int kPadChunk = 16 * kPrepThreads;   // padded texels per block
constexpr int kFillChunk = 32 * kPrepThreads;  // words per block
static_assert(kPrepThreads == kScanThreads, "the counting role scans with the block's threads");

typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at a 4-byte aligned address
}  // namespace

// exclusive scan of one value per thread over a block of kScanThreads; returns the block total in *total. kAgain: another one
// follows in the block.
template <bool kAgain>
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t* total) {
    __shared__ uint32_t wsum[kScanThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const uint32_t inc = wave_incl_scan(v);
    if (lane == kWave - 1) wsum[wid] = inc;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < kScanThreads / kWave; ++k) {
        before += (k < wid) ? wsum[k] : 0u;
        tot += wsum[k];
    }
    if (kAgain) __syncthreads();
    *total = tot;
    return before + inc - v;
}

// the 16 mask bytes of a thread, [base, base + 16): one 16-byte load when all of them are in range and the
// address is 16-byte aligned (a lane per 16 bytes, so a wave reads 1 KiB contiguously), else byte by byte with
// the bytes past n read as 0
__device__ inline uint4 mask16(const uint8_t* __restrict__ mask, int64_t base, int64_t n) {
    static_assert(kScanPerThread == 16, "one 16-byte load per thread");
    if (base + 16 <= n && (reinterpret_cast<uintptr_t>(mask + base) & 15) == 0)
        return *reinterpret_cast<const uint4*>(mask + base);
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    for (int k = 0; k < 16; ++k)
        if (base + k < n) w[k >> 2] |= (uint32_t)mask[base + k] << (8 * (k & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// bit 7 of each byte of the result is set iff that byte of w is nonzero
__device__ inline uint32_t nonzero_bytes(uint32_t w) {
    return (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u;
}

__device__ inline uint32_t count16(const uint4 m) {
    return __popc(nonzero_bytes(m.x)) + __popc(nonzero_bytes(m.y)) + __popc(nonzero_bytes(m.z)) +
           __popc(nonzero_bytes(m.w));
}

// The DEM with a one-texel border replicating the edge texels: (H + 2) x (W + 2), row-major. Its texel (r + 1, c + 1)
// holds dem[clamp(r)][clamp(c)] for r in [-1, H], c in [-1, W], which is what the clamped bilinear patch reads, so the
// padded lookup needs no clamps. Four texels a thread in one 16-byte load (4-byte aligned: the rows are shifted by one
// texel against the source's) and store; only the four that hold a border column go one by one.
__device__ __forceinline__ void pad_role(const float* __restrict__ dem, float* __restrict__ out, int H, int W,
                                         const DivU32& wpdiv, uint32_t block) {
    const uint32_t Wp = (uint32_t)W + 2u, np = (uint32_t)padded_cells(H, W);  // < 2^30
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t i0 = block * (uint32_t)kPadChunk + ((uint32_t)k * kPrepThreads + threadIdx.x) * 4u;
        if (i0 >= np) return;
        uint32_t r = udiv(i0, wpdiv), c = i0 - r * Wp;
        if (c >= 1u && c + 3u <= (uint32_t)W) {  // source columns c - 1 .. c + 2, the last at most W - 1
            const int64_t sr = min(max((int)r - 1, 0), H - 1);
            *reinterpret_cast<u32x4a4*>(out + i0) = *reinterpret_cast<const u32x4a4*>(dem + sr * W + (c - 1u));
        } else {
            for (uint32_t q = 0; q < 4u && i0 + q < np; ++q) {
                const int64_t sr = min(max((int)r - 1, 0), H - 1), sc = min(max((int)c - 1, 0), W - 1);
                out[i0 + q] = dem[sr * W + sc];
                if (++c == Wp) {
                    c = 0;
                    ++r;
                }
            }
        }
    }
}

__device__ __forceinline__ void fill_role(const Fill& f, uint32_t block) {
    const int64_t base = (int64_t)block * kFillChunk;
#pragma unroll
    for (int k = 0; k < kFillChunk / (4 * kPrepThreads); ++k) {
        const int64_t i0 = base + ((int64_t)k * kPrepThreads + threadIdx.x) * 4;
        if (i0 + 4 <= f.n) {
            const u32x4a4 v = {f.v, f.v, f.v, f.v};
            *reinterpret_cast<u32x4a4*>(f.p + i0) = v;
        } else {
            for (int64_t i = i0; i < f.n; ++i) f.p[i] = f.v;
        }
    }
}

__global__ __launch_bounds__(kPrepThreads) void k_prepare(PrepArgs a) {
    uint32_t b = a.first + blockIdx.x;
    if (b < a.count_blocks) {
        const uint32_t m = a.n_masks == 1u ? 0u : b / a.nb, chunk = b - m * a.nb;
        const int64_t base = (int64_t)chunk * kScanChunk + (int64_t)threadIdx.x * kScanPerThread;
        uint32_t total;
        (void)block_excl_scan<false>(count16(mask16(a.mask + (int64_t)m * a.n, base, a.n)), &total);
        if (threadIdx.x == 0) a.blk[b] = total;
        return;
    }
    b -= a.count_blocks;
    if (b < a.pad_blocks) {
        const uint32_t t = b / a.pad_nb;
        pad_role(a.dem + (int64_t)t * a.H * a.W, a.dem_pad + (int64_t)t * padded_cells(a.H, a.W), a.H, a.W, a.wpdiv,
                 b - t * a.pad_nb);
        return;
    }
    b -= a.pad_blocks;
#pragma unroll
    for (int k = 0; k < kFills; ++k) {
        if (b < a.fill_blocks[k]) {
            fill_role(a.fill[k], b);
            return;
        }
        b -= a.fill_blocks[k];
    }
}

hipError_t launch_prepare(PrepArgs a, hipStream_t s) {
    uint64_t total = 0;
    a.nb = 0;
    a.count_blocks = a.pad_blocks = a.pad_nb = 0;
    if (a.mask) {
        a.nb = (uint32_t)scan_blocks(a.n);
        a.count_blocks = a.nb * a.n_masks;
        total += (uint64_t)a.nb * a.n_masks;
    }
    if (a.dem) {
        a.wpdiv = make_divu32((uint32_t)a.W + 2u);
        a.pad_nb = (uint32_t)((padded_cells(a.H, a.W) + kPadChunk - 1) / kPadChunk);
        a.pad_blocks = a.pad_nb * a.n_tiles;
        total += (uint64_t)a.pad_nb * a.n_tiles;
    }
    for (int k = 0; k < kFills; ++k) {
        const uint64_t nb = a.fill[k].p && a.fill[k].n > 0 ? (uint64_t)((a.fill[k].n + kFillChunk - 1) / kFillChunk) : 0;
        a.fill_blocks[k] = (uint32_t)nb;
        total += nb;
    }
    // a launch holds less than 2^32 threads (more wrap, without an error), and a batch of very many small tiles or masks has a block for each; its entry
    // limits keep the blocks of all roles below 2^32
    constexpr uint64_t kMaxBlocks = uint64_t(1) << 23;
    hipError_t e = hipSuccess;
    for (uint64_t at = 0; at < total && e == hipSuccess; at += kMaxBlocks) {
        a.first = (uint32_t)at;
        hipLaunchKernelGGL(k_prepare, dim3((unsigned)std::min(total - at, kMaxBlocks)), dim3(kPrepThreads), 0, s, a);
        e = hipGetLastError();
    }
    return e;
}

// ------------------------------------------------------------------------------------------ scan of the counts
// Block m: exclusive scan of mask m's nb counts in place, its total into n_cells[m]. Only where there are many
// (kDirectScan): else every block of the next kernel sums the counts before its own itself.
__global__ __launch_bounds__(1024) void k_scan_counts(uint32_t* __restrict__ blk, uint32_t nb, int32_t* __restrict__ n_cells) {
    __shared__ uint32_t wsum[1024 / kWave];
    uint32_t* const p = blk + (uint64_t)blockIdx.x * nb;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    uint32_t carry = 0;
    uint32_t v[4], next[4];
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) next[k] = threadIdx.x * 4u + k < nb ? p[threadIdx.x * 4u + k] : 0u;
    for (uint32_t base = 0; base < nb; base += 4096u) {
        const uint32_t i0 = base + threadIdx.x * 4u;
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            v[k] = next[k];
            next[k] = i0 + 4096u + k < nb ? p[i0 + 4096u + k] : 0u;
        }
        const uint32_t local = v[0] + v[1] + v[2] + v[3];
        const uint32_t inc = wave_incl_scan(local);
        if (lane == kWave - 1) wsum[wid] = inc;
        __syncthreads();
        uint32_t before = 0, tot = 0;
#pragma unroll
        for (int k = 0; k < 1024 / kWave; ++k) {
            before += (k < wid) ? wsum[k] : 0u;
            tot += wsum[k];
        }
        uint32_t run = carry + before + inc - local;
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            if (i0 + k < nb) p[i0 + k] = run;
            run += v[k];
        }
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) n_cells[blockIdx.x] = (int32_t)carry;
}

// ------------------------------------------------------------------------------------------ cells and records

// Block (chunk, mask): the chunk's release texels in order behind those of the chunks before it, and per texel its start
// record and particle mass (single runs; a batch's records depend on its run table). The texels are gathered in LDS
// first, so that the records are computed and written by consecutive threads however sparse the mask is. The last
// chunk's block knows the mask's total: n_cells, and a single run's table.
__global__ __launch_bounds__(kScanThreads) void k_release_list(ListArgs a) {
    __shared__ uint16_t list[kScanChunk];
    const uint32_t m = blockIdx.y, b = blockIdx.x;
    const uint8_t* const mask = a.mask + (int64_t)m * a.n;
    const int64_t chunk = (int64_t)b * kScanChunk;
    const uint4 w4 = mask16(mask, chunk + (int64_t)threadIdx.x * kScanPerThread, a.n);
    const uint32_t* const blk = a.blk + (uint64_t)m * a.nb;
    uint32_t base, total;
    if (a.scanned) {
        base = blk[b];
    } else {
        uint32_t sum = 0;
        for (uint32_t i = threadIdx.x; i < b; i += kScanThreads) sum += blk[i];
        (void)block_excl_scan<true>(sum, &base);
    }
    uint32_t pos = block_excl_scan<false>(count16(w4), &total);
    const uint32_t w[4] = {nonzero_bytes(w4.x), nonzero_bytes(w4.y), nonzero_bytes(w4.z), nonzero_bytes(w4.w)};
#pragma unroll
    for (int q = 0; q < 4; ++q)  // bytes past n were read as 0
        for (uint32_t v = w[q]; v != 0u; v &= v - 1u)
            list[pos++] = (uint16_t)(threadIdx.x * kScanPerThread + 4 * q + (__builtin_ctz(v) >> 3));
    __syncthreads();
    int32_t* const cells = a.cells + (int64_t)m * a.cells_stride;
    for (uint32_t i = threadIdx.x; i < total; i += kScanThreads) {
        const uint32_t cell = (uint32_t)(chunk + list[i]);
        const int64_t at = (int64_t)base + i;
        cells[at] = (int32_t)cell;
        if (a.starts && at < a.cap) {
            a.starts[at] = start_state(a.dem, a.H, a.W, a.mult, cell);
            if (a.mpc) a.mpc[at] = (a.mass ? a.mass[cell] : 1.0f) / (float)a.setup.P;
        }
    }
    if (b == a.nb - 1u && threadIdx.x == 0) {
        const uint32_t n = base + total;
        a.n_cells[m] = (int32_t)n;
        if (a.setup.run) setup_one(a.setup, a.H, a.W, (int64_t)n);
    }
}

// Chunks of one mask up to which the list's blocks sum the counts before them themselves instead of a scan of its own. Those
// sums read nb^2 / 2 counts a mask (at 2048 chunks, 8 M texels: 4 loads a thread on average, 8.4 MB from L2 in all), the scan
// costs a launch; so for several masks nb^2 times their number decides. A batch with nothing else to do, summed and scanned: one
// mask of 1024 chunks 42.4 and 44.0 us, of 2048 53.4 and 55.1, of 4096 82.1 and 81.7; 4 of 1024 48.7 and 49.4, 16 of 1024 74.7 and
// 71.1, 64 of 1024 186 and 161; 4 of 2048 66.4 and 65.4, 64 of 2048 390 and 298. Up to kScanThreads chunks a thread reads one
// count at most and a scan never pays (64 of 256 66.6 and 65.0, 16 of 256 40.2 and 41.2); that also bounds the scan's grid.
constexpr uint64_t kDirectScan = 2048;

hipError_t launch_release_list(ListArgs a, uint32_t n_masks, hipStream_t s) {
    a.nb = (uint32_t)scan_blocks(a.n);
    if (a.nb == 0) return hipErrorInvalidValue;
    a.scanned = a.nb > (uint32_t)kScanThreads && (uint64_t)a.nb * a.nb * n_masks > kDirectScan * kDirectScan ? 1 : 0;
    if (a.scanned) hipLaunchKernelGGL(k_scan_counts, dim3(n_masks), dim3(1024), 0, s, a.blk, a.nb, a.n_cells);
    for (uint32_t m = 0; m < n_masks; m += 65535u) {  // the grid's y limit
        ListArgs c = a;
        c.mask += (int64_t)m * a.n;
        c.blk += (uint64_t)m * a.nb;
        c.cells += (int64_t)m * a.cells_stride;
        c.n_cells += m;
        hipLaunchKernelGGL(k_release_list, dim3(a.nb, std::min(n_masks - m, 65535u)), dim3(kScanThreads), 0, s, c);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ run table of a batch

// One block: per run, derived constants and slot counts, then the exclusive scan of the padded slot
// counts. A run with an index out of range or invalid parameters gets no slots and status != 0.
__global__ __launch_bounds__(1024) void k_setup_runs(const RunSpec* __restrict__ specs,
                                                     const ::avl_params* __restrict__ params, uint32_t n_params,
                                                     const int32_t* __restrict__ n_cells_per_scen, uint32_t n_scen,
                                                     uint32_t n_tiles, uint32_t n_runs, int32_t H, int32_t W,
                                                     float cs, uint32_t P, RunConst* __restrict__ runs,
                                                     unsigned long long* __restrict__ run_off,
                                                     int32_t* __restrict__ status, int32_t* __restrict__ rec_run) {
    __shared__ unsigned long long wsum[1024 / kWave];
    const uint32_t per_thread = (n_runs + 1023) / 1024;
    const uint32_t b0 = threadIdx.x * per_thread;
    const uint64_t HW = (uint64_t)H * W;
    unsigned long long local = 0;
    for (uint32_t k = 0; k < per_thread; ++k) {
        const uint32_t r = b0 + k;
        if (r >= n_runs) break;
        const RunSpec sp = specs[r];
        int32_t bad = 0;
        if (sp.tile >= n_tiles || sp.scenario >= n_scen || sp.param >= n_params) bad = 1;
        ::avl_params p{};
        if (!bad) {
            p = params[sp.param];
            bad = param_status(p);
        }
        RunConst c = run_const(sp, p, H, W, cs, P);
        c.raster_off = (uint32_t)(r * HW);
        c.n_slots = bad ? 0ull : (unsigned long long)(uint32_t)n_cells_per_scen[sp.scenario] * P;
        runs[r] = c;
        if (status) status[r] = bad;
        if (!bad) atomicMin(rec_run + sp.scenario, (int32_t)r);
        local += (c.n_slots + kChunk - 1) / kChunk * kChunk;
    }
    // exclusive scan of the per-thread sums
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    unsigned long long inc = local;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const unsigned long long t = __shfl_up(inc, d, kWave);
        if (lane >= d) inc += t;
    }
    if (lane == kWave - 1) wsum[wid] = inc;
    __syncthreads();
    unsigned long long before = 0, tot = 0;
    for (int k = 0; k < 1024 / kWave; ++k) {
        before += (k < wid) ? wsum[k] : 0ull;
        tot += wsum[k];
    }
    unsigned long long run = before + inc - local;
    for (uint32_t k = 0; k < per_thread; ++k) {
        const uint32_t r = b0 + k;
        if (r >= n_runs) break;
        run_off[r] = run;
        run += (runs[r].n_slots + kChunk - 1) / kChunk * kChunk;
        // every run's atomicMin has completed at the barrier above; read the result past the L1
        if (specs[r].scenario < n_scen && specs[r].tile < n_tiles) {
            const int32_t first =
                __hip_atomic_load(rec_run + specs[r].scenario, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            runs[r].use_rec = (first != 0x7FFFFFFF && specs[first].tile == specs[r].tile) ? 1u : 0u;
        }
    }
    if (threadIdx.x == 0) run_off[n_runs] = tot;
}

hipError_t launch_setup_runs(const RunSpec* specs, const ::avl_params* params, uint32_t n_params,
                             const int32_t* n_cells_per_scen, uint32_t n_scen, uint32_t n_tiles, uint32_t n_runs,
                             int32_t H, int32_t W, float cell_size, uint32_t P, RunConst* runs,
                             unsigned long long* run_off, int32_t* status, int32_t* rec_run, hipStream_t s) {
    hipLaunchKernelGGL(k_setup_runs, dim3(1), dim3(1024), 0, s, specs, params, n_params, n_cells_per_scen, n_scen,
                       n_tiles, n_runs, H, W, cell_size, P, runs, run_off, status, rec_run);
    return hipGetLastError();
}

// Batch start records: scenario s's cells on the tile of its first valid run, from the padded tile (the
// same values the trajectory kernel would read, so the same start states).
__global__ __launch_bounds__(256) void k_batch_records(const RunSpec* __restrict__ specs,
                                                       const int32_t* __restrict__ rec_run,
                                                       const int32_t* __restrict__ n_cells_per_scen, uint32_t n_scen,
                                                       const int32_t* __restrict__ cells, const float* dem_pad, int H,
                                                       int W, StartRec* __restrict__ starts) {
    const uint64_t HW = (uint64_t)H * W;
    const uint32_t Wp = (uint32_t)W + 2u, row_bytes = 4u * Wp;
    const uint64_t np = (uint64_t)padded_cells(H, W);
    for (uint32_t sc = blockIdx.y; sc < n_scen; sc += gridDim.y) {
        const int32_t first = rec_run[sc];
        if (first == 0x7FFFFFFF) continue;  // no valid run uses this scenario
        const __amdgpu_buffer_rsrc_t rs =
            buffer_rsrc(dem_pad + (uint64_t)specs[first].tile * np, (uint32_t)(np * sizeof(float)));
        const int64_t nc = n_cells_per_scen[sc];
        for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nc; i += (int64_t)gridDim.x * blockDim.x)
            starts[sc * HW + i] = start_state_pad(rs, Wp, row_bytes, W, (uint32_t)cells[sc * HW + i]);
    }
}

hipError_t launch_batch_records(const RunSpec* specs, const int32_t* rec_run, const int32_t* n_cells_per_scen,
                                uint32_t n_scen, const int32_t* cells, const float* dem_pad, int32_t H, int32_t W,
                                StartRec* starts, hipStream_t s) {
    const uint32_t gy = n_scen < 1024u ? n_scen : 1024u;
    hipLaunchKernelGGL(k_batch_records, dim3(64, gy), dim3(256), 0, s, specs, rec_run, n_cells_per_scen, n_scen, cells,
                       dem_pad, H, W, starts);
    return hipGetLastError();
}

}  // namespace avl

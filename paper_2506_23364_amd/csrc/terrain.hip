// Terrain passes of the avalanche overlay (section 5.2 of arXiv 2506.23364): surface normals and
// steepness per DEM texel, the release-point map from a steepness range and an elevation window. Plus the
// finalize pass of the trajectory pass and the overlay mipmap.
//
// These are streaming passes, written for 64-wide wavefronts with every wave touching whole 256-byte
// stretches of consecutive cells, and bound by HBM bandwidth.
#include "particle.h"

namespace avl {

// ------------------------------------------------------------------------------------------ normals
// Block = 64 x 16 texels, 256 threads (one wave per row, four rows per thread); the tile plus a
// one-texel halo is staged in LDS so every DEM value is read from L2/HBM about once. Gradient: central
// difference inside, one-sided at the grid edges (the textbook finite difference);
// n = (-gx, -gy, 1)/sqrt(gx^2 + gy^2 + 1). Each texel takes five correctly rounded quotients, two square roots and an
// arctangent. The quotients share two divisors, so they come from two reciprocals (of the cell size, correctly rounded
// on the host, and of the root, from the same estimate as the root itself) by one residual step each, and the pass is
// bound by HBM where the compiler's five divisions bound it by VALU issue (3000 x 5001: 73 -> 64 us).
// kMask: the release map of the same texels as well (the release-mask pass below on the nz just computed and
// the staged height, so the map is the one that pass writes from these normals, without reading them back).
struct MaskArgs {
    float cmin, cmax, zmin, zmax;
    uint8_t* mask;
};
struct CellSize {
    float cs, cs2;    // the texel edge, twice it
    float rcs, rcs2;  // their reciprocals, correctly rounded
    int mid;          // both in [2^-40, 2^40]
};
constexpr int kNTX = 64, kNTY = 16, kNRows = 4;  // tile columns, tile rows, rows of threads

// The texel's outputs from its height differences dx, dy over sx, sy (reciprocals rx, ry). The short quotients are those
// of the compiler's divisions (Markstein's residual step from a correctly rounded reciprocal) where no operand, quotient
// or residual comes near the subnormal or overflow range: a wave with a lane outside takes the divisions.
__device__ __forceinline__ float4 normal_of(float dx, float dy, float sx, float sy, float rx, float ry, int mid) {
    auto quotient = [](float a, float b, float r) {
        const float q = a * r;
        return __builtin_fmaf(__builtin_fmaf(-b, q, a), r, q);
    };
    // |g| in [2^-60, 2^60], or the difference is +0; one of -0 (+0.0 and -0.0 side by side) keeps its sign only in a division,
    // for the residual step adds a +0
    auto in_range = [](float d, float g) {
        return __float_as_uint(d) == 0u || (__float_as_uint(g) & 0x7FFFFFFFu) - 0x21800000u <= 0x5D800000u - 0x21800000u;
    };
    float gx = quotient(dx, sx, rx), gy = quotient(dy, sy, ry);
    float gg = gx * gx + gy * gy;
    // 0 < gg < 2^-96 falls outside the short root's range; gg = 0 has the root 0
    const bool odd = !in_range(dx, gx) || !in_range(dy, gy) || !(gg == 0.0f || gg >= 0x1p-96f);
    float4 o;
    if (mid && __builtin_expect(__ballot(odd) == 0ull, 1)) {
        const dev::RootEst e = dev::sqrt_est(gg + 1.0f);
        const float r = dev::recip_root(e);
        o.x = -quotient(gx, e.s, r);
        o.y = -quotient(gy, e.s, r);
        o.z = r;
        o.w = atanf(gg > 0.0f ? dev::sqrt_est(gg).s : 0.0f) * 57.295779513082320876798f;
    } else {
        gx = dx / sx;
        gy = dy / sy;
        gg = gx * gx + gy * gy;
        const float l = sqrtf(gg + 1.0f);
        o.x = -(gx / l);
        o.y = -(gy / l);
        o.z = 1.0f / l;
        o.w = atanf(sqrtf(gg)) * 57.295779513082320876798f;
    }
    return o;
}

template <bool kMask>
__global__ __launch_bounds__(kNTX * kNRows) void k_normals(const float* __restrict__ dem, int H, int W, CellSize s,
                                                           float4* __restrict__ out, MaskArgs m) {
    __shared__ float tile[kNTY + 2][kNTX + 2];
    const int tx = threadIdx.x & (kNTX - 1), ty = threadIdx.x / kNTX;
    const int c0 = blockIdx.x * kNTX, r0 = blockIdx.y * kNTY;
    // stage (kNTY + 2) x (kNTX + 2) texels with clamped indices
    for (int i = threadIdx.x; i < (kNTY + 2) * (kNTX + 2); i += kNTX * kNRows) {
        int lr = i / (kNTX + 2), lc = i - lr * (kNTX + 2);
        int r = min(max(r0 + lr - 1, 0), H - 1);
        int c = min(max(c0 + lc - 1, 0), W - 1);
        tile[lr][lc] = dem[(size_t)r * W + c];
    }
    __syncthreads();
    const int c = c0 + tx;
    if (c >= W) return;
    // an edge texel's neighbour outside the grid is staged as the texel itself, so the one-sided difference is the
    // staged one over the single edge
    const bool ex = c == 0 || c == W - 1;
    const float sx = ex ? s.cs : s.cs2, rx = ex ? s.rcs : s.rcs2;
#pragma unroll
    for (int k = 0; k < kNTY / kNRows; ++k) {
        const int r = r0 + ty + k * kNRows;
        if (r >= H) break;
        const int lr = ty + k * kNRows + 1, lc = tx + 1;
        const bool ey = r == 0 || r == H - 1;
        const float4 o = normal_of(tile[lr][lc + 1] - tile[lr][lc - 1], tile[lr + 1][lc] - tile[lr - 1][lc], sx,
                                   ey ? s.cs : s.cs2, rx, ey ? s.rcs : s.rcs2, s.mid);
        out[(size_t)r * W + c] = o;
        if constexpr (kMask) {
            const float z = tile[lr][lc];  // dem[r][c]: an in-grid texel is staged unclamped
            m.mask[(size_t)r * W + c] = (m.cmin <= o.z && o.z <= m.cmax && m.zmin <= z && z <= m.zmax) ? 1 : 0;
        }
    }
}

static CellSize cell_size_of(float cs) {
    CellSize s;
    s.cs = cs;
    s.cs2 = 2.0f * cs;
    s.rcs = 1.0f / s.cs;
    s.rcs2 = 1.0f / s.cs2;
    s.mid = cs >= 0x1p-40f && s.cs2 <= 0x1p40f;
    return s;
}

hipError_t launch_normals(const float* dem, int H, int W, float cs, float* out4, hipStream_t s) {
    dim3 grid((W + kNTX - 1) / kNTX, (H + kNTY - 1) / kNTY);
    hipLaunchKernelGGL(k_normals<false>, grid, dim3(kNTX * kNRows), 0, s, dem, H, W, cell_size_of(cs),
                       reinterpret_cast<float4*>(out4), MaskArgs{});
    return hipGetLastError();
}

hipError_t launch_normals_mask(const float* dem, int H, int W, float cs, float cmin, float cmax, float zmin,
                               float zmax, float* out4, uint8_t* mask, hipStream_t s) {
    dim3 grid((W + kNTX - 1) / kNTX, (H + kNTY - 1) / kNTY);
    hipLaunchKernelGGL(k_normals<true>, grid, dim3(kNTX * kNRows), 0, s, dem, H, W, cell_size_of(cs),
                       reinterpret_cast<float4*>(out4), MaskArgs{cmin, cmax, zmin, zmax, mask});
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ release mask
// Streaming passes over normals and heights, bound by HBM: kStream texels a thread, kStreamThreads apart, so that every
// load and store of a wave is one contiguous stretch (nz alone: 1 KiB). The blocks run from the last texels to the
// first: the normals were just written in the other order, and what the memory-side cache still holds of them is their
// end (3000 x 5001 snow pass, 240 MB of normals: 91 -> 60 us).
constexpr int kStream = 4, kStreamThreads = 256, kStreamBlock = kStream * kStreamThreads;

__device__ __forceinline__ int64_t stream_base() {
    return (int64_t)(gridDim.x - 1u - blockIdx.x) * kStreamBlock + threadIdx.x;
}

__global__ __launch_bounds__(kStreamThreads) void k_release_mask(const float4* __restrict__ nrm, const float* __restrict__ dem,
                                                                 int64_t n, float cmin, float cmax, float zmin, float zmax,
                                                                 uint8_t* __restrict__ mask) {
    const int64_t i0 = stream_base();
    float nz[kStream], z[kStream];
#pragma unroll
    for (int k = 0; k < kStream; ++k) {
        const int64_t i = i0 + k * kStreamThreads;
        nz[k] = i < n ? nrm[i].z : 0.0f;
        z[k] = i < n ? dem[i] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < kStream; ++k) {
        const int64_t i = i0 + k * kStreamThreads;
        if (i < n) mask[i] = (cmin <= nz[k] && nz[k] <= cmax && zmin <= z[k] && z[k] <= zmax) ? 1 : 0;
    }
}

static unsigned stream_blocks(int64_t n) { return (unsigned)((n + kStreamBlock - 1) / kStreamBlock); }

hipError_t launch_release_mask(const float* normals4, const float* dem, int64_t n, float cmin, float cmax,
                               float zmin, float zmax, uint8_t* mask, hipStream_t s) {
    hipLaunchKernelGGL(k_release_mask, dim3(stream_blocks(n)), dim3(kStreamThreads), 0, s,
                       reinterpret_cast<const float4*>(normals4), dem, n, cmin, cmax, zmin, zmax, mask);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ snow cover
// alpha = ramp(z; snow line, + alt blend) * ramp(nz; cos max slope, cos(max slope - slope blend)), a ramp
// being (v - lo) / (hi - lo) clamped to [0, 1] (NaN -> 0), or the step v >= lo when hi <= lo.
__device__ __forceinline__ float snow_ramp(float v, float lo, float hi, bool step) {
    if (step) return v >= lo ? 1.0f : 0.0f;
    const float t = (v - lo) / (hi - lo);
    return t > 0.0f ? (t < 1.0f ? t : 1.0f) : 0.0f;
}

__global__ __launch_bounds__(kStreamThreads) void k_snow_cover(const float4* __restrict__ nrm, const float* __restrict__ dem,
                                                               int64_t n, float z_lo, float z_hi, float c_lo, float c_hi,
                                                               float* __restrict__ alpha) {
    const bool zstep = !(z_hi > z_lo), cstep = !(c_hi > c_lo);
    const int64_t i0 = stream_base();
    float nz[kStream], z[kStream];
#pragma unroll
    for (int k = 0; k < kStream; ++k) {
        const int64_t i = i0 + k * kStreamThreads;
        nz[k] = i < n ? nrm[i].z : 0.0f;
        z[k] = i < n ? dem[i] : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < kStream; ++k) {
        const int64_t i = i0 + k * kStreamThreads;
        if (i < n) alpha[i] = snow_ramp(z[k], z_lo, z_hi, zstep) * snow_ramp(nz[k], c_lo, c_hi, cstep);
    }
}

hipError_t launch_snow_cover(const float* normals4, const float* dem, int64_t n, float z_lo, float z_hi, float c_lo,
                             float c_hi, float* alpha, hipStream_t s) {
    hipLaunchKernelGGL(k_snow_cover, dim3(stream_blocks(n)), dim3(kStreamThreads), 0, s,
                       reinterpret_cast<const float4*>(normals4), dem, n, z_lo, z_hi, c_lo, c_hi, alpha);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ fine release map
// Release texture with mult x mult texels per DEM cell: texel (R, C) is centred at ((C + 1/2) / mult,
// (R + 1/2) / mult) in DEM cell units, where nz and the height are filtered bilinearly between texel centres
// with clamped indices and tested against the same bounds as the plain map. A block covers kFineSpan
// consecutive texels of one row (row and span from the block index, once per block). The block first
// stages nz and the height of the two DEM rows and the column range its texels touch in LDS (coalesced
// reads; the column range is exact because the texel centres and their floors grow with C), then each
// thread filters four texels from LDS and stores their four bytes at once.
constexpr int kFineThreads = 256;
constexpr int kFineSpan = 4 * kFineThreads;
constexpr int kFineCols = kFineSpan + 3;  // columns a span can touch at mult = 1 (kFineSpan + 1), with margin

__device__ __forceinline__ int fine_col(int64_t C, float fm) {  // floor(x - 1/2) of texel column C's centre
    const float x = ((float)C + 0.5f) / fm;
    return (int)floorf(x - 0.5f);
}

__global__ __launch_bounds__(kFineThreads) void k_release_mask_fine(const float4* __restrict__ nrm,
                                                                    const float* __restrict__ dem, int H, int W,
                                                                    int mult, uint32_t spans_per_row, float cmin,
                                                                    float cmax, float zmin, float zmax,
                                                                    uint8_t* __restrict__ mask) {
    __shared__ float s_n[2][kFineCols], s_z[2][kFineCols];
    const uint32_t rr = blockIdx.x / spans_per_row;  // uniform
    const uint32_t span = blockIdx.x - rr * spans_per_row;
    const int64_t Wf = (int64_t)W * mult;
    const int64_t cs0 = (int64_t)span * kFineSpan;
    const int64_t cs1 = min(cs0 + kFineSpan, Wf) - 1;  // last texel column of the span
    const float fm = (float)mult;
    const int lo = min(max(fine_col(cs0, fm), 0), W - 1);
    const int hi = min(max(fine_col(cs1, fm) + 1, 0), W - 1);
    const float y = ((float)rr + 0.5f) / fm;
    const float sy = y - 0.5f;
    const float fr = floorf(sy);
    const float fy = sy - fr;
    const int r0 = (int)fr;
    const int64_t ra = (int64_t)min(max(r0, 0), H - 1) * W;
    const int64_t rb = (int64_t)min(max(r0 + 1, 0), H - 1) * W;
    for (int k = threadIdx.x; k <= hi - lo; k += kFineThreads) {
        s_n[0][k] = nrm[ra + lo + k].z;
        s_n[1][k] = nrm[rb + lo + k].z;
        s_z[0][k] = dem[ra + lo + k];
        s_z[1][k] = dem[rb + lo + k];
    }
    __syncthreads();
    const int64_t c0 = cs0 + 4 * threadIdx.x;
    if (c0 >= Wf) return;
    uint32_t packed = 0;
    const int nk = (int)min((int64_t)4, Wf - c0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (k < nk) {
            const float x = ((float)(c0 + k) + 0.5f) / fm;
            const float sx = x - 0.5f;
            const float fc = floorf(sx);
            const float fx = sx - fc;
            const int cc = (int)fc;
            const int ca = min(max(cc, 0), W - 1) - lo, cb = min(max(cc + 1, 0), W - 1) - lo;
            const float n00 = s_n[0][ca], n01 = s_n[0][cb], n10 = s_n[1][ca], n11 = s_n[1][cb];
            const float ntop = n00 + fx * (n01 - n00), nbot = n10 + fx * (n11 - n10);
            const float nz = ntop + fy * (nbot - ntop);
            const float z00 = s_z[0][ca], z01 = s_z[0][cb], z10 = s_z[1][ca], z11 = s_z[1][cb];
            const float ztop = z00 + fx * (z01 - z00), zbot = z10 + fx * (z11 - z10);
            const float z = ztop + fy * (zbot - ztop);
            const uint32_t m = (cmin <= nz && nz <= cmax && zmin <= z && z <= zmax) ? 1u : 0u;
            packed |= m << (8 * k);
        }
    }
    uint8_t* out = mask + (int64_t)rr * Wf + c0;
    if (nk == 4 && (reinterpret_cast<uintptr_t>(out) & 3) == 0) {
        *reinterpret_cast<uint32_t*>(out) = packed;
    } else {
        for (int k = 0; k < nk; ++k) out[k] = (uint8_t)(packed >> (8 * k));
    }
}

hipError_t launch_release_mask_fine(const float* normals4, const float* dem, int H, int W, int mult, float cmin,
                                    float cmax, float zmin, float zmax, uint8_t* mask, hipStream_t s) {
    const int64_t Wf = (int64_t)W * mult, Hf = (int64_t)H * mult;
    const int64_t spans = (Wf + kFineSpan - 1) / kFineSpan;
    const int64_t blocks = spans * Hf;  // < 2^31 / 1024 * 2 + Hf: fits a 32-bit grid
    hipLaunchKernelGGL(k_release_mask_fine, dim3((unsigned)blocks), dim3(kFineThreads), 0, s,
                       reinterpret_cast<const float4*>(normals4), dem, H, W, mult, (uint32_t)spans, cmin, cmax, zmin,
                       zmax, mask);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ raster helpers
// v^2 bits -> speed, in place: vmax = sqrt(max v^2). Bound by HBM; texels no particle visited (most of a large region)
// are read and not written back.
__global__ __launch_bounds__(256) void k_finalize_vmax(uint32_t* __restrict__ bits, int64_t n) {
    const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i0 + 4 <= n && (reinterpret_cast<uintptr_t>(bits + i0) & 15) == 0) {
        uint4 b = *reinterpret_cast<uint4*>(bits + i0);
        if ((b.x | b.y | b.z | b.w) == 0u) return;  // no particle came here: its zeros are the speeds already
        b.x = __float_as_uint(sqrtf(__uint_as_float(b.x)));
        b.y = __float_as_uint(sqrtf(__uint_as_float(b.y)));
        b.z = __float_as_uint(sqrtf(__uint_as_float(b.z)));
        b.w = __float_as_uint(sqrtf(__uint_as_float(b.w)));
        *reinterpret_cast<uint4*>(bits + i0) = b;
    } else {
        for (int64_t i = i0; i < n && i < i0 + 4; ++i) bits[i] = __float_as_uint(sqrtf(__uint_as_float(bits[i])));
    }
}

static unsigned blocks_for(int64_t items, int per_thread) {
    const int64_t threads = (items + per_thread - 1) / per_thread;
    return (unsigned)((threads + 255) / 256);
}

// ------------------------------------------------------------------------------------------ mipmap

// Up to kMipPass levels of the overlay mipmap in one pass, bound by HBM. A wave's lane takes 4 x 4 cells of the input (four
// 16-byte loads of each raster, 1 KiB contiguous per wave and row), which makes 2 x 2 cells of the first output level and
// one of the second in registers; a block's 64 x 16 second-level cells are reduced further in LDS. Each level halves the
// previous one rounding up, so the children of a cell never leave the block's cells. Counts add in 64 bits; speeds (>= 0)
// take the maximum; cells past a level's edge count as empty. (2 x 2 cells a lane by 4-byte loads, 64 input columns a
// block: 8192 x 8191 in 195 us, now 174; a copy of its 790 MB takes 151.)
constexpr int kMipCols = 64, kMipRows = 16;  // second-level cells of a block
template <typename T>
struct Vec4 {
    typedef T type __attribute__((ext_vector_type(4), aligned(sizeof(T))));
};
template <typename T>
struct Vec2 {
    typedef T type __attribute__((ext_vector_type(2), aligned(sizeof(T))));
};

template <typename Tin>
__global__ __launch_bounds__(256) void k_mip(const Tin* __restrict__ cin, const float* __restrict__ vin, int h0, int w0,
                                             int nlev, MipLevels o) {
    __shared__ unsigned long long sc[kMipRows * kMipCols];
    __shared__ float sv[kMipRows * kMipCols];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    const int cu = blockIdx.x * kMipCols + lane;
    const int64_t c0 = 4 * (int64_t)cu;
#pragma unroll
    for (int k = 0; k < kMipRows / 4; ++k) {
        const int lr = wid + 4 * k;
        const int ru = blockIdx.y * kMipRows + lr;
        const int64_t r0 = 4 * (int64_t)ru;
        unsigned long long s1[2][2] = {{0, 0}, {0, 0}};
        float m1[2][2] = {{0.0f, 0.0f}, {0.0f, 0.0f}};
        if (r0 + 4 <= h0 && c0 + 4 <= w0) {
            typename Vec4<Tin>::type c[4];
            typename Vec4<float>::type v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = *reinterpret_cast<const typename Vec4<Tin>::type*>(cin + (r0 + q) * w0 + c0);
                v[q] = *reinterpret_cast<const typename Vec4<float>::type*>(vin + (r0 + q) * w0 + c0);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    s1[q / 2][p / 2] += (unsigned long long)c[q][p];
                    m1[q / 2][p / 2] = fmaxf(m1[q / 2][p / 2], v[q][p]);
                }
        } else {
            for (int q = 0; q < 4; ++q)
                for (int p = 0; p < 4; ++p)
                    if (r0 + q < h0 && c0 + p < w0) {
                        s1[q / 2][p / 2] += (unsigned long long)cin[(r0 + q) * w0 + c0 + p];
                        m1[q / 2][p / 2] = fmaxf(m1[q / 2][p / 2], vin[(r0 + q) * w0 + c0 + p]);
                    }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int64_t r = 2 * (int64_t)ru + q, c = 2 * (int64_t)cu, at = r * o.w[0] + c;
            if (r < o.h[0] && c + 1 < o.w[0]) {
                *reinterpret_cast<typename Vec2<unsigned long long>::type*>(o.c[0] + at) = {s1[q][0], s1[q][1]};
                *reinterpret_cast<typename Vec2<float>::type*>(o.v[0] + at) = {m1[q][0], m1[q][1]};
            } else if (r < o.h[0] && c < o.w[0]) {
                o.c[0][at] = s1[q][0];
                o.v[0][at] = m1[q][0];
            }
        }
        const unsigned long long s2 = (s1[0][0] + s1[0][1]) + (s1[1][0] + s1[1][1]);
        const float m2 = fmaxf(fmaxf(m1[0][0], m1[0][1]), fmaxf(m1[1][0], m1[1][1]));
        if (nlev > 1 && ru < o.h[1] && cu < o.w[1]) {
            o.c[1][(int64_t)ru * o.w[1] + cu] = s2;
            o.v[1][(int64_t)ru * o.w[1] + cu] = m2;
        }
        sc[lr * kMipCols + lane] = s2;
        sv[lr * kMipCols + lane] = m2;
    }
    int cols = kMipCols, rows = kMipRows;
    for (int l = 2; l < nlev; ++l) {
        __syncthreads();
        const int c2 = cols / 2, r2 = rows / 2;
        const int t = threadIdx.x;
        const bool mine = t < c2 * r2;
        const int i = t / c2, j = t - i * c2;
        unsigned long long sum = 0;
        float mx = 0.0f;
        if (mine) {
#pragma unroll
            for (int dr = 0; dr < 2; ++dr)
#pragma unroll
                for (int dc = 0; dc < 2; ++dc) {
                    sum += sc[(2 * i + dr) * cols + 2 * j + dc];
                    mx = fmaxf(mx, sv[(2 * i + dr) * cols + 2 * j + dc]);
                }
        }
        __syncthreads();
        if (mine) {
            sc[i * c2 + j] = sum;
            sv[i * c2 + j] = mx;
            const int r = blockIdx.y * r2 + i, c = blockIdx.x * c2 + j;
            if (r < o.h[l] && c < o.w[l]) {
                o.c[l][(size_t)r * o.w[l] + c] = sum;
                o.v[l][(size_t)r * o.w[l] + c] = mx;
            }
        }
        cols = c2;
        rows = r2;
    }
}
static_assert(kMipPass == 6 && kMipRows >> 4 == 1, "level 6 of a block is one row of cells");

hipError_t launch_mip_pass(const void* cin, bool cin64, const float* vin, int h0, int w0, int nlev,
                           const MipLevels& o, hipStream_t s) {
    const dim3 grid((unsigned)(((int64_t)w0 + 4 * kMipCols - 1) / (4 * kMipCols)),
                    (unsigned)(((int64_t)h0 + 4 * kMipRows - 1) / (4 * kMipRows)));
    if (cin64)
        hipLaunchKernelGGL(k_mip<unsigned long long>, grid, dim3(256), 0, s,
                           static_cast<const unsigned long long*>(cin), vin, h0, w0, nlev, o);
    else
        hipLaunchKernelGGL(k_mip<uint32_t>, grid, dim3(256), 0, s, static_cast<const uint32_t*>(cin), vin, h0, w0,
                           nlev, o);
    return hipGetLastError();
}

hipError_t launch_finalize_vmax(uint32_t* vmax_bits, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_finalize_vmax, dim3(blocks_for(n, 4)), dim3(256), 0, s, vmax_bits, n);
    return hipGetLastError();
}

}  // namespace avl

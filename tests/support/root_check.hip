// Exhaustive check of the particle step's short square roots and quotients by a root against the compiler's correctly
// rounded ones, over every binary32 number of their range: prints the mismatches of each.
#include <cstdio>

#include "../../paper_2506_23364_amd/csrc/particle.h"

using namespace avl::dev;

__global__ void k_check(unsigned lo, unsigned hi, float q, unsigned long long* bad) {
    unsigned long long n[3] = {0, 0, 0};
    for (unsigned long long i = lo + blockIdx.x * (unsigned long long)blockDim.x + threadIdx.x; i < hi;
         i += (unsigned long long)gridDim.x * blockDim.x) {
        const float x = __uint_as_float((unsigned)i);
        const RootEst e = sqrt_est(x);
        const float s = sqrtf(x);
        n[0] += e.s != s;
        n[1] += recip_root(e) != 1.0f / s;
        n[2] += div_root(q, e) != q / s;
    }
    for (int j = 0; j < 3; ++j)
        if (n[j]) atomicAdd(bad + j, n[j]);
}

static int run(unsigned lo, unsigned hi, float q, unsigned long long* dev) {
    unsigned long long h[3] = {0, 0, 0};
    if (hipMemcpy(dev, h, sizeof h, hipMemcpyHostToDevice) != hipSuccess) return 1;
    hipLaunchKernelGGL(k_check, dim3(4096), dim3(256), 0, nullptr, lo, hi, q, dev);
    if (hipDeviceSynchronize() != hipSuccess) return 1;
    if (hipMemcpy(h, dev, sizeof h, hipMemcpyDeviceToHost) != hipSuccess) return 1;
    std::printf("%08x %08x %a %llu %llu %llu\n", lo, hi, q, h[0], h[1], h[2]);
    return 0;
}

int main() {
    unsigned long long* dev = nullptr;
    if (hipMalloc(&dev, 3 * sizeof(unsigned long long)) != hipSuccess) return 1;
    // roots and reciprocal roots: [2^-96, max]
    if (run(0x0F800000u, 0x7F800000u, 1.0f, dev)) return 1;
    // quotients: [2^-80, 2^80] by 1 - persistence, powers of two and the type's neighbours of one among them
    const float q[] = {1.0f - 0.9f, 0.0f, 1.0f, 0.5f, 0x1p-24f, 0x1.fffffep-1f, 1.0f - 0.95f, 0.3f, 0x1.000002p-5f, 0x1.87e6b8p-1f};
    for (float v : q)
        if (run(0x17800000u, 0x67800001u, v, dev)) return 1;
    return hipFree(dev) == hipSuccess ? 0 : 1;
}

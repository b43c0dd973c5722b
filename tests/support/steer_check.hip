// The step's direction against the plain formula, bit for bit, for waves whose lanes lie in and out of the short form's range:
// prints per pattern of the wave's odd lane whether the wave may keep the short form, and the mismatches.
#include <cstdio>

#include "../../paper_2506_23364_amd/csrc/particle.h"

using namespace avl::dev;

// lane 17 of each wave has the gradient (g, 0) and the direction (d, 0), the others ordinary ones
__global__ void k_check(float g, float d, float per, float rnd, unsigned* out) {
    const unsigned i = blockIdx.x * blockDim.x + threadIdx.x, lane = threadIdx.x & 63u;
    const float gx = lane == 17u ? g : 0.3f + 1e-4f * (float)i, gy = lane == 17u ? 0.0f : -0.2f + 1e-5f * (float)i;
    const float rx = lane == 17u ? 0.0f : 0.7f - 1e-4f * (float)i, ry = lane == 17u ? 0.0f : 1e-4f * (float)i - 0.4f;
    float dx = lane == 17u ? d : 0.6f, dy = lane == 17u ? 0.0f : -0.8f;
    const float Q = 1.0f - per;
    const float gg = gx * gx + gy * gy;
    const float t = gg > 0.0f ? Q / sqrtf(gg) : 0.0f;
    const float wx = (per * dx - t * gx) + rnd * rx, wy = (per * dy - t * gy) + rnd * ry;
    const float ww = wx * wx + wy * wy;
    float ex = dx, ey = dy;
    if (ww > 0.0f) {
        const float inv = 1.0f / sqrtf(ww);
        ex = wx * inv;
        ey = wy * inv;
    }
    const bool keeps = all_mid_range_or_unused(gg);
    steer(dx, dy, gx, gy, per, Q, rnd, rx, ry);
    const bool nan = (ex != ex && dx != dx) || (ey != ey && dy != dy);
    const bool same = nan || (__float_as_uint(ex) == __float_as_uint(dx) && __float_as_uint(ey) == __float_as_uint(dy));
    if (!same) atomicAdd(out, 1u);
    if (i == 0) out[1] = keeps ? 1u : 0u;
}

int main() {
    unsigned* dev = nullptr;
    if (hipMalloc(&dev, 2 * sizeof(unsigned)) != hipSuccess) return 1;
    const float inf = __builtin_inff(), nan = __builtin_nanf("");
    const float gs[] = {0.0f, -0.0f, 0.5f, 0x1p-39f, 0x1p39f, 0x1p-41f, 0x1p41f, 0x1p-60f, 0x1p-74f, 1e-38f, 1e25f, inf, nan};
    const float ds[] = {0.0f, 1.0f}, pers[] = {0.0f, 0.9f, 1.0f}, rnds[] = {0.0f, 0.16f};
    for (float g : gs)
        for (float d : ds)
            for (float per : pers)
                for (float rnd : rnds) {
                    unsigned h[2] = {0, 0};
                    if (hipMemcpy(dev, h, sizeof h, hipMemcpyHostToDevice) != hipSuccess) return 1;
                    hipLaunchKernelGGL(k_check, dim3(8), dim3(256), 0, nullptr, g, d, per, rnd, dev);
                    if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(h, dev, sizeof h, hipMemcpyDeviceToHost) != hipSuccess)
                        return 1;
                    std::printf("%a %u %u\n", g, h[1], h[0]);
                }
    return hipFree(dev) == hipSuccess ? 0 : 1;
}

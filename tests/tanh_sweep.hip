// tanh_sweep.hip -- every float of a range through the forward pass's tanh
// (csrc/net_tanh.h) beside tanhf, for tests/test_gpu_tanh.py.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../paper_2605_07083_amd/csrc/net_tanh.h"

namespace {

struct Counts {
    unsigned long long closed, closed_wrong, settled_wrong, a_wrong;   // a_wrong: bits of one of them
};

__device__ bool differs(uint32_t got, uint32_t want)
{
    const bool nan = (got & 0x7FFFu) > 0x7F80u && (want & 0x7FFFu) > 0x7F80u;
    return got != want && !nan;
}

// Four consecutive floats per thread and round; every lane of a wave stays in
// the loop for as long as one of them has work.
__global__ __launch_bounds__(256) void k_sweep(uint32_t first, unsigned long long groups, Counts *out)
{
    unsigned long long closed = 0, closed_wrong = 0, settled_wrong = 0;
    const unsigned long long stride = (unsigned long long)gridDim.x * 256u;
    const unsigned long long rounds = (groups + stride - 1) / stride;
    for (unsigned long long r = 0; r < rounds; ++r) {
        const unsigned long long g = r * stride + blockIdx.x * 256u + threadIdx.x;
        const bool live = g < groups;
        const uint32_t bits = first + (uint32_t)((live ? g : 0ull) * 4ull);
        sur::f32x4 x;
        for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(bits + (uint32_t)i);
        uint2 open, h = sur::tanh4(x, open);
        const uint2 before = h;
        sur::tanh4_settle(x, open, h);
        for (int i = 0; i < 4; ++i) {
            const uint32_t want = sur::pack_bf16(tanhf(x[i]), 0.0f) & 0xFFFFu;
            const int shift = 16 * (i & 1);
            const uint32_t o = (i < 2 ? open.x : open.y) >> shift & 0xFFFFu;
            const uint32_t b = (i < 2 ? before.x : before.y) >> shift & 0xFFFFu;
            const uint32_t s = (i < 2 ? h.x : h.y) >> shift & 0xFFFFu;
            if (!live) continue;
            if (o == 0u) {
                ++closed;
                if (differs(b, want)) {
                    ++closed_wrong;
                    out->a_wrong = bits + (uint32_t)i;
                }
            }
            if (differs(s, want)) ++settled_wrong;
        }
    }
    atomicAdd(&out->closed, closed);
    atomicAdd(&out->closed_wrong, closed_wrong);
    atomicAdd(&out->settled_wrong, settled_wrong);
}

}  // namespace

// The floats of bits first .. first + 4 groups - 1; counts to out[4].
extern "C" int tanh_sweep(uint32_t first, unsigned long long groups, unsigned long long *out)
{
    if (!out || groups < 1 || groups > (1ull << 30) || first % 4u) return -1;
    Counts *dev = nullptr, host{};
    if (hipMalloc(reinterpret_cast<void **>(&dev), sizeof(Counts)) != hipSuccess) return -2;
    int rc = 0;
    if (hipMemcpy(dev, &host, sizeof(host), hipMemcpyHostToDevice) != hipSuccess) rc = -3;
    if (!rc) {
        hipLaunchKernelGGL(k_sweep, dim3(4096), dim3(256), 0, 0, first, groups, dev);
        if (hipGetLastError() != hipSuccess || hipMemcpy(&host, dev, sizeof(host), hipMemcpyDeviceToHost) != hipSuccess)
            rc = -4;
    }
    (void)hipFree(dev);
    out[0] = host.closed;
    out[1] = host.closed_wrong;
    out[2] = host.settled_wrong;
    out[3] = host.a_wrong;
    return rc;
}

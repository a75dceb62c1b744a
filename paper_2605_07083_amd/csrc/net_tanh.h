// net_tanh.h -- the forward pass's activation: tanh rounded to bfloat16, as a
// 35-instruction tanhf would round it, in a third of its time.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sur {

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    const bf16x2 r = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, r);
}

// bf16(tanhf(x)) of four values.  tanh x = 1 - 2 / (1 + e^2x) from the
// hardware's exp2 and reciprocal is off by a few 1e-7 in absolute terms; the
// two ends of that error interval almost always round to the same bfloat16,
// which then is the one tanhf's result rounds to (tests/test_gpu_tanh.py: every
// float x).  Where they differ, for one value in some thousands, tanhf itself
// decides.  About 13 instructions' time per value instead of tanhf's 35.
//
// The value, and what is open: nonzero bits of `open` where the ends differ.
__device__ __forceinline__ uint2 tanh4(f32x4 x, uint2 &open)
{
    constexpr float MARGIN = 1.2e-7f;
    float lo[4], hi[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float t = __builtin_amdgcn_exp2f(x[i] * 2.8853900817779268f);   // 2 / ln 2
        const float r = __builtin_amdgcn_rcpf(t + 1.0f);
        lo[i] = __builtin_fmaf(-2.0f * (1.0f + MARGIN), r, 1.0f - MARGIN);
        hi[i] = __builtin_fmaf(-2.0f * (1.0f - MARGIN), r, 1.0f + MARGIN);
    }
    const uint2 a = make_uint2(pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]));
    open = make_uint2(a.x ^ pack_bf16(hi[0], hi[1]), a.y ^ pack_bf16(hi[2], hi[3]));
    return a;
}

// tanhf where it is open in some lane (a lane whose ends agree gets the same
// bits from it).
__device__ __forceinline__ void tanh4_settle(f32x4 x, uint2 open, uint2 &h)
{
    if (__any(open.x)) h.x = pack_bf16(tanhf(x[0]), tanhf(x[1]));
    if (__any(open.y)) h.y = pack_bf16(tanhf(x[2]), tanhf(x[3]));
}

}  // namespace sur

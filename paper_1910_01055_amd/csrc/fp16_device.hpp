// What the half-precision kernels share.
#pragma once
#include "common.hpp"

namespace aq {

// tanh of a value about to be rounded to binary16, relative error below 1e-6 (far inside half a binary16 spacing,
// 2.4e-4): odd polynomial near zero, where the exponential form would cancel, 1 - 2 / (e^{2|x|} + 1) elsewhere
__device__ __forceinline__ float tanh_rel(float x) {
    const float ax = fabsf(x);
    const float u = x * x;
    float p = 0.0035921280f;         // Taylor series of tanh(x) / x in u = x^2 up to u^6
    p = fmaf(p, u, -0.0088632355f);  // (remainder below 2e-7 relative at |x| = 0.5)
    p = fmaf(p, u, 0.0218694885f);
    p = fmaf(p, u, -0.0539682540f);
    p = fmaf(p, u, 0.1333333333f);
    p = fmaf(p, u, -0.3333333333f);
    const float small = fmaf(x * u, p, x);
    const float e = __builtin_amdgcn_exp2f(fminf(ax, 20.0f) * 2.885390081777927f);  // e^{2|x|}
    const float big = copysignf(fmaf(__builtin_amdgcn_rcpf(e + 1.0f), -2.0f, 1.0f), x);
    return ax < 0.5f ? small : big;
}

}  // namespace aq

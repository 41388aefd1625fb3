// fp32 products on the bf16 matrix cores: a value as the exact sum of three bf16 parts (see fp32_conv_stack.hip), and what the
// fp32 kernels share.
#pragma once
#include "int8_device.hpp"

namespace aq {

namespace {
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f_u __attribute__((ext_vector_type(4), aligned(4)));  // rows of floats start at any 4-byte address
typedef uint32_t u32_u __attribute__((aligned(1)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

// ---- min / max of a tensor through order-preserving unsigned keys
__device__ __forceinline__ uint32_t f2key(float f) {
    uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key2f(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
// A wave's (lo, hi) joins slot `who` of a tensor's kRangeSlots.  (With one pair of words per tensor every wave of the
// chip queued at the same address: 90 us per tensor of a frame policy's calibration.)  All lanes of the wave call it.
__device__ __forceinline__ void range_note(RangeSlot* __restrict__ slots, uint32_t who, float lo, float hi) {
    lo = wave_min(lo);
    hi = wave_max(hi);
    if ((threadIdx.x & 63) == 0 && lo <= hi) {
        RangeSlot* s = slots + who % kRangeSlots;
        atomicMax(&s->not_lo, ~f2key(lo));
        atomicMax(&s->hi, f2key(hi));
    }
}

// the wave's minimum and maximum (in the lanes of every row of 16 without a trip through LDS)
__device__ __forceinline__ void wave_range(float& lo, float& hi) {
    auto step = [&](auto ctrl_c) __attribute__((always_inline)) {
        constexpr int ctrl = decltype(ctrl_c)::value;
        lo = fminf(lo, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(lo), ctrl, 15, 15, true)));
        hi = fmaxf(hi, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(hi), ctrl, 15, 15, true)));
    };
    step(std::integral_constant<int, 0xB1>{});   // quad_perm: lane ^ 1
    step(std::integral_constant<int, 0x4E>{});   // lane ^ 2
    step(std::integral_constant<int, 0x141>{});  // row_half_mirror
    step(std::integral_constant<int, 0x140>{});  // row_mirror
#pragma unroll
    for (int o = 16; o <= 32; o *= 2) {
        lo = fminf(lo, __shfl_xor(lo, o, 64));
        hi = fmaxf(hi, __shfl_xor(hi, o, 64));
    }
}
// not finite, or rounding to bf16 would make it so, or so small that its last part would be a denormal cut short: bits of the
// magnitude below kSplitLeast (2^-100) and not zero, or from kSplitMost on
constexpr uint32_t kSplitLeast = 0x0D800000u, kSplitMost = 0x7F7F8000u;
__device__ __forceinline__ bool split_special(float v) {
    const uint32_t u = __float_as_uint(v) & 0x7fffffffu;
    return u != 0 && u - kSplitLeast >= kSplitMost - kSplitLeast;
}
// two values into the words of their three parts: each the rest of the one before, rounded to bf16 (the rests are exact in fp32)
__device__ __forceinline__ uint32_t pack_bf16(float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{x, y}), bf2)); }
__device__ __forceinline__ void split2(float x, float y, int& a, int& b, int& c) {
    const uint32_t p = pack_bf16(x, y);
    x -= __uint_as_float(p << 16);
    y -= __uint_as_float(p & 0xffff0000u);
    const uint32_t q = pack_bf16(x, y);
    x -= __uint_as_float(q << 16);
    y -= __uint_as_float(q & 0xffff0000u);
    a = (int)p;
    b = (int)q;
    c = (int)pack_bf16(x, y);
}
__device__ __forceinline__ void split8(const v4f& lo, const v4f& hi, bf8 (&x)[3]) {
    v4i p[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const v4f& v = i < 2 ? lo : hi;
        int a, b, c;
        split2(v[2 * (i & 1)], v[2 * (i & 1) + 1], a, b, c);
        p[0][i] = a;
        p[1][i] = b;
        p[2][i] = c;
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) x[q] = __builtin_bit_cast(bf8, p[q]);
}
__device__ __forceinline__ v4f mfma_bf16(const bf8& a, const bf8& b, const v4f& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// 32 k of FT feature tiles by one row tile, the smallest terms first; the tiles alternate, so that an MFMA does not wait for
// the one before it
template <int FT>
__device__ __forceinline__ void mfma_split(const bf8 (&w)[FT][3], const bf8 (&x)[3], v4f (&c)[FT]) {
    constexpr int wi[6] = {2, 0, 1, 1, 0, 0}, xi[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int f = 0; f < FT; ++f) c[f] = mfma_bf16(w[f][wi[t]], x[xi[t]], c[f]);
}
// the same on the fp32 instructions: lane group g holds k = 8 g + j of both operands for MFMA j
__device__ __forceinline__ v4f mfma_whole(const v4f& wl, const v4f& wh, const v4f& xl, const v4f& xh, v4f c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_16x16x4f32(wl[j], xl[j], c, 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_16x16x4f32(wh[j], xh[j], c, 0, 0, 0);
    return c;
}
}  // namespace

}  // namespace aq

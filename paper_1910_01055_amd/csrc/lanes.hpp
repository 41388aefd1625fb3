// Values that are the same for a whole wavefront, and exchanges among its four rows of 16 lanes.
#pragma once
#include "common.hpp"

namespace aq {

// readfirstlane keeps a value scalar wherever the compiler cannot prove it uniform, so that loop bounds and branches stay scalar
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float unif(float v) { return __int_as_float(uni(__float_as_int(v))); }
template <class T>
__device__ __forceinline__ T* uni_ptr(T* p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T*)(((uint64_t)hi << 32) | lo);
}

// lane N of every 16-lane row, broadcast to that row (the old value is left undefined, as the broadcast writes
// every lane): no move that clears the destination first.
template <int N>
__device__ __forceinline__ int row_bcast(int v) {
    return __builtin_amdgcn_mov_dpp(v, 0x150 + N, 0xF, 0xF, true);
}
// ... through an instruction of its own, so that no consumer folds it: folded into v_ashrrev_i32_dpp the broadcast is
// applied to the shifted value instead of the amount (additions and plain moves are right).
template <int N>
__device__ __forceinline__ int row_bcast_mov(int v) {
    int r = row_bcast<N>(v);
    asm volatile("" : "+v"(r));
    return r;
}

// sum over the four 16-lane rows of a wavefront (lane ^ 16, then lane ^ 32), the same value in every lane
__device__ __forceinline__ float sum_rows4(float s) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    s = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}
__device__ __forceinline__ int sum_rows4(int s) {
    const auto p = __builtin_amdgcn_permlane16_swap((uint32_t)s, (uint32_t)s, false, false);
    s = (int)(p[0] + p[1]);
    const auto q = __builtin_amdgcn_permlane32_swap((uint32_t)s, (uint32_t)s, false, false);
    return (int)(q[0] + q[1]);
}

}  // namespace aq

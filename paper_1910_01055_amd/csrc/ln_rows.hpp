// LayerNorm over rows that lie in memory (layers that run on their own), shared by the three precisions.
#pragma once
#include <type_traits>

#include "kernels.hpp"

namespace aq {

// W wavefronts of a workgroup of four hold one row in registers, P pieces of four values a thread: all of the row is requested at
// once, and the gains and offsets with it, where one wavefront that walked the row three times, 64 values at a time, paid a round
// trip for each (8 bits, 2048 values, 16 rows: 24 us).  Piece i of thread t holds values 4 (t + T i) ... (VEC; rows of whole,
// aligned pieces) or t + T (4 i + j) (any other), T = 64 W threads to a row; values past the row are zeros.
template <int W, int P>
struct LnRow {
    static constexpr int T = 64 * W;
    static constexpr int kMost = 4 * P * T;  // the longest row
    float v[P][4];

    template <bool VEC>
    static __device__ __forceinline__ int at(int t, int i, int j) {
        return VEC ? 4 * (t + T * i) + j : t + T * (4 * i + j);
    }
    // sum over the row's threads; `red` has a word for each of the workgroup's wavefronts
    static __device__ __forceinline__ float row_sum(float s, float* red) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (W == 1) return s;
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        return (red[0] + red[1]) + (red[2] + red[3]);
    }
    // mean and 1 / sqrt(biased variance + eps) of the row's N values
    template <bool VEC>
    __device__ __forceinline__ void stats(int t, int N, float eps, float (&red)[2][4], float& mean, float& inv) const {
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < P; ++i) s += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
        mean = row_sum(s, red[0]) / (float)N;
        float ss = 0.0f;
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float d = at<VEC>(t, i, j) < N ? v[i][j] - mean : 0.0f;
                ss += d * d;
            }
        inv = 1.0f / sqrtf(row_sum(ss, red[1]) / (float)N + eps);
    }
    // four fp32 values of piece i (zeros past the row; `fill` where there is no array)
    template <bool VEC>
    static __device__ __forceinline__ void load(const float* __restrict__ x, int t, int i, int N, float fill, float (&o)[4]) {
        if (VEC) {
            const int n = at<true>(t, i, 0);
            float4 q = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (x) {
                if (n < N) q = *(const float4*)(x + n);
            } else {
                q = make_float4(fill, fill, fill, fill);
            }
            o[0] = q.x;
            o[1] = q.y;
            o[2] = q.z;
            o[3] = q.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = at<false>(t, i, j);
                o[j] = x ? (n < N ? x[n] : 0.0f) : fill;
            }
        }
    }
};

// Which form a launch takes: four wavefronts to a row where a row is longer than 1024 or where one each would leave most of the
// chip's 1024 SIMDs without one, and the fewest pieces.  False: the row is longer than any holds, or a workgroup for each would be more
// threads than a launch holds.
struct LnForm {
    int w, p;
};
inline bool ln_form(int64_t rows, int N, LnForm* f) {
    f->w = N > 1024 || rows < 1024 ? 4 : 1;
    const int per = (N + 256 * f->w - 1) / (256 * f->w);
    f->p = per <= 1 ? 1 : per <= 2 ? 2 : 4;
    return per <= 4 && (f->w == 1 || grid_ok(rows, 256));
}
// calls go(W, P) as constants
template <class Go>
inline void ln_dispatch(const LnForm& f, Go&& go) {
    auto p = [&](auto w) {
        if (f.p == 1) go(w, std::integral_constant<int, 1>());
        else if (f.p == 2) go(w, std::integral_constant<int, 2>());
        else go(w, std::integral_constant<int, 4>());
    };
    if (f.w == 1) p(std::integral_constant<int, 1>());
    else p(std::integral_constant<int, 4>());
}

}  // namespace aq

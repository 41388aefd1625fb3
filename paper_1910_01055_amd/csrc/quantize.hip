// Quantizer block (Sec. 3.1, Sec. 3.2): fp32 weights -> 8-bit codes + scales + integer layer constants.
//
// The weight passes are HBM-bandwidth bound (4 bytes read + 1 byte written per parameter);
// they are written as coalesced float4 streams with wavefront-shuffle reductions.  A whole
// output channel is kept in registers between the range reduction and the rounding, so a
// per-channel tensor is read from HBM exactly once.
#include "kernels.hpp"

#include <float.h>

namespace aq {

// ---------------------------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t* p, int n, uint32_t v) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__device__ __forceinline__ bool finite_f(float v) { return fabsf(v) <= FLT_MAX; }
typedef float f4v __attribute__((ext_vector_type(4)));

// Sec. 3.2: delta = (|min(W,0)| + |max(W,0)|) / D ; zero-point z = round(-lo / delta).
// (n bits: D = 2^n - 1 or 2^n, codes and zero-point in [0, qmax = 2^n - 1])
__device__ __forceinline__ void asym_qparams(float hi, float nlo, float qdenom, int qmax, float& s, int& z) {
    float lo = -nlo;
    s = (hi - lo) / qdenom;
    if (hi == lo) s = 1.0f;
    z = rint_clamp(-lo / s, 0, qmax);
}

// ---------------------------------------------------------------------------------------------
// per-tensor range of a workgroup's share of a tensor: hi = max(W, 0), nlo = max(-W, 0), non-finite flag; thread 0
// publishes the three words.  Nothing has to be cleared first.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void range_partial_block(const float* __restrict__ w, int64_t n, int64_t first, int64_t stride,
                                                    uint32_t* __restrict__ part) {
    float hi = 0.0f, nlo = 0.0f;
    int bad = 0;
    auto take = [&](float e) {
        bad |= !finite_f(e);
        hi = e > hi ? e : hi;
        const float t = -e;
        nlo = t > nlo ? t : nlo;
    };
    const f4v AQ_GLOBAL* w4 = (const f4v AQ_GLOBAL*)w;
    const int64_t n4 = ((uintptr_t)w & 15) == 0 ? n / 4 : 0;
    for (int64_t i = first; i < n4; i += stride) {
        const f4v v = w4[i];
#pragma unroll
        for (int j = 0; j < 4; ++j) take(v[j]);
    }
    for (int64_t i = n4 * 4 + first; i < n; i += stride) take(((const float AQ_GLOBAL*)w)[i]);
    hi = wave_max(hi);
    nlo = wave_max(nlo);
    bad = wave_or_i32(bad);
    __shared__ float s_hi[4], s_nlo[4];
    __shared__ int s_bad[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        s_hi[wv] = hi;
        s_nlo[wv] = nlo;
        s_bad[wv] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        part[0] = __float_as_uint(fmaxf(fmaxf(s_hi[0], s_hi[1]), fmaxf(s_hi[2], s_hi[3])));
        part[1] = __float_as_uint(fmaxf(fmaxf(s_nlo[0], s_nlo[1]), fmaxf(s_nlo[2], s_nlo[3])));
        part[2] = (uint32_t)(s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3]);
    }
}

// Pass 1 of the per-tensor scheme for a large flat tensor: every workgroup publishes its partial
// range (hi bits, -lo bits, non-finite flag) in part[3 * block]; nothing has to be cleared first.
__global__ __launch_bounds__(256) void k_range_partials(const float* __restrict__ w, int64_t n, uint32_t* __restrict__ part) {
    range_partial_block(w, n, (int64_t)blockIdx.x * 256 + threadIdx.x, (int64_t)gridDim.x * 256, part + 3 * blockIdx.x);
}

// Pass 2: every workgroup folds the partials (a few KiB, cache resident), then streams its share of
// the tensor: 16 bytes in, 4 codes out per thread and iteration.  The second read of the tensor
// comes from the last-level cache for tensors that fit it.
__global__ __launch_bounds__(256) void k_quant_asym_flat(const float4* __restrict__ w4, int64_t n4,
                                                         const uint32_t* __restrict__ part, int n_part, float qdenom,
                                                         int qmax, uint32_t* __restrict__ codes, float* __restrict__ scale,
                                                         int32_t* __restrict__ zp, uint32_t* __restrict__ flag) {
    float hi = 0.0f, nlo = 0.0f;
    int bad = 0;
    for (int b = threadIdx.x; b < n_part; b += 256) {
        hi = fmaxf(hi, __uint_as_float(part[3 * b + 0]));
        nlo = fmaxf(nlo, __uint_as_float(part[3 * b + 1]));
        bad |= (int)part[3 * b + 2];
    }
    hi = wave_max(hi);
    nlo = wave_max(nlo);
    bad = wave_or_i32(bad);
    __shared__ float s_hi[4], s_nlo[4];
    __shared__ int s_bad[4];
    if ((threadIdx.x & 63) == 0) {
        s_hi[threadIdx.x >> 6] = hi;
        s_nlo[threadIdx.x >> 6] = nlo;
        s_bad[threadIdx.x >> 6] = bad;
    }
    __syncthreads();
    hi = fmaxf(fmaxf(s_hi[0], s_hi[1]), fmaxf(s_hi[2], s_hi[3]));
    nlo = fmaxf(fmaxf(s_nlo[0], s_nlo[1]), fmaxf(s_nlo[2], s_nlo[3]));
    float s;
    int z;
    asym_qparams(hi, nlo, qdenom, qmax, s, z);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        scale[0] = s;
        zp[0] = z;
        if (s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3]) flag[0] = 1u;
    }
    const QuantScale qs = make_quant_scale(s);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
        const f4v q = __builtin_nontemporal_load((const f4v*)w4 + i);  // (last use of the tensor)
        __builtin_nontemporal_store(quant_code4(make_float4(q[0], q[1], q[2], q[3]), qs, -z, qmax - z, z), codes + i);
    }
}

// per-channel symmetric codes, canonical order, short rows: G lanes per row, V float4 of it each, in registers between the |w|
// reduction and the rounding; U such sets of rows per wavefront, all requested at once, so that 32 to 64 bytes a thread are in flight
// however short the rows.  Bound by memory: 100000 x 64 (26 MB in, 6 MB out) took 24.9 us with a wavefront per row (one float4
// a thread, three quarters of the lanes idle), 8.3 so.
template <int G, int V, int U>
__global__ __launch_bounds__(256) void k_quant_sym_rows_short(const float4* __restrict__ w4, int64_t rows, int cols4, int qw,
                                                              uint32_t* __restrict__ codes, float* __restrict__ scale,
                                                              int32_t* __restrict__ zp, uint32_t* __restrict__ mm) {
    constexpr int RW = 64 / G;
    const int lane = threadIdx.x & 63, li = lane & (G - 1);
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (RW * U) + lane / G;
    f4v v[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int c = li + G * i;
            const int64_t row = row0 + u * RW;
            v[u][i] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
            if (row < rows && c < cols4) v[u][i] = __builtin_nontemporal_load((const f4v*)w4 + row * cols4 + c);
        }
    int bad = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t row = row0 + u * RW;
        float amax = 0.0f;
#pragma unroll
        for (int i = 0; i < V; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x = fabsf(v[u][i][j]);
                bad |= !(x <= FLT_MAX);
                amax = fmaxf(amax, x);
            }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
        float s = amax / (float)qw;
        if (amax == 0.0f) s = 1.0f;
        if (row >= rows) continue;
        if (li == 0) {
            scale[row] = s;
            zp[row] = 0;
        }
        const QuantScale qs = make_quant_scale(s);
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int c = li + G * i;
            if (c < cols4)
                __builtin_nontemporal_store(quant_code4(make_float4(v[u][i][0], v[u][i][1], v[u][i][2], v[u][i][3]), qs, -qw, qw, 0),
                                            codes + row * cols4 + c);
        }
    }
    if (bad) atomicOr(&mm[2], 1u);
}

// Longer rows: one workgroup per row, R float4 per thread held in registers between the |w|
// reduction and the rounding (still one pass over HBM).  Many small workgroups keep the memory
// pipeline of every CU busy while others are in their arithmetic phase.
template <int R>
__global__ __launch_bounds__(256) void k_quant_sym_row_wg(const float4* __restrict__ w4, int cols4, int qw,
                                                          uint32_t* __restrict__ codes, float* __restrict__ scale,
                                                          int32_t* __restrict__ zp, uint32_t* __restrict__ mm) {
    const int64_t row = blockIdx.x;
    const float4* src = w4 + row * cols4;
    float4 v[R];
    float amax = 0.0f;
    int bad = 0;
    // (the tensor is read once and the codes are written once: both bypass the cache hierarchy's retention)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int c = threadIdx.x + 256 * r;
        if (c < cols4) {
            const f4v q = __builtin_nontemporal_load((const f4v*)src + c);
            v[r] = make_float4(q[0], q[1], q[2], q[3]);
        } else {
            v[r] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float a0 = fabsf(v[r].x), a1 = fabsf(v[r].y), a2 = fabsf(v[r].z), a3 = fabsf(v[r].w);
        bad |= !(a0 <= FLT_MAX) | !(a1 <= FLT_MAX) | !(a2 <= FLT_MAX) | !(a3 <= FLT_MAX);
        amax = fmaxf(fmaxf(amax, fmaxf(a0, a1)), fmaxf(a2, a3));
    }
    amax = wave_max(amax);
    __shared__ float s_max[4];
    if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = amax;
    if (bad) atomicOr(&mm[2], 1u);
    __syncthreads();
    amax = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
    float s = amax / (float)qw;
    if (amax == 0.0f) s = 1.0f;
    if (threadIdx.x == 0) {
        scale[row] = s;
        zp[row] = 0;
    }
    const QuantScale qs = make_quant_scale(s);
    uint32_t* dst = codes + row * cols4;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int c = threadIdx.x + 256 * r;
        if (c < cols4) __builtin_nontemporal_store(quant_code4(v[r], qs, -qw, qw, 0), dst + c);
    }
}

// rows too long for the register-resident kernel: one workgroup per row, the row is read twice
// (the second read comes from cache for any realistic channel length).
__global__ __launch_bounds__(256) void k_quant_sym_rows_long(const float4* __restrict__ w4, int64_t rows, int cols4, int qw,
                                                             uint32_t* __restrict__ codes, float* __restrict__ scale,
                                                             int32_t* __restrict__ zp, uint32_t* __restrict__ mm) {
    const int64_t row = blockIdx.x;
    const float4* src = w4 + row * cols4;
    float amax = 0.0f;
    int bad = 0;
    for (int c = threadIdx.x; c < cols4; c += 256) {
        float4 v = src[c];
        float a0 = fabsf(v.x), a1 = fabsf(v.y), a2 = fabsf(v.z), a3 = fabsf(v.w);
        bad |= !(a0 <= FLT_MAX) | !(a1 <= FLT_MAX) | !(a2 <= FLT_MAX) | !(a3 <= FLT_MAX);
        amax = fmaxf(fmaxf(amax, fmaxf(a0, a1)), fmaxf(a2, a3));
    }
    amax = wave_max(amax);
    bad = wave_or_i32(bad);
    __shared__ float s_max[4];
    __shared__ int s_bad[4];
    if ((threadIdx.x & 63) == 0) {
        s_max[threadIdx.x >> 6] = amax;
        s_bad[threadIdx.x >> 6] = bad;
    }
    __syncthreads();
    amax = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
    bad = s_bad[0] | s_bad[1] | s_bad[2] | s_bad[3];
    float s = amax / (float)qw;
    if (amax == 0.0f) s = 1.0f;
    if (threadIdx.x == 0) {
        scale[row] = s;
        zp[row] = 0;
        if (bad) atomicOr(&mm[2], 1u);
    }
    uint32_t* dst = codes + row * cols4;
    const QuantScale qs = make_quant_scale(s);
    for (int c = threadIdx.x; c < cols4; c += 256) {
        dst[c] = quant_code4(src[c], qs, -qw, qw, 0);
    }
}

// packed signed-domain weights -> canonical codes (the inverse permutation), for export
__global__ void k_unpack_weights(const int8_t* __restrict__ wp, int N, int K, int KS, int asym,
                                 uint8_t* __restrict__ codes) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)N * K) return;
    int n = (int)(i / K), k = (int)(i % K);
    int8_t v = wp[(((int64_t)(n >> 5) * KS + (k >> 5)) * 64 + (n & 31) + 32 * ((k & 31) >> 4)) * 16 + (k & 15)];
    codes[i] = asym ? (uint8_t)((int)v + 128) : (uint8_t)v;
}

// ---------------------------------------------------------------------------------------------
// activation (scale, zero-point) from the supplied ranges: the same formula as for weights,
// the range being extended to contain zero.
// ---------------------------------------------------------------------------------------------
// What opens a quantize pass, done by one wavefront of its first launch: activation parameters, a clear status word,
// the short-form flags (1 for requantized layers; a channel that does not qualify clears its layer's flag later), and
// the caller's parameter pointers in device memory, where the row kernel reads them (a launch is 0.7 us dearer with
// them among its arguments).
__device__ __forceinline__ void open_pass(const QTab& tab, const QPtrs& p, const RangesArg& r, const QOut& o) {
    const int i = threadIdx.x;
    const int nl = tab.n_layers;
    if (i == 63) *o.status = 0;
    if (i >= 32 && i < 32 + nl) o.fast[i - 32] = tab.L[i - 32].requant;
    if (i >= nl) return;
    o.ptrs->w[i] = p.w[i];
    o.ptrs->b[i] = p.b[i];
    o.ptrs->gamma[i] = p.gamma[i];
    o.ptrs->beta[i] = p.beta[i];
    if (i == 0 && tab.in_u8) {
        o.actq[0].s = 1.0f;
        o.actq[0].z = 0;
        return;
    }
    float hi = r.hi[i] > 0.0f ? r.hi[i] : 0.0f;
    float nlo = -r.lo[i] > 0.0f ? -r.lo[i] : 0.0f;
    float s;
    int z;
    asym_qparams(hi, nlo, tab.qdenom, 255, s, z);  // activations stay at 8 bits
    o.actq[i].s = s;
    o.actq[i].z = z;
}
__global__ void k_qp_prep(const QTab* __restrict__ tab, const QPtrs p, const RangesArg r, const QOut o) {
    open_pass(*tab, p, r, o);
}

// ---------------------------------------------------------------------------------------------
// per-channel layer constants:
//   m[n]      = s_in * s_w[n]                                   (fp32)
//   bias_q[n] = round(b[n] / (s_in * s_w[n]))                   (fp64, saturated)
//   M[n]      = s_in * s_w[n] / s_out = f * 2^e, f in [0.5,1);  M0 = round(f * 2^31), r = 31 - e
//   bias_fold = bias_q + zero-point terms of the signed-domain product:
//       sum_k (a_u - z_a)(w_u - z_w) = sum_k a_s w_s - z_a' sum_k w_s - z_w' sum_k a_s + K z_a' z_w'
//   with a_s = a_u - 128, z_a' = z_a - 128, and for unsigned weight codes w_s = w_u - 128,
//   z_w' = z_w - 128 (symmetric codes: w_s = w, z_w' = 0).  The "- z_w' sum_k a_s" term depends on
//   the batch row and is applied inside the forward kernel.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void layer_consts_channel(const QLayerTab& L, int asym, ActQ in, ActQ out, float s_w, int z_w, float bias,
                                                     int rowsum, int n, int* __restrict__ fast, int* __restrict__ status) {
    const float s_in = in.s;
    const int z_a = in.z;
    L.m[n] = s_in * s_w;
    double sw = (double)s_in * (double)s_w;
    double bq = rint((double)bias / sw);
    if (!(bq >= -2147483647.0)) bq = -2147483647.0;
    if (bq > 2147483647.0) bq = 2147483647.0;
    int32_t bqi = (int32_t)bq;
    L.bias_q[n] = bqi;
    if (L.requant) {
        double M = sw / (double)out.s;
        int e;
        double f = frexp(M, &e);
        long long q = llround(f * 2147483648.0);
        if (q == 2147483648LL) {
            q = 1073741824LL;
            e += 1;
        }
        int r = 31 - e;
        if (r < 1 || r > 62 || !(M > 0.0) || !(M <= DBL_MAX)) {
            atomicOr(status, kStatRange);
            q = 0;
            r = 1;
        }
        L.M0[n] = (int32_t)q;
        L.pack1[n] = (int32_t)q;
        L.rshift[n] = r;
        // Short form of the same requantization for 33 <= r <= 54: the rounding constant 2^(r-1) has a
        // zero low word, so (acc*M0 + 2^(r-1)) >> r = (mulhi(acc, M0) + 2^(r-33)) >> (r-32), and the
        // output zero-point can ride along as z_out << (r-32).  One layer-wide flag says whether every
        // channel qualifies.
        if (r >= 33 && r <= 54) {
            L.sh[n] = r - 32;
            L.rz[n] = (1 << (r - 33)) + (out.z << (r - 32));
        } else {
            L.sh[n] = 0;
            L.rz[n] = 0;
            atomicAnd(fast, 0);
        }
    } else {
        L.M0[n] = 0;
        L.rshift[n] = 0;
        L.pack1[n] = __float_as_int(s_in * s_w);
    }
    const int za_s = z_a - 128;
    const int zw_s = asym ? z_w - 128 : 0;
    // (a saturated integer bias can push the folded value out of the accumulator's range: reported, like a
    // multiplier outside the shift range, instead of wrapping silently)
    const long long bf = (long long)bqi - (long long)za_s * rowsum + (long long)L.K * za_s * zw_s;
    if (bf > 2147483647LL || bf < -2147483648LL) atomicOr(status, kStatRange);
    L.bias_fold[n] = (int32_t)bf;
}

// ---------------------------------------------------------------------------------------------
// The whole policy in two launches: what opens the pass (with the per-tensor scheme: together with every layer's
// partial ranges), then the rows of every layer with their constants.  A grid covers all layers; a workgroup finds its
// layer from the table's first-workgroup indices (at most 8 compares).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ int layer_of_block(const QTab& t, int blk, bool rows) {
    // (entries past the last layer hold INT_MAX; all eight in one scalar load instead of a chain of them)
    int l = 0;
#pragma unroll
    for (int i = 1; i < AQ_MAX_LAYERS; ++i) l += blk >= (rows ? t.row_blk0[i] : t.rng_blk0[i]);
    return l;
}

__global__ __launch_bounds__(256) void k_qp_ranges(const QTab* __restrict__ tab, const QPtrs p, const RangesArg r, const QOut o) {
    const QTab& t = *tab;
    if (blockIdx.x == 0 && threadIdx.x < 64) open_pass(t, p, r, o);
    const int l = layer_of_block(t, blockIdx.x, false);
    const QLayerTab& L = t.L[l];
    range_partial_block(p.w[l], (int64_t)L.N * L.K, (int64_t)((int)blockIdx.x - t.rng_blk0[l]) * 256 + threadIdx.x,
                        (int64_t)L.rng_blks * 256, o.part + 3 * blockIdx.x);
}

// Policy weights: a workgroup of 8 wavefronts quantizes 8 output channels of W[N][K], one per wavefront.  Codes go,
// in the signed domain (unsigned codes minus 128; symmetric codes as they are), into the MFMA operand order the forward
// kernels read:
//   tile (nt = n / 32, ks = k / 32) is 1 KiB: lane = n % 32 + 32 * ((k % 32) / 16), byte = k % 16.
// The 8 rows' bytes of a k-half of a tile are 128 consecutive bytes: the codes are collected row by row in LDS, 2048 k at
// a time, and leave as 16-byte pieces in that order.  Rows of up to 2048 floats stay in registers between the range
// and the rounding (read from HBM once, all of a row's requests in flight); longer ones are read again.
// Per channel also: scale, zero-point, the sum of the signed-domain codes (it folds the activation zero-point into
// the integer bias) and, from them, the layer constants - so they need no launch of their own.
// Bound by memory and its latency: 8.6 M parameters (three hidden layers of 2048) 26 us with one wavefront per row storing
// single bytes, plus 4.5 us for the constants' launch.
constexpr int QR_CHUNK = 2048, QR_LD = QR_CHUNK + 16;
template <bool SYM>
__global__ __launch_bounds__(512) void k_qp_rows(const QTab* __restrict__ tab, const QOut o) {
    __shared__ __align__(16) int8_t codes[QR_ROWS * QR_LD];
    __shared__ float s_red[2][8];
    __shared__ int s_bad[8];
    const QTab& t = *tab;
    const int l = layer_of_block(t, blockIdx.x, true);
    const QLayerTab L = t.L[l];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = L.N, K = L.K, n0 = ((int)blockIdx.x - t.row_blk0[l]) * QR_ROWS;
    const float AQ_GLOBAL* w = (const float AQ_GLOBAL*)o.ptrs->w[l];
    const bool vec = (K & 3) == 0 && ((uintptr_t)o.ptrs->w[l] & 15) == 0;
    const bool held = K <= QR_CHUNK;
    constexpr int R = QR_CHUNK / 256;  // float4 per lane and row chunk

    // (rows past the end re-read the last one)
    const float AQ_GLOBAL* src = w + (int64_t)(n0 + wave < N ? n0 + wave : N - 1) * K;
    f4v v[R];
    auto load = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const int k = k0 + 4 * (lane + 64 * c);
            v[c] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
            if (k0 + 256 * c >= K) continue;  // (scalar)
            if (vec) {
                if (k < K) v[c] = *(const f4v AQ_GLOBAL*)(src + k);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k + j < K) v[c][j] = src[k + j];
            }
        }
    };
    if (held) load(0);
    // what the constants of this wavefront's channel need, requested now: at the end of the kernel each of these was a
    // round trip of its own
    const int n_own = n0 + wave;
    float c_bias = 0.0f, c_gamma = 1.0f, c_beta = 0.0f;
    const ActQ a_in = o.actq[l], a_out = o.actq[l + 1];
    if (n_own < N) {
        if (const float* p = o.ptrs->b[l]) c_bias = ((const float AQ_GLOBAL*)p)[n_own];
        if (L.ln) {
            if (const float* p = o.ptrs->gamma[l]) c_gamma = ((const float AQ_GLOBAL*)p)[n_own];
            if (const float* p = o.ptrs->beta[l]) c_beta = ((const float AQ_GLOBAL*)p)[n_own];
        }
    }

    float s;
    int z = 0;
    bool bounded = false;  // no value beyond the largest code
    if (SYM) {
        // the largest magnitude by its bits (in order for finite values; anything above them is not finite)
        uint32_t most = 0;
        for (int k0 = 0; k0 < K; k0 += QR_CHUNK) {
            if (!held) load(k0);
#pragma unroll
            for (int c = 0; c < R; ++c)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t u = __float_as_uint(v[c][j]) & 0x7fffffffu;
                    most = most > u ? most : u;
                }
        }
        const bool bad = __ballot(most > 0x7f7fffffu) != 0;
        float amax = __uint_as_float(most);
        if (bad) {  // the same over what is no NaN
            amax = 0.0f;
            for (int k0 = 0; k0 < K; k0 += QR_CHUNK) {
                if (!held) load(k0);
#pragma unroll
                for (int c = 0; c < R; ++c)
#pragma unroll
                    for (int j = 0; j < 4; ++j) amax = fmaxf(amax, fabsf(v[c][j]));
            }
        }
        bounded = !bad;
        amax = wave_max(amax);
        s = amax / (float)t.w_qw;
        if (amax == 0.0f) s = 1.0f;
        if (bad && lane == 0) atomicOr(o.status, kStatNonFinite);
    } else {
        // the layer's range from its workgroups' partial ones (at most 256)
        float hi = 0.0f, nlo = 0.0f;
        int bad = 0;
        for (int i = tid; i < L.rng_blks; i += 512) {
            const uint32_t* q = o.part + 3 * (t.rng_blk0[l] + i);
            hi = fmaxf(hi, __uint_as_float(q[0]));
            nlo = fmaxf(nlo, __uint_as_float(q[1]));
            bad |= (int)q[2];
        }
        hi = wave_max(hi);
        nlo = wave_max(nlo);
        bad = wave_or_i32(bad);
        if (lane == 0) {
            s_red[0][wave] = hi;
            s_red[1][wave] = nlo;
            s_bad[wave] = bad;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            hi = fmaxf(hi, s_red[0][i]);
            nlo = fmaxf(nlo, s_red[1][i]);
            bad |= s_bad[i];
        }
        asym_qparams(hi, nlo, t.w_qdenom, t.w_qmax, s, z);
        if (bad && n0 == 0 && tid == 0) atomicOr(o.status, kStatNonFinite);
    }

    const QuantScale qs = make_quant_scale(s);
    bounded = bounded && qs.rcp_ok;
    const float lo = SYM ? -(float)t.w_qw : -(float)z, hi = SYM ? (float)t.w_qw : (float)(t.w_qmax - z), add = SYM ? 128.0f : (float)z;
    int sum = 0;
    for (int k0 = 0; k0 < K; k0 += QR_CHUNK) {
        if (!held) load(k0);
#pragma unroll
        for (int c = 0; c < R; ++c) {
            if (k0 + 256 * c >= L.KS * 32) continue;  // (scalar)
            const int kk = 4 * (lane + 64 * c);
            const float4 x = make_float4(v[c][0], v[c][1], v[c][2], v[c][3]);
            uint32_t q = SYM && bounded ? quant_s8x4_bounded(x, qs) : quant_s8x4(x, qs, lo, hi, add);
            // entries behind the end of K are zeros in the signed domain (unconditionally: behind a scalar test for the pieces
            // that reach it, the compiler took 95 registers instead of 64, two workgroups per CU instead of four)
            const int left = K - k0 - kk;
            if (left < 4) q = left <= 0 ? 0u : q & (0xffffffffu >> (8 * (4 - left)));
            sum = __builtin_amdgcn_sdot4((int)q, 0x01010101, sum, false);
            *(uint32_t*)(codes + wave * QR_LD + kk) = q;
        }
        __syncthreads();
        const int ks0 = k0 >> 5, halves = 2 * (L.KS - ks0 < QR_CHUNK / 32 ? L.KS - ks0 : QR_CHUNK / 32);
        for (int idx = tid; idx < QR_ROWS * halves; idx += 512) {
            const int row = idx & (QR_ROWS - 1), c = idx / QR_ROWS, n = n0 + row;
            if (n < N)
                *(v4i AQ_GLOBAL*)(L.wp + (((int64_t)(n >> 5) * L.KS + ks0 + (c >> 1)) * 64 + (n & 31) + 32 * (c & 1)) * 16) =
                    *(const v4i*)(codes + row * QR_LD + 16 * c);
        }
        if (k0 + QR_CHUNK < K) __syncthreads();
    }
    sum = wave_sum_i32(sum);
    if (lane != 0 || n_own >= N) return;
    L.s_w[n_own] = s;
    L.z_w[n_own] = z;
    L.rowsum[n_own] = sum;
    layer_consts_channel(L, t.asym, a_in, a_out, s, z, c_bias, sum, n_own, o.fast + l, o.status);
    if (L.ln) {  // LayerNorm gain and offset (defaults 1 and 0) into their slots of the constant pack
        L.rz[n_own] = __float_as_int(c_gamma);
        L.sh[n_own] = __float_as_int(c_beta);
    }
}

// ---------------------------------------------------------------------------------------------
// Policy blob, one launch each way: 64 header bytes (six words, then zeros), 128 bytes of activation parameters and
// short-form flags (padded with zeros), the layer part of the slab.  (As a header launch and two copies an export or
// an import cost the host 8 us.)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void copy16(v4i* __restrict__ dst, const v4i* __restrict__ src, int64_t n, int64_t first, int64_t stride) {
    for (int64_t i = first; i < n; i += 4 * stride) {
        v4i v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * stride < n) v[u] = src[i + u * stride];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * stride < n) dst[i + u * stride] = v[u];
    }
}
// header and tail of a blob, by the first 64 threads of one workgroup
__device__ __forceinline__ void blob_head_out(uint32_t* __restrict__ blob, const uint32_t (&w)[6], const uint32_t* __restrict__ tail,
                                              int tail_words) {
    const int i = threadIdx.x;
    if (i < 16) {
        uint32_t v = 0u;
#pragma unroll
        for (int j = 0; j < 6; ++j) v = i == j ? w[j] : v;
        blob[i] = v;
    } else if (i < 48) {
        blob[i] = i - 16 < tail_words ? tail[i - 16] : 0u;
    }
}
__device__ __forceinline__ void blob_head_in(const uint32_t* __restrict__ blob, const uint32_t (&w)[6], uint32_t* __restrict__ tail,
                                             int tail_words, int* __restrict__ status) {
    const int i = threadIdx.x;
    bool wrong = false;
#pragma unroll
    for (int j = 0; j < 6; ++j) wrong |= i == j && blob[j] != w[j];
    if (i < tail_words) tail[i] = blob[16 + i];
    const uint64_t any = __ballot(wrong);
    if (i == 0) *status = any ? kStatBlob : 0;
}
__global__ __launch_bounds__(256) void k_blob_export(const BlobHead h, const uint32_t* __restrict__ tail, const v4i* __restrict__ slab,
                                                     int64_t n16, uint32_t* __restrict__ blob) {
    if (blockIdx.x == 0) {
        if (threadIdx.x < 64) blob_head_out(blob, h.w, tail, h.tail_words);
        return;
    }
    copy16((v4i*)(blob + 48), slab, n16, (int64_t)(blockIdx.x - 1) * 256 + threadIdx.x, (int64_t)(gridDim.x - 1) * 256);
}
__global__ __launch_bounds__(256) void k_blob_import(const BlobHead h, uint32_t* __restrict__ tail, v4i* __restrict__ slab, int64_t n16,
                                                     const uint32_t* __restrict__ blob, int* __restrict__ status) {
    if (blockIdx.x == 0) {
        if (threadIdx.x < 64) blob_head_in(blob, h.w, tail, h.tail_words, status);
        return;
    }
    copy16(slab, (const v4i*)(blob + 48), n16, (int64_t)(blockIdx.x - 1) * 256 + threadIdx.x, (int64_t)(gridDim.x - 1) * 256);
}

// ---------------------------------------------------------------------------------------------
// n-bit weight codes stored sub-byte (the packed policy blob): eight consecutive codes of the operand
// order -> n bytes and back.  Codes are kept in the signed domain in the library (symmetric: the code
// itself, in [-qw, qw]; per tensor: unsigned code - 128), the stored field is the code plus `off`
// (qw resp. 128), an n-bit unsigned number.  Padding entries (feature >= N or k >= K) are zero in the
// signed domain, which the per-tensor scheme cannot store in n < 8 bits: they are written as field 0
// and restored from their position when unpacking.
// ---------------------------------------------------------------------------------------------
// One launch each way for the whole packed blob: workgroup 0 does header and tail, then every layer has its workgroups
// for the codes (a thread takes 32 codes = n words) and for its constants, copied as they are.
__device__ __forceinline__ int packed_layer_of(const PackedArgs& a, int blk) {
    int l = a.n_layers - 1;
    while (l > 0 && blk < a.L[l].blk0) --l;
    return l;
}
__global__ __launch_bounds__(256) void k_packed_export(const BlobHead h, const PackedArgs a, const uint32_t* __restrict__ tail,
                                                       const char* __restrict__ slab, uint32_t* __restrict__ blob) {
    if (blockIdx.x == 0) {
        if (threadIdx.x < 64) blob_head_out(blob, h.w, tail, h.tail_words);
        return;
    }
    const PackedLayer& L = a.L[packed_layer_of(a, blockIdx.x)];
    const int rel = blockIdx.x - L.blk0, bits = a.bits, off = a.off;
    if (rel >= L.code_blks) {
        copy16((v4i*)((char*)blob + L.c_off), (const v4i*)(slab + L.c_src), L.c_bytes / 16, (int64_t)(rel - L.code_blks) * 256 + threadIdx.x,
               (int64_t)L.const_blks * 256);
        return;
    }
    uint32_t* out = (uint32_t*)((char*)blob + L.w_off);
    if (rel == 0 && threadIdx.x < 64) {  // alignment padding behind the codes: kept zero
        const int64_t end = (int64_t)L.groups * bits, padded = (L.c_off - L.w_off) / 4;
        if (end + threadIdx.x < padded) out[end + threadIdx.x] = 0u;
    }
    const int64_t g = (int64_t)rel * 256 + threadIdx.x;
    if (g >= L.groups) return;
    const int8_t* wp = (const int8_t*)(slab + L.w_src) + 32 * g;
    const v4i c[2] = {((const v4i*)wp)[0], ((const v4i*)wp)[1]};
    const int fmax = (1 << bits) - 1;
    uint64_t acc = 0;
    int have = 0, word = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        int u = (int)(int8_t)((uint32_t)c[j >> 4][(j >> 2) & 3] >> (8 * (j & 3))) + off;
        u = u < 0 ? 0 : (u > fmax ? 0 : u);
        acc |= (uint64_t)u << have;
        have += bits;
        if (have >= 32) {
            out[g * bits + word++] = (uint32_t)acc;
            acc >>= 32;
            have -= 32;
        }
    }
}
__global__ __launch_bounds__(256) void k_packed_import(const BlobHead h, const PackedArgs a, uint32_t* __restrict__ tail,
                                                       char* __restrict__ slab, const uint32_t* __restrict__ blob, int* __restrict__ status) {
    if (blockIdx.x == 0) {
        if (threadIdx.x < 64) blob_head_in(blob, h.w, tail, h.tail_words, status);
        return;
    }
    const PackedLayer& L = a.L[packed_layer_of(a, blockIdx.x)];
    const int rel = blockIdx.x - L.blk0, bits = a.bits, off = a.off;
    if (rel >= L.code_blks) {
        copy16((v4i*)(slab + L.c_src), (const v4i*)((const char*)blob + L.c_off), L.c_bytes / 16,
               (int64_t)(rel - L.code_blks) * 256 + threadIdx.x, (int64_t)L.const_blks * 256);
        return;
    }
    const int64_t g = (int64_t)rel * 256 + threadIdx.x;
    if (g >= L.groups) return;
    const uint32_t* src = (const uint32_t*)((const char*)blob + L.w_off) + g * bits;
    // position of the group's two 16-byte pieces in the operand order: tile (n / 32, k / 32) = 1 KiB,
    // lane = n % 32 + 32 * ((k % 32) / 16), byte = k % 16
    const uint32_t fmask = (1u << bits) - 1u;
    uint64_t acc = 0;
    int have = 0, word = 0;
    v4i v[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int64_t e = 32 * g + 16 * p;
        const uint32_t tile = (uint32_t)(e >> 10);
        const int nt = (int)(tile / (uint32_t)L.KS), ks = (int)(tile - (uint32_t)nt * (uint32_t)L.KS);
        const int lane = (int)((e & 1023) >> 4);
        const int n = nt * 32 + (lane & 31), k0 = ks * 32 + 16 * (lane >> 5);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            if (have < bits) {
                acc |= (uint64_t)src[word++] << have;
                have += 32;
            }
            int sgn = (int)((uint32_t)acc & fmask) - off;
            acc >>= bits;
            have -= bits;
            if (n >= L.N || k0 + j >= L.K) sgn = 0;
            const uint32_t b = (uint32_t)(uint8_t)(int8_t)sgn << (8 * (j & 3));
            v[p][j >> 2] = (j & 3) == 0 ? (int)b : (int)((uint32_t)v[p][j >> 2] | b);
        }
    }
    v4i* dst = (v4i*)(slab + L.w_src) + 2 * g;
    dst[0] = v[0];
    dst[1] = v[1];
}

// ---------------------------------------------------------------------------------------------
// Measurement aid: the memory traffic of the flat quantize pass without its arithmetic (4 bytes read and
// 1 byte written per element, no reduction, no dependence between the loads and the stores of a thread
// other than the data itself).  What this kernel reaches at a given size is the ceiling for the quantizer
// at that size.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_stream_reference(const float4* __restrict__ in4, int64_t n4,
                                                          uint32_t* __restrict__ out) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += 2 * stride) {
        const f4v a = __builtin_nontemporal_load((const f4v*)in4 + i);
        const bool two = i + stride < n4;
        f4v b = a;
        if (two) b = __builtin_nontemporal_load((const f4v*)in4 + i + stride);
        __builtin_nontemporal_store((__float_as_uint(a[0]) >> 24) | ((__float_as_uint(a[1]) >> 24) << 8) |
                                        ((__float_as_uint(a[2]) >> 24) << 16) | ((__float_as_uint(a[3]) >> 24) << 24),
                                    out + i);
        if (two)
            __builtin_nontemporal_store((__float_as_uint(b[0]) >> 24) | ((__float_as_uint(b[1]) >> 24) << 8) |
                                            ((__float_as_uint(b[2]) >> 24) << 16) | ((__float_as_uint(b[3]) >> 24) << 24),
                                        out + i + stride);
    }
}

aq_status launch_stream_reference(const float* d_in, int64_t n, void* d_out, hipStream_t st) {
    const int64_t n4 = n / 4;
    int64_t g = (n4 + 511) / 512;  // two 16-byte pieces per thread, like the per-channel kernel on 2048-wide rows
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_stream_reference, dim3((unsigned)g), dim3(256), 0, st, (const float4*)d_in, n4, (uint32_t*)d_out);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

// ---------------------------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------------------------
aq_status launch_blob_export(const BlobHead& h, const void* d_tail, const void* slab, int64_t bytes, void* blob, hipStream_t st) {
    const unsigned g = 1 + (unsigned)blob_copy_blocks(bytes);
    hipLaunchKernelGGL(k_blob_export, dim3(g), dim3(256), 0, st, h, (const uint32_t*)d_tail, (const v4i*)slab, bytes / 16, (uint32_t*)blob);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}
aq_status launch_blob_import(const BlobHead& h, void* d_tail, void* slab, int64_t bytes, const void* blob, int* status, hipStream_t st) {
    const unsigned g = 1 + (unsigned)blob_copy_blocks(bytes);
    hipLaunchKernelGGL(k_blob_import, dim3(g), dim3(256), 0, st, h, (uint32_t*)d_tail, (v4i*)slab, bytes / 16, (const uint32_t*)blob, status);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}
aq_status launch_packed_export(const BlobHead& h, const PackedArgs& a, const void* d_tail, const void* slab, void* blob, hipStream_t st) {
    hipLaunchKernelGGL(k_packed_export, dim3((unsigned)a.blocks), dim3(256), 0, st, h, a, (const uint32_t*)d_tail, (const char*)slab, (uint32_t*)blob);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}
aq_status launch_packed_import(const BlobHead& h, const PackedArgs& a, void* d_tail, void* slab, const void* blob, int* status, hipStream_t st) {
    hipLaunchKernelGGL(k_packed_import, dim3((unsigned)a.blocks), dim3(256), 0, st, h, a, (uint32_t*)d_tail, (char*)slab, (const uint32_t*)blob, status);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

static int grid_for(int64_t work_items, int per_block, int cap) {
    int64_t g = (work_items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

aq_status launch_fill_u32(uint32_t* p, int n, uint32_t v, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_u32, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_quantize_tensor(const float* d_w, int64_t rows, int64_t cols, int wscheme, float qdenom,
                                 int qmax, int qw, void* d_codes, float* d_scale, int32_t* d_zp, uint32_t* d_ws, hipStream_t st) {
    const int64_t n = rows * cols;
    const float4* w4 = (const float4*)d_w;
    uint32_t* c4 = (uint32_t*)d_codes;
    if (wscheme == AQ_W_TENSOR_ASYM_U8) {
        const int64_t n4 = n / 4;
        // enough workgroups to keep every CU's memory pipeline full; partial ranges go to d_ws[16..]
        const int g1 = grid_for(n4, 256 * 4, 1024);
        hipLaunchKernelGGL(k_range_partials, dim3(g1), dim3(256), 0, st, d_w, n, d_ws + 16);
        const int g2 = grid_for(n4, 256 * 4, 2048);
        hipLaunchKernelGGL(k_quant_asym_flat, dim3(g2), dim3(256), 0, st, w4, n4, d_ws + 16, g1, qdenom, qmax, c4, d_scale,
                           d_zp, d_ws + 2);
    } else {
        const int cols4 = (int)(cols / 4);
#define AQ_SHORT(G, V, U)                                                                                                     \
    hipLaunchKernelGGL((k_quant_sym_rows_short<G, V, U>), dim3((unsigned)((rows + 4 * (64 / G) * U - 1) / (4 * (64 / G) * U))), \
                       dim3(256), 0, st, w4, rows, cols4, qw, c4, d_scale, d_zp, d_ws)
        // Fewer, fuller wavefronts from the row counts on where they fill the chip, us so / with a wavefront or a workgroup per row:
        // 500000 x 32 25.4 / 107, 2000 x 400 5.2 / 4.6, 20000 x 400 9.3 / 17.9, 2000 x 1000 4.8 / 4.5, 5000 x 700 5.4 / 6.7, 30000 x 1000
        // 25.1 / 32.1.  Rows of 132 to 256 at any count, two to a wavefront / one to a wavefront / four of one each in flight:
        // 25000 x 212 from HBM 7.7 / 8.9 / 10.0, in cache 7.1 / 7.4 / 9.0; 100000 x 160 18.2 / 25.7 / 22.2.
        if (cols4 <= 16) AQ_SHORT(16, 1, 4);
        else if (cols4 <= 32) AQ_SHORT(16, 2, 2);
        else if (cols4 <= 64) AQ_SHORT(32, 2, 1);
        else if (cols4 <= 128 && rows >= 6000) AQ_SHORT(64, 2, 2);
        else if (cols4 <= 256 && rows >= 4096) AQ_SHORT(64, 4, 1);
#undef AQ_SHORT
        else {
#define AQ_ROW_WG(R) \
    hipLaunchKernelGGL(k_quant_sym_row_wg<R>, dim3((unsigned)rows), dim3(256), 0, st, w4, cols4, qw, c4, d_scale, d_zp, d_ws)
            if (cols4 <= 256) AQ_ROW_WG(1);
            else if (cols4 <= 512) AQ_ROW_WG(2);
            else if (cols4 <= 1024) AQ_ROW_WG(4);
            else if (cols4 <= 2048) AQ_ROW_WG(8);
            else
                hipLaunchKernelGGL(k_quant_sym_rows_long, dim3((unsigned)rows), dim3(256), 0, st, w4, rows, cols4, qw, c4,
                                   d_scale, d_zp, d_ws);
#undef AQ_ROW_WG
        }
    }
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_unpack_weights(const int8_t* wp, int N, int K, int KS, int asym, uint8_t* codes, hipStream_t st) {
    const int64_t n = (int64_t)N * K;
    hipLaunchKernelGGL(k_unpack_weights, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, wp, N, K, KS, asym,
                       codes);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_quantize_policy(const QTab* d_tab, const QTab& h_tab, const QPtrs& ptrs, const RangesArg& r, const QOut& o,
                                 hipStream_t st) {
    if (h_tab.asym) {
        hipLaunchKernelGGL(k_qp_ranges, dim3(h_tab.rng_blks_total), dim3(256), 0, st, d_tab, ptrs, r, o);
        hipLaunchKernelGGL(k_qp_rows<false>, dim3(h_tab.row_blks), dim3(512), 0, st, d_tab, o);
    } else {
        hipLaunchKernelGGL(k_qp_prep, dim3(1), dim3(64), 0, st, d_tab, ptrs, r, o);
        hipLaunchKernelGGL(k_qp_rows<true>, dim3(h_tab.row_blks), dim3(512), 0, st, d_tab, o);
    }
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

}  // namespace aq

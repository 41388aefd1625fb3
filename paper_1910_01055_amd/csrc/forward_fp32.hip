// The full-precision actor (the paper's fp32 baseline policy, Sec. 3.1) and the min/max calibration of activation
// ranges, on the fp32 matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and sums, 256 flop per clock and CU).
//
// Operand mapping, shared by both kernels below: weights are the A operand (rows = output features), batch rows (or
// output positions) the B operand, so that a lane owns one row and four consecutive features per accumulator quad and
// stores them as one float4.  A lane's k values within a stage of 16 are 4 g .. 4 g + 3 (g = lane / 16): the sum over
// k is free to be taken in any order, so the four MFMAs of a stage take element 0 .. 3 of one float4 per operand
// instead of one float each.
//
// Weights are read packed: 1 KiB per 16 features x 16 k, lane l's float4 at 16 l, zeros beyond N and K
// (k_keep_params; written together with the handle's copy of the learner's parameters).  An operand read straight from
// the row-major array takes its 64 float4 from 16 rows, neighbouring lanes from different rows, and the vector memory
// path then spends 75 clocks on the instruction instead of 16: 1024 x 1024 on 2000 rows 65 us at best, bound by that.
//
// k_fp32_layer: one layer (fully connected or implicit-GEMM convolution) from and to global memory, inputs staged in
//   LDS.  k_fp32_mlp: a whole small MLP in one launch, activations in LDS.
#include "fp32_split.hpp"
#include "ln_rows.hpp"

namespace aq {

namespace {

typedef const float AQ_GLOBAL* gf_ptr;
typedef const v4f AQ_GLOBAL* gv4f_ptr;

constexpr int FW_ = 8;            // waves per workgroup
constexpr int FT_ = FW_ * 64;
constexpr int MW_ = 16;           // ... of the whole-MLP kernel: four on each SIMD hide the first weights of a tile
constexpr int MT_ = MW_ * 64;

// one stage of 16 k for FT x RT quads; the quads alternate, so that an MFMA does not wait for the one before it
template <int FT, int RT, int AF>
__device__ __forceinline__ void mma_stage(const v4f (&w)[FT], const v4f (&x)[RT], v4f (&acc)[AF][RT]) {
    static_assert(FT <= AF, "");
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[f][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[f][i], x[r][i], acc[f][r], 0, 0, 0);
}

__device__ __forceinline__ float head_value(float y, int head) { return head == AQ_HEAD_TANH ? tanhf(y) : y; }

}  // namespace

// ---------------------------------------------------------------------------------------------- one layer
// Eight waves as WN x WM x WK (features, rows, K); a wave owns 16 FT features x 16 RT rows of the workgroup's tile and
// KS stages of 16 k of each LDS stage of BK = 16 KS WK.  LDS stages alternate between two buffers: while one is
// multiplied, the next one's values sit in registers on their way to the other and the one after that is requested;
// one barrier per stage.  Weights are one LDS stage ahead in registers.  Bound by the matrix cores where the tiles fill
// the chip (1024 x 1024 on 2000 rows: 41 us = 102 TFLOP/s; with every load taken out 35 us), by the last, partly filled
// round of workgroups elsewhere (conv 512 -> 64 on 20736 rows: 23 us for 9 us of MFMAs).  Row stride = BK + 4 floats: an operand
// read's 16 rows fall on 64 different banks.
// two staged inputs, or the partial sums of every wave
constexpr size_t fp32_layer_lds(int ft, int rt, int wm, int wk, int ks) {
    const size_t x = (size_t)2 * 16 * rt * wm * (16 * ks * wk + 4) * 4, p = wk > 1 ? (size_t)FW_ * ft * rt * 1024 : 0;
    return x > p ? x : p;
}
template <int FT, int RT, int WN, int WM, int WK, int KS, bool CONV, bool U8>
__global__ __launch_bounds__(FT_) void k_fp32_layer(const Fp32Layer L, const void* __restrict__ in, float* __restrict__ out,
                                                    const int64_t rows, RangeSlot* __restrict__ slots) {
    static_assert(WN * WM * WK == FW_, "eight waves");
    constexpr int BM = 16 * RT * WM, BK = 16 * KS * WK, LD = BK + 4, NQ = FT * RT;
    constexpr int CPR = BK / 4;               // float4 per row of a stage: a power of two, at most the workgroup's threads
    constexpr int XS = BM * CPR / FT_;        // ... per thread, all in the same column
    static_assert(CPR <= FT_ && BM * CPR % FT_ == 0, "whole columns");
    extern __shared__ __align__(16) float smx[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int wk = wave % WK, wn = (wave / WK) % WN, wm = wave / (WK * WN);
    const uint32_t bx = L.features_first ? blockIdx.y : blockIdx.x, by = L.features_first ? blockIdx.x : blockIdx.y;
    const int64_t row0 = (int64_t)bx * BM;
    const int t0 = (by * WN + wn) * FT;  // this wave's first feature tile
    const int K = L.K, N = L.N, nst = (K + 15) >> 4, tiles = (N + 15) >> 4;

    // where the rows this thread stages begin; rows past the end re-read the last one and are not stored
    const int c4 = 4 * (tid & (CPR - 1));
    int64_t xoff[XS];
    const bool r32 = rows <= 0x7fffffffLL;
#pragma unroll
    for (int u = 0; u < XS; ++u) {
        int64_t row = row0 + tid / CPR + u * (FT_ / CPR);
        if (row >= rows) row = rows - 1;
        if (CONV) {
            const int per_img = L.oh * L.ow;
            const int64_t b = r32 ? (int64_t)((uint32_t)row / (uint32_t)per_img) : row / per_img;
            const int p = (int)(row - b * per_img);
            const int oy = p / L.ow, ox = p - oy * L.ow;
            xoff[u] = ((b * L.in_h + (int64_t)oy * L.stride) * L.in_w + (int64_t)ox * L.stride) * L.in_c;
        } else {
            xoff[u] = row * K;
        }
    }
    const int run = CONV ? L.kw * L.in_c : K;     // consecutive k of one window row
    const int line = CONV ? L.in_w * L.in_c : 0;  // from one window row to the next
    const float inv_run = 1.0f / (float)run;
    auto koff = [&](int k) {                       // where k lies relative to the row's first input
        if (!CONV) return k;
        // (k < 65536: the quotient plus a half over `run` is far from an integer compared with the rounding error)
        const int ky = (int)(((float)k + 0.5f) * inv_run);
        return ky * line + (k - ky * run);
    };
    const bool quads = !CONV || (run & 3) == 0;    // four consecutive k are four consecutive inputs
    auto one = [&](int64_t o) { return U8 ? (float)((const uint8_t*)in)[o] : ((const float*)in)[o]; };
    v4f xr[XS];
    auto fetch_x = [&](int s) __attribute__((always_inline)) {
        const int k = s * BK + c4;
        if (quads && s * BK + BK <= K) {
            const int ko = koff(k);
#pragma unroll
            for (int u = 0; u < XS; ++u) {
                if (U8) {
                    const uint32_t q = *(const u32_u*)((const uint8_t*)in + xoff[u] + ko);
#pragma unroll
                    for (int i = 0; i < 4; ++i) xr[u][i] = (float)((q >> (8 * i)) & 255u);
                } else {
                    xr[u] = *(const v4f_u*)((const float*)in + xoff[u] + ko);
                }
            }
        } else {  // the stage that ends K, or a convolution whose window rows are no multiple of 4 long
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool ok = k + i < K;
                const int ko = ok ? koff(k + i) : 0;
#pragma unroll
                for (int u = 0; u < XS; ++u) xr[u][i] = ok ? one(xoff[u] + ko) : 0.0f;
            }
        }
    };
    auto store_x = [&](int buf) __attribute__((always_inline)) {
        float* d = smx + buf * (BM * LD) + (tid / CPR) * LD + c4;
#pragma unroll
        for (int u = 0; u < XS; ++u) *(v4f*)(d + u * (FT_ / CPR) * LD) = xr[u];
    };
    // this wave's weight operands of LDS stage s; past the last 16 k zeros, like the inputs there (a weight may be
    // infinite: no weight but its own input's may meet a zero), from a block of them instead of behind a branch
    const float* wbase[FT];
#pragma unroll
    for (int f = 0; f < FT; ++f) {
        const int t = t0 + f < tiles ? t0 + f : tiles - 1;
        wbase[f] = L.wpk + (int64_t)t * nst * 256;
    }
    v4f wr[KS][FT];
    auto fetch_w = [&](auto j_c, int s) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        const int k16 = (s * WK + wk) * KS + j;
#pragma unroll
        for (int f = 0; f < FT; ++f) wr[j][f] = *(const v4f*)((k16 < nst ? wbase[f] + (int64_t)k16 * 256 : L.zeros) + lane * 4);
    };

    v4f acc[FT][RT];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[f][r] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const int ns = (K + BK - 1) / BK;
    static_for<0, KS>([&](auto j_c) __attribute__((always_inline)) { fetch_w(j_c, 0); });
    fetch_x(0);
    store_x(0);
    if (ns > 1) fetch_x(1);
    lds_barrier();
    const float* xop = smx + (wm * RT * 16 + i16) * LD + wk * (16 * KS) + 4 * g;
    for (int s = 0; s < ns; ++s) {
        const float* xb = xop + (s & 1) * (BM * LD);
        v4f x[2][RT];  // operands are read one 16-k stage ahead of their MFMAs
#pragma unroll
        for (int r = 0; r < RT; ++r) x[0][r] = *(const v4f*)(xb + r * 16 * LD);
        static_for<0, KS>([&](auto j_c) __attribute__((always_inline)) {
            constexpr int j = decltype(j_c)::value;
            if (j + 1 < KS) {
#pragma unroll
                for (int r = 0; r < RT; ++r) x[(j + 1) & 1][r] = *(const v4f*)(xb + r * 16 * LD + 16 * (j + 1));
            }
            mma_stage<FT, RT, FT>(wr[j], x[j & 1], acc);
            fetch_w(j_c, s + 1 < ns ? s + 1 : s);
            asm volatile("" ::: "memory");  // (or the compiler moves the request down to its use)
        });
        if (s + 1 < ns) {
            store_x((s + 1) & 1);
            if (s + 2 < ns) fetch_x(s + 2);
        }
        lds_barrier();
    }

    float lo = INFINITY, hi = -INFINITY;
    const bool relu = L.relu != 0;
    auto emit = [&](const v4f& a, int f, int r) __attribute__((always_inline)) {
        const int64_t row = row0 + (wm * RT + r) * 16 + i16;
        const int n = (t0 + f) * 16 + 4 * g;
        if (row >= rows || n >= N) return;
        v4f v = a;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (n + i < N) {
                if (L.b) v[i] += L.b[n + i];
                if (relu) v[i] = v[i] > 0.0f ? v[i] : 0.0f;
                lo = fminf(lo, v[i]);
                hi = fmaxf(hi, v[i]);
                if (L.head >= 0) v[i] = head_value(v[i], L.head);
            }
        }
        float* o = out + row * N + n;
        if ((N & 3) == 0) {
            *(v4f_u*)o = v;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (n + i < N) o[i] = v[i];
        }
    };
    if constexpr (WK == 1) {
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int r = 0; r < RT; ++r) emit(acc[f][r], f, r);
    } else {
        // the partial sums of the WK waves of a tile meet in LDS (the last barrier freed it); quad q is summed by wave q % WK
        v4f* p4 = (v4f*)smx;
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int r = 0; r < RT; ++r) p4[(wave * NQ + f * RT + r) * 64 + lane] = acc[f][r];
        lds_barrier();
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                if (wk != (f * RT + r) % WK) continue;
                v4f t = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 0; k < WK; ++k) t += p4[((wave - wk + k) * NQ + f * RT + r) * 64 + lane];
                emit(t, f, r);
            }
    }
    if (slots) range_note(slots, (uint32_t)((blockIdx.y * gridDim.x + blockIdx.x) * FW_ + wave), lo, hi);
}

// ------------------------------------------------------------------------------------- a fully connected layer at few rows
// One workgroup owns FT tiles of 16 features x RT tiles of 16 rows and splits K over its eight waves: every byte of weights and
// inputs passes the CU's vector memory path once, straight into operand registers, PF stages of 16 k in flight, no barrier
// before the partial sums meet in LDS.  Inputs are requested along the rows (four lanes to 64 bytes; lanes down the rows
// take 75 clocks a request instead of 16) and change lanes on the way.  Bound by the fp32 matrix cores, 32 clocks an MFMA,
// and the vector memory path, 47 bytes a clock beside them at 16 x 32.  With a layer of 4 behind it, us on the tiles of the
// kernel above (inputs through LDS, a barrier every 128 to 512 k) and so: 3136-512 at 128 rows 16.4, 12.3, at 256 19.9, 17.3;
// 700-523 at 16 rows 9.9, 8.1, at 512 18.5, 16.5; 2048-2048 at 128 22.5, 19.6.
template <int FT, int RT, bool U8>
__global__ __launch_bounds__(FT_) void k_fp32_rows(const Fp32Layer L, const void* __restrict__ in, float* __restrict__ out,
                                                   const int64_t rows, RangeSlot* __restrict__ slots) {
    constexpr int PF = 4, NQ = FT * RT;
    __shared__ v4f part[FW_][NQ][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const uint32_t bx = L.features_first ? blockIdx.y : blockIdx.x, by = L.features_first ? blockIdx.x : blockIdx.y;
    const int64_t row0 = (int64_t)bx * (16 * RT);
    const int K = L.K, N = L.N, nst = (K + 15) >> 4, tiles = (N + 15) >> 4, t0 = by * FT;
    const int per = (nst + FW_ - 1) / FW_, s0 = wave * per, s1 = s0 + per < nst ? s0 + per : nst;
    gf_ptr wbase[FT];
#pragma unroll
    for (int f = 0; f < FT; ++f) wbase[f] = (gf_ptr)L.wpk + (int64_t)(t0 + f < tiles ? t0 + f : tiles - 1) * nst * 256 + lane * 4;
    int64_t xoff[RT];  // rows past the end re-read the last one and are not stored
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int64_t row = row0 + r * 16 + (lane >> 2);
        xoff[r] = (row < rows ? row : rows - 1) * K + 4 * (lane & 3);
    }
    const int swap = (i16 * 4 + g) * 4;
    v4f acc[FT][RT];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[f][r] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    v4f w[PF][FT], x[PF][RT];
    auto fetch = [&](auto p_c, int s) __attribute__((always_inline)) {
        constexpr int p = decltype(p_c)::value;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int64_t o = xoff[r] + 16 * s;
            if (16 * s + 16 <= K) {
                if (U8) {
                    const uint32_t q = *(const u32_u*)((const uint8_t*)in + o);
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[p][r][i] = (float)((q >> (8 * i)) & 255u);
                } else {
                    x[p][r] = *(const v4f_u AQ_GLOBAL*)((const float*)in + o);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool ok = 16 * s + 4 * (lane & 3) + i < K;
                    x[p][r][i] = 0.0f;
                    if (ok) x[p][r][i] = U8 ? (float)((const uint8_t*)in)[o + i] : ((const float*)in)[o + i];
                }
            }
        }
#pragma unroll
        for (int f = 0; f < FT; ++f) w[p][f] = *(gv4f_ptr)(wbase[f] + (s << 8));
    };
    auto stage = [&](auto p_c) __attribute__((always_inline)) {
        constexpr int p = decltype(p_c)::value;
        v4f y[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) y[r][i] = __int_as_float(__builtin_amdgcn_ds_bpermute(swap, __float_as_int(x[p][r][i])));
        mma_stage<FT, RT, FT>(w[p], y, acc);
    };
    if (s0 < s1) {
        static_for<0, PF>([&](auto p_c) __attribute__((always_inline)) {
            constexpr int p = decltype(p_c)::value;
            fetch(p_c, s0 + p < s1 ? s0 + p : s1 - 1);
        });
        int s = s0;
        for (; s + 2 * PF <= s1; s += PF) {
            static_for<0, PF>([&](auto p_c) __attribute__((always_inline)) {
                constexpr int p = decltype(p_c)::value;
                stage(p_c);
                fetch(p_c, s + p + PF);
                asm volatile("" ::: "memory");
            });
        }
        // (the last requests of a share behind scalar tests: clamped to its end instead, up to PF of them were re-reads that
        // took their turn on the vector memory path: 1024-1024 at 256 rows 13.5 us, 12.9 so, 2048-2048 at 128 20.5, 19.6; eight
        // stages in flight instead of four are slower, 18.5 for 17.3 of 3136-512 at 256)
        if (s + PF <= s1) {
            static_for<0, PF>([&](auto p_c) __attribute__((always_inline)) {
                constexpr int p = decltype(p_c)::value;
                stage(p_c);
                if (s + p + PF < s1) fetch(p_c, s + p + PF);
                asm volatile("" ::: "memory");
            });
            s += PF;
        }
        static_for<0, PF - 1>([&](auto p_c) __attribute__((always_inline)) {
            if (s + decltype(p_c)::value < s1) stage(p_c);
        });
    }
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int r = 0; r < RT; ++r) part[wave][f * RT + r][lane] = acc[f][r];
    lds_barrier();
    // quad q of the tile is summed and finished by wave q
    float lo = INFINITY, hi = -INFINITY;
    if (wave < NQ) {
        const int f = wave / RT, r = wave - f * RT, n = (t0 + f) * 16 + 4 * g;
        const int64_t row = row0 + r * 16 + i16;
        v4f v = part[0][wave][lane];
#pragma unroll
        for (int k = 1; k < FW_; ++k) v += part[k][wave][lane];
        if (row < rows && n < N) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (n + i < N) {
                    if (L.b) v[i] += L.b[n + i];
                    if (L.relu) v[i] = v[i] > 0.0f ? v[i] : 0.0f;
                    lo = fminf(lo, v[i]);
                    hi = fmaxf(hi, v[i]);
                    if (L.head >= 0) v[i] = head_value(v[i], L.head);
                }
            }
            float* o = out + row * N + n;
            if ((N & 3) == 0) {
                *(v4f_u*)o = v;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (n + i < N) o[i] = v[i];
            }
        }
        if (slots) range_note(slots, (uint32_t)((blockIdx.y * gridDim.x + blockIdx.x) * NQ + wave), lo, hi);
    }
}

// ---------------------------------------------------------------------------------------- a whole small MLP
// One workgroup owns 16 RT batch rows from the observation to the action; layer inputs and outputs alternate between
// two LDS buffers, weights come from L2 into operand registers.  A wave takes feature tiles wave, wave + 16, ... of
// a layer, in pairs; a last layer of at most four tiles is split over K instead.  Row stride = width + 4 floats: the 16
// rows of an operand read fall on 64 different banks.
// Bound by the fp32 matrix cores at large batch (16 rows x 256 x 256: 3.4 us per CU), by the chain of layers at small:
// 111-400-300-8 with LayerNorm on 3001 rows 115 us as five launches of vector-ALU kernels, 24 us in this one (eight
// waves instead of sixteen: 26.6 us).
template <int RT, bool U8, bool BYVAL>
__global__ __launch_bounds__(MT_) void k_fp32_mlp(const NetDev* __restrict__ netp, const F32Call c, const F32PtrArg<BYVAL> pa) {
    extern __shared__ __align__(16) float smf[];
    const NetDev& a = *netp;
    const F32Ptrs& P = f32_ptrs(pa);
    constexpr int ROWS = 16 * RT;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int ld = c.ld, nl = a.n_layers;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int64_t left = c.batch - row0;
    const int vrows = left < ROWS ? (int)left : ROWS;
    const uint32_t who = blockIdx.x * MW_ + wave;
    float* xin = smf;
    float* xout = smf + ROWS * ld;

    {   // observations -> LDS, zeros behind row ends (up to whole stages) and past the batch
        const int K = a.L[0].K, K16 = (K + 15) & ~15;
        float lo = INFINITY, hi = -INFINITY;
        const int total = ROWS * K16;
        const float inv = 1.0f / (float)K16;
#pragma unroll 4
        for (int idx = tid; idx < total; idx += MT_) {
            const int m = (int)(((float)idx + 0.5f) * inv), k = idx - m * K16;
            float v = 0.0f;
            if (m < vrows && k < K) {
                const int64_t off = (row0 + m) * K + k;
                v = U8 ? (float)((const uint8_t*)c.obs)[off] : ((const float*)c.obs)[off];
                lo = fminf(lo, v);
                hi = fmaxf(hi, v);
            }
            xin[m * ld + k] = v;
        }
        if (c.slots) range_note(c.slots, who, lo, hi);
    }

    for (int l = 0; l < nl; ++l) {
        const bool last = l == nl - 1;
        if (last && !c.actions) break;  // calibration stops in front of the head
        const int K = a.L[l].K, N = a.L[l].N, act = a.L[l].act;
        const gf_ptr w = (gf_ptr)P.wpk[l], bias = (gf_ptr)P.b[l];
        const int nst = (K + 15) >> 4, tiles = (N + 15) >> 4;
        const float* xrow = xin + i16 * ld + 4 * g;
        lds_barrier();  // this layer's inputs are in LDS

        // tiles t0 and t0 + MW_ (two = false: t0 alone) over stages [s0, s1)
        auto run = [&](auto nf_c, int t0, int s0, int s1, v4f (&acc)[2][RT]) __attribute__((always_inline)) {
            constexpr int NF = decltype(nf_c)::value;
            constexpr int PD = 4;
            gf_ptr wrow[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) wrow[f] = w + (int64_t)(t0 + MW_ * f) * nst * 256 + lane * 4;
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int r = 0; r < RT; ++r) acc[f][r] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
            if (s0 < s1) {
                v4f wa[PD][NF];
                static_for<0, PD>([&](auto p_c) __attribute__((always_inline)) {
                    constexpr int p = decltype(p_c)::value;
                    const int s = s0 + p < s1 ? s0 + p : s1 - 1;
#pragma unroll
                    for (int f = 0; f < NF; ++f) wa[p][f] = *(gv4f_ptr)(wrow[f] + (s << 8));
                });
                v4f x[2][RT];  // operands are read one stage ahead of their MFMAs
#pragma unroll
                for (int r = 0; r < RT; ++r) x[0][r] = *(const v4f*)(xrow + r * 16 * ld + (s0 << 4));
                auto stage = [&](auto p_c, int s) __attribute__((always_inline)) {
                    constexpr int p = decltype(p_c)::value;
                    const int nx = s + p + 1 < s1 ? s + p + 1 : s1 - 1;
#pragma unroll
                    for (int r = 0; r < RT; ++r) x[(p + 1) & 1][r] = *(const v4f*)(xrow + r * 16 * ld + (nx << 4));
                    mma_stage<NF, RT, 2>(wa[p], x[p & 1], acc);
                };
                int s = s0;
                for (; s + PD <= s1; s += PD) {
                    static_for<0, PD>([&](auto p_c) __attribute__((always_inline)) {
                        constexpr int p = decltype(p_c)::value;
                        stage(p_c, s);
                        const int nx = s + p + PD < s1 ? s + p + PD : s1 - 1;
#pragma unroll
                        for (int f = 0; f < NF; ++f) wa[p][f] = *(gv4f_ptr)(wrow[f] + (nx << 8));
                        asm volatile("" ::: "memory");
                        __builtin_amdgcn_sched_barrier(0);
                    });
                }
                static_for<0, PD - 1>([&](auto p_c) __attribute__((always_inline)) {
                    if (s + decltype(p_c)::value < s1) stage(p_c, s);
                });
            }
        };

        if (last && tiles <= 4) {
            // feature tile x K part per wave; partial sums meet in the idle buffer, which holds those of ld / 16 waves
            // (ld >= 132: at least eight)
            const int ntl = tiles <= 1 ? 0 : tiles <= 2 ? 1 : 2, nt2 = 1 << ntl, parts = (ld >= 16 * MW_ ? MW_ : 8) >> ntl;
            const int t = wave & (nt2 - 1), kp = wave >> ntl;
            const int per = (nst + parts - 1) / parts;
            const int s0 = kp * per, s1 = s0 + per < nst ? s0 + per : nst;
            v4f acc[2][RT];
            const float inv_n = 1.0f / (float)N;
            auto row_of = [&](int idx) { return (int)(((float)idx + 0.5f) * inv_n); };
            float b0 = 0.0f;  // the bias of this thread's first output, requested in front of the weights
            if (bias && tid < vrows * N) b0 = bias[tid - row_of(tid) * N];
            if (t < tiles && kp < parts) {
                run(std::integral_constant<int, 1>{}, t, s0, s1, acc);
                v4f* p4 = (v4f*)xout;
#pragma unroll
                for (int r = 0; r < RT; ++r) p4[(wave * RT + r) * 64 + lane] = acc[0][r];
            }
            lds_barrier();
            for (int idx = tid; idx < vrows * N; idx += MT_) {
                const int m = row_of(idx), n = idx - m * N;
                const float* src = xout + ((((n >> 4) * RT + (m >> 4)) * 64 + ((n >> 2) & 3) * 16 + (m & 15)) << 2) + (n & 3);
                float y = 0.0f;
                for (int k = 0; k < parts; ++k) y += src[(k << ntl) * RT * 256];
                if (bias) y += idx == tid ? b0 : bias[n];
                if (a.head == AQ_HEAD_ARGMAX) xin[m * ld + n] = y;
                else ((float*)c.actions)[(row0 + m) * N + n] = head_value(y, a.head);
            }
        } else {
            float lo = INFINITY, hi = -INFINITY;
            const bool ln = !last && act == AQ_ACT_LN_TANH, relu = !last && act == AQ_ACT_RELU;
            // a tile's biases, requested in front of its weights: behind the products they were a round trip per layer
            // (of two row tiles behind them as before: eight registers more and the loop over K spills)
            auto bias4 = [&](int t) __attribute__((always_inline)) {
                const int n = t * 16 + 4 * g;
                v4f b = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                if (bias) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) b[i] = bias[n + i < N ? n + i : N - 1];
                }
                return b;
            };
            auto store = [&](const v4f& s, const v4f& b, int t, int r) __attribute__((always_inline)) {
                const int n = t * 16 + 4 * g, m = r * 16 + i16;
                v4f v = s;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (n + i < N) {
                        if (bias) v[i] += b[i];
                        if (relu) v[i] = v[i] > 0.0f ? v[i] : 0.0f;
                        if (!ln && m < vrows) {
                            lo = fminf(lo, v[i]);
                            hi = fmaxf(hi, v[i]);
                        }
                    } else {
                        v[i] = 0.0f;
                    }
                }
                *(v4f*)(xout + m * ld + n) = v;
            };
            v4f acc[2][RT];
            int t = wave;
            for (; t + MW_ < tiles; t += 2 * MW_) {
                v4f b0, b1;
                if (RT == 1) b0 = bias4(t), b1 = bias4(t + MW_);
                run(std::integral_constant<int, 2>{}, t, 0, nst, acc);
                if (RT != 1) b0 = bias4(t), b1 = bias4(t + MW_);
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    store(acc[0][r], b0, t, r);
                    store(acc[1][r], b1, t + MW_, r);
                }
            }
            if (t < tiles) {
                const v4f b0 = bias4(t);
                run(std::integral_constant<int, 1>{}, t, 0, nst, acc);
#pragma unroll
                for (int r = 0; r < RT; ++r) store(acc[0][r], b0, t, r);
            }
            // LayerNorm of 129 to 64 LNV features: gains, offsets and the row in registers, the former requested in front of the
            // barrier (in the loop over features behind it, each of its turns waited for its own two).  111-400-300-8 on
            // 3001 rows, biases and LayerNorm together: 24.0 -> 23.5 us.  Fewer features are one or two turns of that loop: held, a
            // whole policy took up to 4 % longer with 64 of them, 2 % with 128.
            constexpr int LNV = 8;
            const bool held = ln && N > 128 && N <= 64 * LNV;
            float gv[LNV], bv[LNV];
            if (held) {
                const gf_ptr gam = (gf_ptr)P.gamma[l], bet = (gf_ptr)P.beta[l];
#pragma unroll
                for (int i = 0; i < LNV; ++i) {
                    const int n = lane + 64 * i < N ? lane + 64 * i : N - 1;
                    gv[i] = 1.0f;
                    bv[i] = 0.0f;
                    if (64 * i < N) {
                        if (gam) gv[i] = gam[n];
                        if (bet) bv[i] = bet[n];
                    }
                }
            }
            if (ln || last) lds_barrier();
            if (held) {  // biased variance, eps inside the root; a wave per row
                for (int m = wave; m < ROWS; m += MW_) {
                    float* xr = xout + m * ld;
                    float x[LNV], s = 0.0f;
#pragma unroll
                    for (int i = 0; i < LNV; ++i) {
                        x[i] = 0.0f;
                        if (lane + 64 * i < N) x[i] = xr[lane + 64 * i];
                    }
#pragma unroll
                    for (int i = 0; i < LNV; ++i) s += x[i];
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
                    const float mean = s / (float)N;
                    float ss = 0.0f;
#pragma unroll
                    for (int i = 0; i < LNV; ++i) {
                        const float d = lane + 64 * i < N ? x[i] - mean : 0.0f;
                        ss += d * d;
                    }
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
                    const float rs = 1.0f / sqrtf(ss / (float)N + a.ln_eps);
#pragma unroll
                    for (int i = 0; i < LNV; ++i) {
                        if (64 * i >= N) continue;  // (scalar)
                        const float v = tanhf((x[i] - mean) * rs * gv[i] + bv[i]);
                        if (lane + 64 * i < N) {
                            xr[lane + 64 * i] = v;
                            if (m < vrows) {
                                lo = fminf(lo, v);
                                hi = fmaxf(hi, v);
                            }
                        }
                    }
                }
            } else if (ln) {
                const gf_ptr gam = (gf_ptr)P.gamma[l], bet = (gf_ptr)P.beta[l];
                for (int m = wave; m < ROWS; m += MW_) {
                    float* xr = xout + m * ld;
                    float s = 0.0f;
                    for (int n = lane; n < N; n += 64) s += xr[n];
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
                    const float mean = s / (float)N;
                    float ss = 0.0f;
                    for (int n = lane; n < N; n += 64) {
                        const float d = xr[n] - mean;
                        ss += d * d;
                    }
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
                    const float rs = 1.0f / sqrtf(ss / (float)N + a.ln_eps);
                    for (int n = lane; n < N; n += 64) {
                        const float v = tanhf((xr[n] - mean) * rs * (gam ? gam[n] : 1.0f) + (bet ? bet[n] : 0.0f));
                        xr[n] = v;
                        if (m < vrows) {
                            lo = fminf(lo, v);
                            hi = fmaxf(hi, v);
                        }
                    }
                }
            }
            if (last) {
                if (a.head == AQ_HEAD_ARGMAX) {  // (scanned below, from the other buffer)
                    float* tmp = xin;
                    xin = xout;
                    xout = tmp;
                } else {
                    const float inv_n = 1.0f / (float)N;
                    for (int idx = tid; idx < vrows * N; idx += MT_) {
                        const int m = (int)(((float)idx + 0.5f) * inv_n), n = idx - m * N;
                        ((float*)c.actions)[(row0 + m) * N + n] = head_value(xout[m * ld + n], a.head);
                    }
                }
            } else if (c.slots) {
                range_note(c.slots + (l + 1) * kRangeSlots, who, lo, hi);
            }
        }
        if (last && a.head == AQ_HEAD_ARGMAX) {
            lds_barrier();
            if (tid < vrows) {
                const float* yr = xin + tid * ld;
                int best = 0;
                for (int n = 1; n < N; ++n)
                    if (yr[n] > yr[best]) best = n;
                ((int32_t*)c.actions)[row0 + tid] = best;
            }
        }
        float* tmp = xin;
        xin = xout;
        xout = tmp;
    }
}

// LayerNorm (biased variance, eps inside the root) + tanh in place (layers that run on their own), rows in registers (ln_rows.hpp)
template <int W, int P, bool VEC>
__global__ __launch_bounds__(256) void k_fp32_ln_tanh(float* __restrict__ x, int64_t rows, int N,
                                                      const float* __restrict__ gamma, const float* __restrict__ beta,
                                                      float eps, RangeSlot* __restrict__ slots) {
    using Row = LnRow<W, P>;
    __shared__ float red[2][4];
    const int t = threadIdx.x & (Row::T - 1);
    const int64_t row = W == 1 ? (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6) : (int64_t)blockIdx.x;
    if (row >= rows) return;  // (a whole wavefront, or nobody)
    float* const xr = x + row * N;
    Row r;
    float gg[P][4], bb[P][4];
#pragma unroll
    for (int i = 0; i < P; ++i) Row::template load<VEC>(xr, t, i, N, 0.0f, r.v[i]);
#pragma unroll
    for (int i = 0; i < P; ++i) {
        Row::template load<VEC>(gamma, t, i, N, 1.0f, gg[i]);
        Row::template load<VEC>(beta, t, i, N, 0.0f, bb[i]);
    }
    float mean, inv;
    r.template stats<VEC>(t, N, eps, red, mean, inv);
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        float o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] = tanhf((r.v[i][j] - mean) * inv * gg[i][j] + bb[i][j]);
            const int n = Row::template at<VEC>(t, i, j);
            if (n < N) {
                lo = fminf(lo, o[j]);
                hi = fmaxf(hi, o[j]);
                if (!VEC) xr[n] = o[j];
            }
        }
        if (VEC && Row::template at<true>(t, i, 0) < N) *(float4*)(xr + Row::template at<true>(t, i, 0)) = make_float4(o[0], o[1], o[2], o[3]);
    }
    if (slots) range_note(slots, W == 1 ? (uint32_t)row : (uint32_t)row * 4 + (threadIdx.x >> 6), lo, hi);
}

// rows longer than those hold, or too many for them (ln_form): one wavefront per row, which is read three times
__global__ __launch_bounds__(256) void k_fp32_ln_tanh_long(float* __restrict__ x, int64_t rows, int N,
                                                      const float* __restrict__ gamma, const float* __restrict__ beta,
                                                      float eps, RangeSlot* __restrict__ slots) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    float* xr = x + row * N;
    float s = 0.0f;
    for (int n = lane; n < N; n += 64) s += xr[n];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    const float mean = s / (float)N;
    float ss = 0.0f;
    for (int n = lane; n < N; n += 64) {
        float d = xr[n] - mean;
        ss += d * d;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
    const float inv = 1.0f / sqrtf(ss / (float)N + eps);
    float lo = INFINITY, hi = -INFINITY;
    for (int n = lane; n < N; n += 64) {
        float g = gamma ? gamma[n] : 1.0f, b = beta ? beta[n] : 0.0f;
        const float v = tanhf((xr[n] - mean) * inv * g + b);
        xr[n] = v;
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
    }
    if (slots) range_note(slots, (uint32_t)row, lo, hi);
}

__global__ void k_fp32_argmax(const float* __restrict__ y, int64_t rows, int N, int32_t* __restrict__ actions) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows) return;
    const float* yr = y + i * N;
    int best = 0;
    for (int n = 1; n < N; ++n)
        if (yr[n] > yr[best]) best = n;
    actions[i] = best;
}

// range of the network input: 16 bytes per load where the buffer is aligned, the ends one by one
__global__ __launch_bounds__(256) void k_input_range(const void* __restrict__ x, int is_u8, int64_t n, RangeSlot* __restrict__ slots) {
    float lo = INFINITY, hi = -INFINITY;
    const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, stride = (int64_t)gridDim.x * 256;
    const int per = is_u8 ? 16 : 4;
    const int64_t whole = ((uintptr_t)x & 15) == 0 ? n / per : 0;
#pragma unroll 4
    for (int64_t i = first; i < whole; i += stride) {
        const uint4 q = ((const uint4*)x)[i];
        const uint32_t d[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (is_u8) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float v = (float)((d[j] >> (8 * k)) & 255u);
                    lo = fminf(lo, v);
                    hi = fmaxf(hi, v);
                }
            } else {
                const float v = __uint_as_float(d[j]);
                lo = fminf(lo, v);
                hi = fmaxf(hi, v);
            }
        }
    }
    for (int64_t i = whole * per + first; i < n; i += stride) {
        const float v = is_u8 ? (float)((const uint8_t*)x)[i] : ((const float*)x)[i];
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
    }
    range_note(slots, blockIdx.x * 4 + (threadIdx.x >> 6), lo, hi);
}

// Reduces every tensor's slots to (min, max) and leaves the slots neutral for the next calibration.  `ready`, if
// given, is host memory: it is set once the ranges are there.
__global__ __launch_bounds__(64 * AQ_MAX_LAYERS) void k_ranges_out(RangeSlot* __restrict__ slots, int n, float* __restrict__ out,
                                                                   uint32_t* __restrict__ ready, uint32_t ticket) {
    const int t = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (t < n) {
        RangeSlot* s = slots + t * kRangeSlots;
        RangeSlot v[kRangeSlots / 64];
#pragma unroll
        for (int i = 0; i < kRangeSlots / 64; ++i) v[i] = s[lane + 64 * i];
        uint32_t nlo = 0u, hi = 0u;
#pragma unroll
        for (int i = 0; i < kRangeSlots / 64; ++i) {
            nlo = nlo > v[i].not_lo ? nlo : v[i].not_lo;
            hi = hi > v[i].hi ? hi : v[i].hi;
            s[lane + 64 * i] = RangeSlot{0u, 0u};
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t l2 = (uint32_t)__shfl_xor((int)nlo, o, 64), h2 = (uint32_t)__shfl_xor((int)hi, o, 64);
            nlo = nlo > l2 ? nlo : l2;
            hi = hi > h2 ? hi : h2;
        }
        if (lane == 0) {
            out[2 * t] = key2f(~nlo);
            out[2 * t + 1] = key2f(hi);
        }
    }
    if (ready) {
        __threadfence_system();
        __syncthreads();
        if (threadIdx.x == 0) __hip_atomic_store(ready, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// The learner's parameters -> the handle's copies, every array of every layer in one launch: workgroup -> array and
// piece of it by the table; an absent source is its default value.  (As one copy or fill per array this was 15 to 20
// launches of 2.6 us.)  Per layer: weights row-major (the quantizer reads them), bias, gain, offset, and the weights in
// the operand order of the kernels above (all that is written of parameters passed with a call).
__global__ __launch_bounds__(256) void k_keep_params(const F32Ptrs src, const F32KeepTab* __restrict__ tab, char* __restrict__ to) {
    const int blk = (int)blockIdx.x;
    // the last array that starts at or before this workgroup (5 * AQ_MAX_LAYERS + 4 <= 64: one lane each)
    const int lane = threadIdx.x & 63;
    const uint64_t before = __ballot(lane < tab->n && blk >= tab->blk0[lane < tab->n ? lane : 0]);
    const int a = __builtin_amdgcn_readfirstlane(63 - __builtin_clzll(before));
    const int kind = tab->e[a].kind, l = tab->e[a].layer;
    const int64_t n = tab->e[a].count, base = (int64_t)(blk - tab->blk0[a]) * kKeepPiece;
    const float* s = kind == 1 ? src.b[l] : kind == 2 ? src.gamma[l] : kind == 3 ? src.beta[l] : src.w[l];
    float AQ_GLOBAL* d = (float AQ_GLOBAL*)(to + tab->e[a].off);
    if (kind == 4) {  // 16 blocks of 16 features x 16 k
        const int N = tab->e[a].N, K = tab->e[a].K, nst = (K + 15) >> 4;
        const int i16 = lane & 15, g = lane >> 4;
        const uint32_t nblk = (uint32_t)(n / 256);
        const bool al = (K & 3) == 0 && ((uintptr_t)s & 15) == 0;
        v4f v[kKeepPiece / 1024];
#pragma unroll
        for (int i = 0; i < kKeepPiece / 1024; ++i) {
            // (neighbouring lanes take neighbouring pieces of one row: the rows' order is restored on the way out)
            const uint32_t q = (uint32_t)(base / 256) + i * 4 + (threadIdx.x >> 6);  // block
            const int t = (int)(q / (uint32_t)nst), st = (int)(q - (uint32_t)t * (uint32_t)nst);
            const int n_ = t * 16 + (lane >> 2), k = st * 16 + (lane & 3) * 4;
            v[i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
            if (q < nblk && n_ < N && k < K) {
                const float* p = s + (int64_t)n_ * K + k;
                if (al) {
                    v[i] = *(const v4f AQ_GLOBAL*)p;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (k + j < K) v[i][j] = p[j];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kKeepPiece / 1024; ++i) {
            const uint32_t q = (uint32_t)(base / 256) + i * 4 + (threadIdx.x >> 6);
            v4f w;
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = __shfl(v[i][j], i16 * 4 + g, 64);
            if (q < nblk) *(v4f AQ_GLOBAL*)(d + (int64_t)q * 256 + lane * 4) = w;
        }
        return;
    }
    if (kind == 5) {  // kKeepSplit blocks of 16 features x 32 k, each value as three bf16 parts; then a word per block
        const int N = tab->e[a].N, K = tab->e[a].K, nst = (K + 31) >> 5, nblk = (N + 15) / 16 * nst;
        const int i16 = lane & 15, g = lane >> 4;
        const bool al = (K & 3) == 0 && ((uintptr_t)s & 15) == 0;
        v4f v[kKeepSplit / 4][2];
#pragma unroll
        for (int i = 0; i < kKeepSplit / 4; ++i) {
            const int q = (blk - tab->blk0[a]) * kKeepSplit + i * 4 + (threadIdx.x >> 6);
            const int t = q / nst, n_ = t * 16 + (lane >> 2), k = (q - t * nst) * 32 + (lane & 3) * 8;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v[i][h] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                if (q < nblk && n_ < N) {
                    const float* p = s + (int64_t)n_ * K + k + 4 * h;
                    if (al && k + 4 * h < K) {
                        v[i][h] = *(const v4f AQ_GLOBAL*)p;
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (k + 4 * h + j < K) v[i][h][j] = p[j];
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kKeepSplit / 4; ++i) {
            const int q = (blk - tab->blk0[a]) * kKeepSplit + i * 4 + (threadIdx.x >> 6);
            bool odd = false;
#pragma unroll
            for (int j = 0; j < 8; ++j) odd |= split_special(v[i][j >> 2][j & 3]);
            bf8 x[3];
            split8(v[i][0], v[i][1], x);
            const uint64_t any = __ballot(odd);
#pragma unroll
            for (int part = 0; part < 3; ++part) {
                const v4i from = __builtin_bit_cast(v4i, x[part]);
                v4i w;
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = __shfl(from[j], i16 * 4 + g, 64);
                if (q < nblk) *(v4i AQ_GLOBAL*)((char AQ_GLOBAL*)d + (int64_t)q * 3072 + part * 1024 + lane * 16) = w;
            }
            if (q < nblk && lane == 0) ((uint32_t AQ_GLOBAL*)d)[(int64_t)nblk * 768 + q] = any != 0;
        }
        return;
    }
    const float fill = kind == 2 ? 1.0f : 0.0f;
    const int64_t end = base + kKeepPiece < n ? base + kKeepPiece : n;
    if (s && ((uintptr_t)s & 15) == 0 && end - base == kKeepPiece) {
        const v4f AQ_GLOBAL* s4 = (const v4f AQ_GLOBAL*)(s + base);
        v4f AQ_GLOBAL* d4 = (v4f AQ_GLOBAL*)(d + base);
        v4f v[kKeepPiece / 1024];
#pragma unroll
        for (int i = 0; i < kKeepPiece / 1024; ++i) v[i] = s4[threadIdx.x + 256 * i];
#pragma unroll
        for (int i = 0; i < kKeepPiece / 1024; ++i) d4[threadIdx.x + 256 * i] = v[i];
    } else {
        for (int64_t i = base + threadIdx.x; i < end; i += 256) d[i] = s ? s[i] : fill;
    }
}

// ------------------------------------------------------------------------------------------------- launches
namespace {
// The compiled tiles: FT, RT, WN, WM, WK, KS of k_fp32_layer.
struct TileShape {
    int ft, rt, wn, wm, wk, ks;
};
constexpr TileShape kTiles[] = {
    {2, 2, 2, 4, 1, 4},  // 64 features x 128 rows
    {2, 2, 1, 4, 2, 2},  // 32 x 128: narrow layers
    {2, 2, 2, 2, 2, 2},  // 64 x 64, K in two
    {2, 2, 1, 1, 8, 2},  // 32 x 32, K in eight
    {1, 2, 1, 1, 8, 2},  // 16 x 32
    {1, 1, 1, 1, 8, 4},  // 16 x 16: few rows
};
constexpr int kNTiles = sizeof(kTiles) / sizeof(kTiles[0]);
// The cheapest of them by the clocks a CU's matrix cores are busy (32 per MFMA, two of the eight waves on each SIMD), in
// whole rounds of one workgroup per CU, plus what a workgroup spends before its first and behind its last MFMA.
int pick_tile(const Fp32Layer& L, int64_t rows) {
    int best = 0;
    double best_c = 1e300;
    const int64_t nst = (L.K + 15) / 16;
    for (int i = 0; i < kNTiles; ++i) {
        const TileShape& t = kTiles[i];
        const int64_t bn = 16 * t.ft * t.wn, bm = 16 * t.rt * t.wm, bs = t.ks * t.wk;
        const int64_t ny = (L.N + bn - 1) / bn, nx = (rows + bm - 1) / bm;
        if (ny > 65535 || !grid_ok(nx, FT_)) continue;
        const double stages = (double)((nst + bs - 1) / bs);
        const double per = stages * (t.ks * t.ft * t.rt * 256.0 + 150.0) + (t.wk > 1 ? 1200.0 : 600.0);
        const double c = (double)((nx * ny + 255) / 256) * per + 1500.0;
        if (c < best_c) {
            best_c = c;
            best = i;
        }
    }
    return best;
}
// Workgroups that follow each other go to the eight XCDs in turn, so the faster grid dimension decides what an XCD's L2 must
// hold: all of the other dimension's operand and an eighth of its own.  The larger operand takes the faster one.
dim3 layer_grid(Fp32Layer& L, int64_t nx, int64_t ny, int64_t rows) {
    const double w = 4.0 * L.K * L.N, x = 4.0 * (double)rows * L.K;
    L.features_first = w > x && nx <= 65535;
    return L.features_first ? dim3((unsigned)ny, (unsigned)nx) : dim3((unsigned)nx, (unsigned)ny);
}
template <int I, bool CONV, bool U8>
aq_status launch_tile(Fp32Layer L, const void* in, float* out, int64_t rows, RangeSlot* slots, hipStream_t st) {
    constexpr TileShape t = kTiles[I];
    const dim3 grid = layer_grid(L, (rows + 16 * t.rt * t.wm - 1) / (16 * t.rt * t.wm), (L.N + 16 * t.ft * t.wn - 1) / (16 * t.ft * t.wn), rows);
    auto* const kernel = k_fp32_layer<t.ft, t.rt, t.wn, t.wm, t.wk, t.ks, CONV, U8>;
    constexpr size_t lds = fp32_layer_lds(t.ft, t.rt, t.wm, t.wk, t.ks);
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
        if (hip_failed(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds))) return AQ_EHIP;
        attr_set = true;
    }
    hipLaunchKernelGGL(kernel, grid, dim3(FT_), lds, st, L, in, out, rows, slots);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}
template <int I>
aq_status launch_tile_kind(const Fp32Layer& L, bool fc, int in_u8, const void* in, float* out, int64_t rows, RangeSlot* slots, hipStream_t st) {
    if constexpr (kTiles[I].wk == FW_) {
        constexpr TileShape t = kTiles[I];
        if (fc) {
            Fp32Layer q = L;
            const dim3 grid = layer_grid(q, (rows + 16 * t.rt - 1) / (16 * t.rt), (L.N + 16 * t.ft - 1) / (16 * t.ft), rows);
            if (in_u8) hipLaunchKernelGGL((k_fp32_rows<t.ft, t.rt, true>), grid, dim3(FT_), 0, st, q, in, out, rows, slots);
            else hipLaunchKernelGGL((k_fp32_rows<t.ft, t.rt, false>), grid, dim3(FT_), 0, st, q, in, out, rows, slots);
            return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
        }
        return in_u8 ? launch_tile<I, true, true>(L, in, out, rows, slots, st) : launch_tile<I, true, false>(L, in, out, rows, slots, st);
    }
    if (fc) return in_u8 ? launch_tile<I, false, true>(L, in, out, rows, slots, st) : launch_tile<I, false, false>(L, in, out, rows, slots, st);
    return in_u8 ? launch_tile<I, true, true>(L, in, out, rows, slots, st) : launch_tile<I, true, false>(L, in, out, rows, slots, st);
}
}  // namespace

void fp32_layer_tile(const Fp32Layer& L, int64_t rows, int* features, int* tile_rows) {
    const TileShape& t = kTiles[pick_tile(L, rows)];
    *features = 16 * t.ft * t.wn;
    *tile_rows = 16 * t.rt * t.wm;
}

aq_status launch_fp32_layer(const Fp32Layer& L, const void* in, int in_u8, float* out, int64_t rows, RangeSlot* slots,
                            hipStream_t st) {
    const bool fc = L.kh == 1 && L.kw == 1 && L.in_h == 1 && L.in_w == 1;
    switch (pick_tile(L, rows)) {
        case 0: return launch_tile_kind<0>(L, fc, in_u8, in, out, rows, slots, st);
        case 1: return launch_tile_kind<1>(L, fc, in_u8, in, out, rows, slots, st);
        case 2: return launch_tile_kind<2>(L, fc, in_u8, in, out, rows, slots, st);
        case 3: return launch_tile_kind<3>(L, fc, in_u8, in, out, rows, slots, st);
        case 4: return launch_tile_kind<4>(L, fc, in_u8, in, out, rows, slots, st);
        default: return launch_tile_kind<5>(L, fc, in_u8, in, out, rows, slots, st);
    }
}

namespace {
size_t mlp_lds(int rt, int ld) { return (size_t)2 * 16 * rt * ld * 4; }
int mlp_ld(const NetDev& n) {
    int w = 128;
    for (int l = 0; l < n.n_layers; ++l) {
        const LayerDev& L = n.L[l];
        const int k = (L.K + 15) & ~15, o = (L.N + 15) & ~15;
        w = w > k ? w : k;
        w = w > o ? w : o;
    }
    return w + 4;
}
}  // namespace

// Whether the whole MLP goes in one launch: its two activation buffers must fit LDS, and a workgroup streams every
// weight, so at batches that leave most CUs idle the layers' own launches win once the weights are large.
bool fp32_mlp_fits(const NetDev& n, int64_t batch, int* rt_out) {
    double wbytes = 0.0;
    for (int l = 0; l < n.n_layers; ++l) {
        const LayerDev& L = n.L[l];
        if (L.kh != 1 || L.kw != 1 || L.in_h != 1 || L.in_w != 1) return false;
        wbytes += 4.0 * L.K * L.N;
    }
    const int ld = mlp_ld(n);
    if (mlp_lds(1, ld) > 160 * 1024) return false;
    // (two row tiles from the second round of single ones on: 256-wide policies at 4100 to 8192 rows take 0.76 of the time, up to 4096
    // 1.5 times as long)
    const int rt = batch > 16 * 256 && mlp_lds(2, ld) <= 80 * 1024 ? 2 : 1;
    *rt_out = rt;
    const int64_t workgroups = (batch + 16 * rt - 1) / (16 * rt);
    if (!grid_ok(workgroups, MT_)) return false;
    // clocks: one launch (weights at 40 B per clock and CU, or 32 per MFMA and SIMD) against a launch per layer
    const double rounds = (double)((workgroups + 255) / 256);
    const double mm = wbytes / 4.0 / 1024.0 * rt * 128.0 / 4.0, mem = wbytes / 40.0;
    const double fused = rounds * (mm > mem ? mm : mem);
    const double flops = wbytes / 2.0 * (double)batch;
    const double layers = 7000.0 * n.n_layers + flops / (256.0 * 256.0 * 0.6) + wbytes / 2000.0;
    return fused <= layers;
}

aq_status launch_fp32_mlp(const NetDev& n, const NetDev* d_net, const F32Ptrs& ptrs, const F32Ptrs* d_ptrs, const void* obs,
                          int64_t batch, void* actions, RangeSlot* slots, int rt, hipStream_t st) {
    F32Call c{};
    c.obs = obs;
    c.actions = actions;
    c.batch = batch;
    c.slots = slots;
    c.ld = mlp_ld(n);
    const size_t lds = mlp_lds(rt, c.ld);
    const dim3 grid((unsigned)((batch + 16 * rt - 1) / (16 * rt)));
#define AQ_MLP(RTV, U, BV)                                                                                              \
    do {                                                                                                                \
        static std::atomic<bool> attr_set{false};                                                                       \
        if (!attr_set) {                                                                                                \
            if (hip_failed(hipFuncSetAttribute((const void*)k_fp32_mlp<RTV, U, BV>,                                     \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)))                \
                return AQ_EHIP;                                                                                         \
            attr_set = true;                                                                                            \
        }                                                                                                               \
        hipLaunchKernelGGL((k_fp32_mlp<RTV, U, BV>), grid, dim3(MT_), lds, st, d_net, c, F32PtrArg<BV>(ptrs, d_ptrs));   \
    } while (0)
#define AQ_MLP_U(RTV, U)                 \
    do {                                 \
        if (d_ptrs) AQ_MLP(RTV, U, false); \
        else AQ_MLP(RTV, U, true);       \
    } while (0)
    if (rt == 2) {
        if (n.in_u8) AQ_MLP_U(2, true);
        else AQ_MLP_U(2, false);
    } else {
        if (n.in_u8) AQ_MLP_U(1, true);
        else AQ_MLP_U(1, false);
    }
#undef AQ_MLP_U
#undef AQ_MLP
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_fp32_ln_tanh(float* x, int64_t rows, int N, const float* gamma, const float* beta, float eps,
                              RangeSlot* slots, hipStream_t st) {
    LnForm f;
    if (!ln_form(rows, N, &f)) {
        hipLaunchKernelGGL(k_fp32_ln_tanh_long, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, x, rows, N, gamma, beta, eps, slots);
        return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
    }
    const bool vec = N % 4 == 0 && (((uintptr_t)x | (uintptr_t)gamma | (uintptr_t)beta) & 15) == 0;
    const dim3 grid((unsigned)(f.w == 1 ? (rows + 3) / 4 : rows));
    ln_dispatch(f, [&](auto w, auto p) {
        constexpr int W = decltype(w)::value, P = decltype(p)::value;
        auto go = [&](auto k) { hipLaunchKernelGGL(k, grid, dim3(256), 0, st, x, rows, N, gamma, beta, eps, slots); };
        if (vec) go(k_fp32_ln_tanh<W, P, true>);
        else go(k_fp32_ln_tanh<W, P, false>);
    });
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_fp32_argmax(const float* y, int64_t rows, int N, int32_t* actions, hipStream_t st) {
    hipLaunchKernelGGL(k_fp32_argmax, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, st, y, rows, N, actions);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_input_range(const void* x, int is_u8, int64_t n, RangeSlot* slots, hipStream_t st) {
    int64_t g = (n / (is_u8 ? 16 : 4) + 256 * 4 - 1) / (256 * 4);
    if (g < 1) g = 1;
    if (g > 2048) g = 2048;
    hipLaunchKernelGGL(k_input_range, dim3((unsigned)g), dim3(256), 0, st, x, is_u8, n, slots);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_ranges_out(RangeSlot* slots, int n, float* out, uint32_t* ready, uint32_t ticket, hipStream_t st) {
    hipLaunchKernelGGL(k_ranges_out, dim3(1), dim3(64 * AQ_MAX_LAYERS), 0, st, slots, n, out, ready, ticket);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_keep_params(const F32Ptrs& src, const F32KeepTab* d_tab, void* base, int blocks, hipStream_t st) {
    hipLaunchKernelGGL(k_keep_params, dim3((unsigned)blocks), dim3(256), 0, st, src, d_tab, (char*)base);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

}  // namespace aq

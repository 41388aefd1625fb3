// Half-precision actor (Sec. 3.2: fp16 policies; actors at q = 16): a whole fully connected policy in one launch.
//
// One workgroup of 8 wavefronts owns 16 RT batch rows (RT = 1, 2 or 4) from the observation to the action.  The rows'
// activations live in one LDS buffer that every layer overwrites in place: a layer's outputs stay in accumulators until
// all wavefronts have read its inputs.  That is what lets 64 rows of a 1024-wide policy (132 KB) share a CU, so that a
// weight byte feeds 64 rows.  A wavefront takes feature tiles wave, wave + 8, ... of 32 (up to four, 128 accumulator
// registers at 64 rows); weights stream from L2 through a ring of 16 operands per wavefront; a narrow last layer is
// split over K.
// v_mfma_f32_16x16x32_f16: the chip's clock under matrix load depends on the instruction.  On random operands, the loop
// alone, all CUs: 16x16x32 1790 to 1940 TFLOP/s, 32x32x16 1450 to 1640 (on zeros both 2400).  The library's 32 x 16
// weight tiles serve it unchanged: lane (i = lane % 16, g = lane / 16) of feature half h and k-step s takes piece
// h * 16 + i + 32 * (g % 2) of tile 2 s + g / 2, which holds k = 32 s + 8 g .. + 7 of feature h * 16 + i.
// Sums are fp32 over k, + bias, one rounding per operator, as in the per-layer kernels.
//
// What bounds it: at large batch the matrix cores and the CU's vector memory path together (64 rows x 1024 x 1024: 2 MiB of
// weights at 52 B per clock = 40 k clocks beside as long a run of MFMAs); at small batch the chain of layers of one
// workgroup.
#include "fp16_device.hpp"
#include "int8_device.hpp"
#include "lanes.hpp"

namespace aq {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef const h8 AQ_GLOBAL* gh8_ptr;

namespace {

__device__ __forceinline__ h8 load_operand(__amdgpu_buffer_rsrc_t w, int lane_off, int off) {
    return __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(w, lane_off, off, 0));
}

constexpr int MLW = 8;               // wavefronts per workgroup
constexpr int MLT = MLW * 64;
constexpr int MLMAXW = 1024;         // widest layer input / output
constexpr int MLY_LD = 68;           // halfs per row of a narrow head's logits (at most 64)

// k-steps (of 32) in flight when a wavefront has NB tiles, two operands each
template <int NB>
constexpr int ring_depth() {
    return NB == 1 ? 8 : NB == 2 ? 4 : 2;
}

}  // namespace

template <int RT, bool U8, bool TAPS>
__global__ __launch_bounds__(MLT) void k_fp16_mlp(const Fp16Net* __restrict__ netp, const Fp16Call c, const Fp16Taps<TAPS> tp) {
    extern __shared__ __align__(16) _Float16 sm[];
    constexpr int ROWS = 16 * RT;
    const Fp16Net& a = *netp;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int nl = a.n_layers, ld = c.ld;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int64_t left = c.batch - row0;
    const int vrows = left < ROWS ? (int)left : ROWS;
    _Float16* const xs = sm;                 // the activations
    _Float16* const cs = sm + c.off_const;   // every layer's bias, gain and offset
    float* const red = (float*)(sm + c.off_red);  // a LayerNorm's partial statistics

    // tiles of this wavefront in a layer, and where a tile's weights begin
    auto tiles_of = [&](int l) { return a.L[l].NT > wave ? (a.L[l].NT - wave + MLW - 1) / MLW : 0; };
    auto narrow = [&](int l) { return l == nl - 1 && a.L[l].NT <= 2; };
    // A layer's weights as a buffer: descriptor and tile offset in scalar registers, one 32-bit lane offset for every
    // operand.  (With a 64-bit address per lane and tile, which is what plain pointers compile to, the wide case had
    // registers for two k-steps in flight instead of four.)
    auto weights_of = [&](int l) {
        const int bytes = uni(a.L[l].NT) * uni(a.L[l].KS16) * 1024;
        return __builtin_amdgcn_make_buffer_rsrc((void*)uni_ptr(a.L[l].wp), 0, bytes, 0x00020000);
    };
    const int lane_off = (g >> 1) * 1024 + (i16 + 32 * (g & 1)) * 16;

    for (int i = tid; i < a.cst / 8; i += MLT) ((h8*)cs)[i] = ((gh8_ptr)a.consts)[i];
    {   // Observations, rounded; zeros behind the row ends (up to whole k-steps) and past the batch.  Eight requests per
        // thread are in flight at a time, four values each where the rows allow it (one at a time, 64 rows of 256 took 8 us).
        const int K = a.L[0].K, K32 = (K + 31) & ~31;
        constexpr int U = 8;
        auto stage = [&](auto w_c) __attribute__((always_inline)) {
            constexpr int W = decltype(w_c)::value;  // values per request
            const int cols = K32 / W, total = ROWS * cols;
            const float inv = 1.0f / (float)cols;
            for (int base = tid; base < total; base += U * MLT) {
                v4f v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int idx = base + u * MLT;
                    const int m = (int)(((float)idx + 0.5f) * inv), k = (idx - m * cols) * W;
                    v[u] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                    if (idx < total && m < vrows && k < K) {
                        const int64_t off = (row0 + m) * K + k;
                        if (W == 1) v[u][0] = U8 ? (float)((const uint8_t*)c.obs)[off] : ((const float*)c.obs)[off];
                        else if (!U8) v[u] = *(const v4f*)((const float*)c.obs + off);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int idx = base + u * MLT;
                    const int m = (int)(((float)idx + 0.5f) * inv), k = (idx - m * cols) * W;
                    if (idx >= total) break;
                    if (W == 1) {
                        xs[m * ld + k] = (_Float16)v[u][0];
                    } else {
                        h4 o;
#pragma unroll
                        for (int j = 0; j < 4; ++j) o[j] = (_Float16)v[u][j];
                        *(h4*)(xs + m * ld + k) = o;
                    }
                }
            }
        };
        if (!U8 && (K & 3) == 0 && ((uintptr_t)c.obs & 15) == 0) stage(std::integral_constant<int, 4>{});
        else stage(std::integral_constant<int, 1>{});
    }
    const _Float16* const xrow = xs + i16 * ld + 8 * g;

    // One layer for a wavefront with NB tiles.  (The accumulators live inside this one block: with the k-loop and the
    // epilogue in separate switches over NB the compiler spilled hundreds of registers.  At 64 rows it still spills 36 or
    // 37: 128 accumulators, the ring of operands and the rows' operands share 256.)
    auto layer_nb = [&](auto nb_c, int l) __attribute__((always_inline)) {
        constexpr int NB = decltype(nb_c)::value, PF = ring_depth<NB>();
        const int ks = (uni(a.L[l].K) + 31) >> 5;
        const auto w = weights_of(l);
        const int w0 = wave * uni(a.L[l].KS16) * 1024, step = MLW * uni(a.L[l].KS16) * 1024;
        v4f acc[2 * NB][RT];
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i)
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[i][r] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        // (the first ones requested in front of the barrier that completes the layer's inputs)
        h8 ring[PF][2 * NB];
        auto fetch = [&](auto p_c, int k) __attribute__((always_inline)) {
            constexpr int p = decltype(p_c)::value;
#pragma unroll
            for (int i = 0; i < 2 * NB; ++i)
                ring[p][i] = load_operand(w, lane_off + 256 * (i & 1), w0 + (i >> 1) * step + k * 2048);
        };
        static_for<0, PF>([&](auto p_c) __attribute__((always_inline)) {
            if (decltype(p_c)::value < ks) fetch(p_c, decltype(p_c)::value);
        });
        lds_barrier();  // this layer's inputs (and the constants) are in LDS
        h8 x[RT];  // a row tile's operand of the next k-step is read as soon as this k-step's MFMAs with it are issued
#pragma unroll
        for (int r = 0; r < RT; ++r) x[r] = *(const h8*)(xrow + r * 16 * ld);
        auto one = [&](auto p_c, int s) __attribute__((always_inline)) {
            constexpr int p = decltype(p_c)::value;
            const _Float16* const nx = xrow + (s + p + 1 < ks ? s + p + 1 : s + p) * 32;
#pragma unroll
            for (int r = 0; r < RT; ++r) {
#pragma unroll
                for (int i = 0; i < 2 * NB; ++i)
                    acc[i][r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ring[p][i], x[r], acc[i][r], 0, 0, 0);
                x[r] = *(const h8*)(nx + r * 16 * ld);
            }
        };
        // Whole groups of PF k-steps as straight-line code.  The last ones request nothing (a request past the end would
        // still take its 16 clocks of the memory path), the one in front of a partial group only what is left.
        int s = 0;
        for (; s + 2 * PF <= ks; s += PF) {
            static_for<0, PF>([&](auto p_c) __attribute__((always_inline)) {
                one(p_c, s);
                fetch(p_c, s + decltype(p_c)::value + PF);
                asm volatile("" ::: "memory");
            });
        }
        if (s + PF < ks) {
            static_for<0, PF>([&](auto p_c) __attribute__((always_inline)) {
                one(p_c, s);
                if (s + decltype(p_c)::value + PF < ks) fetch(p_c, s + decltype(p_c)::value + PF);
                asm volatile("" ::: "memory");
            });
            s += PF;
        }
        static_for<0, PF>([&](auto p_c) __attribute__((always_inline)) {
            if (s + decltype(p_c)::value < ks) one(p_c, s);
        });
        const int N = uni(a.L[l].N), act = l < nl - 1 ? uni(a.L[l].act) : AQ_ACT_NONE;
        const _Float16* const bias = cs + a.L[l].c_off;
        auto n0_of = [&](int i) { return (wave + MLW * (i >> 1)) * 32 + 16 * (i & 1) + 4 * g; };
        if (__builtin_expect(act != AQ_ACT_LN_TANH, 1)) {
            lds_barrier();  // all inputs read: the outputs take their place
            const bool relu = act == AQ_ACT_RELU;
#pragma unroll
            for (int i = 0; i < 2 * NB; ++i) {
                const h4 b4 = *(const h4*)(bias + n0_of(i));
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    h4 o;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        _Float16 v = (_Float16)(acc[i][r][j] + (float)b4[j]);
                        if (relu) v = v > (_Float16)0.0f ? v : (_Float16)0.0f;
                        o[j] = v;
                    }
                    *(h4*)(xs + (r * 16 + i16) * ld + n0_of(i)) = o;
                }
            }
            return;
        }
        // LayerNorm (biased variance, eps inside the root) of the rounded outputs, rounded, then tanh, rounded.  The values stay in
        // the accumulators; a wavefront's features give (sum, squared deviations from their own mean) per row, and the wavefronts'
        // pairs meet by the pairwise update (Chan, Golub, LeVeque) over the barrier that frees the inputs.  (Through LDS, a wavefront
        // a row at a time with twelve lane exchanges each: 19-125-102-34 at 9785 rows 21.9 us.)
        const int NT = uni(a.L[l].NT);
        auto count_of = [&](int w) {
            const int tiles = NT > w ? (NT - w + MLW - 1) / MLW : 0;
            return 32 * tiles - (((NT - 1) & (MLW - 1)) == w ? NT * 32 - N : 0);
        };
        const float inv_nw = 1.0f / (float)count_of(wave);  // (of a wavefront with a tile: at least one feature)
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i) {
            const h4 b4 = *(const h4*)(bias + n0_of(i));
#pragma unroll
            for (int r = 0; r < RT; ++r) {
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][r][j] = (float)(_Float16)(acc[i][r][j] + (float)b4[j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            float s = 0.0f, q = 0.0f;
#pragma unroll
            for (int i = 0; i < 2 * NB; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (i < 2 * NB - 2 || n0_of(i) + j < N) s += acc[i][r][j];  // (only a wavefront's last tile has padding)
            s = sum_rows4(s);
            const float mean_w = s * inv_nw;
#pragma unroll
            for (int i = 0; i < 2 * NB; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float d = acc[i][r][j] - mean_w;
                    if (i < 2 * NB - 2 || n0_of(i) + j < N) q += d * d;
                }
            q = sum_rows4(q);
            if (g == 0) *(float2*)(red + ((16 * r + i16) * MLW + wave) * 2) = float2{s, q};
            __builtin_amdgcn_sched_barrier(0);
        }
        // the row's four lanes take two wavefronts' pairs each
        float cnt[2], inv_cnt[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int n = count_of(2 * g + k);
            cnt[k] = (float)n;
            inv_cnt[k] = 1.0f / (float)(n > 0 ? n : 1);
        }
        lds_barrier();  // statistics of all wavefronts; all inputs read: the outputs take their place
        float mean[RT], inv[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const float4 v = *(const float4*)(red + (16 * r + i16) * MLW * 2 + 4 * g);
            const float sw[2] = {cnt[0] > 0.0f ? v.x : 0.0f, cnt[1] > 0.0f ? v.z : 0.0f};
            const float qw[2] = {cnt[0] > 0.0f ? v.y : 0.0f, cnt[1] > 0.0f ? v.w : 0.0f};
            mean[r] = sum_rows4(sw[0] + sw[1]) / (float)N;
            const float d0 = sw[0] * inv_cnt[0] - mean[r], d1 = sw[1] * inv_cnt[1] - mean[r];
            const float m2 = sum_rows4((cnt[0] * d0 * d0 + qw[0]) + (cnt[1] * d1 * d1 + qw[1]));
            inv[r] = 1.0f / sqrtf(m2 / (float)N + a.eps);
        }
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i) {
            const h4 g4 = *(const h4*)(bias + NT * 32 + n0_of(i)), o4 = *(const h4*)(bias + 2 * NT * 32 + n0_of(i));
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                h4 o;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const _Float16 t = (_Float16)((acc[i][r][j] - mean[r]) * inv[r] * (float)g4[j] + (float)o4[j]);
                    o[j] = (_Float16)tanh_rel((float)t);
                }
                *(h4*)(xs + (r * 16 + i16) * ld + n0_of(i)) = o;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    auto tap = [&](int l) {
        if constexpr (TAPS) {
            _Float16* const d = (_Float16*)tp.p[l];
            if (!d) return;
            const int N = a.L[l].N;
            for (int idx = tid; idx < vrows * N; idx += MLT) {
                const int m = idx / N, n = idx - m * N;
                d[(row0 + m) * N + n] = xs[m * ld + n];
            }
        }
    };

    for (int l = 0; l < nl; ++l) {
        const bool last = l == nl - 1;
        const int N = a.L[l].N, NT = a.L[l].NT;
        if (narrow(l)) {
            // feature tile of 16 x K part per wavefront
            const int tiles = (N + 15) >> 4, ntl = tiles <= 1 ? 0 : tiles <= 2 ? 1 : 2, parts = MLW >> ntl;
            const int t = wave & ((1 << ntl) - 1), kp = wave >> ntl;
            const int ks = (uni(a.L[l].K) + 31) >> 5, per = (ks + parts - 1) / parts;
            const int k0 = kp * per, k1 = k0 + per < ks ? k0 + per : ks;
            v4f acc[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
            const auto w = weights_of(l);
            const int w0 = (t >> 1) * uni(a.L[l].KS16) * 1024;
            auto operand = [&](int k) { return load_operand(w, lane_off + 256 * (t & 1), w0 + k * 2048); };
            constexpr int PN = 8;
            h8 wr[PN];
            if (t < tiles) {
#pragma unroll
                for (int p = 0; p < PN; ++p)
                    if (k0 + p < k1) wr[p] = operand(k0 + p);
            }
            lds_barrier();
            if (t < tiles) {
                for (int s = k0; s < k1; s += PN) {
#pragma unroll
                    for (int p = 0; p < PN; ++p)
                        if (s + p < k1) {
                            if (s > k0) wr[p] = operand(s + p);
#pragma unroll
                            for (int r = 0; r < RT; ++r)
                                acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                                    wr[p], *(const h8*)(xrow + r * 16 * ld + (s + p) * 32), acc[r], 0, 0, 0);
                        }
                }
            }
            lds_barrier();  // all inputs read: the partial sums take their place
            float* const part = (float*)xs;
#pragma unroll
            for (int r = 0; r < RT; ++r) ((v4f*)part)[(wave * RT + r) * 64 + lane] = acc[r];
            lds_barrier();
            _Float16* const ys = sm + c.off_y;
            const float inv_n = 1.0f / (float)N;
            for (int idx = tid; idx < vrows * N; idx += MLT) {
                const int m = (int)(((float)idx + 0.5f) * inv_n), n = idx - m * N;
                const float* src = part + ((((n >> 4) * RT + (m >> 4)) * 64 + ((n >> 2) & 3) * 16 + (m & 15)) << 2) + (n & 3);
                float v = 0.0f;
                for (int k = 0; k < parts; ++k) v += src[(k << ntl) * RT * 256];
                const _Float16 o = (_Float16)(v + (float)cs[a.L[l].c_off + n]);
                if constexpr (TAPS) {
                    if (tp.p[l]) ((_Float16*)tp.p[l])[(row0 + m) * N + n] = o;
                }
                if (a.head == AQ_HEAD_ARGMAX) ys[m * MLY_LD + n] = o;
                else ((float*)c.actions)[(row0 + m) * N + n] = a.head == AQ_HEAD_TANH ? (float)(_Float16)tanh_rel((float)o) : (float)o;
            }
            if (a.head == AQ_HEAD_ARGMAX) {
                lds_barrier();
                if (tid < vrows) {
                    const _Float16* yr = ys + tid * MLY_LD;
                    int best = 0;
                    for (int n = 1; n < N; ++n)
                        if (yr[n] > yr[best]) best = n;
                    ((int32_t*)c.actions)[row0 + tid] = best;
                }
            }
            return;
        }
        switch (tiles_of(l)) {
            case 1: layer_nb(std::integral_constant<int, 1>{}, l); break;
            case 2: layer_nb(std::integral_constant<int, 2>{}, l); break;
            case 3: layer_nb(std::integral_constant<int, 3>{}, l); break;
            case 4: layer_nb(std::integral_constant<int, 4>{}, l); break;
            default:
                lds_barrier();
                lds_barrier();
                break;
        }
        // The features that pad the layer to whole tiles become zeros, by the wavefront that wrote them (its LDS writes stay
        // in order): zero weights times an infinite input were no zeros, and the next layer's sums would take them in.
        // (Selected in the epilogue above, it cost the wide case 8 us in spilled registers.)
        if (!last && (N & 31) && wave == ((NT - 1) & (MLW - 1)) && lane < ROWS)
            for (int n = N; n < NT * 32; ++n) xs[lane * ld + n] = (_Float16)0.0f;
        if (TAPS || last) lds_barrier();
        tap(l);
        if (last) {
            if (a.head == AQ_HEAD_ARGMAX) {
                if (tid < vrows) {
                    const _Float16* yr = xs + tid * ld;
                    int best = 0;
                    for (int n = 1; n < N; ++n)
                        if (yr[n] > yr[best]) best = n;
                    ((int32_t*)c.actions)[row0 + tid] = best;
                }
            } else {
                for (int idx = tid; idx < vrows * N; idx += MLT) {
                    const int m = idx / N, n = idx - m * N;
                    const float o = (float)xs[m * ld + n];
                    ((float*)c.actions)[(row0 + m) * N + n] = a.head == AQ_HEAD_TANH ? (float)(_Float16)tanh_rel(o) : o;
                }
            }
        }
    }
}

namespace {
struct MlpPlan {
    int rt, ld, off_const, off_red, off_y;
    size_t lds;
};
bool plan_rows(const Fp16Net& n, int rt, MlpPlan* p) {
    int w = 0;
    for (int l = 0; l < n.n_layers; ++l) {
        const Fp16LayerDev& L = n.L[l];
        const int k = (L.K + 31) & ~31;
        if (k > MLMAXW || L.NT * 32 > MLMAXW) return false;
        w = w > k ? w : k;
        if (l < n.n_layers - 1 || L.NT > 2) w = w > L.NT * 32 ? w : L.NT * 32;
    }
    p->rt = rt;
    p->ld = w + 8;  // (16-byte reads of consecutive rows fall on different banks: 4 words further each)
    size_t halfs = (size_t)16 * rt * p->ld;
    const size_t part = (size_t)MLW * rt * 256 * 2;  // a narrow head's partial sums
    if (n.L[n.n_layers - 1].NT <= 2 && part > halfs) halfs = part;
    halfs = (halfs + 7) & ~(size_t)7;
    p->off_const = (int)halfs;
    halfs += (size_t)n.cst;
    p->off_red = (int)halfs;
    for (int l = 0; l < n.n_layers - 1; ++l)
        if (n.L[l].act == AQ_ACT_LN_TANH) {
            halfs += (size_t)16 * rt * MLW * 4;
            break;
        }
    p->off_y = (int)halfs;
    if (n.L[n.n_layers - 1].NT <= 2 && n.head == AQ_HEAD_ARGMAX) halfs += (size_t)16 * rt * MLY_LD;
    p->lds = halfs * 2;
    return p->lds <= 160 * 1024;
}
// Rows per workgroup, or none.  Clocks of a workgroup: its weights through the CU's vector memory path at 58 B per clock
// and its MFMAs (20 clocks each at the clock the chip holds, on four SIMDs), half of the shorter of the two hidden
// behind the longer; barriers and epilogue per layer; a LayerNorm's statistics and tanh; rounds of one
// workgroup per CU.  Fitted to 67-w-w-w-21: w = 128, 256, 512 at batch 4096 7.0, 9.2, 16.6 us; at 16384 12.9, 16.6,
// 27.7 us; 256-1024x3-64 at 16384 75.8 us; LayerNorms of 64, 256, 512, 1024 features in front add 2.8, 4.6, 7.9, 12.9 us at 64 rows.
// Against a launch per layer, which spreads a layer's weights over the chip.  Two estimates of that, of which the larger counts
// (the launches write maps that two streams would share): 4 us each and 371 k flop per clock, what the widest layers reach; and three
// quarters of 3.96 us each, per 10^6 of output tiles x K 12 us on the few-row kernel, 4 on the tiled one, 20 there for rows of no
// whole 8 values, 4 us per 10^6 values of a LayerNorm, fitted to 16000 pairs (one to five hidden layers of 50 to 1300, 320 to
// 27600 rows).  Three quarters, because it is up to 1.4 times too long for layers of 1024 at some hundred to 2400 rows: 36-1024x3-30 at
// 1067 rows takes 46.0 us whole and 32.6 by layers, 55-1024x2-9 at 974 22.4 and 19.5, 104-1024x3-19 at 4096 54 and 49.8, which the whole of
// it calls faster here.  Elsewhere it costs: 396 drawn policies are 1.3 % from the better way (the whole estimate 0.8 %), 500 at row
// counts just above whole rounds of workgroups 3.2 % (0.6 %).  With the first estimate alone 13.6 and 29 %: 19-125-102-34 took 40.0 us
// at 28000 rows and 80 at 65536 (18.4 and 33.7 here), 111-400-300-8 134 at 65536 (58).
bool plan_mlp(const Fp16Net& n, int64_t batch, MlpPlan* best) {
    double best_c = 0.0;
    bool found = false;
    for (int rt = 1; rt <= 4; rt *= 2) {
        MlpPlan p;
        if (!plan_rows(n, rt, &p)) continue;
        double per = 5000.0;
        for (int l = 0; l < n.n_layers; ++l) {
            const double tiles = n.L[l].NT, ks = (n.L[l].K + 31) / 32;
            const double mem = tiles * ks * 2048.0 / 58.0, mm = tiles * ks * rt * 2 * 20.0 / 4.0;
            per += (mem > mm ? mem + 0.5 * mm : mm + 0.5 * mem) + 2000.0 * (1.0 + 0.15 * rt);
            if (l < n.n_layers - 1 && n.L[l].act == AQ_ACT_LN_TANH) per += 1200.0 + rt * (1100.0 + 6.0 * n.L[l].N);
        }
        const int64_t wgs = (batch + 16 * rt - 1) / (16 * rt);
        if (!grid_ok(wgs, MLT)) continue;
        const double c = (double)((wgs + 255) / 256) * per;
        if (!found || c < best_c) {
            best_c = c;
            *best = p;
            found = true;
        }
    }
    if (!found) return false;
    double flop = 0.0, us = 0.0;
    for (int l = 0; l < n.n_layers; ++l) {
        const Fp16LayerDev& D = n.L[l];
        flop += 9500.0 + 2.0 * D.NT * 32.0 * D.K * (double)batch / 371e3;
        Fp16Layer L{};
        L.fc = 1;
        L.K = D.K;
        L.N = D.N;
        L.NT = D.NT;
        const double tiles = (double)((batch + 31) / 32) * D.NT * D.K * 1e-6;
        us += 3.96 + tiles * (fp16_layer_is_skinny(L, l == 0 ? 1 : 0, batch) ? 12.0 : D.K % 8 ? 20.0 : 4.0);
        if (l < n.n_layers - 1 && D.act == AQ_ACT_LN_TANH) {
            flop += 8000.0 + 10.0 * D.N * (double)batch / 4096.0;
            us += 3.96 + 4e-6 * D.N * (double)batch;
        }
    }
    const double second = 0.75 * 2375.0 * us;
    return best_c <= (flop > second ? flop : second);
}
}  // namespace

int fp16_mlp_rows(const Fp16Net& n, int64_t batch) {
    MlpPlan p;
    return n.n_layers > 0 && plan_mlp(n, batch, &p) ? 16 * p.rt : 0;
}

aq_status launch_fp16_mlp(const Fp16Net& n, const Fp16Net* d_net, const void* obs, int in_u8, int64_t batch, void* actions,
                          void* const* taps, hipStream_t st) {
    MlpPlan p;
    if (!plan_mlp(n, batch, &p)) return AQ_ESHAPE;
    const Fp16Call c{obs, actions, batch, p.ld, p.off_const, p.off_red, p.off_y};
    const dim3 grid((unsigned)((batch + 16 * p.rt - 1) / (16 * p.rt)));
#define AQ_MLP16(RT, U, TP)                                                                                                   \
    do {                                                                                                                      \
        static std::atomic<bool> attr_set{false};                                                                             \
        if (!attr_set) {                                                                                                      \
            if (hip_failed(hipFuncSetAttribute((const void*)k_fp16_mlp<RT, U, TP>,                                            \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)))                      \
                return AQ_EHIP;                                                                                               \
            attr_set = true;                                                                                                  \
        }                                                                                                                     \
        hipLaunchKernelGGL((k_fp16_mlp<RT, U, TP>), grid, dim3(MLT), p.lds, st, d_net, c, Fp16Taps<TP>(taps, n.n_layers));    \
    } while (0)
#define AQ_MLP16_T(RT, U)             \
    do {                              \
        if (taps) AQ_MLP16(RT, U, true); \
        else AQ_MLP16(RT, U, false);  \
    } while (0)
    if (p.rt == 4) {
        if (in_u8) AQ_MLP16_T(4, true);
        else AQ_MLP16_T(4, false);
    } else if (p.rt == 2) {
        if (in_u8) AQ_MLP16_T(2, true);
        else AQ_MLP16_T(2, false);
    } else {
        if (in_u8) AQ_MLP16_T(1, true);
        else AQ_MLP16_T(1, false);
    }
#undef AQ_MLP16_T
#undef AQ_MLP16
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

}  // namespace aq

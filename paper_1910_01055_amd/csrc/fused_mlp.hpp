// The general whole-network int8 MLP kernel (Sec. 3.1 actor inference on the 8-bit policy of Sec. 3.2): every fully connected
// policy up to 1024 wide, either weight scheme, LayerNorms of any of these widths, any K and N.
//
// One workgroup of 8 wavefronts owns 16 RT batch rows from the observation to the action.  The rows' codes live in one LDS buffer
// that every layer overwrites in place: a layer's outputs wait in registers until all wavefronts have read its inputs, so that a
// whole LayerNorm row is at hand between its accumulators and its codes and never leaves the chip.  A wavefront takes feature
// tiles wave, wave + 8, ... of 32 (up to NBM); both halves of a tile are v_mfma_i32_16x16x64_i8 on the library's 32 x 32 operand
// tiles: lane (b = lane % 16, g = lane / 16) of half h and k-step s takes piece 16 h + b + 32 (g % 2) of tile 2 s + g / 2, which
// holds bytes 64 s + 16 g .. + 15 of feature 16 h + b; its results are features 4 g .. 4 g + 3 of row b.
// Two barriers a layer: its inputs are complete; all of them are read (and the LayerNorm's partial statistics are there).
// A requantized layer's codes are made in front of the second one, so that the wavefronts ahead do not just wait there.
// An epilogue's constants: a lane fetches one 16-byte piece per four halves (array lane % 16 / 4 of half lane % 4) and the row's
// lanes hand them to each other by DPP.
// Per-tensor weights need sum_k a_s of every row: the epilogue that writes the codes adds them up, four bytes at a time.
// Columns that nobody computes are zeros wherever a k-step of 64 reads them.
//
// NBM = 2 (hidden layers up to 512 wide) keeps within 128 registers up to 64 rows, so that two workgroups share a CU.
#pragma once
#include "explore_device.hpp"
#include "int8_device.hpp"
#include "lanes.hpp"

namespace aq {
namespace fused {

constexpr int IW = 8;              // wavefronts per workgroup
constexpr int IT = IW * 64;
constexpr int IMAXN = 1024;        // widest layer
constexpr int IMAXK = 2496;        // longest input row
constexpr int INARROW = 64;        // most outputs of a last layer that is split over K
constexpr float K2_LOG2E = 2.885390081777927f;  // 2 log2(e): tanh(y) = 1 - 2 / (2^(K2 y) + 1)

// 1 / n for n >= 1 and 1 / sqrt(v), the units' results (1 ulp) with one Newton step: as near as the correctly rounded operations, for
// a fifth of their instructions
__device__ __forceinline__ float recip(float n) {
    const float r = __builtin_amdgcn_rcpf(n);
    return fmaf(fmaf(-n, r, 1.0f), r, r);
}
__device__ __forceinline__ float rsqrt_near(float v) {
    const bool tiny = v < 1e-30f;  // (a constant row and next to no eps: below, the unit takes v for zero)
    v = tiny ? v * 0x1p64f : v;
    const float r = __builtin_amdgcn_rsqf(v);
    const float n = fmaf(0.5f * r, fmaf(-v * r, r, 1.0f), r) * (tiny ? 0x1p32f : 1.0f);
    return v < INFINITY ? n : r;  // (a variance beyond the largest float: 0)
}

struct Call {
    const void* obs;
    void* actions;
    int64_t batch;
    const float* ex_sigma;  // Gaussian exploration noise added where the actions are written (narrow last layer), or NULL
    uint32_t ex_k0, ex_k1, ex_s0, ex_s1;
    int ld;                        // LDS row stride, bytes: a multiple of 64, plus 16
    int off_red, off_sum, off_cst, off_y;  // LDS: statistics, row sums, a narrow last layer's constants and argmax logits
};

// registers of the weight ring: k-steps (of 64) in flight when a wavefront has NB tiles, two operands of four registers each
template <int RT, int NBM, int NB>
constexpr int ring_depth() {
    constexpr int regs = NBM == 2 ? (RT >= 4 ? 16 : 32) : 64;
    constexpr int d = regs / (8 * NB);
    return d >= 8 ? 8 : d >= 4 ? 4 : d >= 2 ? 2 : 1;
}

template <int RT, int NBM, bool ASYM, bool TAPS>
__global__ __launch_bounds__(IT, NBM == 2 && RT <= 4 ? 4 : 2) void k_mlp_fused(const NetDev* __restrict__ netp, const Call c,
                                                                       const TapParam<TAPS> tp) {
    const TapArgs t = taps_of(tp);
    extern __shared__ __align__(16) int8_t sm[];
    constexpr int ROWS = 16 * RT;
    const NetDev& a = *netp;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int b = lane & 15, g = lane >> 4;
    const int nl = uni(a.n_layers), ld = c.ld;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int64_t left = c.batch - row0;
    const int vrows = left < ROWS ? (int)left : ROWS;
    int8_t* const xs = sm;
    float* const red = (float*)(sm + c.off_red);
    int32_t* const cst = (int32_t*)(sm + c.off_cst);
    int32_t* const rsum = (int32_t*)(sm + c.off_sum);  // per-tensor weights: [layer & 1][row], sum_k a_s of its inputs
    const int Nl = uni(a.L[nl - 1].N), NTl = uni(a.L[nl - 1].NT);
    const bool narrow_last = Nl <= INARROW;

    // ---- observations: codes, kept in the signed domain; zeros past the row ends (up to whole k-steps) and past the batch.
    // A thread has four quads of values in flight.  fp32 rows: one 16-byte request at a 4-byte aligned address, whose words past
    // the row's end are the next row's first ones; only the quad that ends the batch goes word by word.
    {
        const int K = uni(a.L[0].K), cols = ((K + 63) & ~63) >> 2, total = ROWS * cols;
        const float inv = 1.0f / (float)cols;  // (idx + 0.5) / cols is 0.5 / cols away from every integer, idx < 2^16
        const bool u8 = uni(a.in_u8) != 0;
        const bool words = u8 && (K & 3) == 0 && ((uintptr_t)c.obs & 3) == 0;
        const QuantScale qs0 = make_quant_scale(unif(a.actq[0].s));
        const float zf0 = (float)uni(a.actq[0].z);
        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
        constexpr int U = 4;
        for (int base = tid; base < total; base += U * IT) {
            float4 v[U];
            int m[U], k[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int idx = base + u * IT;
                m[u] = (int)(((float)idx + 0.5f) * inv);
                k[u] = (idx - m[u] * cols) * 4;
                v[u] = float4{0.0f, 0.0f, 0.0f, 0.0f};
                if (idx >= total || m[u] >= vrows || k[u] >= K) continue;
                const int64_t off = (row0 + m[u]) * K + k[u];
                const int last = K - 1 - k[u];  // values of the row behind the quad's first
                if (u8) {
                    const uint8_t* src = (const uint8_t*)c.obs + off;
                    uint32_t w;
                    if (words) {
                        w = *(const uint32_t*)src;
                    } else {  // (bytes past the row's end re-read its last one)
                        const uint32_t b0 = src[0], b1 = src[last < 1 ? last : 1], b2 = src[last < 2 ? last : 2],
                                       b3 = src[last < 3 ? last : 3];
                        w = b0 | (b1 << 8) | (b2 << 16) | (b3 << 24);
                    }
                    v[u].x = __uint_as_float(w);
                } else {
                    const float* src = (const float*)c.obs + off;
                    if (last >= 3 || row0 + m[u] + 1 < c.batch - 2) {  // (two rows behind: at least three values exist there)
                        const f4u w = *(const f4u*)src;
                        v[u] = float4{w[0], w[1], w[2], w[3]};
                    } else {
                        v[u].x = src[0];
                        if (last >= 1) v[u].y = src[1];
                        if (last >= 2) v[u].z = src[2];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int idx = base + u * IT;
                if (idx >= total) break;
                uint32_t pack = 0;
                if (m[u] < vrows && k[u] < K) {
                    const int have = K - k[u];  // real values in this quad: 1 .. 4, or more
                    pack = u8 ? __float_as_uint(v[u].x) : quant_u8x4(v[u], qs0, zf0);
                    if (TAPS) {
                        if (t.a0)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (i < have) t.a0[(row0 + m[u]) * K + k[u] + i] = (uint8_t)(pack >> (8 * i));
                    }
                    pack ^= 0x80808080u;
                    if (have < 4) pack &= (1u << (8 * have)) - 1u;
                }
                *(uint32_t*)(xs + m[u] * ld + k[u]) = pack;
            }
        }
    }
    if (narrow_last && tid < 2 * INARROW) {  // bias and scale
        const int n = tid & (INARROW - 1);
        if (n < NTl * 32) cst[tid] = *(gint_ptr)((gint_ptr)uni_ptr(a.L[nl - 1].bias_fold) + (tid >= INARROW ? NTl * 32 : 0) + n);
    }

    // A layer's weights as a buffer: descriptor and tile offset in scalar registers, one 32-bit lane offset.  (The last tile's
    // k-step past an odd number of k-tiles reads zeros, another tile's the next tile's weights: they meet zero activations.)
    const int lane_off = (g >> 1) * 1024 + (b + 32 * (g & 1)) * 16;
    auto weights_of = [&](int l) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)uni_ptr(a.L[l].wp), 0, uni(a.L[l].NT) * uni(a.L[l].KS) * 1024, 0x00020000);
    };
    auto operand = [&](__amdgpu_buffer_rsrc_t w, int off) __attribute__((always_inline)) {
        return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w, lane_off, off, 0));
    };
    const int8_t* const xrow = xs + b * ld + 16 * g;
    auto dot_ones = [&](const v4i& x, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_sdot4(x[i], 0x01010101, s, false);
        return s;
    };

    // Row sums of a layer's inputs: the first layer's from the codes, the others' from the layer before, whose epilogue adds them
    // to the buffer that is cleared here (between a layer's two barriers nobody reads or writes the other layer's).
    auto row_sums = [&](int l, int (&rs)[RT]) __attribute__((always_inline)) {
        const int zw = uni(*(gint_ptr)uni_ptr(a.L[l].z_w)) - 128;
        if (l == 0) {
            const int ks = (uni(a.L[0].KS) + 1) >> 1;
#pragma unroll
            for (int r = 0; r < RT; ++r) rs[r] = 0;
            for (int s = 0; s < ks; ++s)
#pragma unroll
                for (int r = 0; r < RT; ++r) rs[r] = dot_ones(*(const v4i*)(xrow + r * 16 * ld + s * 64), rs[r]);
#pragma unroll
            for (int r = 0; r < RT; ++r) rs[r] = -zw * sum_rows4(rs[r]);
        } else {
#pragma unroll
            for (int r = 0; r < RT; ++r) rs[r] = -zw * rsum[(l & 1) * ROWS + 16 * r + b];
        }
        if (tid < ROWS) rsum[((l + 1) & 1) * ROWS + tid] = 0;
    };
    auto add_row_sum = [&](int l, int r, int s) __attribute__((always_inline)) {
        atomicAdd(&rsum[((l + 1) & 1) * ROWS + 16 * r + b], s);  // (the row's four lanes each their own)
    };
    // per-tensor weights: features past N are zeros (the next layer sums whole padded rows); only a wavefront's last tile has any
    auto mask_padding = [&](auto h_c, auto nb_c, int n0, int N, uint32_t word) __attribute__((always_inline)) {
        if (!ASYM || decltype(h_c)::value < 2 * decltype(nb_c)::value - 2) return word;
        const int keep = N - n0;  // may be <= 0, or 4 and more
        return keep >= 4 ? word : keep <= 0 ? 0u : word & ((1u << (8 * keep)) - 1u);
    };

    auto layer_nb = [&](auto nb_c, int l) __attribute__((always_inline)) {
        constexpr int NB = decltype(nb_c)::value, H = 2 * (NB ? NB : 1), PF = ring_depth<RT, NBM, (NB ? NB : 1)>();
        const int N = uni(a.L[l].N), NT = uni(a.L[l].NT), KS = uni(a.L[l].KS), act = uni(a.L[l].act), Np = NT * 32;
        const bool ln = act == AQ_ACT_LN_TANH;
        const int ks = (KS + 1) >> 1;
        LayerTaps T{nullptr, nullptr, nullptr};
        if (TAPS) T = LayerTaps{t.acc[l], t.act[l], t.ln[l]};
        v4i acc[H][RT];
        int rs[RT];  // - z_w' sum_k a_s
        v4i cm[(H + 3) / 4];  // lane 4 A + h % 4 of a 16-lane row holds its four features' constants of array A, half h
        bool fast = false;
        if constexpr (NB == 0) {
            lds_barrier();
            if (ASYM) row_sums(l, rs);
        } else {
            fast = uni(a.fast[l]) != 0;
            const auto w = weights_of(l);
            const int w0 = wave * KS * 1024, step = IW * KS * 1024;
            v4i ring[PF][H];
            auto fetch = [&](auto p_c, int s) __attribute__((always_inline)) {
                constexpr int p = decltype(p_c)::value;
#pragma unroll
                for (int h = 0; h < H; ++h) ring[p][h] = operand(w, w0 + (h >> 1) * step + s * 2048 + 256 * (h & 1));
            };
            static_for<0, PF>([&](auto p_c) __attribute__((always_inline)) {
                if (decltype(p_c)::value < ks) fetch(p_c, decltype(p_c)::value);
            });
            {
                const int arr = b >> 2;
                const int32_t* base = uni_ptr(a.L[l].bias_fold) + arr * Np;
                if (arr == 3 && !ln && !fast) base = uni_ptr(a.L[l].rshift);
#pragma unroll
                for (int q = 0; q < (H + 3) / 4; ++q) {
                    const int h = 4 * q + (b & 3);
                    int nt = wave + IW * (h >> 1);
                    nt = nt < NT ? nt : NT - 1;
                    cm[q] = *(gv4i_ptr)(base + 32 * nt + 16 * (h & 1) + 4 * g);
                }
            }
            lds_barrier();  // this layer's inputs are in LDS
            if (ASYM) {
                row_sums(l, rs);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int h = 0; h < H; ++h) acc[h][r] = v4i{0, 0, 0, 0};
            v4i x[RT];  // a row tile's operand of the next k-step is read as soon as this k-step's MFMAs with it are issued
#pragma unroll
            for (int r = 0; r < RT; ++r) x[r] = *(const v4i*)(xrow + r * 16 * ld);
            auto one = [&](auto p_c, int s) __attribute__((always_inline)) {
                constexpr int p = decltype(p_c)::value;
                const int8_t* const nx = xrow + (s + p + 1 < ks ? s + p + 1 : s + p) * 64;
#pragma unroll
                for (int r = 0; r < RT; ++r) {
#pragma unroll
                    for (int h = 0; h < H; ++h) acc[h][r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ring[p][h], x[r], acc[h][r], 0, 0, 0);
                    x[r] = *(const v4i*)(nx + r * 16 * ld);
                }
            };
            // whole groups of PF k-steps as straight-line code; the last one requests nothing, the one in front of a partial
            // group only what is left
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
        }
        auto n0_of = [&](int h) { return (wave + IW * (h >> 1)) * 32 + 16 * (h & 1) + 4 * g; };
        // what makes the accumulators of half h the exact integers; taps of them
        auto exact = [&](auto h_c, int r, const int (&bias)[4], int (&val)[4]) __attribute__((always_inline)) {
            constexpr int h = decltype(h_c)::value;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                val[i] = acc[h][r][i] + bias[i];
                if (ASYM) val[i] += rs[r];
                if (TAPS) {
                    const int n = n0_of(h) + i;
                    const int64_t row = row0 + 16 * r + b;
                    if (T.acc && row < c.batch && n < N) T.acc[row * N + n] = val[i];
                }
            }
        };
        auto consts4 = [&](auto h_c, auto arr_c, int (&o)[4]) __attribute__((always_inline)) {
            constexpr int h = decltype(h_c)::value, arr = decltype(arr_c)::value;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = row_bcast_mov<4 * arr + (h & 3)>(cm[h >> 2][i]);
        };
        using A0 = std::integral_constant<int, 0>;
        using A1 = std::integral_constant<int, 1>;
        using A2 = std::integral_constant<int, 2>;
        using A3 = std::integral_constant<int, 3>;

        const int z_out = uni(a.actq[l + 1].z);
        if (!ln) {
            uint32_t pk[H][RT];
            const int lo = act == AQ_ACT_RELU ? z_out : 0;
            int lo_v = lo;
            asm volatile("" : "+v"(lo_v));
            auto tiles = [&](auto fast_c) __attribute__((always_inline)) {
                constexpr bool FAST = decltype(fast_c)::value;
                static_for<0, 2 * NB>([&](auto h_c) __attribute__((always_inline)) {
                    constexpr int h = decltype(h_c)::value;
                    int bias[4], mul[4], rz[4], sh[4];
                    consts4(h_c, A0{}, bias);
                    consts4(h_c, A1{}, mul);
                    if (FAST) consts4(h_c, A2{}, rz);
                    consts4(h_c, A3{}, sh);
                    const int n0 = n0_of(h);
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        int val[4];
                        exact(h_c, r, bias, val);
                        uint32_t pack = 0;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            int code;
                            if (FAST) code = clamp_code((__mulhi(val[i], mul[i]) + rz[i]) >> sh[i], lo_v, 255);
                            else code = requant_code(val[i], mul[i], sh[i], z_out, lo);
                            if (TAPS) {
                                const int64_t row = row0 + 16 * r + b;
                                if (T.act && row < c.batch && n0 + i < N) T.act[row * N + n0 + i] = (uint8_t)code;
                            }
                            pack |= (uint32_t)code << (8 * i);
                        }
                        pk[h][r] = mask_padding(h_c, nb_c, n0, N, pack ^ 0x80808080u);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
            };
            if (NB > 0) {
                if (fast) tiles(std::true_type{});
                else tiles(std::false_type{});
            }
            lds_barrier();  // all inputs read: the outputs take their place
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                int sum = 0;
#pragma unroll
                for (int h = 0; h < 2 * NB; ++h) {
                    *(uint32_t*)(xs + (16 * r + b) * ld + n0_of(h)) = pk[h][r];
                    if (ASYM) sum = __builtin_amdgcn_sdot4((int)pk[h][r], 0x01010101, sum, false);
                }
                if (ASYM && NB > 0) add_row_sum(l, r, sum);
            }
        } else {
            // LayerNorm over the layer's N features, tanh, re-quantize.  x = acc * (s_in s_w) in fp32, in the accumulators' place;
            // this wavefront's features give (sum, squared deviations from their own mean) per row, the wavefronts' pairs meet
            // by the pairwise update (Chan, Golub, LeVeque).
            auto count_of = [&](int w) {
                const int tiles = NT > w ? (NT - w + IW - 1) / IW : 0;
                return 32 * tiles - (((NT - 1) & (IW - 1)) == w ? Np - N : 0);
            };
            const int n_w = count_of(wave);
            const float inv_nw = recip((float)(n_w > 0 ? n_w : 1));
            static_for<0, 2 * NB>([&](auto h_c) __attribute__((always_inline)) {
                constexpr int h = decltype(h_c)::value;
                int bias[4], ms[4];
                consts4(h_c, A0{}, bias);
                consts4(h_c, A1{}, ms);  // (zero for padding features)
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    int val[4];
                    exact(h_c, r, bias, val);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[h][r][i] = __float_as_int((float)val[i] * __int_as_float(ms[i]));
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            if (NB > 0) {
                const bool whole = ((NT - 1) & (IW - 1)) != wave || Np == N;  // no padding among this wavefront's features
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    float s = 0.0f;
#pragma unroll
                    for (int h = 0; h < 2 * NB; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i) s += __int_as_float(acc[h][r][i]);
                    s = sum_rows4(s);
                    const float mean_w = s * inv_nw;
                    float q = 0.0f;
#pragma unroll
                    for (int h = 0; h < 2 * NB; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float d = __int_as_float(acc[h][r][i]) - mean_w;
                            if (h < 2 * NB - 2 || whole) q = fmaf(d, d, q);
                            else if (n0_of(h) + i < N) q = fmaf(d, d, q);
                        }
                    q = sum_rows4(q);
                    if (g == 0) *(float2*)(red + ((16 * r + b) * IW + wave) * 2) = float2{s, q};
                }
            }
            const float s_out = unif(a.actq[l + 1].s), eps = unif(a.ln_eps);
            const QuantScale qs_out = make_quant_scale(s_out);
            const float c0 = qs_out.inv + (float)z_out, c1 = 2.0f * qs_out.inv;
            // the row's four lanes take two wavefronts' pairs each
            float cnt[2], inv_cnt[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = count_of(2 * g + j);
                cnt[j] = (float)n;
                inv_cnt[j] = recip((float)(n > 0 ? n : 1));
            }
            lds_barrier();  // statistics of all wavefronts; all inputs read
            float sc[RT], mean[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const float4 v = *(const float4*)(red + (16 * r + b) * IW * 2 + 4 * g);
                const float sw[2] = {cnt[0] > 0.0f ? v.x : 0.0f, cnt[1] > 0.0f ? v.z : 0.0f};
                const float qw[2] = {cnt[0] > 0.0f ? v.y : 0.0f, cnt[1] > 0.0f ? v.w : 0.0f};
                mean[r] = sum_rows4(sw[0] + sw[1]) / (float)N;
                const float d0 = sw[0] * inv_cnt[0] - mean[r], d1 = sw[1] * inv_cnt[1] - mean[r];
                const float m2 = sum_rows4(fmaf(cnt[0] * d0, d0, qw[0]) + fmaf(cnt[1] * d1, d1, qw[1]));
                // (2 log2 e rides on the row's scale and on the offset: exp2 then yields e^{2y})
                sc[r] = rsqrt_near(m2 / (float)N + eps) * K2_LOG2E;
            }
            // Up to 256 features: code = round(t / s + z) with t = 1 - 2 / (e^{2y} + 1), straight from the reciprocal: 9 codes in a million off
            // the 64-bit ones.  More, what rows in memory get (ln_rows.hpp, 5 in a million): tanh from |y|, and t (1 / s) rounded once,
            // straight to an integer (in MAGIC's last place), before z is added: 4 in a million, tanh's error 3.5e-8 instead of 5.3e-8.
            // It is three more instructions a value: 61-1024x2-36 at 16379 rows 34.3 -> 35.5 us, 61-263-163-2 at 32768 17.8 -> 18.9.
            auto codes = [&](auto wide_c) __attribute__((always_inline)) {
                constexpr bool WIDE = decltype(wide_c)::value;
                constexpr float MAGIC = 12582912.0f;  // 1.5 * 2^23
                const float unmagic = MAGIC - (float)z_out;
                static_for<0, 2 * NB>([&](auto h_c) __attribute__((always_inline)) {
                    constexpr int h = decltype(h_c)::value;
                    int gi[4], bi[4];
                    consts4(h_c, A2{}, gi);
                    consts4(h_c, A3{}, bi);
                    float gv[4], bv[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        gv[i] = __int_as_float(gi[i]);
                        bv[i] = __int_as_float(bi[i]) * K2_LOG2E;
                    }
                    const int n0 = n0_of(h);
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        float rv[4], tv[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float y = fmaf((__int_as_float(acc[h][r][i]) - mean[r]) * sc[r], gv[i], bv[i]);
                            rv[i] = __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(WIDE ? fabsf(y) : y) + 1.0f);
                            tv[i] = fmaf(rv[i], -2.0f, 1.0f);
                            if (WIDE) tv[i] = copysignf(tv[i], y);
                        }
                        uint32_t pack = 0;
                        if (!qs_out.rcp_ok) {
                            pack = quant_u8x4(make_float4(tv[0], tv[1], tv[2], tv[3]), qs_out, (float)z_out);
                        } else {  // the conversion rounds half to even and saturates
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                pack = __builtin_amdgcn_cvt_pk_u8_f32(
                                    WIDE ? fmaf(tv[i], qs_out.inv, MAGIC) - unmagic : fmaf(rv[i], -c1, c0), i, pack);
                        }
                        if (TAPS) {
                            const int64_t row = row0 + 16 * r + b;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                if (row < c.batch && n0 + i < N) {
                                    if (T.ln) T.ln[row * N + n0 + i] = tv[i];
                                    if (T.act) T.act[row * N + n0 + i] = (uint8_t)(pack >> (8 * i));
                                }
                            }
                        }
                        const uint32_t word = mask_padding(h_c, nb_c, n0, N, pack ^ 0x80808080u);
                        *(uint32_t*)(xs + (16 * r + b) * ld + n0) = word;
                        if (ASYM) rs[r] = __builtin_amdgcn_sdot4((int)word, 0x01010101, h == 0 ? 0 : rs[r], false);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
            };
            if (N > 256) codes(std::true_type{});
            else if (NB <= 1) codes(std::false_type{});  // (a second tile of a wavefront's is past 256)
            if (ASYM && NB > 0)
#pragma unroll
                for (int r = 0; r < RT; ++r) add_row_sum(l, r, rs[r]);
        }
        // an odd number of tiles: the next layer's last k-step reads 32 columns nobody computes
        if ((NT & 1) && wave == (NT & (IW - 1))) {
#pragma unroll
            for (int i = 0; i < 2 * RT; ++i) {
                const int e = lane + 64 * i;  // ROWS rows x 8 words
                *(uint32_t*)(xs + (e >> 3) * ld + 32 * NT + 4 * (e & 7)) = 0u;
            }
        }
    };

    for (int l = 0; l < nl - 1; ++l) {
        const int NT = uni(a.L[l].NT);
        switch (NT > wave ? (NT - wave + IW - 1) / IW : 0) {
            case 1: layer_nb(std::integral_constant<int, 1>{}, l); break;
            case 2: layer_nb(std::integral_constant<int, 2>{}, l); break;
            case 3:
                if constexpr (NBM > 2) layer_nb(std::integral_constant<int, 3>{}, l);
                break;
            case 4:
                if constexpr (NBM > 2) layer_nb(std::integral_constant<int, 4>{}, l);
                break;
            default: layer_nb(std::integral_constant<int, 0>{}, l); break;
        }
    }

    if (!narrow_last) {
        // ---- a wide last layer: a tile at a time, straight from the accumulators to the caller's memory
        const int l = nl - 1, N = Nl, head = uni(a.head), KS = uni(a.L[l].KS), ks = (KS + 1) >> 1;
        const auto w = weights_of(l);
        const gint_ptr pack = (gint_ptr)uni_ptr(a.L[l].bias_fold);
        int rs[RT];
        float by[RT];
        int bn[RT];
        lds_barrier();
        if (ASYM) row_sums(l, rs);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            by[r] = 0.0f;
            bn[r] = -1;
        }
        for (int nt = wave; nt < NTl; nt += IW) {
            v4i acc[2][RT], wr[2][2];
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[0][r] = acc[1][r] = v4i{0, 0, 0, 0};
            auto fetch = [&](int p, int s) __attribute__((always_inline)) {
#pragma unroll
                for (int h = 0; h < 2; ++h) wr[p][h] = operand(w, nt * KS * 1024 + s * 2048 + 256 * h);
            };
            auto one = [&](int p, int s) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    const v4i x = *(const v4i*)(xrow + r * 16 * ld + s * 64);
                    acc[0][r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wr[p][0], x, acc[0][r], 0, 0, 0);
                    acc[1][r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wr[p][1], x, acc[1][r], 0, 0, 0);
                }
            };
            fetch(0, 0);
            for (int s = 0; s < ks; s += 2) {
                if (s + 1 < ks) fetch(1, s + 1);
                one(0, s);
                if (s + 2 < ks) fetch(0, s + 2);
                if (s + 1 < ks) one(1, s + 1);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int n = 32 * nt + 16 * h + 4 * g + i;
                    const int bias = pack[n];
                    const float ms = __int_as_float(pack[NTl * 32 + n]);
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        const int64_t row = row0 + 16 * r + b;
                        const bool ok = row < c.batch && n < N;
                        int v = acc[h][r][i] + bias;
                        if (ASYM) v += rs[r];
                        const float y = (float)v * ms;
                        if (TAPS) {
                            if (t.acc[l] && ok) t.acc[l][row * N + n] = v;
                            if (t.y && ok) t.y[row * N + n] = y;
                        }
                        if (head == AQ_HEAD_ARGMAX) {
                            if (ok && (bn[r] < 0 || y > by[r])) {
                                by[r] = y;
                                bn[r] = n;
                            }
                        } else if (ok) {
                            ((float*)c.actions)[row * N + n] = head == AQ_HEAD_TANH ? tanh_head(y) : y;
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (head != AQ_HEAD_ARGMAX) return;
        // lowest index of the largest value: over the row's four lanes, then over the wavefronts
        int* const redn = (int*)red;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                const float oy = __shfl_xor(by[r], o, 64);
                const int on = __shfl_xor(bn[r], o, 64);
                if (on >= 0 && (bn[r] < 0 || oy > by[r] || (oy == by[r] && on < bn[r]))) {
                    by[r] = oy;
                    bn[r] = on;
                }
            }
            if (g == 0) {
                red[((16 * r + b) * IW + wave) * 2] = by[r];
                redn[((16 * r + b) * IW + wave) * 2 + 1] = bn[r];
            }
        }
        lds_barrier();
        if (tid < vrows) {
            float y = 0.0f;
            int n = -1;
            for (int w = 0; w < IW; ++w) {
                const float oy = red[(tid * IW + w) * 2];
                const int on = redn[(tid * IW + w) * 2 + 1];
                if (on >= 0 && (n < 0 || oy > y || (oy == y && on < n))) {
                    y = oy;
                    n = on;
                }
            }
            ((int32_t*)c.actions)[row0 + tid] = n;
        }
        return;
    }

    // ---- a narrow last layer: feature tiles of 16 x parts of K over the wavefronts
    {
        const int l = nl - 1, N = Nl;
        const int tiles = (N + 15) >> 4, lg = tiles <= 1 ? 0 : tiles <= 2 ? 1 : 2, parts = IW >> lg;
        const int tile = wave & ((1 << lg) - 1), kp = wave >> lg;
        const int KS = uni(a.L[l].KS), ks = (KS + 1) >> 1, per = (ks + parts - 1) / parts;
        const int k0 = kp * per, k1 = k0 + per < ks ? k0 + per : ks;
        const auto w = weights_of(l);
        const int w0 = (tile >> 1) * KS * 1024 + 256 * (tile & 1);
        v4i acc[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[r] = v4i{0, 0, 0, 0};
        constexpr int PN = 4;
        v4i wr[PN];
        if (tile < tiles) {
#pragma unroll
            for (int p = 0; p < PN; ++p)
                if (k0 + p < k1) wr[p] = operand(w, w0 + (k0 + p) * 2048);
        }
        lds_barrier();
        if (ASYM && l == 0) {  // (the only layer: the sums of its inputs, where the reduction below finds them)
            int rs[RT];
            row_sums(0, rs);
            if (wave == 0 && g == 0)
#pragma unroll
                for (int r = 0; r < RT; ++r) rsum[16 * r + b] = rs[r];
        }
        if (tile < tiles) {
            for (int s = k0; s < k1; s += PN) {
#pragma unroll
                for (int p = 0; p < PN; ++p)
                    if (s + p < k1) {
                        if (s > k0) wr[p] = operand(w, w0 + (s + p) * 2048);
#pragma unroll
                        for (int r = 0; r < RT; ++r) {
                            const v4i x = *(const v4i*)(xrow + r * 16 * ld + (s + p) * 64);
                            acc[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wr[p], x, acc[r], 0, 0, 0);
                        }
                    }
            }
        }
        lds_barrier();  // all inputs read: the partial sums take their place
        int32_t* const part = (int32_t*)xs;
#pragma unroll
        for (int r = 0; r < RT; ++r) ((v4i*)part)[(wave * RT + r) * 64 + lane] = acc[r];
        int zw = 0;
        if (ASYM) zw = l == 0 ? 1 : 128 - uni(*(gint_ptr)uni_ptr(a.L[l].z_w));
        lds_barrier();
        float* const ys = (float*)(sm + c.off_y);
        const int head = uni(a.head), ldy = INARROW + 1;
        const float inv_n = 1.0f / (float)N;
        auto outputs = [&](auto ex_c) __attribute__((always_inline)) {
            constexpr bool EX = decltype(ex_c)::value;
            for (int idx = tid; idx < vrows * N; idx += IT) {
                const int m = (int)(((float)idx + 0.5f) * inv_n), n = idx - m * N;
                const int32_t* src = part + ((((n >> 4) * RT + (m >> 4)) * 64 + ((n >> 2) & 3) * 16 + (m & 15)) << 2) + (n & 3);
                int v = cst[n];
                for (int k = 0; k < parts; ++k) v += src[(k << lg) * RT * 256];
                if (ASYM) v += zw * rsum[(l & 1) * ROWS + m];
                const int64_t o = (row0 + m) * N + n;
                if (TAPS) {
                    if (t.acc[l]) t.acc[l][o] = v;
                }
                const float y = (float)v * __int_as_float(cst[INARROW + n]);
                if (TAPS) {
                    if (t.y) t.y[o] = y;
                }
                if (head == AQ_HEAD_ARGMAX) {
                    ys[m * ldy + n] = y;
                } else {
                    float act = head == AQ_HEAD_TANH ? tanh_head(y) : y;
                    if (EX) act += c.ex_sigma[row0 + m] * gaussian_draw((uint32_t)(row0 + m), n, c.ex_k0, c.ex_k1, c.ex_s0, c.ex_s1);
                    ((float*)c.actions)[o] = act;
                }
            }
        };
        if (c.ex_sigma) outputs(std::true_type{});
        else outputs(std::false_type{});
        if (head == AQ_HEAD_ARGMAX) {
            lds_barrier();
            if (tid < vrows) {
                const float* yr = ys + tid * ldy;
                int best = 0;
                for (int n = 1; n < N; ++n)
                    if (yr[n] > yr[best]) best = n;
                ((int32_t*)c.actions)[row0 + tid] = best;
            }
        }
    }
}

}  // namespace fused

// 16 rows (HALF) or 32 MT per workgroup, up to 2 NB feature tiles per wavefront
template <int MT, int NB, bool ASYM, bool TAPS, bool HALF>
aq_status launch_fused_t(const NetDev* d_net, const fused::Call& c, const TapArgs& t, size_t lds, hipStream_t st) {
    constexpr int RT = HALF ? 1 : 2 * MT;
    auto* const k = fused::k_mlp_fused<RT, 2 * NB, ASYM, TAPS>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
        if (hip_failed(hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024))) return AQ_EHIP;
        attr_set = true;
    }
    const unsigned grid = (unsigned)((c.batch + 16 * RT - 1) / (16 * RT));
    hipLaunchKernelGGL(k, dim3(grid), dim3(fused::IT), lds, st, d_net, c, TapParam<TAPS>(t));
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}
#define AQ_FUSED_INST(MT, NB, ASYM, TAPS, HALF) \
    template aq_status launch_fused_t<MT, NB, ASYM, TAPS, HALF>(const NetDev*, const fused::Call&, const TapArgs&, size_t, hipStream_t)
#define AQ_FUSED_DECL(MT, NB, ASYM, TAPS, HALF) extern AQ_FUSED_INST(MT, NB, ASYM, TAPS, HALF)

}  // namespace aq

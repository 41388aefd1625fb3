// Fully connected layer at few rows (Sec. 3.1: the paper's actors run their policy on one observation
// at a time; Sec. 4.1: three hidden layers of 2048 units): the time goes into the launch and the round trips for the
// layer's 8-bit weights, so the layer is cut into as many independent weight streams as possible, all requested at once.
//
// One workgroup of 8 waves owns FT tiles of 16 features x RT tiles of 16 rows (v_mfma_i32_16x16x64_i8); its waves split
// K eight ways, so every byte of either operand passes the CU's vector memory path once, straight into operand
// registers, up to PF k-steps of 64 in flight.  Each wave leaves a partial tile in LDS; after the one barrier a thread
// sums the eight partial sums of an output and runs the layer's epilogue (requantize, or dequantize for a LayerNorm /
// last layer).  The library's 32 x 32 weight tiles serve unchanged: lane (i = lane % 16, g = lane / 16) of feature half
// h and k-step s takes piece h * 16 + i + 32 * (g % 2) of tile 2 s + g / 2.
//
// Between two such layers the activations go in operand order too (blocked): byte k of row m at
// ((k / 16) * R + m) * 16 + k % 16 with R = rows rounded up to 16, zeros behind K.  A lane's 16 bytes of row-major
// activations lie in another row than its neighbour's, and the vector memory path then takes 75 clocks for the request
// instead of 16; row-major inputs (observations, maps of a convolution stack, LayerNorm rows) are therefore requested
// with neighbouring lanes along a row and change lanes on the way (ds_bpermute).
//
// Measured, 67-2048x3-21 at 16 rows, four launches: 18.5 us with one 32 x 32 tile per workgroup (v_mfma_i32_32x32x32_i8,
// activations through LDS), 13.0 so (host-bound: 3.1 us a launch).
//
// Weights of at most 4 bits (the precision sweep of the paper's appendix on quantization-aware training; per-channel
// symmetric codes in [-7, 7]) can stay sub-byte in device memory (W4): two codes per byte, stored as c + 8, half
// the bytes to stream.  A wave expands them on the way into the operand registers with three vector instructions
// per 8 codes -- mask, shift, mask: the nibbles enter the MFMA as the unsigned values c + 8, and the surplus
// 8 * sum_k a[k] leaves again in the epilogue through the row sums of the activations, which a second MFMA against
// all-ones collects as for the per-tensor scheme -- the accumulator the epilogue sees is the 8-bit path's, bit for bit.
#pragma once
#include "int8_device.hpp"

namespace aq {

constexpr int SK_W = 8;       // waves per workgroup = K split
constexpr int SK_LD = 65;     // words per register row of a partial tile (64 lanes + 1: the feature-major reduction
                              // then spreads over the banks)
// how a layer's input lies in memory
enum { IN_F32 = 0, IN_ROWS = 1, IN_BLOCKED = 2 };  // fp32 observations; 8-bit rows of any length; operand order

// What the host knows of the layer at launch time, by value: with the pointers among the kernel arguments the
// weight requests go out after one scalar round trip instead of two (arguments, then the layer's entry of the
// device-resident description); only what the quantizer kernels write (activation scales and zero-points, the
// short-form flag, the weight zero-point) is still read from the description, off the critical path.
// As few bytes as carry it: the host writes the arguments into uncached memory, about 0.3 us for each 100 bytes of them,
// and four such launches are a whole forward pass.
struct SkinnyLayer {
    const NetDev* net;
    const void* w;        // packed 8-bit weights, or the same as nibbles (k_pack_nibbles)
    const int32_t* pack;  // four arrays of N rounded up to 32: bias | M0 or m | rz | sh (LayerDev::bias_fold)
    const int32_t *rshift, *z_w;
    const void* in;
    void* out;            // 8-bit codes, or the fp32 rows in front of a LayerNorm; last layer: actions, indices or NULL
    float* y;             // last layer: dequantized outputs, or NULL
    int32_t K, N, rows, flags;  // flags: SF_* and the layer's index
};
enum { SF_FIRST = 1, SF_LAST = 2, SF_LN = 4, SF_RELU = 8, SF_TANH = 16, SF_ARGMAX = 32, SF_BLOCKED = 64, SF_LAYER = 8 /* shift */ };

typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_u __attribute__((ext_vector_type(4), aligned(4)));
typedef int v4i_u __attribute__((ext_vector_type(4), aligned(1)));

// W4: weights read as nibbles (per-channel symmetric only).  FT, RT: see above.  IN: how the input lies in memory.
template <bool ASYM, bool TAPS, bool W4, int FT, int RT, int IN>
__global__ __launch_bounds__(SK_W * 64) void k_layer_skinny(const SkinnyLayer L, const TapParam<TAPS> tp) {
    static_assert(!(ASYM && W4), "nibble weights are per-channel symmetric codes");
    constexpr bool RS = ASYM || W4;  // the epilogue needs the row sums of the activations
    constexpr int NF = 16 * FT, NQ = FT * RT;
    // k-steps in flight: behind a scalar test each, so that none is requested that the share does not have
    constexpr int PF = IN == IN_F32 ? 2 : NQ == 4 ? 4 : 8;
    __shared__ int32_t part[SK_W][NQ * 4][SK_LD];
    __shared__ int32_t part_rs[RS ? SK_W : 1][RS ? 16 * RT : 1];
    const TapArgs t = taps_of(tp);
    const NetDev& a = *L.net;
    // (the wave index as a scalar: what depends on it - this wave's k-steps - then branches on the scalar unit.
    // Left in a vector register it makes those tests lane masks, and a block that holds nothing but an MFMA may
    // lose its skip branch: the matrix cores do not honour an empty lane mask, the k-step would be added anyway)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * NF;
    const int64_t row0 = (int64_t)blockIdx.y * (16 * RT);
    const bool first = L.flags & SF_FIRST, last = L.flags & SF_LAST, ln = L.flags & SF_LN, blocked = L.flags & SF_BLOCKED;
    const int K = L.K, KS = (K + 31) >> 5, N = L.N;
    const int64_t rows = L.rows;
    const int KS64 = (KS + 1) >> 1, kc = (KS64 + SK_W - 1) / SK_W;
    const int k0 = wave * kc, k1 = k0 + kc < KS64 ? k0 + kc : KS64;
    const int64_t rtiles = (rows + 15) >> 4;

    // this thread's epilogue constants (its outputs share one feature): requested up front
    const int n_e = n0 + (tid & (NF - 1));  // < N rounded up to 32: the constant arrays are padded
    const int np = (N + 31) & ~31;
    const int c_bias = L.pack[n_e], c_M0 = L.pack[np + n_e], c_rz = L.pack[2 * np + n_e], c_sh = L.pack[3 * np + n_e], c_r = L.rshift[n_e];
    const float c_m = __int_as_float(c_M0);  // LayerNorm and last layers

    v4i acc[FT][RT], rs[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
#pragma unroll
        for (int f = 0; f < FT; ++f) acc[f][r] = v4i{0, 0, 0, 0};
        rs[r] = v4i{0, 0, 0, 0};
    }

    // row-major input: lane -> row lane / 4 of a tile, piece lane % 4 of a k-step; rows past the batch re-read the last
    // one (a batch row is a column of the MFMA's second operand: they only reach outputs that are not stored)
    int64_t rrow[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int64_t row = row0 + r * 16 + (lane >> 2);
        rrow[r] = row < rows ? row : rows - 1;
    }
    auto load_bytes = [&](int r, int ks) __attribute__((always_inline)) {
        const int k = ks * 64 + (lane & 3) * 16;
        v4i v = {0, 0, 0, 0};
        const int8_t* p = (const int8_t*)L.in + rrow[r] * K + k;
        if (k + 16 <= K) {
            v = (v4i)*(const v4i_u*)p;
            if (first) v ^= (int)0x80808080;  // 8-bit observations: into the signed domain
        } else if (k < K) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                if (k + j < K) v[j >> 2] |= (int)(uint32_t)((uint8_t)p[j] ^ (first ? 128u : 0u)) << (8 * (j & 3));
            }
        }
        return v;
    };
    auto load_f32 = [&](int r, int ks, const QuantScale& qs, int z0) __attribute__((always_inline)) {
        const int k = ks * 64 + (lane & 3) * 16;
        const float* p = (const float*)L.in + rrow[r] * K + k;
        v4f x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (k + 4 * q + 4 <= K) {
                x[q] = *(const v4f_u*)(p + 4 * q);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[q][j] = k + 4 * q + j < K ? p[4 * q + j] : 0.0f;
            }
        }
        v4i v;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t c = quant_u8x4(make_float4(x[q][0], x[q][1], x[q][2], x[q][3]), qs, (float)z0);
            if (TAPS) {
                if (t.a0 && blockIdx.x == 0 && row0 + r * 16 + (lane >> 2) < rows) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (k + 4 * q + j < K) t.a0[rrow[r] * K + k + 4 * q + j] = (uint8_t)(c >> (8 * j));
                }
            }
            c ^= 0x80808080u;
            const int left = K - (k + 4 * q);  // zeros in the signed domain behind K
            if (left < 4) c = left <= 0 ? 0u : c & ((1u << (8 * left)) - 1u);
            v[q] = (int)c;
        }
        return v;
    };
    const int swap = (i16 * 4 + g) * 4;  // where the row-major request left this lane's operand
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    // pieces of this lane in a weight tile pair
    const int wl = i16 + 32 * (g & 1);
    const int nt = FT == 1 ? (int)blockIdx.x >> 1 : (int)blockIdx.x;
    const int h0 = FT == 1 ? (int)blockIdx.x & 1 : 0;

    for (int g0 = k0; g0 < k1; g0 += PF) {
        v4i w[W4 ? 1 : PF][FT], x[PF][RT];
        v2i w4[W4 ? PF : 1][FT];
        if constexpr (IN == IN_BLOCKED) {
            static_for<0, PF>([&](auto u_c) __attribute__((always_inline)) {
                constexpr int u = decltype(u_c)::value;
                if (g0 + u < k1) {
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        // (rows past the batch re-read the last one: nobody writes theirs, and they would come from HBM)
                        const int64_t row_r = row0 + r * 16 + i16, row = row_r < rows ? row_r : rows - 1;
                        const int k = (g0 + u) * 64 + g * 16;
                        x[u][r] = v4i{0, 0, 0, 0};
                        if (k < K) x[u][r] = *(gv4i_ptr)((const int8_t*)L.in + ((int64_t)(k >> 4) * rtiles * 16 + row) * 16);
                    }
                }
            });
        } else if constexpr (IN == IN_ROWS) {
            static_for<0, PF>([&](auto u_c) __attribute__((always_inline)) {
                constexpr int u = decltype(u_c)::value;
                if (g0 + u < k1) {
#pragma unroll
                    for (int r = 0; r < RT; ++r) x[u][r] = load_bytes(r, g0 + u);
                }
            });
        }
        static_for<0, PF>([&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;
            if (g0 + u < k1) {
                const int kt = 2 * (g0 + u) + (g >> 1);  // (the second half of an odd last pair meets zeros)
                const int64_t piece = ((int64_t)nt * KS + (kt < KS ? kt : KS - 1)) * 64 + wl;
#pragma unroll
                for (int f = 0; f < FT; ++f) {
                    if constexpr (W4) w4[u][f] = ((const v2i AQ_GLOBAL*)L.w)[piece + 16 * (h0 + f)];
                    else w[u][f] = ((gv4i_ptr)L.w)[piece + 16 * (h0 + f)];
                }
            }
        });
        if constexpr (IN == IN_F32) {
            const float s0 = a.actq[0].s;
            const int z0 = a.actq[0].z;
            const QuantScale qs0 = make_quant_scale(s0);
            static_for<0, PF>([&](auto u_c) __attribute__((always_inline)) {
                constexpr int u = decltype(u_c)::value;
                if (g0 + u < k1) {
#pragma unroll
                    for (int r = 0; r < RT; ++r) x[u][r] = load_f32(r, g0 + u, qs0, z0);
                }
            });
        }
        if constexpr (IN != IN_BLOCKED) {
            static_for<0, PF>([&](auto u_c) __attribute__((always_inline)) {
                constexpr int u = decltype(u_c)::value;
                if (g0 + u < k1) {
#pragma unroll
                    for (int r = 0; r < RT; ++r)
#pragma unroll
                        for (int j = 0; j < 4; ++j) x[u][r][j] = __builtin_amdgcn_ds_bpermute(swap, x[u][r][j]);
                }
            });
        }
        static_for<0, PF>([&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;
            if (g0 + u < k1) {
#pragma unroll
                for (int f = 0; f < FT; ++f) {
                    v4i wv;
                    if constexpr (W4) {
                        const v2i q = w4[u][f];
                        wv[0] = q[0] & 0x0F0F0F0F;
                        wv[1] = (int)((uint32_t)q[0] >> 4) & 0x0F0F0F0F;
                        wv[2] = q[1] & 0x0F0F0F0F;
                        wv[3] = (int)((uint32_t)q[1] >> 4) & 0x0F0F0F0F;
                    } else {
                        wv = w[u][f];
                    }
#pragma unroll
                    for (int r = 0; r < RT; ++r) acc[f][r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wv, x[u][r], acc[f][r], 0, 0, 0);
                }
                if (RS) {
#pragma unroll
                    for (int r = 0; r < RT; ++r) rs[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, x[u][r], rs[r], 0, 0, 0);
                }
            }
        });
    }
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) part[wave][(f * RT + r) * 4 + i][lane] = acc[f][r][i];
    if (RS) {
        if (lane < 16) {
#pragma unroll
            for (int r = 0; r < RT; ++r) part_rs[wave][r * 16 + lane] = rs[r][0];
        }
    }
    // (what the quantizer wrote, read behind the operands)
    const int l = L.flags >> SF_LAYER;
    const int z_out = last ? 0 : a.actq[l + 1].z;
    const int lo = (L.flags & SF_RELU) ? z_out : 0;
    const int zw_s = W4 ? 8 : (ASYM ? L.z_w[0] - 128 : 0);
    const bool fast = !last && !ln && a.fast[l] != 0;
    const bool argmax_here = L.flags & SF_ARGMAX;  // last layer, argmax head, all features in this workgroup
    LayerTaps T{nullptr, nullptr, nullptr};
    if (TAPS) T = LayerTaps{t.acc[l], t.act[l], t.ln[l]};
    __syncthreads();

    // reduction + epilogue: thread -> (row m, feature n) with the feature index fastest, so that the
    // global stores of a row are contiguous
    constexpr int MP = SK_W * 64 / NF;  // rows per turn
#pragma unroll
    for (int it = 0; it < (16 * RT + MP - 1) / MP; ++it) {
        const int m = tid / NF + MP * it, nl = tid & (NF - 1);
        if (m >= 16 * RT) break;
        const int q = (nl >> 4) * RT + (m >> 4), reg = q * 4 + (nl & 3), lsrc = (m & 15) + 16 * ((nl >> 2) & 3);
        int v = c_bias, rsum = 0;
#pragma unroll
        for (int kp = 0; kp < SK_W; ++kp) {
            v += part[kp][reg][lsrc];
            if (RS) rsum += part_rs[kp][m];
        }
        if (RS) v -= zw_s * rsum;
        const int n = n0 + nl;
        const int64_t row = row0 + m;
        if (TAPS) {
            if (T.acc && row < rows && n < N) T.acc[row * N + n] = v;
        }
        if (argmax_here) {
            // the whole output row sits in this workgroup, one feature per lane of an NF-lane group: the
            // action index (lowest index among equal logits) is a shuffle reduction away
            const bool ok = row < rows && n < N;
            float y = ok ? (float)v * c_m : -INFINITY;
            if (ok && L.y) L.y[row * N + n] = y;
            int best = n;
#pragma unroll
            for (int o = NF / 2; o > 0; o >>= 1) {
                const float yo = __shfl_xor(y, o, NF);
                const int bo = __shfl_xor(best, o, NF);
                if (yo > y || (yo == y && bo < best)) {
                    y = yo;
                    best = bo;
                }
            }
            if (nl == 0 && row < rows) ((int32_t*)L.out)[row] = best;
            continue;
        }
        if (row >= rows) continue;
        if (n >= N) {
            if (blocked && n < ((N + 15) & ~15)) ((int8_t*)L.out)[((int64_t)(n >> 4) * rtiles * 16 + row) * 16 + (n & 15)] = 0;
            continue;
        }
        if (ln) {
            ((float*)L.out)[row * N + n] = (float)v * c_m;
        } else if (last) {
            const float y = (float)v * c_m;
            if (L.y) L.y[row * N + n] = y;
            if (L.out) ((float*)L.out)[row * N + n] = L.flags & SF_TANH ? tanh_head(y) : y;
        } else {
            int code;
            if (fast) code = min(max((__mulhi(v, c_M0) + c_rz) >> c_sh, lo), 255);
            else code = requant_code(v, c_M0, c_r, z_out, lo);
            if (TAPS) {
                if (T.act) T.act[row * N + n] = (uint8_t)code;
            }
            const int64_t o = blocked ? ((int64_t)(n >> 4) * rtiles * 16 + row) * 16 + (n & 15) : row * N + n;
            ((int8_t*)L.out)[o] = (int8_t)(code - 128);
        }
    }
}

struct SkinnyCall {
    hipStream_t st;
    SkinnyLayer sl;
    const TapArgs& t;
    bool taps;
    int ft, rt, in;
};
template <bool AS, bool TP, bool W4, int FT, int RT, int IN>
void skinny_launch(const SkinnyCall& c) {
    const dim3 grid((unsigned)((c.sl.N + 16 * FT - 1) / (16 * FT)), (unsigned)((c.sl.rows + 16 * RT - 1) / (16 * RT)));
    hipLaunchKernelGGL((k_layer_skinny<AS, TP, W4, FT, RT, IN>), grid, dim3(SK_W * 64), 0, c.st, c.sl, TapParam<TP>(c.t));
}
template <bool AS, bool TP, bool W4, int FT, int RT>
void skinny_input(const SkinnyCall& c) {
    if (c.in == IN_F32) skinny_launch<AS, TP, W4, FT, RT, IN_F32>(c);
    else if (c.in == IN_ROWS) skinny_launch<AS, TP, W4, FT, RT, IN_ROWS>(c);
    else skinny_launch<AS, TP, W4, FT, RT, IN_BLOCKED>(c);
}
template <bool AS, bool TP, bool W4>
void skinny_tile(const SkinnyCall& c) {
    if (c.ft == 1 && c.rt == 1) skinny_input<AS, TP, W4, 1, 1>(c);
    else if (c.ft == 1) skinny_input<AS, TP, W4, 1, 2>(c);
    else if (c.rt == 1) skinny_input<AS, TP, W4, 2, 1>(c);
    else skinny_input<AS, TP, W4, 2, 2>(c);
}
// per weight form (compiled one file each): per-channel symmetric, per-tensor asymmetric, nibbles
void skinny_go_sym(const SkinnyCall& c);
void skinny_go_asym(const SkinnyCall& c);
void skinny_go_w4(const SkinnyCall& c);

}  // namespace aq

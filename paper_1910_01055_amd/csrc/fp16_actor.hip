// The half-precision actor (the paper's fp16 policies, Sec. 3.2, and actors at q = 16): parameters,
// observation and every operator's output are IEEE binary16 values; products are exact and sums are
// kept in fp32 by v_mfma_f32_32x32x16_f16, rounded to binary16 once per operator.
//
//   k_fp16_convert        fp32 parameters -> binary16: weights in MFMA operand order (tile (n/32, k/16) = 1 KiB,
//                         lane = n % 32 + 32 * ((k % 16) / 8), 8 consecutive k per lane), zero padded;
//                         biases / LayerNorm gain and offset rounded to binary16 (kept widened, and as halfs)
//   k_layer_fp16          affine layer (FC or implicit-GEMM convolution) + bias (+ReLU), one launch per layer
//                         (whole fully connected policies in one launch: fp16_mlp.hip)
//   k_fp16_ln_tanh        LayerNorm, rounded, then tanh, rounded, in place
//   k_fp16_head           tanh / identity / argmax on the last layer's rows
#include "fp16_device.hpp"
#include "int8_device.hpp"
#include "ln_rows.hpp"

namespace aq {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f16acc __attribute__((ext_vector_type(16)));

namespace {

constexpr int HW = 4;     // waves per workgroup
constexpr int HKC = 64;   // k per staged chunk
constexpr int HLD = HKC + 8;  // LDS row stride in halfs (144 bytes: 16-byte reads of 8 rows hit 32 banks)

// One launch for the whole policy (as one launch per array it cost the host 2.6 us each).  Weights: a wave makes four
// tiles, a lane's 8 consecutive k of one feature per tile.
__global__ __launch_bounds__(256) void k_fp16_convert(const F32Ptrs src, const Fp16ConvTab* __restrict__ tab, int* status) {
    const int blk = (int)blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t before = __ballot(lane < tab->n && blk >= tab->blk0[lane < tab->n ? lane : 0]);
    const int a = __builtin_amdgcn_readfirstlane(63 - __builtin_clzll(before));
    const Fp16ConvTab::Entry e = tab->e[a];
    const int l = e.layer, rel = blk - tab->blk0[a];
    bool bad = false;
    if (e.kind == 0) {
        const float AQ_GLOBAL* w = (const float AQ_GLOBAL*)src.w[l];
        const bool al = (e.K & 3) == 0 && ((uintptr_t)src.w[l] & 15) == 0;
        typedef float f4 __attribute__((ext_vector_type(4)));
        const uint32_t tiles = (uint32_t)e.NT * (uint32_t)e.KS16;
        h8 v[kConvTiles / 4];
#pragma unroll
        for (int i = 0; i < kConvTiles / 4; ++i) {
            const uint32_t t = (uint32_t)rel * kConvTiles + i * 4 + wave;
            const int nt = (int)(t / (uint32_t)e.KS16), ks = (int)(t - (uint32_t)nt * (uint32_t)e.KS16);
            const int n = nt * 32 + (lane & 31), k = ks * 16 + 8 * (lane >> 5);
            f4 q[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
            if (t < tiles && n < e.N) {
                const float AQ_GLOBAL* p = w + (int64_t)n * e.K + k;
                if (al) {
                    if (k < e.K) q[0] = *(const f4 AQ_GLOBAL*)p;
                    if (k + 4 < e.K) q[1] = *(const f4 AQ_GLOBAL*)(p + 4);
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (k + j < e.K) q[j >> 2][j & 3] = p[j];
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                v[i][j] = (_Float16)q[j >> 2][j & 3];
                bad |= !(fabsf((float)v[i][j]) <= 65504.0f);
            }
        }
#pragma unroll
        for (int i = 0; i < kConvTiles / 4; ++i) {
            const uint32_t t = (uint32_t)rel * kConvTiles + i * 4 + wave;
            if (t < tiles) ((h8 AQ_GLOBAL*)e.dst)[(int64_t)t * 64 + lane] = v[i];
        }
    } else {
        const float* s = e.kind == 1 ? src.b[l] : e.kind == 2 ? src.gamma[l] : src.beta[l];
        const int i = rel * 256 + threadIdx.x;
        if (i < e.NT * 32) {
            _Float16 v = (_Float16)(e.kind == 2 ? 1.0f : 0.0f);
            if (s && i < e.N) {
                v = (_Float16)s[i];
                bad = !(fabsf((float)v) <= 65504.0f);
            }
            ((float*)e.dst)[i] = (float)v;
            if (e.dst_h) ((_Float16*)e.dst_h)[i] = v;
        }
    }
    if (bad) atomicOr(status, kStatNonFinite);
}

struct RowPos {
    int64_t base;  // element offset of (row, k = 0) in the layer's input
    bool ok;
};

__device__ __forceinline__ RowPos row_pos(const Fp16Layer& L, int64_t row, int64_t rows) {
    RowPos r;
    r.ok = row < rows;
    if (L.fc) {
        r.base = row * L.K;
    } else {
        const int per_img = L.oh * L.ow;
        const int64_t b = row / per_img;
        const int q = (int)(row - b * per_img);
        const int oy = q / L.ow, ox = q - oy * L.ow;
        r.base = ((b * L.in_h + (int64_t)oy * L.stride) * L.in_w + (int64_t)ox * L.stride) * L.in_c;
    }
    return r;
}

// offset of reduction index k relative to the row's base
__device__ __forceinline__ int64_t k_offset(const Fp16Layer& L, int k) {
    if (L.fc) return k;
    const int run = L.kw * L.in_c;
    const int ky = k / run, kr = k - ky * run;
    return (int64_t)ky * L.in_w * L.in_c + kr;
}

// IN: 0 = binary16 activations, 1 = fp32 observations, 2 = uint8 observations (exact in binary16)
// PIECE: every run of 8 consecutive k starting at a multiple of 8 is contiguous in the input, whole
//        (K is a multiple of 8) and aligned for vector loads (16 bytes for binary16 and fp32, 4 for uint8)
// One workgroup = 4 waves = 32*MT rows x 128*NB features; a wave owns NB feature tiles and all MT row tiles.
// Operands are requested one chunk ahead: weights straight into registers in operand order, the
// activation chunk into registers and from there into the other LDS buffer after the chunk's MFMAs.
// Loads are unconditional from clamped addresses (a row past the end reads the last row, a piece
// past K reads piece 0) and the value is zeroed afterwards, so that no branch separates a load from
// its use.
// (compiled for two waves per SIMD: within 256 registers the accumulators stay in ordinary vector
// registers; with more the compiler parks them in accumulation registers and copies them back and
// forth around every chunk)
template <int MT, int NB, int IN, bool PIECE>
__global__ __launch_bounds__(256, 2) void k_layer_fp16(const Fp16Layer L, const void* __restrict__ in,
                                                    _Float16* __restrict__ out, const int64_t rows) {
    constexpr int ROWS = 32 * MT;
    constexpr int SW = NB * 32 + 8;  // row stride (halfs) of a wave's output staging tile
    constexpr int XBUF = ROWS * HLD;
    constexpr int XS = 2 * XBUF > HW * 32 * SW ? 2 * XBUF : HW * 32 * SW;
    __shared__ __align__(16) _Float16 xs[XS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const int nt0 = (blockIdx.y * HW + wave) * NB;  // this wave's first feature tile
    const bool wave_on = nt0 < L.NT;
    const int KC = L.KS16 / 4;  // chunks of 64

    // staging: thread -> rows (tid >> 3) + 32 j, k piece (tid & 7) * 8 of each chunk
    const int sr = tid >> 3, sk = (tid & 7) * 8;
    RowPos rp[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const int64_t row = row0 + sr + 32 * j;
        rp[j] = row_pos(L, row < rows ? row : rows - 1, rows);
        rp[j].ok = row < rows;
    }

    auto load_x = [&](int c, h8 (&x)[MT]) __attribute__((always_inline)) {
        const int k0 = c * HKC + sk;
        if (PIECE) {
            const bool kok = k0 < L.K;
            const int64_t off = k_offset(L, kok ? k0 : 0);
            const h8 z = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                h8 v;
                {
                    if (IN == 0) {
                        v = *(const h8*)((const _Float16*)in + rp[j].base + off);
                    } else if (IN == 1) {
                        const float4* s4 = (const float4*)((const float*)in + rp[j].base + off);
                        const float4 a = s4[0], b = s4[1];
                        v[0] = (_Float16)a.x; v[1] = (_Float16)a.y; v[2] = (_Float16)a.z; v[3] = (_Float16)a.w;
                        v[4] = (_Float16)b.x; v[5] = (_Float16)b.y; v[6] = (_Float16)b.z; v[7] = (_Float16)b.w;
                    } else {
                        const uint32_t* s1 = (const uint32_t*)((const uint8_t*)in + rp[j].base + off);
                        const uint32_t a = s1[0], b = s1[1];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            v[i] = (_Float16)(float)((a >> (8 * i)) & 0xffu);
                            v[4 + i] = (_Float16)(float)((b >> (8 * i)) & 0xffu);
                        }
                    }
                }
                x[j] = (rp[j].ok && kok) ? v : z;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int k = k0 + i;
                const bool kok = k < L.K;
                const int64_t off = k_offset(L, kok ? k : 0);
#pragma unroll
                for (int j = 0; j < MT; ++j) {
                    _Float16 a;
                    if (IN == 0) a = ((const _Float16*)in)[rp[j].base + off];
                    else if (IN == 1) a = (_Float16)((const float*)in)[rp[j].base + off];
                    else a = (_Float16)(float)((const uint8_t*)in)[rp[j].base + off];
                    x[j][i] = (kok && rp[j].ok) ? a : (_Float16)0.0f;
                }
            }
        }
    };
    auto store_x = [&](int buf, const h8 (&x)[MT]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < MT; ++j) *(h8*)&xs[buf * XBUF + (sr + 32 * j) * HLD + sk] = x[j];
    };
    // this wave's weights of one chunk: 4 k-steps x NB tiles, 16 bytes per lane each
    const h8* wbase = (const h8*)L.wp + lane;
    auto load_w = [&](int c, h8 (&wr)[4][NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int nt = nt0 + nb < L.NT ? nt0 + nb : L.NT - 1;  // (clamped: the tile is not stored)
                wr[s][nb] = wbase[((int64_t)nt * L.KS16 + c * 4 + s) * 64];
            }
    };

    f16acc acc[NB][MT];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[nb][mt][i] = 0.0f;

    h8 wc[4][NB], wn[4][NB];  // weights of chunks c, c + 1
    h8 xn[MT];                 // activations of chunk c + 1
    auto compute = [&](int buf, const h8 (&w)[4][NB]) __attribute__((always_inline)) {
        const _Float16* xb = xs + buf * XBUF;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            h8 bx[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                bx[mt] = *(const h8*)&xb[(mt * 32 + (lane & 31)) * HLD + s * 16 + 8 * (lane >> 5)];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    acc[nb][mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[s][nb], bx[mt], acc[nb][mt], 0, 0, 0);
        }
    };
    if (MT < 4 && KC <= 2) {  // (the 128-row tile has no registers for it and never meets a short K)
        // short K (first layers: 17 or 67 observation features): everything is requested at once and both
        // LDS buffers are filled before the only barrier
        h8 x1[MT];
        load_w(0, wc);
        load_w(KC - 1, wn);
        load_x(0, xn);
        load_x(KC - 1, x1);
        store_x(0, xn);
        store_x(1, x1);
        __syncthreads();
        if (wave_on) {
            compute(0, wc);
            if (KC == 2) compute(1, wn);
        }
        __syncthreads();  // the epilogue reuses the buffers
    } else {
        load_w(0, wc);
        load_x(0, xn);
        store_x(0, xn);
        __syncthreads();
        for (int c = 0; c < KC; ++c) {
            const bool more = c + 1 < KC;
            {
                const int cn = more ? c + 1 : c;  // (clamped: loaded again, not used)
                load_w(cn, wn);
                load_x(cn, xn);
            }
            if (wave_on) compute(c & 1, wc);
            if (more) store_x((c + 1) & 1, xn);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) wc[s][nb] = wn[s][nb];
            __syncthreads();
        }
    }
    if (!wave_on) return;

    // epilogue: + bias, rounded to binary16 once, ReLU; lane = one row, four consecutive features per quad.
    // An elementwise action head (tanh / identity) is applied to the rounded value in the same sweep.
    auto quad_out = [&](int nb, int mt, int q, int n0) __attribute__((always_inline)) {
        const float4 bv = *(const float4*)(L.bias + n0);  // padded to the tile
        const float b4[4] = {bv.x, bv.y, bv.z, bv.w};
        h4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            _Float16 v = (_Float16)(acc[nb][mt][4 * q + i] + b4[i]);
            if (L.relu) v = v > (_Float16)0.0f ? v : (_Float16)0.0f;
            o[i] = v;
        }
        return o;
    };
    if ((L.N & 7) == 0) {
        // Rows of 16-byte pieces: each tile goes through a wave-private LDS region (the activation
        // buffers are idle after the last barrier) and leaves as whole contiguous runs of an output row,
        // NB * 64 bytes per row and wave, instead of 8 bytes per lane 2 * N bytes apart.
        _Float16* wsp = xs + wave * (32 * SW);
        constexpr int LPR = NB * 4;      // lanes per row on the way out
        constexpr int RPI = 64 / LPR;    // rows per store instruction
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n0 = (nt0 + nb) * 32 + 8 * q + 4 * (lane >> 5);
                    h4 o = {0, 0, 0, 0};
                    if (nt0 + nb < L.NT) o = quad_out(nb, mt, q, n0);
                    *(h4*)&wsp[(lane & 31) * SW + nb * 32 + 8 * q + 4 * (lane >> 5)] = o;
                }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 32 / RPI; ++j) {
                const int r = j * RPI + lane / LPR, pc = lane % LPR;
                const h8 v = *(const h8*)&wsp[r * SW + pc * 8];
                const int64_t row = row0 + mt * 32 + r;
                const int n = nt0 * 32 + pc * 8;
                if (row < rows && n < L.N) {
                    *(h8*)(out + row * L.N + n) = v;
                    if (L.head_actions) {
                        float a8[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            a8[i] = L.head_tanh ? (float)(_Float16)tanh_rel((float)v[i]) : (float)v[i];
                        float4* ad = (float4*)(L.head_actions + row * L.N + n);
                        ad[0] = make_float4(a8[0], a8[1], a8[2], a8[3]);
                        ad[1] = make_float4(a8[4], a8[5], a8[6], a8[7]);
                    }
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_wave_barrier();
        }
        return;
    }
    const bool vec_out = (L.N & 3) == 0;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        if (nt0 + nb >= L.NT) continue;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int64_t row = row0 + mt * 32 + (lane & 31);
            if (row >= rows) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n0 = (nt0 + nb) * 32 + 8 * q + 4 * (lane >> 5);
                if (n0 >= L.N) continue;
                const h4 o = quad_out(nb, mt, q, n0);
                _Float16* dst = out + row * L.N + n0;
                if (vec_out) {
                    *(h4*)dst = o;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (n0 + i < L.N) dst[i] = o[i];
                }
                if (L.head_actions) {
                    float* ad = L.head_actions + row * L.N + n0;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (n0 + i < L.N)
                            ad[i] = L.head_tanh ? (float)(_Float16)tanh_rel((float)o[i]) : (float)o[i];
                }
            }
        }
    }
}

// Fully connected layer at few rows (the paper's actors run one observation at a time, Sec. 3.1, on layers of 2048 units,
// Sec. 4.1), the binary16 counterpart of the 8-bit few-row kernel: one workgroup of 8 waves owns FT tiles of 16 features x RT
// tiles of 16 rows (v_mfma_f32_16x16x32_f16), its waves split K, both operands go straight from memory into operand
// registers, up to PF k-steps in flight; partial tiles meet in LDS, then a thread sums eight partial sums of an output, adds the
// bias, rounds once and stores.  Between two such layers the activations lie in operand order (value k of row m at
// ((k / 8) * R + m) * 8 + k % 8, R = rows rounded up to 16, zeros behind K); row-major inputs are requested along the rows and
// change lanes on the way.  The library's 32 x 16 weight tiles serve it unchanged: lane (i = lane % 16, g = lane / 16) of
// feature half h and k-step s takes piece h * 16 + i + 32 * (g % 2) of tile 2 s + g / 2.
// Bound by the launch and the round trips: 67-2048x3-21 at one row, four launches, 15.3 us with row-major activations, 200
// bytes of arguments and the tiled kernel for the first layer, 13.4 so; 67-700-523-21, whose rows are no multiples of 8 values, at
// 16 rows 43.9 (the tiled kernel's element-wise staging), 9.9.
constexpr int SKH_W = 8;
constexpr int SKH_LD = 65;  // words per register row of a partial tile (conflict-free feature-major reads)
typedef float f4acc __attribute__((ext_vector_type(4)));
typedef float f4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef _Float16 h8_u __attribute__((ext_vector_type(8), aligned(2)));
enum { HIN_ROWS = 0, HIN_F32 = 1, HIN_BLOCKED = 2 };
struct HalfRows {
    const void* w;
    const float* bias;
    const void* in;
    _Float16* out;
    void* head;  // fp32 actions, or action indices, or NULL
    int K, N, KS16, rows, flags;
};
enum { HF_RELU = 1, HF_TANH = 2, HF_ARGMAX = 4, HF_BLOCKED = 8 };
template <int FT, int RT, int IN>
__global__ __launch_bounds__(SKH_W * 64) void k_layer_fp16_rows(const HalfRows L) {
    constexpr int NF = 16 * FT, NQ = FT * RT, PF = IN == HIN_F32 ? 2 : NQ == 4 ? 4 : 8;
    __shared__ float part[SKH_W][NQ * 4][SKH_LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * NF, row0 = blockIdx.y * (16 * RT);
    const int K = L.K, N = L.N, rows = L.rows, rtiles = (rows + 15) >> 4;
    const int KS = (K + 31) >> 5, kc = (KS + SKH_W - 1) / SKH_W;  // (the weight tiles are padded to 64 k)
    const int k0 = wave * kc, k1 = k0 + kc < KS ? k0 + kc : KS;
    const float bias = L.bias[n0 + (tid & (NF - 1))];  // (padded to whole tiles of 32)
    f4acc acc[FT][RT];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[f][r] = f4acc{0.0f, 0.0f, 0.0f, 0.0f};
    // Rows past the batch re-read the last one; they only reach outputs that are not stored.  (In operand order they exist in
    // memory, but nobody writes them, and a first pass over new maps fetched them from HBM: 67-2048x3-21 at one row 40.7 us, 39.4
    // without; later passes 13.8 -> 13.5.)
    int64_t roff[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int row = row0 + r * 16 + (IN == HIN_BLOCKED ? i16 : lane >> 2), rr = row < rows ? row : rows - 1;
        roff[r] = IN == HIN_BLOCKED ? (int64_t)rr * 8 : (int64_t)rr * K + 8 * (lane & 3);
    }
    auto load_x = [&](int r, int ks) __attribute__((always_inline)) {
        h8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if constexpr (IN == HIN_BLOCKED) {
            const int k = ks * 32 + 8 * g;
            if (k < K) v = *(const h8 AQ_GLOBAL*)((const _Float16*)L.in + (int64_t)(k >> 3) * rtiles * 128 + roff[r]);
        } else if constexpr (IN == HIN_ROWS) {
            const int k = ks * 32 + 8 * (lane & 3);
            const _Float16* p = (const _Float16*)L.in + roff[r] + ks * 32;
            if (k + 8 <= K) {
                v = (h8)*(const h8_u*)p;
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (k + j < K) v[j] = p[j];
            }
        } else {
            const int k = ks * 32 + 8 * (lane & 3);
            const float* p = (const float*)L.in + roff[r] + ks * 32;
            f4acc x[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (k + 4 * q + 4 <= K) {
                    x[q] = *(const f4_u*)(p + 4 * q);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[q][j] = k + 4 * q + j < K ? p[4 * q + j] : 0.0f;
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = (_Float16)x[j >> 2][j & 3];
        }
        return v;
    };
    const int swap = (i16 * 4 + g) * 4;  // where the row-major request left this lane's operand
    const int nt = FT == 1 ? (int)blockIdx.x >> 1 : (int)blockIdx.x, h0 = FT == 1 ? (int)blockIdx.x & 1 : 0;
    const h8 AQ_GLOBAL* wsrc = (const h8 AQ_GLOBAL*)L.w + (int64_t)nt * L.KS16 * 64 + (g >> 1) * 64 + h0 * 16 + i16 + 32 * (g & 1);
    for (int g0 = k0; g0 < k1; g0 += PF) {
        h8 w[PF][FT], x[PF][RT];
        // (behind a scalar test each: none is requested that the share does not have)
        static_for<0, PF>([&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;
            if (g0 + u < k1) {
#pragma unroll
                for (int r = 0; r < RT; ++r) x[u][r] = load_x(r, g0 + u);
            }
        });
        static_for<0, PF>([&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;
            if (g0 + u < k1) {
#pragma unroll
                for (int f = 0; f < FT; ++f) w[u][f] = wsrc[(int64_t)(g0 + u) * 128 + 16 * f];
            }
        });
        static_for<0, PF>([&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;
            if (g0 + u < k1) {
                if constexpr (IN != HIN_BLOCKED) {
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        v4i t = __builtin_bit_cast(v4i, x[u][r]);
#pragma unroll
                        for (int j = 0; j < 4; ++j) t[j] = __builtin_amdgcn_ds_bpermute(swap, t[j]);
                        x[u][r] = __builtin_bit_cast(h8, t);
                    }
                }
#pragma unroll
                for (int f = 0; f < FT; ++f)
#pragma unroll
                    for (int r = 0; r < RT; ++r) acc[f][r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[u][f], x[u][r], acc[f][r], 0, 0, 0);
            }
        });
    }
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) part[wave][(f * RT + r) * 4 + i][lane] = acc[f][r][i];
    __syncthreads();
    constexpr int MP = SKH_W * 64 / NF;  // rows per turn
#pragma unroll
    for (int it = 0; it < (16 * RT + MP - 1) / MP; ++it) {
        const int m = tid / NF + MP * it, nl = tid & (NF - 1);
        if (m >= 16 * RT) break;
        const int reg = ((nl >> 4) * RT + (m >> 4)) * 4 + (nl & 3), lsrc = (m & 15) + 16 * ((nl >> 2) & 3);
        float v = 0.0f;
#pragma unroll
        for (int kp = 0; kp < SKH_W; ++kp) v += part[kp][reg][lsrc];
        const int n = n0 + nl, row = row0 + m;
        const bool ok = row < rows && n < N;
        _Float16 o = (_Float16)(v + bias);
        if (L.flags & HF_RELU) o = o > (_Float16)0.0f ? o : (_Float16)0.0f;
        if (L.flags & HF_BLOCKED) {
            if (row < rows && n < ((N + 15) & ~15)) L.out[((int64_t)(n >> 3) * rtiles * 16 + row) * 8 + (n & 7)] = ok ? o : (_Float16)0.0f;
        } else if (ok) {
            L.out[(int64_t)row * N + n] = o;
        }
        if (L.flags & HF_ARGMAX) {
            // the whole output row sits in this workgroup, one feature per lane of an NF-lane group: the action
            // index (lowest index among equal values) is a shuffle reduction away
            float y = ok ? (float)o : -INFINITY;
            int best = n;
#pragma unroll
            for (int d = NF / 2; d > 0; d >>= 1) {
                const float yo = __shfl_xor(y, d, NF);
                const int bo = __shfl_xor(best, d, NF);
                if (yo > y || (yo == y && bo < best)) {
                    y = yo;
                    best = bo;
                }
            }
            if (nl == 0 && row < rows) ((int32_t*)L.head)[row] = best;
        } else if (L.head && ok) {
            ((float*)L.head)[(int64_t)row * N + n] = L.flags & HF_TANH ? (float)(_Float16)tanh_rel((float)o) : (float)o;
        }
    }
}

// LayerNorm (biased variance, eps inside the root) rounded to binary16, then tanh rounded to binary16, in place, rows in
// registers (ln_rows.hpp)
template <int W, int P, bool VEC>
__global__ __launch_bounds__(256) void k_fp16_ln_tanh(_Float16* __restrict__ x, int64_t rows, int N,
                                                      const float* __restrict__ gamma, const float* __restrict__ beta,
                                                      float eps) {
    using Row = LnRow<W, P>;
    __shared__ float red[2][4];
    const int t = threadIdx.x & (Row::T - 1);
    const int64_t row = W == 1 ? (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6) : (int64_t)blockIdx.x;
    if (row >= rows) return;  // (a whole wavefront, or nobody)
    _Float16* const xr = x + row * N;
    Row r;
    float gg[P][4], bb[P][4];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        if (VEC) {
            const int n = Row::template at<true>(t, i, 0);
            h4 q = {0, 0, 0, 0};
            if (n < N) q = *(const h4*)(xr + n);
#pragma unroll
            for (int j = 0; j < 4; ++j) r.v[i][j] = (float)q[j];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = Row::template at<false>(t, i, j);
                r.v[i][j] = n < N ? (float)xr[n] : 0.0f;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < P; ++i) {
        Row::template load<VEC>(gamma, t, i, N, 1.0f, gg[i]);
        Row::template load<VEC>(beta, t, i, N, 0.0f, bb[i]);
    }
    float mean, inv;
    r.template stats<VEC>(t, N, eps, red, mean, inv);
#pragma unroll
    for (int i = 0; i < P; ++i) {
        h4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const _Float16 ln = (_Float16)((r.v[i][j] - mean) * inv * gg[i][j] + bb[i][j]);
            o[j] = (_Float16)tanh_rel((float)ln);
        }
        if (VEC) {
            const int n = Row::template at<true>(t, i, 0);
            if (n < N) *(h4*)(xr + n) = o;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = Row::template at<false>(t, i, j);
                if (n < N) xr[n] = o[j];
            }
        }
    }
}

// rows longer than those hold, or too many for them (ln_form): one wavefront per row, which is read three times
__global__ __launch_bounds__(256) void k_fp16_ln_tanh_long(_Float16* __restrict__ x, int64_t rows, int N,
                                                           const float* __restrict__ gamma,
                                                           const float* __restrict__ beta, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    _Float16* xr = x + row * N;
    float s = 0.0f;
    for (int n = lane; n < N; n += 64) s += (float)xr[n];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    const float mean = s / (float)N;
    float ss = 0.0f;
    for (int n = lane; n < N; n += 64) {
        const float d = (float)xr[n] - mean;
        ss += d * d;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
    const float inv = 1.0f / sqrtf(ss / (float)N + eps);
    for (int n = lane; n < N; n += 64) {
        const _Float16 ln = (_Float16)(((float)xr[n] - mean) * inv * gamma[n] + beta[n]);
        xr[n] = (_Float16)tanh_rel((float)ln);
    }
}

__global__ __launch_bounds__(256) void k_fp16_head(const _Float16* __restrict__ y, int64_t rows, int N, int head,
                                                   void* __restrict__ actions) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (head == AQ_HEAD_ARGMAX) {
        if (i >= rows) return;
        const _Float16* yr = y + i * N;
        int best = 0;
        float bv = (float)yr[0];
        for (int n = 1; n < N; ++n) {
            const float v = (float)yr[n];
            if (v > bv) {
                bv = v;
                best = n;
            }
        }
        ((int32_t*)actions)[i] = best;
    } else {
        if (i >= rows * N) return;
        const float v = (float)y[i];
        ((float*)actions)[i] = head == AQ_HEAD_TANH ? (float)(_Float16)tanh_rel(v) : v;
    }
}

}  // namespace

aq_status launch_fp16_convert(const F32Ptrs& src, const Fp16ConvTab* d_tab, int blocks, int* status, hipStream_t st) {
    hipLaunchKernelGGL(k_fp16_convert, dim3((unsigned)blocks), dim3(256), 0, st, src, d_tab, status);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

namespace {
template <int MT, int NB>
void launch_layer_cfg(const Fp16Layer& L, const void* in, int in_mode, bool piece, _Float16* o, int64_t rows,
                      hipStream_t st) {
    const dim3 grid((unsigned)((rows + 32 * MT - 1) / (32 * MT)), (unsigned)((L.NT + HW * NB - 1) / (HW * NB)));
#define AQ_F16_GO(IN, PC) hipLaunchKernelGGL((k_layer_fp16<MT, NB, IN, PC>), grid, dim3(256), 0, st, L, in, o, rows)
    if constexpr (MT == 4) {  // (the 128-row tile serves hidden layers only)
        if (piece) AQ_F16_GO(0, true);
        else AQ_F16_GO(0, false);
    } else {
        if (in_mode == 0) {
            if (piece) AQ_F16_GO(0, true);
            else AQ_F16_GO(0, false);
        } else if (in_mode == 1) {
            if (piece) AQ_F16_GO(1, true);
            else AQ_F16_GO(1, false);
        } else {
            if (piece) AQ_F16_GO(2, true);
            else AQ_F16_GO(2, false);
        }
    }
#undef AQ_F16_GO
}
}  // namespace

// The few-row kernel spreads a layer of few workgroups of the tiled one (32 rows x 128 features) over the chip, for longer where that
// one stages rows of no whole 8 values one by one.  Narrow layers, of at most eight 32-feature tiles, count those instead: the
// tiled kernel is the faster one sooner where K is short, and not in the measured range where a single tile leaves three of its
// four wavefronts without one, unless 16-bit rows are short.  8-bit observations take the tiled kernel.  us on the few-row / the tiled
// kernel, wide: 67-1024x3-21 at 512 rows 19.6 / 31.9, 1500 35.3 / 36.7, 2000 44.2 / 38.5; 67-2048x3-21 at 700 45.7 / 57.5;
// 67-1100-900-21 at 2000 38.4 / 51.6.  Narrow, over 6676 layers of K 16 to 3136 and 60 to 66000 rows: the rule is 1.1 % behind the faster
// kernel on average, 6.3 with the workgroups' line: 16-512-128-9 at 2048 rows 14.3 / 16.3, 6400 21.8 / 17.0; 384-256-9 at 1024 7.0 / 8.3,
// 3200 12.9 / 9.7.  (Layers wider than that by their tiles too: 7200 whole policies 4 % slower on average than so, since a layer's
// neighbours then lose the maps in operand order.)
bool fp16_layer_is_skinny(const Fp16Layer& L, int in_mode, int64_t rows) {
    if (in_mode == 2 || !L.fc || (rows + 15) / 16 > 65535) return false;
    const int64_t row_tiles = (rows + 31) / 32;
    if (L.NT > 8) return row_tiles * ((L.NT + HW - 1) / HW) < (L.K % 8 ? 512 : 400);
    double most = L.K >= 1000 ? 1000.0 : 500.0;
    if (L.K % 8) most *= L.K < 150 ? 1.4 : 2.5;
    if (L.NT == 1 && (L.K >= 200 || in_mode == 1)) most = 2100.0;
    return (double)row_tiles * L.NT < most;
}

namespace {
template <int FT, int RT>
void launch_rows(const HalfRows& q, int in, hipStream_t st) {
    const dim3 grid((unsigned)((q.N + 16 * FT - 1) / (16 * FT)), (unsigned)((q.rows + 16 * RT - 1) / (16 * RT)));
    if (in == HIN_F32) hipLaunchKernelGGL((k_layer_fp16_rows<FT, RT, HIN_F32>), grid, dim3(SKH_W * 64), 0, st, q);
    else if (in == HIN_ROWS) hipLaunchKernelGGL((k_layer_fp16_rows<FT, RT, HIN_ROWS>), grid, dim3(SKH_W * 64), 0, st, q);
    else hipLaunchKernelGGL((k_layer_fp16_rows<FT, RT, HIN_BLOCKED>), grid, dim3(SKH_W * 64), 0, st, q);
}
}  // namespace

aq_status launch_layer_fp16(const Fp16Layer& L, const void* in, int in_mode, void* out, int64_t rows,
                            hipStream_t st) {
    if (rows < 1) return AQ_OK;
    if (L.KS16 % 4 != 0 || L.NT < 1) return AQ_ESHAPE;
    _Float16* o = (_Float16*)out;
    // whole aligned pieces of 8 consecutive k: runs of consecutive k are multiples of 8 long, and every
    // run starts at an element offset that is a multiple of 8 (binary16: 16 bytes) or 4 (fp32: 16 bytes,
    // uint8: 4 bytes)
    const int unit = in_mode == 0 ? 8 : 4;
    const bool piece = ((uintptr_t)in & 15) == 0 &&
                       (L.fc ? L.K % 8 == 0 : ((L.kw * L.in_c) % 8 == 0 && L.in_c % unit == 0));
    // Tile: 128 rows x 256 features (hidden layers: the conversion of an fp32 observation piece does not
    // fit the register budget beside 128 accumulators) when that still gives every CU two workgroups,
    // 64 x 256 when it gives one, else 32 x 128 (few rows or few features: as many workgroups as possible).
    auto wgs = [&](int mt, int nb) {
        return ((rows + 32 * mt - 1) / (32 * mt)) * (int64_t)((L.NT + HW * nb - 1) / (HW * nb));
    };
    // few rows: small output tiles with K split over a workgroup's waves, whenever the tiled kernel would leave most CUs
    // without a workgroup
    if (fp16_layer_is_skinny(L, in_mode, rows)) {
        int ft = 1, rt = 1;
        few_row_tile(L.N, rows, L.head_argmax != nullptr, &ft, &rt);
        const int flags = (L.relu ? HF_RELU : 0) | (L.head_tanh ? HF_TANH : 0) | (L.head_argmax ? HF_ARGMAX : 0) | (L.out_blocked ? HF_BLOCKED : 0);
        const HalfRows q{L.wp, L.bias, in, o, L.head_argmax ? (void*)L.head_argmax : (void*)L.head_actions, L.K, L.N, L.KS16, (int)rows, flags};
        const int mode = L.in_blocked ? HIN_BLOCKED : in_mode == 1 ? HIN_F32 : HIN_ROWS;
        if (ft == 1 && rt == 1) launch_rows<1, 1>(q, mode, st);
        else if (ft == 1) launch_rows<1, 2>(q, mode, st);
        else if (rt == 1) launch_rows<2, 1>(q, mode, st);
        else launch_rows<2, 2>(q, mode, st);
        return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
    }
    if (in_mode == 0 && L.NT > HW && wgs(4, 2) >= 512) launch_layer_cfg<4, 2>(L, in, in_mode, piece, o, rows, st);
    else if (in_mode == 0 && L.NT > HW && wgs(2, 2) >= 256) launch_layer_cfg<2, 2>(L, in, in_mode, piece, o, rows, st);
    else launch_layer_cfg<1, 1>(L, in, in_mode, piece, o, rows, st);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_fp16_ln_tanh(void* x, int64_t rows, int N, const float* gamma, const float* beta, float eps,
                              hipStream_t st) {
    if (rows < 1) return AQ_OK;
    _Float16* xh = (_Float16*)x;
    LnForm f;
    if (!ln_form(rows, N, &f)) {
        hipLaunchKernelGGL(k_fp16_ln_tanh_long, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st, xh, rows, N, gamma, beta, eps);
        return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
    }
    const bool vec = N % 4 == 0 && ((uintptr_t)x & 7) == 0 && (((uintptr_t)gamma | (uintptr_t)beta) & 15) == 0;
    const dim3 grid((unsigned)(f.w == 1 ? (rows + 3) / 4 : rows));
    ln_dispatch(f, [&](auto w, auto p) {
        constexpr int W = decltype(w)::value, P = decltype(p)::value;
        auto go = [&](auto k) { hipLaunchKernelGGL(k, grid, dim3(256), 0, st, xh, rows, N, gamma, beta, eps); };
        if (vec) go(k_fp16_ln_tanh<W, P, true>);
        else go(k_fp16_ln_tanh<W, P, false>);
    });
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

aq_status launch_fp16_head(const void* y, int64_t rows, int N, int head, void* actions, hipStream_t st) {
    const int64_t n = head == AQ_HEAD_ARGMAX ? rows : rows * N;
    hipLaunchKernelGGL(k_fp16_head, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const _Float16*)y, rows, N,
                       head, actions);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

}  // namespace aq

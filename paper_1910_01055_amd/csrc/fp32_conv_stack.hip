// The leading convolutions of a frame policy in full precision, one launch, one workgroup per image: the counterpart of the
// 8-bit and half-precision convolution stacks for the learner's calibration and the fp32 actor.  The frame (8-bit codes)
// and every intermediate map (fp32) stay in LDS; only the last map goes to global memory.  Ranges of the input and of
// every map are collected on the way.
//
// Products.  The fp32 matrix instructions run at a sixteenth of the bf16 rate.  An fp32 value is exactly the sum of three
// bf16 values (8 + 8 + 8 bits of significand, each the rounded rest of the one before), so w x is the sum of nine bf16
// products, exact in fp32; the three smallest (together below 2^-23 of |w x|, 2^-25 of it typically) are left out and six
// v_mfma_f32_16x16x32_bf16 take the place of eight v_mfma_f32_16x16x4_f32 of twice their time, 3 for the first layer, whose
// codes are bf16 values as they are.  Sums stay in fp32, with one rounding per 32 products and term instead of one per 4.
// Error against 64 bits (2-norm, whole fp32 forwards of 150 random frame policies: 52 to 100 pixels a side, 1 to 4 channels): 3.36e-7
// on average, with the fp32 instructions throughout 3.53e-7; 0.95 times theirs by the geometric mean, 0.8 to 1.2 times on single ones.
// A layer with weights or inputs whose parts would leave bf16's range (not finite, rounding to infinity, or below 2^-100 and
// not zero) takes the fp32 instructions on the values themselves: no part of an infinite value meets a zero.
//
// A wavefront owns 32 or 64 features x a group of 16-position tiles x a part of K: weights pass the CU's vector memory path
// once per group, and each activation operand, split on its way from LDS (5.5 vector instructions a value), feeds two or four
// feature tiles.  The parts of K lie side by side in LDS; then all threads add them up and finish the map (bias, ReLU, range).
// Layer sizes and what LDS is left set groups and parts (plan_layer).
//
// Bound by the splitting and the matrix cores in turn: 84 x 84 x 4 through 32, 64 and 64 channels at 256 images takes 35 us, vector
// instructions 46 % and matrix instructions 30 % of it, hardly at once (the two wavefronts of a SIMD reach the same phase together);
// a third of the LDS time is bank conflicts (3.6 k of 71 k clocks), 11 registers are spilled.  As three launches of the per-layer
// fp32 kernel with the input's range in front 5 + 35 + 29.5 + 20 us.
#include "fp32_split.hpp"

namespace aq {

namespace {
constexpr int CF_W = 8;             // wavefronts per workgroup, two on a SIMD
constexpr int CF_T = CF_W * 64;
constexpr int CF_MAXC = 4;          // convolution layers at most
constexpr size_t CF_MAX_LDS = 160 * 1024;
constexpr int CF_ACC = 16;          // accumulator tiles of a wavefront at most: 2 x 8 or 4 x 4 (features x positions)
constexpr int CF_LOAD = 6;          // 16-byte pieces of the frame that a thread has in flight

struct CfLayer {
    const char* w;     // split weights (k_keep_params), then a word per block: special values in it
    const float* wrow; // the weights as given
    const float* b;
    int K, N, KS, ft;  // k-steps of 32, tiles of 16 features
    int fw;            // feature tiles of a wavefront: 2 or 4
    int R, ow;         // output positions, per row
    int px, py;        // LDS bytes (frame) or floats (maps) from a position's window to the next one's, along x and y
    int in_off, out_off, part_off;  // LDS bytes: input, output (part 0 of K), the other parts
    int out_ld;        // floats from position to position of the output map
    int run, row, pix; // of the input: values per window row; LDS distance of rows; map: LDS floats per pixel
    int in_c;
    int b_at;          // where its biases begin among all
    int k_off;         // LDS: where each piece of 8 k lies relative to a window's first value
    int per, pg, kp;   // wavefronts per feature group, as position groups x parts of K
    int relu;
};
struct CfArgs {
    int nc, in_h, row_bytes, row_ld;
    int64_t frame_bytes;
    int flag_off, range_off, bias_off, biases;  // LDS: per layer whether it holds special values; per tensor and wavefront
                                                // the range; all layers' biases
    CfLayer L[CF_MAXC];
};

// eight bytes -> bf16 (exact: at most 8 bits)
__device__ __forceinline__ bf8 codes_bf16(uint32_t a, uint32_t b) {
    v4i r;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        r[i] = (int)pack_bf16((float)((a >> (16 * i)) & 255u), (float)((a >> (16 * i + 8)) & 255u));
        r[2 + i] = (int)pack_bf16((float)((b >> (16 * i)) & 255u), (float)((b >> (16 * i + 8)) & 255u));
    }
    return __builtin_bit_cast(bf8, r);
}

// One wavefront's share of a layer: feature tiles f0 .. f0 + FT - 1, PT position tiles, k-steps [s0, s1).  x0[p]: LDS address
// of the lane's window in tile p.  No branches around the products: tiles past the end repeat the last one and are not stored.
template <int FT, int PT, bool U8>
__device__ __forceinline__ void cf_run(const CfLayer& L, const char* smem, const int* __restrict__ koff, int f0, int s0, int s1,
                                       const int (&x0)[8], v4f (&acc)[CF_ACC], int lane) {
    const int g = lane >> 4, pieces = L.K >> 3;
    typedef const bf8 AQ_GLOBAL* gbf8_ptr;
    const char* const w0 = L.w + (int64_t)f0 * L.KS * 3072 + lane * 16;
    int wf[FT];
#pragma unroll
    for (int f = 0; f < FT; ++f) wf[f] = (f0 + f < L.ft ? f : L.ft - 1 - f0) * L.KS * 3072;
    bf8 wr[2][FT][3];  // [step parity][feature tile][part]
    auto fetch_w = [&](auto slot_c, int s) __attribute__((always_inline)) {
        constexpr int slot = decltype(slot_c)::value;
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int f = 0; f < FT; ++f) wr[slot][f][q] = *(gbf8_ptr)(w0 + (wf[f] + s * 3072 + q * 1024));
    };
    v4f c[PT][FT];
#pragma unroll
    for (int p = 0; p < PT; ++p)
#pragma unroll
        for (int f = 0; f < FT; ++f) c[p][f] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    auto off = [&](int s) { const int q = 4 * s + g; return koff[q < pieces ? q : pieces - 1]; };
    auto step = [&](auto slot_c, int ko) __attribute__((always_inline)) {
        constexpr int slot = decltype(slot_c)::value;
        if constexpr (U8) {
            uint2 b[PT];
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const uint32_t* q = (const uint32_t*)(smem + x0[p] + ko);
                b[p] = make_uint2(q[0], q[1]);
            }
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                const bf8 x = codes_bf16(b[p].x, b[p].y);
#pragma unroll
                for (int q = 2; q >= 0; --q)
#pragma unroll
                    for (int f = 0; f < FT; ++f) c[p][f] = mfma_bf16(wr[slot][f][q], x, c[p][f]);
            }
        } else {
            // a tile's values are read two tiles ahead and its parts made between the products of the one before it
            v4f xa[2], xb[2];
            bf8 x[2][3];
#pragma unroll
            for (int p = 0; p < 2 && p < PT; ++p) {
                xa[p] = *(const v4f*)(smem + x0[p] + ko);
                xb[p] = *(const v4f*)(smem + x0[p] + ko + 16);
            }
            split8(xa[0], xb[0], x[0]);
#pragma unroll
            for (int p = 0; p < PT; ++p) {
                if (p + 2 < PT) {
                    xa[p & 1] = *(const v4f*)(smem + x0[p + 2 < PT ? p + 2 : p] + ko);
                    xb[p & 1] = *(const v4f*)(smem + x0[p + 2 < PT ? p + 2 : p] + ko + 16);
                }
                if (p + 1 < PT) split8(xa[(p + 1) & 1], xb[(p + 1) & 1], x[(p + 1) & 1]);
                mfma_split<FT>(wr[slot], x[p & 1], c[p]);
            }
        }
    };
    const int last = s1 - 1;
    int ko = off(s0);
    fetch_w(std::integral_constant<int, 0>{}, s0);
    int s = s0;
    for (; s + 1 < s1; s += 2) {
        fetch_w(std::integral_constant<int, 1>{}, s + 1);
        const int k1 = off(s + 1);
        step(std::integral_constant<int, 0>{}, ko);
        const int nx = s + 2 < s1 ? s + 2 : last;
        fetch_w(std::integral_constant<int, 0>{}, nx);
        ko = off(nx);
        step(std::integral_constant<int, 1>{}, k1);
    }
    if (s < s1) step(std::integral_constant<int, 0>{}, ko);
#pragma unroll
    for (int p = 0; p < PT; ++p)
#pragma unroll
        for (int f = 0; f < FT; ++f) acc[p * FT + f] = c[p][f];
}
// The same on the fp32 instructions, weights as given, zeros behind K on both sides
template <int FT>
__device__ __forceinline__ void cf_run_whole(const CfLayer& L, const char* smem, const int* koff, int f0, int s0, int s1, bool u8,
                                             const int (&x0)[8], v4f (&acc)[CF_ACC], int lane) {
    const int g = lane >> 4;
    const v4f z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < CF_ACC; ++i) acc[i] = z;
    for (int s = s0; s < s1; ++s) {
        const int k = 32 * s + 8 * g, ko = koff[k < L.K ? k >> 3 : 0];
        v4f w[FT][2];
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            const int n = (f0 + f) * 16 + (lane & 15);
            const bool ok = n < L.N && k < L.K;
            const float* p = L.wrow + (ok ? (int64_t)n * L.K + k : 0);
            w[f][0] = *(const v4f_u*)p;
            w[f][1] = *(const v4f_u*)(p + 4);
            if (!ok) w[f][0] = w[f][1] = z;
        }
#pragma unroll
        for (int p = 0; p < CF_ACC / FT; ++p) {
            v4f lo, hi;
            if (u8) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    lo[i] = (float)(uint8_t)smem[x0[p] + ko + i];
                    hi[i] = (float)(uint8_t)smem[x0[p] + ko + 4 + i];
                }
            } else {
                lo = *(const v4f*)(smem + x0[p] + ko);
                hi = *(const v4f*)(smem + x0[p] + ko + 16);
            }
            if (k >= L.K) lo = hi = z;
#pragma unroll
            for (int f = 0; f < FT; ++f) acc[p * FT + f] = mfma_whole(w[f][0], w[f][1], lo, hi, acc[p * FT + f]);
        }
    }
}

__global__ __launch_bounds__(CF_T) void k_fp32_conv_stack(const CfArgs A, const uint8_t* __restrict__ frames, float* __restrict__ out,
                                                         RangeSlot* __restrict__ slots) {
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int64_t img = blockIdx.x;
    uint32_t* const flags = (uint32_t*)(smem + A.flag_off);
    // this wavefront's share of a layer
    struct Share {
        int f0, s0, s1, kpi, t0, np, ptn;
        bool busy;
    };
    auto share_of = [&](const CfLayer& L) {
        Share h;
        const int grp = wave / L.per, sub = wave - grp * L.per, pgi = sub / L.kp;
        const int tiles = (L.R + 15) >> 4, spk = (L.KS + L.kp - 1) / L.kp;
        h.kpi = sub - pgi * L.kp;
        h.ptn = (tiles + L.pg - 1) / L.pg;
        h.t0 = pgi * h.ptn;
        h.np = tiles - h.t0 < h.ptn ? tiles - h.t0 : h.ptn;
        h.s0 = h.kpi * spk;
        h.s1 = h.s0 + spk < L.KS ? h.s0 + spk : L.KS;
        h.f0 = grp * L.fw;
        h.busy = h.f0 < L.ft && h.np > 0;
        return h;
    };
    float2* const ranges = (float2*)(smem + A.range_off);  // per tensor and wavefront
    float* const biases = (float*)(smem + A.bias_off);
    // The frame's range is collected from the registers it passes through.
    uint32_t lo8 = 255, hi8 = 0;
    auto note4 = [&](uint32_t v) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t c = (v >> (8 * j)) & 255u;
            lo8 = lo8 < c ? lo8 : c;
            hi8 = hi8 > c ? hi8 : c;
        }
    };
    const uint8_t* const src = frames + img * A.frame_bytes;
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    typedef u4 u4_u __attribute__((aligned(1)));
    // (biases first, so that they wait for nothing of the frame)
    for (int i = tid; i < A.biases; i += CF_T) {
        const float* b = nullptr;
        int j = i;
#pragma unroll
        for (int l = 0; l < CF_MAXC; ++l) {
            if (l >= A.nc || b) continue;
            if (j < A.L[l].N) b = A.L[l].b ? A.L[l].b + j : (const float*)-1;
            else j -= A.L[l].N;
        }
        biases[i] = b == (const float*)-1 ? 0.0f : *b;
    }
    const bool whole_rows = A.row_ld == A.row_bytes;  // the frame is one run of bytes in LDS too
    const int nq = whole_rows ? (int)(A.frame_bytes >> 4) : 0;
    u4 fr[CF_LOAD];
#pragma unroll
    for (int u = 0; u < CF_LOAD; ++u) {
        const int i = tid + u * CF_T;
        if (i < nq) fr[u] = *(const u4_u*)(src + (int64_t)i * 16);
    }
    // meanwhile: wave l: where each piece of 8 k of layer l lies, and whether a block of its weights holds special values
    if (wave < A.nc) {
        const CfLayer& L = A.L[wave];
        int* ko = (int*)(smem + L.k_off);
        const float inv_run = 1.0f / (float)L.run, inv_c = 1.0f / (float)L.in_c;
        for (int q = lane; q < L.K >> 3; q += 64) {
            const int k = q * 8, ky = (int)(((float)k + 0.5f) * inv_run), r = k - ky * L.run;
            const int pc = (int)(((float)r + 0.5f) * inv_c);
            // first layer: bytes; maps: floats, padded from pixel to pixel
            ko[q] = wave == 0 ? ky * L.row + r : 4 * (ky * L.row + pc * L.pix + (r - pc * L.in_c));
        }
        const uint32_t* f = (const uint32_t*)(L.w + (int64_t)L.ft * L.KS * 3072);
        uint32_t any = 0;
        for (int i = lane; i < L.ft * L.KS; i += 64) any |= f[i];
        const bool sp = __ballot(any != 0) != 0;
        if (lane == 0) flags[wave] = sp;
    }
#pragma unroll
    for (int u = 0; u < CF_LOAD; ++u) {
        const int i = tid + u * CF_T;
        if (i < nq) {
            *(u4*)(smem + A.L[0].in_off + i * 16) = fr[u];
#pragma unroll
            for (int j = 0; j < 4; ++j) note4(fr[u][j]);
        }
    }
    for (int i = tid + CF_LOAD * CF_T; i < nq; i += CF_T) {
        const u4 v = *(const u4_u*)(src + (int64_t)i * 16);
        *(u4*)(smem + A.L[0].in_off + i * 16) = v;
#pragma unroll
        for (int j = 0; j < 4; ++j) note4(v[j]);
    }
    if (whole_rows) {  // the last bytes
        for (int64_t i = (int64_t)nq * 16 + tid; i < A.frame_bytes; i += CF_T) {
            smem[A.L[0].in_off + i] = src[i];
            note4(src[i] * 0x01010101u);
        }
    } else {  // row by row, each padded to 8 bytes
        const int wpr = A.row_ld >> 2, words = wpr * A.in_h;
        const float inv = 1.0f / (float)wpr;
#pragma unroll 8
        for (int i = tid; i < words; i += CF_T) {
            const int y = (int)(((float)i + 0.5f) * inv), x = (i - y * wpr) * 4, left = A.row_bytes - x;
            const uint8_t* p = src + (int64_t)y * A.row_bytes + x;
            uint32_t v = 0;
            if (left >= 4) {
                v = *(const u32_u*)p;
                note4(v);
            } else {
                for (int j = 0; j < left; ++j) {
                    v |= (uint32_t)p[j] << (8 * j);
                    note4(p[j] * 0x01010101u);
                }
            }
            *(uint32_t*)(smem + A.L[0].in_off + y * A.row_ld + x) = v;
        }
    }
    if (slots) {
        float lo = lo8 <= hi8 ? (float)lo8 : INFINITY, hi = lo8 <= hi8 ? (float)hi8 : -INFINITY;
        wave_range(lo, hi);
        if (lane == 0) ranges[wave] = make_float2(lo, hi);
    }
    lds_barrier();
#pragma unroll 1
    for (int l = 0; l < A.nc; ++l) {
        const CfLayer& L = A.L[l];
        const Share sh = share_of(L);
        const int f0 = sh.f0, s0 = sh.s0, s1 = sh.s1, kpi = sh.kpi, t0 = sh.t0, np = sh.np, ptn = sh.ptn;
        const bool busy = sh.busy;
        const bool special = __builtin_amdgcn_readfirstlane(flags[l]) != 0;  // (a scalar: MFMAs stand behind it)
        if (busy) {
            v4f acc[CF_ACC];
            int x0[8];
            const float inv_ow = 1.0f / (float)L.ow;
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                int r = (t0 + p) * 16 + i16;
                r = r < L.R ? r : L.R - 1;
                const int oy = (int)(((float)r + 0.5f) * inv_ow), ox = r - oy * L.ow;
                const int o = oy * L.py + ox * L.px;
                x0[p] = L.in_off + (l == 0 ? o : 4 * o);
            }
            const int* koff = (const int*)(smem + L.k_off);
            if (special || s0 >= s1) {
                if (L.fw == 4) cf_run_whole<4>(L, smem, koff, f0, s0, s1, l == 0, x0, acc, lane);
                else cf_run_whole<2>(L, smem, koff, f0, s0, s1, l == 0, x0, acc, lane);
            } else {
                switch (l == 0 ? ptn : L.fw == 2 ? 8 + ptn : 16 + ptn) {
#define CF_CASE(PT)                                                                          \
    case PT: cf_run<2, PT, true>(L, smem, koff, f0, s0, s1, x0, acc, lane); break;            \
    case 8 + PT: cf_run<2, PT, false>(L, smem, koff, f0, s0, s1, x0, acc, lane); break
                    CF_CASE(1); CF_CASE(2); CF_CASE(3); CF_CASE(4); CF_CASE(5); CF_CASE(6); CF_CASE(7); CF_CASE(8);
#undef CF_CASE
                    case 17: cf_run<4, 1, false>(L, smem, koff, f0, s0, s1, x0, acc, lane); break;
                    case 18: cf_run<4, 2, false>(L, smem, koff, f0, s0, s1, x0, acc, lane); break;
                    case 19: cf_run<4, 3, false>(L, smem, koff, f0, s0, s1, x0, acc, lane); break;
                }
            }
            // this part of K's sums
            float* map = (float*)(smem + (kpi ? L.part_off : L.out_off)) + (kpi ? (int64_t)(kpi - 1) * L.R * L.out_ld : 0);
            auto store = [&](auto fw_c) __attribute__((always_inline)) {
                constexpr int FT = decltype(fw_c)::value;
#pragma unroll
                for (int p = 0; p < CF_ACC / FT; ++p) {
                    if (p >= np) break;
                    const int r = (t0 + p) * 16 + i16;
                    float* d = map + r * L.out_ld + f0 * 16 + 4 * g;
#pragma unroll
                    for (int f = 0; f < FT; ++f)
                        if (r < L.R && (f0 + f) * 16 + 4 * g < L.N) *(v4f*)(d + 16 * f) = acc[p * FT + f];
                }
            };
            if (L.fw == 4) store(std::integral_constant<int, 4>{});
            else store(std::integral_constant<int, 2>{});
        }
        lds_barrier();
        // all threads: the parts' sum, bias, ReLU, range; the map in place, or the last one on its way out
        const bool last = l == A.nc - 1;
        float lo = INFINITY, hi = -INFINITY;
        uint32_t least = 0xffffffffu, most = 0;  // of the magnitudes' bits; zero minus one is the largest
        const int n4 = L.N >> 2, total = L.R * n4;
        const float inv_n4 = 1.0f / (float)n4;
        const int part = L.R * L.out_ld;
#pragma unroll 4
        for (int i = tid; i < total; i += CF_T) {
            const int r = (int)(((float)i + 0.5f) * inv_n4), n = (i - r * n4) * 4;
            float* d = (float*)(smem + L.out_off) + r * L.out_ld + n;
            const float* q = (const float*)(smem + L.part_off) + r * L.out_ld + n;
            v4f v = *(const v4f*)d;
            for (int k = 1; k < L.kp; ++k) v += *(const v4f*)(q + (k - 1) * part);
            v += *(const v4f*)(biases + L.b_at + n);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (L.relu) v[j] = v[j] > 0.0f ? v[j] : 0.0f;
                lo = fminf(lo, v[j]);
                hi = fmaxf(hi, v[j]);
                const uint32_t u = __float_as_uint(v[j]) & 0x7fffffffu;
                least = least < u - 1 ? least : u - 1;
                most = most > u ? most : u;
            }
            if (last) *(v4f_u*)(out + (img * L.R + r) * L.N + n) = v;
            else *(v4f*)d = v;
        }
        if (!last && __ballot(least < kSplitLeast - 1 || most >= kSplitMost) != 0 && lane == 0) atomicOr(&flags[l + 1], 1u);
        if (slots) {
            wave_range(lo, hi);
            if (lane == 0) ranges[(l + 1) * CF_W + wave] = make_float2(lo, hi);
        }
        lds_barrier();
    }
    if (slots && tid <= A.nc) {  // thread t: tensor t
        float lo = INFINITY, hi = -INFINITY;
#pragma unroll
        for (int i = 0; i < CF_W; ++i) {
            lo = fminf(lo, ranges[tid * CF_W + i].x);
            hi = fmaxf(hi, ranges[tid * CF_W + i].y);
        }
        RangeSlot* s = slots + tid * kRangeSlots + blockIdx.x % kRangeSlots;
        if (lo <= hi) {
            atomicMax(&s->not_lo, ~f2key(lo));
            atomicMax(&s->hi, f2key(hi));
        }
    }
}

// Feature tiles of a wavefront, position groups and parts of K of a layer: so that the slowest of the matrix cores (16 clocks
// an MFMA, two wavefronts on each SIMD), the splitting (48 instructions of 4 clocks for an operand) and the weights' way through the
// vector memory path (52 bytes a clock, once per position group) takes least; `spare` bytes of LDS hold parts of K.  (Two
// wavefronts on a SIMD hide about a quarter of matrix and vector instructions behind each other: measured.)  Returns those
// clocks, 0 where nothing fits.
double plan_layer(CfLayer& q, bool u8, int64_t spare) {
    double best = 1e300;
    const int tiles = (q.R + 15) / 16;
    const int64_t map = (int64_t)q.R * q.out_ld * 4;
    for (int fw = 2; fw <= (u8 || q.ft < 4 ? 2 : 4); fw += 2) {
        const int groups = (q.ft + fw - 1) / fw;
        if (groups > CF_W) continue;
        const int per = CF_W / groups;
        for (int kp = 1; kp <= per; ++kp) {
            const int pg = per / kp, pt = (tiles + pg - 1) / pg;
            if (pt > (fw == 4 ? 3 : 8) || (int64_t)(kp - 1) * map > spare) continue;
            const int steps = (q.KS + kp - 1) / kp;
            const int waves = groups * kp * ((tiles + pt - 1) / pt);  // with anything to do
            const double simd = (waves + 3) / 4;
            const double mm = simd * steps * pt * fw * (u8 ? 3 : 6) * 16, va = simd * steps * pt * (u8 ? 16 : 48) * 4;
            const double mem = (double)q.ft * q.KS * 3072 * pg / 52.0;
            const double busy = 0.75 * (mm + va), c = (busy > mem ? busy : mem) + 0.2 * (busy < mem ? busy : mem) + 150.0 * kp;
            if (c < best) {
                best = c;
                q.fw = fw;
                q.per = per;
                q.pg = pg;
                q.kp = kp;
            }
        }
    }
    return best < 1e300 ? best : 0.0;
}

bool plan_cf(const NetDev& net, CfArgs* A, size_t* lds, double* clocks) {
    if (!net.in_u8) return false;
    int nc = 0;
    while (nc < net.n_layers && !(net.L[nc].kh == 1 && net.L[nc].kw == 1 && net.L[nc].in_h == 1 && net.L[nc].in_w == 1)) ++nc;
    if (nc < 1 || nc > CF_MAXC || nc >= net.n_layers) return false;
    const LayerDev& F = net.L[0];
    A->nc = nc;
    A->in_h = F.in_h;
    A->row_bytes = F.in_w * F.in_c;
    A->row_ld = (A->row_bytes + 7) & ~7;
    A->frame_bytes = (int64_t)F.in_h * A->row_bytes;
    if ((int64_t)A->row_ld * F.in_h > (int64_t)CF_MAX_LDS) return false;
    // LDS: flags, tables and ranges, then what the maps share: even ones from its begin, odd ones from its end
    size_t at = 64;
    for (int l = 0; l < nc; ++l) {
        const LayerDev& X = net.L[l];
        CfLayer& q = A->L[l];
        if (X.act == AQ_ACT_LN_TANH) return false;
        const int run = X.kw * X.in_c;
        if (l == 0 ? run % 8 != 0 || (X.stride * X.in_c) % 4 != 0 : X.in_c % 8 != 0) return false;
        if (X.N % (l == nc - 1 ? 4 : 8) != 0) return false;
        if ((int64_t)X.oh * X.ow > 16 * CF_ACC * CF_W || X.K > 32768) return false;
        q.K = X.K;
        q.N = X.N;
        q.KS = (X.K + 31) / 32;
        q.ft = (X.N + 15) / 16;
        q.R = X.oh * X.ow;
        q.ow = X.ow;
        q.in_c = X.in_c;
        q.run = run;
        q.pix = X.in_c + 4;
        q.row = l == 0 ? A->row_ld : X.in_w * q.pix;
        q.px = X.stride * (l == 0 ? X.in_c : q.pix);
        q.py = X.stride * q.row;
        q.out_ld = X.N + 4;
        q.relu = X.act == AQ_ACT_RELU;
        q.k_off = (int)at;
        at += (size_t)(q.K / 8) * 4;
    }
    A->flag_off = 0;
    at = (at + 15) & ~(size_t)15;
    A->range_off = (int)at;
    at += (size_t)(nc + 1) * CF_W * sizeof(float2);
    A->bias_off = (int)at;
    for (int l = 0; l < nc; ++l) {
        A->L[l].b_at = A->biases;
        A->biases += A->L[l].N;
    }
    at = (at + (size_t)A->biases * 4 + 15) & ~(size_t)15;
    int64_t in = ((int64_t)A->row_ld * F.in_h + 8 + 15) & ~(int64_t)15;
    for (int l = 0; l < nc; ++l) {
        CfLayer& q = A->L[l];
        const int64_t out = (int64_t)q.R * q.out_ld * 4, spare = (int64_t)CF_MAX_LDS - (int64_t)at - in - out;
        const double c = spare < 0 ? 0.0 : plan_layer(q, l == 0, spare);
        if (c == 0.0) return false;
        *clocks += c;
        q.in_off = l & 1 ? (int)(CF_MAX_LDS - in) : (int)at;
        q.out_off = l & 1 ? (int)at : (int)(CF_MAX_LDS - out);
        q.part_off = (int)at + (int)(l & 1 ? out : in);
        in = out;
    }
    *lds = CF_MAX_LDS;
    return true;
}
}  // namespace

int fp32_conv_stack_layers(const NetDev& net, Fp32StackWork* w) {
    CfArgs A{};
    size_t lds = 0;
    double clocks = 0.0;
    if (!plan_cf(net, &A, &lds, &clocks)) return 0;
    *w = Fp32StackWork{};
    w->round = clocks / 2400.0;
    w->ragged = 1e-3 * (double)A.frame_bytes * (A.row_bytes & 3 ? 2 : A.row_bytes & 7 ? 1 : 0);
    for (int l = 0; l < A.nc; ++l) {
        w->operands += 1e-6 * A.L[l].R * A.L[l].K;
        w->products += 1e-6 * A.L[l].R * A.L[l].K * A.L[l].N;
    }
    return A.nc;
}

// One launch, an image per CU and a round of 256 images after the other, or the layers' own launches, which spread a few images
// over several CUs, keep the chip full between rounds and, on many small frames, run at a rate that one image per CU does not
// reach.  fp32 forward, us (one launch / the layers'): 84 x 84 x 4 through 32, 64, 64 at 32 images 41.4 / 35.6, 49 41.4 / 40.9, 64
// 41.7 / 48.0, 256 45.9 / 86.4, 257 78.1 / 93.2, 768 113 / 181; 61 x 61 x 3 through 16, 32, 32 at 256 25.4 / 35.5, 512 42.0 / 64.1,
// 900 79.7 / 70.0, 2048 155 / 122; 52 x 52 x 1 through the same at 256 20.2 / 27.5, 513 42.5 / 37.2, 768 42.5 / 43.1, 2048 96.7 / 72.2.
// The estimates are fitted to 1639 measured pairs, 56 stacks of one to four layers on frames of 20 to 100 pixels a side and 1 to 4
// channels at 8 to 4096 images; what the rule takes is within 4 % of the faster one in 1588 of them and at most 13 % behind the layers'
// launches (tiny frames of a second round just begun).
bool fp32_conv_stack_faster(const Fp32StackWork& w, int nc, int64_t batch) {
    const double n = (double)batch, rounds = (double)((batch + 255) / 256);
    // (in the first round the layers' launches do not fill the chip and hide less behind each other)
    if (batch <= 256) return 3.15 * nc + n * (0.41 * w.operands + 0.0235 * w.products) > 3.4 + 1.5 * w.round + 0.07 * w.ragged;
    return 5.0 * nc + n * (0.556 * w.operands + 0.009 * w.products) > rounds * (4.07 + 1.36 * w.round + 0.24 * w.ragged);
}

aq_status launch_fp32_conv_stack(const NetDev& net, const F32Ptrs& ptrs, const void* frames, int64_t batch, float* out, RangeSlot* slots,
                                 hipStream_t st) {
    CfArgs A{};
    size_t lds = 0;
    double clocks = 0.0;
    if (!plan_cf(net, &A, &lds, &clocks)) return AQ_ESHAPE;
    for (int l = 0; l < A.nc; ++l) {
        A.L[l].w = (const char*)ptrs.wsp[l];
        A.L[l].wrow = ptrs.w[l];
        A.L[l].b = ptrs.b[l];
    }
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
        if (hip_failed(hipFuncSetAttribute((const void*)k_fp32_conv_stack, hipFuncAttributeMaxDynamicSharedMemorySize, (int)CF_MAX_LDS)))
            return AQ_EHIP;
        attr_set = true;
    }
    // (a grid's threads are counted in 32 bits)
    for (int64_t i0 = 0; i0 < batch; i0 += 1 << 22) {
        const int64_t n = batch - i0 < 1 << 22 ? batch - i0 : 1 << 22;
        hipLaunchKernelGGL(k_fp32_conv_stack, dim3((unsigned)n), dim3(CF_T), lds, st, A, (const uint8_t*)frames + i0 * A.frame_bytes,
                           out + i0 * A.L[A.nc - 1].R * A.L[A.nc - 1].N, slots);
    }
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

}  // namespace aq

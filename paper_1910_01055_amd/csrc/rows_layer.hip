// Wide fully connected 8-bit layers at some hundred to some thousand rows (Sec. 3.1 actor inference on the 8-bit policy of Sec. 3.2;
// policies wider than the whole-network kernels hold): one launch per layer, the layers' maps in operand order (blocked_map_bytes).
//
// A workgroup of 8 wavefronts takes 64 rows x 256 features; a wavefront 32 features, both halves of a tile by four row tiles of
// v_mfma_i32_16x16x64_i8.  Weights go from memory straight into operand registers, each byte once per workgroup; the rows' codes go
// through LDS, since all wavefronts read them: in operand order 16 bytes of K of all the workgroup's rows are contiguous in memory
// and in LDS.  Chunks of 256 bytes of K alternate between two buffers, requested one chunk ahead with their weights.  fp32 observations
// (first layer) are quantized on their way into LDS, all of K at once.
//
// What bounds it: the vector memory path, 20 KiB per k-step of 64 at 52 bytes a clock for 256 clocks of matrix work.  128 rows a
// workgroup, which ask for less, were slower up to 8000 rows (67-2048x3-21 at 2000 rows 56 us, at 4500 98): too few workgroups.
// The few-row kernel re-reads both operands for each 32 x 32 tile, the tiled one stages all of K before the first product with one
// wavefront per SIMD, byte by byte where rows are no whole pieces.  us before / now: 67-2048x3-21 at 640 rows 44.6 / 33.3, 1300
// 71.9 / 36.4, 4500 173 / 76; with a LayerNorm at 3000 160 / 78; 67-1300-1500-21 at 900 32.4 / 20.1, at 3000 336 / 30.
#include <atomic>

#include "int8_device.hpp"
#include "lanes.hpp"

namespace aq {
namespace {

constexpr int RL_W = 8, RL_T = RL_W * 64, RL_RT = 4;  // wavefronts, threads, 16-row tiles of a workgroup
constexpr int RL_KC = 16;                // pieces of 16 bytes of K per chunk
constexpr int RL_MAXK0 = 512;            // longest observation row
enum { RL_RELU = 1, RL_LN = 2 };

struct RowsLayer {
    const NetDev* net;
    const int8_t* wp;
    const int32_t *pack, *rshift, *z_w;
    const void* in;
    void* out;  // codes, or fp32 rows in front of a LayerNorm
    int64_t rows;
    int32_t K, N, KS, NT, layer, flags;
};

template <bool F32, bool ASYM, bool TAPS>
__global__ __launch_bounds__(RL_T) void k_layer_rows(const RowsLayer L, const TapParam<TAPS> tp) {
    extern __shared__ __align__(16) int8_t sm[];
    constexpr int RT = RL_RT, ROWS = 16 * RT, CHUNK = RL_KC * ROWS * 16;
    const TapArgs t = taps_of(tp);
    const NetDev& a = *L.net;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), b = lane & 15, g = lane >> 4;
    const int64_t row0 = (int64_t)blockIdx.y * ROWS, rows = L.rows, rpad = (rows + 15) / 16 * 16;
    const int K = L.K, KS = L.KS, N = L.N, NT = L.NT, ks = (KS + 1) >> 1, k16 = (K + 15) >> 4;
    const int own = (int)blockIdx.x * RL_W + wave;
    const bool active = own < NT;
    const int nt = active ? own : NT - 1;  // (a wavefront past the last tile goes along and stores nothing)
    // (pieces of K past the stored tiles read zeros: past the buffer's end)
    const int bytes = NT * KS * 1024;
    const auto w = __builtin_amdgcn_make_buffer_rsrc((void*)L.wp, 0, bytes, 0x00020000);
    const int lane_off = (g >> 1) * 1024 + (b + 32 * (g & 1)) * 16;
    auto weights = [&](int s, v4i (&o)[2]) __attribute__((always_inline)) {
        const int off = 2 * s + (g >> 1) < KS ? lane_off : bytes;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            o[h] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w, off, nt * KS * 1024 + s * 2048 + 256 * h, 0));
    };
    v4i acc[2][RT];
    int rs[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        acc[0][r] = acc[1][r] = v4i{0, 0, 0, 0};
        rs[r] = 0;
    }
    auto step = [&](const int8_t* x0, const v4i (&wr)[2], int s) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const v4i x = *(const v4i*)(x0 + r * 256);
            acc[0][r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wr[0], x, acc[0][r], 0, 0, 0);
            acc[1][r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wr[1], x, acc[1][r], 0, 0, 0);
            if (ASYM) {
                if (4 * s + g < k16)
#pragma unroll
                    for (int i = 0; i < 4; ++i) rs[r] = __builtin_amdgcn_sdot4(x[i], 0x01010101, rs[r], false);
            }
        }
    };
    const int8_t* const xl = sm + (g * ROWS + b) * 16;  // this lane's operand of a buffer's first k-step; a k-step is 4 pieces of K
    // this lane's constants: array lane % 16 / 4 of half lane % 4 (two halves), handed along the row's lanes
    const bool ln = L.flags & RL_LN;
    const bool fast = !ln && a.fast[L.layer] != 0;
    v4i cm = {0, 0, 0, 0};
    {
        const int arr = b >> 2;
        const int32_t* base = L.pack + arr * NT * 32;
        if (arr == 3 && !ln && !fast) base = L.rshift;
        cm = *(gv4i_ptr)(base + 32 * nt + 16 * (b & 1) + 4 * g);
    }

    if constexpr (F32) {
        const QuantScale qs0 = make_quant_scale(a.actq[0].s);
        const float zf0 = (float)a.actq[0].z;
        const int quads = ks * 16, total = ROWS * quads;  // up to whole k-steps
        const float inv = 1.0f / (float)quads;
        typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
        constexpr int U = 4;
        for (int base = tid; base < total; base += U * RL_T) {
            float4 v[U];
            int m[U], k[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int idx = base + u * RL_T;
                m[u] = (int)(((float)idx + 0.5f) * inv);
                k[u] = (idx - m[u] * quads) * 4;
                v[u] = float4{0.0f, 0.0f, 0.0f, 0.0f};
                const int64_t row = row0 + m[u];
                if (idx >= total || row >= rows || k[u] >= K) continue;
                const float* src = (const float*)L.in + row * K + k[u];
                const int last = K - 1 - k[u];
                if (last >= 3 || row + 1 < rows - 2) {  // (words past the row's end are the next rows', which exist)
                    const f4u x = *(const f4u*)src;
                    v[u] = float4{x[0], x[1], x[2], x[3]};
                } else {
                    v[u].x = src[0];
                    if (last >= 1) v[u].y = src[1];
                    if (last >= 2) v[u].z = src[2];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int idx = base + u * RL_T;
                if (idx >= total) break;
                uint32_t pack = 0;
                if (k[u] < K) {
                    const int have = K - k[u];
                    pack = quant_u8x4(v[u], qs0, zf0);
                    if (TAPS) {
                        if (t.a0 && blockIdx.x == 0 && row0 + m[u] < rows)
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (i < have) t.a0[(row0 + m[u]) * K + k[u] + i] = (uint8_t)(pack >> (8 * i));
                    }
                    pack ^= 0x80808080u;
                    if (have < 4) pack &= (1u << (8 * have)) - 1u;
                }
                *(uint32_t*)(sm + ((k[u] >> 4) * ROWS + m[u]) * 16 + (k[u] & 15)) = pack;
            }
        }
        v4i wr[2][2];
        weights(0, wr[0]);
        lds_barrier();
        for (int s = 0; s < ks; s += 2) {
            if (s + 1 < ks) weights(s + 1, wr[1]);
            step(xl + s * 4 * ROWS * 16, wr[0], s);
            if (s + 2 < ks) weights(s + 2, wr[0]);
            if (s + 1 < ks) step(xl + (s + 1) * 4 * ROWS * 16, wr[1], s + 1);
        }
    } else {
        // rows past the batch re-read the last one, pieces past K the last one (the weights are zeros there)
        constexpr int PER = RL_KC * ROWS / RL_T;  // pieces of a chunk per thread
        v4i st[PER];
        auto fetch = [&](int c, auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;
            const int e = u * RL_T + tid, p = c * RL_KC + e / ROWS;
            const int64_t row = row0 + e % ROWS;
            st[u] = *(gv4i_ptr)((const int8_t*)L.in + ((int64_t)(p < k16 ? p : k16 - 1) * rpad + (row < rows ? row : rows - 1)) * 16);
        };
        auto store = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < PER; ++u) *(v4i*)(sm + (c & 1) * CHUNK + (u * RL_T + tid) * 16) = st[u];
        };
        constexpr int S = RL_KC / 4;  // k-steps of a chunk
        const int chunks = (ks + S - 1) / S;
        v4i wr[S][2];
        // The next chunk's requests go out one k-step's at a time, each behind the products that free its registers: in one run in
        // front of the chunk's products they kept all wavefronts from those.  (And without a condition: with one the compiler cannot
        // count what is in flight and waits for all of it.)
        static_for<0, PER>([&](auto u_c) __attribute__((always_inline)) { fetch(0, u_c); });
#pragma unroll
        for (int j = 0; j < S; ++j) weights(j, wr[j]);
        store(0);
        auto chunk = [&](auto more_c, int c) __attribute__((always_inline)) {
            constexpr bool more = decltype(more_c)::value;
            lds_barrier();  // the chunk is in LDS, and nobody reads the other buffer any more
            static_for<0, S>([&](auto j_c) __attribute__((always_inline)) {
                constexpr int j = decltype(j_c)::value;
                step(xl + (c & 1) * CHUNK + j * 4 * ROWS * 16, wr[j], c * S + j);
                if constexpr (more) {
                    if constexpr (j < PER) fetch(c + 1, j_c);
                    weights((c + 1) * S + j, wr[j]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            if (more) store(c + 1);
        };
        static_assert(PER <= S, "a piece of the rows per k-step at most");
        for (int c = 0; c + 1 < chunks; ++c) chunk(std::true_type{}, c);
        chunk(std::false_type{}, chunks - 1);
    }
    if (!active) return;

    const int z_out = a.actq[L.layer + 1].z;
    const int lo = (L.flags & RL_RELU) ? z_out : 0;
    int lo_v = lo;
    asm volatile("" : "+v"(lo_v));
    if (ASYM) {
        const int zw = L.z_w[0] - 128;
#pragma unroll
        for (int r = 0; r < RT; ++r) rs[r] = -zw * sum_rows4(rs[r]);
    }
    LayerTaps T{nullptr, nullptr, nullptr};
    if (TAPS) T = LayerTaps{t.acc[L.layer], t.act[L.layer], t.ln[L.layer]};
    static_for<0, 2>([&](auto h_c) __attribute__((always_inline)) {
        constexpr int h = decltype(h_c)::value;
        const int n0 = nt * 32 + 16 * h + 4 * g;
        int bias[4], mul[4], rz[4], sh[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bias[i] = row_bcast_mov<h>(cm[i]);
            mul[i] = row_bcast_mov<4 + h>(cm[i]);
            rz[i] = row_bcast_mov<8 + h>(cm[i]);
            sh[i] = row_bcast_mov<12 + h>(cm[i]);
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int64_t row = row0 + 16 * r + b;
            int val[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                val[i] = acc[h][r][i] + bias[i];
                if (ASYM) val[i] += rs[r];
                if (TAPS) {
                    if (T.acc && row < rows && n0 + i < N) T.acc[row * N + n0 + i] = val[i];
                }
            }
            if (ln) {
                float* o = (float*)L.out + row * N + n0;
                if (row < rows) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (n0 + i < N) o[i] = (float)val[i] * __int_as_float(mul[i]);
                }
            } else {
                uint32_t pack = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    int code;
                    if (fast) code = clamp_code((__mulhi(val[i], mul[i]) + rz[i]) >> sh[i], lo_v, 255);
                    else code = requant_code(val[i], mul[i], sh[i], z_out, lo);
                    if (TAPS) {
                        if (T.act && row < rows && n0 + i < N) T.act[row * N + n0 + i] = (uint8_t)code;
                    }
                    pack |= (uint32_t)code << (8 * i);
                }
                pack ^= 0x80808080u;
                const int keep = N - n0;  // features past N up to the end of their 16: zeros
                if (keep < 4) pack = keep <= 0 ? 0u : pack & ((1u << (8 * keep)) - 1u);
                if (row < rows && n0 < ((N + 15) & ~15)) *(uint32_t*)((int8_t*)L.out + ((int64_t)(n0 >> 4) * rpad + row) * 16 + (n0 & 15)) = pack;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    });
}

template <bool F32, bool ASYM, bool TAPS>
aq_status go(const RowsLayer& q, const TapArgs& t, hipStream_t st) {
    auto* const k = k_layer_rows<F32, ASYM, TAPS>;
    constexpr int RT = RL_RT;
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
        if (hip_failed(hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024))) return AQ_EHIP;
        attr_set = true;
    }
    const size_t lds = F32 ? (size_t)((q.KS + 1) / 2 * 64) * 16 * RT : (size_t)2 * RL_KC * 16 * RT * 16;
    const dim3 grid((unsigned)((q.NT + RL_W - 1) / RL_W), (unsigned)((q.rows + 16 * RT - 1) / (16 * RT)));
    hipLaunchKernelGGL(k, grid, dim3(RL_T), lds, st, q, TapParam<TAPS>(t));
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}
}  // namespace

// From 450 rows on: us on the few-row kernel / here, the first layer of 67-2048-2048-256-21 at 470 rows 31.5 / 23.3 for the policy; but not
// while the few-row kernel takes that layer in tiles of 16 rows, four rounds of them at most: 384-1100-300-9 at 450 rows 13.7 / 16.3,
// 384-512-2048-9 at 560 16.6 / 20.3, per-tensor 200-700-1500-9 at 466 16.1 / 17.9.  A
// layer behind the first, which the few-row kernel reads in the same order, comes here where the grid holds enough workgroups; for
// whole policies us there / here, per-channel weights: N = 512 at 1800 rows 18.6 / 19.1, 2200 20.6 / 19.2; 700 at 1400 18.0 / 18.9, 1600
// 19.9 / 19.3; 900 at 1100 17.6 / 18.5, 1300 19.3 / 18.8; two of 1100 at 900 25.1 / 28.4, 1200 30.0 / 29.3; two of 2048 at 512 29.8 / 34.2,
// 700 36.7 / 35.4.  Per-tensor weights, whose row sums all wavefronts add up here: two of 2048 at 768 38.9 / 43.3; 700 at 1600 21.1 / 22.1,
// 2000 23.3 / 22.9.  Rows of more than 2048 values always come here (2500 of 2500 at 512 rows 29.6 / 24.4).  The caller ends it where no
// layer behind reads its maps any more: layers of fewer than 16 feature tiles, the last one among them, read them on the few-row kernel
// (layer_uses_skinny), at up to eight tiles for 8128 rows.
bool layer_uses_rows(const FwdArgs& a, int l) {
    const NetDev& n = a.net;
    const LayerDev& L = n.L[l];
    auto fc = [](const LayerDev& X) { return X.kh == 1 && X.kw == 1 && X.in_h == 1 && X.in_w == 1; };
    if (l >= n.n_layers - 1 || !fc(L) || L.NT < 16 || a.c.batch < 450 || a.w4[l]) return false;
    if ((int64_t)L.NT * L.KS * 1024 >= 0x7fffffff) return false;
    if (l == 0) {
        int ft = 0, rt = 0;
        few_row_tile(L.N, a.c.batch, false, &ft, &rt);
        return !n.in_u8 && L.K <= RL_MAXK0 && (rt > 1 || !layer_uses_skinny(a, l));
    }
    const int64_t groups = (L.NT + RL_W - 1) / RL_W, blocks = (a.c.batch + 16 * RL_RT - 1) / (16 * RL_RT);
    if (L.K <= 2048 && groups * blocks < 60 + 5 * groups + (n.asym ? 20 : 0) && layer_uses_skinny(a, l)) return false;
    return fc(n.L[l - 1]);
}

aq_status launch_layer_rows(const FwdArgs& a, int l, const LayerIO& io, hipStream_t st) {
    const LayerDev& L = a.net.L[l];
    const bool ln = L.act == AQ_ACT_LN_TANH, f32 = l == 0, taps = any_taps(a), as = a.net.asym != 0;
    const RowsLayer q{a.d_net, L.wp, L.bias_fold, L.rshift, L.z_w, io.in, ln ? (void*)io.ln_x : (void*)io.out, a.c.batch,
                      L.K, L.N, L.KS, L.NT, l, (L.act == AQ_ACT_RELU ? RL_RELU : 0) | (ln ? RL_LN : 0)};
    if (f32) {
        if (as) return taps ? go<true, true, true>(q, a.t, st) : go<true, true, false>(q, a.t, st);
        return taps ? go<true, false, true>(q, a.t, st) : go<true, false, false>(q, a.t, st);
    }
    if (as) return taps ? go<false, true, true>(q, a.t, st) : go<false, true, false>(q, a.t, st);
    return taps ? go<false, false, true>(q, a.t, st) : go<false, false, false>(q, a.t, st);
}

}  // namespace aq

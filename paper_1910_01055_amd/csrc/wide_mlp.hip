// Whole-network int8 MLP for wide layers at large batch (Sec. 3.1 actor inference on the 8-bit policy of
// Sec. 3.2), software-pipelined: one workgroup of 8 wavefronts owns 64 batch rows from the observation to
// the action, as in the general fused kernel, but a wavefront never sits in a phase that uses only one of
// the CU's pipes.
//
// A layer's output features are split into passes of 512 (8 wavefronts x 2 feature tiles x 32); a wavefront
// keeps two sets of accumulators, the pass being multiplied and the pass before it.  While the matrix cores
// run the MFMAs of pass i, the vector ALU requantizes the accumulators of pass i - 1, two register quads a
// k-step, written between the MFMAs of that k-step.  Across a layer boundary this still works: the first
// k-steps of layer l + 1 read the features that layer l's earlier passes wrote, so the epilogue of layer l's
// last pass runs under them; one workgroup barrier in the middle of that pass then publishes the remaining
// features, and the k-steps that read them follow it.  Weights stream L2 -> registers in operand order, two
// k-steps of 64 in flight per wavefront, and the stream does not stop at a pass boundary: the last k-steps of a
// pass already request the first k-steps of the next one.
//
// v_mfma_i32_16x16x64_i8 on the 32 x 32 operand tiles, as in the general kernel: a weight stream beside it keeps the matrix pipe waiting
// less than beside 32x32x32 (the loop alone: busy 80 % of the cycles instead of 72; this kernel 102.6 k cycles -> 97.0 k at the same
// clock, 256-1024x3-64 at 16384 rows 46.5 -> 43.7 us).  Four quads of the epilogue in a k-step
// instead of two, so that layers of K = 256 hide theirs too, spilled 41 registers and took 47.
//
// Shapes: per-channel symmetric weights, fp32 observations at a 16-byte aligned address, every hidden layer
// ReLU / none (no LayerNorm) with a width that is a multiple of 64, every layer's K a multiple of 128, a
// last layer of at most 64 outputs.  Everything else takes the general fused kernel.
#include <atomic>

#include "explore_device.hpp"
#include "int8_device.hpp"
#include "lanes.hpp"

namespace aq {
namespace {

constexpr int FW = 8;            // wavefronts per workgroup
constexpr int FT = FW * 64;      // threads per workgroup
constexpr int CST_MAXN = 1024;   // widest layer


// The narrow last layer, read through the kernel's pointer argument with uniform indices, i.e. by scalar loads into scalar
// registers.  Its constants: bias, then scale, [Np] each.
struct LastLayer {
    const int8_t* wp;
    gv4i_ptr pack;
    int N, NT, KS, pieces;  // pieces of 16 bytes of the constants: one a thread at most
};
__device__ __forceinline__ LastLayer last_layer(const LayerDev& s) {
    const int NT = uni(s.NT);
    return LastLayer{uni_ptr(s.wp), (gv4i_ptr)uni_ptr(s.bias_fold), uni(s.N), NT, uni(s.KS), 2 * NT * 8};
}

// A last layer of at most two feature tiles would leave most waves idle.  It is spread over all
// eight instead: its (feature tile, row tile) pairs go to different waves, and the waves left over
// split K.  Partial accumulators meet in LDS (PART_WORDS ints per wave: 16 accumulator registers, lane-major).
constexpr int NARROW_NT = 2;
constexpr int PART_WORDS = 16 * 64;
constexpr int PART_BYTES = FW * PART_WORDS * 4;
struct NarrowMap {
    int pairs, ksplit, pair, nt, mt, k0, k1;
};
template <int MT>
__device__ __forceinline__ NarrowMap narrow_map(int NT, int KS, int wave) {
    NarrowMap x;
    x.pairs = NT * MT;                        // 1, 2, 4 or 8
    const int lg = 31 - __builtin_clz(x.pairs);
    x.ksplit = FW >> lg;
    x.pair = wave & (x.pairs - 1);
    const int kpart = wave >> lg;
    x.nt = x.pair & (NT - 1);
    x.mt = x.pair >> (NT - 1);                // NT is 1 or 2
    const int kchunk = (KS + x.ksplit - 1) >> (3 - lg);
    x.k0 = kpart * kchunk;
    x.k1 = x.k0 + kchunk < KS ? x.k0 + kchunk : KS;
    return x;
}

// Sums the K-split partial accumulators of a narrow last layer and dequantizes: every thread owns
// 2 * NT * MT outputs (lane-major, so its LDS reads are conflict-free) and reads the KSPLIT partial
// sums of each; all reads of one output are independent and issued together.
template <int MT, int NT, bool TAPS>
__device__ __forceinline__ void narrow_reduce(const int32_t* part, const int32_t* cst, const LayerTaps& T, int N,
                                              int64_t row0, int64_t batch, float* yrow, int ldy, int tid, int head,
                                              float* actions, float* tap_y, const CallArgs& c) {
    constexpr int PAIRS = NT * MT, KSPLIT = FW / PAIRS;
#pragma unroll
    for (int it = 0; it < 2 * PAIRS; ++it) {
        const int e = tid + it * FT, pr = it >> 1;  // FT = 512 outputs per step, 1024 per pair
        const int reg = (e >> 6) & 15, ln = tid & 63;
        int v = 0;
#pragma unroll
        for (int kp = 0; kp < KSPLIT; ++kp) {
            const int32_t* src = part + (kp * PAIRS + pr) * PART_WORDS + ln;
            v += src[reg * 64];
        }
        const int nt = pr & (NT - 1), mt = pr / NT;
        const int n = nt * 32 + 8 * (reg >> 2) + 4 * (ln >> 5) + (reg & 3);
        const int m = mt * 32 + (ln & 31);
        v += cst[n];
        const int64_t row = row0 + m;
        const bool ok = row < batch && n < N;
        if (TAPS) {
            if (T.acc && ok) T.acc[row * N + n] = v;
        }
        const float y = (float)v * __int_as_float(cst[NT * 32 + n]);
        if (actions) {
            // elementwise heads leave from here; only argmax needs the whole row in one place
            if (ok) {
                if (TAPS) {
                    if (tap_y) tap_y[row * N + n] = y;
                }
                float act = head == AQ_HEAD_TANH ? tanh_head(y) : y;
                if (c.ex_sigma)  // exploration noise of Sec. 4.1, sigma per actor (= per batch row)
                    act = act + c.ex_sigma[row] * gaussian_draw((uint32_t)row, n, c.ex_k0, c.ex_k1, c.ex_s0, c.ex_s1);
                actions[row * N + n] = act;
            }
        } else {
            yrow[m * ldy + n] = y;
        }
    }
}


constexpr int WROWS = 64;    // batch rows per workgroup: two row tiles per wavefront
constexpr int WPF = 2;       // weight k-steps (of 64) in flight per wavefront
constexpr int WSLOT = 256;   // words of one wave-private constant slot: four arrays of 64 features
constexpr int WGROUP = 8;    // k-steps of a pass that carry the epilogue of the pass before (two quads each)

typedef const char AQ_GLOBAL* gbytes;

__host__ __device__ inline size_t wide_lds_bytes(int ld) {
    return (size_t)2 * WROWS * ld + (size_t)FW * 2 * WSLOT * 4 + 256 * 4;
}

template <bool TAPS>
__global__ __launch_bounds__(FT) void k_mlp_wide(const NetDev* __restrict__ netp, const CallArgs c, const TapParam<TAPS> tp) {
    const TapArgs t = taps_of(tp);
    extern __shared__ __align__(16) int8_t smem[];
    const NetDev& a = *netp;
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int b16 = lane & 15, g = lane >> 4;  // this lane's batch row and k-group (operands) / feature quad (results)
    const int64_t row0 = (int64_t)blockIdx.x * WROWS;
    const int ld = c.ld;
    int32_t* const cst_all = (int32_t*)(smem + 2 * WROWS * ld);
    int32_t* const my_cst = cst_all + wave * 2 * WSLOT;   // two slots: this pass's constants, the previous pass's
    int32_t* const cst_last = cst_all + FW * 2 * WSLOT;   // the narrow last layer's bias | scale
    auto buf = [&](int i) { return smem + (i & 1) * WROWS * ld; };
    const int n_layers = uni(a.n_layers), nh = n_layers - 1;

    // the weight stream of one pass of this wavefront: its two feature tiles, KS k-steps of 2 KiB each
    struct Stream {
        gbytes b0, b1;
        int KS;
    };
    const uint32_t lane_off = (uint32_t)((g >> 1) * 1024 + (b16 + 32 * (g & 1)) * 16);
    // half h of the stream's tiles at k-step ks
    auto wload = [&](gbytes t0, gbytes t1, int h, int ks) {
        return *(gv4i_ptr)((h >> 1 ? t1 : t0) + (int64_t)ks * 2048 + (lane_off + 256 * (h & 1)));
    };

    // first pass's first weights: requested before the observations are touched
    v4i wreg[WPF][4];
    {
        const int KS0 = c.KS0;
        gbytes wp = (gbytes)c.wp0;
        const int grp0 = 2 * wave < c.NT0 ? wave : 0;
#pragma unroll
        for (int p = 0; p < WPF; ++p)
#pragma unroll
            for (int h = 0; h < 4; ++h)
                wreg[p][h] = wload(wp + (int64_t)(2 * grp0) * KS0 * 1024, wp + (int64_t)(2 * grp0 + 1) * KS0 * 1024, h, p);
    }

    // observation quantize: a0 = clamp(round(x / s0) + z0, 0, 255), kept in the signed domain.  The block's
    // rows are one contiguous 16-byte aligned run (the launcher checked the address; K0 is a multiple of 128):
    // 16-byte pieces, four in flight per lane, four codes at a time into their row of the LDS buffer.
    {
        const int K0 = c.K0;
        const float s0 = a.actq[0].s;
        const int z0 = a.actq[0].z;
        const QuantScale qs0 = make_quant_scale(s0);
        const float zf0 = (float)z0;
        int8_t* buf_in = buf(0);
        const int64_t left = c.batch - row0;
        const int vrows = left < WROWS ? (int)left : WROWS;
        const int n4 = (vrows * K0) >> 2, k4 = K0 >> 2;
        // idx / k4 by a reciprocal: (idx + 0.5) / k4 stays at least 0.5 / k4 away from every integer, far more
        // than the rounding error at these magnitudes (idx < 2^16)
        const float inv_k4 = __builtin_amdgcn_rcpf((float)k4);
        const float4* src = (const float4*)((const float*)c.obs + row0 * K0);
        for (int i0 = tid; i0 < n4; i0 += 4 * FT) {
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + u * FT < n4) v[u] = src[i0 + u * FT];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int idx = i0 + u * FT;
                if (idx < n4) {
                    uint32_t pack = quant_u8x4(v[u], qs0, zf0);
                    if (TAPS) {
                        if (t.a0) *(uint32_t*)(t.a0 + row0 * K0 + 4 * idx) = pack;
                    }
                    const int m = (int)(((float)idx + 0.5f) * inv_k4), kq = idx - m * k4;
                    *(uint32_t*)(buf_in + m * ld + 4 * kq) = pack ^ 0x80808080u;
                }
            }
        }
        // rows past the batch: zero in the signed domain
        for (int m = vrows + wave; m < WROWS; m += FW)
            for (int k = lane * 4; k < K0; k += 256) *(uint32_t*)(buf_in + m * ld + k) = 0u;
    }
    lds_barrier();

    v4i cur[4][4], prev[4][4];  // [16-feature half][16-row tile]
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) cur[h][r] = prev[h][r] = v4i{0, 0, 0, 0};

    // what the epilogue of the previous pass needs (all uniform)
    bool have_prev = false, prev_active = false;
    int prev_grp = 0, prev_N = 0, prev_zout = 0, prev_lo = 0, prev_fast = 0, prev_slot = 0;
    const int32_t* prev_rshift = nullptr;
    int8_t* prev_out = nullptr;
    int32_t* prev_tacc = nullptr;  // intermediate outputs asked for by a test (TAPS only)
    uint8_t* prev_tact = nullptr;

    // ---- epilogue of the previous pass, in pieces: quad Q = (half h, row tile r), piece i = output i of the quad.
    // Constants of a half are read from the wave's LDS slot one half ahead of their use.
    QuadConsts qc{}, qn{};
    uint32_t pack = 0;
    auto quad_consts = [&](int h) {
        const int32_t* s = my_cst + prev_slot * WSLOT + 16 * h + 4 * g;
        QuadConsts q;
        q.bf = *(const int4*)(s);
        q.M = *(const int4*)(s + 64);
        q.Z = *(const int4*)(s + 128);
        q.S = *(const int4*)(s + 192);
        return q;
    };
    int lo_v = 0;
    auto epi_piece = [&](auto q_c, auto i_c, auto fast_c) __attribute__((always_inline)) {
        constexpr int Q = decltype(q_c)::value, i = decltype(i_c)::value;
        constexpr bool FAST = decltype(fast_c)::value;
        constexpr int h = Q >> 2, r = Q & 3;
        if (i == 0 && r == 0) {
            qc = qn;
            if (h + 1 < 4) qn = quad_consts(h + 1);
        }
        const int bfv = i == 0 ? qc.bf.x : i == 1 ? qc.bf.y : i == 2 ? qc.bf.z : qc.bf.w;
        const int Mv = i == 0 ? qc.M.x : i == 1 ? qc.M.y : i == 2 ? qc.M.z : qc.M.w;
        const int Zv = i == 0 ? qc.Z.x : i == 1 ? qc.Z.y : i == 2 ? qc.Z.z : qc.Z.w;
        const int Sv = i == 0 ? qc.S.x : i == 1 ? qc.S.y : i == 2 ? qc.S.z : qc.S.w;
        const int val = prev[h][r][i] + bfv;
        const int n = 64 * prev_grp + 16 * h + 4 * g + i;
        int code;
        if (FAST) code = clamp_code((__mulhi(val, Mv) + Zv) >> Sv, lo_v, 255);
        else code = requant_code(val, Mv, prev_rshift[n], prev_zout, prev_lo);
        if (TAPS) {
            const int64_t row = row0 + r * 16 + b16;
            if (row < c.batch) {
                if (prev_tacc) prev_tacc[row * prev_N + n] = val;
                if (prev_tact) prev_tact[row * prev_N + n] = (uint8_t)code;
            }
        }
        pack = i == 0 ? (uint32_t)code : pack | ((uint32_t)code << (8 * i));
        if (i == 3) *(uint32_t*)(prev_out + (r * 16 + b16) * ld + n - 3) = pack ^ 0x80808080u;
    };
    auto epi_begin = [&]() __attribute__((always_inline)) {
        qn = quad_consts(0);
        lo_v = prev_lo;
        asm volatile("" : "+v"(lo_v));
    };
    // the whole epilogue of the previous pass with nothing under it
    auto epi_standalone = [&](auto fast_c) __attribute__((always_inline)) {
        epi_begin();
        static_for<0, 16>([&](auto q_c) __attribute__((always_inline)) {
            static_for<0, 4>([&](auto i_c) __attribute__((always_inline)) { epi_piece(q_c, i_c, fast_c); });
        });
    };

    // ---- one k-step (of 64) of this wavefront's 4 x 4 tiles of 16 x 16; Q >= 0: with quads Q and Q + 1 of the previous
    // pass's epilogue between its MFMAs.  A row tile's operand of the next k-step is read as soon as this one's MFMAs with it
    // are issued; then the weight slot's refill: k-step k + WPF of this pass, or, past its end, of the next pass (clamped to an
    // address that exists when there is nothing left to request; those registers are then never used).
    Stream sc{nullptr, nullptr, 1}, sn{nullptr, nullptr, 1};
    const int8_t* xrow = nullptr;
    v4i xf[4];
    auto kstep = [&](int k, auto p_c, auto q_c) __attribute__((always_inline)) {
        constexpr int p = decltype(p_c)::value, Q = decltype(q_c)::value;
        const int8_t* const nx = xrow + (k + 1 < sc.KS ? k + 1 : sc.KS - 1) * 64;
        static_for<0, 4>([&](auto r_c) __attribute__((always_inline)) {
            constexpr int r = decltype(r_c)::value;
            static_for<0, 4>([&](auto h_c) __attribute__((always_inline)) {
                constexpr int h = decltype(h_c)::value;
                cur[h][r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wreg[p][h], xf[r], cur[h][r], 0, 0, 0);
                if constexpr (Q >= 0 && (h & 1) == 1)  // eight pieces a k-step
                    epi_piece(std::integral_constant<int, Q + r / 2>{}, std::integral_constant<int, 2 * (r & 1) + h / 2>{}, std::true_type{});
            });
            xf[r] = *(const v4i*)(nx + r * 16 * ld);
        });
        const int idx = k + WPF;
        const bool in = idx < sc.KS;
        const int past = idx - sc.KS < sn.KS ? idx - sc.KS : sn.KS - 1;
        const int ks = in ? idx : past;
#pragma unroll
        for (int h = 0; h < 4; ++h) wreg[p][h] = wload(in ? sc.b0 : sn.b0, in ? sc.b1 : sn.b1, h, ks);
        __builtin_amdgcn_sched_barrier(0);
    };
    using NoQ = std::integral_constant<int, -1>;
    auto group = [&](int k) __attribute__((always_inline)) {
        static_for<0, WPF>([&](auto p_c) __attribute__((always_inline)) { kstep(k + decltype(p_c)::value, p_c, NoQ{}); });
    };
    // the activation operands of k-step k
    auto start_ring = [&](int k) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) xf[r] = *(const v4i*)(xrow + r * 16 * ld + k * 64);
    };
    // Everything uniform a pass needs.  It is read from the network description one pass ahead of its use, so
    // that the scalar loads' round trips run under the previous pass's k-steps.
    struct Pass {
        bool valid, active;
        int l, p, grp, npass, N, Np, KS, act, z_out, fast;
        gbytes b0, b1;
        gv4i_ptr pack;
        const int32_t* rshift;
    };
    auto pass_of = [&](int l, int p) {
        Pass q{};
        q.valid = l < nh;
        q.l = l;
        q.p = p;
        if (q.valid) {
            const LayerDev& L = a.L[l];
            const int NT = uni(L.NT), ngroups = NT >> 1;
            q.npass = (ngroups + FW - 1) / FW;
            q.grp = p * FW + wave;
            q.active = q.grp < ngroups;
            q.N = uni(L.N);
            q.Np = NT * 32;
            q.KS = uni(L.KS) >> 1;
            q.act = uni(L.act);
            q.z_out = uni(a.actq[l + 1].z);
            q.fast = uni(a.fast[l]);
            gbytes wp = (gbytes)uni_ptr(L.wp);
            const int grp = q.active ? q.grp : 0;
            q.b0 = wp + (int64_t)(2 * grp) * q.KS * 2048;
            q.b1 = wp + (int64_t)(2 * grp + 1) * q.KS * 2048;
            q.pack = (gv4i_ptr)uni_ptr(L.bias_fold);
            q.rshift = uni_ptr(L.rshift);
        }
        return q;
    };
    int npass_prev_layer = 0;
    int pass_no = 0;
    bool w_ready = 2 * wave < c.NT0;  // this wavefront's next pass finds its first weights requested already
    Pass P = pass_of(0, 0);
    while (P.valid) {
        const bool more = P.p + 1 < P.npass;
        const Pass Nx = pass_of(more ? P.l : P.l + 1, more ? P.p + 1 : 0);
        const int l = P.l;
        const bool active = P.active;
        sc = Stream{P.b0, P.b1, P.KS};
        // the pass after this one, for the weight stream (nothing to request: this pass's last tile again)
        if (Nx.valid && Nx.active) sn = Stream{Nx.b0, Nx.b1, Nx.KS};
        else sn = Stream{sc.b0 + (int64_t)(sc.KS - 1) * 2048, sc.b1 + (int64_t)(sc.KS - 1) * 2048, 1};
        // this pass's per-channel constants: one 16-byte piece per lane (four arrays x 64 features), parked in
        // the wave's slot at the end of the pass
        v4i cw = {0, 0, 0, 0};
        const int cw_word = (lane >> 4) * P.Np + 64 * P.grp + 4 * (lane & 15);
        if (active) cw = P.pack[cw_word >> 2];
        xrow = buf(l) + b16 * ld + g * 16;
        if (active && !w_ready) {  // (the pass before this one was not this wavefront's, or requested nothing)
#pragma unroll
            for (int q = 0; q < WPF; ++q)
#pragma unroll
                for (int h = 0; h < 4; ++h) wreg[q][h] = wload(sc.b0, sc.b1, h, q);
        }
        // k-steps that may run before the previous pass's outputs are visible to every wavefront: all of them
        // within a layer; in a layer's first pass those that read what the previous layer's earlier passes wrote
        const int n_over = P.p > 0 ? sc.KS : WGROUP * (npass_prev_layer - 1);
        int k0 = 0;
        if (have_prev) {
            if (prev_active) {
                if (active && prev_fast && n_over >= WGROUP && sc.KS >= WGROUP) {
                    start_ring(0);
                    epi_begin();
                    static_for<0, WGROUP>([&](auto q_c) __attribute__((always_inline)) {
                        constexpr int q = decltype(q_c)::value;
                        kstep(q, std::integral_constant<int, q % WPF>{}, std::integral_constant<int, 2 * q>{});
                    });
                    k0 = WGROUP;
                } else if (prev_fast) {
                    epi_standalone(std::true_type{});
                } else {
                    epi_standalone(std::false_type{});
                }
            }
            // the previous pass's features are in LDS for every wavefront (the k-steps below, or a later pass of
            // any wavefront, read them)
            lds_barrier();
        }
        if (active) {
            if (k0 < sc.KS) start_ring(k0);  // (after the barrier: operands are read a k-step ahead)
            for (int k = k0; k < sc.KS; k += WPF) group(k);
            // park the constants: [bias_fold | M0 | rz | sh] x 64 features
            *(v4i*)(my_cst + (pass_no & 1) * WSLOT + (lane >> 4) * 64 + 4 * (lane & 15)) = cw;
        }
        w_ready = active && sn.KS > 1;  // (KS is at least 2: a one-step stream is the placeholder)
        // hand the accumulators to the next pass's epilogue
        have_prev = true;
        prev_active = active;
        prev_grp = P.grp;
        prev_N = P.N;
        prev_zout = P.z_out;
        prev_lo = P.act == AQ_ACT_RELU ? P.z_out : 0;
        prev_fast = P.fast;
        prev_slot = pass_no & 1;
        prev_rshift = P.rshift;
        prev_out = buf(l + 1);
        if (TAPS) {
            prev_tacc = t.acc[l];
            prev_tact = t.act[l];
        }
#pragma unroll
        for (int h = 0; h < 4; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                prev[h][r] = cur[h][r];
                cur[h][r] = v4i{0, 0, 0, 0};
            }
        if (!more) npass_prev_layer = P.npass;
        P = Nx;
        ++pass_no;
    }
    // The narrow last layer's constants and this wavefront's first weights of it do not depend on the hidden
    // layers: requested before the last epilogue.
    const LastLayer LL = last_layer(a.L[nh]);
    const NarrowMap nm = narrow_map<2>(LL.NT, LL.KS, wave);
    v4i cv = {0, 0, 0, 0};
    if (tid < LL.pieces) cv = LL.pack[tid];
    gv4i_ptr nwptr[1];
    nwptr[0] = (gv4i_ptr)LL.wp + (int64_t)nm.nt * LL.KS * 64 + lane;
    v4i nw[4][1];
    if (nm.k0 < nm.k1) mma_prefetch<1, 4>(nwptr, nm.k0, nm.k1, nw);
    // the last hidden pass has nothing to hide under
    if (have_prev && prev_active) {
        if (prev_fast) epi_standalone(std::true_type{});
        else epi_standalone(std::false_type{});
    }

    // ---- narrow last layer (at most two feature tiles): spread over all eight wavefronts by splitting K
    {
        const int l = nh;
        const LastLayer& L = LL;
        LayerTaps T{nullptr, nullptr, nullptr};
        if (TAPS) T = LayerTaps{t.acc[l], t.act[l], t.ln[l]};
        const int Np = L.NT * 32;
        lds_barrier();  // every hidden feature is in LDS
        const int8_t* in = buf(l);
        v16i pacc[1][1], prs[1];
        pacc[0][0] = zero16();
        prs[0] = zero16();
        if (nm.k0 < nm.k1)
            mma_run<1, 1, false, 4>(nwptr, nw, in + nm.mt * 32 * ld, ld, nm.k0, nm.k1, 0, pacc, prs, lane);
        int32_t* part = (int32_t*)buf(l + 1);  // the idle activation buffer (64 * ld >= PART_BYTES, checked by the launcher)
        {
            int32_t* mine = part + wave * PART_WORDS + lane;
#pragma unroll
            for (int r = 0; r < 16; ++r) mine[r * 64] = pacc[0][0][r];
        }
        if (tid < L.pieces) ((v4i*)cst_last)[tid] = cv;
        lds_barrier();  // partial sums and the layer's constants are in LDS; the layer's input is free
        float* yrow = (float*)buf(l);
        const int ldy = Np + 1;
        const int head = uni(a.head);
        float* direct = head != AQ_HEAD_ARGMAX ? (float*)c.actions : nullptr;
        float* tap_y = TAPS ? t.y : nullptr;
        if (L.NT == 1)
            narrow_reduce<2, 1, TAPS>(part, cst_last, T, L.N, row0, c.batch, yrow, ldy, tid, head, direct, tap_y, c);
        else
            narrow_reduce<2, 2, TAPS>(part, cst_last, T, L.N, row0, c.batch, yrow, ldy, tid, head, direct, tap_y, c);
        if (direct) return;
        lds_barrier();
        // argmax over the dequantized rows (lowest index wins ties)
        for (int m = tid; m < WROWS; m += FT) {
            const int64_t row = row0 + m;
            if (row >= c.batch) continue;
            int best = 0;
            for (int n = 0; n < L.N; ++n) {
                const float y = yrow[m * ldy + n];
                if (TAPS) {
                    if (t.y) t.y[row * L.N + n] = y;
                }
                if (y > yrow[m * ldy + best]) best = n;
            }
            ((int32_t*)c.actions)[row] = best;
        }
    }
}

template <bool TAPS>
aq_status launch_wide_t(const FwdArgs& a, size_t lds, hipStream_t st) {
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
        if (hip_failed(hipFuncSetAttribute((const void*)k_mlp_wide<TAPS>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)))
            return AQ_EHIP;
        attr_set = true;
    }
    const unsigned grid = (unsigned)((a.c.batch + WROWS - 1) / WROWS);
    hipLaunchKernelGGL((k_mlp_wide<TAPS>), dim3(grid), dim3(FT), lds, st, a.d_net, a.c, TapParam<TAPS>(a.t));
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

}  // namespace

// Shapes the pipelined kernel takes (see the head of this file); `ld_out`: its LDS row stride.
bool wide_mlp_supported(const FwdArgs& a, int* ld_out) {
    const NetDev& n = a.net;
    if (n.asym || n.in_u8 || n.n_layers < 2) return false;
    int maxw = 0;
    for (int l = 0; l < n.n_layers; ++l) {
        const LayerDev& L = n.L[l];
        if (L.kh != 1 || L.kw != 1 || L.in_h != 1 || L.in_w != 1) return false;
        if (L.K % 128 != 0) return false;
        if (l < n.n_layers - 1) {
            if (L.N % 64 != 0 || L.N > CST_MAXN || L.act == AQ_ACT_LN_TANH) return false;
        } else if (L.NT > NARROW_NT) {
            return false;
        }
        maxw = maxw > L.K ? maxw : L.K;
    }
    const int ld = maxw + 16;
    // the narrow last layer parks its K-split partial sums in the idle activation buffer and its fp32 rows
    // (stride 32 * NT + 1 floats) in the other one
    if ((size_t)WROWS * ld < (size_t)PART_BYTES) return false;
    if ((size_t)ld < (size_t)(NARROW_NT * 32 + 1) * 4) return false;
    if (wide_lds_bytes(ld) > 160 * 1024) return false;
    *ld_out = ld;
    return true;
}

aq_status launch_wide_mlp(const FwdArgs& a_in, hipStream_t st) {
    int ld = 0;
    if (!wide_mlp_supported(a_in, &ld)) return AQ_ESHAPE;
    if (((uintptr_t)a_in.c.obs & 15) != 0) return AQ_ESHAPE;
    FwdArgs a = a_in;
    a.c.ld = ld;
    a.c.wp0 = a.net.L[0].wp;
    a.c.NT0 = a.net.L[0].NT;
    a.c.KS0 = a.net.L[0].KS;
    const size_t lds = wide_lds_bytes(ld);
    return any_taps(a) ? launch_wide_t<true>(a, lds, st) : launch_wide_t<false>(a, lds, st);
}

}  // namespace aq

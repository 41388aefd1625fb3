// The leading convolution layers of a frame policy (Sec. 4.1: the Atari-style policies take stacked
// 8-bit frames through three convolutions before the fully connected layers) in one launch: a workgroup
// of 16 wavefronts (or two of 8, see launch_conv_stack) keeps a frame, every intermediate feature map, the layers'
// weights and epilogue constants in LDS and goes from image to image (grid = what the CUs hold at once), so that
// weights and constants are fetched once per workgroup and a frame is fetched under the previous image's convolutions.
//
// No im2col: with NHWC maps a 16-byte piece of the implicit GEMM's K is 16 contiguous bytes of one kernel row of
// the input map, so an MFMA's activation operand is one 16-byte LDS read per lane at an address computed from the
// output position.  v_mfma_i32_16x16x64_i8: lane (i = lane % 16, g = lane / 16) of k-step s holds bytes
// 64 s + 16 g .. + 15 of K, for weights a piece of the 32 x 32 operand tiles the library stores.  A wavefront's task is
// 16 output positions x 32 features.
//
// What bounds it: the chain of phases of one workgroup (arguments, frame round trip, three layers of a barrier, a task's
// operand reads and products, an epilogue) and, within a phase, instruction issue: what all sixteen wavefronts execute
// costs sixteen clocks an instruction.  Hence one wavefront per layer for constants and tables, four per layer for the
// weights (straight into LDS), one code for all layers with arguments read per layer, windows' places from a table.  An
// 84 x 84 x 4 frame through 32, 32 and 16 channels at 256 images takes 7.6 us back to back, 2.6 of them the launch.  The
// same with a copy of the code per layer and weights through registers: 13 us.  One workgroup per image with 32 x 32
// tiles and weights from L2 per tile (what stood here before) took none but rows of 16 bytes: a policy on 65 x 65 x 3
// frames at batch 25 went layer by layer with byte gathers, 55.4 us, now 19.3.  Where both run, whole forwards before
// and now: 84 x 84 x 4 through 32, 32, 16 at 256 / 2048 images 16.0 / 46.6 and 14.5 / 40.9 us; through 32, 64, 64, whose
// weights leave one workgroup to a CU, 18.6 / 56.6 and 17.4 / 61.2 us.
//
// Frames of fewer than four channels whose windows would not begin and end at whole pieces are expanded to four on
// their way into LDS, and the first layer's weights with them (zeros in the channels that do not exist), so that every
// frame has aligned pieces; rows in LDS are padded to 16 bytes.
//
// Shapes it takes (the host checks them, anything else goes one launch per layer): 8-bit frames, per-channel
// symmetric weights, two to four convolutions before a fully connected layer; per layer kw * C and stride * C multiples
// of 16 (C = channels, 4 where the frame is expanded), N a multiple of 4; frame, maps and constants within LDS and the
// registers they pass through.  The frame and the second map have LDS of their own, so that the next frame is stored
// while the last layer is still at work; where that is too much they share it, for one barrier more per image.
#include "int8_device.hpp"

namespace aq {

namespace {
constexpr int CS_W = 16;         // wavefronts per workgroup, or half of them with two workgroups on a CU
constexpr int cs_pieces(int W) { return W == CS_W ? 3 : 4; }  // 16-byte pieces of the frame (in LDS) per thread
constexpr size_t CS_MAX_LDS = 160 * 1024;
constexpr int CS_MAXC = 4;       // convolution layers of a stack at most

// What the host knows of the stack at launch time, by value: no layer begins with a round trip for its own entry of
// the device-resident description.  Only what the quantizer kernels write (activation zero-points, short-form flags)
// comes from there, requested at the start.
struct StackLayer {
    const int8_t* wp;
    const int32_t* pack;  // epilogue constants: bias_fold | M0 | rz | sh, each NT * 32 words
    const int32_t* rsh;   // shifts of the general form (read where they are used)
    int per_nt, per_inv;  // wavefronts per tile of 32 features; 65536 / that, rounded up
    int NT, RT, R, ow;    // tiles of 32 features, tiles of 16 positions, output positions, positions per row
    float inv_ow;
    int pos_x, pos_y;     // bytes from an output position's window to the next one's, in LDS
    int K, N, KS, act;
    int in_off, out_off, out_row;  // LDS: input map, output map and its row stride
    int w_off, w_tiles;   // LDS: weights, and how many 1 KiB tiles of them
    int c_off;            // LDS: constants
    int k_off, k_len;     // LDS: where each 16-byte piece of K lies relative to a window's first byte; entries per g
    int run, row;         // bytes of a window row, of an input map row in LDS
};
struct StackArgs {
    int pieces, pieces_row;  // 16-byte pieces of the frame in LDS, and of one of its rows
    float inv_row;
    int src_piece, src_row;  // bytes of a piece and of a row in the frame as given
    int last;                // where its last 16 bytes begin
    int64_t frame_bytes;
    int ragged;              // a piece reaches past the image's end
    int expand;              // first layer: channels below four, their number; else 0
    int KS0;                 // first layer's k-steps as stored
    int share;               // the second map lies where the frame does
    int batch, nc;
    StackLayer L[CS_MAXC];
};

struct StackPlan {
    int nc;         // leading convolution layers taken
    bool resident;  // weights in LDS
    size_t lds;
};

// For workgroups of W wavefronts, CS_W / W of them on a CU.  `sa` may be NULL: only whether and how many
bool plan_stack(const FwdArgs& a, int W, StackPlan* p, StackArgs* sa) {
    const size_t max_lds = CS_MAX_LDS / (CS_W / W);
    const NetDev& net = a.net;
    if (!net.in_u8 || net.asym) return false;
    int nc = 0;
    while (nc < net.n_layers) {
        const LayerDev& L = net.L[nc];
        const bool fc = L.kh == 1 && L.kw == 1 && L.in_h == 1 && L.in_w == 1;
        if (fc) break;
        ++nc;
    }
    if (nc < 2 || nc > CS_MAXC || nc >= net.n_layers) return false;  // a fully connected layer must follow
    if (a.c.batch > 0x7fffffffLL) return false;
    StackArgs s{};
    const LayerDev& L0 = net.L[0];
    s.expand = L0.in_c < 4 && ((L0.kw * L0.in_c) % 16 || (L0.stride * L0.in_c) % 16) ? L0.in_c : 0;
    const int c0 = s.expand ? 4 : L0.in_c;
    s.pieces_row = (L0.in_w * c0 + 15) / 16;
    s.pieces = L0.in_h * s.pieces_row;
    s.inv_row = 1.0f / (float)s.pieces_row;
    s.src_piece = s.expand ? 4 * L0.in_c : 16;
    s.src_row = L0.in_w * L0.in_c;
    s.frame_bytes = (int64_t)L0.in_h * s.src_row;
    s.KS0 = L0.KS;
    s.ragged = s.pieces_row * s.src_piece > s.src_row || s.src_piece < 16;
    s.last = (int)s.frame_bytes - 16;
    s.batch = (int)a.c.batch;
    s.nc = nc;
    if (s.pieces > cs_pieces(W) * W * 64 || s.frame_bytes < 16) return false;
    size_t map[2] = {0, 0};
    for (int l = 0; l < nc; ++l) {
        const LayerDev& L = net.L[l];
        StackLayer& q = s.L[l];
        const int C = l == 0 ? c0 : L.in_c;
        if (L.act == AQ_ACT_LN_TANH || a.t.ln[l]) return false;
        if ((L.kw * C) % 16 || (L.stride * C) % 16 || (L.N & 3)) return false;
        q.wp = L.wp;
        q.pack = L.bias_fold;
        q.rsh = L.rshift;
        q.R = L.oh * L.ow;
        q.ow = L.ow;
        q.inv_ow = 1.0f / (float)L.ow;
        q.RT = (q.R + 15) / 16;
        q.per_nt = L.NT < W ? W / L.NT : 1;
        q.per_inv = (65536 + q.per_nt - 1) / q.per_nt;
        q.run = L.kw * C;
        q.row = l == 0 ? s.pieces_row * 16 : s.L[l - 1].out_row;
        q.pos_x = L.stride * C;
        q.pos_y = L.stride * q.row;
        q.K = L.kh * L.kw * C;
        q.N = L.N;
        q.NT = L.NT;
        q.KS = (q.K + 31) / 32;
        q.act = L.act;
        q.out_row = round_up(L.ow * L.N, 16);
        const size_t out = (size_t)L.oh * q.out_row;
        if (l < nc - 1 && out > map[l & 1]) map[l & 1] = out;
    }
    // LDS: frame, the two map areas, constants, tables of K
    const size_t frame = (size_t)s.pieces * 16;
    size_t rest = 0;
    for (int l = 0; l < nc; ++l) rest += (size_t)s.L[l].NT * 512 + (size_t)round_up((s.L[l].K + 63) / 64, 4) * 16;
    s.share = frame + map[0] + map[1] + rest > max_lds;
    const size_t first = s.share && map[1] > frame ? map[1] : frame;
    const size_t off_map[2] = {first, s.share ? 0 : first + map[0]};
    size_t at = first + map[0] + (s.share ? 0 : map[1]);
    for (int l = 0; l < nc; ++l) {
        StackLayer& q = s.L[l];
        q.in_off = l == 0 ? 0 : (int)off_map[(l - 1) & 1];
        q.out_off = (int)off_map[l & 1];
        q.c_off = (int)at;
        at += (size_t)q.NT * 512;
        q.k_off = (int)at;
        q.k_len = round_up((q.K + 63) / 64, 4);
        at += (size_t)q.k_len * 16;
    }
    // the weights, if all of them fit; an expanded first layer's have to
    size_t w_at = at;
    for (int l = 0; l < nc; ++l) {
        StackLayer& q = s.L[l];
        q.w_off = (int)w_at;
        q.w_tiles = q.NT * q.KS;
        w_at += (size_t)q.w_tiles * 1024;
    }
    p->nc = nc;
    p->resident = w_at <= max_lds;
    p->lds = p->resident ? w_at : at;
    if (p->lds > max_lds || (s.expand && !p->resident)) return false;
    if (sa) *sa = s;
    return true;
}

typedef v4i v4i_any __attribute__((aligned(1)));
#define AQ_CONST __attribute__((address_space(4)))

// 1 KiB of weights straight into LDS (no registers, nothing to wait for until they are used)
__device__ __forceinline__ void lds_fetch_1k(const int8_t* src, int8_t* dst, int lane) {
    __builtin_amdgcn_global_load_lds((const AQ_GLOBAL void*)(src + lane * 16), (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
}  // namespace

// WLDS: weights in LDS (else from L2, operand by operand)
template <bool TAPS, bool WLDS, int W>
__global__ __launch_bounds__(W * 64, 4) void k_conv_stack(const NetDev* __restrict__ netp, const uint8_t* __restrict__ frames,
                                                     int8_t* __restrict__ out, const StackArgs sa_, const TapParam<TAPS> tp) {
    extern __shared__ __align__(16) int8_t smem[];
    constexpr int T = W * 64, FU = cs_pieces(W);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, i16 = lane & 15;
    const StackArgs AQ_CONST* const sa = (const StackArgs AQ_CONST*)((const char AQ_CONST*)__builtin_amdgcn_kernarg_segment_ptr() + 24);
    (void)sa_;
    // (every cache line of the arguments is a round trip over the host link when it is first read: all of them at once)
    int warm[(sizeof(StackArgs) + 63) / 64];
#pragma unroll
    for (int i = 0; i < (int)(sizeof(warm) / 4); ++i) warm[i] = ((const int AQ_CONST*)sa)[16 * i];
    const int pieces = sa->pieces;

    // ---- frames: pieces of 16 bytes (in LDS).  A piece that would reach past the image's end is read as the image's last
    // 16 bytes and shifted down; past a row's end there is whatever follows, in LDS bytes that no window covers.
    v4i fr[FU];
    auto source = [&](int u, int* back) __attribute__((always_inline)) {
        const int i = tid + u * T, y = (int)(((float)i + 0.5f) * sa->inv_row);
        const int at = __mul24(y, sa->src_row) + __mul24(i - __mul24(y, sa->pieces_row), sa->src_piece);
        *back = at > sa->last ? at - sa->last : 0;
        return at > sa->last ? sa->last : at;
    };
    auto fetch_frame = [&](int64_t img) __attribute__((always_inline)) {
        const uint8_t AQ_GLOBAL* f = (const uint8_t AQ_GLOBAL*)frames + img * sa->frame_bytes;
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            if (u * T >= pieces) continue;  // (scalar)
            int back;
            const uint32_t at = (uint32_t)source(u, &back);
            fr[u] = *(const v4i_any AQ_GLOBAL*)(f + at);
        }
    };
    auto store_frame = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < FU; ++u) {
            if (u * T >= pieces) continue;
            const int i = tid + u * T;
            v4i x = fr[u];
            int back = 0;
            if (sa->ragged) (void)source(u, &back);  // (scalar)
            if (back) {
                uint64_t p0 = (uint32_t)x[0] | (uint64_t)(uint32_t)x[1] << 32, p1 = (uint32_t)x[2] | (uint64_t)(uint32_t)x[3] << 32;
                const int b = (back & 7) * 8;
                if (back & 8) {
                    p0 = p1;
                    p1 = 0;
                }
                if (b) {
                    p0 = p0 >> b | p1 << (64 - b);
                    p1 >>= b;
                }
                x = v4i{(int)p0, (int)(p0 >> 32), (int)p1, (int)(p1 >> 32)};
            }
            if (sa->expand) {  // (scalar) four pixels of one to three bytes
                const uint32_t d0 = x[0], d1 = x[1], d2 = x[2];
                if (sa->expand == 3)
                    x = v4i{(int)(d0 & 0xffffffu), (int)(d0 >> 24 | (d1 & 0xffffu) << 8), (int)(d1 >> 16 | (d2 & 0xffu) << 16), (int)(d2 >> 8)};
                else if (sa->expand == 2)
                    x = v4i{(int)(d0 & 0xffffu), (int)(d0 >> 16), (int)(d1 & 0xffffu), (int)(d1 >> 16)};
                else
                    x = v4i{(int)(d0 & 255u), (int)(d0 >> 8 & 255u), (int)(d0 >> 16 & 255u), (int)(d0 >> 24)};
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] ^= (int)0x80808080;  // into the signed domain (code - 128)
            if (i < pieces) *(v4i*)(smem + 16 * i) = x;
        }
    };

    // ---- the start: the first frame, the weights, the constants and the tables of K.  An instruction that all sixteen
    // wavefronts execute takes 16 clocks of the CU, so that what a single wavefront can do a single one does.
    const int64_t step = gridDim.x;
    int64_t img = blockIdx.x;
    fetch_frame(img);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(warm) / 4); ++i) asm volatile("" ::"s"(warm[i]));
    const int nc = sa->nc;
    if (wave >= W - nc) {  // (scalar) one wavefront per layer
        const StackLayer AQ_CONST& L = sa->L[W - 1 - wave];
        const v4i c0 = ((gv4i_ptr)L.pack)[lane < L.NT * 32 ? lane : 0];
        const float inv_run = 1.0f / (float)L.run;
        for (int i = lane; i < 4 * L.k_len; i += 64) {  // k-step i / 4, piece i % 4
            const int k1 = 16 * i, k = k1 < L.K ? k1 : L.K - 16, ky = (int)(((float)k + 0.5f) * inv_run);
            ((int*)(smem + L.k_off))[(i & 3) * L.k_len + (i >> 2)] = __mul24(ky, L.row) + (k - __mul24(ky, L.run));
        }
        if (lane < L.NT * 32) *(v4i*)(smem + L.c_off + 16 * lane) = c0;
        for (int i = 64 + lane; i < L.NT * 32; i += 64) *(v4i*)(smem + L.c_off + 16 * i) = ((gv4i_ptr)L.pack)[i];
    }
    if (WLDS) {
        constexpr int PER = W / CS_MAXC;
        const int l = wave / PER;  // (scalar) as many wavefronts for each layer
        if (l < nc && !(l == 0 && sa->expand)) {
            const StackLayer AQ_CONST& L = sa->L[l];
            for (int j = wave % PER; j < L.w_tiles; j += PER) lds_fetch_1k(L.wp + j * 1024, smem + L.w_off + j * 1024, lane);
        }
    }
    if (WLDS && sa->expand) {  // the first layer's weights with four channels per tap: a thread makes the four bytes of one
        const StackLayer AQ_CONST& L = sa->L[0];
        const int KS = L.KS, words = L.w_tiles * 256, ch = sa->expand;
        const int8_t AQ_GLOBAL* wp = (const int8_t AQ_GLOBAL*)L.wp;
        for (int i = tid; i < words; i += T) {
            const int tile = i >> 8, ln = (i >> 2) & 63, nt = tile / KS, ks = tile - nt * KS;
            const int tap = (ks * 32 + 16 * (ln >> 5)) / 4 + (i & 3);
            uint32_t w = 0;
            if (4 * tap < L.K)
                for (int c = 0; c < ch; ++c) {
                    const int k = tap * ch + c;
                    const int8_t v = wp[(((int64_t)nt * sa->KS0 + (k >> 5)) * 64 + (ln & 31) + 32 * ((k & 31) >> 4)) * 16 + (k & 15)];
                    w |= (uint32_t)(uint8_t)v << (8 * c);
                }
            *(uint32_t*)(smem + L.w_off + 4 * i) = w;
        }
    }
    store_frame();
    if (WLDS) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (this wavefront's share of the weights is in LDS)

    const int a_lane = (g >> 1) * 1024 + (i16 + 32 * (g & 1)) * 16;  // this lane's piece of a k-step's two weight tiles
    for (;;) {
        const bool more = img + step < sa->batch;
        for (int l = 0; l < nc; ++l) {
            lds_barrier();
            // (read anew each time: kept across the loop, four layers' arguments are more than there are scalar registers)
            const StackLayer AQ_CONST* Lp = &sa->L[l];
            asm volatile("" : "+s"(Lp));
            const StackLayer AQ_CONST& L = *Lp;
            const int N = L.N, np = L.NT * 32, K = L.K, KS = L.KS;
            const int z_out = ((const NetDev AQ_CONST*)netp)->actq[l + 1].z, fast = ((const NetDev AQ_CONST*)netp)->fast[l];
            const int lo = L.act == AQ_ACT_RELU ? z_out : 0;
            int lo_v = lo;
            asm volatile("" : "+v"(lo_v));
            const int32_t* const koff = (const int32_t*)(smem + L.k_off) + g * L.k_len;
            const int w_nt = (wave * L.per_inv) >> 16, w_rt = wave - w_nt * L.per_nt;
            for (int nt = w_nt; nt < L.NT; nt += W) {
                const int8_t* const wl = smem + L.w_off + nt * KS * 1024 + a_lane;
                const int8_t AQ_GLOBAL* const wg = (const int8_t AQ_GLOBAL*)L.wp + nt * KS * 1024 + a_lane;
                auto weights = [&](int off) __attribute__((always_inline)) {
                    return WLDS ? *(const v4i*)(wl + off) : *(const v4i AQ_GLOBAL*)(wg + off);
                };
                const int32_t* const cst = (const int32_t*)(smem + L.c_off) + nt * 32 + 4 * g;
                v4i bias[2];
#pragma unroll
                for (int f = 0; f < 2; ++f) bias[f] = *(const v4i*)(cst + 16 * f);
                for (int rt = w_rt; rt < L.RT; rt += L.per_nt) {
                    const int r = rt * 16 + i16;           // this lane's output position (operand column)
                    const int rc = r < L.R ? r : L.R - 1;  // a ragged last tile re-reads the last position; never stored
                    const int oy = (int)(((float)rc + 0.5f) * L.inv_ow), ox = rc - __mul24(oy, L.ow);
                    const int8_t* const xb = smem + L.in_off + __mul24(oy, L.pos_y) + __mul24(ox, L.pos_x);
                    v4i acc[2] = {bias[0], bias[1]};
                    int s = 0;
                    for (; (s + 4) * 64 <= K; s += 4) {  // (one read for the places of four k-steps)
                        const v4i ko = *(const v4i*)(koff + s);
                        v4i X[4], A[4][2];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            A[j][0] = weights((s + j) * 2048);
                            A[j][1] = weights((s + j) * 2048 + 256);
                        }
#pragma unroll
                        for (int j = 0; j < 4; ++j) X[j] = *(const v4i*)(xb + ko[j]);
                        __builtin_amdgcn_sched_barrier(0);  // (all twelve requests before the first product)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[j][0], X[j], acc[0], 0, 0, 0);
                            acc[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[j][1], X[j], acc[1], 0, 0, 0);
                        }
                    }
                    for (; s * 64 < K; ++s) {
                        // (a k-step that K ends in: zeros from there on, and no weights from past the last tile)
                        const bool ok = 64 * s + 16 * g < K;
                        const int back = 2 * s + (g >> 1) < KS ? 0 : 1024;
                        v4i X = *(const v4i*)(xb + koff[s]);
                        const v4i A0 = weights(s * 2048 - back), A1 = weights(s * 2048 + 256 - back);
#pragma unroll
                        for (int j = 0; j < 4; ++j) X[j] = ok ? X[j] : 0;
                        acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A0, X, acc[0], 0, 0, 0);
                        acc[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A1, X, acc[1], 0, 0, 0);
                    }
                    const int c255 = 255;
                    uint32_t pack[2];
#pragma unroll
                    for (int f = 0; f < 2; ++f) {
                        const v4i val = acc[f], M = *(const v4i*)(cst + np + 16 * f);
                        int code[4];
                        if (fast) {  // (scalar)
                            const v4i Z = *(const v4i*)(cst + 2 * np + 16 * f), S = *(const v4i*)(cst + 3 * np + 16 * f);
#pragma unroll
                            for (int i = 0; i < 4; ++i) code[i] = clamp_code((__mulhi(val[i], M[i]) + Z[i]) >> S[i], lo_v, c255);
                        } else {
                            const v4i S = *(gv4i_ptr)(L.rsh + nt * 32 + 16 * f + 4 * g);
#pragma unroll
                            for (int i = 0; i < 4; ++i) code[i] = requant_code(val[i], M[i], S[i], z_out, lo);
                        }
                        if (TAPS) {
                            const int64_t at = (img * L.R + r) * N + nt * 32 + 16 * f + 4 * g;
                            const TapArgs t = taps_of(tp);
                            int32_t* const t_acc = t.acc[l];
                            uint8_t* const t_act = t.act[l];
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const bool ok = r < L.R && nt * 32 + 16 * f + 4 * g + i < N;
                                if (t_acc && ok) t_acc[at + i] = val[i];
                                if (t_act && ok) t_act[at + i] = (uint8_t)code[i];
                            }
                        }
                        pack[f] = ((uint32_t)code[0] | (uint32_t)code[1] << 8 | (uint32_t)code[2] << 16 | (uint32_t)code[3] << 24) ^ 0x80808080u;
                    }
                    const int n0 = nt * 32 + 4 * g;
                    if (r < L.R) {
                        if (l == nc - 1) {  // (scalar)
                            int8_t AQ_GLOBAL* o = (int8_t AQ_GLOBAL*)out + (img * L.R + r) * N + n0;
                            if (n0 < N) *(uint32_t AQ_GLOBAL*)o = pack[0];
                            if (n0 + 16 < N) *(uint32_t AQ_GLOBAL*)(o + 16) = pack[1];
                        } else {
                            int8_t* o = smem + L.out_off + __mul24(oy, L.out_row) + __mul24(ox, N) + n0;
                            if (n0 < N) *(uint32_t*)o = pack[0];
                            if (n0 + 16 < N) *(uint32_t*)(o + 16) = pack[1];
                        }
                    }
                }
            }
            if (l == 0) {
                if (more) fetch_frame(img + step);
                asm volatile("" ::: "memory");  // (the requests stay in front of the layers)
            }
        }
        if (!more) break;
        if (sa->share) lds_barrier();  // (the last layer may read what lies in the frame's place)
        store_frame();                 // (else the first layer was the frame's only reader)
        img += step;
    }
}

namespace {
template <bool TAPS, bool WLDS, int W>
aq_status launch_stack_t(const FwdArgs& a, const StackPlan& p, const StackArgs& sa, int8_t* out, hipStream_t st) {
    auto* const kernel = k_conv_stack<TAPS, WLDS, W>;
    static std::atomic<bool> attr_set{false};
    if (!attr_set) {
        if (hip_failed(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)CS_MAX_LDS))) return AQ_EHIP;
        attr_set = true;
    }
    const int64_t most = 256 * (CS_W / W);
    const dim3 grid((unsigned)(a.c.batch < most ? a.c.batch : most));
    hipLaunchKernelGGL(kernel, grid, dim3(W * 64), p.lds, st, a.d_net, (const uint8_t*)a.c.obs, out, sa, TapParam<TAPS>(a.t));
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}
}  // namespace

int conv_stack_layers(const FwdArgs& a) {
    StackPlan p;
    return plan_stack(a, CS_W, &p, nullptr) ? p.nc : 0;
}

// Two workgroups of half the wavefronts on a CU hide each other's phases: better from the first image beyond one per CU
// where both hold their weights in LDS (40 x 40 x 4 through 16 and 32 channels, whole forward at 384, 2048 and 16384
// images 13.3, 26.9 and 157 us as one, 11.6, 20.1 and 104 as two).  With weights from L2 it depends: 64 x 64 x 8 through
// 32 and 64 channels at 2048 images 510 us as one, 552 as two; 64 x 64 x 6 through 32 and 32 36.5 and 32.5.
aq_status launch_conv_stack(const FwdArgs& a, int8_t* out, hipStream_t st) {
    StackPlan p;
    StackArgs sa;
    const bool taps = any_taps(a);
    constexpr int H = CS_W / 2;
    if (a.c.batch > 256 && plan_stack(a, H, &p, &sa) && p.resident)
        return taps ? launch_stack_t<true, true, H>(a, p, sa, out, st) : launch_stack_t<false, true, H>(a, p, sa, out, st);
    if (!plan_stack(a, CS_W, &p, &sa)) return AQ_ESHAPE;
    if (p.resident) return taps ? launch_stack_t<true, true, CS_W>(a, p, sa, out, st) : launch_stack_t<false, true, CS_W>(a, p, sa, out, st);
    return taps ? launch_stack_t<true, false, CS_W>(a, p, sa, out, st) : launch_stack_t<false, false, CS_W>(a, p, sa, out, st);
}

}  // namespace aq

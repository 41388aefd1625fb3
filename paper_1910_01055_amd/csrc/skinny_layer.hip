// Host side of the few-row layer kernel (skinny_layer.hpp) and the nibble copies of the weights.
#include "skinny_layer.hpp"

namespace aq {

namespace {
// 16 signed codes in [-7, 7] (one lane's 16 bytes of a k-step, words d0 .. d3) -> 8 bytes: word j holds the codes of
// d(2j) as the low nibbles of its bytes and those of d(2j + 1) as the high nibbles, each stored as c + 8
__global__ __launch_bounds__(256) void k_pack_nibbles(const v4i* __restrict__ wp, v2i* __restrict__ w4, int64_t pieces) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= pieces) return;
    const v4i d = wp[i];
    auto nib = [](int w) {  // per byte: (c + 8) & 15
        uint32_t r = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) r |= ((((uint32_t)w >> (8 * b)) + 8u) & 15u) << (8 * b);
        return r;
    };
    v2i q;
    q[0] = (int)(nib(d[0]) | (nib(d[1]) << 4));
    q[1] = (int)(nib(d[2]) | (nib(d[3]) << 4));
    w4[i] = q;
}
}  // namespace

// the last layer of an argmax policy whose logits fit one workgroup: the action index comes out of the
// same launch
bool skinny_layer_does_argmax(const FwdArgs& a, int l) {
    return l == a.net.n_layers - 1 && a.net.head == AQ_HEAD_ARGMAX && a.net.L[l].NT == 1;
}

bool skinny_layer_supported(const LayerDev& L, int64_t rows) {
    const bool fc = L.kh == 1 && L.kw == 1 && L.in_h == 1 && L.in_w == 1;
    return fc && (rows + 15) / 16 <= 65535;
}

aq_status launch_pack_nibbles(const int8_t* wp, uint8_t* w4, int64_t pieces, hipStream_t st) {
    hipLaunchKernelGGL(k_pack_nibbles, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st, (const v4i*)wp, (v2i*)w4, pieces);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

// Tiles of 16 per workgroup, by what a CU spends behind the fixed part of a launch: the operand bytes of the workgroups
// it takes, row tiles counted twice (their requests are the shorter ones, and each is another set of partial sums), and
// 1.4 times that where no second workgroup fills the waits of the first.  Layers of 2048 x 2048, four launches, us with
// 1 x 1, 2 x 1 (features x rows), 1 x 2, 2 x 2: 16 rows 12.7 13.4 14.3 15.8, 64 rows 14.8 14.3 15.5 17.3, 128 rows 21.8
// 16.6 18.7 17.9, 256 rows 32.9 24.9 27.7 24.5, 900 rows 83.7 66.5 77.5 66.1.
void few_row_tile(int N, int64_t rows, bool argmax, int* ft, int* rt) {
    double best = 1e300;
    for (int f = 1; f <= 2; ++f) {
        if (argmax && 16 * f < N) continue;
        for (int r = 1; r <= 2; ++r) {
            const int64_t wgs = ((N + 16 * f - 1) / (16 * f)) * ((rows + 16 * r - 1) / (16 * r));
            const double c = (wgs > 256 ? (double)((wgs + 255) / 256) : 1.4) * (f + 2 * r);
            if (c < best) {
                best = c;
                *ft = f;
                *rt = r;
            }
        }
    }
}

// A whole-network kernel passes every weight through the vector memory path of one CU, however few the rows; the layers'
// own launches spread them over the chip.  Measured, us (whole network / layers), 16 rows, 61 inputs: 512x3 10.4 / 11.9, with a
// LayerNorm 11.2 / 15.0; 1024x2 15.2 / 9.8, with a LayerNorm 15.8 / 12.6; 1024x3 23.6 / 12.3, with a LayerNorm 24.3 / 15.3; 300 rows
// 1024x3 23.8 / 18.3, with a LayerNorm 24.8 / 21.7; 400-300 6.3 / 9.5; per-tensor weights 1024x3 24.2 / 12.4, 512x3 11.2 / 12.0.
// An event behind the forward (streams other than the default one) costs 2.8 to 3.5.  The first forward behind a quantize or an
// import finds its weights in no L2, and each launch waits for its own: a whole pull of 28-512x2-1 24.8 us in one launch, 27.8 layer
// by layer.
bool few_rows_faster(const FwdArgs& a, bool noise, bool guarded, bool cold) {
    const int nl = a.net.n_layers;
    if (a.c.batch > kFewMaxRows || nl < 2) return false;
    double weights = 0.0;  // millions
    int widest = 0, lns = 0;
    for (int l = 0; l < nl; ++l) {
        const LayerDev& L = a.net.L[l];
        weights += 1e-6 * L.K * L.N;
        if (l == nl - 1) break;
        if (L.act == AQ_ACT_LN_TANH) ++lns;
        widest = widest > L.N ? widest : L.N;
    }
    if (widest < kFewMinWidth) return false;
    if (a.net.head == AQ_HEAD_ARGMAX && !skinny_layer_does_argmax(a, nl - 1)) return false;
    for (int l = 0; l < nl; ++l)
        if (!layer_uses_skinny(a, l)) return false;
    const double whole = 7.0 + 8.2 * weights + 0.9 * lns;  // (an upper bound: between 512x2 and 512x3 the two are within 1 us)
    const double layers = nl * (a.c.batch > 256 ? 5.0 : a.c.batch > 128 ? 3.5 : 3.1) + 3.0 * lns + (noise ? 3.1 : 0.0) + (guarded ? 3.3 : cold ? 1.6 : 0.0);
    return layers < whole;
}

aq_status launch_layer_skinny(const FwdArgs& a, int l, const LayerIO& io, hipStream_t st) {
    const LayerDev& L = a.net.L[l];
    const int64_t rows = a.c.batch;
    const bool first = l == 0, last = l == a.net.n_layers - 1, ln = !last && L.act == AQ_ACT_LN_TANH;
    const int in = io.in_blocked ? IN_BLOCKED : first && !a.net.in_u8 ? IN_F32 : IN_ROWS;
    const bool argmax = skinny_layer_does_argmax(a, l);
    int ft = 1, rt = 1;
    few_row_tile(L.N, rows, argmax, &ft, &rt);
    const bool asym = a.net.asym != 0;
    const uint8_t* w4 = asym ? nullptr : a.w4[l];
    void* out = !last ? (ln ? (void*)io.ln_x : (void*)io.out) : argmax || a.net.head != AQ_HEAD_ARGMAX ? a.c.actions : nullptr;
    const int flags = (first ? SF_FIRST : 0) | (last ? SF_LAST : 0) | (ln ? SF_LN : 0) | (!last && L.act == AQ_ACT_RELU ? SF_RELU : 0) |
                      (a.net.head == AQ_HEAD_TANH ? SF_TANH : 0) | (argmax ? SF_ARGMAX : 0) | (io.out_blocked ? SF_BLOCKED : 0) | l << SF_LAYER;
    const SkinnyCall call{st, SkinnyLayer{a.d_net, w4 ? (const void*)w4 : L.wp, L.bias_fold, L.rshift, L.z_w, io.in, out,
                                          last ? io.y : nullptr, L.K, L.N, (int32_t)rows, flags},
                          a.t, any_taps(a), ft, rt, in};
    if (asym) skinny_go_asym(call);
    else if (w4) skinny_go_w4(call);
    else skinny_go_sym(call);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

}  // namespace aq

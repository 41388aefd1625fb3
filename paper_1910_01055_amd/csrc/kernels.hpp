// Host-side launchers of the HIP kernels (internal to the library).
#pragma once
#include "common.hpp"

namespace aq {

// ---- quantizer block (quantize.hip)
aq_status launch_fill_u32(uint32_t* p, int n, uint32_t v, hipStream_t st);
// a grid's threads along one dimension are counted in 32 bits
inline bool grid_ok(int64_t workgroups, int threads) { return workgroups <= 0xffffffffLL / threads; }
// qdenom, qmax (largest unsigned code) and qw (largest symmetric code) describe the n-bit code range
aq_status launch_quantize_tensor(const float* d_w, int64_t rows, int64_t cols, int wscheme, float qdenom,
                                 int qmax, int qw, void* d_codes, float* d_scale, int32_t* d_zp, uint32_t* d_ws, hipStream_t st);
// The whole policy: activation parameters, weight ranges (per-tensor scheme), packed 8-bit weights and
// per-channel constants of every layer, in two launches.
aq_status launch_quantize_policy(const QTab* d_tab, const QTab& h_tab, const QPtrs& ptrs, const RangesArg& r, const QOut& o,
                                 hipStream_t st);
// the quantize pass's traffic without its arithmetic (n a multiple of 4)
aq_status launch_stream_reference(const float* d_in, int64_t n, void* d_out, hipStream_t st);
// the pipelined wide kernel's k-step loop alone (mfma_reference.hip); sizes as in aq_mfma_loop_reference
aq_status launch_mfma_reference(const void* d_weights, const void* d_acts, int ksteps, bool stream_weights, int workgroups,
                                int32_t* d_acc, hipStream_t st);
aq_status launch_unpack_weights(const int8_t* wp, int N, int K, int KS, int asym, uint8_t* codes, hipStream_t st);

// ---- policy blob (quantize.hip): header words [0..15] = magic, version, hash lo/hi, payload bytes lo/hi, 0...; then
// 32 words of which tail_words are the activation parameters and short-form flags; then the layer part of the slab
struct BlobHead {
    uint32_t w[6];
    int tail_words;
};
inline int64_t blob_copy_blocks(int64_t bytes) {  // 16 KiB per workgroup, at most four resident workgroups per CU
    const int64_t g = (bytes + 16383) / 16384;
    return g < 1 ? 1 : g > 2048 ? 2048 : g;
}
aq_status launch_blob_export(const BlobHead& h, const void* d_tail, const void* slab, int64_t bytes, void* blob, hipStream_t st);
aq_status launch_blob_import(const BlobHead& h, void* d_tail, void* slab, int64_t bytes, const void* blob, int* status, hipStream_t st);
// The packed blob: per layer the weight codes (operand order, signed domain) as n-bit fields, padded to 256 bytes, then
// the layer's constants as they are; offsets in bytes within blob and slab.
struct PackedLayer {
    int64_t w_off, w_src, c_off, c_src, c_bytes, groups;  // groups of 32 codes
    int N, K, KS, blk0, code_blks, const_blks;
};
struct PackedArgs {
    PackedLayer L[AQ_MAX_LAYERS];
    int n_layers, bits, off, blocks;
};
aq_status launch_packed_export(const BlobHead& h, const PackedArgs& a, const void* d_tail, const void* slab, void* blob, hipStream_t st);
aq_status launch_packed_import(const BlobHead& h, const PackedArgs& a, void* d_tail, void* slab, const void* blob, int* status, hipStream_t st);

// ---- exploration on the produced actions (explore.hip)
aq_status launch_explore(void* d_actions, int64_t rows, int A, int head, const float* d_sigma, float epsilon,
                         uint64_t seed, uint64_t step, hipStream_t st);

// ---- 8-bit forward (forward_int8.hip)
struct FwdArgs {
    explicit FwdArgs(const NetDev& n) : net(n) {}
    const NetDev& net;              // the handle's host copy, for planning
    const NetDev* d_net = nullptr;  // the same, in device memory
    CallArgs c{};
    TapArgs t{};
    bool taps = false;              // any pointer of `t` is set
    // host side only: per layer, the weights as nibbles for the few-row kernel (policies of at most 4 bits), or NULL
    const uint8_t* w4[AQ_MAX_LAYERS] = {};
};

// whole-network fused MLP kernel; returns AQ_ESHAPE when the network does not fit it
bool any_taps(const FwdArgs& a);
bool fused_mlp_supported(const FwdArgs& a, int* rows_per_wg_out, int* tiles_per_wave_out = nullptr);
aq_status launch_fused_mlp(const FwdArgs& a, hipStream_t st);
// software-pipelined whole-network kernel for wide layers (wide_mlp.hip); launch_fused_mlp hands it the shapes it takes
bool wide_mlp_supported(const FwdArgs& a, int* ld_out);
aq_status launch_wide_mlp(const FwdArgs& a, hipStream_t st);
// whole-network kernel for small networks, 16, 32 or 64 rows per workgroup (rows16_mlp.hpp / .hip);
// launch_fused_mlp hands it the shapes it takes
bool rows16_mlp_supported(const FwdArgs& a);
int rows16_mlp_row_tiles(int64_t batch);  // 16-row tiles per workgroup at this batch: 1, 2 or 4
bool rows16_mlp_alone_on_cu(int64_t batch);  // at most one 16-row workgroup per CU at this batch
aq_status launch_rows16_mlp(const FwdArgs& a, hipStream_t st);
// which kernel launch_fused_mlp runs for this network and batch (observations 16-byte aligned): 0 = the general
// fused kernel, 1 = the pipelined kernel for wide layers, 2 = the 16-row kernel for small networks
int fused_mlp_kernel_kind(const FwdArgs& a);

// one launch per layer (FC and implicit-GEMM convolution), activations in global memory
struct LayerIO {
    const void* in;   // layer 0: observations (fp32 or uint8); else int8 signed-domain [rows][K]
    int8_t* out;      // hidden layers: int8 signed-domain [rows][N] (row stride N)
    float* ln_x;      // LN layers: fp32 scratch [rows][N]
    float* y;         // last layer: dequantized outputs [rows][N]
    // the few-row and the many-row kernel leave their maps in operand order for each other (skinny_layer.hip, rows_layer.hip); the tiled
    // one refuses such a map
    int in_blocked = 0, out_blocked = 0;
};
// bytes of such a map of `rows` rows and N features
inline size_t blocked_map_bytes(int64_t rows, int N) { return (size_t)((rows + 15) / 16 * 16) * (size_t)((N + 15) / 16 * 16); }
aq_status launch_layer_int8(const FwdArgs& a, int layer, const LayerIO& io, hipStream_t st);
// FC layers at few rows: small output tiles, K split over a workgroup's waves (skinny_layer.hip)
bool skinny_layer_supported(const LayerDev& L, int64_t rows);
// 16-feature and 16-row tiles per workgroup that such a layer takes (argmax: all features in one workgroup)
void few_row_tile(int N, int64_t rows, bool argmax, int* ft, int* rt);
bool skinny_layer_does_argmax(const FwdArgs& a, int l);
// whether an MLP that fits the whole-network kernels is faster layer by layer at this batch (at most kFewMaxRows rows, a
// hidden layer of at least kFewMinWidth); noise: exploration then takes a launch of its own; guarded: an event behind the forward;
// cold: the weights were just written
constexpr int kFewMaxRows = 512, kFewMinWidth = 257;
bool few_rows_faster(const FwdArgs& a, bool noise, bool guarded, bool cold);
// the leading convolution layers in one launch (0 layers = shapes it does not take); writes the last
// convolution's signed codes to `out` ([batch * oh * ow][N])
int conv_stack_layers(const FwdArgs& a);
aq_status launch_conv_stack(const FwdArgs& a, int8_t* out, hipStream_t st);
// whether launch_layer_int8 hands layer l at this batch to the K-split kernel
bool layer_uses_skinny(const FwdArgs& a, int l);
// fully connected layers at many rows (rows_layer.hip): input fp32 observations or a map in operand order, output such a map or fp32
// rows.  Whether layer l takes it, given that the next one reads such a map
bool layer_uses_rows(const FwdArgs& a, int l);
aq_status launch_layer_rows(const FwdArgs& a, int l, const LayerIO& io, hipStream_t st);
aq_status launch_layer_skinny(const FwdArgs& a, int l, const LayerIO& io, hipStream_t st);
// the few-row kernel's nibble weights from a layer's packed 8-bit operands: `pieces` = NT * KS * 64 (16 bytes -> 8)
aq_status launch_pack_nibbles(const int8_t* wp, uint8_t* w4, int64_t pieces, hipStream_t st);
// blocked: `out` in the few-row kernel's operand order
aq_status launch_ln_tanh_rows(const FwdArgs& a, int layer, const float* x, int8_t* out, int64_t rows, bool blocked, hipStream_t st);
aq_status launch_head_rows(const float* y, int64_t rows, int N, int head, void* actions, hipStream_t st);

// ---- fp32 actor (forward_fp32.hip)
struct Fp32Layer {
    const float* wpk;  // weights in operand order, see forward_fp32.hip
    const float* zeros;  // 1 KiB of them
    const float* b;
    int K, N;
    int relu;
    int head;  // last layer with an elementwise head applied to the outputs (aq_head), else -1
    int in_h, in_w, in_c, kh, kw, stride, oh, ow;
    int features_first;  // the grid's faster dimension is the features' (set at the launch)
};
// (min, max) of an activation tensor as it is collected: kRangeSlots pairs per tensor, each an order-preserving key of
// the float (the minimum's complemented, so that both are maxima and zero is neutral)
constexpr int kRangeSlots = 512;
struct RangeSlot {
    uint32_t not_lo, hi;
};
struct F32Ptrs {
    const float* w[AQ_MAX_LAYERS];    // row-major
    const float* wpk[AQ_MAX_LAYERS];  // in operand order
    const float* wsp[AQ_MAX_LAYERS];  // split into bf16 parts (a convolution stack's layers)
    const float* b[AQ_MAX_LAYERS];
    const float* gamma[AQ_MAX_LAYERS];
    const float* beta[AQ_MAX_LAYERS];
};
// the whole-MLP kernel's view of them: by value (parameters passed with the call) or one pointer to the handle's
// table, which keeps 320 bytes out of every launch
template <bool BYVAL>
struct F32PtrArg {
    F32Ptrs p;
    F32PtrArg(const F32Ptrs& v, const F32Ptrs*) : p(v) {}
};
template <>
struct F32PtrArg<false> {
    const F32Ptrs* p;
    F32PtrArg(const F32Ptrs&, const F32Ptrs* d) : p(d) {}
};
__device__ __forceinline__ const F32Ptrs& f32_ptrs(const F32PtrArg<true>& a) { return a.p; }
__device__ __forceinline__ const F32Ptrs& f32_ptrs(const F32PtrArg<false>& a) { return *a.p; }
struct F32Call {
    const void* obs;
    void* actions;  // NULL: calibration, the last layer is not run
    int64_t batch;
    RangeSlot* slots;  // kRangeSlots per activation tensor, or NULL
    int ld;            // LDS row stride, floats
};
// where a set of fp32 parameters goes: each array starts at workgroup blk0 of the copy's grid, one workgroup per
// kKeepPiece values
constexpr int kKeepPiece = 4096;
constexpr int kKeepSplit = 8;  // blocks of split weights (kind 5) per workgroup
struct F32KeepTab {
    struct Entry {
        int64_t off;  // bytes from where the set begins
        int64_t count;
        int kind, layer, N, K;  // kind: 0 weights, 1 bias, 2 gain, 3 offset, 4 packed weights,
                                  // 5 weights split into bf16 parts (a convolution stack's)
    };
    Entry e[5 * AQ_MAX_LAYERS + 4];  // (split weights: at most four layers)
    int blk0[5 * AQ_MAX_LAYERS + 4];
    int n, blocks;
};
aq_status launch_fp32_layer(const Fp32Layer& L, const void* in, int in_u8, float* out, int64_t rows, RangeSlot* slots,
                            hipStream_t st);
// features and rows of the tile that a layer takes at this number of rows
void fp32_layer_tile(const Fp32Layer& L, int64_t rows, int* features, int* tile_rows);
// whether the network runs as one launch at this batch; rt = 16-row tiles per workgroup then
bool fp32_mlp_fits(const NetDev& n, int64_t batch, int* rt);
aq_status launch_fp32_mlp(const NetDev& n, const NetDev* d_net, const F32Ptrs& ptrs, const F32Ptrs* d_ptrs, const void* obs,
                          int64_t batch, void* actions, RangeSlot* slots, int rt, hipStream_t st);
// the leading convolutions of a frame policy in one launch (fp32_conv_stack.hip): how many layers (0: none of these shapes;
// their weights are also kept split), and the launch, which writes the last one's map to `out`; with slots also the
// ranges of the frames and of every map
// What the choice between it and the layers' own launches goes by: the launch's time for a round of 256 images by its plan, us;
// kilobytes of a frame whose rows are no whole pieces of 8 bytes, twice where they are none of 4; of the layers, millions of operand
// values and of products an image
struct Fp32StackWork {
    double round = 0.0, ragged = 0.0, operands = 0.0, products = 0.0;
};
bool fp32_conv_stack_faster(const Fp32StackWork& w, int nc, int64_t batch);
int fp32_conv_stack_layers(const NetDev& n, Fp32StackWork* w);
aq_status launch_fp32_conv_stack(const NetDev& n, const F32Ptrs& ptrs, const void* frames, int64_t batch, float* out, RangeSlot* slots,
                                 hipStream_t st);
aq_status launch_fp32_ln_tanh(float* x, int64_t rows, int N, const float* gamma, const float* beta, float eps,
                              RangeSlot* slots, hipStream_t st);
aq_status launch_fp32_argmax(const float* y, int64_t rows, int N, int32_t* actions, hipStream_t st);
aq_status launch_input_range(const void* x, int is_u8, int64_t n, RangeSlot* slots, hipStream_t st);
aq_status launch_ranges_out(RangeSlot* slots, int n, float* out, uint32_t* ready, uint32_t ticket, hipStream_t st);
aq_status launch_keep_params(const F32Ptrs& src, const F32KeepTab* d_tab, void* base, int blocks, hipStream_t st);


// ---- half-precision actor (fp16_actor.hip)
struct Fp16Layer {
    const void* wp;     // binary16 weights in MFMA operand order, [NT][KS16] tiles of 1 KiB
    const float* bias;  // binary16 values widened to fp32, padded to NT * 32
    int K, N, KS16, NT, fc, relu;
    int in_h, in_w, in_c, kh, kw, stride, oh, ow;
    float* head_actions;  // last layer with an elementwise head: fp32 actions [rows][N], else NULL
    int head_tanh;
    int32_t* head_argmax;  // last layer of an argmax policy run by the few-row kernel with one feature tile:
                           // action indices [rows], else NULL
    int in_blocked, out_blocked;  // input / output in the few-row kernel's operand order
};
// The learner's parameters -> binary16, every array of every layer in one launch: entry i starts at workgroup blk0[i].
// Weights go into operand order (kind 0: 16 tiles of 32 features x 16 k per workgroup), biases, gains and offsets
// (kinds 1 to 3, padded to NT * 32) into a vector of widened values and one of halfs.
struct Fp16ConvTab {
    struct Entry {
        void* dst;
        void* dst_h;
        int kind, layer, N, K, KS16, NT;
    };
    Entry e[4 * AQ_MAX_LAYERS];
    int blk0[4 * AQ_MAX_LAYERS];
    int n, blocks;
};
constexpr int kConvTiles = 16;
aq_status launch_fp16_convert(const F32Ptrs& src, const Fp16ConvTab* d_tab, int blocks, int* status, hipStream_t st);

// ---- whole fully connected policies in half precision (fp16_mlp.hip)
struct Fp16LayerDev {
    const void* wp;
    int K, N, KS16, NT, act;
    int c_off;  // where the layer's constants begin among the network's, in halfs: bias, then gain and offset, NT * 32 each
};
struct Fp16Net {
    Fp16LayerDev L[AQ_MAX_LAYERS];
    const void* consts;
    int n_layers;  // 0: not a fully connected policy
    int head, cst;  // cst: halfs of constants, a multiple of 8
    float eps;
};
struct Fp16Call {
    const void* obs;
    void* actions;
    int64_t batch;
    // LDS, in halfs: row stride of the activations, the constants, a LayerNorm's statistics, a narrow argmax head's logits
    int ld, off_const, off_red, off_y;
};
template <bool TAPS>
struct Fp16Taps {
    void* p[AQ_MAX_LAYERS];
    Fp16Taps(void* const* t, int n) {
        for (int l = 0; l < AQ_MAX_LAYERS; ++l) p[l] = l < n ? t[l] : nullptr;
    }
};
template <>
struct Fp16Taps<false> {
    int none;
    Fp16Taps(void* const*, int) : none(0) {}
};
// rows per workgroup where the policy runs as one launch at this batch size, else 0
int fp16_mlp_rows(const Fp16Net& n, int64_t batch);
aq_status launch_fp16_mlp(const Fp16Net& n, const Fp16Net* d_net, const void* obs, int in_u8, int64_t batch, void* actions,
                          void* const* taps, hipStream_t st);
// in_mode: 0 = binary16 activations, 1 = fp32 observations, 2 = uint8 observations
aq_status launch_layer_fp16(const Fp16Layer& L, const void* in, int in_mode, void* out, int64_t rows,
                            hipStream_t st);
// whether launch_layer_fp16 takes the few-row (K-split) kernel for this layer
bool fp16_layer_is_skinny(const Fp16Layer& L, int in_mode, int64_t rows);
aq_status launch_fp16_ln_tanh(void* x, int64_t rows, int N, const float* gamma, const float* beta, float eps,
                              hipStream_t st);
aq_status launch_fp16_head(const void* y, int64_t rows, int N, int head, void* actions, hipStream_t st);
// the leading convolutions of a frame policy in one launch (fp16_conv_stack.hip): how many layers it takes
// (0 = none of these shapes), and the launch, which writes the last convolution's map to `out`
int fp16_conv_stack_layers(const Fp16Layer* L, int n_layers, const void* obs, int in_mode0, int64_t batch);
aq_status launch_fp16_conv_stack(const Fp16Layer* L, int n_layers, const void* obs, int in_mode0, int64_t batch,
                                 void* out, hipStream_t st);

}  // namespace aq

// C ABI of the library: the policy handle, argument checks and the launch sequences.
#include <algorithm>
#include <cstddef>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "kernels.hpp"

using namespace aq;

// Scratch of aq_policy_forward_int8_static: the intermediate activations of the one-launch-per-layer plan for
// callers that cannot allocate.  The array is part of the library's device image, so every GPU the library
// runs on holds its own copy at its own address until the process ends; host code never uses the array's
// name as an address (it is only a host-side stand-in), but the per-device pointer looked up below.
static __device__ __align__(256) unsigned char scratch[AQ_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];  // per device, filled on first use with that device current

// device address of `scratch` on the current device (AQ_EHIP when the lookup fails)
aq_status static_scratch(unsigned char** out) {
    int dev = -1;
    if (hip_failed(hipGetDevice(&dev)) || dev < 0 || dev >= kMaxDevices) return AQ_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hip_failed(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) || !ptr) return AQ_EHIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = (unsigned char*)g_scratch_ptr[dev];
    return AQ_OK;
}
}  // namespace

namespace {

struct LayerBuf {
    aq_layer d;
    int K, N, K_pad, N_pad, KS, NT, oh, ow;
    bool fc;
    int8_t* wp;
    float* s_w;
    int32_t* z_w;
    int32_t* rowsum;
    int32_t* bias_q;
    int32_t* M0;
    int32_t* rshift;
    float* m;
    // The constants an epilogue reads per output channel sit in one contiguous pack of four
    // [N_pad] arrays, so that the fused kernel stages them with one linear copy:
    //   [0] bias_fold   [1] M0 (requantized layers) or m (LayerNorm and last layers)
    //   [2] rz or gamma [3] sh or beta          (a layer is either requantized or normalised)
    int32_t* bias_fold;
    int32_t* pack1;
    int32_t* rz;
    int32_t* sh;
    float* gamma;
    float* beta;
};

}  // namespace

struct F32Store {
    void* slab = nullptr;
    F32Ptrs ptrs{};            // host copy, and its device copy for the whole-MLP kernel
    F32Ptrs* d_ptrs = nullptr;
    F32KeepTab* d_tab = nullptr;
    int blocks = 0;            // of the launch that fills it
};

constexpr int kFewPairs = 4;

struct aq_policy {
    aq_net net;
    std::vector<LayerBuf> L;
    void* slab = nullptr;  // all per-layer buffers live in one allocation
    ActQ* actq = nullptr;
    int* status = nullptr;
    QOut qout{};
    RangeSlot* slots = nullptr;   // kRangeSlots per activation tensor, neutral between calls
    bool slots_dirty = false;     // a calibration ended early: clear them first
    const float* f32_zeros = nullptr;  // 1 KiB: the fp32 layers' weights past the end of K
    NetDev h_net{};            // host copy of the device-resident network description
    NetDev* d_net = nullptr;
    QTab h_qtab{};             // the quantizer's table of the policy, host copy and device copy
    QTab* d_qtab = nullptr;
    bool quantized = false;
    size_t layer_bytes = 0;    // the slab's leading part: every layer's packed weights and constants
    uint64_t net_hash = 0;     // of the network description (blob header)
    int path = 0;  // 0 auto, 1 fused only, 2 one launch per layer, 3 one launch per layer also for the convolutions
    bool conv_stack = true;
    bool subbyte = false;  // plan 4: plan 2 with the few-row layers streaming the nibble copies of their weights
    // activation scratch of the per-layer path (8-bit maps, the fp32 rows a LayerNorm layer hands to its row
    // kernel, the logits of an argmax head) and of the fp32 actor, grown on demand
    int64_t cap_i8 = 0, cap_f32 = 0;
    // ... and the maps of a policy that fits the whole-network kernels but runs few rows layer by layer (few_rows_faster):
    // kFewPairs pairs of them, since a forward that needs no scratch may overlap another on a second stream.  Made with the
    // policy: such a forward allocates nothing, as on the whole-network kernels.  Pair 0 belongs to the default stream,
    // which is the same one for good.  Any other handle may name a new stream once its own is destroyed, perhaps with work
    // in flight: those pairs are guarded by an event behind their last forward, whatever stream it was on.
    size_t few_bytes = 0;  // of one map; 0: the policy never takes that route
    size_t few_ln_bytes = 0;  // of a pair's fp32 rows into a LayerNorm
    int8_t* few_slab = nullptr;
    hipStream_t few_stream[kFewPairs] = {};  // of the pair's last forward
    hipEvent_t few_done[kFewPairs] = {};
    int8_t* act_i8[2] = {nullptr, nullptr};
    float* ln_x = nullptr;
    float* y_rows = nullptr;
    float* act_f32[2] = {nullptr, nullptr};
    int64_t ln_elems = 0;  // per sample: widest LayerNorm layer output
    int64_t y_elems = 0;   // per sample: logits kept for an argmax head
    // half-precision actor: binary16 weights in operand order and rounded bias / gain / offset per layer
    // (one allocation, made by the first aq_convert_params_fp16), and its activation scratch
    void* h16_slab = nullptr;
    std::vector<void*> h16_wp;
    std::vector<float*> h16_bias, h16_gamma, h16_beta;
    bool h16_ready = false;
    Fp16Net h16_net{};              // a fully connected policy's description for the whole-network kernel ...
    Fp16Net* d_h16_net = nullptr;   // ... and its device copy
    Fp16ConvTab* d_h16_tab = nullptr;
    int h16_blocks = 0;
    int64_t cap_f16 = 0;
    void* act_f16[2] = {nullptr, nullptr};
    // the learner's fp32 parameters, copied by aq_policy_set_params_fp32, and the packed weights of parameters passed
    // with a call (one allocation each)
    F32Store f32_kept;    // made by the first aq_policy_set_params_fp32
    F32Store f32_passed;  // made by the first aq_policy_forward_fp32_params (its table with the policy)
    bool f32_ready = false;
    int f32_stack = 0;    // leading convolutions that the fp32 actor runs in one launch
    Fp32StackWork f32_work;
    // policies of at most 4 bits, per-channel symmetric, under launch plan 4: the fully connected layers' weights
    // once more as nibbles, for the few-row kernel (one allocation when the plan is first chosen; rewritten by
    // the first forward pass after every quantize / import)
    void* w4_slab = nullptr;
    std::vector<uint8_t*> w4;
    bool w4_stale = true;
    bool cold = false;  // the 8-bit weights were quantized or imported since the last forward
    // aq_calibrate_fp32's answer, in host memory that the GPU writes (made by its first call): the number of the
    // calibration that is ready, then (min, max) per activation tensor
    uint32_t* calib = nullptr;
    uint32_t calib_ticket = 0;
    int64_t max_hidden_elems = 0;  // per sample, over hidden layer outputs
    int64_t max_out_elems = 0;     // per sample, over all layer outputs
};

static void fill_layer_dev(const aq_policy* p, int l, LayerDev& d) {
    const LayerBuf& b = p->L[l];
    d.wp = b.wp;
    d.bias_fold = b.bias_fold;
    d.M0 = b.M0;
    d.rshift = b.rshift;
    d.m = b.m;
    d.gamma = b.gamma;
    d.beta = b.beta;
    d.z_w = b.z_w;
    d.rz = b.rz;
    d.sh = b.sh;
    d.K = b.K;
    d.N = b.N;
    d.KS = b.KS;
    d.NT = b.NT;
    d.act = b.d.act;
    d.in_h = b.d.in_h;
    d.in_w = b.d.in_w;
    d.in_c = b.d.in_c;
    d.kh = b.d.kh;
    d.kw = b.d.kw;
    d.stride = b.d.stride;
    d.oh = b.oh;
    d.ow = b.ow;
}

// workgroups that share a layer's range reduction (per-tensor scheme)
static int range_blocks(int N, int K) {
    const int64_t b = ((int64_t)N * K / 4 + 1 + 255) / 256;
    return b > 256 ? 256 : (int)b;
}

static hipStream_t as_stream(void* s) { return (hipStream_t)s; }

constexpr int kMaxK = 1 << 16, kMaxN = 1 << 20, kMaxSide = 1 << 14;

extern "C" const char* aq_status_string(aq_status s) {
    switch (s) {
        case AQ_OK: return "ok";
        case AQ_EINVAL: return "invalid argument";
        case AQ_ESHAPE: return "unsupported or inconsistent layer shapes";
        case AQ_ENONFINITE: return "non-finite weights";
        case AQ_ENOTQUANT: return "policy not quantized yet";
        case AQ_EHIP: return "HIP runtime error";
        case AQ_ENOMEM: return "out of device memory";
        case AQ_ERANGE: return "requantization multiplier out of range";
        case AQ_ETOOBIG: return "needs more scratch memory than is available without allocating";
    }
    return "unknown";
}

// A set of fp32 parameters: the packed weights, with `keep` also row-major copies, biases, gains and offsets.  Fills the
// table that the launch filling the set reads, and returns the bytes the set takes.
static size_t f32_store_layout(const aq_policy* p, bool keep, F32KeepTab& tab) {
    size_t bytes = 0;
    int blk = 0;
    auto add = [&](int64_t n, int kind, int l) {
        tab.blk0[tab.n] = blk;
        tab.e[tab.n++] = F32KeepTab::Entry{(int64_t)bytes, n, kind, l, p->L[l].N, p->L[l].K};
        bytes += ((size_t)n * 4 + 255) / 256 * 256;
        blk += kind == 5 ? (int)((n / 769 + kKeepSplit - 1) / kKeepSplit) : (int)((n + kKeepPiece - 1) / kKeepPiece);
    };
    for (int l = 0; l < p->net.n_layers; ++l) {
        const LayerBuf& b = p->L[l];
        if (keep) {
            add((int64_t)b.N * b.K, 0, l);
            for (int i = 1; i < 4; ++i) add(b.N, i, l);
        }
        if (l < p->f32_stack) add((int64_t)((b.N + 15) / 16) * ((b.K + 31) / 32) * 769, 5, l);
        add((int64_t)((b.N + 15) / 16) * ((b.K + 15) / 16) * 256, 4, l);
    }
    tab.blocks = blk;
    return bytes;
}

// ... and where its arrays are, given where it begins
static F32Ptrs f32_store_ptrs(const F32KeepTab& tab, char* base) {
    F32Ptrs ptrs{};
    for (int i = 0; i < tab.n; ++i) {
        const F32KeepTab::Entry& e = tab.e[i];
        (e.kind == 0 ? ptrs.w : e.kind == 1 ? ptrs.b : e.kind == 2 ? ptrs.gamma : e.kind == 3 ? ptrs.beta : e.kind == 4 ? ptrs.wpk : ptrs.wsp)[e.layer] =
            (float*)(base + e.off);
    }
    return ptrs;
}

static void few_free(aq_policy* p) {
    if (p->few_slab) (void)hipFree(p->few_slab);
    for (hipEvent_t e : p->few_done)
        if (e) (void)hipEventDestroy(e);
}

extern "C" aq_status aq_policy_create(const aq_net* net, aq_policy** out) {
    if (!net || !out || !net->layers) return AQ_EINVAL;
    if (net->n_layers < 1 || net->n_layers > AQ_MAX_LAYERS) return AQ_EINVAL;
    if (net->head < 0 || net->head > AQ_HEAD_LINEAR) return AQ_EINVAL;
    if (net->wscheme != AQ_W_TENSOR_ASYM_U8 && net->wscheme != AQ_W_CHANNEL_SYM_S8) return AQ_EINVAL;
    if (net->in_type != AQ_IN_F32 && net->in_type != AQ_IN_U8) return AQ_EINVAL;
    if (net->qdenom != 255 && net->qdenom != 256) return AQ_EINVAL;
    if (!(net->ln_eps > 0.0f)) return AQ_EINVAL;
    if (net->wbits != 0 && (net->wbits < 2 || net->wbits > 8)) return AQ_EINVAL;
    int dev_count = 0;
    if (hip_failed(hipGetDeviceCount(&dev_count)) || dev_count < 1) return AQ_EHIP;

    aq_policy* p = new (std::nothrow) aq_policy();
    if (!p) return AQ_ENOMEM;
    p->net = *net;
    p->net.layers = nullptr;
    int64_t prev_elems = -1;
    int prev_h = 0, prev_w = 0, prev_c = 0;
    bool prev_conv = false;
    size_t bytes = 0;
    auto take = [&](size_t n) {
        size_t off = bytes;
        bytes += (n + 255) / 256 * 256;
        return off;
    };
    std::vector<size_t> offs;
    for (int l = 0; l < net->n_layers; ++l) {
        const aq_layer& d = net->layers[l];
        LayerBuf b{};
        b.d = d;
        if (d.act < 0 || d.act > AQ_ACT_LN_TANH || d.out_c < 1 || d.in_c < 1) {
            delete p;
            return AQ_EINVAL;
        }
        // Size limits: K products of two signed 8-bit values (each at most 2^14 in magnitude) must stay
        // inside the int32 accumulator, and tile counts and per-sample element counts inside int32.
        if (d.in_c > kMaxK || d.out_c > kMaxN ||
            (d.kind == AQ_CONV2D && (d.in_h > kMaxSide || d.in_w > kMaxSide ||
                                     (int64_t)d.kh * d.kw * d.in_c > kMaxK))) {
            delete p;
            return AQ_ESHAPE;
        }
        if (d.kind == AQ_FC) {
            b.fc = true;
            b.K = d.in_c;
            b.oh = b.ow = 1;
            b.d.in_h = b.d.in_w = b.d.kh = b.d.kw = b.d.stride = 1;
            if (prev_elems >= 0 && prev_elems != d.in_c) {
                delete p;
                return AQ_ESHAPE;
            }
        } else if (d.kind == AQ_CONV2D) {
            b.fc = false;
            if (d.kh < 1 || d.kw < 1 || d.stride < 1 || d.in_h < d.kh || d.in_w < d.kw) {
                delete p;
                return AQ_ESHAPE;
            }
            if (l > 0 && (!prev_conv || prev_h != d.in_h || prev_w != d.in_w || prev_c != d.in_c)) {
                delete p;
                return AQ_ESHAPE;
            }
            if (d.act == AQ_ACT_LN_TANH) {
                delete p;
                return AQ_ESHAPE;
            }
            b.K = d.kh * d.kw * d.in_c;
            b.oh = (d.in_h - d.kh) / d.stride + 1;
            b.ow = (d.in_w - d.kw) / d.stride + 1;
        } else {
            delete p;
            return AQ_EINVAL;
        }
        b.N = d.out_c;
        b.K_pad = round_up(b.K, kTile);
        b.N_pad = round_up(b.N, kTile);
        b.KS = b.K_pad / kTile;
        b.NT = b.N_pad / kTile;
        prev_conv = !b.fc;
        prev_h = b.oh;
        prev_w = b.ow;
        prev_c = b.N;
        prev_elems = (int64_t)b.oh * b.ow * b.N;
        if (l < net->n_layers - 1 && prev_elems > p->max_hidden_elems) p->max_hidden_elems = prev_elems;
        if (prev_elems > p->max_out_elems) p->max_out_elems = prev_elems;
        if (l < net->n_layers - 1 && d.act == AQ_ACT_LN_TANH && prev_elems > p->ln_elems) p->ln_elems = prev_elems;
        if (l == net->n_layers - 1 && net->head == AQ_HEAD_ARGMAX) p->y_elems = prev_elems;
        offs.push_back(take((size_t)b.NT * b.KS * 1024));
        for (int i = 0; i < 7; ++i) offs.push_back(take((size_t)b.N_pad * 4));
        offs.push_back(take((size_t)b.N_pad * 4 * 4));  // the epilogue constant pack, see LayerBuf
        p->L.push_back(b);
    }
    p->layer_bytes = bytes;
    size_t off_status = take(256);
    int rng_blks = 0;
    for (const LayerBuf& b : p->L) rng_blks += range_blocks(b.N, b.K);
    size_t off_part = take((size_t)rng_blks * 3 * 4);
    size_t off_qptrs = take(sizeof(QPtrs));
    size_t off_slots = take(sizeof(RangeSlot) * kRangeSlots * AQ_MAX_LAYERS);
    size_t off_zeros = take(1024);
    // what the host writes, side by side: one copy
    size_t off_net = take(sizeof(NetDev));
    size_t off_qtab = take(sizeof(QTab));
    size_t off_ftab = take(sizeof(F32KeepTab));
    if (hip_failed(hipMalloc(&p->slab, bytes))) {
        delete p;
        return AQ_ENOMEM;
    }
    // zero once: padding rows / k-steps of the packed weights and padded constants stay zero for good
    if (hip_failed(hipMemset(p->slab, 0, bytes))) {
        (void)hipFree(p->slab);
        delete p;
        return AQ_EHIP;
    }
    p->w4.assign(p->L.size(), nullptr);
    char* base = (char*)p->slab;
    size_t oi = 0;
    for (auto& b : p->L) {
        b.wp = (int8_t*)(base + offs[oi++]);
        b.s_w = (float*)(base + offs[oi++]);
        b.z_w = (int32_t*)(base + offs[oi++]);
        b.rowsum = (int32_t*)(base + offs[oi++]);
        b.bias_q = (int32_t*)(base + offs[oi++]);
        b.M0 = (int32_t*)(base + offs[oi++]);
        b.rshift = (int32_t*)(base + offs[oi++]);
        b.m = (float*)(base + offs[oi++]);
        int32_t* pack = (int32_t*)(base + offs[oi++]);
        b.bias_fold = pack;
        b.pack1 = pack + b.N_pad;
        b.rz = pack + 2 * b.N_pad;
        b.sh = pack + 3 * b.N_pad;
        b.gamma = (float*)b.rz;
        b.beta = (float*)b.sh;
    }
    p->status = (int*)(base + off_status);
    p->slots = (RangeSlot*)(base + off_slots);
    p->f32_zeros = (const float*)(base + off_zeros);
    p->d_net = (NetDev*)(base + off_net);
    p->d_qtab = (QTab*)(base + off_qtab);
    p->actq = p->d_net->actq;  // device address arithmetic only
    p->qout = QOut{p->actq, p->d_net->fast, p->status, (QPtrs*)(base + off_qptrs), (uint32_t*)(base + off_part)};
    for (int l = 0; l < net->n_layers; ++l) {
        fill_layer_dev(p, l, p->h_net.L[l]);
    }
    p->h_net.n_layers = net->n_layers;
    p->h_net.head = net->head;
    p->h_net.in_u8 = net->in_type == AQ_IN_U8;
    p->h_net.asym = net->wscheme == AQ_W_TENSOR_ASYM_U8;
    p->h_net.ln_eps = net->ln_eps;
    p->f32_stack = fp32_conv_stack_layers(p->h_net, &p->f32_work);
    F32KeepTab ftab{};  // of parameters passed with a call
    (void)f32_store_layout(p, false, ftab);
    {
        FwdArgs probe(p->h_net);
        probe.c.batch = 1;
        int r = 0, few_n = 0;
        for (int l = 0; l < net->n_layers - 1; ++l) few_n = std::max(few_n, p->L[l].N);
        // (one row: if the layers' launches are not faster there, they are at no batch)
        if (fused_mlp_supported(probe, &r) && few_rows_faster(probe, false, false, false)) {
            p->few_bytes = (blocked_map_bytes(kFewMaxRows, few_n) + 255) & ~(size_t)255;
            p->few_ln_bytes = ((size_t)kFewMaxRows * (size_t)p->ln_elems * 4 + 255) & ~(size_t)255;
            if (hip_failed(hipMalloc((void**)&p->few_slab, kFewPairs * (2 * p->few_bytes + p->few_ln_bytes)))) {
                (void)hipFree(p->slab);
                delete p;
                return AQ_ENOMEM;
            }
            for (int i = 1; i < kFewPairs; ++i) {
                if (hip_failed(hipEventCreateWithFlags(&p->few_done[i], hipEventDisableTiming))) {
                    p->few_done[i] = nullptr;
                    few_free(p);
                    (void)hipFree(p->slab);
                    delete p;
                    return AQ_ENOMEM;
                }
            }
        }
    }
    {   // the quantizer's table: outputs per layer and each layer's first workgroup in the shared grids
        QTab& q = p->h_qtab;
        q.n_layers = net->n_layers;
        q.asym = p->h_net.asym;
        q.in_u8 = p->h_net.in_u8;
        q.qdenom = (float)net->qdenom;
        const int wbits = net->wbits ? net->wbits : 8;
        q.w_qmax = (1 << wbits) - 1;
        q.w_qw = (1 << (wbits - 1)) - 1;
        q.w_qdenom = net->qdenom == 256 ? (float)(q.w_qmax + 1) : (float)q.w_qmax;
        int row_blk = 0, rng_blk = 0;
        for (int l = 0; l < AQ_MAX_LAYERS; ++l) q.row_blk0[l] = q.rng_blk0[l] = 0x7fffffff;
        for (int l = 0; l < net->n_layers; ++l) {
            const LayerBuf& b = p->L[l];
            QLayerTab& t = q.L[l];
            t.wp = b.wp; t.s_w = b.s_w; t.z_w = b.z_w; t.rowsum = b.rowsum; t.bias_q = b.bias_q; t.M0 = b.M0;
            t.rshift = b.rshift; t.m = b.m; t.bias_fold = b.bias_fold; t.pack1 = b.pack1; t.rz = b.rz; t.sh = b.sh;
            t.N = b.N; t.K = b.K; t.KS = b.KS;
            t.ln = b.d.act == AQ_ACT_LN_TANH;
            t.requant = l < net->n_layers - 1 && !t.ln;
            q.row_blk0[l] = row_blk;
            q.rng_blk0[l] = rng_blk;
            t.rng_blks = range_blocks(b.N, b.K);
            row_blk += (b.N + QR_ROWS - 1) / QR_ROWS;
            rng_blk += t.rng_blks;
        }
        q.row_blks = row_blk;
        q.rng_blks_total = rng_blk;
    }
    {   // FNV-1a over everything that fixes the blob's layout and meaning
        uint64_t h = 1469598103934665603ull;
        auto mix = [&](int64_t v) {
            for (int i = 0; i < 8; ++i) {
                h ^= (uint64_t)(v >> (8 * i)) & 0xffu;
                h *= 1099511628211ull;
            }
        };
        mix(net->n_layers);
        mix(net->head);
        mix(net->wscheme);
        mix(net->in_type);
        mix(net->qdenom);
        mix(net->wbits ? net->wbits : 8);
        for (const auto& b : p->L) {
            mix(b.d.kind); mix(b.d.in_h); mix(b.d.in_w); mix(b.d.in_c); mix(b.d.out_c);
            mix(b.d.kh); mix(b.d.kw); mix(b.d.stride); mix(b.d.act);
        }
        mix((int64_t)p->layer_bytes);
        p->net_hash = h;
    }
    p->f32_passed.d_tab = (F32KeepTab*)(base + off_ftab);
    p->f32_passed.blocks = ftab.blocks;
    std::vector<char> up(off_ftab + sizeof(F32KeepTab) - off_net);
    memcpy(up.data(), &p->h_net, sizeof(NetDev));
    memcpy(up.data() + (off_qtab - off_net), &p->h_qtab, sizeof(QTab));
    memcpy(up.data() + (off_ftab - off_net), &ftab, sizeof(F32KeepTab));
    if (hip_failed(hipMemcpy(p->d_net, up.data(), up.size(), hipMemcpyHostToDevice))) {
        (void)hipFree(p->slab);
        few_free(p);
        delete p;
        return AQ_EHIP;
    }
    {   // set-up of the allocation-free forward: this device's address of the static scratch
        unsigned char* sc = nullptr;
        if (static_scratch(&sc) != AQ_OK) {
            (void)hipFree(p->slab);
            few_free(p);
            delete p;
            return AQ_EHIP;
        }
    }
    *out = p;
    return AQ_OK;
}

extern "C" aq_status aq_policy_destroy(aq_policy* p) {
    if (!p) return AQ_EINVAL;
    (void)hipDeviceSynchronize();
    if (p->slab) (void)hipFree(p->slab);
    if (p->w4_slab) (void)hipFree(p->w4_slab);
    few_free(p);
    for (int i = 0; i < 2; ++i) {
        if (p->act_i8[i]) (void)hipFree(p->act_i8[i]);
        if (p->act_f32[i]) (void)hipFree(p->act_f32[i]);
        if (p->act_f16[i]) (void)hipFree(p->act_f16[i]);
    }
    if (p->ln_x) (void)hipFree(p->ln_x);
    if (p->y_rows) (void)hipFree(p->y_rows);
    if (p->h16_slab) (void)hipFree(p->h16_slab);
    if (p->f32_kept.slab) (void)hipFree(p->f32_kept.slab);
    if (p->f32_passed.slab) (void)hipFree(p->f32_passed.slab);
    if (p->calib) (void)hipHostFree(p->calib);
    delete p;
    return AQ_OK;
}

// Growing a buffer frees and allocates device memory and waits for the device: not possible while the
// caller's stream is being captured into a graph, which the forward then reports instead of breaking the capture.
static bool capturing(hipStream_t st) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    return !hip_failed(hipStreamIsCapturing(st, &cs)) && cs != hipStreamCaptureStatusNone;
}

// bytes of one 8-bit activation map of the per-layer plan (a little slack behind the last row), and the same where
// fully connected layers' maps may lie in operand order
static size_t i8_map_bytes(const aq_policy* p, int64_t batch) {
    return (size_t)batch * (size_t)(p->max_hidden_elems > 0 ? p->max_hidden_elems : 1) + 64;
}
static size_t i8_map_bytes_blocked(const aq_policy* p, int64_t batch) {
    size_t n = i8_map_bytes(p, batch);
    for (const LayerBuf& b : p->L)
        if (b.fc) n = std::max(n, blocked_map_bytes(batch, b.N));
    return n;
}

static aq_status ensure_i8(aq_policy* p, int64_t batch, hipStream_t st) {
    if (batch <= p->cap_i8) return AQ_OK;
    if (capturing(st)) return AQ_ETOOBIG;
    (void)hipDeviceSynchronize();
    for (int i = 0; i < 2; ++i) {
        if (p->act_i8[i]) (void)hipFree(p->act_i8[i]);
        p->act_i8[i] = nullptr;
    }
    if (p->ln_x) (void)hipFree(p->ln_x);
    if (p->y_rows) (void)hipFree(p->y_rows);
    p->ln_x = p->y_rows = nullptr;
    p->cap_i8 = 0;
    for (int i = 0; i < 2; ++i)
        if (hip_failed(hipMalloc((void**)&p->act_i8[i], i8_map_bytes_blocked(p, batch)))) return AQ_ENOMEM;
    // fp32 rows exist only where the 8-bit path needs them: LayerNorm inputs, argmax logits
    if (p->ln_elems && hip_failed(hipMalloc((void**)&p->ln_x, (size_t)batch * p->ln_elems * 4 + 256))) return AQ_ENOMEM;
    if (p->y_elems && hip_failed(hipMalloc((void**)&p->y_rows, (size_t)batch * p->y_elems * 4 + 256))) return AQ_ENOMEM;
    p->cap_i8 = batch;
    return AQ_OK;
}

static aq_status ensure_f32(aq_policy* p, int64_t batch, hipStream_t st) {
    if (batch <= p->cap_f32) return AQ_OK;
    if (capturing(st)) return AQ_ETOOBIG;
    (void)hipDeviceSynchronize();
    for (int i = 0; i < 2; ++i) {
        if (p->act_f32[i]) (void)hipFree(p->act_f32[i]);
        p->act_f32[i] = nullptr;
    }
    p->cap_f32 = 0;
    size_t n = ((size_t)batch * (size_t)p->max_out_elems + 64) * sizeof(float);
    for (int i = 0; i < 2; ++i)
        if (hip_failed(hipMalloc((void**)&p->act_f32[i], n))) return AQ_ENOMEM;
    p->cap_f32 = batch;
    return AQ_OK;
}

static aq_status ensure_f16(aq_policy* p, int64_t batch, hipStream_t st) {
    if (batch <= p->cap_f16) return AQ_OK;
    if (capturing(st)) return AQ_ETOOBIG;
    (void)hipDeviceSynchronize();
    for (int i = 0; i < 2; ++i) {
        if (p->act_f16[i]) (void)hipFree(p->act_f16[i]);
        p->act_f16[i] = nullptr;
    }
    p->cap_f16 = 0;
    size_t n = ((size_t)batch * (size_t)p->max_out_elems + 64) * 2;
    for (const LayerBuf& b : p->L)  // (fully connected layers' maps may lie in operand order)
        if (b.fc) n = std::max(n, 2 * blocked_map_bytes(batch, b.N));
    for (int i = 0; i < 2; ++i)
        if (hip_failed(hipMalloc(&p->act_f16[i], n))) return AQ_ENOMEM;
    p->cap_f16 = batch;
    return AQ_OK;
}

// Storage of the parameters that aq_policy_set_params_fp32 keeps, made once.
static aq_status ensure_f32_kept(aq_policy* p, hipStream_t st) {
    F32Store& S = p->f32_kept;
    if (S.slab) return AQ_OK;
    if (capturing(st)) return AQ_ETOOBIG;
    struct {
        F32Ptrs ptrs;
        F32KeepTab tab;
    } up{};
    const size_t bytes = f32_store_layout(p, true, up.tab);
    char* slab = nullptr;
    if (hip_failed(hipMalloc((void**)&slab, bytes + sizeof(up)))) return AQ_ENOMEM;
    up.ptrs = f32_store_ptrs(up.tab, slab);
    if (hip_failed(hipMemcpy(slab + bytes, &up, sizeof(up), hipMemcpyHostToDevice))) {
        (void)hipFree(slab);
        return AQ_EHIP;
    }
    S.d_ptrs = (F32Ptrs*)(slab + bytes);
    S.d_tab = (F32KeepTab*)(slab + bytes + offsetof(decltype(up), tab));
    S.slab = slab;
    S.ptrs = up.ptrs;
    S.blocks = up.tab.blocks;
    return AQ_OK;
}

// Memory for the packed weights of parameters passed with a call, made once (their table is there from the start, so
// that this is an allocation and nothing else).  The call may be one into a graph: an allocation is no part of it,
// and the relaxed mode of this thread says that it is meant to happen now.
static aq_status ensure_f32_passed(aq_policy* p) {
    F32Store& S = p->f32_passed;
    if (S.slab) return AQ_OK;
    F32KeepTab tab{};
    const size_t bytes = f32_store_layout(p, false, tab);
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    AQ_HIP_CHECK(hipThreadExchangeStreamCaptureMode(&mode));
    const bool failed = hip_failed(hipMalloc(&S.slab, bytes));
    AQ_HIP_CHECK(hipThreadExchangeStreamCaptureMode(&mode));
    if (failed) {
        S.slab = nullptr;
        return AQ_ENOMEM;
    }
    S.ptrs = f32_store_ptrs(tab, (char*)S.slab);
    return AQ_OK;
}

// The pair of maps for a forward on `st`, which waits for what may still use it; -1: `st` is being captured (or cannot say so),
// or every pair is at work on another stream.
static int few_pair_of(aq_policy* p, hipStream_t st) {
    if (!st) return 0;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hip_failed(hipStreamIsCapturing(st, &cs)) || cs != hipStreamCaptureStatusNone) return -1;
    int mine = -1, idle = -1;
    for (int i = 1; i < kFewPairs && mine < 0; ++i) {
        if (p->few_stream[i] == st) mine = i;
        else if (!p->few_stream[i] && idle < 0) idle = i;
    }
    // (on the stream of the pair's last forward there is nothing to wait for and the runtime sees that, 0.1 us; the handle
    // may name a new one)
    if (mine > 0) return hip_failed(hipStreamWaitEvent(st, p->few_done[mine], 0)) ? -1 : mine;
    if (idle < 0) {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;  // (another thread may be capturing)
        if (hip_failed(hipThreadExchangeStreamCaptureMode(&mode))) return -1;
        for (int i = 1; i < kFewPairs && idle < 0; ++i)
            if (!hip_failed(hipEventQuery(p->few_done[i]))) idle = i;
        if (hip_failed(hipThreadExchangeStreamCaptureMode(&mode))) return -1;
    }
    if (idle > 0) p->few_stream[idle] = st;
    return idle;
}

extern "C" aq_status aq_policy_reserve(aq_policy* p, int64_t max_batch) {
    if (!p || max_batch < 0) return AQ_EINVAL;
    aq_status s = ensure_i8(p, max_batch, nullptr);
    if (s != AQ_OK) return s;
    if (p->h16_ready) {
        s = ensure_f16(p, max_batch, nullptr);
        if (s != AQ_OK) return s;
    }
    return ensure_f32(p, max_batch, nullptr);
}

extern "C" aq_status aq_policy_set_path(aq_policy* p, int32_t path) {
    if (!p || path < 0 || path > 4) return AQ_EINVAL;
    if (path == 4 && !p->w4_slab && p->net.wbits != 0 && p->net.wbits <= 4 && p->net.wscheme == AQ_W_CHANNEL_SYM_S8) {
        size_t w4_bytes = 0;
        std::vector<size_t> need(p->L.size(), 0);
        for (size_t l = 0; l < p->L.size(); ++l) {
            const LayerBuf& b = p->L[l];
            LayerDev probe{};
            probe.kh = probe.kw = probe.in_h = probe.in_w = b.fc ? 1 : 2;
            probe.KS = b.KS;
            if (skinny_layer_supported(probe, 1)) need[l] = (size_t)b.NT * b.KS * 512;
            w4_bytes += need[l];
        }
        if (w4_bytes) {
            if (hip_failed(hipMalloc(&p->w4_slab, w4_bytes))) return AQ_ENOMEM;
            size_t o4 = 0;
            for (size_t l = 0; l < p->L.size(); ++l) {
                if (!need[l]) continue;
                p->w4[l] = (uint8_t*)p->w4_slab + o4;
                o4 += need[l];
            }
            p->w4_stale = true;
        }
    }
    p->conv_stack = path != 3;
    p->subbyte = path == 4;
    p->path = path >= 3 ? 2 : path;
    return AQ_OK;
}

extern "C" aq_status aq_policy_conv_stack_layers(const aq_policy* p, int32_t* n_layers) {
    if (!p || !n_layers) return AQ_EINVAL;
    FwdArgs a(p->h_net);
    a.c.batch = 1;
    *n_layers = p->conv_stack ? conv_stack_layers(a) : 0;
    return AQ_OK;
}

extern "C" aq_status aq_policy_fused_plan(const aq_policy* p, int64_t batch, int32_t* rows, int32_t* tiles,
                                          int32_t* kind) {
    if (!p || !rows || !tiles || !kind || batch < 1) return AQ_EINVAL;
    FwdArgs a(p->h_net);
    a.c.batch = batch;
    int r = 0, t = 0;
    if (p->path == 2 || !fused_mlp_supported(a, &r, &t) || (p->path == 0 && p->few_bytes && few_rows_faster(a, false, false, false))) r = t = 0;
    *rows = r;
    *tiles = t;
    *kind = r != 0 ? fused_mlp_kernel_kind(a) : 0;
    return AQ_OK;
}

extern "C" aq_status aq_policy_subbyte_layers(const aq_policy* p, int64_t batch, int32_t* n_layers) {
    if (!p || !n_layers || batch < 1) return AQ_EINVAL;
    FwdArgs a(p->h_net);
    a.c.batch = batch;
    int r = 0;
    int n = 0;
    if (p->path == 2 || !fused_mlp_supported(a, &r)) {
        const int nc = p->conv_stack ? conv_stack_layers(a) : 0;
        for (int l = nc; l < (int)p->L.size(); ++l)
            n += p->subbyte && p->w4[l] && !p->h_net.asym && layer_uses_skinny(a, l);
    }
    *n_layers = n;
    return AQ_OK;
}

// how many convolutions of a frame policy run in one launch at this batch
static int f32_stack_layers(const aq_policy* p, int64_t batch) {
    return p->conv_stack && p->f32_stack && fp32_conv_stack_faster(p->f32_work, p->f32_stack, batch) ? p->f32_stack : 0;
}

extern "C" aq_status aq_policy_fp32_plan(const aq_policy* p, int64_t batch, int32_t* rows, int32_t* tiles) {
    if (!p || !rows || !tiles || batch < 1) return AQ_EINVAL;
    int rt = 1;
    *rows = fp32_mlp_fits(p->h_net, batch, &rt) ? 16 * rt : 0;
    for (int l = 0; l < p->net.n_layers; ++l) {
        const LayerBuf& b = p->L[l];
        Fp32Layer L{};
        L.K = b.K;
        L.N = b.N;
        tiles[2 * l] = tiles[2 * l + 1] = 0;
        if (!*rows && l >= f32_stack_layers(p, batch)) fp32_layer_tile(L, batch * b.oh * b.ow, &tiles[2 * l], &tiles[2 * l + 1]);
    }
    return AQ_OK;
}

extern "C" aq_status aq_policy_fp16_plan(const aq_policy* p, int64_t batch, int32_t* rows) {
    if (!p || !rows || batch < 1) return AQ_EINVAL;
    if (!p->h16_ready) return AQ_ENOTQUANT;
    *rows = fp16_mlp_rows(p->h16_net, batch);
    return AQ_OK;
}

extern "C" aq_status aq_policy_status(aq_policy* p, void* stream) {
    if (!p) return AQ_EINVAL;
    int h2[2] = {0, 0};  // [0] the 8-bit policy's status word, [1] the half-precision policy's
    AQ_HIP_CHECK(hipStreamSynchronize(as_stream(stream)));
    AQ_HIP_CHECK(hipMemcpy(h2, p->status, sizeof(h2), hipMemcpyDeviceToHost));
    const int h = h2[0] | (h2[1] & kStatNonFinite);
    if (h & kStatNonFinite) return AQ_ENONFINITE;
    if (h & kStatRange) return AQ_ERANGE;
    if (h & kStatBlob) return AQ_EINVAL;
    return AQ_OK;
}

// ---- policy blob: [64-byte header][128-byte tail: activation (scale, zero-point) pairs and
// short-form flags][the slab's layer part]
namespace {
constexpr size_t kBlobHeader = 64, kBlobTail = 128;
constexpr uint32_t kBlobMagic = 0x42515141u;  // "AQQB"
constexpr uint32_t kBlobVersion = 1;
static_assert(sizeof(ActQ) * (AQ_MAX_LAYERS + 1) + sizeof(int) * AQ_MAX_LAYERS <= kBlobTail, "tail fits");
static_assert(offsetof(NetDev, fast) == offsetof(NetDev, actq) + sizeof(ActQ) * (AQ_MAX_LAYERS + 1),
              "scales, zero-points and flags are contiguous");
void blob_words(const aq_policy* p, uint32_t (&w)[6]) {
    const uint64_t payload = kBlobTail + p->layer_bytes;
    w[0] = kBlobMagic;
    w[1] = kBlobVersion;
    w[2] = (uint32_t)p->net_hash;
    w[3] = (uint32_t)(p->net_hash >> 32);
    w[4] = (uint32_t)payload;
    w[5] = (uint32_t)(payload >> 32);
}
constexpr size_t kTailBytes = sizeof(ActQ) * (AQ_MAX_LAYERS + 1) + sizeof(int) * AQ_MAX_LAYERS;
}  // namespace

// the nibble copies of the weights follow every change of the packed 8-bit operands: written by the first forward
// pass under launch plan 4 after such a change
static aq_status refresh_w4(aq_policy* p, hipStream_t st) {
    for (size_t l = 0; l < p->L.size(); ++l) {
        if (!p->w4[l]) continue;
        const LayerBuf& b = p->L[l];
        const aq_status s = launch_pack_nibbles(b.wp, p->w4[l], (int64_t)b.NT * b.KS * 64, st);
        if (s != AQ_OK) return s;
    }
    p->w4_stale = false;
    return AQ_OK;
}

extern "C" aq_status aq_policy_blob_size(const aq_policy* p, uint64_t* bytes) {
    if (!p || !bytes) return AQ_EINVAL;
    *bytes = kBlobHeader + kBlobTail + p->layer_bytes;
    return AQ_OK;
}

static BlobHead blob_head(const uint32_t (&w)[6]) {
    BlobHead h;
    for (int i = 0; i < 6; ++i) h.w[i] = w[i];
    h.tail_words = (int)(kTailBytes / 4);
    return h;
}

extern "C" aq_status aq_policy_export_blob(const aq_policy* p, void* d_blob, uint64_t bytes, void* stream) {
    if (!p || !d_blob || ((uintptr_t)d_blob & 15)) return AQ_EINVAL;
    if (bytes < kBlobHeader + kBlobTail + p->layer_bytes) return AQ_EINVAL;
    if (!p->quantized) return AQ_ENOTQUANT;
    uint32_t w[6];
    blob_words(p, w);
    return launch_blob_export(blob_head(w), p->d_net->actq, p->slab, (int64_t)p->layer_bytes, d_blob, as_stream(stream));
}

extern "C" aq_status aq_policy_import_blob(aq_policy* p, const void* d_blob, uint64_t bytes, void* stream) {
    if (!p || !d_blob || ((uintptr_t)d_blob & 15)) return AQ_EINVAL;
    if (bytes < kBlobHeader + kBlobTail + p->layer_bytes) return AQ_EINVAL;
    uint32_t w[6];
    blob_words(p, w);
    const aq_status s = launch_blob_import(blob_head(w), p->d_net->actq, p->slab, (int64_t)p->layer_bytes, d_blob, p->status,
                                           as_stream(stream));
    if (s != AQ_OK) return s;
    p->w4_stale = p->cold = true;
    p->quantized = true;
    return AQ_OK;
}

// ---- packed policy blob: the same header (other magic) and tail, then per layer the weight codes as
// n-bit fields (n = the policy's weight precision) followed by the layer's constants verbatim.
namespace {
constexpr uint32_t kPackedMagic = 0x50515141u;  // "AQQP"
int policy_wbits(const aq_policy* p) { return p->net.wbits ? p->net.wbits : 8; }
// (also the grid of the launch: workgroup 0 for header and tail, then a layer's codes and its constants)
PackedArgs packed_layout(const aq_policy* p, size_t* total) {
    PackedArgs a{};
    a.n_layers = p->net.n_layers;
    a.bits = policy_wbits(p);
    a.off = p->h_net.asym ? 128 : (1 << (a.bits - 1)) - 1;
    a.blocks = 1;
    size_t at = kBlobHeader + kBlobTail;
    const char* base = (const char*)p->slab;
    for (size_t l = 0; l < p->L.size(); ++l) {
        const LayerBuf& b = p->L[l];
        PackedLayer& q = a.L[l];
        const size_t wb = (size_t)b.NT * b.KS * 1024;
        const size_t begin = (size_t)((const char*)b.wp - base);
        const size_t end = l + 1 < p->L.size() ? (size_t)((const char*)p->L[l + 1].wp - base) : p->layer_bytes;
        q.w_off = (int64_t)at;
        q.w_src = (int64_t)begin;
        q.groups = (int64_t)(wb / 32);
        at += (wb / 8 * a.bits + 255) / 256 * 256;
        q.c_off = (int64_t)at;
        q.c_src = (int64_t)(begin + wb);
        q.c_bytes = (int64_t)(end - begin - wb);
        at += (size_t)q.c_bytes;
        q.N = b.N;
        q.K = b.K;
        q.KS = b.KS;
        q.blk0 = a.blocks;
        q.code_blks = (int)((q.groups + 255) / 256);
        q.const_blks = (int)blob_copy_blocks(q.c_bytes);
        a.blocks += q.code_blks + q.const_blks;
    }
    *total = at;
    return a;
}
void packed_words(const aq_policy* p, size_t total, uint32_t (&w)[6]) {
    blob_words(p, w);
    w[0] = kPackedMagic;
    w[4] = (uint32_t)(total - kBlobHeader);
    w[5] = (uint32_t)((uint64_t)(total - kBlobHeader) >> 32);
}
}  // namespace

extern "C" aq_status aq_policy_packed_blob_size(const aq_policy* p, uint64_t* bytes) {
    if (!p || !bytes) return AQ_EINVAL;
    size_t total = 0;
    packed_layout(p, &total);
    *bytes = total;
    return AQ_OK;
}

extern "C" aq_status aq_policy_export_packed_blob(const aq_policy* p, void* d_blob, uint64_t bytes, void* stream) {
    if (!p || !d_blob || ((uintptr_t)d_blob & 15)) return AQ_EINVAL;
    size_t total = 0;
    const PackedArgs a = packed_layout(p, &total);
    if (bytes < total) return AQ_EINVAL;
    if (!p->quantized) return AQ_ENOTQUANT;
    uint32_t w[6];
    packed_words(p, total, w);
    return launch_packed_export(blob_head(w), a, p->d_net->actq, p->slab, d_blob, as_stream(stream));
}

extern "C" aq_status aq_policy_import_packed_blob(aq_policy* p, const void* d_blob, uint64_t bytes, void* stream) {
    if (!p || !d_blob || ((uintptr_t)d_blob & 15)) return AQ_EINVAL;
    size_t total = 0;
    const PackedArgs a = packed_layout(p, &total);
    if (bytes < total) return AQ_EINVAL;
    uint32_t w[6];
    packed_words(p, total, w);
    const aq_status s = launch_packed_import(blob_head(w), a, p->d_net->actq, p->slab, d_blob, p->status, as_stream(stream));
    if (s != AQ_OK) return s;
    p->w4_stale = true;
    p->cold = false;  // (the codes' expansion takes long enough: what follows it is launched by then)
    p->quantized = true;
    return AQ_OK;
}

static aq_status explore_args_ok(const aq_policy* p, const aq_explore* ex, int64_t batch) {
    if (batch > 0xffffffffLL) return AQ_EINVAL;
    const bool discrete = p->net.head == AQ_HEAD_ARGMAX;
    if (!discrete && !ex->d_sigma) return AQ_EINVAL;
    if (discrete && !(ex->epsilon >= 0.0f && ex->epsilon <= 1.0f)) return AQ_EINVAL;
    return AQ_OK;
}

extern "C" aq_status aq_policy_explore(const aq_policy* p, void* d_actions, int64_t batch, const aq_explore* ex,
                                       void* stream) {
    if (!p || !d_actions || !ex || batch < 0) return AQ_EINVAL;
    const aq_status es = explore_args_ok(p, ex, batch);
    if (es != AQ_OK) return es;
    if (batch == 0) return AQ_OK;
    const int A = p->L.back().N * p->L.back().oh * p->L.back().ow;
    return launch_explore(d_actions, batch, A, p->net.head, ex->d_sigma, ex->epsilon, ex->seed, ex->step,
                          as_stream(stream));
}

extern "C" aq_status aq_quantize_tensor(const float* d_w, int64_t rows, int64_t cols, int32_t wscheme,
                                        int32_t qdenom, void* d_codes, float* d_scale, int32_t* d_zp,
                                        void* d_workspace, void* stream) {
    if (!d_w || !d_codes || !d_scale || !d_zp || !d_workspace) return AQ_EINVAL;
    if (rows < 0 || cols < 0) return AQ_EINVAL;
    // qdenom = 2^n - 1 (default reading) or 2^n (literal) for n = 2..8 bits
    int bits = 0;
    for (int n = 2; n <= 8; ++n)
        if (qdenom == (1 << n) - 1 || qdenom == (1 << n)) bits = n;
    if (bits == 0) return AQ_EINVAL;
    if (wscheme != AQ_W_TENSOR_ASYM_U8 && wscheme != AQ_W_CHANNEL_SYM_S8) return AQ_EINVAL;
    if (cols % 4 != 0 || ((uintptr_t)d_w & 15) || ((uintptr_t)d_codes & 3)) return AQ_ESHAPE;
    if (rows > 0x7fffffffLL || cols / 4 > 0x7fffffffLL) return AQ_ESHAPE;
    if (rows == 0 || cols == 0) return AQ_OK;
    return launch_quantize_tensor(d_w, rows, cols, wscheme, (float)qdenom, (1 << bits) - 1, (1 << (bits - 1)) - 1,
                                  d_codes, d_scale, d_zp, (uint32_t*)d_workspace, as_stream(stream));
}

extern "C" aq_status aq_stream_reference(const float* d_in, int64_t n, void* d_out, void* stream) {
    if (!d_in || !d_out || n < 0) return AQ_EINVAL;
    if (n % 4 != 0 || ((uintptr_t)d_in & 15) || ((uintptr_t)d_out & 3)) return AQ_ESHAPE;
    if (n == 0) return AQ_OK;
    return launch_stream_reference(d_in, n, d_out, as_stream(stream));
}

extern "C" aq_status aq_mfma_loop_reference(const void* d_weights, const void* d_acts, int32_t ksteps, int32_t stream_weights,
                                             int32_t workgroups, int32_t* d_acc, void* stream) {
    if (!d_weights || !d_acts || !d_acc) return AQ_EINVAL;
    if (ksteps < 4 || ksteps % 4 != 0 || workgroups < 1 || workgroups > 65536) return AQ_EINVAL;
    if (((uintptr_t)d_weights & 15) || ((uintptr_t)d_acts & 15) || ((uintptr_t)d_acc & 3)) return AQ_ESHAPE;
    return launch_mfma_reference(d_weights, d_acts, ksteps, stream_weights != 0, workgroups, d_acc, as_stream(stream));
}

extern "C" aq_status aq_quantize_params(aq_policy* p, const float* const* h_d_w, const float* const* h_d_b,
                                        const float* const* h_d_gamma, const float* const* h_d_beta,
                                        const aq_range* h_ranges, void* stream) {
    if (!p || !h_ranges) return AQ_EINVAL;
    const int nl = p->net.n_layers;
    if (!h_d_w) {  // the parameters kept by aq_policy_set_params_fp32
        if (h_d_b || h_d_gamma || h_d_beta) return AQ_EINVAL;
        if (!p->f32_ready) return AQ_ENOTQUANT;
        h_d_w = p->f32_kept.ptrs.w;
        h_d_b = p->f32_kept.ptrs.b;
        h_d_gamma = p->f32_kept.ptrs.gamma;
        h_d_beta = p->f32_kept.ptrs.beta;
    }
    for (int l = 0; l < nl; ++l)
        if (!h_d_w[l]) return AQ_EINVAL;
    hipStream_t st = as_stream(stream);
    RangesArg r{};
    QPtrs ptrs{};
    for (int l = 0; l < nl; ++l) {
        r.lo[l] = h_ranges[l].lo;
        r.hi[l] = h_ranges[l].hi;
        ptrs.w[l] = h_d_w[l];
        ptrs.b[l] = h_d_b ? h_d_b[l] : nullptr;
        ptrs.gamma[l] = h_d_gamma ? h_d_gamma[l] : nullptr;
        ptrs.beta[l] = h_d_beta ? h_d_beta[l] : nullptr;
    }
    aq_status s = launch_quantize_policy(p->d_qtab, p->h_qtab, ptrs, r, p->qout, st);
    if (s != AQ_OK) return s;
    p->w4_stale = p->cold = true;
    p->quantized = true;
    return AQ_OK;
}

extern "C" aq_status aq_policy_export_layer(const aq_policy* p, int32_t layer, void* d_codes, float* d_w_scale,
                                            int32_t* d_w_zp, int32_t* d_bias_q, int32_t* d_mult, int32_t* d_rshift,
                                            float* d_m, void* stream) {
    if (!p || layer < 0 || layer >= p->net.n_layers) return AQ_EINVAL;
    if (!p->quantized) return AQ_ENOTQUANT;
    hipStream_t st = as_stream(stream);
    const LayerBuf& b = p->L[layer];
    if (d_codes) {
        aq_status s = launch_unpack_weights(b.wp, b.N, b.K, b.KS, p->net.wscheme == AQ_W_TENSOR_ASYM_U8,
                                            (uint8_t*)d_codes, st);
        if (s != AQ_OK) return s;
    }
    const size_t nb = sizeof(float) * b.N;
    if (d_w_scale) AQ_HIP_CHECK(hipMemcpyAsync(d_w_scale, b.s_w, nb, hipMemcpyDeviceToDevice, st));
    if (d_w_zp) AQ_HIP_CHECK(hipMemcpyAsync(d_w_zp, b.z_w, nb, hipMemcpyDeviceToDevice, st));
    if (d_bias_q) AQ_HIP_CHECK(hipMemcpyAsync(d_bias_q, b.bias_q, nb, hipMemcpyDeviceToDevice, st));
    if (d_mult) AQ_HIP_CHECK(hipMemcpyAsync(d_mult, b.M0, nb, hipMemcpyDeviceToDevice, st));
    if (d_rshift) AQ_HIP_CHECK(hipMemcpyAsync(d_rshift, b.rshift, nb, hipMemcpyDeviceToDevice, st));
    if (d_m) AQ_HIP_CHECK(hipMemcpyAsync(d_m, b.m, nb, hipMemcpyDeviceToDevice, st));
    return AQ_OK;
}

__global__ void k_split_actq(const ActQ* q, int n, float* s, int32_t* z) {
    int i = threadIdx.x;
    if (i < n) {
        if (s) s[i] = q[i].s;
        if (z) z[i] = q[i].z;
    }
}

extern "C" aq_status aq_policy_export_act_qparams(const aq_policy* p, float* d_scale, int32_t* d_zp, void* stream) {
    if (!p) return AQ_EINVAL;
    if (!p->quantized) return AQ_ENOTQUANT;
    hipLaunchKernelGGL(k_split_actq, dim3(1), dim3(64), 0, as_stream(stream), p->actq, p->net.n_layers, d_scale,
                       d_zp);
    return hipGetLastError() == hipSuccess ? AQ_OK : AQ_EHIP;
}

// where the one-launch-per-layer plan keeps its intermediate tensors
struct FwdScratch {
    int8_t* i8[2];  // 8-bit activation maps, ping-pong
    bool blocked;   // they hold maps in operand order too (whole tiles of 16 rows and features)
    float* ln_x;    // fp32 rows into a LayerNorm row kernel
    float* y;       // logits of an argmax head
};

// `fixed`: scratch the caller of this function provides (the allocation-free entry point); NULL = the handle's
// own buffers, grown on demand
static aq_status forward_int8_impl(aq_policy* p, const void* d_obs, int64_t batch, void* d_actions,
                                   const aq_taps* taps, const aq_explore* ex, void* stream,
                                   const FwdScratch* fixed = nullptr) {
    if (!p || batch < 0) return AQ_EINVAL;
    if (ex) {
        const aq_status es = explore_args_ok(p, ex, batch);
        if (es != AQ_OK) return es;
    }
    if (!p->quantized) return AQ_ENOTQUANT;
    if (batch == 0) return AQ_OK;
    if (!d_obs || !d_actions) return AQ_EINVAL;
    if (batch > (1LL << 40)) return AQ_EINVAL;
    hipStream_t st = as_stream(stream);
    const int nl = p->net.n_layers;
    FwdArgs a(p->h_net);
    a.d_net = p->d_net;
    a.c.obs = d_obs;
    a.c.actions = d_actions;
    a.c.batch = batch;
    a.c.K0 = p->L[0].K;
    a.c.in_u8 = p->h_net.in_u8;
    if (p->subbyte && p->w4_slab && p->w4_stale) {
        const aq_status ws = refresh_w4(p, st);
        if (ws != AQ_OK) return ws;
    }
    for (int l = 0; l < nl; ++l) a.w4[l] = p->subbyte ? p->w4[l] : nullptr;
    if (taps) {
        a.taps = true;
        for (int l = 0; l < nl; ++l) {
            a.t.acc[l] = taps->acc ? taps->acc[l] : nullptr;
            a.t.act[l] = taps->act ? taps->act[l] : nullptr;
            a.t.ln[l] = taps->ln_t ? taps->ln_t[l] : nullptr;
        }
        a.t.a0 = taps->a0;
        a.t.y = taps->y;
    }

    int rows;
    bool can_fuse = p->path != 2 && fused_mlp_supported(a, &rows);
    if (p->path == 1 && !can_fuse) return AQ_ESHAPE;
    // An MLP that fits a whole-network kernel runs there, but for few rows on wide layers.  (Not under capture, nor for
    // the allocation-free entry point: what is captured may be replayed on any stream beside any other, and needs no
    // scratch with the whole-network kernels.)
    const bool noise = ex && p->net.head != AQ_HEAD_ARGMAX;
    const bool cold = p->cold;
    p->cold = false;
    int pair = -1;
    if (can_fuse && p->path == 0 && p->few_bytes && !fixed && few_rows_faster(a, noise, st != nullptr, cold)) pair = few_pair_of(p, st);
    if (pair >= 0) can_fuse = false;
    // on every way out: the event behind this forward's last use of the pair
    struct Done {
        hipEvent_t e;
        hipStream_t st;
        ~Done() {
            if (e && hip_failed(hipEventRecord(e, st))) (void)hip_failed(hipStreamSynchronize(st));
        }
    } const done{pair > 0 ? p->few_done[pair] : nullptr, st};
    const int A = p->L.back().N * p->L.back().oh * p->L.back().ow;
    if (can_fuse) {
        // Gaussian noise rides in the kernel where it writes the actions itself (an elementwise head on
        // a narrow last layer); every other case takes the separate exploration launch below
        const bool fuse_ex = ex && p->net.head != AQ_HEAD_ARGMAX && p->L.back().NT <= 2;
        if (fuse_ex) {
            a.c.ex_sigma = ex->d_sigma;
            a.c.ex_k0 = (uint32_t)ex->seed;
            a.c.ex_k1 = (uint32_t)(ex->seed >> 32);
            a.c.ex_s0 = (uint32_t)ex->step;
            a.c.ex_s1 = (uint32_t)(ex->step >> 32);
        }
        const aq_status fs = launch_fused_mlp(a, st);
        if (fs != AQ_OK || !ex || fuse_ex) return fs;
        return launch_explore(d_actions, batch, A, p->net.head, ex->d_sigma, ex->epsilon, ex->seed, ex->step, st);
    }

    // one launch per layer
    aq_status s = AQ_OK;
    FwdScratch sc;
    if (fixed) {
        sc = *fixed;
    } else if (pair >= 0) {
        int8_t* const maps = p->few_slab + (size_t)pair * (2 * p->few_bytes + p->few_ln_bytes);
        sc = FwdScratch{{maps, maps + p->few_bytes}, true, (float*)(maps + 2 * p->few_bytes), nullptr};
    } else {
        s = ensure_i8(p, batch, st);
        if (s != AQ_OK) return s;
        sc = FwdScratch{{p->act_i8[0], p->act_i8[1]}, true, p->ln_x, p->y_rows};
    }
    if (a.net.in_u8 && a.t.a0) {
        const LayerBuf& b0 = p->L[0];
        const size_t n = (size_t)batch * b0.d.in_h * b0.d.in_w * b0.d.in_c;
        AQ_HIP_CHECK(hipMemcpyAsync(a.t.a0, d_obs, n, hipMemcpyDeviceToDevice, st));
        a.t.a0 = nullptr;
    }
    // the dequantized last-layer rows are only materialised for the y tap or for an argmax head
    float* ybuf = a.t.y ? a.t.y : (p->net.head == AQ_HEAD_ARGMAX ? sc.y : nullptr);
    // a frame policy's convolutions run as one launch where their shapes allow it
    const int nc = p->conv_stack ? conv_stack_layers(a) : 0;
    if (nc) {
        s = launch_conv_stack(a, sc.i8[(nc - 1) & 1], st);
        if (s != AQ_OK) return s;
    }
    // Wide layers at many rows may take a kernel that writes operand order only (and reads it, behind the first layer).  Settled from
    // the last layer backwards: one takes it if the next one reads that order, as one of its kind or of the few-row kernel's; and
    // in the loop only where its own input lies so.
    bool takes_many[AQ_MAX_LAYERS] = {}, reads_blocked[AQ_MAX_LAYERS + 1] = {};
    for (int l = nl - 1; l >= nc && sc.blocked; --l) {
        if (!p->L[l].fc) continue;
        takes_many[l] = nc == 0 && pair < 0 && reads_blocked[l + 1] && layer_uses_rows(a, l);
        reads_blocked[l] = takes_many[l] || layer_uses_skinny(a, l);
    }
    int blocked = 0;  // how the layer before left its output
    for (int l = nc; l < nl; ++l) {
        const LayerBuf& b = p->L[l];
        const int64_t rows_l = batch * b.oh * b.ow;
        LayerIO io;
        io.in_blocked = blocked;
        const bool ln = l < nl - 1 && b.d.act == AQ_ACT_LN_TANH;  // (its rows' kernel writes either order)
        const bool many = takes_many[l] && (l == 0 || blocked);
        blocked = many || (b.fc && reads_blocked[l + 1] && (ln || layer_uses_skinny(a, l)));
        io.out_blocked = ln ? 0 : blocked;
        io.in = l == 0 ? d_obs : (const void*)sc.i8[(l - 1) & 1];
        io.out = sc.i8[l & 1];
        io.ln_x = sc.ln_x;
        io.y = ybuf;
        s = many ? launch_layer_rows(a, l, io, st) : launch_layer_int8(a, l, io, st);
        if (s != AQ_OK) return s;
        if (ln) {
            s = launch_ln_tanh_rows(a, l, io.ln_x, io.out, rows_l, blocked, st);
            if (s != AQ_OK) return s;
        }
        if (l == nl - 1 && p->net.head == AQ_HEAD_ARGMAX && !(layer_uses_skinny(a, l) && skinny_layer_does_argmax(a, l))) {
            s = launch_head_rows(ybuf, rows_l, b.N, p->net.head, d_actions, st);
            if (s != AQ_OK) return s;
        }
    }
    if (ex) return launch_explore(d_actions, batch, A, p->net.head, ex->d_sigma, ex->epsilon, ex->seed, ex->step, st);
    return AQ_OK;
}

extern "C" aq_status aq_policy_forward_int8(aq_policy* p, const void* d_obs, int64_t batch, void* d_actions,
                                            const aq_taps* taps, void* stream) {
    return forward_int8_impl(p, d_obs, batch, d_actions, taps, nullptr, stream);
}

extern "C" aq_status aq_policy_step_int8(aq_policy* p, const void* d_obs, int64_t batch, void* d_actions,
                                         const aq_explore* ex, const aq_taps* taps, void* stream) {
    return forward_int8_impl(p, d_obs, batch, d_actions, taps, ex, stream);
}

extern "C" aq_status aq_policy_forward_int8_static(aq_policy* p, const void* d_obs, int64_t batch, void* d_actions,
                                                   void* stream) {
    if (!p || batch < 0) return AQ_EINVAL;
    unsigned char* base = nullptr;
    const aq_status ss = static_scratch(&base);
    if (ss != AQ_OK) return ss;
    // carve the static array: two 8-bit maps, LayerNorm rows, argmax logits (each piece 256-byte aligned)
    auto up = [](size_t n) { return (n + 255) / 256 * 256; };
    size_t map = up(i8_map_bytes(p, batch));
    const size_t ln = up((size_t)batch * (size_t)p->ln_elems * 4);
    const size_t y = up((size_t)batch * (size_t)p->y_elems * 4);
    FwdArgs probe(p->h_net);
    probe.c.batch = batch > 0 ? batch : 1;
    int rows = 0;
    const bool fused = p->path != 2 && fused_mlp_supported(probe, &rows);
    FwdScratch sc{{nullptr, nullptr}, false, nullptr, nullptr};
    if (!fused) {  // (the whole-network kernel keeps everything in LDS and needs none of it)
        if ((double)batch * (double)(p->max_hidden_elems + 4 * (p->ln_elems + p->y_elems)) > 1e12 ||
            2 * map + ln + y > (size_t)AQ_STATIC_SCRATCH_BYTES)
            return AQ_ETOOBIG;
        const size_t map_b = up(i8_map_bytes_blocked(p, batch));
        sc.blocked = 2 * map_b + ln + y <= (size_t)AQ_STATIC_SCRATCH_BYTES;
        if (sc.blocked) map = map_b;
        sc.i8[0] = (int8_t*)base;
        sc.i8[1] = (int8_t*)(base + map);
        sc.ln_x = (float*)(base + 2 * map);
        sc.y = (float*)(base + 2 * map + ln);
    }
    return forward_int8_impl(p, d_obs, batch, d_actions, nullptr, nullptr, stream, &sc);
}

// The fp32 actor on explicit parameter arrays (d_ptrs: the same table in device memory, or NULL).  d_actions may be
// NULL (calibration only: the last layer is not run).  d_ranges_out, if given, receives the ranges; with `ready` it is
// host memory and *ready becomes `ticket` once they are there.
static aq_status forward_fp32_impl(aq_policy* p, const F32Ptrs& ptrs, const F32Ptrs* d_ptrs, const void* d_obs,
                                   int64_t batch, void* d_actions, float* d_ranges_out, uint32_t* ready, uint32_t ticket,
                                   hipStream_t st) {
    const int nl = p->net.n_layers;
    const int in_u8 = p->net.in_type == AQ_IN_U8;
    RangeSlot* const slots = d_ranges_out ? p->slots : nullptr;
    aq_status s = AQ_OK;
    if (slots) {
        if (p->slots_dirty) {
            s = launch_fill_u32((uint32_t*)slots, (int)(sizeof(RangeSlot) / 4) * kRangeSlots * AQ_MAX_LAYERS, 0u, st);
            if (s != AQ_OK) return s;
        }
        p->slots_dirty = true;
    }
    int rt = 1;
    if (fp32_mlp_fits(p->h_net, batch, &rt)) {
        s = launch_fp32_mlp(p->h_net, p->d_net, ptrs, d_ptrs, d_obs, batch, d_actions, slots, rt, st);
        if (s != AQ_OK) return s;
    } else {
        s = ensure_f32(p, batch, st);
        if (s != AQ_OK) return s;
        const int nc = f32_stack_layers(p, batch);
        if (nc) {
            s = launch_fp32_conv_stack(p->h_net, ptrs, d_obs, batch, p->act_f32[(nc - 1) & 1], slots, st);
            if (s != AQ_OK) return s;
        } else if (slots) {
            const LayerBuf& b0 = p->L[0];
            s = launch_input_range(d_obs, in_u8, batch * (int64_t)b0.d.in_h * b0.d.in_w * b0.d.in_c, slots, st);
            if (s != AQ_OK) return s;
        }
        for (int l = nc; l < nl; ++l) {
            const LayerBuf& b = p->L[l];
            const bool last = l == nl - 1;
            if (last && !d_actions) break;
            const bool ln = !last && b.d.act == AQ_ACT_LN_TANH, argmax = last && p->net.head == AQ_HEAD_ARGMAX;
            Fp32Layer L{};
            L.wpk = ptrs.wpk[l];
            L.zeros = p->f32_zeros;
            L.b = ptrs.b[l];
            L.K = b.K;
            L.N = b.N;
            L.relu = !last && b.d.act == AQ_ACT_RELU;
            L.head = last && !argmax ? p->net.head : -1;
            L.in_h = b.d.in_h;
            L.in_w = b.d.in_w;
            L.in_c = b.d.in_c;
            L.kh = b.d.kh;
            L.kw = b.d.kw;
            L.stride = b.d.stride;
            L.oh = b.oh;
            L.ow = b.ow;
            const int64_t rows_l = batch * b.oh * b.ow;
            const void* in = l == 0 ? d_obs : (const void*)p->act_f32[(l - 1) & 1];
            float* out = last && !argmax ? (float*)d_actions : p->act_f32[l & 1];
            RangeSlot* const sl = slots && !last ? slots + (l + 1) * kRangeSlots : nullptr;
            s = launch_fp32_layer(L, in, l == 0 ? in_u8 : 0, out, rows_l, ln ? nullptr : sl, st);
            if (s != AQ_OK) return s;
            if (ln) {
                s = launch_fp32_ln_tanh(out, rows_l, b.N, ptrs.gamma[l], ptrs.beta[l], p->net.ln_eps, sl, st);
                if (s != AQ_OK) return s;
            }
            if (argmax) {
                s = launch_fp32_argmax(out, rows_l, b.N, (int32_t*)d_actions, st);
                if (s != AQ_OK) return s;
            }
        }
    }
    if (slots) {
        s = launch_ranges_out(slots, nl, d_ranges_out, ready, ticket, st);
        if (s != AQ_OK) return s;
        p->slots_dirty = false;
    }
    return AQ_OK;
}

// the caller's arrays of per-layer pointers (the optional ones may be absent) as one table
static F32Ptrs f32_ptr_table(int nl, const float* const* w, const float* const* b, const float* const* gamma,
                             const float* const* beta) {
    F32Ptrs t{};
    for (int l = 0; l < nl; ++l) {
        t.w[l] = w[l];
        t.b[l] = b ? b[l] : nullptr;
        t.gamma[l] = gamma ? gamma[l] : nullptr;
        t.beta[l] = beta ? beta[l] : nullptr;
    }
    return t;
}

extern "C" aq_status aq_policy_forward_fp32_params(aq_policy* p, const float* const* h_d_w, const float* const* h_d_b,
                                                   const float* const* h_d_gamma, const float* const* h_d_beta,
                                                   const void* d_obs, int64_t batch, void* d_actions,
                                                   float* d_ranges_out, void* stream) {
    if (!p || !h_d_w || batch < 0) return AQ_EINVAL;
    if (batch == 0) return AQ_OK;
    if (!d_obs || !d_actions) return AQ_EINVAL;
    for (int l = 0; l < p->net.n_layers; ++l)
        if (!h_d_w[l]) return AQ_EINVAL;
    hipStream_t st = as_stream(stream);
    F32Ptrs ptrs = f32_ptr_table(p->net.n_layers, h_d_w, h_d_b, h_d_gamma, h_d_beta);
    aq_status s = ensure_f32_passed(p);
    if (s != AQ_OK) return s;
    s = launch_keep_params(ptrs, p->f32_passed.d_tab, p->f32_passed.slab, p->f32_passed.blocks, st);
    if (s != AQ_OK) return s;
    for (int l = 0; l < p->net.n_layers; ++l) {
        ptrs.wpk[l] = p->f32_passed.ptrs.wpk[l];
        ptrs.wsp[l] = p->f32_passed.ptrs.wsp[l];
    }
    return forward_fp32_impl(p, ptrs, nullptr, d_obs, batch, d_actions, d_ranges_out, nullptr, 0, st);
}

extern "C" aq_status aq_policy_set_params_fp32(aq_policy* p, const float* const* h_d_w, const float* const* h_d_b,
                                               const float* const* h_d_gamma, const float* const* h_d_beta,
                                               void* stream) {
    if (!p || !h_d_w) return AQ_EINVAL;
    const int nl = p->net.n_layers;
    for (int l = 0; l < nl; ++l)
        if (!h_d_w[l]) return AQ_EINVAL;
    hipStream_t st = as_stream(stream);
    aq_status s = ensure_f32_kept(p, st);
    if (s != AQ_OK) return s;
    // (absent biases, gains and offsets take their defaults 0, 1, 0)
    s = launch_keep_params(f32_ptr_table(nl, h_d_w, h_d_b, h_d_gamma, h_d_beta), p->f32_kept.d_tab,
                           p->f32_kept.slab, p->f32_kept.blocks, st);
    if (s != AQ_OK) return s;
    p->f32_ready = true;
    return AQ_OK;
}

extern "C" aq_status aq_policy_forward_fp32(aq_policy* p, const void* d_obs, int64_t batch, void* d_actions,
                                            void* stream) {
    if (!p || batch < 0) return AQ_EINVAL;
    if (!p->f32_ready) return AQ_ENOTQUANT;
    if (batch == 0) return AQ_OK;
    if (!d_obs || !d_actions) return AQ_EINVAL;
    return forward_fp32_impl(p, p->f32_kept.ptrs, p->f32_kept.d_ptrs, d_obs, batch, d_actions, nullptr, nullptr, 0, as_stream(stream));
}

extern "C" aq_status aq_calibrate_fp32(aq_policy* p, const void* d_obs, int64_t batch, aq_range* h_ranges_out,
                                       void* stream) {
    if (!p || !d_obs || !h_ranges_out || batch < 1) return AQ_EINVAL;
    if (!p->f32_ready) return AQ_ENOTQUANT;
    hipStream_t st = as_stream(stream);
    if (capturing(st)) return AQ_EINVAL;  // the call has to wait for its result
    const int nl = p->net.n_layers;
    // The ranges come back through host memory that the last kernel writes and this thread watches: a copy to pageable
    // memory and a stream synchronization cost 23 us, a third of a frame policy's whole calibration.
    if (!p->calib) {
        if (hip_failed(hipHostMalloc((void**)&p->calib, 64 + sizeof(float) * 2 * AQ_MAX_LAYERS, hipHostMallocDefault))) {
            p->calib = nullptr;
            return AQ_ENOMEM;
        }
        __atomic_store_n(p->calib, 0u, __ATOMIC_RELEASE);
    }
    void* d_calib = nullptr;
    AQ_HIP_CHECK(hipHostGetDevicePointer(&d_calib, p->calib, 0));
    if (++p->calib_ticket == 0) p->calib_ticket = 1;
    const uint32_t ticket = p->calib_ticket;
    const aq_status s = forward_fp32_impl(p, p->f32_kept.ptrs, p->f32_kept.d_ptrs, d_obs, batch, nullptr, (float*)((char*)d_calib + 64),
                                          (uint32_t*)d_calib, ticket, st);
    if (s != AQ_OK) return s;
    // (the stream is asked now and then: a failed one never sets the word)
    for (int64_t i = 1; __atomic_load_n(p->calib, __ATOMIC_ACQUIRE) != ticket; ++i) {
        if (i % 65536) {
            __builtin_ia32_pause();
            continue;
        }
        const hipError_t e = hipStreamQuery(st);
        if (hip_failed(e) && e == hipErrorNotReady) continue;
        if (e != hipSuccess || __atomic_load_n(p->calib, __ATOMIC_ACQUIRE) != ticket) return AQ_EHIP;
    }
    const float* h = (const float*)((const char*)p->calib + 64);
    for (int l = 0; l < nl; ++l) {
        h_ranges_out[l].lo = h[2 * l];
        h_ranges_out[l].hi = h[2 * l + 1];
    }
    return AQ_OK;
}

// ---- half-precision actor: storage of its parameters (one allocation, made once) and the tables over it
static aq_status ensure_h16(aq_policy* p, hipStream_t st) {
    if (p->h16_slab) return AQ_OK;
    if (capturing(st)) return AQ_ETOOBIG;
    const int nl = p->net.n_layers;
    size_t bytes = 0;
    auto take = [&](size_t n) {
        size_t off = bytes;
        bytes += (n + 255) / 256 * 256;
        return off;
    };
    std::vector<size_t> offs;
    bool fc = true;
    int cst = 0;
    std::vector<int> c_off;
    for (const LayerBuf& b : p->L) {
        offs.push_back(take((size_t)b.NT * (round_up(b.K, 64) / 16) * 1024));
        for (int i = 0; i < 3; ++i) offs.push_back(take((size_t)b.N_pad * 4));
        fc = fc && b.fc;
        c_off.push_back(cst);
        cst += b.N_pad * (b.d.act == AQ_ACT_LN_TANH ? 3 : 1);
    }
    struct {  // one copy
        Fp16Net net;
        Fp16ConvTab tab;
    } up{};
    const size_t off_h = take((size_t)cst * 2), off_up = take(sizeof(up));
    void* slab = nullptr;
    if (hip_failed(hipMalloc(&slab, bytes))) return AQ_ENOMEM;
    char* base = (char*)slab;
    Fp16Net& net = up.net;
    Fp16ConvTab& tab = up.tab;
    int blk = 0;
    net.n_layers = fc ? nl : 0;
    net.head = p->net.head;
    net.cst = cst;
    net.eps = p->net.ln_eps;
    net.consts = base + off_h;
    for (int l = 0; l < nl; ++l) {
        const LayerBuf& b = p->L[l];
        const int ks16 = round_up(b.K, 64) / 16;
        net.L[l] = Fp16LayerDev{base + offs[4 * l], b.K, b.N, ks16, b.NT, b.d.act, c_off[l]};
        for (int i = 0; i < 4; ++i) {
            const bool ln = b.d.act == AQ_ACT_LN_TANH;
            if (i >= 2 && !ln) continue;
            void* half = i == 0 ? nullptr : base + off_h + 2 * ((size_t)c_off[l] + (size_t)(i - 1) * b.N_pad);
            tab.blk0[tab.n] = blk;
            tab.e[tab.n++] = Fp16ConvTab::Entry{base + offs[4 * l + i], half, i, l, b.N, b.K, ks16, b.NT};
            blk += i == 0 ? (int)(((int64_t)b.NT * ks16 + kConvTiles - 1) / kConvTiles) : (b.N_pad + 255) / 256;
        }
    }
    tab.blocks = blk;
    if (hip_failed(hipMemcpy(base + off_up, &up, sizeof(up), hipMemcpyHostToDevice))) {
        (void)hipFree(slab);
        return AQ_EHIP;
    }
    for (int l = 0; l < nl; ++l) {
        p->h16_wp.push_back(base + offs[4 * l]);
        p->h16_bias.push_back((float*)(base + offs[4 * l + 1]));
        p->h16_gamma.push_back((float*)(base + offs[4 * l + 2]));
        p->h16_beta.push_back((float*)(base + offs[4 * l + 3]));
    }
    p->h16_slab = slab;
    p->h16_net = net;
    p->d_h16_net = (Fp16Net*)(base + off_up);
    p->d_h16_tab = (Fp16ConvTab*)(base + off_up + offsetof(decltype(up), tab));
    p->h16_blocks = blk;
    return AQ_OK;
}

extern "C" aq_status aq_convert_params_fp16(aq_policy* p, const float* const* h_d_w, const float* const* h_d_b,
                                            const float* const* h_d_gamma, const float* const* h_d_beta,
                                            void* stream) {
    if (!p || !h_d_w) return AQ_EINVAL;
    const int nl = p->net.n_layers;
    for (int l = 0; l < nl; ++l)
        if (!h_d_w[l]) return AQ_EINVAL;
    hipStream_t st = as_stream(stream);
    aq_status s = ensure_h16(p, st);
    if (s != AQ_OK) return s;
    int* st16 = p->status + 1;
    s = launch_fill_u32((uint32_t*)st16, 1, 0u, st);
    if (s != AQ_OK) return s;
    s = launch_fp16_convert(f32_ptr_table(nl, h_d_w, h_d_b, h_d_gamma, h_d_beta), p->d_h16_tab, p->h16_blocks, st16, st);
    if (s != AQ_OK) return s;
    p->h16_ready = true;
    return AQ_OK;
}

static void fp16_layers(const aq_policy* p, Fp16Layer* Ls) {
    const int nl = p->net.n_layers;
    for (int l = 0; l < nl; ++l) {
        const LayerBuf& b = p->L[l];
        const bool last = l == nl - 1;
        Fp16Layer L{};
        L.wp = p->h16_ready ? p->h16_wp[l] : nullptr;
        L.bias = p->h16_ready ? p->h16_bias[l] : nullptr;
        L.K = b.K;
        L.N = b.N;
        L.KS16 = round_up(b.K, 64) / 16;
        L.NT = b.NT;
        L.fc = b.fc;
        L.relu = !last && b.d.act == AQ_ACT_RELU;
        L.in_h = b.d.in_h;
        L.in_w = b.d.in_w;
        L.in_c = b.d.in_c;
        L.kh = b.d.kh;
        L.kw = b.d.kw;
        L.stride = b.d.stride;
        L.oh = b.oh;
        L.ow = b.ow;
        Ls[l] = L;
    }
}

extern "C" aq_status aq_policy_fp16_conv_stack_layers(const aq_policy* p, int32_t* n_layers) {
    if (!p || !n_layers) return AQ_EINVAL;
    Fp16Layer Ls[AQ_MAX_LAYERS];
    fp16_layers(p, Ls);
    *n_layers = p->conv_stack ? fp16_conv_stack_layers(Ls, p->net.n_layers, nullptr,
                                                       p->net.in_type == AQ_IN_U8 ? 2 : 1, 1)
                              : 0;
    return AQ_OK;
}

extern "C" aq_status aq_policy_forward_fp16(aq_policy* p, const void* d_obs, int64_t batch, void* d_actions,
                                            void* const* taps_out, void* stream) {
    if (!p || batch < 0) return AQ_EINVAL;
    if (!p->h16_ready) return AQ_ENOTQUANT;
    if (batch == 0) return AQ_OK;
    if (!d_obs || !d_actions) return AQ_EINVAL;
    hipStream_t st = as_stream(stream);
    if (fp16_mlp_rows(p->h16_net, batch))
        return launch_fp16_mlp(p->h16_net, p->d_h16_net, d_obs, p->h_net.in_u8, batch, d_actions, taps_out, st);
    aq_status s = ensure_f16(p, batch, st);
    if (s != AQ_OK) return s;
    const int nl = p->net.n_layers;
    const int in_mode0 = p->net.in_type == AQ_IN_U8 ? 2 : 1;
    Fp16Layer Ls[AQ_MAX_LAYERS];
    fp16_layers(p, Ls);
    // a frame policy's convolutions run as one launch where their shapes allow it (their maps then stay in
    // LDS, so a tap on any but the last of them takes the per-layer launches)
    int nc = p->conv_stack ? fp16_conv_stack_layers(Ls, nl, d_obs, in_mode0, batch) : 0;
    for (int l = 0; l + 1 < nc; ++l)
        if (taps_out && taps_out[l]) nc = 0;
    if (nc) {
        const LayerBuf& b = p->L[nc - 1];
        void* out = p->act_f16[(nc - 1) & 1];
        s = launch_fp16_conv_stack(Ls, nl, d_obs, in_mode0, batch, out, st);
        if (s != AQ_OK) return s;
        if (taps_out && taps_out[nc - 1])
            AQ_HIP_CHECK(hipMemcpyAsync(taps_out[nc - 1], out, (size_t)batch * b.oh * b.ow * b.N * 2,
                                        hipMemcpyDeviceToDevice, st));
    }
    int blocked = 0;
    for (int l = nc; l < nl; ++l) {
        const LayerBuf& b = p->L[l];
        const bool last = l == nl - 1;
        Fp16Layer L = Ls[l];
        const int64_t rows_l = batch * b.oh * b.ow;
        const void* in = l == 0 ? d_obs : (const void*)p->act_f16[(l - 1) & 1];
        void* out = p->act_f16[l & 1];
        // (the layer kernel writes actions in 16-byte pieces)
        const bool fused_head = last && p->net.head != AQ_HEAD_ARGMAX && ((uintptr_t)d_actions & 15) == 0;
        if (fused_head) {
            L.head_actions = (float*)d_actions;
            L.head_tanh = p->net.head == AQ_HEAD_TANH;
        }
        // an argmax policy whose logits fit one tile of the few-row kernel: the action index leaves the same launch
        const bool fused_argmax = last && p->net.head == AQ_HEAD_ARGMAX && L.NT == 1 &&
                                  fp16_layer_is_skinny(L, l == 0 ? in_mode0 : 0, rows_l);
        if (fused_argmax) L.head_argmax = (int32_t*)d_actions;
        // between two layers of the few-row kernel the activations lie in its operand order
        L.in_blocked = blocked;
        blocked = !last && b.d.act != AQ_ACT_LN_TANH && !(taps_out && taps_out[l]) && Ls[l + 1].fc &&
                  fp16_layer_is_skinny(L, l == 0 ? in_mode0 : 0, rows_l) && fp16_layer_is_skinny(Ls[l + 1], 0, rows_l);
        L.out_blocked = blocked;
        s = launch_layer_fp16(L, in, l == 0 ? in_mode0 : 0, out, rows_l, st);
        if (s != AQ_OK) return s;
        if (!last && b.d.act == AQ_ACT_LN_TANH) {
            s = launch_fp16_ln_tanh(out, rows_l, b.N, p->h16_gamma[l], p->h16_beta[l], p->net.ln_eps, st);
            if (s != AQ_OK) return s;
        }
        if (taps_out && taps_out[l])
            AQ_HIP_CHECK(hipMemcpyAsync(taps_out[l], out, (size_t)rows_l * b.N * 2, hipMemcpyDeviceToDevice, st));
        if (last && !fused_head && !fused_argmax) {
            s = launch_fp16_head(out, rows_l, b.N, p->net.head, d_actions, st);
            if (s != AQ_OK) return s;
        }
    }
    return AQ_OK;
}

// Host side of the whole-network int8 MLP kernels: decides whether a network fits the general one, picks its rows per workgroup,
// and hands each call to the kernel that takes its shape.
#include "fused_mlp.hpp"

namespace aq {

AQ_FUSED_DECL(1, 1, false, false, true);
AQ_FUSED_DECL(1, 1, false, true, true);
AQ_FUSED_DECL(1, 1, false, false, false);
AQ_FUSED_DECL(1, 1, false, true, false);
AQ_FUSED_DECL(2, 1, false, false, false);
AQ_FUSED_DECL(2, 1, false, true, false);
AQ_FUSED_DECL(4, 1, false, false, false);
AQ_FUSED_DECL(4, 1, false, true, false);
AQ_FUSED_DECL(1, 2, false, false, false);
AQ_FUSED_DECL(1, 2, false, true, false);
AQ_FUSED_DECL(2, 2, false, false, false);
AQ_FUSED_DECL(2, 2, false, true, false);
AQ_FUSED_DECL(1, 1, true, false, true);
AQ_FUSED_DECL(1, 1, true, true, true);
AQ_FUSED_DECL(1, 1, true, false, false);
AQ_FUSED_DECL(1, 1, true, true, false);
AQ_FUSED_DECL(2, 1, true, false, false);
AQ_FUSED_DECL(2, 1, true, true, false);
// hidden layers wider than 512: 16 rows per workgroup, and per-tensor weights
extern AQ_FUSED_INST(1, 2, false, false, true);
extern AQ_FUSED_INST(1, 2, false, true, true);
extern AQ_FUSED_INST(1, 2, true, false, true);
extern AQ_FUSED_INST(1, 2, true, true, true);
extern AQ_FUSED_INST(1, 2, true, false, false);
extern AQ_FUSED_INST(1, 2, true, true, false);
extern AQ_FUSED_INST(2, 2, true, false, false);
extern AQ_FUSED_INST(2, 2, true, true, false);

namespace {
struct Plan {
    int rt, nb, ld, off_red, off_sum, off_cst, off_y;
    size_t lds;
};

// LDS of a workgroup of 16 rt rows; false where the network is none of this kernel's.
bool layout(const NetDev& n, int rt, Plan* p) {
    int w = 0, nt = 0;
    const LayerDev& last = n.L[n.n_layers - 1];
    for (int l = 0; l < n.n_layers; ++l) {
        const LayerDev& L = n.L[l];
        if (L.kh != 1 || L.kw != 1 || L.in_h != 1 || L.in_w != 1 || L.NT * 32 > fused::IMAXN || L.K > fused::IMAXK) return false;
        const int k = (L.K + 63) & ~63;
        w = w > k ? w : k;
        if (l < n.n_layers - 1) nt = nt > L.NT ? nt : L.NT;
    }
    p->rt = rt;
    p->nb = nt > 2 * fused::IW ? 2 : 1;
    p->ld = w + 16;  // (16-byte reads of consecutive rows are 4 banks further each)
    size_t bytes = (size_t)16 * rt * p->ld;
    const size_t part = (size_t)fused::IW * rt * 1024;  // a narrow last layer's partial sums
    if (bytes < part) bytes = part;
    auto take = [&](size_t more) {
        const int at = (int)bytes;
        bytes += more;
        return at;
    };
    p->off_red = take((size_t)16 * rt * fused::IW * 8);
    p->off_sum = take(n.asym ? (size_t)2 * 16 * rt * 4 : 0);
    p->off_cst = take(2 * fused::INARROW * 4);
    p->off_y = take(n.head == AQ_HEAD_ARGMAX && last.N <= fused::INARROW ? (size_t)16 * rt * (fused::INARROW + 1) * 4 : 0);
    p->lds = bytes;
    return p->lds <= 160 * 1024;
}

// Rows per workgroup, by measurement (us at 16 / 32 / 64 / 128 rows; -: not measured, or no such variant).  More rows pass fewer weight
// bytes per row through the CU's vector memory path, fewer leave fewer CUs idle.
// Above 512 wide one workgroup fills a CU: 61-1024x3-40 at 4096 rows 27 / 30 / 42, at 8000 50 / 30 / 37, at 16379 97 / 58 / 41.
// Up to 512, where two of up to 64 rows share one: 61-512x3-17 at 8000 17.1 / 14.4 / 18.1, at 16384 - / 19.5 / 19.4 / 26.2, at 20000 - / 27.9 /
// 25.4 / 26.2, at 65536 - / 65.8 / 54.6 / 52.4; 200-512-256-17 at 16384 - / 12.5 / 17.7 / 21.1, at 20000 - / 19.2 / 21.9 / 21.3; 111-400-300-8 at
// 16379 16.7 / 10.9 / 14.5, at 24000 - / 17.0 / 18.6 / 17.6, at 65536 - / 37.8 / 37.7 / 34.4.  Between one and one and a half rounds of 32
// rows (16385 to 24576) 64 serve policies of 512 with a quarter of a million weights behind the first layer: 61-512x2-17 at 20000
// 19.9 (32) / 18.7, 256 inputs 22.9 / 23.2; 61-512-512-256-17 24.3 / 22.4; but 61-480x2-17 19.7 / 19.9, 256 inputs 22.8 / 25.2; 61-480x3-17
// 27.5 / 27.2, 256 inputs 30.9 / 32.0; with a LayerNorm 61-512x3-17 31.9 / 34.3; per-tensor 29.9 / 30.3.  128 rows are the best at whole rounds
// of 32768; a second round that is nearly empty loses to 32 rows (61-512x3-17 at 40000 - / 42.9 / 46.7 / 51.5).
// Per-tensor weights, which have no variant of 128 rows: 512x3 at 65536 - / 70.6 / 65.9; 111-400-300-8 at 65536 - / 42.2 / 41.4.
bool make_plan(const FwdArgs& a, Plan* p) {
    const NetDev& n = a.net;
    const int64_t b = a.c.batch;
    Plan q;
    if (!layout(n, 1, &q)) return false;
    int widest = 0, lns = 0;
    int64_t weights = 0;
    for (int l = 0; l < n.n_layers; ++l) {
        if (l > 0) weights += (int64_t)n.L[l].K * n.L[l].N;
        if (l == n.n_layers - 1) break;
        widest = widest > n.L[l].N ? widest : n.L[l].N;
        lns += n.L[l].act == AQ_ACT_LN_TANH;
    }
    int rt;
    if (b <= 16 * 256) rt = 1;
    else if (q.nb == 2) rt = b <= 32 * 256 ? 2 : 4;
    else if (b <= 32 * 768) rt = b > 32 * 512 && widest > 480 && weights > 250000 && !lns && !n.asym ? 4 : 2;
    else rt = !n.asym ? 8 : widest > 480 ? 4 : 2;
    while (rt > 1 && !layout(n, rt, &q)) rt /= 2;
    if (rt == 1) (void)layout(n, 1, &q);
    if (!grid_ok((b + 16 * rt - 1) / (16 * rt), fused::IT)) return false;
    *p = q;
    return true;
}
}  // namespace

bool any_taps(const FwdArgs& a) {
    if (!a.taps) return false;
    if (a.t.a0 || a.t.y) return true;
    for (int l = 0; l < a.net.n_layers; ++l)
        if (a.t.acc[l] || a.t.act[l] || a.t.ln[l]) return true;
    return false;
}

bool fused_mlp_supported(const FwdArgs& a, int* rows_out, int* tiles_out) {
    if (rows16_mlp_supported(a)) {  // (given a 16-byte aligned observation buffer; every such network also has a plan)
        *rows_out = 16 * rows16_mlp_row_tiles(a.c.batch);
        if (tiles_out) *tiles_out = 1;
        return true;
    }
    Plan p;
    if (!make_plan(a, &p)) return false;
    *rows_out = 16 * p.rt;
    if (tiles_out) *tiles_out = p.nb;
    return true;
}

int fused_mlp_kernel_kind(const FwdArgs& a) {
    if (rows16_mlp_supported(a)) return rows16_mlp_alone_on_cu(a.c.batch) ? 3 : 2;
    Plan p;
    int ld;
    if (!make_plan(a, &p)) return 0;
    if (p.nb == 2 && p.rt == 4 && wide_mlp_supported(a, &ld)) return 1;
    return 0;
}

aq_status launch_fused_mlp(const FwdArgs& a, hipStream_t st) {
    // 16-row workgroups on small networks: the kernel built for that case (asked first, before any planning: at
    // these sizes the call's host time is what a launch costs)
    const bool aligned = ((uintptr_t)a.c.obs & 15) == 0;
    if (aligned && rows16_mlp_supported(a)) return launch_rows16_mlp(a, st);
    Plan p;
    if (!make_plan(a, &p)) return AQ_ESHAPE;
    // 64-row workgroups on wide layers: the pipelined kernel where the shapes and the address allow it
    int wide_ld;
    if (aligned && p.nb == 2 && p.rt == 4 && wide_mlp_supported(a, &wide_ld)) return launch_wide_mlp(a, st);
    const fused::Call c{a.c.obs, a.c.actions, a.c.batch, a.c.ex_sigma, a.c.ex_k0, a.c.ex_k1, a.c.ex_s0, a.c.ex_s1,
                        p.ld, p.off_red, p.off_sum, p.off_cst, p.off_y};
    const bool taps = any_taps(a), as = a.net.asym != 0;
#define AQ_GO(MT, NB, AS, HF)                                                            \
    return taps ? launch_fused_t<MT, NB, AS, true, HF>(a.d_net, c, a.t, p.lds, st)       \
                : launch_fused_t<MT, NB, AS, false, HF>(a.d_net, c, a.t, p.lds, st)
#define AQ_GO_ROWS(NB, AS)                 \
    do {                                   \
        if (p.rt == 1) AQ_GO(1, NB, AS, true);  \
        if (p.rt == 2) AQ_GO(1, NB, AS, false); \
        if (p.rt == 4) AQ_GO(2, NB, AS, false); \
    } while (0)
    if (p.nb == 2) {
        if (as) AQ_GO_ROWS(2, true);
        else AQ_GO_ROWS(2, false);
        return AQ_ESHAPE;
    }
    if (as) {
        AQ_GO_ROWS(1, true);
        return AQ_ESHAPE;
    }
    AQ_GO_ROWS(1, false);
    AQ_GO(4, 1, false, false);
#undef AQ_GO_ROWS
#undef AQ_GO
}

}  // namespace aq

// The inference-system core (section "The inference system") on one GPU and its C interface.
//
// The paper's processes become: the segment broadcaster -> a host loop that hands every segment
// once to every member; a worker (batcher, predictor, prediction sender) -> an activation arena
// and the launches of a gang on one of the process's four streams (lanes), whose kernels write
// logits straight into the member's row block, so there is nothing to reassemble; the prediction
// accumulator -> one fused softmax-and-mean kernel behind every lane, of which the last to arrive
// for a row does the work (members in a fixed order).
#include "engine.h"

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>

#include "chain.h"
#include "planner.h"
#include "resident.h"
#include "seedgen.h"
#include "static_scratch.h"

using namespace ens;

#define HIP_TRY(expr)                                                                       \
    do {                                                                                    \
        hipError_t e_ = (expr);                                                             \
        if (e_ != hipSuccess) {                                                             \
            fprintf(stderr, "ens: %s failed: %s (%s:%d)\n", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
            return e_ == hipErrorOutOfMemory ? ENS_E_NOMEM : ENS_E_HIP;                     \
        }                                                                                   \
    } while (0)

namespace ens {

const char* conv_bf16_variant_name(const ConvArgs& a, int G);
bool conv_bneck_applicable(const ConvArgs& a1, const ConvArgs& a2, const ConvArgs& a3, int nb, int G);
const char* conv_bneck_name(const ConvArgs& a1);
hipError_t launch_conv_bneck(const ConvArgs& a1, const ConvArgs& a2, const ConvArgs& a3, const ConvArgs* argv, int G, int nb,
                             hipStream_t s);
bool conv_dense_applicable(const ConvArgs& a1, const ConvArgs& a2, int nb, int G);
bool conv_pw_applicable(const ConvArgs& a, int nb, int G);
bool conv_stempool_applicable(const ConvArgs& a, const ConvArgs& pool, int nb, int G);
const char* conv_stempool_name();
hipError_t launch_conv_stempool(const ConvArgs& a, const ConvArgs& pool, const ConvArgs* argv, int G, int nb, hipStream_t s);
const char* conv_dense_name();
hipError_t launch_conv_dense(const ConvArgs& a1, const ConvArgs& a2, const ConvArgs* argv, int G, int nb, hipStream_t s);

static int prof_class(ens_handle* h, const std::string& name) {
    for (size_t i = 0; i < h->prof.size(); i++)
        if (h->prof[i].name == name) return (int)i;
    h->prof.push_back(ProfClass{name});
    return (int)h->prof.size() - 1;
}

// Tensor 0 (the staged input) is shared by a gang: only the leader's copy is written.
static View view_of(const Worker& w, const Worker& leader, const Member& m, int t, int c0) {
    const Worker& src = t == 0 ? leader : w;
    View v;
    v.p = src.arena + src.layout.offset[t];
    v.stride = m.tensors[t].cs;
    v.c0 = c0;
    return v;
}

static bool same_network(const Member& a, const Member& b) {
    if (a.bf16 != b.bf16 || a.ops.size() != b.ops.size() || a.tensors.size() != b.tensors.size()) return false;
    for (size_t t = 0; t < a.tensors.size(); t++)
        if (a.tensors[t].h != b.tensors[t].h || a.tensors[t].w != b.tensors[t].w || a.tensors[t].c != b.tensors[t].c) return false;
    for (size_t i = 0; i < a.ops.size(); i++)
        if (memcmp(&a.ops[i].op, &b.ops[i].op, sizeof(ens_op)) != 0) return false;
    return true;
}

// Fills one member's argument block for operation `pl`; `L` receives kind, class and work.
// `images`: the batch size the launch is planned for (tile choices and names; work is counted at the worker's full batch).
// `sub`: which of the operation's pl.sub argument blocks (sub-convolutions of a grouped convolution)
static int fill_args(ens_handle* h, const Worker& w, const Worker& leader, int G, int images, const OpPlan& pl, Launch& L, int sub = 0) {
    const Member& m = h->members[w.member];
    const int es = m.bf16 ? 2 : 4;
    const ens_op& o = pl.op;
    const TensorInfo& ts = m.tensors[o.src];
    const TensorInfo& td = m.tensors[o.dst];
    const char* P = m.dev_params;
    const double nb = w.batch;
    switch (o.kind) {
        case ENS_OP_CONV: {
            L.kind = L_CONV;
            ConvArgs& a = L.conv;
            a.x = view_of(w, leader, m, o.src, o.src_c0);
            a.y = view_of(w, leader, m, o.dst, o.dst_c0);
            a.res.p = nullptr; a.res.stride = 0; a.res.c0 = 0;
            if (o.res >= 0) a.res = view_of(w, leader, m, o.res, o.res_c0);
            a.w = P + pl.w;
            a.bias = (const float*)(P + pl.b);
            a.scale = (const float*)(P + pl.scale);
            a.pre_scale = pl.pre_scale != SIZE_MAX ? (const float*)(P + pl.pre_scale) : nullptr;
            a.pre_shift = pl.pre_shift != SIZE_MAX ? (const float*)(P + pl.pre_shift) : nullptr;
            a.ws = nullptr; a.ws_floats = 0;
            a.gate = nullptr; a.gate_stride = 0;
            a.pair = 0;
            a.few = 2 * images <= w.batch;
            a.zeros = P + m.zeros_off;
            a.wpk = pl.w_packed != SIZE_MAX ? P + pl.w_packed : nullptr;
            if (w.layout.scratch_offset != SIZE_MAX) {
                a.ws = (float*)(w.arena + w.layout.scratch_offset);
                a.ws_floats = (long long)SPLIT_WS_FLOATS;
            }
            a.nb = images; a.H = ts.h; a.W = ts.w; a.cin = pl.cin_s; a.Ho = td.h; a.Wo = td.w; a.cout = pl.sub_cout;
            a.kh = o.kh; a.kw = o.kw; a.sh = o.sh; a.sw = o.sw; a.pt = o.pt; a.pl = o.pl; a.act = o.act;
            a.inv_hw = 1.0 / ((double)td.h * td.w); a.inv_w = 1.0 / (double)td.w;
            L.sub = pl.sub;
            if (pl.sub > 1) {                                    // this block's slice of channels, weights and bias
                a.x.c0 += sub * pl.cin_s;
                a.y.c0 += sub * pl.sub_cout;
                if (a.res.p) a.res.c0 += sub * pl.sub_cout;
                a.w = (const char*)a.w + (size_t)sub * pl.sub_cout * o.kh * o.kw * pl.cin_s * es;
                a.bias += (size_t)sub * pl.sub_cout;
                a.scale += (size_t)sub * pl.sub_cout;
            }
            const int groups = o.r > 1 ? o.r : 1;
            L.flop = 2.0 * nb * td.h * td.w * o.cout * (pl.alg_k > 0 ? pl.alg_k : o.kh * o.kw * o.cin / groups);
            L.bytes = nb * ((double)ts.h * ts.w * o.cin + (double)td.h * td.w * o.cout * (o.res >= 0 ? 2 : 1)) * es +
                      (double)o.kh * o.kw * o.cin / groups * o.cout * es;
            L.klass = prof_class(h, m.bf16 ? conv_bf16_variant_name(a, G * pl.sub) : "conv_f32_kernel");
            break;
        }
        case ENS_OP_DWCONV:
        case ENS_OP_MAXPOOL:
        case ENS_OP_AVGPOOL: {
            L.kind = o.kind == ENS_OP_DWCONV ? L_DWCONV : L_POOL;
            L.is_max = o.kind == ENS_OP_MAXPOOL;
            PoolArgs& a = L.pool;
            a.x = view_of(w, leader, m, o.src, o.src_c0);
            a.y = view_of(w, leader, m, o.dst, o.dst_c0);
            a.w = o.kind == ENS_OP_DWCONV ? P + pl.w : nullptr;
            a.bias = o.kind == ENS_OP_DWCONV ? (const float*)(P + pl.b) : nullptr;
            a.scale = o.kind == ENS_OP_DWCONV ? (const float*)(P + pl.scale) : nullptr;
            a.nb = images; a.H = ts.h; a.W = ts.w; a.c = o.cin; a.Ho = td.h; a.Wo = td.w;
            a.kh = o.kh; a.kw = o.kw; a.sh = o.sh; a.sw = o.sw; a.pt = o.pt; a.pl = o.pl;
            a.act = o.kind == ENS_OP_DWCONV ? o.act : ACT_NONE;  // a pool has none of its own
            a.sums = nullptr; a.sums_stride = 0;
            a.pre_scale = a.pre_shift = nullptr;
            L.flop = o.kind == ENS_OP_DWCONV ? 2.0 * nb * td.h * td.w * o.cin * o.kh * o.kw : 0.0;
            L.bytes = nb * ((double)ts.h * ts.w + (double)td.h * td.w) * o.cin * es;
            L.klass = prof_class(h, o.kind == ENS_OP_DWCONV ? "window_kernel<dwconv>"
                                    : L.is_max ? "window_kernel<maxpool>" : "window_kernel<avgpool>");
            break;
        }
        case ENS_OP_GAP: {
            L.kind = L_GAP;
            GapArgs& a = L.gap;
            a.x = view_of(w, leader, m, o.src, o.src_c0);
            a.y = (float*)(w.arena + w.layout.offset[o.dst]) + o.dst_c0;
            a.pre_scale = pl.pre_scale != SIZE_MAX ? (const float*)(P + pl.pre_scale) : nullptr;
            a.pre_shift = pl.pre_shift != SIZE_MAX ? (const float*)(P + pl.pre_shift) : nullptr;
            a.nb = images; a.HW = ts.h * ts.w; a.c = o.cin;
            if (td.c != o.cin) return ENS_E_UNSUPPORTED;         // the pooled vector is dense
            L.bytes = nb * (double)ts.h * ts.w * o.cin * es;
            L.klass = prof_class(h, "gap_kernel");
            break;
        }
        case ENS_OP_FC: {
            L.kind = L_FC;
            FcArgs& a = L.fc;
            a.x = (const float*)(w.arena + w.layout.offset[o.src]);
            a.w = P + pl.w;
            a.wpk = pl.w_packed != SIZE_MAX ? P + pl.w_packed : nullptr;
            a.bias = (const float*)(P + pl.b);
            a.y = h->d_logits[w.member];                         // rows of the whole request
            a.nb = images; a.cin = o.cin; a.cout = o.cout; a.ldy = o.cout;
            L.flop = 2.0 * nb * o.cin * o.cout;
            L.bytes = (double)o.cin * o.cout * es + nb * (o.cin + o.cout) * 4.0;
            L.klass = prof_class(h, m.bf16 && fc_mfma_applicable(a) ? "fc_mfma_bf16" : "fc_kernel");
            break;
        }
        case ENS_OP_SE: {
            L.kind = L_SE;
            SeArgs& a = L.se;
            a.x = view_of(w, leader, m, o.src, o.src_c0);
            a.y = view_of(w, leader, m, o.dst, o.dst_c0);
            a.w1 = (const float*)(P + pl.w); a.b1 = (const float*)(P + pl.b);
            a.w2 = (const float*)(P + pl.w2); a.b2 = (const float*)(P + pl.b2);
            a.scratch = (float*)(w.arena + w.layout.offset[pl.scratch]);
            a.nb = images; a.HW = ts.h * ts.w; a.c = o.cin; a.r = o.r;
            a.gate_only = 0;
            a.cap = pl.se_cap; a.have_sums = 0;
            L.flop = 4.0 * nb * o.cin * o.r;
            L.bytes = nb * 3.0 * ts.h * ts.w * o.cin * es;
            L.klass = prof_class(h, "se_kernels");
            break;
        }
        default:
            return ENS_E_INVALID;
    }
    return ENS_OK;
}

// Which operations of a gang's member run together, for batches of up to `images` images.
struct Fusions {
    bool few = false;              // the batches do not fill half of the worker's batch size
    std::vector<char> chain, fused, gated, summed, swapped;
    bool operator==(const Fusions& o) const {
        return few == o.few && chain == o.chain && fused == o.fused && gated == o.gated && summed == o.summed && swapped == o.swapped;
    }
};

// The pooled output of a stem in the convolution's argument form.
static ConvArgs pool_as_conv(ens_handle* h, const Worker& w, const OpPlan& pl, int images) {
    const Member& mw = h->members[w.member];
    ConvArgs p;
    memset(&p, 0, sizeof(p));
    p.y = view_of(w, w, mw, pl.op.dst, pl.op.dst_c0);
    p.Ho = mw.tensors[pl.op.dst].h;
    p.Wo = mw.tensors[pl.op.dst].w;
    p.nb = images;
    return p;
}

// Turns the arguments of a 1x1 convolution round: its input is the squeeze-excite block's, times the block's gates.
static void gate_args(ens_handle* h, const Worker& w, const Worker& leader, const OpPlan& se, ConvArgs& c) {
    const Member& mw = h->members[w.member];
    c.x = view_of(w, leader, mw, se.op.src, se.op.src_c0);
    c.gate = (const float*)(w.arena + w.layout.offset[se.scratch]) + se_gate_offset(se.op.cin, se.op.r, se.se_cap);
    c.gate_stride = se_scratch_floats(se.op.cin, se.op.r, se.se_cap);
}

static Fusions decide_fusions(ens_handle* h, Gang& g, int images) {
    const Worker& leader = h->workers[g.workers[0]];
    const Member& m = h->members[leader.member];
    const int G = (int)g.workers.size();
    Fusions F;
    F.few = 2 * images <= leader.batch;
    std::vector<char>&chain = F.chain, &fused = F.fused, &gated = F.gated, &summed = F.summed, &swapped = F.swapped;
    auto fill = [&](size_t i, Launch& L) { return fill_args(h, leader, leader, G, images, m.ops[i], L) == ENS_OK; };
    // Which bottlenecks run as one kernel: planned as such and within the kernel's shapes at this batch
    // size.  The tensors in between are then not written (not wanted when they are to be read back).
    chain.assign(m.ops.size(), 0);                               // 1: runs the next two operations too, 2: run by it
    for (size_t i = 0; i + 2 < m.ops.size(); i++) {
        if (!m.ops[i].fuse_chain || h->keeps) continue;
        Launch a, b, c;
        if (!fill(i, a) || !fill(i + 1, b) || !fill(i + 2, c)) continue;
        if (conv_bneck_applicable(a.conv, b.conv, c.conv, images, G)) {
            chain[i] = 1;
            chain[i + 1] = chain[i + 2] = 2;
        }
    }
    // Which layers of dense blocks run as one kernel: chain[] 3 marks the head (two operations), 2 the one it runs
    for (size_t i = 0; i + 1 < m.ops.size(); i++) {
        if (!m.ops[i].fuse_dense || h->keeps || chain[i] || chain[i + 1]) continue;
        Launch a, b;
        if (!fill(i, a) || !fill(i + 1, b)) continue;
        if (conv_dense_applicable(a.conv, b.conv, images, G)) {
            chain[i] = 3;
            chain[i + 1] = 2;
        }
    }
    // The stem and the max-pool behind it as one kernel: chain[] 4 marks the stem, 2 the pool it runs
    for (size_t i = 0; i + 1 < m.ops.size(); i++) {
        if (!m.ops[i].fuse_pool || h->keeps || chain[i] || chain[i + 1]) continue;
        Launch a;
        if (!fill(i, a)) continue;
        if (conv_stempool_applicable(a.conv, pool_as_conv(h, leader, m.ops[i + 1], images), images, G)) {
            chain[i] = 4;
            chain[i + 1] = 2;
        }
    }
    // Which pairs of convolutions run as one launch: planned as such, and both on the generic kernel or both on the one
    // for few pixels at this batch size (their workgroups read every field of their own argument block).
    fused.assign(m.ops.size(), 0);                               // 1: takes the next operation along, 2: taken along
    for (size_t i = 0; i + 1 < m.ops.size(); i++) {
        if (!m.ops[i].fuse_next || chain[i] || chain[i + 1]) continue;   // a bottleneck kernel takes precedence
        Launch a, b;
        if (!fill(i, a) || !fill(i + 1, b)) continue;
        auto both_on = [&](const char* kernel) {
            return strncmp(conv_bf16_variant_name(a.conv, 2 * G), kernel, strlen(kernel)) == 0 &&
                   strncmp(conv_bf16_variant_name(b.conv, 2 * G), kernel, strlen(kernel)) == 0;
        };
        a.conv.wpk = b.conv.wpk = nullptr;                       // the 1x1 kernel runs no pairs
        bool pair = both_on("conv_igemm_bf16");
        a.conv.pair = b.conv.pair = 1;
        if (pair || both_on("conv_small_bf16")) {
            fused[i] = 1;
            fused[i + 1] = 2;
        }
    }
    // Squeeze-excite blocks that stop at the gates, which the 1x1 convolution behind them applies to its
    // input: gated[] 1 marks the block, 2 the convolution.
    gated.assign(m.ops.size(), 0);
    for (size_t i = 0; i + 1 < m.ops.size(); i++) {
        if (!m.ops[i].fuse_gate || h->keeps || chain[i] || chain[i + 1] || fused[i] || fused[i + 1]) continue;
        Launch c;
        if (!fill(i + 1, c)) continue;
        gate_args(h, leader, leader, m.ops[i], c.conv);
        if (c.conv.wpk && conv_pw_applicable(c.conv, images, G)) {
            gated[i] = 1;
            gated[i + 1] = 2;
        }
    }
    // Depthwise convolutions whose kernel leaves the channel sums for the squeeze-excite block behind them:
    // summed[] 1 marks the convolution, 2 the block.
    summed.assign(m.ops.size(), 0);
    for (size_t i = 0; i + 1 < m.ops.size(); i++) {
        if (!m.ops[i].fuse_sums || h->keeps || m.ops[i + 1].op.kind != ENS_OP_SE) continue;
        Launch d;
        if (!fill(i, d)) continue;
        if (dwconv_sums_applicable(d.pool, m.bf16) && dwconv_sums_blocks(d.pool.Ho, d.pool.Wo, d.pool.c) <= m.ops[i + 1].se_cap) {
            summed[i] = 1;
            summed[i + 1] = 2;
        }
    }
    // Average pools that change places with the 1x1 convolution behind them: swapped[] 1 marks the pool's place
    // (the convolution runs there), 2 the convolution's (the pool runs there, on the convolution's channels).
    swapped.assign(m.ops.size(), 0);
    for (size_t i = 0; i + 1 < m.ops.size(); i++) {
        if (!m.ops[i].swap_pool || h->keeps || chain[i] || chain[i + 1] || fused[i] || fused[i + 1] || gated[i + 1]) continue;
        swapped[i] = 1;
        swapped[i + 1] = 2;
    }
    // ... and pre-activated 1x1 convolutions that let the 2x2 average pool behind them go first: 3 marks the
    // convolution's place (the pool runs there, on the convolution's input), 4 the pool's (the convolution, on the pooled map)
    for (size_t i = 0; i + 1 < m.ops.size(); i++) {
        if (!m.ops[i].swap_conv || h->keeps || chain[i] || chain[i + 1] || fused[i] || fused[i + 1] || gated[i] || swapped[i] ||
            swapped[i + 1])
            continue;
        swapped[i] = 3;
        swapped[i + 1] = 4;
    }
    return F;
}

constexpr size_t ARG_SLOT = 512;                                 // bytes reserved per argument block
static_assert(sizeof(ConvArgs) <= ARG_SLOT && sizeof(PoolArgs) <= ARG_SLOT && sizeof(SeArgs) <= ARG_SLOT, "argument block");

// The launches of a gang for batches of up to `images` images, their argument blocks appended to `blocks`; d_argv holds
// offsets into `blocks` until the caller knows where they are on the device.
static int build_plan(ens_handle* h, Gang& g, int images, const Fusions& F, std::vector<Launch>& launches, std::vector<char>& blocks) {
    const Worker& leader = h->workers[g.workers[0]];
    const Member& m = h->members[leader.member];
    const int G = (int)g.workers.size();
    const size_t slot = ARG_SLOT;
    const std::vector<char>&chain = F.chain, &fused = F.fused, &gated = F.gated, &summed = F.summed, &swapped = F.swapped;
    std::vector<size_t> first_blk(m.ops.size() + 1, 0);          // argument blocks: G * sub per operation
    for (size_t i = 0; i < m.ops.size(); i++)
        first_blk[i + 1] = first_blk[i] + (fused[i] == 2 || chain[i] == 2 ? 0
                                           : (size_t)G * (chain[i] == 1 ? 3 : chain[i] == 3 || chain[i] == 4 || fused[i] == 1 ? 2 : (m.ops[i].sub > 1 ? m.ops[i].sub : 1)));
    const size_t n_blk = first_blk[m.ops.size()];
    std::vector<char> host(n_blk * slot, 0);
    const size_t at = blocks.size();
    launches.clear();
    for (size_t i = 0; i < m.ops.size(); i++) {
        Launch L;
        if (fused[i] == 2 || chain[i] == 2) {                    // its argument blocks are in an earlier launch
            L.kind = L_SKIP;
            launches.push_back(L);
            continue;
        }
        if (chain[i] == 4) {                                     // stem and pool: G blocks of the convolution, then G of the pooled output
            for (int k = G - 1; k >= 0; k--) {
                const Worker& wk = h->workers[g.workers[k]];
                const Member& mk = h->members[wk.member];
                const ConvArgs p = pool_as_conv(h, wk, mk.ops[i + 1], images);
                const int rc = fill_args(h, wk, leader, G, images, mk.ops[i], L);
                if (rc != ENS_OK) return rc;
                L.conv.ws = nullptr;
                L.conv.ws_floats = 0;
                if (k == 0) L.conv2 = p;
                memcpy(host.data() + (first_blk[i] + (size_t)k) * slot, &L.conv, sizeof(ConvArgs));
                memcpy(host.data() + (first_blk[i] + (size_t)G + k) * slot, &p, sizeof(ConvArgs));
            }
            // algorithmic bytes: the image once, the pooled map once, the filter
            L.bytes = (double)leader.batch * ((double)L.conv.H * L.conv.W * L.conv.cin + (double)L.conv2.Ho * L.conv2.Wo * L.conv.cout) * 2.0 +
                      2.0 * L.conv.kh * L.conv.kw * L.conv.cin * L.conv.cout;
            L.kind = L_STEMPOOL;
            L.sub = 2;
            L.klass = prof_class(h, conv_stempool_name());
            L.d_argv = (const void*)(at + first_blk[i] * slot);
            launches.push_back(L);
            continue;
        }
        if (chain[i] == 3) {                                     // a layer of a dense block: G blocks of each of its two convolutions
            double flop = 0, bytes = 0;
            for (int sub = 1; sub >= 0; sub--)
                for (int k = G - 1; k >= 0; k--) {
                    const Member& mk = h->members[h->workers[g.workers[k]].member];
                    const int rc = fill_args(h, h->workers[g.workers[k]], leader, G, images, mk.ops[i + sub], L);
                    if (rc != ENS_OK) return rc;
                    L.conv.ws = nullptr;
                    L.conv.ws_floats = 0;
                    if (k == 0) {
                        flop += L.flop;
                        if (sub == 1) {                          // algorithmic bytes: the block's input and weights, the appended channels
                            L.conv2 = L.conv;
                            bytes += (double)leader.batch * L.conv.H * L.conv.W * L.conv.cout * 2.0 + 2.0 * 9 * L.conv.cin * L.conv.cout;
                        } else {
                            bytes += (double)leader.batch * L.conv.H * L.conv.W * L.conv.cin * 2.0 + 2.0 * L.conv.cin * L.conv.cout;
                        }
                    }
                    memcpy(host.data() + (first_blk[i] + (size_t)sub * G + k) * slot, &L.conv, sizeof(ConvArgs));
                }
            L.kind = L_DENSE;
            L.sub = 2;
            L.flop = flop;
            L.bytes = bytes;
            L.klass = prof_class(h, conv_dense_name());
            L.d_argv = (const void*)(at + first_blk[i] * slot);
            launches.push_back(L);
            continue;
        }
        if (chain[i] == 1) {                                     // G blocks of each of the three convolutions
            double flop = 0, wbytes = 0;
            for (int sub = 2; sub >= 0; sub--)
                for (int k = G - 1; k >= 0; k--) {
                    const Member& mk = h->members[h->workers[g.workers[k]].member];
                    const int rc = fill_args(h, h->workers[g.workers[k]], leader, G, images, mk.ops[i + sub], L);
                    if (rc != ENS_OK) return rc;
                    L.conv.ws = nullptr;
                    L.conv.ws_floats = 0;
                    if (k == 0) {
                        flop += L.flop;
                        wbytes += 2.0 * L.conv.kh * L.conv.kw * L.conv.cin * L.conv.cout;
                        if (sub == 2) L.conv3 = L.conv;
                        if (sub == 1) L.conv2 = L.conv;
                    }
                    memcpy(host.data() + (first_blk[i] + (size_t)sub * G + k) * slot, &L.conv, sizeof(ConvArgs));
                }
            // algorithmic bytes of the block: input once (it is the residual too, unless that is another tensor), output, weights
            const double px = (double)leader.batch * L.conv.H * L.conv.W;
            const bool own_res = L.conv3.res.p && L.conv3.res.p != L.conv.x.p;
            L.kind = L_BNECK;
            L.sub = 3;
            L.flop = flop;
            L.bytes = px * 2.0 * (L.conv.cin + L.conv3.cout * (own_res ? 2 : 1)) + wbytes;
            L.klass = prof_class(h, conv_bneck_name(L.conv));
            L.d_argv = (const void*)(at + first_blk[i] * slot);
            launches.push_back(L);
            continue;
        }
        const int nsub = fused[i] == 1 ? 2 : (m.ops[i].sub > 1 ? m.ops[i].sub : 1);
        // the one with more output channels leads (the grid is sized for the first argument block), the
        // deeper of two equals (so is the tile shape)
        const bool second_leads = fused[i] == 1 &&
            (m.ops[i + 1].sub_cout > m.ops[i].sub_cout ||
             (m.ops[i + 1].sub_cout == m.ops[i].sub_cout &&
              m.ops[i + 1].op.kh * m.ops[i + 1].op.kw * m.ops[i + 1].cin_s > m.ops[i].op.kh * m.ops[i].op.kw * m.ops[i].cin_s));
        double flop2 = 0, bytes2 = 0;
        for (int sub = nsub - 1; sub >= 0; sub--)
            for (int k = G - 1; k >= 0; k--) {                   // (k, sub) == (0, 0) last: L keeps the leader's first block
                const Member& mk = h->members[h->workers[g.workers[k]].member];
                const OpPlan& pl = swapped[i] == 1 || swapped[i] == 3 ? mk.ops[i + 1] : swapped[i] == 2 || swapped[i] == 4 ? mk.ops[i - 1]
                                   : fused[i] == 1 && (sub == 1) != second_leads ? mk.ops[i + 1] : mk.ops[i];
                const int rc = fill_args(h, h->workers[g.workers[k]], leader, G, images, pl, L, fused[i] == 1 ? 0 : sub);
                if (rc != ENS_OK) return rc;
                if (swapped[i] >= 3) {
                    // the pool first: pre-activation and average of the convolution's input into the convolution's output
                    // memory, as many channels wide as that input; then the convolution over the pooled map, nothing in front
                    const Worker& wk = h->workers[g.workers[k]];
                    const OpPlan& c = swapped[i] == 3 ? mk.ops[i] : mk.ops[i - 1];
                    const OpPlan& q = swapped[i] == 3 ? mk.ops[i + 1] : mk.ops[i];
                    const TensorInfo &tx = mk.tensors[c.op.src], &tq = mk.tensors[q.op.dst];
                    View mid;
                    mid.p = wk.arena + wk.layout.offset[c.op.dst];
                    mid.stride = c.op.cin;
                    mid.c0 = 0;
                    const char* P = mk.dev_params;
                    if (swapped[i] == 3) {
                        L.pool.x = view_of(wk, leader, mk, c.op.src, c.op.src_c0);
                        L.pool.y = mid;
                        L.pool.c = c.op.cin;
                        L.pool.H = tx.h; L.pool.W = tx.w;
                        L.pool.pre_scale = (const float*)(P + c.pre_scale);
                        L.pool.pre_shift = (const float*)(P + c.pre_shift);
                        L.bytes = (double)wk.batch * ((double)tx.h * tx.w + (double)tq.h * tq.w) * c.op.cin * 2.0;
                        L.klass = prof_class(h, "window_kernel<avgpool,pre>");
                    } else {
                        L.conv.x = mid;
                        L.conv.y = view_of(wk, leader, mk, q.op.dst, q.op.dst_c0);
                        L.conv.pre_scale = L.conv.pre_shift = nullptr;
                        L.conv.H = L.conv.Ho = tq.h; L.conv.W = L.conv.Wo = tq.w;
                        L.conv.inv_hw = 1.0 / ((double)tq.h * tq.w); L.conv.inv_w = 1.0 / (double)tq.w;
                        L.flop = 2.0 * wk.batch * tq.h * tq.w * (double)c.op.cout * c.op.cin;
                        L.bytes = (double)wk.batch * tq.h * tq.w * (c.op.cin + c.op.cout) * 2.0 + (double)c.op.cin * c.op.cout * 2.0;
                        L.klass = prof_class(h, conv_bf16_variant_name(L.conv, G));
                    }
                } else if (swapped[i]) {
                    // the convolution first: from the pool's input into the pool's output memory, as many channels wide
                    // as the convolution has, batch-norm but no activation; then the pool over that, with the activation
                    const Worker& wk = h->workers[g.workers[k]];
                    const OpPlan& q = swapped[i] == 1 ? mk.ops[i] : mk.ops[i - 1];
                    const OpPlan& c = swapped[i] == 1 ? mk.ops[i + 1] : mk.ops[i];
                    View mid;
                    mid.p = wk.arena + wk.layout.offset[q.op.dst];
                    mid.stride = c.op.cout;
                    mid.c0 = 0;
                    const double px = (double)wk.batch * mk.tensors[q.op.dst].h * mk.tensors[q.op.dst].w;
                    if (swapped[i] == 1) {
                        L.conv.x = view_of(wk, leader, mk, q.op.src, q.op.src_c0);
                        L.conv.y = mid;
                        L.conv.act = ACT_NONE;
                        L.klass = prof_class(h, conv_bf16_variant_name(L.conv, G));
                    } else {
                        L.pool.x = mid;
                        L.pool.y = view_of(wk, leader, mk, c.op.dst, c.op.dst_c0);
                        L.pool.c = c.op.cout;
                        L.pool.act = c.op.act;
                        L.bytes = px * c.op.cout * 2.0 * 2.0;
                        L.klass = prof_class(h, "window_kernel<avgpool,act>");
                    }
                }
                const double se_pass = L.bytes / 3.0;            // squeeze-excite: the tensor is read twice and written once
                if (summed[i] == 1) {                            // the sums go to the scratch of the block behind
                    const Worker& wk = h->workers[g.workers[k]];
                    const OpPlan& se = mk.ops[i + 1];
                    L.pool.sums = (float*)(wk.arena + wk.layout.offset[se.scratch]);
                    L.pool.sums_stride = se_scratch_floats(se.op.cin, se.op.r, se.se_cap);
                    L.klass = prof_class(h, "window_kernel<dwconv,sums>");
                } else if (summed[i] == 2) {                     // one pass over the input less
                    L.se.have_sums = dwconv_sums_blocks(mk.tensors[pl.op.src].h, mk.tensors[pl.op.src].w, pl.op.cin);
                    L.bytes -= se_pass;
                }
                if (gated[i] == 1) {                             // the block stops at the gates: one pass over its input
                    L.se.gate_only = 1;
                    L.bytes -= 2.0 * se_pass;
                    if (summed[i] == 2) L.bytes = (double)L.se.nb * L.se.have_sums * L.se.c * sizeof(float);   // only the rows of sums
                } else if (gated[i] == 2) {
                    gate_args(h, h->workers[g.workers[k]], leader, mk.ops[i - 1], L.conv);
                    L.klass = prof_class(h, conv_bf16_variant_name(L.conv, G));
                }
                if (fused[i] == 1) {                             // no split of the depth: the two would share one workspace
                    L.conv.pair = 1;                             // a kernel that can run both
                    L.conv.ws = nullptr;
                    L.conv.ws_floats = 0;
                    if (sub == 1) { flop2 = L.flop; bytes2 = L.bytes; }
                }
                char* dst = host.data() + (first_blk[i] + (size_t)sub * G + k) * slot;
                switch (L.kind) {
                    case L_CONV: memcpy(dst, &L.conv, sizeof(ConvArgs)); break;
                    case L_DWCONV:
                    case L_POOL: memcpy(dst, &L.pool, sizeof(PoolArgs)); break;
                    case L_GAP: memcpy(dst, &L.gap, sizeof(GapArgs)); break;
                    case L_FC: memcpy(dst, &L.fc, sizeof(FcArgs)); break;
                    case L_SE: memcpy(dst, &L.se, sizeof(SeArgs)); break;
                    default: break;
                }
            }
        if (fused[i] == 1) {
            L.sub = 2;
            L.flop += flop2;
            L.bytes += bytes2;
            L.klass = prof_class(h, conv_bf16_variant_name(L.conv, 2 * G));
        }
        L.d_argv = (const void*)(at + first_blk[i] * slot);
        launches.push_back(L);
    }
    // The device arrays are indexed by element size, so every block is re-packed densely.
    for (size_t i = 0; i < m.ops.size(); i++) {
        const Launch& L = launches[i];
        size_t sz = 0;
        switch (L.kind) {
            case L_CONV:
            case L_BNECK:
            case L_DENSE:
            case L_STEMPOOL: sz = sizeof(ConvArgs); break;
            case L_DWCONV:
            case L_POOL: sz = sizeof(PoolArgs); break;
            case L_GAP: sz = sizeof(GapArgs); break;
            case L_FC: sz = sizeof(FcArgs); break;
            case L_SE: sz = sizeof(SeArgs); break;
            default: break;
        }
        char* base = host.data() + first_blk[i] * slot;
        const size_t nb_i = first_blk[i + 1] - first_blk[i];
        for (size_t k = 1; k < nb_i; k++) memmove(base + k * sz, base + k * slot, sz);
    }
    blocks.insert(blocks.end(), host.begin(), host.end());
    return ENS_OK;
}

// Translates the gang's operations into kernel argument arrays in device memory, once for every range of batch sizes with
// fusions of its own: a request smaller than a worker's batch size runs the layers as its own size wants them.  Ranges end at
// powers of two, at half the worker's batch size and at the whole.
// may_alloc false: the device block of the gang must already be large enough (it is once the
// allocation has been installed); the function then only rewrites it.
static int build_launches(ens_handle* h, Gang& g, bool may_alloc = true) {
    const Worker& leader = h->workers[g.workers[0]];
    const Member& m = h->members[leader.member];
    std::vector<std::pair<int, Fusions>> ranges;
    for (int images = 1;; images *= 2) {
        const int most = 2 * images < leader.batch ? images : ranges.empty() || ranges.back().first < leader.batch / 2 ? std::max(1, leader.batch / 2) : leader.batch;
        Fusions F = decide_fusions(h, g, most);
        if (!ranges.empty() && ranges.back().second == F) ranges.back().first = most;
        else ranges.emplace_back(most, std::move(F));
        if (most == leader.batch) break;
    }
    g.plans.assign(ranges.size(), GangPlan());
    std::vector<char> blocks;
    for (size_t i = 0; i < ranges.size(); i++) {
        g.plans[i].most = ranges[i].first;
        const int rc = build_plan(h, g, ranges[i].first, ranges[i].second, g.plans[i].launches, blocks);
        if (rc != ENS_OK) return rc;
    }
    if (!may_alloc && (!g.d_args || g.d_args_bytes < blocks.size())) return ENS_E_INVALID;
    if (g.d_args && g.d_args_bytes < blocks.size()) { (void)hipFree(g.d_args); g.d_args = nullptr; }
    if (!g.d_args) { HIP_TRY(hipMalloc((void**)&g.d_args, blocks.size())); g.d_args_bytes = blocks.size(); }
    for (GangPlan& p : g.plans)
        for (Launch& L : p.launches) L.d_argv = g.d_args + (size_t)L.d_argv;
    g.stage.src = nullptr;                                       // named per request
    g.stage.slot = nullptr;
    g.stage.dst = leader.arena + leader.layout.offset[0];
    g.stage.nb = leader.batch; g.stage.sh = h->base_h; g.stage.sw = h->base_w;
    g.stage.dh = m.in_h; g.stage.dw = m.in_w; g.stage.dc = m.tensors[0].cs; g.stage.s2d = m.stem_s2d ? 1 : 0;
    // (not on the null stream, which would wait for the lanes of every handle)
    HIP_TRY(hipMemcpyAsync(g.d_args, blocks.data(), blocks.size(), hipMemcpyHostToDevice, h->main_stream));
    HIP_TRY(hipStreamSynchronize(h->main_stream));
    g.stale = false;
    return ENS_OK;
}

static int ensure_buffers(ens_handle* h, int64_t n);

// The last replay may have been waited for on the flag alone (see wait_lanes): the runtime is done with it when its lanes are synchronised.
static void destroy_graph(ens_handle* h, RequestGraph& r) {
    for (int l = 0; l < r.lanes; l++)
        if (r.exec[l]) (void)hipStreamSynchronize(h->lanes[l]);
    for (hipGraphExec_t& e : r.exec) {
        if (e) (void)hipGraphExecDestroy(e);
        e = nullptr;
    }
}

// Recorded requests hold launch geometry, argument block addresses, the batches' sizes and the addresses of the library's own logits
// buffers.  What the argument blocks name may change beneath them and back: a request that runs on the fixed device array leaves
// them as they are, and the next one of ens_predict has the blocks of its gangs rewritten before it replays one.
static void drop_graphs(ens_handle* h) {
    for (RequestGraph& r : h->graphs) destroy_graph(h, r);
    h->graphs.clear();
    h->sizes_seen.clear();
}

// A small request that is answered through pinned host memory ends in finish_kernel on every lane, and the last one to arrive
// writes the request's number there too.  Waiting for that instead of for the streams saves 10 us and more per lane.
// A request that takes longer than the spin is waited for the ordinary way, and so is one in SYNC_EVERY, which lets the runtime
// give back what it holds for finished launches.  (Not for answers on the device: the caller's next synchronisation of a stream of its
// own would pay for that, 0.6 us per launch.)
constexpr double SPIN_S = 5e-3;
constexpr uint64_t SYNC_EVERY = 64;

static hipError_t wait_lanes(ens_handle* h) {
    if (h->flagged && h->requests % SYNC_EVERY) {
        const auto t0 = std::chrono::steady_clock::now();
        for (unsigned i = 1;; i++) {
            if (__atomic_load_n(h->flag, __ATOMIC_ACQUIRE) == (uint32_t)h->requests) return hipSuccess;
            __builtin_ia32_pause();
            if (i % 64 == 0 && std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() > SPIN_S) break;
        }
    }
    for (int l = 0; l < h->lanes_used; l++) {
        const hipError_t e = hipStreamSynchronize(h->lanes[l]);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

static void drop_chains(ens_handle* h) {
    h->chains.clear();
    if (h->d_chain) (void)hipFree(h->d_chain);
    h->d_chain = nullptr;
    h->chain_bytes = 0;
    h->chain_plans.clear();
    for (Worker& w : h->workers) w.last_programs.clear();
}

static void drop_residents(ens_handle* h) {
    h->residents.clear();
    if (h->d_resident) (void)hipFree(h->d_resident);
    h->d_resident = nullptr;
    h->resident_bytes = 0;
}

static void destroy_workers(ens_handle* h) {
    h->flagged = false;                                          // the streams themselves
    (void)wait_lanes(h);
    drop_graphs(h);
    for (Gang& g : h->gangs)
        if (g.d_args) (void)hipFree(g.d_args);
    h->gangs.clear();
    h->own_gangs = 0;
    for (Worker& w : h->workers)
        if (w.arena) (void)hipFree(w.arena);
    h->workers.clear();
    drop_chains(h);
    drop_residents(h);
    h->have_alloc = false;
}

static int64_t alloc_bytes(const ens_handle* h, const ens_alloc& a) {
    int64_t total = 0;
    for (const Member& m : h->members) total += (int64_t)m.weight_bytes();
    for (int r = 0; r < a.rows; r++)
        for (int c = 0; c < a.cols; c++)
            if (a.batch[r][c] > 0) total += (int64_t)plan_arena(h->members[c], a.batch[r][c], h->keep_tensors).bytes;
    return total;
}

// What a launch counts on of the chip: its gang's share.  (Of the gangs at most LANES run at once, and the copies of a single gang do so
// too: the share that a launch has can be twice this, or a quarter.  The kernels' thresholds were measured with this number.)
static int stream_share(const ens_handle* h) {
    const int streams = std::max(1, h->own_gangs);
    return std::max(32, 256 / streams);
}

static int64_t copy_bytes(const ens_handle* h) {
    int64_t total = 0;
    for (const Worker& w : h->workers)
        if (w.copy) total += (int64_t)std::max<size_t>(w.arena_bytes, 256);
    return total;
}

// Gives the copies up, and the recorded requests, which run on them, and the chains.
static void drop_copies(ens_handle* h) {
    h->flagged = false;                                          // the streams themselves
    (void)wait_lanes(h);
    drop_graphs(h);
    h->alloc.bytes -= copy_bytes(h) + h->chain_bytes;
    drop_chains(h);
    while ((int)h->gangs.size() > h->own_gangs) {
        if (h->gangs.back().d_args) (void)hipFree(h->gangs.back().d_args);
        h->gangs.pop_back();
    }
    while (!h->workers.empty() && h->workers.back().copy) {
        (void)hipFree(h->workers.back().arena);
        h->workers.pop_back();
    }
    for (size_t i = 0; i < h->gangs.size(); i++) h->gangs[i].copies.assign(1, (int)i);
    (void)hipGetLastError();
}

// fn, which allocates device memory; once more without the copies and the recorded requests if there is not enough of it, and once more
// without the members in LDS, which are much faster than their launches and take a few hundred KB.
template <typename F>
static int with_room(ens_handle* h, F&& fn) {
    int rc = fn();
    if (rc != ENS_E_NOMEM) return rc;
    (void)hipGetLastError();
    if ((int)h->gangs.size() > h->own_gangs || !h->graphs.empty() || !h->chains.empty()) {
        drop_copies(h);
        rc = fn();
        if (rc != ENS_E_NOMEM) return rc;
        (void)hipGetLastError();
    }
    if (h->residents.empty()) return rc;
    h->flagged = false;
    (void)wait_lanes(h);
    h->alloc.bytes -= h->resident_bytes;
    drop_residents(h);
    rc = fn();
    if (rc == ENS_E_NOMEM) (void)hipGetLastError();
    return rc;
}

// Copies of the gangs (see Gang): LANES - 1 of a single gang, one each of two; of three or four, which have lanes enough, one of
// those with batches of up to 64 images (see takes_turns).  They are an extra: no more than a quarter of the memory that is free,
// nothing that a budget does not have room for beside the workers and the request buffers, none while every tensor is kept for
// inspection; and they go when something else finds no memory (with_room).
static int copy_gangs(ens_handle* h, int64_t need) {
    const int own = h->own_gangs;
    if (own > LANES || h->keep_tensors) return ENS_OK;
    std::vector<int> copies(own);
    size_t extra = 0, free_bytes = 0, total = 0;
    for (int i = 0; i < own; i++) {
        copies[i] = own == 1 ? LANES - 1 : own == 2 || h->workers[h->gangs[i].workers[0]].batch <= 64 ? 1 : 0;
        for (int wi : h->gangs[i].workers) extra += copies[i] * std::max<size_t>(h->workers[wi].arena_bytes, 256);
    }
    if (hipMemGetInfo(&free_bytes, &total) != hipSuccess || extra > free_bytes / 4) { (void)hipGetLastError(); return ENS_OK; }
    if (h->budget && (uint64_t)need + extra + (uint64_t)h->reserve > h->budget) return ENS_OK;
    for (int k = 0; k < LANES - 1; k++)
        for (int i = 0; i < own; i++) {
            if (k >= copies[i]) continue;
            Gang g = h->gangs[i];
            g.copy = true;
            g.copies.clear();
            g.d_args = nullptr;
            g.d_args_bytes = 0;
            const size_t had = h->workers.size();
            for (int& wi : g.workers) {
                Worker w = h->workers[wi];
                w.copy = true;
                w.gang = (int)h->gangs.size();
                w.arena = nullptr;
                if (hipMalloc((void**)&w.arena, std::max<size_t>(w.arena_bytes, 256)) != hipSuccess) {
                    (void)hipGetLastError();
                    for (size_t j = had; j < h->workers.size(); j++) (void)hipFree(h->workers[j].arena);
                    h->workers.resize(had);
                    return ENS_OK;
                }
                wi = (int)h->workers.size();
                h->workers.push_back(w);
            }
            h->gangs[i].copies.push_back((int)h->gangs.size());
            h->gangs.push_back(g);
            const int rc = build_launches(h, h->gangs.back());
            if (rc != ENS_OK) return rc;
        }
    return ENS_OK;
}

// The members' chains, for requests of a few images (run_chains).  For ensembles of deep bf16 members: a chain saves a launch per layer,
// and one of a few layers has little to save.  They run in the arenas of the members' first workers; a matrix whose workers of one member
// differ in batch size is left alone, since which of them takes a batch is what it is about (hand_out).
constexpr size_t CHAIN_MIN_OPS = 16;

static void install_chains(ens_handle* h, int64_t need) {
    std::vector<Chain> chains(h->members.size());
    h->chains_off = false;
    if (h->keeps || !h->gangs_enabled || h->planning) return;
    for (const Worker& w : h->workers)
        for (const Worker& u : h->workers)
            if (u.member == w.member && u.batch != w.batch) return;
    size_t steps = 0;
    std::vector<size_t> at;
    for (size_t c = 0; c < h->members.size(); c++) {
        const Member& m = h->members[c];
        if (!m.bf16 || m.ops.size() < CHAIN_MIN_OPS) return;
        const Worker* own = nullptr;
        for (const Worker& w : h->workers)
            if (w.member == (int)c && w.rank == 0 && !w.copy) own = &w;
        if (!own) return;
        Worker w = *own;                                         // its tensors apart, and every operation for itself
        w.layout = plan_arena(m, 1, true);
        w.batch = 1;
        const size_t arena_bytes = own->arena_bytes;
        const int batch = own->batch;
        char* const arena = own->arena;
        Fusions F;
        F.chain.assign(m.ops.size(), 0);
        F.fused = F.gated = F.summed = F.swapped = F.chain;
        for (size_t i = 0; i + 1 < m.ops.size(); i++)
            if (!F.swapped[i] && (m.ops[i].swap_pool || m.ops[i].swap_conv)) {
                F.swapped[i] = m.ops[i].swap_pool ? 1 : 3;
                F.swapped[i + 1] = m.ops[i].swap_pool ? 2 : 4;
            }
        Gang g;
        g.workers.push_back((int)h->workers.size());
        std::vector<Launch> launches;
        std::vector<char> blocks;
        const std::vector<size_t> places = w.layout.offset;
        h->workers.push_back(w);
        const int rc = build_plan(h, g, 1, F, launches, blocks);
        h->workers.pop_back();
        if (rc != ENS_OK || !build_chain(m, launches, arena, places, arena_bytes, batch, &chains[c])) return;
        at.push_back(steps);
        steps += chains[c].steps.size();
    }
    // the steps, and behind them the weights that are not in operand order elsewhere
    size_t bytes = steps * sizeof(ChainStep);
    for (const Chain& c : chains) bytes += c.pack_bytes;
    size_t free_bytes = 0, total = 0;
    if (hipMemGetInfo(&free_bytes, &total) != hipSuccess || bytes > free_bytes / 4) { (void)hipGetLastError(); return; }
    if (h->budget && (uint64_t)need + bytes + (uint64_t)h->reserve > h->budget) return;
    if (hipMalloc((void**)&h->d_chain, bytes) != hipSuccess) { h->d_chain = nullptr; (void)hipGetLastError(); return; }
    bool ok = true;
    char* packed = (char*)(h->d_chain + steps);
    for (size_t c = 0; c < chains.size() && ok; c++) {
        for (const Chain::Pack& p : chains[c].packs) {
            ChainStep& s = chains[c].steps[p.step];
            ok = ok && launch_chain_pack(s.w, packed + p.at, p.groups, p.rows, p.K, h->main_stream) == hipSuccess;
            for (ChainStep& q : chains[c].steps)
                for (int k = 0; k < 2; k++)
                    if (q.ahead[k] == s.w) q.ahead[k] = packed + p.at;
            s.w = packed + p.at;
        }
        packed += chains[c].pack_bytes;
        ok = ok && hipMemcpyAsync(h->d_chain + at[c], chains[c].steps.data(), chains[c].steps.size() * sizeof(ChainStep), hipMemcpyHostToDevice, h->main_stream) == hipSuccess;
    }
    ok = hipStreamSynchronize(h->main_stream) == hipSuccess && ok;
    if (!ok) {
        (void)hipGetLastError();
        (void)hipFree(h->d_chain);
        h->d_chain = nullptr;
        return;
    }
    h->chain_bytes = (int64_t)bytes;
    h->chain_at = at;
    h->chains = std::move(chains);
}

// The members in LDS, when all of them are small fp32 networks.
static void install_residents(ens_handle* h, int64_t need) {
    if (h->keeps || h->planning || h->members.size() > RESIDENT_MAX_MEMBERS) return;
    std::vector<Resident> all(h->members.size());
    std::vector<size_t> at;
    std::vector<float> fixed;
    for (size_t c = 0; c < h->members.size(); c++) {
        for (const Worker& w : h->workers)
            if (w.member == (int)c && w.rank == 0 && !w.copy && !build_resident(h->members[c], &all[c])) return;
        at.push_back(fixed.size());
        fixed.insert(fixed.end(), all[c].fixed.begin(), all[c].fixed.end());
    }
    const size_t queue = fixed.size();                           // zeros: the words that a launch's workgroups draw images by
    fixed.resize(fixed.size() + RESIDENT_MAX_MEMBERS + 1, 0.f);
    if (h->budget && (uint64_t)need + fixed.size() * sizeof(float) + (uint64_t)h->reserve > h->budget) return;
    if (hipMalloc((void**)&h->d_resident, fixed.size() * sizeof(float)) != hipSuccess) { h->d_resident = nullptr; (void)hipGetLastError(); return; }
    if (hipMemcpyAsync(h->d_resident, fixed.data(), fixed.size() * sizeof(float), hipMemcpyHostToDevice, h->main_stream) != hipSuccess ||
        hipStreamSynchronize(h->main_stream) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(h->d_resident);
        h->d_resident = nullptr;
        return;
    }
    h->resident_bytes = (int64_t)(fixed.size() * sizeof(float));
    h->resident_at = at;
    h->resident_queue = (unsigned*)(h->d_resident + queue);
    h->residents = std::move(all);
}

static int install_alloc(ens_handle* h, const ens_alloc& a, int segment_size) {
    const int M = (int)h->members.size();
    if (a.rows <= 0 || a.rows > ENS_MAX_SLOTS || a.cols != M) return ENS_E_INVALID;
    int max_batch = 0;
    for (int c = 0; c < M; c++) {
        bool any = false;
        for (int r = 0; r < a.rows; r++) {
            if (a.batch[r][c] < 0) return ENS_E_INVALID;
            any = any || a.batch[r][c] > 0;
            max_batch = std::max(max_batch, a.batch[r][c]);
        }
        if (!any) return ENS_E_INVALID;                          // a column of zeros is illegal
    }
    if (segment_size <= 0) segment_size = 128;
    segment_size = std::max(segment_size, max_batch);           // segment >= the largest batch size
    const int64_t need = alloc_bytes(h, a);
    if (h->budget && (uint64_t)need > h->budget) return ENS_E_NOMEM;
    destroy_workers(h);
    for (int r = 0; r < a.rows; r++)
        for (int c = 0; c < M; c++) {
            if (a.batch[r][c] == 0) continue;
            Worker w;
            w.member = c; w.batch = a.batch[r][c]; w.slot = r;
            w.layout = plan_arena(h->members[c], w.batch, h->keep_tensors);
            w.arena_bytes = w.layout.bytes;
            h->workers.push_back(w);
        }
    for (Worker& w : h->workers) {                               // rank among the member's workers
        w.rank = 0; w.of = 0;
        for (const Worker& u : h->workers)
            if (u.member == w.member) { if (u.slot < w.slot) w.rank++; w.of++; }
    }
    for (Worker& w : h->workers) {
        hipError_t e = hipMalloc((void**)&w.arena, std::max<size_t>(w.arena_bytes, 256));
        if (e != hipSuccess) {
            (void)hipGetLastError();
            destroy_workers(h);
            return e == hipErrorOutOfMemory ? ENS_E_NOMEM : ENS_E_HIP;
        }
    }
    // gangs: same row, same network shape and the same column of the matrix (hence the same batch size
    // here, the same fellow workers and so the same share of the segments)
    auto same_column = [&](int c1, int c2) {
        for (int r = 0; r < a.rows; r++)
            if (a.batch[r][c1] != a.batch[r][c2]) return false;
        return true;
    };
    for (size_t i = 0; i < h->workers.size(); i++) {
        Worker& w = h->workers[i];
        for (size_t gi = 0; gi < h->gangs.size() && w.gang < 0 && h->gangs_enabled; gi++) {
            const Worker& l = h->workers[h->gangs[gi].workers[0]];
            if (l.slot == w.slot && same_column(l.member, w.member) && same_network(h->members[l.member], h->members[w.member])) {
                w.gang = (int)gi;
                h->gangs[gi].workers.push_back((int)i);
            }
        }
        if (w.gang < 0) {
            Gang g;
            g.workers.push_back((int)i);
            g.rank = w.rank; g.of = w.of;
            w.gang = (int)h->gangs.size();
            g.copies.push_back(w.gang);
            h->gangs.push_back(g);
        }
    }
    h->own_gangs = (int)h->gangs.size();
    if (!h->d_logits.empty() && !h->d_logits[0]) {               // argument blocks hold the logits pointers
        const int rc0 = ensure_buffers(h, 1);
        if (rc0 != ENS_OK) { destroy_workers(h); return rc0; }
    }
    cu_budget() = stream_share(h);
    lanes_busy() = lanes_in_use() = std::min(LANES, std::max(1, h->own_gangs));
    h->keeps = h->keep_tensors;
    for (Gang& g : h->gangs) {
        const int rc = build_launches(h, g);
        if (rc != ENS_OK) { destroy_workers(h); return rc; }
    }
    h->args_stale = false;
    h->alloc = a;
    h->alloc.bytes = need;
    if (copy_gangs(h, need) != ENS_OK) drop_copies(h);
    install_chains(h, need + copy_bytes(h));                     // (what large requests gain from goes first where room is scarce)
    install_residents(h, need + copy_bytes(h) + h->chain_bytes);
    h->alloc.bytes = need + copy_bytes(h) + h->chain_bytes + h->resident_bytes;
    h->segment_size = segment_size;
    h->have_alloc = true;
    return ENS_OK;
}

static hipEvent_t take_event(ens_handle* h) {
    if (!h->event_pool.empty()) {
        hipEvent_t e = h->event_pool.back();
        h->event_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

static hipError_t issue(const Launch& L, bool bf16, int G, int nb, long long first, hipStream_t s) {
    switch (L.kind) {
        case L_CONV: return bf16 ? launch_conv_bf16(L.conv, (const ConvArgs*)L.d_argv, G * L.sub, nb, s)
                                 : launch_conv_f32(L.conv, (const ConvArgs*)L.d_argv, G * L.sub, nb, s);
        case L_DWCONV: return launch_dwconv(L.pool, (const PoolArgs*)L.d_argv, G, nb, bf16, s);
        case L_POOL: return launch_pool(L.pool, (const PoolArgs*)L.d_argv, G, nb, L.is_max, bf16, s);
        case L_GAP: return launch_gap(L.gap, (const GapArgs*)L.d_argv, G, nb, bf16, s);
        case L_FC: return launch_fc(L.fc, (const FcArgs*)L.d_argv, G, nb, first, bf16, s);
        case L_SE: return launch_se(L.se, (const SeArgs*)L.d_argv, G, nb, bf16, s);
        case L_BNECK: return launch_conv_bneck(L.conv, L.conv2, L.conv3, (const ConvArgs*)L.d_argv, G, nb, s);
        case L_DENSE: return launch_conv_dense(L.conv, L.conv2, (const ConvArgs*)L.d_argv, G, nb, s);
        case L_STEMPOOL: return launch_conv_stempool(L.conv, L.conv2, (const ConvArgs*)L.d_argv, G, nb, s);
        case L_SKIP: return hipSuccess;
    }
    return hipErrorInvalidValue;
}

static void note_batch(ens_handle* h, const Gang& g, int64_t first, int nb) {
    for (int wi : g.workers) {
        Worker& w = h->workers[wi];
        w.last_nb = nb;
        w.input_only = false;
        w.last_programs.clear();
        w.last_request = h->requests;
        w.last_first = first;
    }
}

// One batch of one gang: stage the images into the leader's arena, run every member, write the
// logits rows of the batch.
// The images are at `src`, or where `slot` says when the launches are being recorded.
static int forward_batch(ens_handle* h, Gang& g, int64_t first, int nb, const float* src, const RequestSlot* slot, hipStream_t st) {
    const Worker& leader = h->workers[g.workers[0]];
    const Member& m = h->members[leader.member];
    const int G = (int)g.workers.size();
    const double scale = (double)nb / leader.batch;
    auto timed = [&](int klass, double flop, double bytes, auto&& fn) -> hipError_t {
        if (!h->profiling) return fn();
        ProfRec r{klass, take_event(h), take_event(h), flop * scale, bytes * scale};
        if (!r.start || !r.stop) return hipErrorOutOfMemory;
        next_launch_events() = LaunchEvents{r.start, r.stop};    // stamped with the kernels' own begin and end
        const hipError_t e = fn();
        next_launch_events() = LaunchEvents{};
        h->prof_recs.push_back(r);
        return e;
    };
    if (h->fake_predictor) {                                     // zeros for the rows of this batch, nothing else
        for (int wi : g.workers) {
            const Worker& w = h->workers[wi];
            HIP_TRY(launch_fill_zero(h->d_logits[w.member] + first * h->classes, (int64_t)nb * h->classes, st));
        }
        note_batch(h, g, first, nb);
        return ENS_OK;
    }
    const double stage_bytes = (double)leader.batch * (h->base_h * h->base_w * 12.0 + (double)m.tensors[0].h * m.tensors[0].w * g.stage.dc * (m.bf16 ? 2 : 4));
    g.stage.src = src;
    g.stage.slot = slot;
    g.stage.sh = h->base_h; g.stage.sw = h->base_w;
    HIP_TRY(timed(h->stage_klass, 0.0, stage_bytes, [&] { return launch_stage(g.stage, nb, first, m.bf16, st); }));
    for (const Launch& L : g.plan_for(nb).launches) {
        if (L.kind == L_SKIP) continue;
        HIP_TRY(timed(L.klass, L.flop * G, L.bytes * G, [&] { return issue(L, m.bf16, G, nb, first, st); }));
    }
    note_batch(h, g, first, nb);
    return ENS_OK;
}

static int ensure_buffers(ens_handle* h, int64_t n) {
    const size_t rows = (size_t)n;
    bool moved = false;
    if (rows > h->d_logits_heap_rows) {
        for (float*& p : h->d_logits_heap) {
            if (p) (void)hipFree(p);
            p = nullptr;
        }
        h->d_logits_heap.assign(h->members.size(), nullptr);
        h->d_logits_heap_rows = 0;
        for (size_t m = 0; m < h->members.size(); m++)
            HIP_TRY(hipMalloc((void**)&h->d_logits_heap[m], rows * h->members[m].classes * sizeof(float)));
        h->d_logits_heap_rows = rows;
        moved = true;
        drop_graphs(h);                                        // they end in a combination of the old ones
    }
    if (moved || h->logits_static) {                           // (back) to the library's own buffers
        h->d_logits = h->d_logits_heap;
        h->d_logits_rows = h->d_logits_heap_rows;
        h->logits_static = false;
        h->args_stale = true;                                  // the FC argument blocks name these buffers
    }
    return ENS_OK;
}

// Points the per-member logits at slices of the fixed device array: behind its reserved head one block of
// `rows` x classes floats per member.  Allocates nothing.
static int use_static_logits(ens_handle* h, int64_t n) {
    void* base = nullptr;
    size_t bytes = 0;
    HIP_TRY(static_scratch(&base, &bytes));
    const size_t M = h->members.size();
    const size_t row_bytes = M * (size_t)h->classes * sizeof(float);
    const size_t rows_cap = (bytes - STATIC_SCRATCH_TABLE_BYTES) / row_bytes;
    if ((size_t)n > rows_cap) {
        fprintf(stderr, "ens_predict_static: %lld images x %zu members x %d classes of fp32 logits exceed the %zu-byte "
                "static scratch (at most %zu images for this ensemble)\n", (long long)n, M, h->classes, bytes, rows_cap);
        return ENS_E_TOOBIG;
    }
    float* first = (float*)((char*)base + STATIC_SCRATCH_TABLE_BYTES);
    const bool there = h->logits_static && !h->d_logits.empty() && h->d_logits[0] == first;
    if (!there) {
        h->d_logits.assign(M, nullptr);
        for (size_t m = 0; m < M; m++) h->d_logits[m] = first + m * rows_cap * (size_t)h->classes;
        h->d_logits_rows = rows_cap;
        h->logits_static = true;
        h->args_stale = true;                                  // the FC argument blocks name these buffers
    }
    return ENS_OK;
}

static int grow(float** p, size_t* cap, size_t want_floats) {
    if (want_floats <= *cap) return ENS_OK;
    if (*p) (void)hipFree(*p);
    *p = nullptr;
    *cap = 0;
    HIP_TRY(hipMalloc((void**)p, want_floats * sizeof(float)));
    *cap = want_floats;
    return ENS_OK;
}

// Does a gang with `batches` batches in a request share them with its copies?  One or two gangs always: 512 images through a
// ResNet-50 in batches of 128, 64 and 32 8.7 -> 7.4, 10.4 -> 7.7 and 12.6 -> 8.9 ms.  Three or four from four batches on: four members,
// 256 images in batches of 64, 32 and 16 16.2 -> 15.5, 20.7 -> 18.2 and 28.9 -> 23.4 ms; with two batches each (100 images,
// batches of 64) the lanes were loaded less evenly than by one gang each, 10.1 -> 10.5 ms, and with batches of 128 images three lanes
// fill the GPU: 38.5 -> 39.1 ms.
static bool takes_turns(const ens_handle* h, const Gang& g, int64_t batches) {
    return !h->one_stream && g.copies.size() > 1 && (h->own_gangs <= 2 || batches >= 4);
}

// Calls fn(gang, first image, images) for every batch of a request of n images, in the order of issue.  A gang's copies take its
// batches in turn.
template <typename F>
static int each_batch(ens_handle* h, int64_t n, uint64_t mask, const std::vector<std::vector<int32_t>>& owner, F&& fn) {
    const int seg = h->segment_size;
    const int64_t n_seg = (n + seg - 1) / seg;
    std::vector<size_t> turn(h->own_gangs, 0);
    for (int64_t s = 0; s < n_seg; s++) {
        const int64_t start = s * seg, end = std::min<int64_t>((s + 1) * seg, n);
        for (int i = 0; i < h->own_gangs; i++) {
            Gang& g = h->gangs[i];
            const int member0 = h->workers[g.workers[0]].member;
            if (g.of > 1 && owner[member0][s] != g.rank) continue;
            bool wanted = false;
            for (int wi : g.workers) wanted = wanted || ((mask >> h->workers[wi].member) & 1);
            if (!wanted) continue;
            const int b = h->workers[g.workers[0]].batch;
            const bool turns = takes_turns(h, g, (n + b - 1) / b / g.of);
            for (int64_t a = start; a < end; a += b) {
                Gang& taker = turns ? h->gangs[g.copies[turn[i]++ % g.copies.size()]] : g;
                const int rc = fn(taker, a, (int)std::min<int64_t>(b, end - a));
                if (rc != ENS_OK) return rc;
            }
        }
    }
    return ENS_OK;
}

// Requests recorded as graphs (see below): the launches of a request that is still recorded, recorded requests and noted sizes that
// a handle keeps, and requests from one recording that takes another's place to the next (see worth_recording); below three lanes the GPU takes as long for a launch as the host.  Average launch of the
// requests that are handed out batch by batch instead.  What a graph costs the host per kernel in it, and what
// it costs to start and to wait for one lane more (a graph's launch 30 us, a wait 10 to 20).
constexpr int64_t GRAPH_MAX_LAUNCHES = 2048;
constexpr size_t GRAPHS_KEPT = 16, SIZES_KEPT = 32;
constexpr uint64_t RECORD_EVERY = 32;
constexpr int GRAPH_MIN_LANES = 3;
constexpr double HAND_OUT_LAUNCH_S = 9e-6, LANE_S = 30e-6, GRAPH_NODE_S = 0.4e-6;

// What a launch takes whatever its batch (one image, other lanes busy): most are a chain of two or three round trips to memory.
static double launch_floor(int kind) {
    switch (kind) {
        case L_SE: return 12e-6;
        case L_DWCONV: return 9e-6;
        case L_BNECK: return 25e-6;
        case L_DENSE: return 17e-6;
        case L_STEMPOOL: return 20e-6;
        default: return 7e-6;
    }
}

// What a launch of a large batch takes: its work at the rates the kernels reach (measured alone on batches of 128).
static double launch_work(const Launch& L, double share) {
    double tflops = 6e14, gbs = 3.1e12;
    switch (L.kind) {
        case L_CONV: tflops = L.conv.kh * L.conv.kw > 1 && L.conv.sh == 1 ? 8e14 : 5.5e14; break;
        case L_DENSE: tflops = 2.8e14; break;
        case L_BNECK: tflops = 5.6e14; break;
        case L_STEMPOOL: tflops = 2.5e14; break;
        case L_DWCONV: gbs = 2.7e12; break;
        case L_SE: gbs = 1e12; break;
        default: break;
    }
    return share * std::max(L.flop / tflops, L.bytes / gbs);
}

static double batch_estimate(ens_handle* h, const Gang& g, int nb) {
    const double share = (double)nb / h->workers[g.workers[0]].batch * (double)g.workers.size();
    double t = launch_floor(L_POOL);                             // input staging
    for (const Launch& L : g.plan_for(nb).launches)
        if (L.kind != L_SKIP) t += std::max(launch_floor(L.kind), launch_work(L, share));
    return t;
}

// What a request comes to: its batches per gang, its launches and their estimated time one after the other.
struct Batch { int64_t first; int nb; double estimate; };
struct Work {
    std::vector<std::vector<Batch>> batches;
    std::vector<double> estimate;                                // per gang
    int64_t launches = 0, most = 0;                              // most: batches of the gang that has the most of them
    double total = 0;
};
static Work plan_work(ens_handle* h, int64_t n, uint64_t mask, const std::vector<std::vector<int32_t>>& owner) {
    Work w;
    w.batches.resize(h->gangs.size());
    w.estimate.assign(h->gangs.size(), 0.0);
    (void)each_batch(h, n, mask, owner, [&](Gang& g, int64_t first, int nb) {
        const size_t i = &g - h->gangs.data();
        std::vector<Batch>& all = w.batches[i];
        const double t = !all.empty() && all.back().nb == nb ? all.back().estimate : batch_estimate(h, g, nb);
        all.push_back(Batch{first, nb, t});
        for (const Launch& L : g.plan_for(nb).launches) w.launches += L.kind != L_SKIP;
        w.launches++;
        w.estimate[i] += t;
        w.total += t;
        w.most = std::max<int64_t>(w.most, (int64_t)all.size());
        return ENS_OK;
    });
    return w;
}

// Deals the gangs to the lanes: the longest first, each to the lane with the least so far.  The host
// reaches a lane after it has issued those before it, which counts as load, and a lane more costs what LANE_S says.
// Returns the number of lanes in use.
static int deal_lanes(ens_handle* h, const Work& work) {
    const std::vector<double>& est = work.estimate;
    std::vector<int> order(h->gangs.size());
    for (size_t i = 0; i < order.size(); i++) order[i] = (int)i;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return est[x] > est[y]; });
    double load[LANES] = {0};
    for (int l = 0; l < LANES; l++) load[l] = l * (LANE_S + (work.launches <= GRAPH_MAX_LAUNCHES ? work.launches / LANES * GRAPH_NODE_S : 0.0));
    int used = 0;
    for (int i : order) {
        if (est[i] == 0.0) continue;
        int best = 0;
        for (int l = 1; l < LANES; l++)
            if (load[l] < load[best]) best = l;
        if (h->one_stream) best = 0;
        h->gangs[i].lane = best;
        load[best] += est[i];
        used = std::max(used, best + 1);                        // lanes fill from the first on
    }
    return used;
}

static CombineArgs combine_args(ens_handle* h, int64_t n, int lanes) {
    CombineArgs a;
    memset(&a, 0, sizeof(a));
    for (size_t m = 0; m < h->members.size(); m++) a.logits[m] = h->d_logits[m];
    a.weights = h->d_weights;
    a.arrivals = h->d_arrivals;
    a.lanes = lanes;
    a.n_members = (int)h->members.size();
    a.classes = h->classes;
    a.rule = h->combine_rule;
    a.n = n;
    return a;
}

// ---- requests recorded as graphs ------------------------------------------------------------------
// Issuing a launch costs the host 2.7 us, so a small request through many layers waits for the host: one image through
// twelve members is 940 launches.  A request of a size that comes again is recorded, one graph of plain kernel launches in a row
// per lane, and from then on costs 0.2 to 0.5 us per launch.  (One graph over all the lanes with its forks and joins was
// measured too: 2.2 us per launch.)  Recording takes 3 us per launch and is done the second time a size is seen; the recorded
// launches find the request's buffers through a slot per lane.  Requests with more launches than this keep the GPU
// busy for longer than the host needs to issue them.

static RequestGraph* find_graph(ens_handle* h, int64_t n) {
    for (RequestGraph& r : h->graphs)
        if (r.n == n) return &r;
    return nullptr;
}

static RequestGraph* oldest_graph(ens_handle* h) {
    return &*std::min_element(h->graphs.begin(), h->graphs.end(), [](const RequestGraph& x, const RequestGraph& y) { return x.used < y.used; });
}

// Is a request of this size to be recorded?  When it comes again, while there is room.  After that only if it came last time since the
// recorded size that would make room for it was used, and once in RECORD_EVERY requests: a front end with more sizes than
// are kept would otherwise pay for a recording (3 us a launch, as much as issuing it) with most of its requests and see it given up
// before it is replayed.  (One to 12 and one to 24 images in turn through twelve members: 5.7 and 6.8 ms a request with each size
// recorded again whenever it came, 4.1 and 5.2 ms now; 5.6 and 6.3 ms launch by launch on a stream per gang.)  Sixteen of them hold some 13 MB of device memory there.  Notes that the size has come.
static bool worth_recording(ens_handle* h, int64_t n) {
    for (SeenSize& s : h->sizes_seen)
        if (s.n == n) {
            const uint64_t before = s.when;
            s.when = h->requests;
            if (s.failed) return false;
            return h->graphs.size() < GRAPHS_KEPT || (before > oldest_graph(h)->used && h->requests - h->last_recorded >= RECORD_EVERY);
        }
    if (h->sizes_seen.size() >= SIZES_KEPT)
        h->sizes_seen.erase(std::min_element(h->sizes_seen.begin(), h->sizes_seen.end(), [](auto& x, auto& y) { return x.when < y.when; }));
    h->sizes_seen.push_back(SeenSize{n, h->requests, false});
    return false;
}

// Records the request on the handle's own stream; nothing runs.  Failure leaves no graph: the request is then issued launch by launch,
// and so are those of its size that follow.
static RequestGraph* record_request(ens_handle* h, int64_t n, int lanes, const std::vector<std::vector<int32_t>>& owner) {
    RequestGraph r;
    r.n = n;
    r.lanes = lanes;
    bool ok = true;
    for (int l = 0; l < lanes && ok; l++) {
        ok = hipStreamBeginCapture(h->main_stream, hipStreamCaptureModeThreadLocal) == hipSuccess;
        if (!ok) break;
        const RequestSlot* slot = h->d_slots + l;
        int rc = each_batch(h, n, ~0ull, owner, [&](Gang& g, int64_t first, int nb) {
            if (g.lane != l) return (int)ENS_OK;
            const int i = (int)(&g - h->gangs.data());
            if (std::find(r.gangs.begin(), r.gangs.end(), i) == r.gangs.end()) r.gangs.push_back(i);
            return forward_batch(h, g, first, nb, nullptr, slot, h->main_stream);
        });
        CombineArgs c = combine_args(h, n, lanes);
        c.slot = slot;
        if (rc == ENS_OK && launch_combine(c, h->main_stream) != hipSuccess) rc = ENS_E_HIP;
        hipGraph_t graph = nullptr;
        ok = hipStreamEndCapture(h->main_stream, &graph) == hipSuccess && rc == ENS_OK && graph;
        ok = ok && hipGraphInstantiate(&r.exec[l], graph, nullptr, nullptr, 0) == hipSuccess;
        if (graph) (void)hipGraphDestroy(graph);
    }
    auto seen = std::find_if(h->sizes_seen.begin(), h->sizes_seen.end(), [&](const SeenSize& x) { return x.n == n; });
    if (!ok) {
        (void)hipGetLastError();
        destroy_graph(h, r);
        if (seen != h->sizes_seen.end()) seen->failed = true;
        return nullptr;
    }
    if (h->graphs.size() >= GRAPHS_KEPT) {
        RequestGraph* const old = oldest_graph(h);
        destroy_graph(h, *old);
        h->graphs.erase(h->graphs.begin() + (old - h->graphs.data()));
    }
    if (seen != h->sizes_seen.end()) h->sizes_seen.erase(seen);      // to be seen twice again once it has been given up
    h->last_recorded = h->requests;
    h->stats.recorded++;
    for (int i : r.gangs) {
        const Worker& w = h->workers[h->gangs[i].workers[0]];
        r.last_batch.emplace_back(w.last_first, w.last_nb);
    }
    h->graphs.push_back(r);
    return &h->graphs.back();
}

// Every segment id goes once to every member; a member's workers share its segments as they would by taking them from one queue, the faster
// worker more of them (planner.cpp, hand_out).
static int hand_out_segments(ens_handle* h, int64_t n, std::vector<std::vector<int32_t>>& owner) {
    for (int c = 0; c < (int)h->members.size(); c++) {
        std::vector<int32_t> batches;
        const Gang* first = nullptr;
        for (const Worker& w : h->workers)                   // in slot order = rank order
            if (w.member == c && !w.copy) {
                batches.push_back(w.batch);
                if (w.rank == 0) first = &h->gangs[w.gang];
            }
        if (batches.size() <= 1 || !first) continue;
        double flop = 0;
        int launches = 1;
        for (const Launch& L : first->plans.back().launches)
            if (L.kind != L_SKIP) { flop += L.flop; launches++; }
        const double launch_cost = launches * 8e-6;          // a kernel of a small batch lasts about this long whatever it does
        const double image_cost = flop / batches[0] / (h->members[c].bf16 ? 4e14 : 2e13);
        const int rc = hand_out(n, h->segment_size, batches.data(), (int)batches.size(), launch_cost, image_cost, &owner[c]);
        if (rc != ENS_OK) return rc;
    }
    return ENS_OK;
}

// The gang that a copy was made from.
static int own_gang(const ens_handle* h, const Gang& copy) {
    const int i = (int)(&copy - h->gangs.data());
    for (int own = 0; own < h->own_gangs; own++)
        if (std::find(h->gangs[own].copies.begin(), h->gangs[own].copies.end(), i) != h->gangs[own].copies.end()) return own;
    return i;
}

// ---- requests of members in LDS -------------------------------------------------------------------------

// The compute units, dealt to the members so that the one that ends last ends first; what an image then takes is the longest of them.
static double deal_blocks(const ens_handle* h, int64_t n, int* blocks) {
    const int M = (int)h->members.size();
    int lds = 0;
    for (const Resident& r : h->residents) lds = std::max(lds, r.lds_floats * 4);
    const int each = lds <= RESIDENT_LDS / 2 ? 2 : 1;             // workgroups per compute unit
    for (int m = 0; m < M; m++) blocks[m] = 1;
    auto end = [&](int m) { return (double)((n + blocks[m] - 1) / blocks[m]) * h->residents[m].seconds * each; };
    for (int left = 256 * each - M;; left--) {
        int slow = 0;
        for (int m = 1; m < M; m++)
            if (end(m) > end(slow)) slow = m;
        if (left <= 0 || blocks[slow] >= n) return end(slow);
        blocks[slow]++;
    }
}

// Beside the launches of a batch at the floor of a launch and at the rate they reach together (measured: 14 TFLOP/s over 8 100 images of 32 x 32).
// Two members of 32 x 32, 1 ... 8 192 images, batches of 8 ... 128: 1.7 to 21 times faster, at no size slower.
static bool resident_wanted(const ens_handle* h, int64_t n) {
    if (h->residents.empty()) return false;
    int blocks[RESIDENT_MAX_MEMBERS];
    double floors = 0, flop = 0;
    for (int i = 0; i < h->own_gangs; i++) {
        const Gang& g = h->gangs[i];
        if (g.rank != 0) continue;
        double t = 0, f = 0;
        for (const Launch& L : g.plans.back().launches)
            if (L.kind != L_SKIP) { t += launch_floor(L.kind); f += L.flop; }
        floors = std::max(floors, t);
        flop += f / h->workers[g.workers[0]].batch * g.workers.size();
    }
    return deal_blocks(h, n, blocks) < floors + (double)n * flop / 14e12;
}

// Images from host memory come in pieces beside the kernels of those before.
constexpr int64_t RESIDENT_PIECE = 1024;

static int run_resident(ens_handle* h, const float* d_images, int64_t n, float* d_probs, const float* host_images) {
    std::vector<std::vector<int32_t>> owner(h->members.size());
    int rc = hand_out_segments(h, n, owner);
    if (rc != ENS_OK) return rc;
    rc = each_batch(h, n, ~0ull, owner, [&](Gang& g, int64_t first, int nb) {   // of a gang and its copies the one that made them tells
        if (g.rank == 0) note_batch(h, h->gangs[own_gang(h, g)], first, nb);
        return (int)ENS_OK;
    });
    if (rc != ENS_OK) return rc;
    ResidentArgs a;
    memset(&a, 0, sizeof(a));
    int blocks[RESIDENT_MAX_MEMBERS], lds = 0;
    const int64_t piece = host_images ? std::min(n, RESIDENT_PIECE) : n;
    (void)deal_blocks(h, piece, blocks);
    a.n_members = (int)h->members.size();
    for (int m = 0, at = 0; m < a.n_members; m++) {
        const Resident& r = h->residents[m];
        ResidentMember& b = a.member[m];
        b.fixed = h->d_resident + h->resident_at[m];
        b.logits = h->d_logits[m];
        b.n_ops = r.n_ops;
        b.fixed_floats = (int)r.fixed.size();
        b.lds_floats = r.lds_floats;
        b.in = r.in; b.in_p = r.in_p; b.in_r = r.in_r;
        b.in_h = h->members[m].in_h; b.in_w = h->members[m].in_w;
        for (Worker& w : h->workers)
            if (w.member == m && w.rank == 0 && !w.copy && w.last_request == h->requests) {
                b.input = (float*)(w.arena + w.layout.offset[0]);
                b.last_first = (int)w.last_first;
                b.last_n = w.last_nb;
                w.input_only = true;
            }
        b.first_block = at;
        b.blocks = blocks[m];
        at += blocks[m];
        lds = std::max(lds, r.lds_floats * 4);
    }
    // images in turn up to two for each workgroup, drawn by who is ready beyond that
    for (int m = 0; m < a.n_members; m++)
        if (piece > 2 * blocks[m]) a.queue = h->resident_queue;
    a.src = d_images;
    a.base_h = h->base_h; a.base_w = h->base_w; a.classes = h->classes;
    const size_t image_floats = (size_t)h->base_h * h->base_w * 3;
    for (int64_t first = 0, k = 0; first < n; first += piece, k++) {
        a.first = (int)first;
        a.n = (int)std::min(piece, n - first);
        if (host_images) {
            HIP_TRY(hipMemcpyAsync((void*)(d_images + first * image_floats), host_images + first * image_floats, (size_t)a.n * image_floats * sizeof(float),
                                   hipMemcpyHostToDevice, h->main_stream));
            while (h->copied.size() <= (size_t)k) {
                hipEvent_t ev = nullptr;
                HIP_TRY(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
                h->copied.push_back(ev);
            }
            HIP_TRY(hipEventRecord(h->copied[k], h->main_stream));
            HIP_TRY(hipStreamWaitEvent(h->lanes[0], h->copied[k], 0));
        }
        HIP_TRY(launch_resident(a, lds, h->lanes[0]));
    }
    h->stats.chained++;
    h->lanes_used = 1;
    CombineArgs c = combine_args(h, n, 1);
    c.y = d_probs;
    HIP_TRY(launch_combine(c, h->lanes[0]));
    if (h->flagged) HIP_TRY(launch_finish(h->d_arrivals + COMBINE_MAX_BLOCKS, 1, h->flag, (uint32_t)h->requests, h->lanes[0]));
    return ENS_OK;
}

// ---- requests as chains -----------------------------------------------------------------------------

// A program's estimate from those of the numbers of images around it (Chain::seconds or ::span).
static double program_seconds(const double (&of)[CHAIN_SIZES], int images) {
    const int z = chain_size(images);
    if (images >= 1 << z) return of[z] * images / (1 << z);
    const double lo = 1 << (z - 1), hi = 1 << z;
    return of[z - 1] + (of[z] - of[z - 1]) * (images - lo) / (hi - lo);
}

// What a request in one launch takes by the spans of its programs (measured beside them: launches_seconds).
constexpr double CHAIN_BASE = 60e-6, CHAIN_SPAN = 1.05;

// Cuts a request into programs for the eight groups: every member's images in the number of parts that ends first by the sums of their
// steps, the longest program first.  None: the request is not one for chains.  (Cut by the spans, four members of batch size 16 on 4 images took
// 832 us instead of 777.)
static ChainPlan plan_programs(const ens_handle* h, int64_t n) {
    ChainPlan best;
    constexpr int GROUPS = 8;                                    // XCDs
    for (int parts = 1; parts <= GROUPS && parts <= n; parts++) {
        std::vector<std::pair<double, ChainProgram>> all;
        const int most = (int)((n + parts - 1) / parts);
        if (parts > 1 && most == (int)((n + parts - 2) / (parts - 1))) continue;
        for (size_t c = 0; c < h->chains.size(); c++)
            for (int first = 0; first < n; first += most) {
                const int images = (int)std::min<int64_t>(most, n - first);
                all.emplace_back(program_seconds(h->chains[c].seconds, images), ChainProgram{(short)c, (short)first, (short)images, (short)chain_size(images)});
            }
        if (all.size() > CHAIN_MAX_PROGRAMS) break;
        std::stable_sort(all.begin(), all.end(), [](const auto& x, const auto& y) { return x.first > y.first; });
        double load[GROUPS] = {0}, end = 0;
        for (const auto& p : all) {
            double& l = *std::min_element(load, load + GROUPS);
            l += p.first;
            end = std::max(end, l);
        }
        if (end < best.seconds) {
            best.seconds = end;
            best.programs.clear();
            for (const auto& p : all) best.programs.push_back(p.second);
        }
    }
    if (best.programs.empty()) return best;
    double load[GROUPS] = {0};                                   // as the groups take them from the queue
    for (const ChainProgram& p : best.programs) *std::min_element(load, load + GROUPS) += program_seconds(h->chains[p.member].span, p.images);
    best.seconds = CHAIN_BASE + CHAIN_SPAN * *std::max_element(load, load + GROUPS);
    return best;
}

// What the launches of the request come to: a launch is a chain of round trips however little it does, one after the other on a lane, and
// the work of all of them takes the GPU besides.
//
// 392 requests were measured both ways: nineteen ensembles of 1 to 12 members, batch sizes 8 to 128, one to 128 images.  The constants here and
// CHAIN_BASE and CHAIN_SPAN were fitted together, to send as few as can be the way that is more than 3 % slower with what comes out even left to the
// launches: 26 of them are, by 25 % at most (three Inception-shaped members on 8 images, whose launches take 1.4 times their estimate).  Chains take
// 0.78 to 1.30 of their estimate (half of them 0.92 to 1.04), launches 0.77 to 1.71 (half of them 0.92 to 1.09; the most a VGG-16, far from either).
// In us, launches / chains: twelve members on 1, 4, 7 and 10 images 2946 / 1226, 3638 / 2534, 4272 / 3980 and 4797 / 5336; four members on 1, 4, 8 and
// 16 818 / 636, 1059 / 767, 1340 / 1154 and 1899 / 1954; a ResNet-50 on 1, 4, 8, 20 and 80 328 / 374, 403 / 397, 487 / 411, 711 / 782 and 1585 / 1806; with
// a DenseNet-121 on 1 924 / 631; an Inception-shaped member on 1, 4 and 16 528 / 521, 600 / 553 and 1064 / 787; three ResNet-18, whose launches carry all
// three, on 1 and 8 189 / 189 and 341 / 357.
static double launches_seconds(ens_handle* h, int64_t n) {
    const std::vector<std::vector<int32_t>> owner(h->members.size(), std::vector<int32_t>(1, 0));   // (one segment: the first worker's)
    std::vector<double> floors(h->gangs.size(), 0.0);
    double work = 0;
    (void)each_batch(h, n, ~0ull, owner, [&](Gang& g, int64_t, int nb) {
        const double share = (double)nb / h->workers[g.workers[0]].batch * (double)g.workers.size();
        floors[&g - h->gangs.data()] += launch_floor(L_POOL);    // input staging
        for (const Launch& L : g.plan_for(nb).launches)
            if (L.kind != L_SKIP) {
                floors[&g - h->gangs.data()] += launch_floor(L.kind);
                work += launch_work(L, share);
            }
        return ENS_OK;
    });
    std::sort(floors.begin(), floors.end(), [](double x, double y) { return x > y; });
    double load[LANES] = {0};
    for (double t : floors) *std::min_element(load, load + LANES) += t;
    // (the floors are those of a launch among others' on four lanes: on a lane of its own a gang is faster)
    const bool several = std::count_if(floors.begin(), floors.end(), [](double t) { return t > 0.0; }) > 1;
    return *std::max_element(load, load + LANES) * (several ? 1.05 : 0.88) + 0.7 * work;
}

// How a request of n images is cut into programs, or null when it goes launch by launch: whichever the estimates have end first.
static const ChainPlan* chain_plan(ens_handle* h, int64_t n) {
    if (h->chains.empty() || h->chains_off) return nullptr;
    for (const Chain& c : h->chains)
        if (n > c.cap) return nullptr;
    if (h->chain_plans.size() <= (size_t)n) h->chain_plans.resize((size_t)n + 1);
    ChainPlan& p = h->chain_plans[(size_t)n];
    if (!p.known) {
        p = plan_programs(h, n);
        p.known = true;
        if (p.seconds > launches_seconds(h, n)) p.programs.clear();
    }
    return p.programs.empty() ? nullptr : &p;
}

// The request in one launch and the combination behind it, on the first lane.
static int run_chains(ens_handle* h, const float* d_images, int64_t n, float* d_probs, const ChainPlan& plan, const float* host_images) {
    const std::vector<ChainProgram>& programs = plan.programs;
    if (host_images)
        HIP_TRY(hipMemcpyAsync((void*)d_images, host_images, (size_t)n * h->base_h * h->base_w * 3 * sizeof(float), hipMemcpyHostToDevice, h->lanes[0]));
    ChainArgs a;
    memset(&a, 0, sizeof(a));
    for (size_t c = 0; c < h->members.size(); c++) {
        a.steps[c] = h->d_chain + h->chain_at[c];
        a.phases[c] = (short)h->chains[c].phases;
        a.image_bytes[c] = (unsigned)h->chains[c].image_bytes;
        a.logits[c] = h->d_logits[c];
    }
    for (Worker& w : h->workers)
        if (w.rank == 0 && !w.copy) {
            a.arena[w.member] = w.arena;
            w.last_nb = (int)n;
            w.input_only = false;
            w.last_request = h->requests;
            w.last_first = 0;
            w.last_programs.clear();
            for (const ChainProgram& p : programs)
                if (p.member == w.member) w.last_programs.push_back(p);
        }
    std::copy(programs.begin(), programs.end(), a.programs);
    a.n_programs = (int)programs.size();
    a.sync = h->d_chain_sync;
    a.failed = h->flag + CHAIN_FAILED_WORD;
    a.src = d_images;
    a.base_h = h->base_h; a.base_w = h->base_w; a.classes = h->classes;
    HIP_TRY(launch_chain(a, h->lanes[0]));
    h->stats.chained++;
    h->lanes_used = 1;
    CombineArgs c = combine_args(h, n, 1);
    c.y = d_probs;
    HIP_TRY(launch_combine(c, h->lanes[0]));
    if (h->flagged) HIP_TRY(launch_finish(h->d_arrivals + COMBINE_MAX_BLOCKS, 1, h->flag, (uint32_t)h->requests, h->lanes[0]));
    return ENS_OK;
}

// f(X, A) -> Y with Y on the device (or in pinned host memory).  The images are at d_images; when host_images is
// given they are still to be copied there from host memory, segment by segment beside the kernels of the segments before.
// `mask` selects the members that take part (all members for a real request; a single member when the BBS baseline
// times it alone).  may_alloc false (the allocation-free entry point): the logits buffers are already in place and
// nothing on the way may allocate or free device memory.  Returns with the work on the lanes: wait_lanes.
static int run_device(ens_handle* h, const float* d_images, int64_t n, float* d_probs, uint64_t mask, bool may_alloc = true,
                      const float* host_images = nullptr) {
    if (n == 0) return ENS_OK;
    cu_budget() = stream_share(h);
    lanes_busy() = std::min(LANES, std::max(1, h->own_gangs));
    int rc = may_alloc ? with_room(h, [&] { return ensure_buffers(h, n); }) : ENS_OK;
    if (rc != ENS_OK) return rc;
    if ((size_t)n > h->d_logits_rows) return ENS_E_INVALID;
    const int M = (int)h->members.size();
    const int seg = h->segment_size;
    const int64_t n_seg = (n + seg - 1) / seg;
    if (h->args_stale) {                                         // other logits than those that the argument blocks name
        for (Gang& g : h->gangs) g.stale = true;
        h->args_stale = false;
    }
    auto refresh = [&](int i) { return h->gangs[i].stale ? build_launches(h, h->gangs[i], may_alloc) : ENS_OK; };
    h->requests++;
    const bool plain_only = !may_alloc || h->profiling || h->fake_predictor || h->one_stream || mask != ~0ull;
    if (!h->profiling && !h->fake_predictor && !h->one_stream && mask == ~0ull) {
        const ChainPlan* plan = chain_plan(h, n);
        if (plan) return run_chains(h, d_images, n, d_probs, *plan, host_images);
        if (n < (int64_t)1 << 30 && resident_wanted(h, n)) return run_resident(h, d_images, n, d_probs, host_images);
    }
    RequestGraph* graph = plain_only || (host_images && n_seg > 1) ? nullptr : find_graph(h, n);
    // every segment id goes once to every member; a member's workers share its segments as they
    // would by taking them from one queue, the faster worker more of them (planner.cpp, hand_out)
    std::vector<std::vector<int32_t>> owner(M);
    int lanes = graph ? graph->lanes : 0;
    Work work;
    bool hand_out_batches = false;
    if (!graph) {
        rc = hand_out_segments(h, n, owner);
        if (rc != ENS_OK) return rc;
        work = plan_work(h, n, mask, owner);
        // More gangs than lanes with several batches each are handed out as the lanes come free (below), unless their launches are so
        // short that the host has to be out of the way.
        hand_out_batches = !h->one_stream && h->gangs.size() > LANES && work.most > 1 && work.total > HAND_OUT_LAUNCH_S * (double)work.launches;
        lanes = lanes_in_use() = hand_out_batches ? LANES : deal_lanes(h, work);
        for (size_t i = 0; i < h->gangs.size(); i++) {
            if (work.batches[i].empty()) continue;
            rc = refresh((int)i);
            if (rc != ENS_OK) return rc;
        }
        if (!plain_only && !(host_images && n_seg > 1) && !hand_out_batches && lanes >= GRAPH_MIN_LANES && work.launches <= GRAPH_MAX_LAUNCHES &&
            worth_recording(h, n))
            graph = record_request(h, n, lanes, owner);
    }
    h->lanes_used = lanes;
    // Host images go to the device in pieces of the smallest batch, beside the kernels; a lane waits for the last piece it needs.
    const size_t image_floats = (size_t)h->base_h * h->base_w * 3;
    int64_t piece = seg;
    for (const Worker& w : h->workers) piece = std::min<int64_t>(piece, w.batch);
    piece = std::max<int64_t>(piece, 16);
    const int64_t pieces = host_images ? (n + piece - 1) / piece : 0;
    int64_t here = 0, waited[LANES] = {0};                       // pieces whose copies have been issued; that a lane has waited for
    auto bring_piece = [&]() -> int {
        const int64_t start = here * piece, end = std::min<int64_t>(start + piece, n);
        HIP_TRY(hipMemcpyAsync((void*)(d_images + start * image_floats), host_images + start * image_floats,
                               (size_t)(end - start) * image_floats * sizeof(float), hipMemcpyHostToDevice, h->main_stream));
        while (h->copied.size() <= (size_t)here) {
            hipEvent_t e = nullptr;
            HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
            h->copied.push_back(e);
        }
        HIP_TRY(hipEventRecord(h->copied[here++], h->main_stream));
        return ENS_OK;
    };
    auto need_images = [&](int l, int64_t end) -> int {          // lane l: images up to `end`
        if (!host_images) return ENS_OK;
        const int64_t p = (end + piece - 1) / piece;
        while (here < p) {
            const int e = bring_piece();
            if (e != ENS_OK) return e;
        }
        if (waited[l] < p) HIP_TRY(hipStreamWaitEvent(h->lanes[l], h->copied[p - 1], 0));   // copies are in order
        waited[l] = std::max(waited[l], p);
        return ENS_OK;
    };
    if (graph) {
        for (int i : graph->gangs) {
            rc = refresh(i);
            if (rc != ENS_OK) return rc;
        }
        graph->used = h->requests;
        h->stats.replayed++;
        for (int l = 0; l < lanes; l++) {
            rc = need_images(l, n);
            if (rc != ENS_OK) return rc;
            HIP_TRY(launch_bind_request(h->d_slots + l, RequestSlot{d_images, d_probs}, h->lanes[l]));
            HIP_TRY(hipGraphLaunch(graph->exec[l], h->lanes[l]));
            if (h->flagged) HIP_TRY(launch_finish(h->d_arrivals + COMBINE_MAX_BLOCKS, lanes, h->flag, (uint32_t)h->requests, h->lanes[l]));
        }
        for (size_t i = 0; i < graph->gangs.size(); i++) note_batch(h, h->gangs[graph->gangs[i]], graph->last_batch[i].first, graph->last_batch[i].second);
        return ENS_OK;
    }
    if (hand_out_batches) {
        // A lane holds two batches, the one that runs and the next; when one ends it gets the next batch of the gang that has the most
        // left to do among those that have nothing on another lane.  (Dealt to the lanes beforehand by the estimates, the twelve-member
        // ensemble's lanes ended between 151 and 191 ms.)
        // A batch ends in finish_kernel, which writes its number to the lane's word in pinned memory (asking the runtime about events
        // in a loop slowed the GPU's own queues down: 21.5 ms instead of 17.2 for three ResNet-18 over 1024 images).
        struct InFlight { int gang = -1; uint32_t number = 0; };
        InFlight flight[LANES][2];
        std::vector<size_t> next(h->gangs.size(), 0);
        std::vector<int> out(h->gangs.size(), 0), on(h->gangs.size(), -1);   // batches in flight, and their lane
        std::vector<double> left = work.estimate;
        uint32_t issued[LANES] = {0};
        for (int l = 0; l < lanes; l++) __atomic_store_n(h->flag + 1 + l, 0u, __ATOMIC_RELEASE);
        size_t remaining = 0;
        for (const auto& b : work.batches) remaining += b.size();
        auto t_moved = std::chrono::steady_clock::now();
        while (remaining) {
            bool moved = false;
            for (int k = 0; k < 2; k++)                          // every lane one batch before any has two
                for (int l = 0; l < lanes; l++) {
                    InFlight& f = flight[l][k];
                    if (f.gang >= 0) {
                        if (__atomic_load_n(h->flag + 1 + l, __ATOMIC_ACQUIRE) < f.number) continue;
                        out[f.gang]--;
                        f.gang = -1;
                    }
                    int pick = -1;
                    double pick_due = 0;
                    for (size_t i = 0; i < h->gangs.size(); i++) {
                        if (next[i] >= work.batches[i].size() || (out[i] > 0 && on[i] != l)) continue;
                        if (host_images && work.batches[i][next[i]].first + work.batches[i][next[i]].nb > here * piece && here < pieces) continue;
                        // a gang stays on its lane unless another has two batches more to do
                        const double due = left[i] + (out[i] > 0 ? 2.0 * work.batches[i][next[i]].estimate : 0.0);
                        if (pick < 0 || due > pick_due) { pick = (int)i; pick_due = due; }
                    }
                    if (pick < 0) continue;
                    const Batch& b = work.batches[pick][next[pick]++];
                    rc = need_images(l, b.first + b.nb);
                    if (rc == ENS_OK) rc = forward_batch(h, h->gangs[pick], b.first, b.nb, d_images, nullptr, h->lanes[l]);
                    if (rc != ENS_OK) return rc;
                    h->stats.handed_out++;
                    f.number = ++issued[l];
                    HIP_TRY(launch_finish(h->d_arrivals, 1, h->flag + 1 + l, f.number, h->lanes[l]));
                    f.gang = pick;
                    out[pick]++;
                    on[pick] = l;
                    left[pick] -= b.estimate;
                    remaining--;
                    moved = true;
                }
            if (moved) {
                t_moved = std::chrono::steady_clock::now();
                continue;
            }
            if (here < pieces) {
                rc = bring_piece();
                if (rc != ENS_OK) return rc;
                continue;
            }
            for (int i = 0; i < 200; i++) __builtin_ia32_pause();       // some 5 us
            if (std::chrono::steady_clock::now() - t_moved > std::chrono::seconds(2)) {   // a lane that is stuck: the runtime knows why
                HIP_TRY(wait_lanes(h));
                t_moved = std::chrono::steady_clock::now();
            }
        }
    } else {
        rc = each_batch(h, n, mask, owner, [&](Gang& g, int64_t first, int nb) {
            const int e = need_images(g.lane, first + nb);
            return e != ENS_OK ? e : forward_batch(h, g, first, nb, d_images, nullptr, h->lanes[g.lane]);
        });
        if (rc != ENS_OK) return rc;
    }
    if (mask == ~0ull || M == 1) {
        CombineArgs c = combine_args(h, n, lanes);
        c.y = d_probs;
        for (int l = 0; l < lanes; l++) {
            ProfRec r{prof_class(h, "combine_kernel"), nullptr, nullptr, 0.0, (double)n * h->classes * 4.0 * (M + 1)};
            if (h->profiling && l == lanes - 1) {
                r.start = take_event(h); r.stop = take_event(h);
                if (!r.start || !r.stop) return ENS_E_HIP;
                next_launch_events() = LaunchEvents{r.start, r.stop};
            }
            HIP_TRY(launch_combine(c, h->lanes[l]));
            if (h->flagged) HIP_TRY(launch_finish(h->d_arrivals + COMBINE_MAX_BLOCKS, lanes, h->flag, (uint32_t)h->requests, h->lanes[l]));
            if (r.start) {
                next_launch_events() = LaunchEvents{};
                h->prof_recs.push_back(r);
            }
        }
    }
    return ENS_OK;
}

// After a request that failed on the way: nothing of it is left in flight, and the arrivals are zeros again.
static void recover(ens_handle* h) {
    (void)hipDeviceSynchronize();
    h->flagged = false;
    if (h->d_arrivals) (void)hipMemset(h->d_arrivals, 0, (COMBINE_MAX_BLOCKS + 1) * sizeof(unsigned));
    if (h->d_chain_sync) (void)hipMemset(h->d_chain_sync, 0, sizeof(ChainSync));
    (void)hipGetLastError();
}

// A request from its launches to its end.  A chain's group that waited for seconds has said so and left: the launches answer that request,
// and those after it until the next allocation is installed.
static int answer(ens_handle* h, const float* d_images, int64_t n, float* d_probs, uint64_t mask = ~0ull, bool may_alloc = true, const float* host_images = nullptr) {
    const bool flagged = h->flagged;
    for (;;) {
        const int64_t rows = rows_taken();
        rows_off() = h->no_rows;
        const int rc = run_device(h, d_images, n, d_probs, mask, may_alloc, host_images);
        h->stats.rows += rows_taken() - rows;
        if (rc != ENS_OK) { recover(h); return rc; }
        HIP_TRY(wait_lanes(h));
        if (!__atomic_load_n(h->flag + CHAIN_FAILED_WORD, __ATOMIC_ACQUIRE)) break;
        recover(h);
        __atomic_store_n(h->flag + CHAIN_FAILED_WORD, 0u, __ATOMIC_RELEASE);
        h->chains_off = true;
        h->flagged = flagged;
    }
    h->flagged = false;
    return ENS_OK;
}

static int finish_profile(ens_handle* h) {
    for (ProfRec& r : h->prof_recs) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, r.start, r.stop) == hipSuccess) {
            ProfClass& c = h->prof[r.klass];
            c.ms += ms; c.flop += r.flop; c.bytes += r.bytes; c.launches++;
        }
        h->event_pool.push_back(r.start);
        h->event_pool.push_back(r.stop);
    }
    h->prof_recs.clear();
    return ENS_OK;
}

static void reset_profile(ens_handle* h) {
    for (ProfClass& c : h->prof) { c.ms = 0; c.flop = 0; c.bytes = 0; c.launches = 0; }
}

static int default_alloc(ens_handle* h) {
    ens_alloc a;
    memset(&a, 0, sizeof(a));
    a.rows = 1;
    a.cols = (int)h->members.size();
    for (int c = 0; c < a.cols; c++) a.batch[0][c] = 8;
    return install_alloc(h, a, 128);
}

static int ensure_calib(ens_handle* h, int64_t n) {
    if ((size_t)n <= h->d_calib_images) return ENS_OK;
    if (h->d_calib) (void)hipFree(h->d_calib);
    h->d_calib = nullptr;
    h->d_calib_images = 0;
    const size_t count = (size_t)n * h->base_h * h->base_w * 3;
    HIP_TRY(hipMalloc((void**)&h->d_calib, count * sizeof(float)));
    HIP_TRY(launch_fill_noise(h->d_calib, (int64_t)count, 0x5EEDCA11Bull, h->main_stream));
    HIP_TRY(hipStreamSynchronize(h->main_stream));
    h->d_calib_images = (size_t)n;
    return ENS_OK;
}

// Small requests from and to host memory: the staging kernels read the images in pinned host memory themselves (each
// gang does, hence the product with their number) and the combination writes the probabilities there, instead of a
// copy on a stream in front of the kernels and one behind them (10 us each, 20 and more from pageable memory).
// Coherent memory for both: what the GPU may cache of other pinned memory is only brought up to date by synchronising a stream, and
// a request that is waited for on the flag synchronises none.  (Images in cached pinned memory were no faster: fp32 pair, 8
// images 63 us against 61, three ResNet-18, one image 192 against 191.)
constexpr size_t DIRECT_IN_BYTES = 1280u << 10, DIRECT_OUT_BYTES = 256u << 10;

static int grow_pinned(float** p, size_t* cap, size_t want_floats) {
    if (want_floats <= *cap) return ENS_OK;
    if (*p) (void)hipHostFree(*p);
    *p = nullptr;
    *cap = 0;
    HIP_TRY(hipHostMalloc((void**)p, want_floats * sizeof(float), hipHostMallocCoherent));
    *cap = want_floats;
    return ENS_OK;
}

// Benchmark Mode on the installed allocation: median images/s of `repeats` runs after a warm-up.
static int time_installed(ens_handle* h, int64_t n, int repeats, uint64_t mask, double* ips) {
    int rc = with_room(h, [&] { return ensure_calib(h, n); });
    if (rc != ENS_OK) return rc;
    rc = with_room(h, [&] { return grow(&h->d_probs, &h->d_probs_cap, (size_t)n * h->classes); });
    if (rc != ENS_OK) return rc;
    std::vector<double> secs;
    for (int i = 0; i < repeats + 1; i++) {
        const auto t0 = std::chrono::steady_clock::now();
        rc = answer(h, h->d_calib, n, h->d_probs, mask);
        if (rc != ENS_OK) return rc;
        const auto t1 = std::chrono::steady_clock::now();
        if (i > 0) secs.push_back(std::chrono::duration<double>(t1 - t0).count());
    }
    if (h->profiling) finish_profile(h);
    std::sort(secs.begin(), secs.end());
    *ips = (double)n / secs[secs.size() / 2];
    return ENS_OK;
}

}  // namespace ens

// ------------------------------------------------------------------------------------ C API
extern "C" {

int ens_load(const ens_member_spec* specs, int32_t n_members, uint64_t seed, ens_handle** out) {
    if (!specs || !out || n_members <= 0 || n_members > ENS_MAX_MEMBERS) return ENS_E_INVALID;
    *out = nullptr;
    ens_handle* h = new ens_handle();
    memset(&h->alloc, 0, sizeof(h->alloc));
    for (int i = 0; i < n_members; i++) {
        const ens_member_spec& sp = specs[i];
        std::vector<float> drawn;
        const float* params = sp.params;
        if (!params) {
            if (!sp.param_specs || sp.n_params <= 0) { delete h; return ENS_E_INVALID; }
            drawn.assign((size_t)sp.n_params, 0.f);
            const int rc = draw_params(sp.param_specs, sp.n_param_specs, seed, i, drawn.data(), sp.n_params);
            if (rc != ENS_OK) { delete h; return rc; }
            params = drawn.data();
        }
        Member m;
        const int rc = build_member(sp, params, &m);
        if (rc != ENS_OK) { delete h; return rc; }
        h->members.push_back(std::move(m));
    }
    h->classes = h->members[0].classes;
    for (const Member& m : h->members)
        if (m.classes != h->classes) { delete h; return ENS_E_INVALID; }
    h->base_h = h->members[0].in_h;
    h->base_w = h->members[0].in_w;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) {
        (void)hipGetLastError();
        delete h;
        return ENS_E_NODEVICE;
    }
    auto fail = [&](int rc) { ens_free(h); return rc; };
    for (Member& m : h->members) {
        hipError_t e = hipMalloc((void**)&m.dev_params, std::max<size_t>(m.host_params.size(), 256));
        if (e == hipSuccess)
            e = hipMemcpy(m.dev_params, m.host_params.data(), m.host_params.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return fail(e == hipErrorOutOfMemory ? ENS_E_NOMEM : ENS_E_HIP);
        }
    }
    if (hipStreamCreateWithFlags(&h->main_stream, hipStreamNonBlocking) != hipSuccess) return fail(ENS_E_HIP);
    if (acquire_lanes(h->lanes) != hipSuccess) return fail(ENS_E_HIP);
    h->have_lanes = true;
    if (hipMalloc((void**)&h->d_slots, LANES * sizeof(RequestSlot)) != hipSuccess) return fail(ENS_E_NOMEM);
    if (hipMalloc((void**)&h->d_arrivals, (COMBINE_MAX_BLOCKS + 1) * sizeof(unsigned)) != hipSuccess) return fail(ENS_E_NOMEM);
    if (hipMemset(h->d_arrivals, 0, (COMBINE_MAX_BLOCKS + 1) * sizeof(unsigned)) != hipSuccess) return fail(ENS_E_HIP);
    if (hipHostMalloc((void**)&h->flag, 64, hipHostMallocCoherent) != hipSuccess) return fail(ENS_E_NOMEM);
    memset(h->flag, 0, 64);
    if (hipMalloc((void**)&h->d_chain_sync, sizeof(ChainSync)) != hipSuccess) return fail(ENS_E_NOMEM);
    if (hipMemset(h->d_chain_sync, 0, sizeof(ChainSync)) != hipSuccess) return fail(ENS_E_HIP);
    h->d_logits.assign(h->members.size(), nullptr);
    h->stage_klass = prof_class(h, "stage_kernel");
    *out = h;
    return ENS_OK;
}

void ens_free(ens_handle* h) {
    if (!h) return;
    (void)hipDeviceSynchronize();
    destroy_workers(h);
    for (Member& m : h->members)
        if (m.dev_params) (void)hipFree(m.dev_params);
    for (float* p : h->d_logits_heap)
        if (p) (void)hipFree(p);
    if (h->d_slots) (void)hipFree(h->d_slots);
    if (h->d_arrivals) (void)hipFree(h->d_arrivals);
    if (h->d_chain_sync) (void)hipFree(h->d_chain_sync);
    if (h->pin_in) (void)hipHostFree(h->pin_in);
    if (h->pin_out) (void)hipHostFree(h->pin_out);
    if (h->flag) (void)hipHostFree(h->flag);
    if (h->d_weights) (void)hipFree(h->d_weights);
    if (h->d_images) (void)hipFree(h->d_images);
    if (h->d_probs) (void)hipFree(h->d_probs);
    if (h->d_calib) (void)hipFree(h->d_calib);
    for (ProfRec& r : h->prof_recs) { (void)hipEventDestroy(r.start); (void)hipEventDestroy(r.stop); }
    for (hipEvent_t e : h->event_pool) (void)hipEventDestroy(e);
    for (hipEvent_t e : h->copied) (void)hipEventDestroy(e);
    if (h->have_lanes) release_lanes(h->lanes);
    if (h->main_stream) (void)hipStreamDestroy(h->main_stream);
    delete h;
}

int ens_set_io(ens_handle* h, int32_t base_h, int32_t base_w, int32_t images_on_device, int32_t probs_on_device) {
    if (!h || base_h <= 0 || base_w <= 0) return ENS_E_INVALID;
    if (base_h != h->base_h || base_w != h->base_w) {
        if (h->d_calib) (void)hipFree(h->d_calib);
        h->d_calib = nullptr;
        h->d_calib_images = 0;
        drop_graphs(h);                                          // the staging launches hold the image size
    }
    h->base_h = base_h;
    h->base_w = base_w;
    h->images_on_device = images_on_device != 0;
    h->probs_on_device = probs_on_device != 0;
    return ENS_OK;
}

int ens_set_alloc(ens_handle* h, const ens_alloc* a, int32_t segment_size) {
    if (!h || !a) return ENS_E_INVALID;
    return install_alloc(h, *a, segment_size);
}

int ens_predict(ens_handle* h, const float* images, int64_t n, float* probs_out) {
    if (!h || n < 0 || (n > 0 && (!images || !probs_out))) return ENS_E_INVALID;
    if (n == 0) return ENS_OK;
    if (!h->have_alloc) {
        const int rc = default_alloc(h);
        if (rc != ENS_OK) return rc;
    }
    const auto t0 = std::chrono::steady_clock::now();
    const size_t img_floats = (size_t)n * h->base_h * h->base_w * 3, out_floats = (size_t)n * h->classes;
    const float *d_in = images, *host_in = nullptr;
    if (!h->images_on_device) {
        if (img_floats * sizeof(float) * h->own_gangs <= DIRECT_IN_BYTES) {
            int rc = grow_pinned(&h->pin_in, &h->pin_in_cap, img_floats);
            if (rc != ENS_OK) return rc;
            memcpy(h->pin_in, images, img_floats * sizeof(float));
            d_in = h->pin_in;
        } else {
            int rc = with_room(h, [&] { return grow(&h->d_images, &h->d_images_cap, img_floats); });
            if (rc != ENS_OK) return rc;
            d_in = h->d_images;
            host_in = images;
        }
    }
    float* d_out = probs_out;
    const bool direct_out = !h->probs_on_device && out_floats * sizeof(float) <= DIRECT_OUT_BYTES;
    if (!h->probs_on_device) {
        int rc = direct_out ? grow_pinned(&h->pin_out, &h->pin_out_cap, out_floats) : with_room(h, [&] { return grow(&h->d_probs, &h->d_probs_cap, out_floats); });
        if (rc != ENS_OK) return rc;
        d_out = direct_out ? h->pin_out : h->d_probs;
    }
    if (h->profiling) reset_profile(h);
    h->flagged = direct_out && !h->profiling;
    const int rc = answer(h, d_in, n, d_out, ~0ull, true, host_in);
    if (rc != ENS_OK) return rc;
    if (direct_out) {
        memcpy(probs_out, h->pin_out, out_floats * sizeof(float));
    } else if (!h->probs_on_device) {
        HIP_TRY(hipMemcpyAsync(probs_out, d_out, out_floats * sizeof(float), hipMemcpyDeviceToHost, h->main_stream));
        HIP_TRY(hipStreamSynchronize(h->main_stream));
    }
    if (h->profiling) finish_profile(h);
    h->last_n = n;
    h->last_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return ENS_OK;
}

int ens_predict_static(ens_handle* h, const float* d_images, int64_t n, float* d_probs_out) {
    if (!h || n < 0 || (n > 0 && (!d_images || !d_probs_out))) return ENS_E_INVALID;
    if (!h->have_alloc || h->profiling) {
        fprintf(stderr, "ens_predict_static: %s\n", !h->have_alloc ? "no allocation installed (ens_plan or ens_set_alloc first)"
                                                                   : "per-kernel profiling creates events: switch it off");
        return ENS_E_INVALID;
    }
    if (n == 0) return ENS_OK;
    const auto t0 = std::chrono::steady_clock::now();
    int rc = use_static_logits(h, n);
    if (rc != ENS_OK) return rc;
    rc = answer(h, d_images, n, d_probs_out, ~0ull, false);
    if (rc != ENS_OK) return rc;
    h->last_n = n;
    h->last_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return ENS_OK;
}

int ens_static_scratch_bytes(void) { return (int)STATIC_SCRATCH_BYTES; }

int ens_bench(ens_handle* h, const ens_alloc* a, int32_t segment_size, int64_t n_calib, int32_t repeats,
              double* img_per_sec) {
    if (!h || !a || !img_per_sec || n_calib <= 0) return ENS_E_INVALID;
    if (repeats <= 0) repeats = 3;
    *img_per_sec = 0.0;
    int rc = install_alloc(h, *a, segment_size);
    if (rc == ENS_E_NOMEM) return ENS_OK;                        // a matrix that does not fit scores zero (Algorithm 2, definition of bench)
    if (rc != ENS_OK) return rc;
    if (h->profiling) reset_profile(h);
    return time_installed(h, n_calib, repeats, ~0ull, img_per_sec);
}

int ens_plan(ens_handle* h, uint64_t mem_budget_bytes, const ens_plan_opts* opts, ens_alloc* out) {
    if (!h || !out) return ENS_E_INVALID;
    ens_plan_opts o;
    memset(&o, 0, sizeof(o));
    if (opts) o = *opts;
    if (o.n_domain <= 0) {
        const int d[5] = {8, 16, 32, 64, 128};
        o.n_domain = 5;
        memcpy(o.domain, d, sizeof(d));
    }
    if (o.n_domain > ENS_MAX_DOMAIN) return ENS_E_INVALID;
    if (o.default_batch <= 0) o.default_batch = *std::min_element(o.domain, o.domain + o.n_domain);
    if (o.segment_size <= 0) o.segment_size = 128;
    if (o.max_neighs <= 0) o.max_neighs = 100;
    if (o.max_iter <= 0) o.max_iter = 10;
    if (o.slots <= 0) o.slots = 1;
    if (o.slots > ENS_MAX_SLOTS) return ENS_E_INVALID;
    if (o.n_calib <= 0) o.n_calib = 1024;
    if (o.repeats <= 0) o.repeats = 3;
    const int M = (int)h->members.size();
    if (mem_budget_bytes == 0) {
        size_t fr = 0, tot = 0;
        HIP_TRY(hipMemGetInfo(&fr, &tot));
        mem_budget_bytes = tot;
    }
    std::vector<int64_t> wbytes(M), abytes((size_t)M * o.n_domain);
    for (int m = 0; m < M; m++) {
        wbytes[m] = (int64_t)h->members[m].weight_bytes();
        for (int j = 0; j < o.n_domain; j++) abytes[(size_t)m * o.n_domain + j] = (int64_t)plan_arena(h->members[m], o.domain[j]).bytes;
    }
    std::vector<int32_t> row_pool(o.slots, 0), row_gpu(o.slots, 1);
    // request buffers (images, logits, probabilities) come out of the same budget
    int64_t reserve = (int64_t)o.n_calib * ((int64_t)h->base_h * h->base_w * 3 + (int64_t)h->classes * (M + 1)) * 4;
    int64_t cap = (int64_t)mem_budget_bytes - reserve;
    if (cap < 0) cap = 0;
    h->budget = mem_budget_bytes;
    h->reserve = reserve;
    ens_plan_problem p;
    p.n_models = M; p.n_rows = o.slots; p.n_pools = 1; p.n_domain = o.n_domain;
    p.domain = o.domain; p.default_batch = o.default_batch;
    p.weight_bytes = wbytes.data(); p.arena_bytes = abytes.data();
    p.row_pool = row_pool.data(); p.row_is_gpu = row_gpu.data(); p.pool_cap = &cap;
    p.max_iter = o.max_iter; p.max_neighs = o.max_neighs; p.seed = o.seed;
    if (!problem_ok(&p)) return ENS_E_INVALID;

    std::vector<int32_t> A((size_t)o.slots * M, 0);
    int rc = wfd(p, A.data());
    if (rc != ENS_OK) return rc;
    auto to_alloc = [&](const int32_t* mat) {
        ens_alloc a;
        memset(&a, 0, sizeof(a));
        a.rows = o.slots; a.cols = M;
        for (int r = 0; r < o.slots; r++)
            for (int c = 0; c < M; c++) a.batch[r][c] = mat[r * M + c];
        return a;
    };
    int hip_rc = ENS_OK;
    int32_t shown = 0;
    auto show = [&](const int32_t* mat, double ips) {             // progress of a long plan
        if (!o.verbose) return;
        std::string line;
        for (int r = 0; r < o.slots; r++) {
            line += r ? " | " : "";
            for (int c = 0; c < M; c++) line += (c ? " " : "") + std::to_string(mat[r * M + c]);
        }
        fprintf(stderr, "ens_plan: benchmark %d: [%s] -> %.1f images/s\n", ++shown, line.c_str(), ips);
        fflush(stderr);
    };
    auto bench = [&](const int32_t* mat) -> double {
        if (!fit_mem(p, mat)) return 0.0;
        const ens_alloc a = to_alloc(mat);
        double ips = 0.0;
        const int r = ens_bench(h, &a, o.segment_size, o.n_calib, o.repeats, &ips);
        if (r != ENS_OK) { hip_rc = r; return 0.0; }
        show(mat, ips);
        return ips;
    };
    // A matrix is judged by its workers' batches: a request that runs in one launch hardly depends on it, and members timed alone go by launches
    double score = 0.0;
    int32_t n_bench = 0;
    h->planning = true;
    if (o.strategy == 0) {
        rc = greedy(p, A.data(), bench, &score, &n_bench);
    } else if (o.strategy == 1) {
        score = bench(A.data());
        n_bench = 1;
    } else if (o.strategy == 2) {
        // each member alone on the GPU, its batch size scanned; then the combined matrix is timed
        std::vector<int32_t> best(M, o.default_batch);
        auto single = [&](int m, int b) -> double {
            std::vector<int32_t> mat((size_t)o.slots * M, 0);
            for (int c = 0; c < M; c++) mat[c] = c == m ? b : o.default_batch;
            if (!fit_mem(p, mat.data())) return 0.0;
            const ens_alloc a = to_alloc(mat.data());
            h->gangs_enabled = false;                            // the member is timed alone
            int r = install_alloc(h, a, o.segment_size);
            h->gangs_enabled = true;
            if (r == ENS_E_NOMEM) return 0.0;
            if (r != ENS_OK) { hip_rc = r; return 0.0; }
            double ips = 0.0;
            r = time_installed(h, o.n_calib, o.repeats, 1ull << m, &ips);
            if (r != ENS_OK) { hip_rc = r; return 0.0; }
            show(mat.data(), ips);
            return ips;
        };
        rc = bbs(p, single, best.data(), &n_bench);
        std::fill(A.begin(), A.end(), 0);
        for (int c = 0; c < M; c++) A[c] = best[c];
        score = bench(A.data());
    } else {
        rc = ENS_E_INVALID;
    }
    h->planning = false;
    if (rc != ENS_OK) return rc;
    if (hip_rc != ENS_OK) return hip_rc;
    ens_alloc a = to_alloc(A.data());
    rc = install_alloc(h, a, o.segment_size);
    if (rc != ENS_OK) return rc;
    *out = h->alloc;
    out->score = score;
    out->n_bench = n_bench;
    h->alloc = *out;
    return ENS_OK;
}

int ens_member_logits(ens_handle* h, int32_t member, int64_t n, float* logits_out) {
    if (!h || member < 0 || member >= (int)h->members.size() || !logits_out) return ENS_E_INVALID;
    if (n <= 0 || n > h->last_n || (size_t)n > h->d_logits_rows) return ENS_E_INVALID;
    HIP_TRY(hipMemcpy(logits_out, h->d_logits[member], (size_t)n * h->members[member].classes * sizeof(float),
                      hipMemcpyDeviceToHost));
    return ENS_OK;
}

int ens_debug_tensor(ens_handle* h, int32_t member, int32_t tensor, int32_t n_images, float* out) {
    if (!h || !out || member < 0 || member >= (int)h->members.size()) return ENS_E_INVALID;
    const Member& m = h->members[member];
    if (tensor < 0 || tensor >= (int)m.tensors.size() || m.tensors[tensor].external) return ENS_E_INVALID;
    const Worker* w = nullptr;
    for (const Worker& x : h->workers)
        if (x.member == member) { w = &x; break; }
    if (!w) return ENS_E_INVALID;
    const Gang& own = h->gangs[w->gang];                         // its batches may have gone to copies of its gang
    const size_t place = std::find(own.workers.begin(), own.workers.end(), (int)(w - h->workers.data())) - own.workers.begin();
    for (int i : own.copies) {
        const Worker& x = h->workers[h->gangs[i].workers[place]];
        if (x.last_request > w->last_request || (x.last_request == w->last_request && x.last_first > w->last_first)) w = &x;
    }
    if (n_images <= 0 || n_images > w->last_nb) return ENS_E_INVALID;
    if (w->input_only) {                                         // the batch ran in LDS: its layers once more, up to the head, as launches
        Gang& g = h->gangs[w->gang];
        if (g.stale) {
            const int rc = build_launches(h, g, false);
            if (rc != ENS_OK) return rc;
        }
        for (const Launch& L : g.plan_for(w->last_nb).launches)
            if (L.kind != L_SKIP && L.kind != L_FC) HIP_TRY(issue(L, m.bf16, (int)g.workers.size(), w->last_nb, 0, h->lanes[0]));
        HIP_TRY(hipStreamSynchronize(h->lanes[0]));
        for (int i : g.workers) h->workers[i].input_only = false;
    }
    const TensorInfo& ti = m.tensors[tensor];
    std::vector<uint8_t> raw(ti.bytes(n_images));
    if (!w->last_programs.empty()) {
        const Chain& c = h->chains[member];
        if (c.place[tensor] == SIZE_MAX) return ENS_E_INVALID;
        for (const ChainProgram& p : w->last_programs) {
            const int images = std::min((int)p.images, n_images - p.first);
            if (images <= 0) continue;
            HIP_TRY(hipMemcpy(raw.data() + ti.bytes(p.first), w->arena + p.first * c.image_bytes + p.images * c.place[tensor], ti.bytes(images), hipMemcpyDeviceToHost));
        }
    } else {
        if (tensor == 0) w = &h->workers[h->gangs[w->gang].workers[0]];   // the staged input lives with the gang's leader
        HIP_TRY(hipMemcpy(raw.data(), w->arena + w->layout.offset[tensor], raw.size(), hipMemcpyDeviceToHost));
    }
    const size_t pixels = (size_t)n_images * ti.h * ti.w;
    for (size_t p = 0; p < pixels; p++)
        for (int c = 0; c < ti.c; c++) {
            float v;
            if (ti.f32) {
                v = ((const float*)raw.data())[p * ti.cs + c];
            } else {
                const uint32_t u = ((uint32_t)((const uint16_t*)raw.data())[p * ti.cs + c]) << 16;
                memcpy(&v, &u, 4);
            }
            out[p * ti.c + c] = v;
        }
    return ENS_OK;
}

int ens_debug_keep_tensors(ens_handle* h, int32_t on) {
    if (!h) return ENS_E_INVALID;
    h->keep_tensors = on != 0;
    return ENS_OK;
}

int ens_classes(const ens_handle* h) { return h ? h->classes : ENS_E_INVALID; }
int ens_n_members(const ens_handle* h) { return h ? (int)h->members.size() : ENS_E_INVALID; }

int ens_member_bytes(const ens_handle* h, int32_t member, int32_t batch, int64_t* weight_bytes, int64_t* arena_bytes) {
    if (!h || member < 0 || member >= (int)h->members.size() || batch <= 0) return ENS_E_INVALID;
    if (weight_bytes) *weight_bytes = (int64_t)h->members[member].weight_bytes();
    if (arena_bytes) *arena_bytes = (int64_t)plan_arena(h->members[member], batch).bytes;
    return ENS_OK;
}

int ens_spec_bytes(const ens_member_spec* spec, int32_t batch, int64_t* weight_bytes, int64_t* arena_bytes) {
    if (!spec || batch <= 0) return ENS_E_INVALID;
    std::vector<float> zeros;
    const float* params = spec->params;
    if (!params) {
        if (spec->n_params <= 0) return ENS_E_INVALID;
        zeros.assign((size_t)spec->n_params, 0.f);
        params = zeros.data();
    }
    Member m;
    const int rc = build_member(*spec, params, &m);
    if (rc != ENS_OK) return rc;
    if (weight_bytes) *weight_bytes = (int64_t)m.weight_bytes();
    if (arena_bytes) *arena_bytes = (int64_t)plan_arena(m, batch).bytes;
    return ENS_OK;
}

int ens_debug_fake_predictor(ens_handle* h, int32_t on) {
    if (!h) return ENS_E_INVALID;
    h->fake_predictor = on != 0;
    return ENS_OK;
}

int ens_set_combination(ens_handle* h, int32_t rule, const float* weights) {
    if (!h) return ENS_E_INVALID;
    if (rule != ENS_COMBINE_MEAN && rule != ENS_COMBINE_WEIGHTED && rule != ENS_COMBINE_VOTE) return ENS_E_INVALID;
    if (rule == ENS_COMBINE_WEIGHTED) {
        if (!weights) return ENS_E_INVALID;
        if (!h->d_weights) HIP_TRY(hipMalloc((void**)&h->d_weights, ENS_MAX_MEMBERS * sizeof(float)));
        HIP_TRY(hipMemcpy(h->d_weights, weights, h->members.size() * sizeof(float), hipMemcpyHostToDevice));
    }
    h->combine_rule = rule;
    drop_graphs(h);                                              // they end in the combination
    return ENS_OK;
}

int ens_debug_one_stream(ens_handle* h, int32_t on) {
    if (!h) return ENS_E_INVALID;
    (void)hipDeviceSynchronize();
    h->one_stream = on != 0;
    return ENS_OK;
}

int ens_debug_rows(ens_handle* h, int32_t on) {
    if (!h) return ENS_E_INVALID;
    if (h->no_rows != (on == 0)) drop_graphs(h);                 // they hold launches of the other kind
    h->no_rows = on == 0;
    return ENS_OK;
}

int ens_debug_stats(const ens_handle* h, ens_stats* out) {
    if (!h || !out) return ENS_E_INVALID;
    *out = h->stats;
    out->graphs = (int64_t)h->graphs.size();
    out->copies = (int64_t)h->gangs.size() - h->own_gangs;
    out->copy_bytes = copy_bytes(h);
    return ENS_OK;
}

int ens_set_profiling(ens_handle* h, int32_t on) {
    if (!h) return ENS_E_INVALID;
    h->profiling = on != 0;
    return ENS_OK;
}

int ens_profile_get(const ens_handle* h, int32_t idx, char* name, int32_t name_len, double* ms, int64_t* launches,
                    double* flop, double* bytes) {
    if (!h || idx < 0 || idx >= (int)h->prof.size()) return ENS_E_INVALID;
    const ProfClass& c = h->prof[idx];
    if (name && name_len > 0) {
        strncpy(name, c.name.c_str(), (size_t)name_len - 1);
        name[name_len - 1] = 0;
    }
    if (ms) *ms = c.ms;
    if (launches) *launches = c.launches;
    if (flop) *flop = c.flop;
    if (bytes) *bytes = c.bytes;
    return ENS_OK;
}

double ens_last_ms(const ens_handle* h) { return h ? h->last_ms : 0.0; }

const char* ens_strerror(int status) {
    switch (status) {
        case ENS_OK: return "ok";
        case ENS_E_INVALID: return "invalid description, matrix or argument";
        case ENS_E_NOMEM: return "not enough device memory for a member or worker";
        case ENS_E_NOFIT: return "no device has enough memory for a member";
        case ENS_E_HIP: return "HIP runtime error";
        case ENS_E_NODEVICE: return "no GPU visible";
        case ENS_E_UNSUPPORTED: return "shape not covered by the GPU kernels";
        case ENS_E_TOOBIG: return "request larger than the static scratch of the allocation-free entry point";
    }
    return "unknown status";
}

const char* ens_version(void) { return "ens-mi355x 0.1 (gfx950)"; }

}  // extern "C"

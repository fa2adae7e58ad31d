// Host side of the chains (chain.h): a member's operations as phases of steps that do not depend on each other, the places of its
// tensors by the phases they live in, and the tiles of its convolutions.  No GPU calls in this file.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>

#include "chain.h"

namespace ens {

namespace {

// What a step reads or writes: channels [lo, hi) of a tensor whose pixels are `stride` elements apart.
struct Access { int tensor, lo, hi, stride; bool write; };
struct Node {
    ChainStep s;
    int kh = 1, kw = 1, sh = 1, sw = 1, pt = 0, pl = 0, act = 0, s2d = 0;   // packed into the step in the end
    std::vector<Access> acc;
    int level = 0;
    bool pack = false;       // a convolution whose weights are not in operand order
};

bool depends(const Node& later, const Node& earlier) {
    for (const Access& a : later.acc)
        for (const Access& b : earlier.acc)
            if (a.tensor == b.tensor && (a.write || b.write) && (a.stride != b.stride || (a.lo < b.hi && b.lo < a.hi))) return true;
    return false;
}

constexpr int GROUP = 32;                    // compute units of an XCD

// What a convolution takes on one group, in microseconds: rounds of workgroups, and in each the chunks of 64 along K of a wavefront, one
// after the other.  Fitted to the phases of nine networks on 1 to 8 images with each tile and split forced in turn (11 352 of them, half
// of them within 9 %); what it picks for a layer by itself is within 1 % of the best there (several in a phase: suit_sides).  A phase costs another PHASE_US.
constexpr double PHASE_US = 1.85;
double conv_us(const ChainStep& s, int images, int side, int lg) {
    const double P = (double)images * s.px;
    const int split = 1 << lg, chunks = (s.K + 63) / 64, per = (chunks + split - 1) / split;
    const double tiles = std::ceil(P / (32 * side)) * s.ctiles[side - 1], rounds = std::ceil(std::ceil(tiles * split / CHAIN_WAVES) / GROUP);
    const double busy = std::min(1.0, std::max(1.0 / CHAIN_WAVES, tiles * split / (GROUP * CHAIN_WAVES)));
    return rounds * (side == 1 ? 1.55 + per * (0.46 + 0.13 * busy) : 2.2 + per * (1.03 + 0.19 * busy));
}

// Pixels of a depthwise strip's window in LDS: its rows and, for whole runs of four outputs, its columns.
int dw_slots(const ChainStep& s) {
    const int h_per = (s.Ho + s.rows - 1) / s.rows, k = s.window & 255, st = s.stride & 255;
    return ((h_per - 1) * st + k) * (((s.Wo + 3) / 4 * 4 - 1) * st + k);
}

double weight_bytes(const ChainStep& s) {
    switch (s.kind) {
        case CH_CONV:
        case CH_CONV_PRE: return s.wsize;
        case CH_DW: return 2.0 * (s.window & 255) * (s.window & 255) * s.cin;
        case CH_FC: return (double)((s.cout + 31) / 32) * ((s.cin + 63) / 64) * 4096;
        case CH_SE_HIDDEN: return 4.0 * s.cin * s.r;
    }
    return 0.0;
}

// What the kernel works out as chain_units when the images are no power of two.
double units(const ChainStep& s, int images, int pick) {
    const double cb = (s.cin + 63) / 64;
    switch (s.kind) {
        case CH_STAGE: return images * std::ceil((double)s.Ho * s.Wo / CHAIN_THREADS);
        case CH_CONV:
        case CH_CONV_PRE: {
            const int side = pick & 255;
            return std::ceil(std::ceil((double)images * s.px / (32 * side)) * s.ctiles[side - 1] * (1 << (pick >> 8 & 255)) / CHAIN_WAVES);
        }
        case CH_DW: return images * s.rows * cb;
        case CH_MAXPOOL:
        case CH_AVGPOOL: return std::ceil((double)images * s.Ho * s.Wo * (s.cin / 8) / (CH_POOL * CHAIN_THREADS));
        case CH_SE_SUM:
        case CH_GAP: return images * cb;
        case CH_SE_HIDDEN: return images * ((s.r + CHAIN_WAVES - 1) / CHAIN_WAVES);
        case CH_SE_APPLY: return images * s.sub * cb;
        case CH_FC: return ((s.cout + 31) / 32) * ((images + 31) / 32);
    }
    return 0.0;
}

// What a step takes on one group beside the phase's own time, in microseconds (fitted as conv_us is: within 2 to 20 %).
double step_us(const ChainStep& s, int images, int size) {
    const double all = std::ceil(units(s, images, s.choice[size]) / GROUP);
    switch (s.kind) {
        case CH_CONV:
        case CH_CONV_PRE: return conv_us(s, images, s.choice[size] & 255, s.choice[size] >> 8 & 255);
        case CH_STAGE: return 1.4 * all;
        case CH_DW: {
            const int k = s.window & 255;
            const double items = std::ceil(std::ceil((double)s.Ho / s.rows) * ((s.Wo + 3) / 4) / 64);
            return all * (1.6 + 0.0034 * dw_slots(s) + items * (k == 3 ? 1.5 : 3.7) + (s.scratch >= 0 ? 1.3 : 0.0));
        }
        case CH_MAXPOOL: return 1.6 + 3.7 * all;
        case CH_AVGPOOL: return 5.1 * all;
        case CH_SE_SUM:
        case CH_GAP: return 2.0 * all;
        case CH_SE_HIDDEN: return all * (0.8 + s.cin / 320.0);
        case CH_SE_APPLY: return all * (2.2 + s.r / 500.0 + 0.0016 * s.H * s.W / s.sub);
        case CH_FC: return 1.0 + all * s.cin / 450.0;
    }
    return 0.0;
}

// What a phase takes on one group beside its own time: its units are dealt to the workgroups in turn, whatever step they are of.
double phase_us(const ChainStep* steps, int count, int images, int size) {
    double load[GROUP] = {0};
    int at = 0;
    for (int i = 0; i < count; i++) {
        const double n = units(steps[i], images, steps[i].choice[size]), whole = std::floor(n / GROUP);
        const double each = step_us(steps[i], images, size) / std::max(1.0, std::ceil(n / GROUP));
        for (double& l : load) l += whole * each;
        for (int u = 0; u < (int)(n - whole * GROUP); u++, at = (at + 1) % GROUP) load[at] += each;
    }
    return *std::max_element(load, load + GROUP);
}

constexpr double MOST_UNITS = 65535.0;       // of a step, in 16 bits of its choice

// The tiles that take a convolution the least time by itself.
int own_tiles(const ChainStep& s, int images) {
    int pick = 0;
    double best = 1e30;
    for (int side = 1; side <= 2; side++)
        for (int split = 0; 1 << split <= CHAIN_WAVES; split++) {
            if (side == 2 && s.sub > 1) continue;
            const double us = conv_us(s, images, side, split);
            if (us < best) { best = us; pick = side | split << 8; }
        }
    return pick;
}

// Several steps of a phase share the workgroups, so that the best tiles of each by itself can make two rounds where larger ones make one (a module's
// branches; a layer and its shortcut, 26 and 25 units): every convolution in turn is given the side of tiles that suits the others'.  The parts
// that its K is cut into stay its own, since its sums are added up in them: a layer's answer does not depend on what runs beside it.
// (An Inception-shaped member on 1 to 16 images 4.5 % faster, four members on 4 images 2 %; members whose phases hold one convolution or two unchanged.)
void suit_sides(ChainStep* steps, int count, int size) {
    const int images = 1 << size;
    double us = phase_us(steps, count, images, size);
    for (bool moved = true; moved;) {
        moved = false;
        for (int i = 0; i < count; i++) {
            ChainStep& s = steps[i];
            if (s.kind > CH_CONV_PRE || s.sub > 1) continue;
            const int was = s.choice[size];
            s.choice[size] = was ^ 3;
            const double t = phase_us(steps, count, images, size);
            if (t < us - 1e-6 && units(s, images, s.choice[size]) <= MOST_UNITS) { us = t; moved = true; }
            else s.choice[size] = was;
        }
    }
}

}  // namespace

int chain_size(int images) {
    int z = 0;
    while (z + 1 < CHAIN_SIZES && (1 << z) < images) z++;
    return z;
}

bool build_chain(const Member& m, const std::vector<Launch>& launches, char* base, const std::vector<size_t>& at, size_t arena_bytes, int batch,
                 Chain* out) {
    if (!m.bf16) return false;
    auto tensor_at = [&](const void* p) {
        const size_t off = (size_t)((const char*)p - base);
        for (size_t t = 0; t < at.size(); t++)
            if (!m.tensors[t].external && m.tensors[t].def != INT32_MAX && at[t] == off) return (int)t;
        return -1;
    };
    std::vector<Node> nodes;
    std::vector<int> scratch_floats(m.tensors.size(), 0);        // of a squeeze-excite block's scratch, with the rows of sums that it has here
    bool ok = true;
    // the slice of view `v` that is `c` channels wide, for reading or writing; its tensor (whose place is filled in below)
    auto touch = [&](Node& n, const View& v, int c, bool write) -> int64_t {
        const int t = tensor_at(v.p);
        if (t < 0) ok = false;
        n.acc.push_back(Access{t, v.c0, v.c0 + c, v.stride, write});
        return t;
    };
    auto blank = [](int kind) {
        Node n;
        memset((void*)&n.s, 0, sizeof(n.s));
        n.s.kind = kind;
        n.s.res = n.s.scratch = -1;
        n.s.sub = 1;
        return n;
    };
    auto pack = [&](Node& n) {
        ok = ok && n.kh < 256 && n.kw < 256 && n.pt < 256 && n.pl < 256 && n.sh < 256 && n.sw < 256;
        n.s.window = n.kh | n.kw << 8 | n.pt << 16 | (int)((unsigned)n.pl << 24);
        n.s.stride = n.sh | n.sw << 8 | n.act << 16 | n.s2d << 24;
    };
    {
        Node n = blank(CH_STAGE);                                // tensor 0 as the staging kernels write it
        const TensorInfo& t0 = m.tensors[0];
        n.s.H = m.in_h; n.s.W = m.in_w; n.s.Ho = t0.h; n.s.Wo = t0.w; n.s.ys = t0.cs; n.s2d = m.stem_s2d ? 1 : 0;
        if (t0.cs != (m.stem_s2d ? 16 : 8)) return false;
        n.s.y = touch(n, View{base + at[0], t0.cs, 0}, t0.cs, true);
        nodes.push_back(n);
    }
    for (size_t i = 0; i < launches.size() && ok; i++) {
        const Launch& L = launches[i];
        switch (L.kind) {
            case L_CONV: {
                const ConvArgs& a = L.conv;
                const int K = a.kh * a.kw * a.cin;
                if (a.gate || a.cin % 8 || a.cout % 8 || a.H > 16384 || a.W > 16384) return false;
                if (a.pre_scale && (a.kh != 1 || a.kw != 1 || a.pt || a.pl || 2 * ((K + 63) / 64 * 64) > CHAIN_TABLE_FLOATS || L.sub > 1)) return false;
                Node n = blank(a.pre_scale ? CH_CONV_PRE : CH_CONV);
                ChainStep& s = n.s;
                s.x = touch(n, a.x, a.cin * L.sub, false);
                s.y = touch(n, a.y, a.cout * L.sub, true);
                if (a.res.p) s.res = touch(n, a.res, a.cout * L.sub, false);
                s.xs = a.x.stride; s.xc0 = a.x.c0; s.ys = a.y.stride; s.yc0 = a.y.c0; s.rs = a.res.stride; s.rc0 = a.res.c0;
                s.w = a.wpk ? a.wpk : a.w; s.bias = a.bias; s.scale = a.scale; s.pre_scale = a.pre_scale; s.pre_shift = a.pre_shift;
                n.pack = !a.wpk;
                s.H = a.H; s.W = a.W; s.Ho = a.Ho; s.Wo = a.Wo; s.cin = a.cin; s.cout = a.cout;
                s.px = a.Ho * a.Wo;
                s.res_present = a.res.p != nullptr;
                s.padded = a.pt || a.pl || (a.Ho - 1) * a.sh + a.kh > a.H || (a.Wo - 1) * a.sw + a.kw > a.W;
                if (s.padded && a.kh * a.kw > 32) return false;  // a bit per tap
                const double wsize = (double)L.sub * ((a.cout + 31) / 32) * ((K + 63) / 64) * 4096;
                if (wsize >= 0x7FFFFF00LL) return false;
                s.wsize = (int)wsize;
                n.kh = a.kh; n.kw = a.kw; n.sh = a.sh; n.sw = a.sw; n.pt = a.pt; n.pl = a.pl; n.act = a.act;
                s.sub = L.sub;
                s.K = K;
                nodes.push_back(n);
                break;
            }
            case L_DWCONV:
            case L_POOL: {
                const PoolArgs& a = L.pool;
                if (a.c % 8) return false;
                if (L.kind == L_DWCONV && (a.kh != a.kw || (a.kh != 3 && a.kh != 5) || a.sh != a.sw || (a.sh != 1 && a.sh != 2))) return false;
                Node n = blank(L.kind == L_DWCONV ? CH_DW : L.is_max ? CH_MAXPOOL : CH_AVGPOOL);
                ChainStep& s = n.s;
                s.x = touch(n, a.x, a.c, false);
                s.y = touch(n, a.y, a.c, true);
                s.xs = a.x.stride; s.xc0 = a.x.c0; s.ys = a.y.stride; s.yc0 = a.y.c0;
                s.w = a.w; s.bias = a.bias; s.scale = a.scale; s.pre_scale = a.pre_scale; s.pre_shift = a.pre_shift;
                s.H = a.H; s.W = a.W; s.Ho = a.Ho; s.Wo = a.Wo; s.cin = s.cout = a.c;
                n.kh = a.kh; n.kw = a.kw; n.sh = a.sh; n.sw = a.sw; n.pt = a.pt; n.pl = a.pl; n.act = a.act;
                pack(n);
                if (L.kind == L_DWCONV) {
                    const Launch* next = i + 1 < launches.size() && launches[i + 1].kind == L_SE ? &launches[i + 1] : nullptr;
                    const bool sums = next && next->se.x.p == a.y.p && next->se.x.c0 == a.y.c0 && next->se.c == a.c;
                    // strips of rows: the window of one fits LDS, and the group has the least to do
                    if (sums) s.scratch = tensor_at(next->se.scratch);
                    if (sums && s.scratch < 0) return false;
                    double best = 1e30;
                    for (int rows = 1; rows <= a.Ho; rows++) {
                        s.rows = rows;
                        const double us = step_us(s, 1, 0);
                        if (dw_slots(s) <= CHAIN_DW_SLOTS && us < best) { best = us; s.r = rows; }
                    }
                    if (best == 1e30) return false;
                    s.rows = s.r;
                    s.r = 0;
                    if (sums) {
                        s.scratch_stride = se_scratch_floats(a.c, next->se.r, s.rows);
                        n.acc.push_back(Access{(int)s.scratch, 0, s.rows * a.c, 1, true});
                    }
                }
                nodes.push_back(n);
                break;
            }
            case L_SE: {
                const SeArgs& a = L.se;
                if (a.c % 8 || a.c > CHAIN_TABLE_FLOATS || a.r > CHAIN_TABLE_FLOATS - 1024) return false;
                const int t = tensor_at(a.scratch);
                if (t < 0) return false;
                const bool have = !nodes.empty() && nodes.back().s.kind == CH_DW && nodes.back().s.scratch == t;
                const int rows = have ? nodes.back().s.rows : 1, sums = rows * a.c;
                scratch_floats[t] = se_scratch_floats(a.c, a.r, rows);
                Node n = blank(CH_SE_SUM);
                ChainStep& s = n.s;
                s.scratch = t;
                s.scratch_stride = scratch_floats[t];
                s.hidden_at = sums;
                s.xs = a.x.stride; s.xc0 = a.x.c0; s.ys = a.y.stride; s.yc0 = a.y.c0;
                s.w = a.w1; s.bias = a.b1; s.scale = a.w2; s.pre_scale = a.b2;
                const TensorInfo& tx = m.tensors[std::max(0, tensor_at(a.x.p))];
                s.H = s.Ho = tx.h; s.W = s.Wo = tx.w; s.cin = s.cout = a.c; s.r = a.r;
                s.rows = rows;
                if (!have) {
                    s.x = touch(n, a.x, a.c, false);
                    n.acc.push_back(Access{t, 0, sums, 1, true});
                    nodes.push_back(n);
                }
                Node hidden = blank(CH_SE_HIDDEN);
                hidden.s = s;
                hidden.s.kind = CH_SE_HIDDEN;
                hidden.acc.push_back(Access{t, 0, sums, 1, false});
                hidden.acc.push_back(Access{t, sums, sums + a.r, 1, true});
                nodes.push_back(hidden);
                Node apply = blank(CH_SE_APPLY);
                apply.s = s;
                apply.s.kind = CH_SE_APPLY;
                apply.s.x = touch(apply, a.x, a.c, false);
                apply.s.y = touch(apply, a.y, a.c, true);
                apply.acc.push_back(Access{t, sums, sums + a.r, 1, false});
                apply.s.sub = std::max(1, std::min((tx.h * tx.w + 63) / 64, (2 * GROUP + (a.c + 63) / 64 - 1) / ((a.c + 63) / 64)));
                nodes.push_back(apply);
                break;
            }
            case L_GAP: {
                const GapArgs& a = L.gap;
                const int t = tensor_at(a.y);                    // (a slice that does not begin its tensor is found nowhere)
                if (t < 0 || a.c % 8) return false;
                Node n = blank(CH_GAP);
                ChainStep& s = n.s;
                s.x = touch(n, a.x, a.c, false);
                s.y = t;
                n.acc.push_back(Access{t, 0, a.c, 1, true});
                const TensorInfo& tx = m.tensors[std::max(0, tensor_at(a.x.p))];
                s.H = tx.h; s.W = tx.w; s.cin = a.c;
                s.xs = a.x.stride; s.xc0 = a.x.c0; s.ys = a.c;
                s.pre_scale = a.pre_scale; s.pre_shift = a.pre_shift;
                nodes.push_back(n);
                break;
            }
            case L_FC: {
                const FcArgs& a = L.fc;
                const int t = tensor_at(a.x);
                if (t < 0 || !a.wpk || a.cin % 8) return false;
                Node n = blank(CH_FC);
                n.s.x = t;
                n.acc.push_back(Access{t, 0, a.cin, 1, false});
                n.s.w = a.wpk; n.s.bias = a.bias; n.s.cin = a.cin; n.s.cout = a.cout;
                nodes.push_back(n);
                break;
            }
            default: return false;
        }
    }
    if (!ok) return false;
    for (Node& n : nodes) {
        ChainStep& s = n.s;
        pack(n);
        for (int i = 0; i < 2; i++) {
            s.ctiles[i] = (s.cout + 32 * i + 31) / (32 * (i + 1)) * s.sub;
            s.inv_ctiles[i] = 1.f / std::max(1, s.ctiles[i]);
        }
        s.inv_wo = 1.f / std::max(1, s.Wo); s.inv_ho = 1.f / std::max(1, s.Ho);
        s.inv_cin = 1.f / std::max(1, s.cin); s.inv_kw = 1.f / n.kw;
    }
    if (!ok) return false;
    // phases: every step right behind the last of those that it depends on
    int phases = 0;
    for (size_t i = 0; i < nodes.size(); i++) {
        for (size_t j = 0; j < i; j++)
            if (nodes[j].level >= nodes[i].level && depends(nodes[i], nodes[j])) nodes[i].level = nodes[j].level + 1;
    }
    std::stable_sort(nodes.begin(), nodes.end(), [](const Node& a, const Node& b) { return a.level < b.level; });
    for (size_t i = 0, level = 0, steps = 0, was = 0; i < nodes.size(); i++) {   // as many steps as a phase holds
        if (i > 0 && ((size_t)nodes[i].level != was || steps == CHAIN_PHASE_STEPS)) { level++; steps = 0; }
        was = (size_t)nodes[i].level;
        nodes[i].level = (int)level;
        steps++;
        phases = (int)level + 1;
    }
    if (phases < 2) return false;
    // places: the lowest that is free in all phases from the first to the last that touches the tensor
    const int NT = (int)m.tensors.size();
    std::vector<int> def(NT, INT32_MAX), last(NT, -1), order;
    for (const Node& n : nodes)
        for (const Access& a : n.acc) {
            def[a.tensor] = std::min(def[a.tensor], n.level);
            last[a.tensor] = std::max(last[a.tensor], n.level);
        }
    for (int t = 0; t < NT; t++)
        if (last[t] >= 0) order.push_back(t);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return def[a] < def[b]; });
    out->place.assign(NT, SIZE_MAX);
    out->image_bytes = 0;
    auto size_of = [&](int t) { return ((scratch_floats[t] ? scratch_floats[t] * sizeof(float) : m.tensors[t].bytes(1)) + 255) / 256 * 256; };
    for (size_t i = 0; i < order.size(); i++) {
        const int t = order[i];
        std::vector<std::pair<size_t, size_t>> busy;
        for (size_t j = 0; j < i; j++) {
            const int u = order[j];
            if (def[u] <= last[t] && def[t] <= last[u]) busy.push_back({out->place[u], out->place[u] + size_of(u)});
        }
        std::sort(busy.begin(), busy.end());
        size_t off = 0;
        for (const auto& b : busy) {
            if (off + size_of(t) <= b.first) break;
            off = std::max(off, b.second);
        }
        out->place[t] = off;
        out->image_bytes = std::max(out->image_bytes, off + size_of(t));
    }
    out->cap = (int)std::min<size_t>((size_t)batch, arena_bytes / out->image_bytes);
    if (out->cap < 1) return false;
    // 32-bit offsets with 2^31 standing for 'outside', quotients by float reciprocals, 24-bit products
    for (const Node& n : nodes) {
        const ChainStep& s = n.s;
        const double bytes = std::max((double)s.H * s.W * s.xs, (double)s.Ho * s.Wo * std::max(s.ys, s.rs)) * 2;
        const double items = (double)s.Ho * s.Wo * (s.kind <= CH_CONV_PRE ? 1 : std::max(1, s.cin / 8));
        out->cap = (int)std::min({(double)out->cap, 2147483000.0 / std::max(1.0, bytes), 8388607.0 / std::max(1.0, items)});
        if (s.kind == CH_FC && (double)((s.cout + 31) / 32) * ((s.cin + 63) / 64) * 4096 >= 0x7FFFFF00LL) return false;
    }
    // what a launch is told of a program in 32 and in 16 bits
    if (out->image_bytes > UINT32_MAX) return false;
    out->cap = std::min(out->cap, (int)INT16_MAX);
    if (out->cap < 1) return false;
    out->steps.clear();
    out->packs.clear();
    out->pack_bytes = 0;
    out->phases = phases;
    for (int z = 0; z < CHAIN_SIZES; z++) out->seconds[z] = out->span[z] = 0.0;
    for (size_t i = 0; i < nodes.size();) {
        size_t e = i;
        while (e < nodes.size() && nodes[e].level == nodes[i].level) e++;
        for (size_t j = i; j < e; j++) {
            ChainStep s = nodes[j].s;
            auto place = [&](int64_t t) { return t >= 0 ? (int64_t)out->place[t] : (int64_t)-1; };
            if (j == i) {
                size_t f = e;
                std::vector<std::pair<double, const void*>> next;
                for (; f < nodes.size() && nodes[f].level == nodes[e].level; f++) next.emplace_back(weight_bytes(nodes[f].s), nodes[f].s.w);
                s.phase_steps = (int)(e - i) | (int)(f - e) << 8;
                std::sort(next.begin(), next.end(), std::greater<>());
                for (size_t k = 0; k < 2 && k < next.size(); k++) {
                    s.ahead[k] = next[k].second;
                    s.ahead_bytes[k] = (int)std::min(next[k].first, 2e9);
                }
            }
            if (s.kind != CH_SE_HIDDEN && s.kind != CH_STAGE) s.x = place(s.x);
            if (s.kind != CH_SE_SUM && s.kind != CH_SE_HIDDEN && s.kind != CH_FC) s.y = place(s.y);
            s.res = place(s.res);
            s.scratch = place(s.scratch);
            for (int z = 0; z < CHAIN_SIZES; z++) {
                if (s.kind <= CH_CONV_PRE) s.choice[z] = own_tiles(s, 1 << z);
                if (units(s, 1 << z, s.choice[z]) > MOST_UNITS) return false;
                out->seconds[z] += 1e-6 * step_us(s, 1 << z, z);
            }
            if (nodes[j].pack) {
                out->packs.push_back(Chain::Pack{(int)out->steps.size(), s.sub, s.cout, s.K, out->pack_bytes, (size_t)s.wsize});
                out->pack_bytes += ((size_t)s.wsize + 255) / 256 * 256;
            }
            out->steps.push_back(s);
        }
        ChainStep* const phase = &out->steps[out->steps.size() - (e - i)];
        for (int z = 0; z < CHAIN_SIZES; z++) {
            if (e - i > 1) suit_sides(phase, (int)(e - i), z);
            out->seconds[z] += 1e-6 * PHASE_US;
            out->span[z] += 1e-6 * (PHASE_US + phase_us(phase, (int)(e - i), 1 << z, z));
            for (size_t j = 0; j < e - i; j++) phase[j].choice[z] |= (int)units(phase[j], 1 << z, phase[j].choice[z]) << 16;
        }
        i = e;
    }
    return true;
}

}  // namespace ens

// Host side of the resident members (resident.h): their operations, weights and tables as LDS holds them.  No GPU calls in this file.
#include <algorithm>
#include <cstring>

#include "resident.h"

namespace ens {

static bool build(const Member& m, Resident* out, bool pairs) {
    if (m.bf16 || m.ops.size() > RESIDENT_MAX_OPS) return false;
    const int NT = (int)m.tensors.size(), NO = (int)m.ops.size();
    // what a convolution's taps reach around a tensor
    struct Pad { int t = 0, b = 0, l = 0, r = 0; bool any() const { return t || b || l || r; } };
    std::vector<Pad> pad(NT);
    std::vector<int> def(NT, -1), last(NT, -1);
    for (int i = 0; i < NO; i++) {
        const OpPlan& pl = m.ops[i];
        const ens_op& o = pl.op;
        const TensorInfo &ts = m.tensors[o.src], &td = m.tensors[o.dst];
        if (o.kind != ENS_OP_CONV && o.kind != ENS_OP_MAXPOOL && o.kind != ENS_OP_AVGPOOL && o.kind != ENS_OP_GAP && o.kind != ENS_OP_FC) return false;
        // whole tensors, each written once, no residuals, groups or pre-activations
        if (o.src_c0 || o.dst_c0 || o.cin != ts.c || o.cout != td.c || def[o.dst] >= 0 || o.dst == 0 || (o.src != 0 && def[o.src] < 0)) return false;
        if (o.kind == ENS_OP_CONV && (o.res >= 0 || o.pre || pl.sub > 1)) return false;
        if (o.kind == ENS_OP_GAP && o.pre) return false;
        if ((long long)td.h * td.w * td.c >= (1 << 20) || (long long)ts.h * ts.w * ts.c >= (1 << 20)) return false;
        def[o.dst] = i;
        last[o.src] = i;
        if (o.kind == ENS_OP_CONV) {
            Pad& p = pad[o.src];
            p.t = std::max(p.t, o.pt);
            p.l = std::max(p.l, o.pl);
            p.b = std::max(p.b, (td.h - 1) * o.sh + o.kh - o.pt - ts.h);
            p.r = std::max(p.r, (td.w - 1) * o.sw + o.kw - o.pl - ts.w);
        }
    }
    if (m.ops.back().op.kind != ENS_OP_FC || m.ops.back().op.dst != m.out_tensor) return false;
    // A convolution whose output goes into 2 x 2 / 2 windows, all of them inside, or into the mean, and nowhere else takes that along
    std::vector<int> pool(NO, RS_NO_POOL), readers(NT, 0);
    std::vector<char> gone(NO, 0);                               // operations that run with the one before
    for (int i = 0; i < NO; i++) readers[m.ops[i].op.src]++;
    for (int i = 0; i + 1 < NO; i++) {
        const ens_op &o = m.ops[i].op, &q = m.ops[i + 1].op;
        if (o.kind != ENS_OP_CONV || q.src != o.dst || readers[o.dst] != 1) continue;
        const TensorInfo &ts = m.tensors[o.dst], &td = m.tensors[q.dst];
        const bool windows = q.kh == 2 && q.kw == 2 && q.sh == 2 && q.sw == 2 && q.pt == 0 && q.pl == 0 && td.h * 2 <= ts.h && td.w * 2 <= ts.w;
        if (q.kind == ENS_OP_GAP) pool[i] = RS_MEAN_POOL;
        else if (q.kind == ENS_OP_MAXPOOL && windows) pool[i] = RS_MAX_POOL;
        else if (q.kind == ENS_OP_AVGPOOL && windows) pool[i] = RS_AVG_POOL;
        else continue;
        gone[i + 1] = 1;
        def[o.dst] = -1;                                         // never in LDS
        def[q.dst] = i;
    }
    // LDS begins with the operations, then weights, biases and tap tables
    std::vector<float>& fixed = out->fixed;
    fixed.assign((size_t)NO * 64, 0.f);
    std::vector<ResidentOp> ops(NO);
    const float* const P = (const float*)m.host_params.data();
    auto pitch = [](int c) { const int p = (c + 3) / 4 * 4; return p % 8 == 0 ? p + 4 : p; };   // a pixel's floats: pixels side by side on different banks
    double macs = 0;
    for (int i = 0; i < NO; i++) {
        const OpPlan& pl = m.ops[i];
        const ens_op& o = pl.op;
        ResidentOp& r = ops[i];
        memset((void*)&r, 0, sizeof(r));
        const TensorInfo &ts = m.tensors[o.src], &td = m.tensors[o.dst];
        r.kind = o.kind == ENS_OP_CONV ? RS_CONV : o.kind == ENS_OP_MAXPOOL ? RS_MAXPOOL : o.kind == ENS_OP_AVGPOOL ? RS_AVGPOOL : o.kind == ENS_OP_GAP ? RS_GAP : RS_FC;
        r.H = ts.h; r.W = ts.w; r.cin = o.cin; r.Ho = td.h; r.Wo = td.w; r.cout = o.cout;
        r.kh = o.kh; r.kw = o.kw; r.sh = o.sh; r.sw = o.sw; r.pt = o.pt; r.pl = o.pl; r.act = o.act;
        if (o.kind == ENS_OP_CONV) {
            // Up to eight channels leave half of a tile's rows empty: two neighbouring pixels share it, with a column of the filter more.  (A weight of zero
            // meets a pixel of the neighbour's then, which only the request's images are known to have finite: resident_kernel.)
            const bool pair = pairs && o.src == 0 && o.cout <= 8 && o.kw > 1 && o.sw == 1 && (pool[i] == RS_MAX_POOL || pool[i] == RS_AVG_POOL);
            const int kw = o.kw + (pair ? 1 : 0), K = o.kh * kw * o.cin, steps = (K + 3) / 4, tiles = o.cout > 16 ? (o.cout + 31) / 32 * 2 : 1;   // in pairs where there are several
            if ((size_t)tiles * steps * 64 > RESIDENT_LDS / 4) return false;
            r.steps = steps;
            r.w = (int)fixed.size();
            fixed.resize(fixed.size() + (size_t)tiles * steps * 64, 0.f);
            const float* const w = P + pl.w / 4;                 // [K][cout]
            r.pair = pair;
            for (int k = 0; k < o.kh * o.kw * o.cin; k++)
                for (int c = 0; c < o.cout; c++) {
                    const int at = (k / (o.kw * o.cin) * kw + k / o.cin % o.kw) * o.cin + k % o.cin;
                    fixed[(size_t)r.w + ((size_t)(c / 16) * steps * 4 + at) * 16 + c % 16] = w[(size_t)k * o.cout + c];
                    if (pair) fixed[(size_t)r.w + (size_t)(at + o.cin) * 16 + 8 + c] = w[(size_t)k * o.cout + c];
                }
            r.taps = (int)fixed.size();                          // filled in when the tensors have their places
            fixed.resize(fixed.size() + (size_t)steps * 4, 0.f);
            macs += (double)td.h * td.w / (pair ? 2 : 1) * tiles * 16 * steps * 4;
        }
        if (o.kind == ENS_OP_FC) {
            if ((size_t)o.cin * o.cout > RESIDENT_LDS / 4) return false;
            r.w = (int)fixed.size();
            fixed.insert(fixed.end(), P + pl.w / 4, P + pl.w / 4 + (size_t)o.cin * o.cout);
            fixed.resize((fixed.size() + 3) / 4 * 4, 0.f);
        }
        if (o.kind == ENS_OP_CONV || o.kind == ENS_OP_FC) {
            r.bias = (int)fixed.size();
            fixed.insert(fixed.end(), P + pl.b / 4, P + pl.b / 4 + o.cout);
            fixed.resize((fixed.size() + 15) / 16 * 16, 0.f);    // whole fours are read
        }
        if (fixed.size() > RESIDENT_LDS / 4) return false;
    }
    // tensors: those with a border for themselves (the zeros stay), the others where memory is free while they live
    struct Place { int at = -1, p = 0, r = 0, floats = 0; };
    std::vector<Place> place(NT);
    bool fours = false;                              // pooling reads pixels of whole fours
    for (int i = 0; i < NO; i++) fours |= m.ops[i].op.src == 0 && !gone[i] && (m.ops[i].op.kind == ENS_OP_MAXPOOL || m.ops[i].op.kind == ENS_OP_AVGPOOL);
    int top = (int)fixed.size();
    for (int pass = 0; pass < 2; pass++) {
        const int floor = top;
        for (int t = 0; t < NT; t++) {
            if (t != 0 && def[t] < 0) continue;
            if (t == m.out_tensor || pad[t].any() != (pass == 0)) continue;
            const TensorInfo& ti = m.tensors[t];
            Place& q = place[t];
            q.p = t == 0 && !fours ? ti.c : ti.h * ti.w == 1 ? (ti.c + 3) / 4 * 4 : pitch(ti.c);
            q.r = (ti.w + pad[t].l + pad[t].r) * q.p;
            q.floats = (ti.h + pad[t].t + pad[t].b) * q.r + 4;
            q.floats = (q.floats + 3) / 4 * 4;
            int at = pass == 0 ? top : floor;
            if (pass == 1) {
                for (bool moved = true; moved;) {
                    moved = false;
                    for (int u = 0; u < NT; u++) {
                        if (u == t || place[u].at < floor) continue;
                        const bool together = def[u] <= std::max(last[t], def[t]) && def[t] <= std::max(last[u], def[u]);
                        if (together && at < place[u].at + place[u].floats && place[u].at < at + q.floats) { at = place[u].at + place[u].floats; moved = true; }
                    }
                }
            }
            q.at = at;
            top = std::max(top, at + q.floats);
            if ((size_t)top > RESIDENT_LDS / 4) return false;
        }
    }
    for (int i = 0; i < NO; i++) {
        if (gone[i]) continue;
        const ens_op& o = m.ops[i].op;
        ResidentOp& r = ops[i];
        const int dst = pool[i] != RS_NO_POOL ? m.ops[i + 1].op.dst : o.dst;
        const Place &s = place[o.src], &d = place[dst];
        const int origin = s.at + pad[o.src].t * s.r + pad[o.src].l * s.p;
        r.x = o.kind == ENS_OP_CONV ? origin - o.pt * s.r - o.pl * s.p : origin;
        r.xp = s.p; r.xr = s.r;
        r.pool = pool[i];
        if (pool[i] == RS_MEAN_POOL) {
            r.sums = top;
            r.sums_p = (o.cout + 3) / 4 * 4;
            top += (m.tensors[o.dst].h * m.tensors[o.dst].w + 31) / 32 * r.sums_p;   // a unit is 32 pixels
            if ((size_t)top > RESIDENT_LDS / 4) return false;
        } else if (pool[i] != RS_NO_POOL) {
            r.Ho = m.tensors[dst].h;
            r.Wo = m.tensors[dst].w;
        }
        if (dst != m.out_tensor) {
            r.y = d.at + pad[dst].t * d.r + pad[dst].l * d.p;
            r.yp = d.p; r.yr = d.r;
        }
        if (o.kind == ENS_OP_CONV)
            for (int k = 0, kw = o.kw + r.pair; k < o.kh * kw * o.cin; k++) {
                const int c = k % o.cin, tap = k / o.cin;
                const int v = tap / kw * s.r + tap % kw * s.p + c;
                memcpy(&fixed[(size_t)r.taps + k], &v, 4);
            }
    }
    const Place& in = place[0];
    out->in = in.at + pad[0].t * in.r + pad[0].l * in.p;
    out->in_p = in.p;
    out->in_r = in.r;
    out->lds_floats = (top + 3) / 4 * 4;
    out->n_ops = 0;
    for (int i = 0; i < NO; i++)
        if (!gone[i]) memcpy(&fixed[(size_t)out->n_ops++ * 64], &ops[i], sizeof(ResidentOp));
    // the matrix cores' 256 operations a clock and compute unit, and the steps between
    out->seconds = 2.0 * macs / 614e9 / 0.6 + 1e-6 * NO;
    return true;
}

bool build_resident(const Member& m, Resident* out) {
    return build(m, out, true) || build(m, out, false);          // (the pairs' weights are larger)
}

}  // namespace ens

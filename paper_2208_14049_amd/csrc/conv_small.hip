// Convolution on the CDNA4 matrix cores for launches with few output pixels: one image or a handful, where the other
// kernels leave most of the chip idle and a workgroup's life is the serial chain of its K loop (a 14x14x256 3x3 layer on one
// image: 8 workgroups, 36 stages of weights one after the other, 13 us).
//
// GEMM view as everywhere: rows = output pixels, columns = output channels, K = taps x input channels.  A workgroup owns a tile
// of 32 pixels x 32 channels and its NW wavefronts split K: each takes a run of 64-element chunks, both operands by
// asynchronous global-to-LDS loads into a part of LDS that is its own, two chunks ahead, so that a wavefront waits for its own
// loads only and there is no barrier before the end, where the NW partial tiles meet in LDS and are added in wavefront order.
// Up to 128 KB are in flight per compute unit and a layer's whole K is one to five round trips to memory.  (The
// same split with fragments straight from memory to registers was measured first: a lane's 16 bytes of 32 different
// rows cost the load path 64 clocks where whole 128-byte rows cost 16, and 14x14x256 took 12.4 us.)  What the kernel pays is
// load traffic, 64 bytes per 1024 multiply-adds through the compute unit's 64 B/clock path: conv_small_pick takes it while that costs
// less than the chain.
//
// Any filter, stride and padding; pre-activation and squeeze-excite gates of 1x1 layers are applied to the pixel fragments
// between LDS and the matrix cores.  Weights in their plain layout [cout][kh][kw][cin]; rows are read with bits 2 and 3 of their
// number swapped, which makes a lane's 16 results two runs of 8 channels.
#include "conv_direct.h"

namespace ens {

enum { SM_PLAIN = 0, SM_PRE = 1, SM_GATE = 2 };
template <int TP, int TC>
constexpr int sm_stage() { return 32 * (TP + TC) * 128; }   // bytes of a chunk: pixel rows and weight rows of 64 values
constexpr int SM_LDS = 160 * 1024;

// NST: chunks of a wavefront in LDS (the one in use and those ahead).  tab: floats of the table behind the rings (pre-activation:
// scale, then shift of every input channel; gates: those of the images a tile touches).
template <int TP, int TC, int NW, int NST, bool TAPS, int MODE>
__global__ __launch_bounds__(64 * NW) void conv_small_bf16(const ConvArgs* __restrict__ argv, const int nb_) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const ConvArgs a = argv[blockIdx.z];
    constexpr int T = 64 * NW, BP = 32 * TP, BC = 32 * TC, SM_STAGE = sm_stage<TP, TC>(), XB = BP * 128;
    constexpr unsigned OOBV = 0x80000000u;           // past the end of every buffer the launcher admits: zeros
    const int P = nb_ * a.Ho * a.Wo, K = a.kh * a.kw * a.cin;
    const int t = threadIdx.x, lane = t & 63, lrow = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int n_ctiles = (a.cout + BC - 1) / BC;
    const int ptile = (int)blockIdx.x / n_ctiles, ctile = (int)blockIdx.x - ptile * n_ctiles;
    const int p0 = ptile * BP, c0 = ctile * BC;
    if (p0 >= P) return;                             // the smaller operation of a pair: the grid is sized for the other one
    const int chunks = (K + 63) / 64, per = (chunks + NW - 1) / NW;
    const int m0 = wave * per, m1 = min(chunks, m0 + per);

    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        (void*)a.x.p, 0, (int)((unsigned)nb_ * (unsigned)(a.H * a.W) * (unsigned)a.x.stride * 2u), 0x00020000);
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, (int)((unsigned)a.cout * (unsigned)K * 2u), 0x00020000);

    // ---- loads: lane fills 16-byte slot lane % 8 of rows lane / 8 + 8 i, with the chunk's piece (lane % 8) ^ (row % 8)
    const int r8 = lane >> 3, piece = (lane & 7) ^ r8;
    unsigned xo[4 * TP], wo[4 * TC];                           // byte offsets of tap (0, 0), channel 0 (pixels: may wrap below zero for padded windows)
    int hi0[4 * TP], wi0[4 * TP];
#pragma unroll
    for (int i = 0; i < 4 * TP; i++) {
        const unsigned p = (unsigned)min(p0 + r8 + 8 * i, P - 1);   // rows past the last pixel repeat it; their results are dropped
        const unsigned row = p / (unsigned)a.Wo, n = row / (unsigned)a.Ho;
        hi0[i] = (int)(row - n * (unsigned)a.Ho) * a.sh - a.pt;
        wi0[i] = (int)(p - row * (unsigned)a.Wo) * a.sw - a.pl;
        xo[i] = (unsigned)((((int)n * a.H + hi0[i]) * a.W + wi0[i]) * a.x.stride * 2 + a.x.c0 * 2);
    }
#pragma unroll
    for (int i = 0; i < 4 * TC; i++) {
        const int lr = r8 + 8 * i, co = c0 + ((lr & ~12) | ((lr & 4) << 1) | ((lr & 8) >> 1));
        wo[i] = co < a.cout ? (unsigned)co * (unsigned)K * 2u : OOBV;
    }
    int k = 64 * m0 + 8 * piece;                     // this lane's next piece, and its tap and channel
    int kh = 0, kw = 0, c = k;
    if constexpr (TAPS) {
        const int tap = k / a.cin;
        c = k - tap * a.cin;
        kh = tap / a.kw;
        kw = tap - kh * a.kw;
    }
    unsigned char* const mine = lds + wave * (NST * SM_STAGE);
    auto ask = [&](int stage) {
        unsigned char* const d = mine + stage * SM_STAGE;
        const bool kok = k < K;
        if constexpr (TAPS) {
            const unsigned to = (unsigned)((kh * a.W + kw) * a.x.stride * 2 + c * 2);
#pragma unroll
            for (int i = 0; i < 4 * TP; i++) {
                const bool ok = kok && (unsigned)(hi0[i] + kh) < (unsigned)a.H && (unsigned)(wi0[i] + kw) < (unsigned)a.W;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_ptr_t)(d + i * 1024), LDS_LOAD_BYTES, ok ? xo[i] + to : OOBV, 0, 0, 0);
            }
            c += 64;
            while (c >= a.cin) {
                c -= a.cin;
                if (++kw == a.kw) { kw = 0; kh++; }
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4 * TP; i++)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_ptr_t)(d + i * 1024), LDS_LOAD_BYTES, kok ? xo[i] + (unsigned)k * 2u : OOBV, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4 * TC; i++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wres, (lds_ptr_t)(d + XB + i * 1024), LDS_LOAD_BYTES,
                                                     kok && wo[i] != OOBV ? wo[i] + (unsigned)k * 2u : OOBV, 0, 0, 0);
        k += 64;
    };
#pragma unroll
    for (int q = 0; q < NST; q++)
        if (m0 + q < m1) ask(q);

    // ---- what the end needs from memory: this thread's groups of V channels
    constexpr int OUT = BP * BC / T, V = OUT >= 8 ? 8 : OUT, NG = OUT / V, GP = BC / V;   // results per thread, groups per thread and per pixel
    static_assert(OUT * T == BP * BC && V >= 2 && T % GP == 0, "results split evenly, a thread keeps its channels over its groups");
    const int px = t / GP, ch = (t - px * GP) * V, oc = c0 + ch;
    const bool ch_ok = oc < a.cout;                  // channel counts are in eights: a group exists as a whole or not at all
    float bias[V], scale[V];
    uint32_t resv[NG][V / 2];
    const uint16_t* const rg = (const uint16_t*)a.res.p;
#pragma unroll
    for (int e = 0; e < V; e++) {
        bias[e] = ch_ok ? ENS_GLOBAL(float, a.bias)[oc + e] : 0.f;
        scale[e] = ch_ok ? ENS_GLOBAL(float, a.scale)[oc + e] : 1.f;
    }
#pragma unroll
    for (int g = 0; g < NG; g++) {
        const int op = p0 + px + g * (T / GP);
#pragma unroll
        for (int e = 0; e < V / 2; e++)
            resv[g][e] = rg && ch_ok && op < P ? ENS_GLOBAL(uint32_t, rg + (size_t)op * a.res.stride + a.res.c0 + oc)[e] : 0u;
    }

    // ---- tables of the pre-activation or the gates, zeros past the last channel
    float* const tab = (float*)(lds + NW * NST * SM_STAGE);
    const int kpad = chunks * 64;
    int tab_row[TP] = {0};                           // gates: this lane's pixels' images among those of the tile
    if constexpr (MODE == SM_PRE) {
        for (int i = t; i < kpad; i += T) {
            tab[i] = i < K ? ENS_GLOBAL(float, a.pre_scale)[i] : 0.f;
            tab[kpad + i] = i < K ? ENS_GLOBAL(float, a.pre_shift)[i] : 0.f;
        }
        __syncthreads();
    } else if constexpr (MODE == SM_GATE) {
        const int HW = a.H * a.W, n_first = p0 / HW, n_last = min(p0 + BP - 1, P - 1) / HW;
        for (int i = t; i < (n_last - n_first + 1) * kpad; i += T) {
            const int n = i / kpad, q = i - n * kpad;
            tab[i] = q < K ? ENS_GLOBAL(float, a.gate)[(long long)(n_first + n) * a.gate_stride + q] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < TP; j++) tab_row[j] = (min(p0 + 32 * j + lrow, P - 1) / HW - n_first) * kpad;
        __syncthreads();
    }

    f32x16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; i++)
#pragma unroll
        for (int j = 0; j < TP; j++) bn_zero(acc[i][j]);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)mine + (uint32_t)(lrow * 128);
    int stage = 0;
    for (int m = m0; m < m1; m++) {
        // chunk m has landed: issued behind it are the chunks up to m + NST - 1
        if (NST > 1 && m + 1 < m1) bn_wait_vm<4 * (TP + TC) * (NST - 1)>(); else bn_wait_vm<0>();
        const uint32_t xs = lds0 + (uint32_t)(stage * SM_STAGE);
        bf16x8 xf[4][TP], wf[4][TC];
        bn_unroll<4>([&](auto ks_c) {
            constexpr int ks = decltype(ks_c)::value;
            const uint32_t at = xs + (uint32_t)(((2 * ks + lhalf) ^ (lrow & 7)) << 4);
            bn_unroll<TP>([&](auto j) { xf[ks][decltype(j)::value] = bn_lds_read<decltype(j)::value * 4096>(at); });
            bn_unroll<TC>([&](auto i) { wf[ks][decltype(i)::value] = bn_lds_read<XB + decltype(i)::value * 4096>(at); });
        });
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
#pragma unroll
            for (int j = 0; j < TP; j++) bn_tie(xf[ks][j]);
#pragma unroll
            for (int i = 0; i < TC; i++) bn_tie(wf[ks][i]);
        }
        if (m + NST < m1) ask(stage);                // into the buffer just read
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            if constexpr (MODE != SM_PLAIN) {
                f32x4 e0, e1, s0, s1;
                if constexpr (MODE == SM_PRE) {
                    const float* tp = tab + 64 * m + 16 * ks + 8 * lhalf;
                    e0 = *(const f32x4*)tp; e1 = *(const f32x4*)(tp + 4);
                    s0 = *(const f32x4*)(tp + kpad); s1 = *(const f32x4*)(tp + kpad + 4);
                }
#pragma unroll
                for (int j = 0; j < TP; j++) {
                    if constexpr (MODE == SM_GATE) {
                        const float* tp = tab + tab_row[j] + 64 * m + 16 * ks + 8 * lhalf;
                        e0 = *(const f32x4*)tp; e1 = *(const f32x4*)(tp + 4);
                    }
                    u32x4 u = __builtin_bit_cast(u32x4, xf[ks][j]);
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        const float lo = __uint_as_float(u[q] << 16), hi = __uint_as_float(u[q] & 0xFFFF0000u);
                        const float m0_ = q < 2 ? e0[2 * q] : e1[2 * q - 4], m1_ = q < 2 ? e0[2 * q + 1] : e1[2 * q - 3];
                        if constexpr (MODE == SM_PRE) {
                            const float f0 = q < 2 ? s0[2 * q] : s1[2 * q - 4], f1 = q < 2 ? s0[2 * q + 1] : s1[2 * q - 3];
                            u[q] = pack_bf16x2(fmaxf(fmaf(lo, m0_, f0), 0.f), fmaxf(fmaf(hi, m1_, f1), 0.f));
                        } else {
                            u[q] = pack_bf16x2(lo * m0_, hi * m1_);
                        }
                    }
                    xf[ks][j] = __builtin_bit_cast(bf16x8, u);
                }
            }
#pragma unroll
            for (int i = 0; i < TC; i++)
#pragma unroll
                for (int j = 0; j < TP; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks][i], xf[ks][j], acc[i][j], 0, 0, 0);
        }
        stage = stage + 1 == NST ? 0 : stage + 1;
    }
    // ---- the partial tiles meet: each wavefront's in its own part of LDS, [pixel][channel], rows padded by 16 bytes where that fits
    constexpr int PART = NST * SM_STAGE / 4, ROW = BP * (BC + 4) <= PART ? BC + 4 : BC;
    static_assert(BP * ROW <= PART, "a partial tile fits a wavefront's part");
    float* const part = (float*)lds;
#pragma unroll
    for (int j = 0; j < TP; j++)
#pragma unroll
        for (int i = 0; i < TC; i++)
#pragma unroll
            for (int q = 0; q < 4; q++)
                *(float4*)&part[wave * PART + (32 * j + lrow) * ROW + 32 * i + 16 * (q >> 1) + 8 * lhalf + 4 * (q & 1)] =
                    make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    __syncthreads();
#pragma unroll
    for (int g = 0; g < NG; g++) {
        const int row = px + g * (T / GP), op = p0 + row;
        float v[V];
#pragma unroll
        for (int e = 0; e < V; e++) v[e] = 0.f;
#pragma unroll
        for (int w = 0; w < NW; w++) {
#pragma unroll
            for (int e = 0; e < V; e++) v[e] += part[w * PART + row * ROW + ch + e];
        }
#pragma unroll
        for (int e = 0; e < V; e++) v[e] = fmaf(v[e], scale[e], bias[e]);
        if (rg) {
#pragma unroll
            for (int e = 0; e < V / 2; e++) {
                v[2 * e] += bf16_to_f32((uint16_t)(resv[g][e] & 0xFFFF));
                v[2 * e + 1] += bf16_to_f32((uint16_t)(resv[g][e] >> 16));
            }
        }
        apply_act_n<V>(v, a.act);
        if (op < P && ch_ok) {
            uint16_t* const d = (uint16_t*)a.y.p + (size_t)op * a.y.stride + a.y.c0 + oc;
            uint32_t u[V / 2];
#pragma unroll
            for (int e = 0; e < V / 2; e++) u[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
            if constexpr (V == 8) *ENS_GLOBAL_W(u32x4, d) = u32x4{u[0], u[1], u[2], u[3]};
            else {
#pragma unroll
                for (int e = 0; e < V / 2; e++) ENS_GLOBAL_W(uint32_t, d)[e] = u[e];
            }
        }
    }
}

// ---- host side -----------------------------------------------------------------------------
static size_t small_table_bytes(const ConvArgs& a, int bp) {
    const size_t kpad = (size_t)(a.cin + 63) / 64 * 64 * sizeof(float);
    return a.pre_scale ? 2 * kpad : a.gate ? (size_t)((bp - 1) / (a.H * a.W) + 2) * kpad : 0;
}

bool conv_small_applicable(const ConvArgs& a, int nb) {
    const long long P = (long long)nb * a.Ho * a.Wo, Pin = (long long)nb * a.H * a.W, K = (long long)a.kh * a.kw * a.cin;
    if (a.cin % 8 || a.cout % 8 || a.x.stride % 8 || a.x.c0 % 8 || a.y.stride % 8 || a.y.c0 % 8) return false;
    if (a.res.p && (a.res.stride % 8 || a.res.c0 % 8)) return false;
    const bool point = a.kh == 1 && a.kw == 1 && a.pt == 0 && a.pl == 0;
    if ((a.pre_scale || a.gate) && !point) return false;
    if (a.pre_scale && a.gate) return false;
    if (a.gate && (a.gate_stride < a.cin || a.sh != 1 || a.sw != 1)) return false;
    if (8 * sm_stage<1, 1>() + small_table_bytes(a, 32) > SM_LDS) return false;
    // 32-bit byte offsets with 2^31 standing for 'outside'
    if (Pin * a.x.stride * 2 >= 0x7FFFFF00LL || a.cout * K * 2 >= 0x7FFFFF00LL || P >= (1LL << 24)) return false;
    return true;
}

template <int TP, int TC, int NW, int NST, bool TAPS, int MODE>
static hipError_t launch_small_variant(const ConvArgs& a, const ConvArgs* argv, int G, int nb, hipStream_t s) {
    const long long P = (long long)nb * a.Ho * a.Wo;
    const dim3 grid((unsigned)(((P + 32 * TP - 1) / (32 * TP)) * ((a.cout + 32 * TC - 1) / (32 * TC))), 1, (unsigned)G);
    const size_t bytes = (size_t)NW * NST * sm_stage<TP, TC>() + small_table_bytes(a, 32 * TP);
    if (bytes > SM_LDS) return hipErrorInvalidValue;
    static bool raised = false;                                  // LDS above 64 KB has to be asked for once
    if (bytes > 64 * 1024 && !raised) {
        hipError_t e = hipFuncSetAttribute((const void*)&conv_small_bf16<TP, TC, NW, NST, TAPS, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, SM_LDS);
        if (e != hipSuccess) return e;
        raised = true;
    }
    ENS_LAUNCH((conv_small_bf16<TP, TC, NW, NST, TAPS, MODE>), grid, dim3(64 * NW), bytes, s, argv, nb);
    return hipGetLastError();
}
template <int TP, int TC, int NW, int NST>
static hipError_t launch_small_split(const ConvArgs& a, const ConvArgs* argv, int G, int nb, hipStream_t s) {
    if (a.pre_scale) return launch_small_variant<TP, TC, NW, NST, false, SM_PRE>(a, argv, G, nb, s);
    if (a.gate) return launch_small_variant<TP, TC, NW, NST, false, SM_GATE>(a, argv, G, nb, s);
    if (!a.pair && a.kh == 1 && a.kw == 1 && a.pt == 0 && a.pl == 0) return launch_small_variant<TP, TC, NW, NST, false, SM_PLAIN>(a, argv, G, nb, s);
    return launch_small_variant<TP, TC, NW, NST, true, SM_PLAIN>(a, argv, G, nb, s);
}

hipError_t launch_conv_small(const ConvArgs& a, const ConvArgs* argv, int G, int nb, int variant, hipStream_t s) {
    if (nb <= 0 || G <= 0 || !argv || !a.w || !a.bias || !a.scale || !conv_small_applicable(a, nb)) return hipErrorInvalidValue;
    switch (variant) {
        case 0: return launch_small_split<1, 1, 8, 2>(a, argv, G, nb, s);
        case 1: return launch_small_split<1, 1, 8, 1>(a, argv, G, nb, s);
        case 2: return launch_small_split<1, 1, 4, 1>(a, argv, G, nb, s);
        case 3: return launch_small_split<2, 2, 4, 2>(a, argv, G, nb, s);
    }
    return hipErrorInvalidValue;
}

const char* conv_small_name(const ConvArgs& a) { return a.gate ? "conv_small_bf16<32x32,gate>" : "conv_small_bf16"; }

// Measured over the layers of residual, dense, inception and inverted-residual networks on 1 to 64 images, one launch after
// the other (us, this kernel against the one that ran before; T = tiles of 32 x 32):
//   T <= 256    every layer                   14x14 1024->256 x1 4.4 / 8.9, 3x3 14x14x256 x4 6.7 / 13.8, 3x3 7x7x512 x4 8.8 / 13.9
//   T <= 512    all but shallow 1x1 layers    3x3 14x14x256 x8 9.8 / 14.5, 28x28 512->128 x4 4.6 / 6.5
//   T <= 800    what is not a plain 1x1       3x3 28x28x128 x8 10.5 / 11.0, 5x5 25x25x48 x16 9.3 / 13.6
// and 64 x 64 tiles (half the load traffic) while they number 256 or fewer: 3x3/2 28x28x128 x32 10.1 / 13.1, 1x7 12x12x160
// x32 10.3 / 15.8, 14x14 1024->256 x16 8.0 / 9.5.  Launches of other lanes count as 0.3 of a launch each.  A worker's full batches
// are for throughput: there the filters along one axis keep their own kernel whatever their number of tiles.
int conv_small_pick(const ConvArgs& a, int nb, int G) {
    if ((!a.few && a.kh != a.kw) || !conv_small_applicable(a, nb)) return -1;
    const long long P = (long long)nb * a.Ho * a.Wo, K = (long long)a.kh * a.kw * a.cin;
    if (K * a.cout < 4096) return -1;                            // a single step of the matrix cores or two
    const double load = 1.0 + 0.3 * (lanes_busy() - 1);
    const double t32 = load * (double)(G * ((P + 31) / 32) * ((a.cout + 31) / 32)), t64 = load * (double)(G * ((P + 63) / 64) * ((a.cout + 63) / 64));
    const bool plain = a.kh == 1 && a.kw == 1 && !a.pre_scale && !a.pair;
    const size_t table = small_table_bytes(a, 32);
    const bool wide = 16 * sm_stage<1, 1>() + table <= SM_LDS;   // two chunks per wavefront, one workgroup per compute unit
    if (t32 <= 256) return K >= 1024 && wide ? 0 : 1;
    if (plain && K <= 128) return -1;
    if (t32 <= 512) return 1;
    if (plain && K < 512) return -1;
    if (t64 <= 256 && 8 * sm_stage<2, 2>() + small_table_bytes(a, 64) <= SM_LDS) return 3;
    return t32 <= 800 && !plain ? 2 : -1;
}

// (28x28 bottleneck x4: 16 us in three launches, 29 us fused; 14x14 dense layer x8: 10 us in two, 17 us fused)
bool conv_small_layers(const ConvArgs& a, int nb, int G) {
    return a.few && (double)nb * a.Ho * a.Wo * G * (1.0 + 0.3 * (lanes_busy() - 1)) <= 6272;
}

}  // namespace ens

// fp32 convolution (members of fp32 precision: fp32 storage, fp32 multiply-adds, fp32 sums).
//
// A lane owns one output pixel and CT output channels: an input value that it fetches serves CT multiply-adds, and the
// CT weights of a (tap, input channel) are the same for the whole wavefront and stand side by side in memory
// ([kh][kw][cin][cout]), so they come through the scalar cache and enter the multiply-adds as scalar operands.  Taps outside
// the image are loaded from the nearest pixel inside and set to zero by a select, so that the loads of a filter row are
// unconditional and in flight together.
//
// With one output value per lane and both operands fetched for every multiply-add the kernel was bound by the vector memory
// path: 110 us per launch (1.5 TFLOP/s) for the 3x3 and 5x5 layers of 32 x 32 and 16 x 16 maps at batch 128.
#include "kernels.h"

namespace ens {

// uniform loads from memory that no kernel writes while this one runs
#define ENS_UNIFORM(p) ((const __attribute__((address_space(4))) float*)(p))

// K: filter size of both axes, 0 = any.  S: input channels fetched together: 4 (16-byte loads; channel count, stride and
// offset in fours), 3 (an image of three channels) or 1.
template <int CT, int K, int S>
__global__ __launch_bounds__(256) void conv_f32_kernel(const ConvArgs* __restrict__ argv, const int nb_, const int tile0) {
    const ConvArgs a = argv[blockIdx.z];
    const unsigned P = (unsigned)nb_ * (unsigned)(a.Ho * a.Wo);
    const unsigned p = blockIdx.x * 256u + threadIdx.x;
    if (p >= P) return;
    const int co0 = (tile0 + (int)blockIdx.y) * CT;
    const unsigned row = p / (unsigned)a.Wo, n = row / (unsigned)a.Ho;
    const int wo = (int)(p - row * (unsigned)a.Wo), ho = (int)(row - n * (unsigned)a.Ho);
    const float* __restrict__ const x = (const float*)a.x.p + (long long)n * a.H * a.W * a.x.stride + a.x.c0;
    const int KH = K ? K : a.kh, KW = K ? K : a.kw;
    constexpr int U = K ? K : 1;                                 // taps fetched together
    float acc[CT];
#pragma unroll
    for (int c = 0; c < CT; c++) acc[c] = 0.f;
    for (int kh = 0; kh < KH; kh++) {
        const int hi = ho * a.sh - a.pt + kh;
        const bool hok = (unsigned)hi < (unsigned)a.H;
        const float* __restrict__ const xr = x + (long long)min(max(hi, 0), a.H - 1) * a.W * a.x.stride;
        for (int kw0 = 0; kw0 < KW; kw0 += U) {
            const float* px[U];
            bool ok[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int wi = wo * a.sw - a.pl + kw0 + u;
                ok[u] = hok && (unsigned)wi < (unsigned)a.W;
                px[u] = xr + (long long)min(max(wi, 0), a.W - 1) * a.x.stride;
            }
            const float* wk = (const float*)a.w + (long long)(kh * KW + kw0) * a.cin * a.cout + co0;
            for (int c0 = 0; c0 < a.cin; c0 += S) {
                float v[U][S];
#pragma unroll
                for (int u = 0; u < U; u++) {
                    if constexpr (S == 4) {
                        const float4 t = *(const float4*)(px[u] + c0);
                        v[u][0] = t.x; v[u][1] = t.y; v[u][2] = t.z; v[u][3] = t.w;
                    } else {
#pragma unroll
                        for (int q = 0; q < S; q++) v[u][q] = px[u][c0 + q];
                    }
                }
                if (a.pre_scale) {
#pragma unroll
                    for (int u = 0; u < U; u++)
#pragma unroll
                        for (int q = 0; q < S; q++)
                            v[u][q] = fmaxf(v[u][q] * ENS_UNIFORM(a.pre_scale)[c0 + q] + ENS_UNIFORM(a.pre_shift)[c0 + q], 0.f);
                }
#pragma unroll
                for (int u = 0; u < U; u++)
#pragma unroll
                    for (int q = 0; q < S; q++) {
                        const float t = ok[u] ? v[u][q] : 0.f;
                        // (a tile past the last channel reads on into the next row or what follows the weights: dropped below)
                        const float* w = wk + (long long)(u * a.cin + c0 + q) * a.cout;
#pragma unroll
                        for (int c = 0; c < CT; c++) acc[c] = fmaf(t, ENS_UNIFORM(w)[c], acc[c]);
                    }
            }
        }
    }
    float* __restrict__ const y = (float*)a.y.p + (long long)p * a.y.stride + a.y.c0;
    const float* __restrict__ const res = a.res.p ? (const float*)a.res.p + (long long)p * a.res.stride + a.res.c0 : nullptr;
#pragma unroll
    for (int c = 0; c < CT; c++) {
        const int co = min(co0 + c, a.cout - 1);
        acc[c] = fmaf(acc[c], ENS_UNIFORM(a.scale)[co], ENS_UNIFORM(a.bias)[co]);   // fp32 members: the scale is in the weights and this one is 1
        if (res) acc[c] += res[co];
    }
    if (a.act == ACT_RELU) {
#pragma unroll
        for (int c = 0; c < CT; c++) acc[c] = fmaxf(acc[c], 0.f);
    } else if (a.act == ACT_SILU) {
#pragma unroll
        for (int c = 0; c < CT; c++) acc[c] = acc[c] / (1.f + expf(-acc[c]));        // the exponential at full precision
    }
    if (co0 + CT <= a.cout && a.y.stride % 4 == 0 && a.y.c0 % 4 == 0) {
#pragma unroll
        for (int c = 0; c < CT; c += 4) *(float4*)(y + co0 + c) = make_float4(acc[c], acc[c + 1], acc[c + 2], acc[c + 3]);
    } else {
#pragma unroll
        for (int c = 0; c < CT; c++)
            if (co0 + c < a.cout) y[co0 + c] = acc[c];
    }
}

template <int CT, int K>
static void launch_f32_variant(const ConvArgs& a, const ConvArgs* argv, int G, int nb, long long P, hipStream_t s) {
    constexpr int MOST = 65535;                                  // channel tiles that a grid can hold: wider layers take more launches
    const int tiles = (a.cout + CT - 1) / CT;
    for (int t0 = 0; t0 < tiles; t0 += MOST) {
        const dim3 grid((unsigned)((P + 255) / 256), (unsigned)(tiles - t0 < MOST ? tiles - t0 : MOST), (unsigned)G);
        const bool first = t0 == 0, last = tiles - t0 <= MOST;
        if (a.cin % 4 == 0 && a.x.stride % 4 == 0 && a.x.c0 % 4 == 0) ENS_LAUNCH_EV(first, last, (conv_f32_kernel<CT, K, 4>), grid, dim3(256), 0, s, argv, nb, t0);
        else if (a.cin == 3) ENS_LAUNCH_EV(first, last, (conv_f32_kernel<CT, K, 3>), grid, dim3(256), 0, s, argv, nb, t0);
        else ENS_LAUNCH_EV(first, last, (conv_f32_kernel<CT, K, 1>), grid, dim3(256), 0, s, argv, nb, t0);
    }
}
template <int CT>
static void launch_f32_channels(const ConvArgs& a, const ConvArgs* argv, int G, int nb, long long P, hipStream_t s) {
    if (a.kh == 3 && a.kw == 3) launch_f32_variant<CT, 3>(a, argv, G, nb, P, s);
    else if (a.kh == 5 && a.kw == 5) launch_f32_variant<CT, 5>(a, argv, G, nb, P, s);
    else launch_f32_variant<CT, 0>(a, argv, G, nb, P, s);
}

hipError_t launch_conv_f32(const ConvArgs& a, const ConvArgs* argv, int G, int nb, hipStream_t s) {
    if (nb <= 0 || a.cin <= 0 || a.cout <= 0 || !a.bias || !a.scale || G <= 0 || !argv) return hipErrorInvalidValue;
    if ((a.pre_scale == nullptr) != (a.pre_shift == nullptr)) return hipErrorInvalidValue;
    const long long P = (long long)nb * a.Ho * a.Wo;
    if (P >= (1LL << 32) - 256) return hipErrorInvalidValue;     // the kernel's pixel numbers, and the threads that a launch can have
    // More channels per lane make more of a fetched value, fewer make more wavefronts: as many channels as leave two
    // wavefronts per SIMD (1024 of them).  A lane's channels past the last one are worked out and dropped.
    const long long waves = (P + 63) / 64 * G;
    if (waves * ((a.cout + 15) / 16) >= 2048 && a.cout > 8) launch_f32_channels<16>(a, argv, G, nb, P, s);
    else if (waves * ((a.cout + 7) / 8) >= 2048 && a.cout > 4) launch_f32_channels<8>(a, argv, G, nb, P, s);
    else launch_f32_channels<4>(a, argv, G, nb, P, s);
    return hipGetLastError();
}

}  // namespace ens

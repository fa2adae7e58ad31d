// A small fp32 member from the request's images to its logits in one launch: a workgroup takes an image at a time, every tensor in LDS.
//
// Launch by launch such a member costs five launches a batch that leave the GPU idle (8 images: 66 us, of which a few are work) and fetches
// every tap through the vector memory path (14 TFLOP/s over 8 100 images).  A 32 x 32 x 16 map is 64 KB: the whole network fits the 160 KB of a
// compute unit.  Weights come once per workgroup, which then walks its share of the images.
//
// Convolutions run on the matrix cores in fp32 (v_mfma_f32_16x16x4: fp32 products, fp32 sums): 16 channels x 16 pixels, K = taps x input
// channels in steps of four.  The value a lane needs for its k is at a distance from the first tap's that is the same for every pixel: a
// table in LDS.  Tensors that a padded convolution reads have a border of zeros of their own, so that no tap is outside.
//
// Measured, two members of 32 x 32 images: 8 images 61 -> 32 us, 1 000 images in batches of 8 2.5 ms -> 117 us, 8 192 images 2.84 -> 0.57 ms.  A first
// form kept every map in LDS (convolution, barrier, pooling): one workgroup a compute unit, 1.50 ms; with windows and means taken in
// registers and the next image's pixels asked for ahead two of them fit.  8 100 images on the device, us, step by step: 710; the request's pixels three floats
// apart instead of four (windows two pixels apart then lie on different banks) 699; two pixels of up to eight channels in a tile 628; the steps
// behind the last whole four asked for at once, sums over lanes without LDS, 16 lanes a class 607; images drawn instead of dealt 584 (dealt, the workgroups of
// a launch ended between 430 and 590 us); a higher priority outside the convolutions' loops 565.
// No unit is full (counters, 8 100 images): the matrix cores are busy 0.52 of the time, LDS 0.28, a sixth of that bank conflicts (before the image's
// pixels lay three floats apart 0.48, half of it), vector units 0.43; of a wavefront's time 0.22 issues, 0.51 waits for its turn to issue (a matrix
// instruction holds its pipe for 32 clocks; for LDS alone it is 0.01) and 0.26 for data and at barriers.
#include "resident.h"
#include "conv_common.h"
#include "stage.h"

#include <cstddef>
#include <type_traits>

namespace ens {

#define RS(f) __builtin_amdgcn_readlane(op, offsetof(ResidentOp, f) / 4)

__device__ __forceinline__ float rs_act(float v, int act) {
    return act == ACT_RELU ? fmaxf(v, 0.f) : act == ACT_SILU ? v / (1.f + expf(-v)) : v;   // the exponential at full precision
}

// p / d for 0 <= p < 2^24
__device__ __forceinline__ int rs_div(int p, int d, float inv) {
    int q = (int)((float)p * inv);
    const int r = p - q * d;
    return q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
}

// the sum over 16 lanes side by side, in each of them
__device__ __forceinline__ float rs_sum16(float v) {
    auto from = [](float x, auto n) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + decltype(n)::value, 0xF, 0xF, false)); };   // row_ror
    v += from(v, std::integral_constant<int, 8>{});
    v += from(v, std::integral_constant<int, 4>{});
    v += from(v, std::integral_constant<int, 2>{});
    v += from(v, std::integral_constant<int, 1>{});
    return v;
}

// PT x 16 pixels times CT x 16 channels at a time.  POOL: a lane's pixels are the four of a 2 x 2 window, whose maximum or mean is what leaves the
// registers; MEAN: the sums over a unit's pixels are, added up at the end.  So the widest maps never are in LDS.
enum { RS_PLAIN, RS_POOL, RS_MEAN };
template <int PT, int CT, int FORM>
__device__ __forceinline__ void rs_conv(const int op, float* const lds) {
    const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // outputs: pixels, or windows of four
    const int Wo = RS(Wo), P = RS(Ho) * Wo, cout = RS(cout), steps = RS(steps), K = RS(kh) * RS(kw) * RS(cin), xs = RS(xp) * RS(sw), xrs = RS(xr) * RS(sh), act = RS(act);
    constexpr int EACH = FORM == RS_POOL ? 16 : 16 * PT;
    const int cts = (cout + 16 * CT - 1) / (16 * CT), units = ((P + EACH - 1) / EACH) * cts;
    const float inv = __builtin_amdgcn_rcpf((float)Wo);
    const int* const taps = (const int*)lds + RS(taps) + kq;
    for (int u = wave; u < units; u += RESIDENT_THREADS / 64) {
        const int pt = u / cts, ct = u - pt * cts;
        const float* x[PT];
        int yo[PT];
#pragma unroll
        for (int j = 0; j < PT; j++) {
            if constexpr (FORM == RS_POOL) {
                static_assert(PT == 4, "a window");
                const int p = pt * 16 + l16, pc = min(p, P - 1), ho = rs_div(pc, Wo, inv), wo = pc - ho * Wo;
                x[j] = lds + RS(x) + (2 * ho + (j >> 1)) * xrs + (2 * wo + (j & 1)) * xs;
                yo[j] = p < P ? RS(y) + ho * RS(yr) + wo * RS(yp) : -1;
            } else {
                const int p = (pt * PT + j) * 16 + l16, pc = min(p, P - 1), ho = rs_div(pc, Wo, inv), wo = pc - ho * Wo;
                x[j] = lds + RS(x) + ho * xrs + wo * xs;
                yo[j] = p < P ? RS(y) + ho * RS(yr) + wo * RS(yp) : -1;
            }
        }
        const float* const w = lds + RS(w) + (ct * CT * 4 * steps + kq) * 16 + l16;
        f32x4 acc[CT][PT];
#pragma unroll
        for (int i = 0; i < CT; i++)
#pragma unroll
            for (int j = 0; j < PT; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        // four steps at a time, the places of the next four on their way
        constexpr int U = 4;
        const int whole = K / (4 * U) * U;
        int off[U];
#pragma unroll
        for (int q = 0; q < U; q++) off[q] = taps[4 * q];        // (behind the table lie other words of LDS)
        __builtin_amdgcn_s_setprio(0);
        for (int s = 0; s < whole; s += U) {
            float a[U][CT], b[U][PT];
#pragma unroll
            for (int q = 0; q < U; q++) {
#pragma unroll
                for (int j = 0; j < PT; j++) b[q][j] = x[j][off[q]];
#pragma unroll
                for (int i = 0; i < CT; i++) a[q][i] = w[(i * steps + s + q) * 64];
            }
#pragma unroll
            for (int q = 0; q < U; q++) off[q] = taps[4 * (s + U + q)];
#pragma unroll
            for (int q = 0; q < U; q++)
#pragma unroll
                for (int i = 0; i < CT; i++)
#pragma unroll
                    for (int j = 0; j < PT; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][i], b[q][j], acc[i][j], 0, 0, 0);
        }
        if (whole < steps) {                                     // (behind K: a weight of zero times what is there could be a NaN)
            float a[U][CT], b[U][PT];
#pragma unroll
            for (int q = 0; q < U; q++) {
                const bool ok = 4 * (whole + q) + kq < K;
#pragma unroll
                for (int j = 0; j < PT; j++) {
                    const float v = x[j][ok ? off[q] : 0];
                    b[q][j] = ok ? v : 0.f;
                }
#pragma unroll
                for (int i = 0; i < CT; i++) a[q][i] = w[(i * steps + min(whole + q, steps - 1)) * 64];
            }
#pragma unroll
            for (int q = 0; q < U; q++) {
                if (whole + q >= steps) break;
#pragma unroll
                for (int i = 0; i < CT; i++)
#pragma unroll
                    for (int j = 0; j < PT; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][i], b[q][j], acc[i][j], 0, 0, 0);
            }
        }
        __builtin_amdgcn_s_setprio(1);
        // register v of a lane: channel 4 (lane / 16) + v of pixel lane % 16; whole fours are written (a pixel has room for them)
#pragma unroll
        for (int i = 0; i < CT; i++) {
            const int c = (ct * CT + i) * 16 + 4 * kq;
            const f32x4 b = *(const f32x4*)(lds + RS(bias) + min(c, cout - 1) / 4 * 4);
            f32x4 v[PT];
#pragma unroll
            for (int j = 0; j < PT; j++)
#pragma unroll
                for (int e = 0; e < 4; e++) v[j][e] = rs_act(acc[i][j][e] + b[e], act);
            if constexpr (FORM == RS_POOL) {
                const bool is_max = RS(pool) == RS_MAX_POOL;
                f32x4 r;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const float most = fmaxf(fmaxf(fmaxf(v[0][e], v[1][e]), fmaxf(v[2][e], v[3][e])), -3.0e38f);   // as rs_pool begins
                    r[e] = is_max ? most : (v[0][e] + v[1][e] + v[2][e] + v[3][e]) * 0.25f;
                }
                if (yo[0] >= 0 && c < cout) *(f32x4*)(lds + yo[0] + c) = r;
            } else if constexpr (FORM == RS_MEAN) {
                f32x4 r{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < PT; j++)
#pragma unroll
                    for (int e = 0; e < 4; e++) r[e] += yo[j] >= 0 ? v[j][e] : 0.f;
#pragma unroll
                for (int e = 0; e < 4; e++) r[e] = rs_sum16(r[e]);
                if (l16 == 0 && c < cout) *(f32x4*)(lds + RS(sums) + pt * RS(sums_p) + c) = r;
            } else if (c < cout) {
#pragma unroll
                for (int j = 0; j < PT; j++)
                    if (yo[j] >= 0) *(f32x4*)(lds + yo[j] + c) = v[j];
            }
        }
    }
    if constexpr (FORM == RS_MEAN) {                 // the units' sums in order
        __syncthreads();
        const int n = (P + EACH - 1) / EACH;
        const int sums_p = RS(sums_p);
        const float *const sums = lds + RS(sums);
        float* const y = lds + RS(y);
        for (int c = t; c < cout; c += RESIDENT_THREADS) {
            float sum = 0.f;
#pragma unroll 8
            for (int q = 0; q < n; q++) sum += sums[q * sums_p + c];
            y[c] = sum / (float)P;
        }
    }
}

// Up to eight channels and windows of 2 x 2: the rows of a tile are the channels of the windows' left pixels and of their right ones, its columns
// 16 windows, and K a column of the filter longer: kh * (kw + 1) * cin for half the tiles (5 x 5 x 3 to 8 channels on 32 x 32: 736 matrix instructions
// instead of 1 216).  Four tiles at a time: 32 windows, both their rows.
__device__ __forceinline__ void rs_conv_pair(const int op, float* const lds) {
    const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int Wo = RS(Wo), P = RS(Ho) * Wo, cout = RS(cout), steps = RS(steps), K = RS(kh) * (RS(kw) + 1) * RS(cin), xs = RS(xp), xrs = RS(xr) * RS(sh), act = RS(act);
    const float inv = __builtin_amdgcn_rcpf((float)Wo);
    const int* const taps = (const int*)lds + RS(taps) + kq;
    const float* const w = lds + RS(w) + kq * 16 + l16;
    const bool is_max = RS(pool) == RS_MAX_POOL;
    for (int u = wave; u < (P + 31) / 32; u += RESIDENT_THREADS / 64) {
        const float* x[4];
        int yo = -1;                                 // of the window that this lane writes: the first 16 are the lower half's
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const int p = u * 32 + j * 16 + l16, pc = min(p, P - 1), ho = rs_div(pc, Wo, inv), wo = pc - ho * Wo;
            x[2 * j] = lds + RS(x) + 2 * ho * xrs + 2 * wo * xs;
            x[2 * j + 1] = x[2 * j] + xrs;
            if (j == kq >> 1 && p < P) yo = RS(y) + ho * RS(yr) + wo * RS(yp);
        }
        f32x4 acc[4];
#pragma unroll
        for (int j = 0; j < 4; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        // four steps at a time, the places of the next four on their way
        constexpr int U = 4;
        const int whole = K / (4 * U) * U;
        int off[U];
#pragma unroll
        for (int q = 0; q < U; q++) off[q] = taps[4 * q];        // (behind the table lie other words of LDS)
        __builtin_amdgcn_s_setprio(0);
        for (int s = 0; s < whole; s += U) {
            float a[U], b[U][4];
#pragma unroll
            for (int q = 0; q < U; q++) {
#pragma unroll
                for (int j = 0; j < 4; j++) b[q][j] = x[j][off[q]];
                a[q] = w[(s + q) * 64];
            }
#pragma unroll
            for (int q = 0; q < U; q++) off[q] = taps[4 * (s + U + q)];
#pragma unroll
            for (int q = 0; q < U; q++)
#pragma unroll
                for (int j = 0; j < 4; j++) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], b[q][j], acc[j], 0, 0, 0);
        }
        if (whole < steps) {                                     // (behind K: a weight of zero times what is there could be a NaN)
            float a[U], b[U][4];
#pragma unroll
            for (int q = 0; q < U; q++) {
                const bool ok = 4 * (whole + q) + kq < K;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const float v = x[j][ok ? off[q] : 0];
                    b[q][j] = ok ? v : 0.f;
                }
                a[q] = w[min(whole + q, steps - 1) * 64];
            }
#pragma unroll
            for (int q = 0; q < U; q++) {
                if (whole + q >= steps) break;
#pragma unroll
                for (int j = 0; j < 4; j++) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], b[q][j], acc[j], 0, 0, 0);
            }
        }
        __builtin_amdgcn_s_setprio(1);
        // register v of a lane: channel 4 (lane / 16 % 2) + v of the left pixel in the lower half, of the right one in the upper
        const int c = 4 * (kq & 1);
        const f32x4 bias = *(const f32x4*)(lds + RS(bias) + min(c, cout - 1) / 4 * 4);
        f32x4 r[2];
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const float v0 = rs_act(acc[2 * j][e] + bias[e], act), v2 = rs_act(acc[2 * j + 1][e] + bias[e], act);
                if (is_max) {
                    const float m = fmaxf(v0, v2);
                    r[j][e] = fmaxf(fmaxf(m, __shfl_xor(m, 32, 64)), -3.0e38f);   // as rs_pool begins
                } else {                             // left and right, above and below
                    const float o0 = __shfl_xor(v0, 32, 64), o2 = __shfl_xor(v2, 32, 64);
                    r[j][e] = ((v0 + o0) + (kq < 2 ? v2 : o2) + (kq < 2 ? o2 : v2)) * 0.25f;
                }
            }
        if (yo >= 0 && c < cout) *(f32x4*)(lds + yo + c) = kq < 2 ? r[0] : r[1];
    }
}

// The same for an image with an infinity or a NaN, whose product with a zero of the pairs' weights would reach the neighbour: a thread per output.
__device__ __forceinline__ void rs_conv_odd(const int op, float* const lds) {
    const int Wo = RS(Wo), cout = RS(cout), cin = RS(cin), kh = RS(kh), each = RS(kw) * cin, P = RS(Ho) * Wo, act = RS(act), xs = RS(xp), xrs = RS(xr) * RS(sh), yr = RS(yr), yp = RS(yp);
    const int* const taps = (const int*)lds + RS(taps);
    const float *const x0 = lds + RS(x), *const w = lds + RS(w), *const bias = lds + RS(bias);
    float* const y = lds + RS(y);
    const bool is_max = RS(pool) == RS_MAX_POOL;
    for (int it = threadIdx.x; it < P * cout; it += RESIDENT_THREADS) {
        const int p = it / cout, c = it - p * cout, ho = p / Wo, wo = p - ho * Wo;
        float most = -3.0e38f, sum = 0.f;
#pragma unroll 1
        for (int q = 0; q < 4; q++) {
            const float* const x = x0 + (2 * ho + (q >> 1)) * xrs + (2 * wo + (q & 1)) * xs;
            float v = 0.f;
            for (int row = 0, k = 0; row < kh; row++, k += cin)  // (the left pixel's weights; the last column of a row is the right one's)
                for (int i = 0; i < each; i++, k++) v = fmaf(x[taps[k]], w[k * 16 + c], v);
            v = rs_act(v + bias[c], act);
            most = fmaxf(most, v);
            sum += v;
        }
        y[ho * yr + wo * yp + c] = is_max ? most : sum * 0.25f;
    }
}

__device__ __forceinline__ void rs_pool(const int op, float* const lds, const bool is_max) {
    const int c4 = (RS(cin) + 3) / 4, Wo = RS(Wo), H = RS(H), W = RS(W), items = RS(Ho) * Wo * c4;
    const float inv_c = __builtin_amdgcn_rcpf((float)c4), inv_w = __builtin_amdgcn_rcpf((float)Wo);
    for (int it = threadIdx.x; it < items; it += RESIDENT_THREADS) {
        const int p = rs_div(it, c4, inv_c), c = (it - p * c4) * 4, ho = rs_div(p, Wo, inv_w), wo = p - ho * Wo;
        const int h0 = ho * RS(sh) - RS(pt), w0 = wo * RS(sw) - RS(pl);
        f32x4 acc = is_max ? f32x4{-3.0e38f, -3.0e38f, -3.0e38f, -3.0e38f} : f32x4{0.f, 0.f, 0.f, 0.f};
        int cnt = 0;
        for (int h = max(h0, 0); h < min(h0 + RS(kh), H); h++)
            for (int w = max(w0, 0); w < min(w0 + RS(kw), W); w++) {
                const f32x4 v = *(const f32x4*)(lds + RS(x) + h * RS(xr) + w * RS(xp) + c);
#pragma unroll
                for (int e = 0; e < 4; e++) acc[e] = is_max ? fmaxf(acc[e], v[e]) : acc[e] + v[e];
                cnt++;
            }
        if (!is_max) {
#pragma unroll
            for (int e = 0; e < 4; e++) acc[e] /= (float)max(cnt, 1);
        }
        *(f32x4*)(lds + RS(y) + ho * RS(yr) + wo * RS(yp) + c) = acc;
    }
}

// mean over the pixels, a wavefront per channel
__device__ __forceinline__ void rs_gap(const int op, float* const lds) {
    const int t = threadIdx.x, lane = t & 63, W = RS(W), HW = RS(H) * W;
    const float inv = __builtin_amdgcn_rcpf((float)W);
    for (int c = t >> 6; c < RS(cin); c += RESIDENT_THREADS / 64) {
        float sum = 0.f;
        for (int p = lane; p < HW; p += 64) {
            const int h = rs_div(p, W, inv);
            sum += lds[RS(x) + h * RS(xr) + (p - h * W) * RS(xp) + c];
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        if (lane == 0) lds[RS(y) + c] = sum / (float)HW;
    }
}

// LANES lanes per class
template <int LANES>
__device__ __forceinline__ void rs_fc(const int op, float* const lds, float* const logits) {
    const int t = threadIdx.x, l = t & (LANES - 1), K = RS(cin), classes = RS(cout);
    const float *const x = lds + RS(x), *const w = lds + RS(w), *const bias = lds + RS(bias);
    for (int c0 = 0; c0 < classes; c0 += RESIDENT_THREADS / LANES) {
        const int c = min(c0 + t / LANES, classes - 1);
        float sum = 0.f;
        for (int k = l; k < K; k += LANES) sum = fmaf(x[k], w[k * classes + c], sum);
        sum = rs_sum16(sum);
#pragma unroll
        for (int off = 16; off < LANES; off <<= 1) sum += __shfl_xor(sum, off, 64);
        if (l == 0 && c0 + t / LANES < classes) logits[c] = sum + bias[c];
    }
}

__global__ __launch_bounds__(RESIDENT_THREADS) void resident_kernel(const ResidentArgs a) {
    extern __shared__ __attribute__((aligned(1024))) float rlds[];
    const int t = threadIdx.x;
    // Of the two workgroups of a compute unit, one of either half of the grid, the earlier one is served first (16 us an image against 20): every
    // other pair changes places, so that a member has as many of both, and still another member's beside them.
    const int half = (int)(gridDim.x + 1) / 2, pair = (int)blockIdx.x % half;
    const int block = pair % 2 && pair + half < (int)gridDim.x ? ((int)blockIdx.x < half ? pair + half : pair) : (int)blockIdx.x;
    int m = 0;
    while (m + 1 < a.n_members && block >= a.member[m + 1].first_block) m++;
    const ResidentMember& mb = a.member[m];
    const int px = mb.in_h * mb.in_w;
    const float inv_w = __builtin_amdgcn_rcpf((float)mb.in_w);
    // the next image's pixels are asked for a network ahead, where a thread has no more than two of them and they are only copied
    constexpr int AHEAD = 2;
    const bool ahead = px <= AHEAD * RESIDENT_THREADS && a.base_h == mb.in_h && a.base_w == mb.in_w;
    float v[AHEAD][3];
    auto ask = [&](int image) {
        const float* const src = a.src + (size_t)image * px * 3;
#pragma unroll
        for (int q = 0; q < AHEAD; q++)
#pragma unroll
            for (int c = 0; c < 3; c++) v[q][c] = t + q * RESIDENT_THREADS < px ? src[(t + q * RESIDENT_THREADS) * 3 + c] : 0.f;
    };
    int image = a.first + block - mb.first_block, next = image + mb.blocks;
    const int end = a.first + a.n;
    if (ahead && image < end) ask(image);
    for (int i = t; i < mb.lds_floats / 4; i += RESIDENT_THREADS)
        ((f32x4*)rlds)[i] = i < mb.fixed_floats / 4 ? ((const f32x4*)mb.fixed)[i] : f32x4{0.f, 0.f, 0.f, 0.f};   // and the borders' zeros
    const int* const ops = (const int*)rlds;         // the operations lie first
    // A workgroup's short phases go before its neighbour's matrix instructions, which fill the gaps: rs_conv and rs_conv_pair step back for their loops
    __builtin_amdgcn_s_setprio(1);
    constexpr int ODD = offsetof(ResidentOp, odd) / 4, DRAWN = offsetof(ResidentOp, drawn) / 4;
    __syncthreads();
    while (image < end) {
        unsigned drawn = 0;
        const bool draw = a.queue && next < end;     // the image after the next one: whoever is faster takes more
        if (draw && t == 0) drawn = __hip_atomic_fetch_add(a.queue + m, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        auto put = [&](int i, const float* p) {
            const int y = rs_div(i, mb.in_w, inv_w), x = i - y * mb.in_w;
            float* const d = rlds + mb.in + y * mb.in_r + x * mb.in_p;
            d[0] = p[0]; d[1] = p[1]; d[2] = p[2];
            if (p[0] * 0.f + p[1] * 0.f + p[2] * 0.f != 0.f) ((int*)rlds)[ODD] = image + 1;
            if (image >= mb.last_first && image < mb.last_first + mb.last_n) {
                float* const k = mb.input + ((size_t)(image - mb.last_first) * px + i) * 3;
                k[0] = p[0]; k[1] = p[1]; k[2] = p[2];
            }
        };
        if (ahead) {
#pragma unroll
            for (int q = 0; q < AHEAD; q++)
                if (t + q * RESIDENT_THREADS < px) put(t + q * RESIDENT_THREADS, v[q]);
            if (next < end) ask(next);
        } else {
            const float* const src = a.src + (size_t)image * a.base_h * a.base_w * 3;
            for (int i = t; i < px; i += RESIDENT_THREADS) {
                const int y = rs_div(i, mb.in_w, inv_w), x = i - y * mb.in_w;
                float p[3];
                stage_sample(a.base_h, a.base_w, mb.in_h, mb.in_w, src, y, x, p);
                put(i, p);
            }
        }
        __syncthreads();
        for (int i = 0; i < mb.n_ops; i++) {
            const int op = ops[i * 64 + (t & 63)];
            switch (RS(kind)) {
                case RS_CONV:
                    if (RS(pool) == RS_NO_POOL) {
                        if (RS(cout) > 16) rs_conv<2, 2, RS_PLAIN>(op, rlds); else rs_conv<4, 1, RS_PLAIN>(op, rlds);
                    } else if (RS(pool) == RS_MEAN_POOL) {
                        if (RS(cout) > 16) rs_conv<2, 2, RS_MEAN>(op, rlds); else rs_conv<2, 1, RS_MEAN>(op, rlds);
                    } else if (RS(pair)) {
                        if (ops[ODD] == image + 1) rs_conv_odd(op, rlds); else rs_conv_pair(op, rlds);
                    } else {
                        if (RS(cout) > 16) rs_conv<4, 2, RS_POOL>(op, rlds); else rs_conv<4, 1, RS_POOL>(op, rlds);
                    }
                    break;
                case RS_GAP: rs_gap(op, rlds); break;
                case RS_FC: {                        // (few products a class: the trips they take cost less than two more rounds of adding lanes up)
                    float* const z = mb.logits + (size_t)image * a.classes;
                    if (RS(cin) <= 256) rs_fc<16>(op, rlds, z); else rs_fc<64>(op, rlds, z);
                    break;
                }
                default: rs_pool(op, rlds, RS(kind) == RS_MAXPOOL);
            }
            if (i == 0 && draw && t == 0) ((int*)rlds)[DRAWN] = (int)drawn;   // (not before everybody has read the one before: the pixels' barrier)
            __syncthreads();
        }
        image = next;
        next = !a.queue ? next + mb.blocks : draw ? a.first + 2 * mb.blocks + ops[DRAWN] : end;
    }
    // the last workgroup of the launch leaves zeros
    if (a.queue && t == 0 && __hip_atomic_fetch_add(a.queue + RESIDENT_MAX_MEMBERS, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1)
        for (int i = 0; i <= RESIDENT_MAX_MEMBERS; i++) __hip_atomic_store(a.queue + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

hipError_t launch_resident(const ResidentArgs& a, int lds_bytes, hipStream_t s) {
    if (!a.src || a.n <= 0 || a.n_members <= 0 || a.n_members > RESIDENT_MAX_MEMBERS || lds_bytes > RESIDENT_LDS) return hipErrorInvalidValue;
    static const hipError_t raised = hipFuncSetAttribute((const void*)&resident_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, RESIDENT_LDS);
    if (raised != hipSuccess) return raised;
    int blocks = 0;
    for (int m = 0; m < a.n_members; m++) {
        if (a.member[m].blocks <= 0 || a.member[m].first_block != blocks || a.member[m].lds_floats * 4 > lds_bytes || !a.member[m].logits) return hipErrorInvalidValue;
        blocks += a.member[m].blocks;
    }
    ENS_LAUNCH(resident_kernel, dim3((unsigned)blocks), dim3(RESIDENT_THREADS), (size_t)lds_bytes, s, a);
    return hipGetLastError();
}

}  // namespace ens

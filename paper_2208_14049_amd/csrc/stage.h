// Input staging: what the staging kernels (layers.hip) and the chains (chain.hip) read of a request's images.
#pragma once
#include "kernels.h"

namespace ens {

// Bilinear sample (half-pixel centres, edge clamp) of the three source channels at destination
// pixel (y, x) of a dh x dw image made from an sh x sw one; a plain copy when the sizes agree.
__device__ __forceinline__ void stage_sample(const int sh, const int sw, const int dh, const int dw, const float* __restrict__ src, int y, int x, float* v) {
    if (sh == dh && sw == dw) {
        const float* p = src + ((long long)y * sw + x) * 3;
        v[0] = p[0]; v[1] = p[1]; v[2] = p[2];
        return;
    }
    float fy = (y + 0.5f) * ((float)sh / (float)dh) - 0.5f;
    float fx = (x + 0.5f) * ((float)sw / (float)dw) - 0.5f;
    fy = fminf(fmaxf(fy, 0.f), (float)(sh - 1));
    fx = fminf(fmaxf(fx, 0.f), (float)(sw - 1));
    const int y0 = (int)floorf(fy), x0 = (int)floorf(fx);
    const int y1 = min(y0 + 1, sh - 1), x1 = min(x0 + 1, sw - 1);
    const float wy = fy - y0, wx = fx - x0;
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const float p00 = src[((long long)y0 * sw + x0) * 3 + c], p01 = src[((long long)y0 * sw + x1) * 3 + c];
        const float p10 = src[((long long)y1 * sw + x0) * 3 + c], p11 = src[((long long)y1 * sw + x1) * 3 + c];
        const float top = p00 * (1.f - wx) + p01 * wx, bot = p10 * (1.f - wx) + p11 * wx;
        v[c] = top * (1.f - wy) + bot * wy;
    }
}

}  // namespace ens

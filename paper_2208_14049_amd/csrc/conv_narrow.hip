// 3x3, stride 1, padding 1 convolution from 32 channels to 32 on the CDNA4 matrix cores, the filter in registers: the parts that a
// grouped convolution is cut into.
//
// A pixel fragment meets one block of weights here, and 9 x 32 of K: on the generic kernel such a layer fetches every pixel nine times, with a
// barrier for every 64 of K, and runs at 60 TFLOP/s and 1.7 TB/s.  Here a wavefront keeps all 18 fragments of the filter (72 registers) for its
// whole life and the workgroups are persistent; all a tile needs is its input window, which comes to LDS once and in one go.  The
// inner loop is LDS reads and matrix-core instructions, two barriers a tile.  Grouped layers of 32 groups, 64 images, us alone, generic kernel and this
// one: 56x56x128 56.1 and 25.2, 28x28x256 32.0 and 16.3, 14x14x512 20.1 and 13.5, 7x7x1024 13.0 and 8.3; 16 images 56x56x128 21.2 and 14.3,
// 14x14x512 8.7 and 7.4.  What bounds it now is memory: 4 TB/s at 56x56.
//
// One window buffer and three workgroups a compute unit (168 registers): while one waits for its window the others compute.  The same form
// for 128 -> 32 channels (dense blocks' growth layers, two wavefronts sharing K, two workgroups a compute unit) takes 34.6 us instead of 48.7 at
// 56x56 and 128 images and 14.0 instead of 14.4 at 28x28, but fills a compute unit's LDS where conv_halo.hip leaves room for other lanes'
// launches: requests of four and twelve members stayed within 0.2 %, so those layers stay there.
//
// Pixels are numbered in the padded raster of conv_halo.hip.  A window row is 64 bytes of LDS, its pieces of 16 swizzled by the row's number.  The
// output leaves straight from the accumulators (conv_wreg.hip).
#include "conv_direct.h"

namespace ens {

constexpr int NARROW_CUS = 256, NARROW_PER_CU = 3, NARROW_LDS = 160 * 1024, NARROW_BP = 256, NARROW_CIN = 32;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NARROW_PER_CU, NARROW_PER_CU)))
void conv3x3_narrow_bf16(const ConvArgs* __restrict__ argv, const int nb_, const int hrows) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const ConvArgs a = argv[blockIdx.z];
    constexpr int BP = NARROW_BP, TP = BP / 128, CIN = NARROW_CIN, ROWB = CIN * 2, PIECES = ROWB / 16, RS = 256 / PIECES;
    constexpr int STEPS = CIN / 16, NSTEP = 9 * STEPS, BLK = 32 * ROWB, NTAB = 2;
    constexpr unsigned OOBV = 0x80000000u;
    auto key = [](uint32_t q) { return (q >> 2) & 3; };      // which piece of its row a row of LDS begins with

    const int W1 = a.W + 1, H1 = a.H + 1, img = H1 * W1, PP = nb_ * img;
    const int t = threadIdx.x, lane = t & 63, lrow = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wp0 = wave * 32 * TP;
    const int n_ptiles = (PP + BP - 1) / BP;
    const TileWalk walk = tile_walk(n_ptiles, blockIdx.z * gridDim.x);
    int ptile = walk.first;
    if (ptile >= walk.end) return;

    // LDS: window | bias and scale of the 32 channels | two tables window row -> pixel index (-1: none)
    float* const sb = (float*)(lds + hrows * ROWB);
    int* const tbl = (int*)(sb + 64);

    // ---- the filter: a lane's row is a channel with bits 2 and 3 swapped.  (A row's 576 bytes are taken 32 at a time, from the L1 after the first; once a
    // workgroup that is nothing beside a copy in operand order.)
    bf16x8 wreg[9][STEPS];
    {
        const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc((void*)a.w, 0, 32 * 9 * CIN * 2, 0x00020000);
        const unsigned row = (unsigned)((lrow & 0x13) | ((lrow & 4) << 1) | ((lrow & 8) >> 1)) * (9 * CIN * 2) + lhalf * 16u;
#pragma unroll
        for (int tap = 0; tap < 9; tap++)
#pragma unroll
            for (int ks = 0; ks < STEPS; ks++) wreg[tap][ks] = bn_wload(wres, row, (tap * STEPS + ks) * 32);
    }

    // ---- the table: a thread keeps the positions of its rows as (image, row, column) and steps them from tile to tile
    int tn[NTAB], thi[NTAB], twi[NTAB];
#pragma unroll
    for (int i = 0; i < NTAB; i++) {
        const int pp = ptile * BP - (W1 + 1) + t + 256 * i + img;   // one image further on: never negative
        const float inv_img = __builtin_amdgcn_rcpf((float)img), inv_w1 = __builtin_amdgcn_rcpf((float)W1);
        int n = (int)((float)pp * inv_img);
        int rem = pp - n * img;
        n += (rem >= img ? 1 : 0) - (rem < 0 ? 1 : 0);
        rem = pp - n * img;
        int hi = (int)((float)rem * inv_w1);
        int wi = rem - hi * W1;
        hi += (wi >= W1 ? 1 : 0) - (wi < 0 ? 1 : 0);
        tn[i] = n - 1; thi[i] = hi; twi[i] = rem - hi * W1;
    }
    const int adv = walk.step * BP, adv_n = adv / img, adv_h = (adv - adv_n * img) / W1, adv_w = adv - adv_n * img - adv_h * W1;
    // writes the table of the tile that the positions stand at, then moves on to the next one
    auto make_table = [&](int slot) {
#pragma unroll
        for (int i = 0; i < NTAB; i++) {
            const bool ok = (unsigned)tn[i] < (unsigned)nb_ && thi[i] < a.H && twi[i] < a.W;
            if (t + 256 * i < hrows) tbl[slot * hrows + t + 256 * i] = ok ? (tn[i] * a.H + thi[i]) * a.W + twi[i] : -1;
            twi[i] += adv_w;
            const int cw = twi[i] >= W1 ? 1 : 0;
            twi[i] -= cw ? W1 : 0;
            thi[i] += adv_h + cw;
            const int ch = thi[i] >= H1 ? 1 : 0;
            thi[i] -= ch ? H1 : 0;
            tn[i] += adv_n + ch;
        }
    };
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc((void*)a.x.p, 0, (int)((unsigned)nb_ * (unsigned)(a.H * a.W) * (unsigned)a.x.stride * 2u), 0x00020000);
    const int r0 = t / PIECES;
    const unsigned xlane = (unsigned)(a.x.c0 * 2) + (((unsigned)(t % PIECES) ^ key(r0)) << 4);
    auto issue_window = [&](int slot) {
        const int* const tb = tbl + slot * hrows;
        const int nsl = (hrows + RS - 1) / RS, wrow = wave * (64 / PIECES);   // (hrows is whole wavefronts' loads)
        for (int s0 = 0; s0 < nsl; s0 += 8) {                    // eight table look-ups in flight at a time
            int p8[8];
#pragma unroll
            for (int j = 0; j < 8; j++) p8[j] = tb[min((s0 + j) * RS + r0, hrows - 1)];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                if ((s0 + j) * RS + wrow >= hrows) break;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_ptr_t)(lds + (s0 + j) * 4096 + wave * 1024), LDS_LOAD_BYTES,
                                                         p8[j] >= 0 ? (unsigned)(p8[j] * a.x.stride * 2) + xlane : OOBV, 0, 0, 0);
            }
        }
    };
    make_table(0);
    if (t < 32) {
        sb[t] = ENS_GLOBAL(float, a.bias)[t];
        sb[32 + t] = ENS_GLOBAL(float, a.scale)[t];
    }
    __syncthreads();
    issue_window(0);

    // ---- fragment side: the nine taps' places in the window do not depend on the tile
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
    uint32_t xoff[9];
#pragma unroll
    for (int tap = 0; tap < 9; tap++) {
        const uint32_t q = (uint32_t)(wp0 + lrow + (tap / 3) * W1 + tap % 3);
        xoff[tap] = lds0 + q * ROWB + (((uint32_t)lhalf ^ key(q)) << 4);
    }
    // ---- output side: channels 16 k + 8 lhalf ... + 7 of this wavefront's positions
    const unsigned npix = (unsigned)nb_ * (unsigned)(a.H * a.W);
    const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc((void*)a.y.p, 0, (int)(npix * (unsigned)a.y.stride * 2u), 0x00020000);
    auto store = [&](const f32x16& acc, int p) {
        const unsigned at = p >= 0 ? (unsigned)(p * a.y.stride + a.y.c0 + 8 * lhalf) * 2u : OOBV;
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const u32x4 o = bn_pack(acc, k, a.act, sb + 8 * lhalf, 32);
            __builtin_amdgcn_raw_buffer_store_b128(o, yres, at, 32 * k, 0);
        }
    };

    for (int slot = 0; ptile < walk.end; ptile += walk.step, slot ^= 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wavefront's part of the window has landed,
        __syncthreads();                                         // and everybody's
        const bool more = ptile + walk.step < walk.end;
        if (more) make_table(slot ^ 1);                          // (the table of the tile before is done with)
        f32x16 acc[TP];
#pragma unroll
        for (int j = 0; j < TP; j++) bn_zero(acc[j]);
        bf16x8 xf[2][TP];
        auto read_frags = [&](auto step_c, auto b_c) {
            constexpr int step = decltype(step_c)::value, b = decltype(b_c)::value;
            const uint32_t xa = xoff[step / STEPS] ^ (uint32_t)(step % STEPS << 5);
            bn_unroll<TP>([&](auto j) { xf[b][decltype(j)::value] = bn_lds_read<decltype(j)::value * BLK>(xa); });
        };
        read_frags(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
        bn_unroll<NSTEP>([&](auto step_c) {
            constexpr int step = decltype(step_c)::value, b = step & 1;
            // the next step's reads are issued first; LDS returns in order
            if constexpr (step + 1 < NSTEP) {
                read_frags(std::integral_constant<int, step + 1>{}, std::integral_constant<int, b ^ 1>{});
                asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(TP) : "memory");
            } else {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
#pragma unroll
            for (int j = 0; j < TP; j++) bn_tie(xf[b][j]);
#pragma unroll
            for (int j = 0; j < TP; j++) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wreg[step / STEPS][step % STEPS], xf[b][j], acc[j], 0, 0, 0);
        });
        int p[TP];                                               // the centre tap's rows: this tile's outputs
#pragma unroll
        for (int j = 0; j < TP; j++) p[j] = tbl[slot * hrows + W1 + 1 + wp0 + lrow + 32 * j];
        __syncthreads();                                         // the window is free
        if (more) issue_window(slot ^ 1);
#pragma unroll
        for (int j = 0; j < TP; j++) store(acc[j], p[j]);
    }
}

// ---- host side -----------------------------------------------------------------------------
struct NarrowPlan { int hrows, wgs; size_t bytes; };

static bool narrow_plan(const ConvArgs& a, int nb, int G, NarrowPlan* pl) {
    if (a.kh != 3 || a.kw != 3 || a.sh != 1 || a.sw != 1 || a.pt != 1 || a.pl != 1 || a.Ho != a.H || a.Wo != a.W) return false;
    if (a.pre_scale || a.gate || a.res.p || a.pair || a.cin != NARROW_CIN || a.cout != 32) return false;
    if (a.x.stride % 8 || a.x.c0 % 8 || a.y.stride % 8 || a.y.c0 % 8) return false;
    // 32-bit byte offsets with 2^31 standing for 'outside'; quotients by float reciprocals
    const long long pixels = (long long)nb * a.H * a.W, img = (long long)(a.H + 1) * (a.W + 1), PP = nb * img;
    if (pixels * a.x.stride * 2 >= 0x7FFFFF00LL || pixels * a.y.stride * 2 >= 0x7FFFFF00LL || PP + img + 2 * NARROW_BP >= (1LL << 24)) return false;
    const int rows_a_load = 64 / (NARROW_CIN / 8);
    if (a.W > 126) return false;                                 // two rows of the table a thread
    pl->hrows = (NARROW_BP + 2 * (a.W + 1) + 2 + rows_a_load - 1) / rows_a_load * rows_a_load;
    pl->bytes = (size_t)pl->hrows * NARROW_CIN * 2 + 64 * 4 + 2 * (size_t)pl->hrows * 4;
    // as many workgroups as the chip holds at once
    const long long tiles = (PP + NARROW_BP - 1) / NARROW_BP;
    pl->wgs = (int)std::min<long long>(tiles, std::max<long long>(1, (long long)NARROW_PER_CU * NARROW_CUS / G));
    return pl->hrows <= 512 && NARROW_PER_CU * (pl->bytes + 1024) <= (size_t)NARROW_LDS;
}

bool conv_narrow_applicable(const ConvArgs& a, int nb, int G) {
    NarrowPlan pl;
    return narrow_plan(a, nb, G, &pl);
}

const char* conv_narrow_name(const ConvArgs&) { return "conv3x3_narrow_bf16<256,c32>"; }

hipError_t launch_conv_narrow(const ConvArgs& a, const ConvArgs* argv, int G, int nb, hipStream_t s) {
    NarrowPlan pl;
    if (!narrow_plan(a, nb, G, &pl)) return hipErrorInvalidValue;
    ENS_LAUNCH(conv3x3_narrow_bf16, dim3((unsigned)pl.wgs, 1, (unsigned)G), dim3(256), pl.bytes, s, argv, nb, pl.hrows);
    return hipGetLastError();
}

}  // namespace ens

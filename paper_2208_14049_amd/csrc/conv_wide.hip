// 1x1 convolution (stride 1, or a stride without padding) with tiles of 128 pixels x 256 output channels: the wide layers of large
// batches.  The work of a chunk of input channels, its ring in LDS and the operand-ordered weights are those of conv_pw.hip; here a
// wavefront owns 128 pixels x 64 channels, so that each pixel fragment it reads from LDS serves two matrix-core instructions.
//
// What bounds it: with 128 x 32 per wavefront, LDS reads and the loads of input and weights through the L1 each took as long as the
// matrix-core instructions they fed (128 and 64 bytes per clock and compute unit); with 128 x 64 they take one half and three
// quarters of that, and half as many tiles read each input value.  The price is registers, 128 of them accumulators: the weights are
// only one chunk ahead, the residual is asked for during the last chunk (half of it, in the registers where that chunk's
// successor's weights would lie) and after it.  Measured against 128 x 128 tiles, four streams at once: 14x14 1024 -> 256, 128
// images 14.6 -> 13.2 us (998 TFLOP/s), 19x19 728 -> 728, 64 images 35.9 -> 30.3 us, 14x14 512 -> 512, 128 images 16.8 -> 14.3 us.
#include "conv_direct.h"

namespace ens {

constexpr int WD_BP = 128, WD_BC = 256, WD_NXB = 3, WD_XS = WD_BP * 128;
constexpr size_t WD_LDS = (size_t)WD_NXB * WD_XS + 2 * WD_BC * sizeof(float);

template <bool RES, bool ROWS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv1x1_wide_bf16(const ConvArgs* __restrict__ argv, const int nb_) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const ConvArgs a = argv[blockIdx.z];
    constexpr int BP = WD_BP, TP = BP / 32, CB = 2, BC = WD_BC, XS = WD_XS, XO = 4;   // XO: input rows per thread and chunk
    const int P = nb_ * a.Ho * a.Wo;                 // output pixels
    const int t = threadIdx.x, lane = t & 63, lrow = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int n_ptiles = (P + BP - 1) / BP, n_ctiles = (a.cout + BC - 1) / BC;
    int ptile, ctile;
    tile_of_block(n_ptiles, n_ctiles, &ptile, &ctile);
    if (ptile >= n_ptiles) return;
    const int p0 = ptile * BP, c0 = ctile * BC;
    const int wc = c0 + wave * 64;                   // this wave's 64 channels; the last ones of a layer may be fewer, or none
    const int nk = (a.cin + 63) / 64, NS = nk * 4;   // input chunks; matrix-core steps per block of weight rows
    constexpr unsigned OOBV = 0x80000000u;           // past the end of every buffer the launcher admits: zeros, or no store
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        (void*)a.wpk, 0, (int)((unsigned)((a.cout + 31) / 32 * 32) * (unsigned)(nk * 64) * 2u), 0x00020000);
    unsigned wv[CB];
#pragma unroll
    for (int b = 0; b < CB; b++) wv[b] = wc + 32 * b < a.cout ? (unsigned)((wc / 32 + b) * NS * 1024 + lane * 16) : OOBV;
    bf16x8 w0[CB][4], w1[CB][4];                     // weights of this chunk and the next
    auto load_w = [&](bf16x8 (&w)[CB][4], int kc) {
#pragma unroll
        for (int ks = 0; ks < 4; ks++)
#pragma unroll
            for (int b = 0; b < CB; b++) w[b][ks] = bn_wload(wres, wv[b], (kc * 4 + ks) * 1024);
    };
    const unsigned npix = (unsigned)P;
    const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc((void*)a.y.p, 0, (int)(npix * (unsigned)a.y.stride * 2u), 0x00020000);
    f32x16 acc[CB][TP];
#pragma unroll
    for (int b = 0; b < CB; b++)
#pragma unroll
        for (int j = 0; j < TP; j++) bn_zero(acc[b][j]);
    float* const sbl = (float*)(lds + WD_NXB * XS);
    const bool sb_ok = c0 + t < a.cout;
    const float bias_r = sb_ok ? ENS_GLOBAL(float, a.bias)[c0 + t] : 0.f;
    const float scale_r = sb_ok ? ENS_GLOBAL(float, a.scale)[c0 + t] : 1.f;
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        (void*)a.x.p, 0, (int)((unsigned)nb_ * (unsigned)(a.H * a.W) * (unsigned)a.x.stride * 2u), 0x00020000);
    const int r8 = t >> 3, c8 = (t & 7) ^ ((r8 >> 1) & 7);
    const bool strided = a.sh != 1 || a.sw != 1;
    unsigned xvo[XO];
#pragma unroll
    for (int s = 0; s < XO; s++) {
        const int p = p0 + r8 + 32 * s;
        const int pin = strided && p < P ? strided_input_pixel(a, p) : p;
        xvo[s] = p < P ? (unsigned)(pin * a.x.stride * 2) + (unsigned)(a.x.c0 * 2 + c8 * 16) : OOBV;
    }
    // in the last chunk of a layer whose input channels are not a multiple of 64 this thread's 8 may lie past the last one
    const bool tail_ok = (nk - 1) * 64 + c8 * 8 < a.cin;
    unsigned char* const mine = lds + wave * 1024;
    auto issue_x = [&](int buf, int kc) {
        const bool live = kc + 1 < nk || tail_ok;
#pragma unroll
        for (int s = 0; s < XO; s++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_ptr_t)(mine + buf * XS + s * 4096), LDS_LOAD_BYTES, live ? xvo[s] : OOBV, kc * 128, 0, 0);
    };
    issue_x(0, 0);
    load_w(w0, 0);
    if (nk > 1) issue_x(1, 1);
    sbl[t] = bias_r;
    sbl[BC + t] = scale_r;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
    const uint32_t xs0 = lds0 + (uint32_t)(lrow * 128 + ((lhalf ^ ((lrow >> 1) & 7)) << 4));
    const __amdgpu_buffer_rsrc_t rres = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(RES ? a.res.p : a.y.p), 0, (int)(npix * (unsigned)(RES ? a.res.stride : a.y.stride) * 2u), 0x00020000);
    // Residual and output come and go half the tile's pixels at a time, in 8 pieces of 8 channels, which exist as a whole or not at all.  ROWS: in rows
    // (bn_row), piece m being pixel pl + 8 m, channels rc ...; otherwise straight from the accumulators, pixel pl + 32 (m / 4), channels rc + 16 (m % 4).
    const int rc = wc + 8 * (ROWS ? lane & 7 : lhalf);
    auto piece = [&](int h, int m, int pl, const View& v) {
        const int p = pl + 64 * h + (ROWS ? 8 * m : m / 4 * 32), c = rc + (ROWS ? 0 : m % 4 * 16);
        return p < P && c < a.cout ? (unsigned)(p * v.stride * 2) + (unsigned)((v.c0 + c) * 2) : OOBV;
    };
    auto load_res = [&](bf16x8 (&res)[CB][4], int h, int pl) {
#pragma unroll
        for (int m = 0; m < 8; m++) res[m / 4][m % 4] = bn_wload(rres, piece(h, m, pl, a.res), 0);
    };
    int pl = p0 + (ROWS ? lane >> 3 : lrow);
    int buf = 0;
    // Order of issue: x(0) w(0) x(1), then w(kc + 1) x(kc + 2) in chunk kc; when chunk kc begins only x(kc + 1) may be outstanding.
    auto chunk = [&](bf16x8 (&wc_)[CB][4], bf16x8 (&wl)[CB][4], const int kc) {
        if (kc + 1 < nk) bn_wait_vm<XO>(); else bn_wait_vm<0>();
#pragma unroll
        for (int b = 0; b < CB; b++)
#pragma unroll
            for (int ks = 0; ks < 4; ks++) bn_tie(wc_[b][ks]);
        __builtin_amdgcn_s_barrier();
        if (kc + 1 < nk) load_w(wl, kc + 1);
        else if constexpr (RES) load_res(wl, 0, pl);
        if (kc + 2 < nk) issue_x(buf == 0 ? 2 : buf - 1, kc + 2);
        const uint32_t xs = xs0 + (uint32_t)(buf * XS);
        buf = buf == 2 ? 0 : buf + 1;
        bf16x8 xf[2][TP];
        auto read_frags = [&](auto ks_c, auto b_c) {
            constexpr int ks = decltype(ks_c)::value, b = decltype(b_c)::value;
            const uint32_t xa = xs ^ (uint32_t)(ks << 5);
            bn_unroll<TP>([&](auto j) { xf[b][decltype(j)::value] = bn_lds_read<decltype(j)::value * 4096>(xa); });
        };
        read_frags(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
        bn_unroll<4>([&](auto ks_c) {
            constexpr int ks = decltype(ks_c)::value, b = ks & 1;
            if constexpr (ks + 1 < 4) {
                read_frags(std::integral_constant<int, ks + 1>{}, std::integral_constant<int, b ^ 1>{});
                asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(TP) : "memory");
            } else {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
#pragma unroll
            for (int j = 0; j < TP; j++) bn_tie(xf[b][j]);
#pragma unroll
            for (int q = 0; q < CB; q++)
#pragma unroll
                for (int j = 0; j < TP; j++) acc[q][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wc_[q][ks], xf[b][j], acc[q][j], 0, 0, 0);
        });
    };
    int kc = 0;
    for (; kc + 1 < nk; kc += 2) {
        chunk(w0, w1, kc);
        chunk(w1, w0, kc + 1);
    }
    if (kc < nk) chunk(w0, w1, kc);
    asm volatile("" : "+v"(pl));
    bf16x8 r1[CB][4];
    if constexpr (RES) {
        if (nk & 1) {                                // the first half's residual lies where the last chunk's successor would
#pragma unroll
            for (int b = 0; b < CB; b++)
#pragma unroll
                for (int ks = 0; ks < 4; ks++) w0[b][ks] = w1[b][ks];
        }
        load_res(r1, 1, pl);
    }
    // turned in the two buffers of the ring that the last chunk is not in: everybody is done with them since its barrier
    unsigned char* const turn = lds + ((wave < 2 ? nk : nk + 1) % 3) * XS + (wave & 1) * 8192;
#pragma unroll
    for (int h = 0; h < 2; h++) {
        auto row = [&](int m) { return (u32x4*)(turn + bn_row<128>(8 * m + (lane >> 3), lane & 7)); };
        auto res = [&](int m) { return __builtin_bit_cast(u32x4, h ? r1[m / 4][m % 4] : w0[m / 4][m % 4]); };
        if constexpr (RES && ROWS) {
#pragma unroll
            for (int m = 0; m < 8; m++) *row(m) = res(m);
            bn_turn();
        }
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int q = 0; q < CB; q++)
#pragma unroll
                for (int k = 0; k < 2; k++) {
                    u32x4* const at = (u32x4*)(turn + bn_row<128>(32 * j + lrow, 4 * q + 2 * k + lhalf));
                    u32x4 r = {0u, 0u, 0u, 0u};
                    if constexpr (RES && ROWS) r = *at;
                    else if constexpr (RES) r = res(4 * j + 2 * q + k);
                    r = bn_pack_res<RES>(acc[q][2 * h + j], k, r, a.act, sbl + (wc + 8 * lhalf + 32 * q - c0), BC);
                    if constexpr (ROWS) *at = r;
                    else __builtin_amdgcn_raw_buffer_store_b128(r, yres, piece(h, 4 * j + 2 * q + k, pl, a.y), 0, 0);
                }
        if constexpr (ROWS) {
            bn_turn();
#pragma unroll
            for (int m = 0; m < 8; m++) __builtin_amdgcn_raw_buffer_store_b128(*row(m), yres, piece(h, m, pl, a.y), 0, 0);
            bn_turn();
        }
    }
}
// ---- host side -----------------------------------------------------------------------------
// The shape has passed conv_pw_applicable.  Wide tiles are taken
//  - among the launches of other lanes from 128 tiles on (14x14 1024 -> 256: 98 tiles 8.2 us against 7.7, 147 tiles 10.1 against
//    11.3);
//  - alone if they nearly fill the 512 places of one round (7x7 512 -> 2048, 392 tiles: 25.8 us against 29.2; with 343 or fewer the
//    smaller tiles are as fast or faster, with 543 and 784 both are within 10 % either way) or several (1371 tiles 128 us against
//    151);
//  - if no more than a quarter of their columns are padding (768 -> 192 gains 12 %, 2048 -> 320 loses as much);
//  - with more than 128 input channels: shorter layers write more than they compute (28x28 128 -> 512: 41 us against 38).
bool conv_wide_wanted(const ConvArgs& a, int nb, int G) {
    const int ctiles = (a.cout + WD_BC - 1) / WD_BC;
    const long long tiles = ((long long)nb * a.Ho * a.Wo + WD_BP - 1) / WD_BP * ctiles * G;
    if (a.gate || a.cin <= 128 || 4 * a.cout < 3 * ctiles * WD_BC) return false;
    return lanes_in_use() >= 3 ? tiles >= 128 : (tiles > 343 && tiles <= 512) || tiles >= 1024;
}

hipError_t launch_conv_wide(const ConvArgs& a, const ConvArgs* argv, int G, int nb, hipStream_t s) {
    const long long P = (long long)nb * a.Ho * a.Wo;
    const dim3 grid((unsigned)(((P + WD_BP - 1) / WD_BP) * ((a.cout + WD_BC - 1) / WD_BC)), 1, G);
    if (rows_wanted()) {
        if (a.res.p) ENS_LAUNCH((conv1x1_wide_bf16<true, true>), grid, dim3(256), WD_LDS, s, argv, nb);
        else ENS_LAUNCH((conv1x1_wide_bf16<false, true>), grid, dim3(256), WD_LDS, s, argv, nb);
    } else {
        if (a.res.p) ENS_LAUNCH((conv1x1_wide_bf16<true, false>), grid, dim3(256), WD_LDS, s, argv, nb);
        else ENS_LAUNCH((conv1x1_wide_bf16<false, false>), grid, dim3(256), WD_LDS, s, argv, nb);
    }
    return hipGetLastError();
}

}  // namespace ens

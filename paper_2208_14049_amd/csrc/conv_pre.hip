// Pre-activated 1x1 convolution (relu(x * scale + shift) per input channel, up to 128 output channels) on the CDNA4 matrix cores: the
// first layer of a dense-block layer on batches that fill the chip, where it and the 3x3 behind it run as two launches.
//
// Organisation as in conv_pw.hip: a workgroup of four wavefronts owns 128 pixels x 128 channels, each wavefront all pixels of 32
// channels, weights straight from memory in matrix-core operand order, input 64 channels at a time by asynchronous
// global-to-LDS loads.  The ring has four buffers, since a chunk is also converted on the way: while the matrix cores work on
// chunk kc, every thread turns the 16-byte pieces that it brought in of chunk kc + 1 into relu(x * scale + shift), in
// place and once per value, and chunks kc + 2 and kc + 3 are on their way.
//
// Against the fused layer (conv_dense.hip), which computes this convolution on the window its 3x3 taps reach: no value is worked out
// twice (there 1.5 times at 14x14, twice at 28x28 and 56x56), for 256 bytes per pixel of the tensor in between written and read.
#include "conv_direct.h"

namespace ens {

constexpr int PR_BP = 128, PR_BC = 128, PR_NXB = 4, PR_XS = PR_BP * 128;

template <bool ROWS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void conv1x1_pre_bf16(const ConvArgs* __restrict__ argv, const int nb_) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const ConvArgs a = argv[blockIdx.z];
    constexpr int TP = PR_BP / 32, XS = PR_XS, XO = PR_BP / 32, WO = 4;   // loads per thread and chunk: input rows, weight fragments
    constexpr unsigned OOBV = 0x80000000u;           // past the end of every buffer the launcher admits
    const int P = nb_ * a.H * a.W;
    const int t = threadIdx.x, lane = t & 63, lrow = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    int ptile, ctile;
    tile_of_block((P + PR_BP - 1) / PR_BP, 1, &ptile, &ctile);
    const int p0 = ptile * PR_BP, wc = wave * 32;
    const bool wave_ok = wc < a.cout;
    const int nk = (a.cin + 63) / 64, NS = nk * 4;   // input chunks; matrix-core steps per block of weight rows

    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        (void*)a.wpk, 0, (int)((unsigned)((a.cout + 31) / 32 * 32) * (unsigned)(nk * 64) * 2u), 0x00020000);
    const unsigned wv = wave_ok ? (unsigned)(wave * NS * 1024 + lane * 16) : OOBV;
    bf16x8 w0[4], w1[4], w2[4];                      // weights of this chunk, the next, the one after
    auto load_w = [&](bf16x8 (&w)[4], int kc) {
#pragma unroll
        for (int ks = 0; ks < 4; ks++) w[ks] = bn_wload(wres, wv, (kc * 4 + ks) * 1024);
    };
    load_w(w0, 0);
    if (nk > 1) load_w(w1, 1);
    // ---- input chunks: thread t fills slot t % 8 of rows t / 8 + 32 s with the swizzled piece
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc((void*)a.x.p, 0, (int)((unsigned)P * (unsigned)a.x.stride * 2u), 0x00020000);
    const int r8 = t >> 3, c8 = (t & 7) ^ ((r8 >> 1) & 7);
    unsigned xvo[XO];
#pragma unroll
    for (int s = 0; s < XO; s++) {
        const int p = p0 + r8 + 32 * s;
        xvo[s] = p < P ? (unsigned)(p * a.x.stride * 2) + (unsigned)(a.x.c0 * 2 + c8 * 16) : OOBV;
    }
    const bool tail_ok = (nk - 1) * 64 + c8 * 8 < a.cin;         // pieces past the last channel are zeros
    unsigned char* const mine = lds + wave * 1024;               // this wave's quarter of a 4 KB load
    auto issue_x = [&](int kc) {
        const bool live = kc + 1 < nk || tail_ok;
#pragma unroll
        for (int s = 0; s < XO; s++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_ptr_t)(mine + (kc & 3) * XS + s * 4096), LDS_LOAD_BYTES, live ? xvo[s] : OOBV,
                                                     kc * 128, 0, 0);
    };
    issue_x(0);
    if (nk > 1) issue_x(1);
    if (nk > 2) issue_x(2);
    // ---- tables: bias, scale of the channels; scale and shift of the inputs, zeros past the last one (relu(0 x + 0) = 0)
    float* const sbl = (float*)(lds + PR_NXB * XS);
    float* const psl = sbl + 2 * PR_BC;
    const int kpad = nk * 64;
    if (t < PR_BC) {
        sbl[t] = t < a.cout ? ENS_GLOBAL(float, a.bias)[t] : 0.f;
        sbl[PR_BC + t] = t < a.cout ? ENS_GLOBAL(float, a.scale)[t] : 1.f;
    }
    for (int i0 = t; i0 < kpad; i0 += 4 * 256) {
        float s[4], h[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int i = i0 + 256 * u;
            s[u] = i < a.cin ? ENS_GLOBAL(float, a.pre_scale)[i] : 0.f;
            h[u] = i < a.cin ? ENS_GLOBAL(float, a.pre_shift)[i] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (i0 + 256 * u < kpad) {
                psl[i0 + 256 * u] = s[u];
                psl[kpad + i0 + 256 * u] = h[u];
            }
    }
    __syncthreads();

    f32x16 acc[TP];
#pragma unroll
    for (int j = 0; j < TP; j++) bn_zero(acc[j]);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
    const uint32_t xs0 = lds0 + (uint32_t)(lrow * 128 + ((lhalf ^ ((lrow >> 1) & 7)) << 4));
    const uint32_t own0 = lds0 + (uint32_t)(wave * 1024 + lane * 16), psl0 = (uint32_t)(uintptr_t)(lds_ptr_t)psl + (uint32_t)(8 * c8 * 4);
    bf16x8 xv[XO], pt[4];                            // this thread's pieces, and scale and shift of their channels (as raw bits)
    auto pre_read = [&](int kc) {
        const uint32_t pa = psl0 + (uint32_t)(kc * 256), ha = pa + (uint32_t)(kpad * 4), own = own0 + (uint32_t)((kc & 3) * XS);
        pt[0] = bn_lds_read<0>(pa); pt[1] = bn_lds_read<16>(pa);
        pt[2] = bn_lds_read<0>(ha); pt[3] = bn_lds_read<16>(ha);
        bn_unroll<XO>([&](auto sc) { xv[decltype(sc)::value] = bn_lds_read<decltype(sc)::value * 4096>(own); });
    };
    auto pre_tie = [&]() {
#pragma unroll
        for (int x = 0; x < 4; x++) bn_tie(pt[x]);
#pragma unroll
        for (int x = 0; x < XO; x++) bn_tie(xv[x]);
    };
    auto pre_math = [&](int x) {
        const f32x4 s0 = __builtin_bit_cast(f32x4, pt[0]), s1 = __builtin_bit_cast(f32x4, pt[1]);
        const f32x4 h0 = __builtin_bit_cast(f32x4, pt[2]), h1 = __builtin_bit_cast(f32x4, pt[3]);
        u32x4 u = __builtin_bit_cast(u32x4, xv[x]);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const float lo = __uint_as_float(u[q] << 16), hi = __uint_as_float(u[q] & 0xFFFF0000u);
            const float sl = q < 2 ? s0[2 * q] : s1[2 * q - 4], sh = q < 2 ? s0[2 * q + 1] : s1[2 * q - 3];
            const float hl = q < 2 ? h0[2 * q] : h1[2 * q - 4], hh = q < 2 ? h0[2 * q + 1] : h1[2 * q - 3];
            typedef short s16x2 __attribute__((ext_vector_type(2)));
            const s16x2 z = {0, 0};                              // relu on the rounded pair: a negative bf16 is a negative 16-bit integer
            u[q] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(
                __builtin_bit_cast(s16x2, pack_bf16x2(fmaf(lo, sl, hl), fmaf(hi, sh, hh))), z));
        }
        xv[x] = __builtin_bit_cast(bf16x8, u);
    };
    auto pre_write = [&](int kc) {
        const uint32_t own = own0 + (uint32_t)((kc & 3) * XS);
#pragma unroll
        for (int x = 0; x < XO; x++) asm volatile("ds_write_b128 %0, %1" ::"v"(own + (uint32_t)(x * 4096)), "v"(xv[x]) : "memory");
    };
    // chunk 0 (the barrier above has waited for it)
    pre_read(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    pre_tie();
#pragma unroll
    for (int x = 0; x < XO; x++) pre_math(x);
    pre_write(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    // One chunk: `wk` holds its weights, `wl` receives those of chunk kc + 2; the three sets rotate by name.  `steady`: chunk kc + 3
    // exists, every load is issued and the wait is one constant.
    auto chunk = [&](auto steady_c, bf16x8 (&wk)[4], bf16x8 (&wl)[4], const int kc) {
        constexpr bool steady = decltype(steady_c)::value;
        if (steady || kc + 3 < nk) issue_x(kc + 3);
        if (steady || kc + 2 < nk) load_w(wl, kc + 2);
        const uint32_t xs = xs0 + (uint32_t)((kc & 3) * XS);
        bf16x8 xf[2][TP];
        auto read_frags = [&](auto ks_c, auto b_c) {
            constexpr int ks = decltype(ks_c)::value, b = decltype(b_c)::value;
            const uint32_t xa = xs ^ (uint32_t)(ks << 5);
            bn_unroll<TP>([&](auto j) { xf[b][decltype(j)::value] = bn_lds_read<decltype(j)::value * 4096>(xa); });
        };
        read_frags(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
        // The input of chunk kc + 1 has landed.  Issued behind it are the inputs of chunks kc + 2 and kc + 3 and the weights of chunks kc + 1
        // and kc + 2, 2 (XO + WO) loads in the steady loop and XO + 2 WO where kc + 2 is the last chunk.  The waits allow XO (WO) fewer:
        // the input of chunk kc + 2 has landed as well.  Not measured with the looser ones.
        if (steady) bn_wait_vm<2 * XO + WO>();
        else if (kc + 2 < nk) bn_wait_vm<XO + WO>();
        else bn_wait_vm<0>();
        const int kn = steady || kc + 1 < nk ? kc + 1 : kc;      // after the last chunk: converted again, not written
        pre_read(kn);
        bn_unroll<4>([&](auto ks_c) {
            constexpr int ks = decltype(ks_c)::value, b = ks & 1;
            if constexpr (ks == 0) {
                asm volatile("s_waitcnt lgkmcnt(8)" ::: "memory");      // the fragments, not the pieces read behind them
            } else {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
#pragma unroll
            for (int j = 0; j < TP; j++) bn_tie(xf[b][j]);
            if constexpr (ks == 1) pre_tie();
            if constexpr (ks + 1 < 4) read_frags(std::integral_constant<int, ks + 1>{}, std::integral_constant<int, b ^ 1>{});
#pragma unroll
            for (int j = 0; j < TP; j++) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wk[ks], xf[b][j], acc[j], 0, 0, 0);
            if constexpr (ks == 1) { pre_math(0); pre_math(1); }
            if constexpr (ks == 2) { pre_math(2); pre_math(3); }
        });
        if (steady || kc + 1 < nk) pre_write(kn);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    };
    constexpr std::false_type near_the_end{};
    constexpr std::true_type all_there{};
    int kc = 0;
    for (; kc + 5 < nk; kc += 3) {
        chunk(all_there, w0, w2, kc);
        chunk(all_there, w1, w0, kc + 1);
        chunk(all_there, w2, w1, kc + 2);
    }
    for (; kc < nk; kc += 3) {
        chunk(near_the_end, w0, w2, kc);
        if (kc + 1 < nk) chunk(near_the_end, w1, w0, kc + 1);
        if (kc + 2 < nk) chunk(near_the_end, w2, w1, kc + 2);
    }
    // ---- output: register v of a lane is channel wc + 16(v/8) + 8(lane/32) + v%8 of its pixel
    const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc((void*)a.y.p, 0, (int)((unsigned)P * (unsigned)a.y.stride * 2u), 0x00020000);
    //      and leaves straight from the accumulators or, ROWS, in rows (bn_row), turned in the ring, which everybody is done with since the last barrier
    unsigned char* const turn = lds + wave * (TP * 32 * 64);
    auto store = [&](const u32x4& v, int px, int c) {
        const int p = p0 + px;
        __builtin_amdgcn_raw_buffer_store_b128(v, yres, p < P && c < a.cout ? (unsigned)(p * a.y.stride * 2) + (unsigned)((a.y.c0 + c) * 2) : OOBV, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < TP; j++)
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const u32x4 o = bn_pack(acc[j], k, a.act, sbl + wc + 8 * lhalf, PR_BC);
            if constexpr (ROWS) *(u32x4*)(turn + bn_row<64>(32 * j + lrow, 2 * k + lhalf)) = o;
            else store(o, 32 * j + lrow, wc + 8 * lhalf + 16 * k);
        }
    if constexpr (ROWS) {
        bn_turn();
#pragma unroll
        for (int i = 0; i < 2 * TP; i++) {
            const int px = 16 * i + (lane >> 2);
            store(*(const u32x4*)(turn + bn_row<64>(px, lane & 3)), px, wc + 8 * (lane & 3));
        }
    }
}

// ---- host side -----------------------------------------------------------------------------
static size_t pre_lds_bytes(const ConvArgs& a) { return (size_t)PR_NXB * PR_XS + (2 * PR_BC + 2 * ((size_t)(a.cin + 63) / 64 * 64)) * sizeof(float); }

bool conv_pre_applicable(const ConvArgs& a, int nb) {
    if (a.kh != 1 || a.kw != 1 || a.sh != 1 || a.sw != 1 || a.pt != 0 || a.pl != 0 || a.Ho != a.H || a.Wo != a.W) return false;
    if (!a.pre_scale || !a.pre_shift || !a.wpk || a.gate || a.pair || a.res.p || a.cin % 8 || a.cout % 8 || a.cout > PR_BC) return false;
    if (a.x.stride % 8 || a.x.c0 % 8 || a.y.stride % 8 || a.y.c0 % 8) return false;
    const long long P = (long long)nb * a.H * a.W;               // 32-bit byte offsets with 2^31 standing for 'outside'
    if (P * a.x.stride * 2 >= 0x7FFFFF00LL || P * a.y.stride * 2 >= 0x7FFFFF00LL) return false;
    return 2 * pre_lds_bytes(a) <= 160 * 1024;                   // two workgroups per compute unit
}

const char* conv_pre_name() { return "conv1x1_pre_bf16<128x128>"; }

template <bool ROWS>
static hipError_t launch_pre_variant(const ConvArgs& a, const ConvArgs* argv, int G, int nb, hipStream_t s) {
    static bool raised = false;                                  // LDS above 64 KB has to be asked for once
    if (!raised) {
        hipError_t e = hipFuncSetAttribute((const void*)&conv1x1_pre_bf16<ROWS>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        raised = true;
    }
    const long long P = (long long)nb * a.H * a.W;
    ENS_LAUNCH(conv1x1_pre_bf16<ROWS>, dim3((unsigned)((P + PR_BP - 1) / PR_BP), 1, (unsigned)G), dim3(256), pre_lds_bytes(a), s, argv, nb);
    return hipGetLastError();
}

hipError_t launch_conv_pre(const ConvArgs& a, const ConvArgs* argv, int G, int nb, hipStream_t s) {
    if (!conv_pre_applicable(a, nb)) return hipErrorInvalidValue;
    return rows_wanted() ? launch_pre_variant<true>(a, argv, G, nb, s) : launch_pre_variant<false>(a, argv, G, nb, s);
}

}  // namespace ens

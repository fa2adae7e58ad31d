// A request of few images in one kernel launch: chains.
//
// One image through a deep member is a chain of 50 to 300 layers of which none fills the GPU, and a launch per layer costs 6 to 10 us
// however little it does (twelve members, one image: 940 launches on four lanes, 2.97 ms).  Here the workgroups of an XCD, one per
// compute unit, form a group that takes a member and some images and runs all its layers, with a barrier between layers that
// depend on each other, and the eight groups take such programs from one queue, the longest first (1.23 ms).  The group's compute units
// share an L2: stores need only reach it (s_waitcnt vmcnt(0)), loads of what others stored bypass the L1 (device scope, sc1: 3.6 TB/s an XCD
// from the L2 with it and without), and a barrier of the 32 workgroups is an atomic and a poll there, 1.0 us (over all eight XCDs it is 4 us,
// and data would have to go through memory).
//
// Nobody waits for a workgroup that is not there: a group is made of the workgroups that have begun by the time the first
// of them closes it (all of them in a few microseconds when the GPU is free), later ones leave at once, and the programs go to whatever
// groups there are.  So the launch needs no place for all its workgroups at once and ends beside anything.  How fast depends on
// the compute units that are empty when it begins (a workgroup takes nearly all of one's LDS), for its groups do not grow: one image through four
// members takes 0.63 ms alone, and while another handle keeps three of the four streams full 0.70 ms (0.93 ms at 90 %, 5.5 ms the worst of
// 284; as launches it waits for those streams, 67 ms), and the other handle's 70 ms become 224 if such requests follow one another all the
// while.  Two handles that send one such request after another: 1.33 ms for both (launches: 1.54).
//
// Convolutions: a wavefront owns a tile of 32 x 32 or 64 x 64 (pixels x channels) or a share of its K; weights come straight to registers,
// pixels through LDS of its own.  A phase is 5 us for a layer of one round and a few chunks along K: 1.9 us between the phases, 1.6 us of
// set-up and ending, 0.5 us a chunk (round trips, some 500 instructions, and 64 bytes a clock of loads; a chunk of a 64 x 64 tile is at the
// L2's 47 bytes a clock and compute unit).  By the counters (twelve members, one image) a wavefront waits for data and at barriers 0.68 of its time; the matrix
// cores are busy 0.04 of it, the L1s 0.23, the L2s give 5.2 TB/s (0.88 of it hits), the memory 0.6.  Tried: four wavefronts and two groups a compute unit, to fill one program's waits with
// another's work: 1.0 to 1.1 times as fast from two images on, 0.75 times on one.
#include "chain.h"
#include "conv_direct.h"
#include "stage.h"
#include <cstddef>

namespace ens {

// A step in a register, a dword a lane.  Fields read from memory where they are needed were twenty round trips to the scalar cache
// on the way to a layer's first load (1.8 us); a lane read is an instruction.
struct Step { int v; };
__device__ __forceinline__ int st_int(const Step s, int at) { return __builtin_amdgcn_readlane(s.v, at); }
__device__ __forceinline__ int64_t st_long(const Step s, int at) { return (int64_t)(((uint64_t)(uint32_t)st_int(s, at + 1) << 32) | (uint32_t)st_int(s, at)); }
// The thread's number, worked out again: what depends on it is not kept in registers over all the kinds of steps.
__device__ __forceinline__ int ch_thread() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}
#define ST(f) st_int(s, offsetof(ChainStep, f) / 4)
#define ST_L(f) st_long(s, offsetof(ChainStep, f) / 4)
#define ST_P(f) ((const char*)ST_L(f))
#define ST_F(f) __int_as_float(ST(f))

constexpr int CH_WAVE_LDS = 16 * 1024;
constexpr int CH_TABLE_AT = CHAIN_WAVES * CH_WAVE_LDS;
constexpr int CH_MISC_AT = CH_TABLE_AT + CHAIN_TABLE_FLOATS * 4;
constexpr int CH_STEPS_AT = CH_MISC_AT + 64;
constexpr int CH_LDS = CH_STEPS_AT + 2 * CHAIN_PHASE_STEPS * 256;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr int SC1 = 16;                              // cache policy of a buffer load: device scope

__device__ __forceinline__ u32x4 ch_load16(const __amdgpu_buffer_rsrc_t& r, unsigned off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, SC1));
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t ch_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}
// p / d for 0 <= p < 2^24 with inv = 1 / d
__device__ __forceinline__ int ch_div(int p, int d, float inv) {
    int q = (int)((float)p * inv);
    const int r = p - q * d;
    return q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
}
__device__ __forceinline__ void ch_unpack(const u32x4& v, float* f) {
#pragma unroll
    for (int e = 0; e < 4; e++) {
        f[2 * e] = __uint_as_float(v[e] << 16);
        f[2 * e + 1] = __uint_as_float(v[e] & 0xFFFF0000u);
    }
}
__device__ __forceinline__ u32x4 ch_pack(const float* f) {
    return u32x4{pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7])};
}

// The group's barrier, in two halves, and what the phases to come need: the steps of the phase after the next one, and the next one's weights,
// which are brought into the L2 (a word of each line, dealt to the group's threads).  Loads come back in the order they were asked for, so
// whatever a wavefront asks for behind those waits for the memory too.  A workgroup that has to wait at the barrier asks for them there; one that
// comes last, and that the others will wait for next, behind its loads of the phase.  (Asked for by all in front of the barrier, the workgroups
// with a share of them came 1 to 3 us later than the others in every phase; twelve members, one image and two: 1.26 and 1.68 ms, now 1.22 and 1.65.)
constexpr int CH_AHEAD = 2;
struct ChainGroup {
    unsigned* arrived;
    unsigned target, size, ticket;
    unsigned* misc;                                  // LDS: [0] is everybody there, [5] verdict of the wait
    int* steps;                                      // LDS: the steps of this phase and of the next one, CHAIN_PHASE_STEPS each
    const int* next;                                 // the next phase's steps in memory
    int next_n, at;                                  // how many; which half of `steps` is this phase's
    bool pending;                                    // arrived at and not waited for yet
    bool dead, fetched;                              // fetched: what the phases to come need has been asked for
    int word;                                        // of the next phase's steps, on its way to LDS
    unsigned ahead[CH_AHEAD];                        // what was touched

    __device__ __forceinline__ Step step(int i) const { return Step{steps[(at * CHAIN_PHASE_STEPS + i) * 64 + (threadIdx.x & 63)]}; }
    __device__ __forceinline__ void arrive() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // this wave's stores are in the L2
#pragma unroll
        for (int i = 0; i < CH_AHEAD; i++) asm volatile("" ::"v"(ahead[i]));
        at ^= 1;
        if (fetched && threadIdx.x >= 64 && (int)threadIdx.x - 64 < next_n * 64) steps[at * CHAIN_PHASE_STEPS * 64 + threadIdx.x - 64] = word;
        fetched = false;
        __syncthreads();
        if (threadIdx.x == 0) (void)__hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);   // at the group's L2
        target += size;
        pending = true;
    }
    __device__ __forceinline__ void prefetch(const Step s0) {     // s0: the first step of the phase
        if (fetched) return;
        fetched = true;
        if (threadIdx.x < 64) return;                            // (the first wavefront polls)
        const int idx = (int)threadIdx.x - 64;
        static_assert(CHAIN_PHASE_STEPS * 64 <= CHAIN_THREADS - 64, "a dword each");
        if (idx < next_n * 64) word = ENS_GLOBAL(int, next)[idx];
        const unsigned first = ticket * (CHAIN_THREADS - 64) + idx, all = size * (CHAIN_THREADS - 64);
        const char* const w0 = (const char*)st_long(s0, offsetof(ChainStep, ahead) / 4);
        const char* const w1 = (const char*)st_long(s0, offsetof(ChainStep, ahead) / 4 + 2);
        const unsigned n0 = (unsigned)st_int(s0, offsetof(ChainStep, ahead_bytes) / 4) / 128u, n1 = (unsigned)st_int(s0, offsetof(ChainStep, ahead_bytes) / 4 + 1) / 128u;
        if (first < n0) ahead[0] = *ENS_GLOBAL(unsigned, w0 + (size_t)first * 128);
        if (n1) {
            if (first < n1) ahead[1] = *ENS_GLOBAL(unsigned, w1 + (size_t)first * 128);
        } else if (first + all < n0) {
            ahead[1] = *ENS_GLOBAL(unsigned, w0 + (size_t)(first + all) * 128);
        }
    }
    __device__ __forceinline__ bool all_there() const { return (int)(__hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) >= 0; }
    __device__ __forceinline__ void wait(const Step s0) {
        if (!pending) return;
        pending = false;
        if (threadIdx.x == 0) misc[0] = all_there();
        __syncthreads();
        if (misc[0]) return;
        if (threadIdx.x == 0) {
            unsigned ok = 0;
            // Every workgroup of the group is running, so this ends; the limit (seconds) is for a mistake elsewhere
            for (int i = 0; i < (1 << 23); i++) {
                if (all_there()) { ok = 1; break; }
                __builtin_amdgcn_s_sleep(1);
            }
            misc[5] = ok;
        }
        prefetch(s0);
        __syncthreads();
        if (!misc[5]) dead = true;
    }
};

// ---- convolution ---------------------------------------------------------------------------
// T: side of a wavefront's tile in 32s.  Weights come in operand order straight to registers (1 KB in a row per load), pixels by asynchronous
// loads into LDS of the wavefront's own, both two chunks of 64 along K ahead.
template <int T, bool PRE>
__device__ __forceinline__ void chain_conv(const Step s, const Step s0_, char* const base, const int images, const int unit, const int lg, unsigned char* const lds, ChainGroup& group) {
    constexpr int TP = T, TC = T, BP = 32 * TP, BC = 32 * TC, STAGE = BP * 128, NST = 2;
    constexpr unsigned OOBV = 0x80000000u;
    static_assert(NST * STAGE <= CH_WAVE_LDS && BP * BC * 4 <= CH_WAVE_LDS, "a wavefront's part");
    static_assert(CHAIN_WAVES == 8, "three bits of wavefronts");
    const int t = ch_thread(), lane = t & 63, lrow = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int split = 1 << lg, kpart = wave & (split - 1), tile = (unit << (3 - lg)) + (wave >> lg);
    const int ctiles = ST(ctiles[T - 1]), ptile = ch_div(tile, ctiles, ST_F(inv_ctiles[T - 1])), cs = tile - ptile * ctiles;
    const int K = ST(K), P = images * ST(px), cout = ST(cout), cin = ST(cin), xs = ST(xs);
    const int chunks = (K + 63) >> 6, per = (chunks + split - 1) >> lg, p0 = ptile * BP;
    const bool live = p0 < P;
    const int m0 = kpart * per, m1 = live ? min(chunks, m0 + per) : 0;

    const __amdgpu_buffer_rsrc_t wres = ch_rsrc(ST_P(w), (unsigned)ST(wsize));
    bf16x8 wf[NST][4][TC];
    unsigned wv[TC];
#pragma unroll
    for (int i = 0; i < TC; i++) wv[i] = i == 0 ? lane * 16u : chain_weight_lane(cs, TC, i, ST(ctiles[0]), lane);
    auto ask_w = [&](auto buf, int m) {
#pragma unroll
        for (int st = 0; st < 4; st++)
#pragma unroll
            for (int i = 0; i < TC; i++) wf[decltype(buf)::value][st][i] = bn_wload(wres, wv[i], (((cs * TC + i) * chunks + m) * 4 + st) * 1024);
    };
    if (m0 < m1) ask_w(std::integral_constant<int, 0>{}, m0);
    if (m0 + 1 < m1) ask_w(std::integral_constant<int, 1>{}, m0 + 1);

    int group_no = 0, c0 = cs * BC;
    if (ST(sub) > 1) {                               // (of 32 channels or whole multiples)
        const int each = (cout + BC - 1) / BC;
        group_no = cs / each;
        c0 = (cs - group_no * each) * BC;
    }
    // ---- pixels of the rows that this lane loads: lane / 8 + 8 i, 16 bytes of the chunk's 128
    const int W = ST(W), H = ST(H), window = ST(window);
    const bool no_pad = window == 0x0101;            // one tap, inside for every output pixel
    const unsigned x_at = (unsigned)(ST(xc0) + group_no * cin) * 2u;
    const __amdgpu_buffer_rsrc_t xres = ch_rsrc(base + ST_L(x) * images, (unsigned)(images * H * W) * (unsigned)xs * 2u);
    const int r8 = lane >> 3, piece = (lane & 7) ^ r8;
    const int kw_n = window >> 8 & 255;
    unsigned xo[4 * TP];
    unsigned taps[4 * TP];                           // bit kh * kw_n + kw: that tap is inside the image
    if (no_pad && (ST(stride) & 0xFFFF) == 0x0101) {
        const int first = __mul24(p0 + r8, xs) * 2 + (int)x_at, step = xs * 16, most = __mul24(P - 1, xs) * 2 + (int)x_at;
#pragma unroll
        for (int i = 0; i < 4 * TP; i++) xo[i] = (unsigned)min(first + i * step, most);
    } else {
        // a lane works one pixel out, the loads pick theirs
        const int Wo = ST(Wo), Ho = ST(Ho), stride = ST(stride), p = min(p0 + (lane & (BP - 1)), P - 1);
        const int row = ch_div(p, Wo, ST_F(inv_wo)), n = ch_div(row, Ho, ST_F(inv_ho));
        const int hi = __mul24(row - __mul24(n, Ho), stride & 255) - (window >> 16 & 255), wi = __mul24(p - __mul24(row, Wo), stride >> 8 & 255) - (int)((unsigned)window >> 24);
        const int off = ((n * H + hi) * W + wi) * xs * 2 + (int)x_at;
        unsigned mask = ~0u;
        if (ST(padded)) {
            // (a filter of up to 32 taps in a row, or a window up to 255 columns outside: counts of 32 are no shifts of 32 bits)
            const unsigned cols = (unsigned)((1ull << min(kw_n, W - wi)) - (1ull << min(kw_n, max(0, -wi))));
            const int kh_n = window & 255;
            mask = 0;
            for (int kh = 0; kh < kh_n; kh++) mask |= (unsigned)(hi + kh) < (unsigned)H ? cols << (kh * kw_n) : 0u;
        }
#pragma unroll
        for (int i = 0; i < 4 * TP; i++) {
            xo[i] = (unsigned)__shfl(off, r8 + 8 * i, 64);
            taps[i] = (unsigned)__shfl((int)mask, r8 + 8 * i, 64);
        }
    }
    int k = 64 * m0 + 8 * piece, tap = 0, kw = 0, c = k, at = 0;   // at: bytes from the first tap's pixel to this tap's
    if (!no_pad) {
        tap = ch_div(min(k, K - 1), cin, ST_F(inv_cin));
        c = k - tap * cin;
        const int kh = ch_div(tap, kw_n, ST_F(inv_kw));
        kw = tap - kh * kw_n;
        at = __mul24(__mul24(kh, W) + kw, xs) * 2;
    }
    unsigned char* const mine = lds + wave * CH_WAVE_LDS;
    auto ask_x = [&](int stage) {
        unsigned char* const d = mine + stage * STAGE;
        const bool kok = k < K;
        if (no_pad) {
            const unsigned to = kok ? (unsigned)k * 2u : OOBV;
#pragma unroll
            for (int i = 0; i < 4 * TP; i++) __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_ptr_t)(d + i * 1024), LDS_LOAD_BYTES, xo[i] + to, 0, 0, SC1);
        } else {
            // (more than 32 taps are taken by layers only of which none is outside: all bits are set)
            const unsigned to = (unsigned)(at + c * 2), bit = kok ? 1u << (tap & 31) : 0u;
#pragma unroll
            for (int i = 0; i < 4 * TP; i++)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_ptr_t)(d + i * 1024), LDS_LOAD_BYTES, taps[i] & bit ? xo[i] + to : OOBV, 0, 0, SC1);
            c += 64;
            while (c >= cin) {
                c -= cin;
                tap++;
                at += xs * 2;
                if (++kw == kw_n) { kw = 0; at += (W - kw_n) * xs * 2; }
            }
        }
        k += 64;
    };
    // ---- scale and bias of the channels whose results this thread finishes: the tile's results are dealt to the threads of its
    // wavefronts in groups of V channels of a pixel
    const int tin = kpart * 64 + lane, lg_v = T == 1 ? min(3, 4 - lg) : 3;
    const int oc = c0 + ((tin << lg_v) & (BC - 1));
    const bool ch_ok = oc < cout;
    f32x4 b0{0.f, 0.f, 0.f, 0.f}, b1 = b0, s0 = b0, s1 = b0;
    if (ch_ok) {
        const float *bp = (const float*)ST_P(bias) + group_no * cout + oc, *sp = (const float*)ST_P(scale) + group_no * cout + oc;
        if (lg_v == 1) {
            b0[0] = ENS_GLOBAL(float, bp)[0]; b0[1] = ENS_GLOBAL(float, bp)[1];
            s0[0] = ENS_GLOBAL(float, sp)[0]; s0[1] = ENS_GLOBAL(float, sp)[1];
        } else {
            b0 = *ENS_GLOBAL(f32x4, bp);
            s0 = *ENS_GLOBAL(f32x4, sp);
            if (lg_v == 3) { b1 = *ENS_GLOBAL(f32x4, bp + 4); s1 = *ENS_GLOBAL(f32x4, sp + 4); }
        }
    }
    float* const tab = (float*)(lds + CH_TABLE_AT);
    const int kpad = chunks * 64;
    if constexpr (PRE) {
        for (int i = t; i < kpad; i += CHAIN_THREADS) {
            tab[i] = i < K ? ENS_GLOBAL(float, (const float*)ST_P(pre_scale))[i] : 0.f;
            tab[kpad + i] = i < K ? ENS_GLOBAL(float, (const float*)ST_P(pre_shift))[i] : 0.f;
        }
    }
    group.wait(s0_);                                 // what the layers before wrote
    if constexpr (PRE) __syncthreads();
    const bool has_res = ST(res_present) != 0;
    constexpr int ALL = BP * BC / 64;                // results of a lane if its wavefront had the tile to itself
    uint32_t resv[ALL / 2];
    auto ask_res = [&](auto lg_c) {
        constexpr int SPLIT = 1 << decltype(lg_c)::value, V = ALL / SPLIT < 8 ? ALL / SPLIT : 8, N = ALL / SPLIT / V, GP = BC / V;
        const int rs = ST(rs), row0 = tin / GP, step = SPLIT * 64 / GP;
        const __amdgpu_buffer_rsrc_t rr = ch_rsrc(base + ST_L(res) * images, (unsigned)P * (unsigned)rs * 2u);
        const unsigned first = (unsigned)(__mul24(p0 + row0, rs) + ST(rc0) + group_no * cout + oc) * 2u;
#pragma unroll
        for (int i = 0; i < N; i++) {
            const unsigned off = ch_ok && p0 + row0 + i * step < P ? first + (unsigned)(i * step * rs * 2) : OOBV;
            if constexpr (V == 8) {
                const u32x4 v = ch_load16(rr, off);
#pragma unroll
                for (int e = 0; e < 4; e++) resv[4 * i + e] = v[e];
            } else {
#pragma unroll
                for (int e = 0; e < V / 2; e++) resv[e] = __builtin_amdgcn_raw_buffer_load_b32(rr, off + 4 * e, 0, SC1);
            }
        }
    };
    auto by_split = [&](auto&& f) {
        switch (lg) {
            case 0: f(std::integral_constant<int, 0>{}); break;
            case 1: f(std::integral_constant<int, 1>{}); break;
            case 2: f(std::integral_constant<int, 2>{}); break;
            default: f(std::integral_constant<int, 3>{}); break;
        }
    };
    if (m0 < m1) ask_x(0);
    if (m0 + 1 < m1) ask_x(1);
    if (T == 1 && has_res) by_split(ask_res);        // (a wide tile has no registers for them before its accumulators are free)

    f32x16 acc[TC][TP];
#pragma unroll
    for (int i = 0; i < TC; i++)
#pragma unroll
        for (int j = 0; j < TP; j++) bn_zero(acc[i][j]);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)mine + (uint32_t)(lrow * 128);
    auto chunk = [&](auto buf, int m) {
        constexpr int B = decltype(buf)::value;
        // issued behind chunk m's pixels: the next chunk's, and what was asked for since (residuals in front of the first chunk)
        if (m + 1 >= m1) bn_wait_vm<0>();
        else if (m == m0) bn_wait_vm<4 * T>();
        else bn_wait_vm<8 * T>();
        const uint32_t at0 = lds0 + (uint32_t)(B * STAGE);
        // two halves of two matrix-core steps: as many fragment registers as the accumulators leave room for
        bn_unroll<2>([&](auto half_c) {
            constexpr int half = decltype(half_c)::value;
            bf16x8 xf[2][TP];
            bn_unroll<2>([&](auto q_c) {
                constexpr int q = decltype(q_c)::value;
                const uint32_t at = at0 + (uint32_t)(((4 * half + 2 * q + lhalf) ^ (lrow & 7)) << 4);
                bn_unroll<TP>([&](auto j) { xf[q][decltype(j)::value] = bn_lds_read<decltype(j)::value * 4096>(at); });
            });
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
                for (int j = 0; j < TP; j++) bn_tie(xf[q][j]);
            if (half == 1 && m + 2 < m1) ask_x(B);   // into the buffer just read
#pragma unroll
            for (int q = 0; q < 2; q++) {
                if constexpr (PRE) {
                    const float* tp = tab + 64 * m + 32 * half + 16 * q + 8 * lhalf;
                    const f32x4 e0 = *(const f32x4*)tp, e1 = *(const f32x4*)(tp + 4), h0 = *(const f32x4*)(tp + kpad), h1 = *(const f32x4*)(tp + kpad + 4);
#pragma unroll
                    for (int j = 0; j < TP; j++) {
                        float f[8];
                        ch_unpack(__builtin_bit_cast(u32x4, xf[q][j]), f);
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            f[e] = fmaxf(fmaf(f[e], e0[e], h0[e]), 0.f);
                            f[4 + e] = fmaxf(fmaf(f[4 + e], e1[e], h1[e]), 0.f);
                        }
                        xf[q][j] = __builtin_bit_cast(bf16x8, ch_pack(f));
                    }
                }
#pragma unroll
                for (int i = 0; i < TC; i++)
#pragma unroll
                    for (int j = 0; j < TP; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[B][2 * half + q][i], xf[q][j], acc[i][j], 0, 0, 0);
            }
        });
        if (m + 2 < m1) ask_w(buf, m + 2);
    };
    for (int m = m0; m < m1; m += 2) {
        chunk(std::integral_constant<int, 0>{}, m);
        if (m + 1 < m1) chunk(std::integral_constant<int, 1>{}, m + 1);
    }
    group.prefetch(s0_);
    // ---- the partial tiles, [pixel][channel] in groups of four that are shuffled by pixel, each wavefront's in its part of LDS
    float* const part = (float*)mine;
    if (live) {
#pragma unroll
        for (int j = 0; j < TP; j++)
#pragma unroll
            for (int i = 0; i < TC; i++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int f = (32 * i + 16 * (q >> 1) + 8 * lhalf + 4 * (q & 1)) / 4;
                    *(f32x4*)&part[(32 * j + lrow) * BC + ((f ^ (lrow & (BC / 4 - 1))) << 2)] =
                        f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                }
    }
    if (T > 1 && has_res) by_split(ask_res);
    __syncthreads();
    if (!live || !ch_ok) return;
    by_split([&](auto lg_c) {
        constexpr int SPLIT = 1 << decltype(lg_c)::value, V = ALL / SPLIT < 8 ? ALL / SPLIT : 8, N = ALL / SPLIT / V, GP = BC / V;
        const int ys = ST(ys), act = (ST(stride) >> 16 & 255), f = (tin & (GP - 1)) * V / 4, row0 = tin / GP, step = SPLIT * 64 / GP;
        const float* const sum0 = (const float*)(lds + (wave & ~(SPLIT - 1)) * CH_WAVE_LDS);
        const __amdgpu_buffer_rsrc_t yr = ch_rsrc(base + ST_L(y) * images, (unsigned)P * (unsigned)ys * 2u);
        const unsigned first = (unsigned)(__mul24(p0 + row0, ys) + ST(yc0) + group_no * cout + oc) * 2u;
#pragma unroll
        for (int i = 0; i < N; i++) {
            const int row = row0 + i * step, key = row & (BC / 4 - 1);
            float v[V];
            if constexpr (V >= 4) {
                f32x4 q[SPLIT][V / 4];
#pragma unroll
                for (int w = 0; w < SPLIT; w++)
#pragma unroll
                    for (int e = 0; e < V / 4; e++) q[w][e] = *(const f32x4*)(sum0 + w * (CH_WAVE_LDS / 4) + row * BC + (((f + e) ^ key) << 2));
#pragma unroll
                for (int e = 0; e < V; e++) {
                    v[e] = q[0][e / 4][e % 4];
#pragma unroll
                    for (int w = 1; w < SPLIT; w++) v[e] += q[w][e / 4][e % 4];
                }
            } else {
                typedef float f32x2 __attribute__((ext_vector_type(2)));
                f32x2 q[SPLIT];
#pragma unroll
                for (int w = 0; w < SPLIT; w++) q[w] = *(const f32x2*)(sum0 + w * (CH_WAVE_LDS / 4) + row * BC + ((f ^ key) << 2) + ((tin & 1) << 1));
#pragma unroll
                for (int e = 0; e < V; e++) {
                    v[e] = q[0][e];
#pragma unroll
                    for (int w = 1; w < SPLIT; w++) v[e] += q[w][e];
                }
            }
#pragma unroll
            for (int e = 0; e < V; e++) {
                v[e] = fmaf(v[e], e < 4 ? s0[e & 3] : s1[e & 3], e < 4 ? b0[e & 3] : b1[e & 3]);
                if (has_res) v[e] += __uint_as_float(e & 1 ? resv[(V * i + e) / 2] & 0xFFFF0000u : resv[(V * i + e) / 2] << 16);
            }
            apply_act_n<V>(v, act);
            uint32_t o[V / 2];
#pragma unroll
            for (int e = 0; e < V / 2; e++) o[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
            const unsigned off = p0 + row < P ? first + (unsigned)(i * step * ys * 2) : OOBV;   // (rows past the last pixel are dropped by the range check)
            if constexpr (V == 8) __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[0], o[1], o[2], o[3]}, yr, off, 0, 0);
            else if constexpr (V == 4) __builtin_amdgcn_raw_buffer_store_b64(u32x2{o[0], o[1]}, yr, off, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b32(o[0], yr, off, 0, 0);
        }
    });
}

// ---- depthwise layer: a unit is an image, 64 channels and a strip of rows, whose window comes into LDS in one round trip; it leaves
// the strip's channel sums when asked to.  (A lane per run of four columns that took its rows from memory one after the other: 11 to 18 us.)
constexpr int CH_DW_SUMS_AT = CHAIN_DW_SLOTS * 128;
static_assert(CH_DW_SUMS_AT + 64 * 68 * 4 <= CH_TABLE_AT, "sums beside the window");
template <int KK, int S>
__device__ __forceinline__ void chain_dw(const Step s, const Step s0_, char* const base, const int images, const int unit, unsigned char* const lds, ChainGroup& group) {
    constexpr int NW = 4, NCOL = (NW - 1) * S + KK;
    const int t = ch_thread(), lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), c_n = ST(cin), cb = (c_n + 63) / 64, rows = ST(rows);
    const int H = ST(H), W = ST(W), Ho = ST(Ho), Wo = ST(Wo), xs = ST(xs), ys = ST(ys);
    const int n = unit / (cb * rows), u = unit - n * (cb * rows), strip = u / cb, c64 = (u - strip * cb) * 64, c = c64 + (t & 7) * 8;
    const int h_per = (Ho + rows - 1) / rows, h0 = strip * h_per, h1 = min(Ho, h0 + h_per);
    const int runs = (Wo + NW - 1) / NW, items = h1 > h0 ? (h1 - h0) * runs : 0;
    const int cols = (runs * NW - 1) * S + KK, slots = h1 > h0 ? ((h1 - h0 - 1) * S + KK) * cols : 0;
    const bool c_ok = c < c_n;
    unsigned char* const wlds = lds + CH_TABLE_AT;
    if (wave * 8 < KK * KK) {                        // the filter: a tap's 64 channels in 128 bytes
        const int tap = wave * 8 + (lane >> 3);
        const __amdgpu_buffer_rsrc_t wr = ch_rsrc(ST_P(w), (unsigned)(KK * KK) * (unsigned)c_n * 2u);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (lds_ptr_t)(wlds + wave * 1024), LDS_LOAD_BYTES, tap < KK * KK && c_ok ? (unsigned)(tap * c_n + c) * 2u : 0x80000000u, 0, 0, 0);
    }
    f32x4 b0{0.f, 0.f, 0.f, 0.f}, b1 = b0, s0 = b0, s1 = b0;
    if (c_ok) {
        b0 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(bias)) + c); b1 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(bias)) + c + 4);
        s0 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(scale)) + c); s1 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(scale)) + c + 4);
    }
    group.wait(s0_);
    {
        const __amdgpu_buffer_rsrc_t xr = ch_rsrc(base + ST_L(x) * images + (size_t)n * H * W * xs * 2, (unsigned)(H * W) * (unsigned)xs * 2u);
        const float inv = __builtin_amdgcn_rcpf((float)cols);
        const int window = ST(window), hi0 = h0 * S - (window >> 16 & 255), wi0 = -(int)((unsigned)window >> 24);
        for (int q0 = wave * 8; q0 < slots; q0 += CHAIN_WAVES * 8) {
            const int q = q0 + (lane >> 3), r = ch_div(q, cols, inv), hi = hi0 + r, wi = wi0 + q - r * cols;
            const bool ok = q < slots && c_ok && (unsigned)hi < (unsigned)H && (unsigned)wi < (unsigned)W;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_ptr_t)(lds + q0 * 128), LDS_LOAD_BYTES, ok ? (unsigned)((hi * W + wi) * xs + ST(xc0) + c) * 2u : 0x80000000u, 0, 0, SC1);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (c_ok) {
        const float inv = __builtin_amdgcn_rcpf((float)runs);
        const int act = (ST(stride) >> 16 & 255);
        uint16_t* const y = (uint16_t*)(base + ST_L(y) * images) + (size_t)n * Ho * Wo * ys + ST(yc0) + c;
        for (int it = t >> 3; it < items; it += CHAIN_THREADS / 8) {
            const int hr = ch_div(it, runs, inv), ho = h0 + hr, wo0 = (it - hr * runs) * NW;
            float acc[NW][8];
#pragma unroll
            for (int o = 0; o < NW; o++)
#pragma unroll
                for (int e = 0; e < 8; e++) acc[o][e] = 0.f;
            const u32x4* const win = (const u32x4*)(lds + ((hr * S) * cols + wo0 * S) * 128 + (t & 7) * 16);
#pragma unroll 1
            for (int kh = 0; kh < KK; kh++) {
                float wf[KK][8];
#pragma unroll
                for (int q = 0; q < KK; q++) ch_unpack(*(const u32x4*)(wlds + (kh * KK + q) * 128 + (t & 7) * 16), wf[q]);
#pragma unroll
                for (int j = 0; j < NCOL; j++) {
                    float xf[8];
                    ch_unpack(win[(kh * cols + j) * 8], xf);
#pragma unroll
                    for (int o = 0; o < NW; o++) {
                        const int q = j - o * S;
                        if (q >= 0 && q < KK) {
#pragma unroll
                            for (int e = 0; e < 8; e++) acc[o][e] = fmaf(xf[e], wf[q][e], acc[o][e]);
                        }
                    }
                }
            }
#pragma unroll
            for (int o = 0; o < NW; o++) {
                if (wo0 + o >= Wo) break;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    acc[o][e] = fmaf(acc[o][e], s0[e], b0[e]);
                    acc[o][4 + e] = fmaf(acc[o][4 + e], s1[e], b1[e]);
                }
                apply_act_n<8>(acc[o], act);
                const u32x4 packed = ch_pack(acc[o]);
                *ENS_GLOBAL_W(u32x4, y + (size_t)(ho * Wo + wo0 + o) * ys) = packed;
                float r[8];
                ch_unpack(packed, r);
#pragma unroll
                for (int e = 0; e < 8; e++) sum[e] += r[e];
            }
        }
    }
    if (ST_L(scratch) < 0) return;
    float* const red = (float*)(lds + CH_DW_SUMS_AT);   // [64 lanes][64 channels], a lane's rows apart by 68 floats
#pragma unroll
    for (int e = 0; e < 8; e++) red[(t >> 3) * 68 + (t & 7) * 8 + e] = sum[e];
    __syncthreads();
    if (t < 64 && c64 + t < c_n) {
        float v = 0.f;
#pragma unroll
        for (int l = 0; l < 64; l++) v += red[l * 68 + t];
        ((float*)(base + ST_L(scratch) * images))[(size_t)n * ST(scratch_stride) + (size_t)strip * c_n + c64 + t] = v;
    }
}

// ---- pooling: a lane per pixel and 8 channels, CH_POOL of them at a time
template <int KK>
__device__ __forceinline__ void chain_pool(const Step s, char* const base, const int images, const int unit, const bool is_max) {
    const int cv = ST(cin) / 8, H = ST(H), W = ST(W), Ho = ST(Ho), Wo = ST(Wo), xs = ST(xs);
    const int window = ST(window), stride = ST(stride), kh_n = KK ? KK : window & 255, kw_n = KK ? KK : window >> 8 & 255, total = images * Ho * Wo * cv;
    const __amdgpu_buffer_rsrc_t xr = ch_rsrc(base + ST_L(x) * images, (unsigned)images * (unsigned)(H * W) * (unsigned)xs * 2u);
    const bool pre = ((const float*)ST_P(pre_scale)) != nullptr;
    const float inv_cv = __builtin_amdgcn_rcpf((float)cv);
    int p[CH_POOL], c[CH_POOL], n[CH_POOL], hi0[CH_POOL], wi0[CH_POOL], cnt[CH_POOL];
    float acc[CH_POOL][8];
#pragma unroll
    for (int k = 0; k < CH_POOL; k++) {
        const int idx = min((unit * CH_POOL + k) * CHAIN_THREADS + ch_thread(), total - 1);
        p[k] = ch_div(idx, cv, inv_cv);
        c[k] = (idx - p[k] * cv) * 8;
        const int row = ch_div(p[k], Wo, ST_F(inv_wo));
        n[k] = ch_div(row, Ho, ST_F(inv_ho));
        hi0[k] = (row - n[k] * Ho) * (stride & 255) - (window >> 16 & 255);
        wi0[k] = (p[k] - row * Wo) * (stride >> 8 & 255) - (int)((unsigned)window >> 24);
        cnt[k] = 0;
#pragma unroll
        for (int e = 0; e < 8; e++) acc[k][e] = is_max ? -3.0e38f : 0.f;
    }
    auto row_of = [&](int kh) {
        constexpr int U = KK ? KK : 1;
        for (int kw0 = 0; kw0 < kw_n; kw0 += U) {
            u32x4 v[CH_POOL][U];
#pragma unroll
            for (int k = 0; k < CH_POOL; k++)
#pragma unroll
                for (int q = 0; q < U; q++) {
                    const int hi = hi0[k] + kh, wi = wi0[k] + kw0 + q;
                    v[k][q] = ch_load16(xr, (unsigned)hi < (unsigned)H && (unsigned)wi < (unsigned)W ? (unsigned)(((n[k] * H + hi) * W + wi) * xs + ST(xc0) + c[k]) * 2u : 0x80000000u);
                }
#pragma unroll
            for (int k = 0; k < CH_POOL; k++)
#pragma unroll
                for (int q = 0; q < U; q++) {
                    const int hi = hi0[k] + kh, wi = wi0[k] + kw0 + q;
                    if (!((unsigned)hi < (unsigned)H && (unsigned)wi < (unsigned)W)) continue;
                    float f[8];
                    ch_unpack(v[k][q], f);
                    if (pre) {
                        const f32x4 e0 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(pre_scale)) + c[k]), e1 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(pre_scale)) + c[k] + 4);
                        const f32x4 h0 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(pre_shift)) + c[k]), h1 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(pre_shift)) + c[k] + 4);
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            f[e] = fmaxf(fmaf(f[e], e0[e], h0[e]), 0.f);
                            f[4 + e] = fmaxf(fmaf(f[4 + e], e1[e], h1[e]), 0.f);
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; e++) acc[k][e] = is_max ? fmaxf(acc[k][e], f[e]) : acc[k][e] + f[e];
                    cnt[k]++;
                }
        }
    };
    if constexpr (KK != 0) {
#pragma unroll
        for (int kh = 0; kh < KK; kh++) row_of(kh);
    } else {
        for (int kh = 0; kh < kh_n; kh++) row_of(kh);
    }
#pragma unroll
    for (int k = 0; k < CH_POOL; k++) {
        if ((unit * CH_POOL + k) * CHAIN_THREADS + ch_thread() >= total) break;
        if (!is_max) {
            const float inv = 1.f / (float)max(cnt[k], 1);
#pragma unroll
            for (int e = 0; e < 8; e++) acc[k][e] *= inv;
        }
        apply_act_n<8>(acc[k], (ST(stride) >> 16 & 255));
        *ENS_GLOBAL_W(u32x4, (uint16_t*)(base + ST_L(y) * images) + (size_t)p[k] * ST(ys) + ST(yc0) + c[k]) = ch_pack(acc[k]);
    }
}

// ---- means over an image's pixels: a unit is an image and 64 channels.  To fp32 (global pooling, CH_GAP) or as a row of sums (CH_SE_SUM)
__device__ __forceinline__ void chain_mean(const Step s, char* const base, const int images, const int unit, unsigned char* const lds) {
    const int t = ch_thread(), c_n = ST(cin), cb = (c_n + 63) / 64, HW = ST(H) * ST(W), xs = ST(xs);
    const int n = unit / cb, c64 = (unit - n * cb) * 64, c = c64 + (t & 7) * 8;
    float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (c < c_n) {
        const __amdgpu_buffer_rsrc_t xr = ch_rsrc(base + ST_L(x) * images + (size_t)n * HW * xs * 2, (unsigned)HW * (unsigned)xs * 2u);
        const bool pre = ((const float*)ST_P(pre_scale)) != nullptr && ST(kind) == CH_GAP;
        f32x4 e0, e1, h0, h1;
        if (pre) {
            e0 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(pre_scale)) + c); e1 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(pre_scale)) + c + 4);
            h0 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(pre_shift)) + c); h1 = *ENS_GLOBAL(f32x4, ((const float*)ST_P(pre_shift)) + c + 4);
        }
        constexpr int U = 4;
        for (int p = t >> 3; p < HW; p += U * (CHAIN_THREADS / 8)) {
            u32x4 v[U];
#pragma unroll
            for (int q = 0; q < U; q++) {
                const int pq = p + q * (CHAIN_THREADS / 8);
                v[q] = ch_load16(xr, pq < HW ? (unsigned)(pq * xs + ST(xc0) + c) * 2u : 0x80000000u);
            }
#pragma unroll
            for (int q = 0; q < U; q++) {
                if (p + q * (CHAIN_THREADS / 8) >= HW) break;
                float f[8];
                ch_unpack(v[q], f);
                if (pre) {
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        f[e] = fmaxf(fmaf(f[e], e0[e], h0[e]), 0.f);
                        f[4 + e] = fmaxf(fmaf(f[4 + e], e1[e], h1[e]), 0.f);
                    }
                }
#pragma unroll
                for (int e = 0; e < 8; e++) sum[e] += f[e];
            }
        }
    }
    float* const red = (float*)lds;
#pragma unroll
    for (int e = 0; e < 8; e++) red[(t >> 3) * 68 + (t & 7) * 8 + e] = sum[e];
    __syncthreads();
    if (t < 64 && c64 + t < c_n) {
        float v = 0.f;
        for (int l = 0; l < 64; l++) v += red[l * 68 + t];
        if (ST(kind) == CH_GAP) ((float*)(base + ST_L(y) * images))[(size_t)n * ST(ys) + ST(yc0) + c64 + t] = v / (float)HW;
        else ((float*)(base + ST_L(scratch) * images))[(size_t)n * ST(scratch_stride) + c64 + t] = v;
    }
}

__device__ __forceinline__ float ch_load_f(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// ---- squeeze-excite, hidden values: a unit is an image and CHAIN_WAVES hidden units, one per wavefront
__device__ __forceinline__ void chain_hidden(const Step s, char* const base, const int images, const int unit, unsigned char* const lds) {
    const int t = ch_thread(), lane = t & 63, wave = t >> 6, c_n = ST(cin), r_n = ST(r), rows = ST(rows);
    const int ub = (r_n + CHAIN_WAVES - 1) / CHAIN_WAVES, n = unit / ub, r = (unit - n * ub) * CHAIN_WAVES + wave;
    float* const mean = (float*)(lds + CH_TABLE_AT);
    float* const sc = (float*)(base + ST_L(scratch) * images) + (size_t)n * ST(scratch_stride);
    const float inv = 1.f / (float)(ST(H) * ST(W));
    for (int c = t; c < c_n; c += CHAIN_THREADS) {
        float m = 0.f;
        for (int k0 = 0; k0 < rows; k0 += 8) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; k++) v[k] = k0 + k < rows ? ch_load_f(sc + (size_t)(k0 + k) * c_n + c) : 0.f;
#pragma unroll
            for (int k = 0; k < 8; k++) m += v[k];
        }
        mean[c] = m * inv;
    }
    __syncthreads();
    if (r >= r_n) return;
    const float* const w1 = (const float*)ST_P(w);
    float acc = 0.f;
    for (int c0 = lane; c0 < c_n; c0 += 64 * 8) {
        float w[8];
#pragma unroll
        for (int u = 0; u < 8; u++) w[u] = c0 + 64 * u < c_n ? ENS_GLOBAL(float, w1)[(size_t)(c0 + 64 * u) * r_n + r] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; u++) acc = fmaf(c0 + 64 * u < c_n ? mean[c0 + 64 * u] : 0.f, w[u], acc);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) {
        const float z = acc + ENS_GLOBAL(float, ((const float*)ST_P(bias)))[r];
        sc[ST(hidden_at) + r] = z / (1.f + __expf(-z));
    }
}

// ---- squeeze-excite, gates and rescaling: a unit is an image, 64 channels and a strip of pixels
__device__ __forceinline__ void chain_apply(const Step s, char* const base, const int images, const int unit, unsigned char* const lds) {
    const int t = ch_thread(), c_n = ST(cin), cb = (c_n + 63) / 64, r_n = ST(r), strips = ST(sub), HW = ST(H) * ST(W);
    const int n = unit / (cb * strips), u = unit - n * (cb * strips), strip = u / cb, c64 = (u - strip * cb) * 64;
    const float* const sc = (const float*)(base + ST_L(scratch) * images) + (size_t)n * ST(scratch_stride) + ST(hidden_at);
    float* const tab = (float*)(lds + CH_TABLE_AT);  // [0, 64) gates, [64, 64 + 512) partial sums, then the hidden values
    for (int r = t; r < r_n; r += CHAIN_THREADS) tab[1024 + r] = ch_load_f(sc + r);
    __syncthreads();
    {
        const int c = c64 + (t & 63), part = t >> 6;
        float acc = 0.f;
        if (c < c_n)
            for (int r0 = part; r0 < r_n; r0 += CHAIN_WAVES * 8) {
                float w[8];
#pragma unroll
                for (int q = 0; q < 8; q++) w[q] = r0 + q * CHAIN_WAVES < r_n ? ENS_GLOBAL(float, ((const float*)ST_P(scale)))[(size_t)(r0 + q * CHAIN_WAVES) * c_n + c] : 0.f;
#pragma unroll
                for (int q = 0; q < 8; q++) acc = fmaf(r0 + q * CHAIN_WAVES < r_n ? tab[1024 + r0 + q * CHAIN_WAVES] : 0.f, w[q], acc);
            }
        tab[64 + t] = acc;
    }
    __syncthreads();
    if (t < 64) {
        float z = c64 + t < c_n ? ENS_GLOBAL(float, ((const float*)ST_P(pre_scale)))[c64 + t] : 0.f;
#pragma unroll
        for (int q = 0; q < CHAIN_WAVES; q++) z += tab[64 + 64 * q + t];
        tab[t] = 1.f / (1.f + __expf(-z));
    }
    __syncthreads();
    const int c = c64 + (t & 7) * 8, per = (HW + strips - 1) / strips, p0 = strip * per, p1 = min(HW, p0 + per);
    if (c >= c_n) return;
    float g[8];
#pragma unroll
    for (int e = 0; e < 8; e++) g[e] = tab[(t & 7) * 8 + e];
    const int xs = ST(xs);
    const __amdgpu_buffer_rsrc_t xr = ch_rsrc(base + ST_L(x) * images + (size_t)n * HW * xs * 2, (unsigned)HW * (unsigned)xs * 2u);
    uint16_t* const y = (uint16_t*)(base + ST_L(y) * images) + (size_t)n * HW * ST(ys) + ST(yc0) + c;
    constexpr int U = 4, STEP = CHAIN_THREADS / 8;
    for (int p = p0 + (t >> 3); p < p1; p += U * STEP) {
        u32x4 v[U];
#pragma unroll
        for (int q = 0; q < U; q++) v[q] = ch_load16(xr, p + q * STEP < p1 ? (unsigned)((p + q * STEP) * xs + ST(xc0) + c) * 2u : 0x80000000u);
#pragma unroll
        for (int q = 0; q < U; q++) {
            if (p + q * STEP >= p1) break;
            float f[8];
            ch_unpack(v[q], f);
#pragma unroll
            for (int e = 0; e < 8; e++) f[e] *= g[e];
            *ENS_GLOBAL_W(u32x4, y + (size_t)(p + q * STEP) * ST(ys)) = ch_pack(f);
        }
    }
}

// ---- FC head (fc_mfma.hip): a unit is 32 classes x 32 images, K split over the wavefronts
__device__ __forceinline__ void chain_fc(const Step s, const Step s0_, char* const base, float* const logits, const int images, const int first, const int unit, unsigned char* const lds, ChainGroup& group) {
    const int t = ch_thread(), lane = t & 63, lrow = lane & 31, lhalf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int K = ST(cin), classes = ST(cout), cblocks = (classes + 31) / 32;
    const int nblk = unit / cblocks, c0 = (unit - nblk * cblocks) * 32, n = nblk * 32 + lrow;
    const int NS = (K + 63) / 64 * 4, steps = (K + 15) / 16, per = (steps + CHAIN_WAVES - 1) / CHAIN_WAVES;
    const int s_begin = wave * per, s_end = min(steps, s_begin + per);
    const __amdgpu_buffer_rsrc_t wres = ch_rsrc(ST_P(w), (unsigned)cblocks * (unsigned)NS * 1024u);
    constexpr unsigned OOBV = 0x80000000u;
    const __amdgpu_buffer_rsrc_t xres = ch_rsrc(base + ST_L(x) * images, (unsigned)images * (unsigned)K * 4u);
    const unsigned wv = (unsigned)((c0 / 32) * NS * 1024 + lane * 16), xv = n < images ? (unsigned)((n * K + 8 * lhalf) * 4) : OOBV;
    f32x16 acc;
    bn_zero(acc);
    constexpr int U = 8;
    bf16x8 wf[U];
    auto ask_w = [&](int q0) {
#pragma unroll
        for (int u = 0; u < U; u++) wf[u] = bn_wload(wres, q0 + u < s_end ? wv : OOBV, (q0 + u) * 1024);
    };
    ask_w(s_begin);
    group.wait(s0_);
    for (int q0 = s_begin; q0 < s_end; q0 += U) {
        u32x4 x0[U], x1[U];
        if (q0 > s_begin) ask_w(q0);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int q = q0 + u;
            const bool live = q < s_end && 16 * q + 8 * lhalf + 8 <= K && xv != OOBV;
            x0[u] = ch_load16(xres, live ? xv + q * 64 : OOBV);
            x1[u] = ch_load16(xres, live ? xv + q * 64 + 16 : OOBV);
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const float f0 = __uint_as_float(e < 2 ? x0[u][2 * e] : x1[u][2 * e - 4]), f1 = __uint_as_float(e < 2 ? x0[u][2 * e + 1] : x1[u][2 * e - 3]);
                hi[e] = pack_bf16x2(f0, f1);
                lo[e] = pack_bf16x2(f0 - __uint_as_float(hi[e] << 16), f1 - __uint_as_float(hi[e] & 0xFFFF0000u));
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u], __builtin_bit_cast(bf16x8, u32x4{hi[0], hi[1], hi[2], hi[3]}), acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u], __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], lo[2], lo[3]}), acc, 0, 0, 0);
        }
    }
    float* const red = (float*)lds;
#pragma unroll
    for (int v = 0; v < 16; v++) red[(wave * 16 + v) * 64 + lane] = acc[v];
    __syncthreads();
    // register v of lane l: class 16 (v / 8) + 8 (l / 32) + v % 8 of image l % 32; 1024 results, two per thread
#pragma unroll
    for (int i = 0; i < 1024 / CHAIN_THREADS; i++) {
        const int id = t + i * CHAIN_THREADS, im = nblk * 32 + (id >> 5), cl = id & 31;
        const int v = 8 * (cl >> 4) + (cl & 7), l = (id >> 5) + 32 * ((cl >> 3) & 1);
        if (im >= images || c0 + cl >= classes) continue;
        float z = 0.f;
#pragma unroll
        for (int w = 0; w < CHAIN_WAVES; w++) z += red[(w * 16 + v) * 64 + l];
        logits[(size_t)(first + im) * classes + c0 + cl] = z + ENS_GLOBAL(float, ((const float*)ST_P(bias)))[c0 + cl];
    }
}

// ---- input staging: a lane per pixel of the member's input tensor (layers.hip)
__device__ __forceinline__ void chain_stage(const Step s, char* const base, const int images, const float* src_all, const int base_h, const int base_w, const int first, const int unit) {
    const int dh = ST(H), dw = ST(W), th = ST(Ho), tw = ST(Wo), px = th * tw, per = (px + CHAIN_THREADS - 1) / CHAIN_THREADS;
    const int n = unit / per, idx = (unit - n * per) * CHAIN_THREADS + ch_thread();
    if (idx >= px) return;
    const int r = ch_div(idx, tw, __builtin_amdgcn_rcpf((float)tw)), q = idx - r * tw;
    const float* const src = src_all + (size_t)(first + n) * base_h * base_w * 3;
    uint16_t* const d = (uint16_t*)(base + ST_L(y) * images) + ((size_t)n * px + idx) * ST(ys);
    if ((unsigned)ST(stride) >> 24) {
        float f[16];
#pragma unroll
        for (int e = 0; e < 16; e++) f[e] = 0.f;
#pragma unroll
        for (int by = 0; by < 2; by++)
#pragma unroll
            for (int bx = 0; bx < 2; bx++) {
                const int y = 2 * r + by, x = 2 * q + bx;
                if (y < dh && x < dw) stage_sample(base_h, base_w, dh, dw, src, y, x, f + (2 * by + bx) * 3);
            }
        *ENS_GLOBAL_W(u32x4, d) = ch_pack(f);
        *ENS_GLOBAL_W(u32x4, d + 8) = ch_pack(f + 8);
    } else {
        float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        stage_sample(base_h, base_w, dh, dw, src, r, q, f);
        *ENS_GLOBAL_W(u32x4, d) = ch_pack(f);
    }
}

// Units of a step: what one workgroup does at a time.
__device__ __forceinline__ int chain_units(const Step s, const int images, const int pick) {
    switch (ST(kind)) {
        case CH_STAGE: return images * ((ST(Ho) * ST(Wo) + CHAIN_THREADS - 1) / CHAIN_THREADS);
        case CH_CONV:
        case CH_CONV_PRE: {
            const int side = pick & 255, tiles = ((images * ST(Ho) * ST(Wo) + 32 * side - 1) >> (4 + side)) * st_int(s, offsetof(ChainStep, ctiles) / 4 + side - 1);
            return ((tiles << (pick >> 8 & 255)) + CHAIN_WAVES - 1) / CHAIN_WAVES;
        }
        case CH_DW: return images * ST(rows) * ((ST(cin) + 63) / 64);
        case CH_MAXPOOL:
        case CH_AVGPOOL: return (images * ST(Ho) * ST(Wo) * (ST(cin) / 8) + CH_POOL * CHAIN_THREADS - 1) / (CH_POOL * CHAIN_THREADS);
        case CH_SE_SUM:
        case CH_GAP: return images * ((ST(cin) + 63) / 64);
        case CH_SE_HIDDEN: return images * ((ST(r) + CHAIN_WAVES - 1) / CHAIN_WAVES);
        case CH_SE_APPLY: return images * ST(sub) * ((ST(cin) + 63) / 64);
        case CH_FC: return ((ST(cout) + 31) / 32) * ((images + 31) / 32);
    }
    return 0;
}

__global__ __launch_bounds__(CHAIN_THREADS) void chain_kernel(const ChainArgs a_) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const ChainArgs& a = a_;
    unsigned* const misc = (unsigned*)(lds + CH_MISC_AT);
    int* const steps = (int*)(lds + CH_STEPS_AT);
    const int t = threadIdx.x;
    const int xcd = (int)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & (CHAIN_GROUPS - 1));   // hwreg(XCC_ID), 4 bits
    auto& g = a.sync->group[xcd];
    constexpr unsigned CLOSED = 0x40000000u;
    if (t == 0) {
        const unsigned ticket = __hip_atomic_fetch_add(&g.count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        unsigned size = 0;
        if (ticket == 0) {
            // close the group when it is complete, or after 100 us: others' kernels hold a compute unit for less than that
            const unsigned want = gridDim.x / 8;
            const long long t0 = wall_clock64();
            while (__hip_atomic_load(&g.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want && wall_clock64() - t0 < 10000) __builtin_amdgcn_s_sleep(1);
            size = __hip_atomic_fetch_or(&g.count, CLOSED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned program = __hip_atomic_fetch_add(&a.sync->queue, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&g.program, program, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned before = __hip_atomic_load(&g.arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&g.arrived_before, before, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __hip_atomic_store(&g.size, size, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (ticket < CLOSED) {
            // (the first workgroup is running and closes the group)
            for (int i = 0; i < (1 << 23) && size == 0; i++) {
                size = __hip_atomic_load(&g.size, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (size == 0) __builtin_amdgcn_s_sleep(1);
            }
        }
        misc[1] = ticket;
        misc[2] = ticket < size ? size : 0;
        misc[3] = size ? __hip_atomic_load(&g.program, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        misc[4] = size ? __hip_atomic_load(&g.arrived_before, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    }
    __syncthreads();
    const unsigned ticket = __builtin_amdgcn_readfirstlane(misc[1]), size = __builtin_amdgcn_readfirstlane(misc[2]);
    if (size) {
        ChainGroup group{&g.arrived, (unsigned)__builtin_amdgcn_readfirstlane(misc[4]), size, ticket, misc, steps, nullptr, 0, 0, false, false, false, 0, {0u, 0u}};
        int program = __builtin_amdgcn_readfirstlane(misc[3]);
        while (program < a.n_programs && !group.dead) {
            const ChainProgram pr = a.programs[program];
            const int images = pr.images, first = pr.first, sz = pr.size;
            const int* words = (const int*)a.steps[pr.member];
            const int phases = a.phases[pr.member];
            char* const base = a.arena[pr.member] + (size_t)first * a.image_bytes[pr.member];
            {                                        // the first two phases' steps
                const int both = ENS_GLOBAL(int, words)[offsetof(ChainStep, phase_steps) / 4], n0 = both & 255, n1 = both >> 8;
                if (t < n0 * 64) steps[t] = ENS_GLOBAL(int, words)[t];
                if (t < n1 * 64) steps[CHAIN_PHASE_STEPS * 64 + t] = ENS_GLOBAL(int, words)[n0 * 64 + t];
                group.at = 0;
                __syncthreads();
            }
            for (int ph = 0; ph < phases && !group.dead; ph++) {
                const Step s0 = group.step(0);
                const int counts = st_int(s0, offsetof(ChainStep, phase_steps) / 4), ns = counts & 255;
                words += ns * 64;
                // while this phase runs the one after the next comes: its steps follow the next one's
                group.next = words;
                group.next_n = counts >> 8;
                int done = 0;                        // units of the steps before
                int u = (int)ticket;
                bool touched = false;                // LDS holds something of a unit of this phase
                for (int i = 0; i < ns; i++) {
                    const Step s = i == 0 ? s0 : group.step(i);
                    const int pick = st_int(s, offsetof(ChainStep, choice) / 4 + sz), kind = ST(kind);
                    const int units = images == 1 << sz ? (int)((unsigned)pick >> 16) : chain_units(s, images, pick);
                    for (; u < done + units; u += (int)size) {
                        if (touched) __syncthreads();
                        touched = true;
                        const int unit = u - done;
                        if (kind <= CH_CONV_PRE) {
                            const int lg = pick >> 8 & 255;
                            const bool narrow = (pick & 255) == 1;
                            if (kind == CH_CONV) {
                                if (narrow) chain_conv<1, false>(s, s0, base, images, unit, lg, lds, group);
                                else chain_conv<2, false>(s, s0, base, images, unit, lg, lds, group);
                            } else {
                                if (narrow) chain_conv<1, true>(s, s0, base, images, unit, lg, lds, group);
                                else chain_conv<2, true>(s, s0, base, images, unit, lg, lds, group);
                            }
                            continue;
                        }
                        if (kind != CH_DW && kind != CH_FC) group.wait(s0);
                        switch (kind) {
                            case CH_STAGE: chain_stage(s, base, images, a.src, a.base_h, a.base_w, first, unit); break;
                            case CH_DW:
                                if ((ST(window) & 255) == 3) {
                                    if ((ST(stride) & 255) == 1) chain_dw<3, 1>(s, s0, base, images, unit, lds, group); else chain_dw<3, 2>(s, s0, base, images, unit, lds, group);
                                } else {
                                    if ((ST(stride) & 255) == 1) chain_dw<5, 1>(s, s0, base, images, unit, lds, group); else chain_dw<5, 2>(s, s0, base, images, unit, lds, group);
                                }
                                break;
                            case CH_MAXPOOL:
                            case CH_AVGPOOL:
                                if ((ST(window) & 0xFFFF) == 0x0303) chain_pool<3>(s, base, images, unit, kind == CH_MAXPOOL);
                                else if ((ST(window) & 0xFFFF) == 0x0202) chain_pool<2>(s, base, images, unit, kind == CH_MAXPOOL);
                                else chain_pool<0>(s, base, images, unit, kind == CH_MAXPOOL);
                                break;
                            case CH_SE_SUM:
                            case CH_GAP: chain_mean(s, base, images, unit, lds); break;
                            case CH_SE_HIDDEN: chain_hidden(s, base, images, unit, lds); break;
                            case CH_SE_APPLY: chain_apply(s, base, images, unit, lds); break;
                            case CH_FC: chain_fc(s, s0, base, a.logits[pr.member], images, first, unit, lds, group); break;
                        }
                    }
                    done += units;
                }
                group.wait(s0);                      // also without a unit: nobody arrives twice
                group.prefetch(s0);
                if (ph + 1 == phases && ticket == 0 && t == 0) {
                    const unsigned next = __hip_atomic_fetch_add(&a.sync->queue, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(&g.program, next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                group.arrive();
            }
            group.next_n = 0;
            group.wait(Step{0});
            group.fetched = false;
            if (t == 0) misc[3] = __hip_atomic_load(&g.program, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            program = __builtin_amdgcn_readfirstlane(misc[3]);
            // nobody overwrites the word before everybody has read it: the next program's first barrier lies in between
        }
        if (group.dead && t == 0) __hip_atomic_store(a.failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    // the last workgroup of the launch leaves zeros
    if (t == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (__hip_atomic_fetch_add(&a.sync->gone, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) {
            for (int i = 0; i < CHAIN_GROUPS; i++) {
                auto& q = a.sync->group[i];
                __hip_atomic_store(&q.count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&q.size, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&q.program, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __hip_atomic_store(&a.sync->queue, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&a.sync->gone, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Weights [rows][K] in matrix-core operand order (conv_direct.h): blocks of 32 rows, steps of 16 columns, K padded to 64 with zeros; `groups` of them.
__global__ void chain_pack_kernel(const uint16_t* __restrict__ w, uint16_t* __restrict__ out, const int rows, const int K, const int blocks, const int steps, const long long total) {
    const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;     // 8 values of a lane
    if (id >= total) return;
    const int lane = (int)(id & 63), r = lane & 31;
    const long long rest = id >> 6;
    const int st = (int)(rest % steps), blk = (int)(rest / steps % blocks), g = (int)(rest / steps / blocks);
    const int row = 32 * blk + ((r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1)), col = 16 * st + 8 * (lane >> 5);
    u32x4 v{0u, 0u, 0u, 0u};
    if (row < rows && col < K) v = *(const u32x4*)(w + ((size_t)g * rows + row) * K + col);
    *(u32x4*)(out + id * 8) = v;
}

hipError_t launch_chain_pack(const void* w, void* out, int groups, int rows, int K, hipStream_t s) {
    if (!w || !out || groups <= 0 || rows <= 0 || K <= 0 || K % 8) return hipErrorInvalidValue;
    const int blocks = (rows + 31) / 32, steps = (K + 63) / 64 * 4;
    const long long total = (long long)groups * blocks * steps * 64;
    ENS_LAUNCH(chain_pack_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (const uint16_t*)w, (uint16_t*)out, rows, K, blocks, steps, total);
    return hipGetLastError();
}

hipError_t launch_chain(const ChainArgs& a, hipStream_t s) {
    if (!a.sync || !a.failed || !a.src || a.n_programs <= 0 || a.n_programs > CHAIN_MAX_PROGRAMS) return hipErrorInvalidValue;
    static const hipError_t raised = hipFuncSetAttribute((const void*)&chain_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, CH_LDS);
    if (raised != hipSuccess) return raised;
    ENS_LAUNCH(chain_kernel, dim3(256), dim3(CHAIN_THREADS), CH_LDS, s, a);
    return hipGetLastError();
}

}  // namespace ens

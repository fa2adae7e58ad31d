// Small fp32 members, an image at a time in the LDS of a compute unit (resident.hip).
#pragma once
#include "engine.h"

namespace ens {

enum ResidentKind { RS_CONV, RS_MAXPOOL, RS_AVGPOOL, RS_GAP, RS_FC };
enum ResidentPool { RS_NO_POOL, RS_MAX_POOL, RS_AVG_POOL, RS_MEAN_POOL };   // none, 2 x 2 / 2 windows, all pixels
constexpr int RESIDENT_THREADS = 512, RESIDENT_MAX_OPS = 32;

// One operation.  Places in LDS are in floats; a tensor's pixels are `p` floats apart, its rows `r`.  A wavefront holds an operation in one register,
// a dword a lane.
struct alignas(256) ResidentOp {
    int kind;
    int x, xp, xr, H, W, cin;  // x: of the first tap of output pixel (0, 0) for a convolution, of pixel (0, 0) otherwise
    int y, yp, yr, Ho, Wo, cout;
    int kh, kw, sh, sw, pt, pl;
    int act, steps;            // convolution: K = kh * kw * cin in steps of four
    int w, bias, taps;         // LDS: weights in tiles [16 channels][K][16] (FC: [K][cout]), biases, place of each k from the first tap's
    int pool;                  // convolution: what follows it in the same operation, RS_*_POOL: Ho x Wo is what that leaves
    int sums, sums_p;          // RS_MEAN_POOL: LDS for a row of sums per unit
    int pair;                  // weights and places for two neighbouring pixels at once: kh * (kw + 1) * cin of them, rows 0..7 and 8..15 the channels of either
    int odd, drawn;            // of operation 0: one more than the last image with an infinity or a NaN; the number last drawn for an image
};
static_assert(sizeof(ResidentOp) == 256, "a dword for each lane");

struct ResidentMember {
    const float* fixed;        // what LDS begins with: the operations, weights, biases and tap tables
    float* logits;
    float* input;              // of the worker's arena: the images that ens_debug_tensor runs the layers on again
    int n_ops, fixed_floats, lds_floats;
    int in, in_p, in_r, in_h, in_w;        // the input tensor
    int last_first, last_n;    // those images: the first worker's last batch
    int first_block, blocks;
};
struct ResidentArgs {
    ResidentMember member[8];
    const float* src;
    unsigned* queue;           // RESIDENT_MAX_MEMBERS + 1 zeros, which the launch leaves as zeros: images drawn by each member's workgroups beyond two each, workgroups gone
    int n_members, first, n, base_h, base_w, classes;   // images [first, first + n) of the request
};
static_assert(sizeof(ResidentArgs) <= 4000, "kernel arguments");
constexpr int RESIDENT_MAX_MEMBERS = 8, RESIDENT_LDS = 160 * 1024;

hipError_t launch_resident(const ResidentArgs& a, int lds_bytes, hipStream_t s);
// A member's operations in LDS, as engine.h's Resident; host only.  False: it does not fit, or has other operations.
bool build_resident(const Member& m, Resident* out);

}  // namespace ens

// A request of few images as chains: the operations of a member, one after the other, inside one kernel launch (chain.hip).
#pragma once
#include "engine.h"

namespace ens {

enum ChainKind { CH_CONV, CH_CONV_PRE, CH_STAGE, CH_DW, CH_MAXPOOL, CH_AVGPOOL, CH_SE_SUM, CH_SE_HIDDEN, CH_SE_APPLY, CH_GAP, CH_FC };

constexpr int CHAIN_THREADS = 512, CHAIN_WAVES = CHAIN_THREADS / 64;
constexpr int CHAIN_GROUPS = 16;             // XCDs that the kernel has a group word for (the GPU has 8)
constexpr int CHAIN_MAX_PROGRAMS = 192;
constexpr int CHAIN_TABLE_FLOATS = 4096;     // of LDS: pre-activation (scale and shift of up to 2048 channels), means, hidden values
constexpr int CHAIN_FAILED_WORD = 8;         // of the 16 words of ens_handle::flag: ChainArgs::failed
constexpr int CHAIN_DW_SLOTS = 880;          // pixels (of 64 channels) of a depthwise layer's strip that LDS holds beside the sums

// One operation; the steps of a phase follow each other, read nothing that another one of them writes and run side by side.
// Tensors are slices (x, y, res) of NHWC bf16 tensors.  A program of k images at `first` has the arena's bytes from first * image_bytes
// on, and there a tensor with place p in the layout of one image begins at k * p and holds its k images in a row: programs of a
// member share nothing, whatever their sizes.
// A wavefront holds a step in one register, a dword a lane, and reads fields by lane (chain.hip): 64 dwords.
struct alignas(256) ChainStep {
    int64_t x, y, res, scratch;   // places in bytes; res < 0: no residual; scratch: of a squeeze-excite block's sums and hidden values (< 0: none)
    const void* w;             // weights, of convolutions and the FC head in operand order; squeeze-excite: W1
    const float* bias;         // squeeze-excite: b1
    const float* scale;        // squeeze-excite: W2
    const float* pre_scale;    // squeeze-excite: b2
    const float* pre_shift;
    const void* ahead[2];      // first step of a phase: weights of the next phase, and their bytes
    int ahead_bytes[2];
    int kind, phase_steps;     // first step of a phase: the steps of that phase, and << 8 those of the next one (0: none)
    int xs, xc0, ys, yc0, rs, rc0;
    int H, W, Ho, Wo, cin, cout;
    int window, stride;        // kh | kw << 8 | pt << 16 | pl << 24; sh | sw << 8 | act << 16 | s2d << 24
    int sub;                   // convolution: > 1 groups of `cout` output and `cin` input channels each; squeeze-excite: strips of pixels
    int r, rows, scratch_stride, hidden_at;   // squeeze-excite: hidden units, rows of sums, floats per image, place of the hidden values
    int px, wsize, res_present, padded;   // convolution: output pixels of an image, bytes of the weights; has it a residual, and taps outside the image?
    int K, ctiles[2];          // convolution: taps x input channels; tiles of 32 and of 64 output channels (of all groups)
    float inv_ctiles[2], inv_wo, inv_ho, inv_cin, inv_kw;
    int choice[CHAIN_SIZES];   // << 16 units for that many images; convolution: side of a wavefront's tile in 32s, << 8 log2 of the wavefronts that share its K
};
static_assert(sizeof(ChainStep) == 256, "a dword for each lane");
constexpr int CH_POOL = 2;                   // outputs of a pooling layer that a lane works on at a time
constexpr int CHAIN_PHASE_STEPS = 7;         // of a phase at most

// Where in a 1 KB fragment of block i of channel tile cs (`side` blocks of 32 output channels each) a lane's weights lie.  The last tile has a block
// less than others when the number of blocks is odd: what it asks for there lies past the end of every buffer and comes as zeros.  (The
// range check is about this offset alone, not about the place of the block, which is a scalar.)
__host__ __device__ inline unsigned chain_weight_lane(int cs, int side, int i, int blocks, int lane) {
    return cs * side + i < blocks ? (unsigned)lane * 16u : 0x80000000u;
}

// Words that the groups of one launch meet at; zeros before a launch, and again after it.
struct ChainSync {
    // (what workgroups of one XCD count at their L2 has a line of its own, is never set back, and is used by nobody else)
    struct { unsigned count; unsigned pad0[31]; unsigned size, program, arrived_before; unsigned pad1[29]; unsigned arrived; unsigned pad2[31]; } group[CHAIN_GROUPS];
    unsigned queue; unsigned pad3[31];
    unsigned gone; unsigned pad4[31];
};

struct ChainArgs {
    const ChainStep* steps[ENS_MAX_MEMBERS];
    char* arena[ENS_MAX_MEMBERS];
    unsigned image_bytes[ENS_MAX_MEMBERS];
    float* logits[ENS_MAX_MEMBERS];          // rows of the whole request
    short phases[ENS_MAX_MEMBERS];
    ChainProgram programs[CHAIN_MAX_PROGRAMS];
    ChainSync* sync;
    uint32_t* failed;                        // pinned host word: set when a group gave up waiting
    const float* src;                        // request images
    int n_programs, base_h, base_w, classes;
};
static_assert(sizeof(ChainArgs) <= 4000, "kernel arguments");

hipError_t launch_chain(const ChainArgs& a, hipStream_t s);
hipError_t launch_chain_pack(const void* w, void* out, int groups, int rows, int K, hipStream_t s);

// `launches`: the member's operations one by one, their tensors at distinct addresses base + at[tensor].  False: not for chains.
// Weights of convolutions are named as the launches have them, and listed in out->packs where they are not in operand order yet: w of those steps
// is to become the place of the packed copy.
bool build_chain(const Member& m, const std::vector<Launch>& launches, char* base, const std::vector<size_t>& at, size_t arena_bytes, int batch,
                 Chain* out);
int chain_size(int images);

}  // namespace ens

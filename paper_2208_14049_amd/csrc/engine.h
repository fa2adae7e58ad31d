// The inference-system core on one GPU: members resident in HBM, workers (one per non-zero
// cell of the allocation matrix) with their own stream and activation arena, the segment /
// batch partition of a request and the fused combination kernel.
#pragma once
#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "../../include/ens.h"
#include "kernels.h"

namespace ens {

struct ChainStep;
struct ChainSync;
// Images [first, first + images) of one member, as a chain (chain.h); size: for what number of images its tiles were chosen.
struct alignas(8) ChainProgram { short member, first, images, size; };

struct TensorInfo {
    int h, w, c;
    int cs;          // stored channels (bf16 tensors are padded to a multiple of 8)
    bool f32;        // stored as fp32
    int def, last;   // first writing / last reading operation (-1: written by the input staging)
    bool external;   // the logits tensor lives in the member's logits buffer, not in an arena
    size_t elems_per_image() const { return (size_t)h * w * cs; }
    size_t bytes(int batch) const { return (size_t)batch * elems_per_image() * (f32 ? 4 : 2); }
};

struct OpPlan {
    ens_op op;
    // byte offsets into the member's device parameter block (SIZE_MAX: absent)
    size_t w, b, scale, pre_scale, pre_shift, w2, b2;
    size_t w_packed; // the convolution's weights once more in matrix-core operand order (members of a fused chain)
    int cin_s;       // stored input channels of the convolution's K axis
    int scratch;     // index of the scratch pseudo-tensor (squeeze-excite), -1 otherwise
    int alg_k;       // multiply-adds per output element as the network defines the layer (0: kh*kw*cin of op)
    // A grouped convolution runs as `sub` dense convolutions on channel slices, sub_cout output channels
    // each over cin_s input channels, weights [sub][sub_cout][kh*kw][cin_s] (zeros where a pair of
    // channels belongs to different groups).  Ordinary convolution: sub = 1, sub_cout = cout.
    int sub, sub_cout;
    // This convolution and the next one read the same input slice and write outputs of the same height
    // and width (a residual block's 3x3 / stride-2 branch and its 1x1 shortcut, the 1x1 heads of an
    // inception module's branches): one launch can run both as further argument blocks when both go
    // to the generic kernel.  The second output counts as written here.
    bool fuse_next;
    // This 1x1 convolution, the 3x3 after it and the 1x1 after that form a residual bottleneck whose two
    // middle tensors nobody else touches: one kernel can run the three without writing them.
    bool fuse_chain;
    // This pre-activated 1x1 convolution (to 128 channels) and the 3x3 after it (to 32 channels) are a layer
    // of a dense block whose middle tensor nobody else touches: one kernel can run both.
    bool fuse_dense;
    // This convolution is the input stem (rewritten to stride 1 over the space-to-depth image, ReLU) and the
    // next operation is a 3x3 / stride-2 / padding-1 max-pool that alone reads its output: one kernel can
    // run both without writing the stem's output.
    bool fuse_pool;
    // This squeeze-excite block is followed by a 1x1 convolution that alone reads its output: the block can
    // stop at the gates and the convolution multiply its input by them, so that the rescaled tensor is
    // never written.
    bool fuse_gate;
    // This depthwise convolution is followed by a squeeze-excite block over its output: its kernel can leave
    // the channel sums the block starts from (one row per workgroup, in the block's scratch, which then lives
    // from this operation on and holds se_cap rows), and the block does not read the tensor for them.
    bool fuse_sums;
    // This 3x3 / stride-1 / padding-1 average pool is followed by a plain 1x1 convolution that alone reads its output
    // and has no more output channels than the pool has channels (the pool branch of an inception module): the
    // two are linear and commute, so the convolution (with its batch-norm, which an average whose weights add up
    // to one also commutes with) can run first, into the pool's output memory, and the pool then averages the
    // narrower tensor and applies the activation.
    bool swap_pool;
    // This pre-activated 1x1 convolution without an activation of its own is followed by a 2x2 / stride-2 average
    // pool that alone reads its output (the transition between two dense blocks): pre-activation and pool can run
    // first, into the convolution's output memory, and the convolution on a quarter of the pixels.
    bool swap_conv;
    int se_cap;      // squeeze-excite: rows of partial sums its scratch holds per image
};

struct Member {
    bool bf16 = false;
    int in_h = 0, in_w = 0, classes = 0, out_tensor = -1;
    std::vector<TensorInfo> tensors;     // description tensors, then scratch pseudo-tensors
    std::vector<OpPlan> ops;
    std::vector<uint8_t> host_params;    // folded, converted, laid out for the device
    size_t zeros_off = 0;                // 256 zero bytes inside the parameter block (padding source)
    // The stride-2 convolution that reads the input image runs as a stride-1 convolution over the
    // image stored space-to-depth (tensor 0 is then ceil(h/2) x ceil(w/2) x 12, stored 16 wide).
    bool stem_s2d = false;
    char* dev_params = nullptr;
    size_t weight_bytes() const { return host_params.size(); }
};

// Scratch the convolution kernel uses when it splits a layer's K range over several workgroups:
// one fp32 slice of partial sums per split.
constexpr size_t SPLIT_WS_FLOATS = 4u << 20;

struct ArenaLayout {
    std::vector<size_t> offset;          // per tensor (unused for external ones)
    size_t scratch_offset = SIZE_MAX;    // split-K scratch (bf16 members)
    size_t bytes = 0;
};

// Builds the device-side form of a member from its description.  Host only.
int build_member(const ens_member_spec& spec, const float* params, Member* out);
// Places the member's tensors for `batch` images by liveness; host only.
// keep_all gives every tensor its own region (debug read-back of intermediate tensors).
ArenaLayout plan_arena(const Member& m, int batch, bool keep_all = false);

enum LaunchKind { L_CONV, L_DWCONV, L_POOL, L_GAP, L_FC, L_SE, L_BNECK, L_DENSE, L_STEMPOOL, L_SKIP };   // L_SKIP: ran with an earlier launch

// One operation of a gang: host copy of the first member's arguments (validation, grid sizing)
// and the device array holding the arguments of every member of the gang.
struct Launch {
    int kind = 0;
    bool is_max = false;
    int klass = 0;                 // profile class
    double flop = 0, bytes = 0;    // algorithmic work of one member's full-batch launch
    ConvArgs conv;
    ConvArgs conv2, conv3;         // L_BNECK: the second and third convolution of the chain; L_DENSE: conv2 is the 3x3;
                                   // L_STEMPOOL: conv2 describes the pooled output
    PoolArgs pool;
    GapArgs gap;
    FcArgs fc;
    SeArgs se;
    const void* d_argv = nullptr;  // device: G * sub argument blocks of this operation's kind
    int sub = 1;                   // argument blocks per member (sub-convolutions of a grouped convolution)
};

struct Worker {
    int member = 0, batch = 0, slot = 0;
    int rank = 0, of = 1;          // this is worker `rank` of the member's `of` workers
    int gang = -1;
    bool copy = false;             // the arena of a gang's copy (see Gang)
    char* arena = nullptr;
    size_t arena_bytes = 0;
    ArenaLayout layout;
    int last_nb = 0;               // images of its last batch
    bool input_only = false;       // of which its arena holds the input and nothing else (ens_debug_tensor runs the layers)
    std::vector<ChainProgram> last_programs;   // not empty: it ran as these (chain.h)
    uint64_t last_request = 0;     // and which one that was: the number of the request, its first image
    int64_t last_first = 0;
};

// The launches of a gang for batches of up to `most` images.
struct GangPlan {
    int most = 0;
    std::vector<Launch> launches;
};

// Workers that run the same network shape at the same batch size on the same segments (the
// replicas of a homogeneous ensemble in one row of the allocation matrix) advance in lockstep:
// one stream, and one kernel launch per operation whose grid spans all of them.
//
// Where there are few of them a gang has copies, gangs of their own over the same members with an arena more each, and its
// batches go to the copies in turn: the batches of one gang ran one after the other on one lane, and its kernels leave compute
// units idle at the end of every launch and wait for memory at its beginning.
struct Gang {
    std::vector<int> workers;      // indices into ens_handle::workers; [0] leads (its input tensor is shared)
    int rank = 0, of = 1;
    int lane = 0;                  // lane of the request in flight
    bool copy = false;
    std::vector<int> copies;       // of the gang they were made from: itself and its copies, indices into ens_handle::gangs
    bool stale = false;            // its argument blocks name request buffers that have moved
    std::vector<GangPlan> plans;   // by the batch sizes they are for, ascending; the last one ends at the workers' batch size
    const GangPlan& plan_for(int images) const {
        for (const GangPlan& p : plans)
            if (images <= p.most) return p;
        return plans.back();
    }
    StageArgs stage;
    char* d_args = nullptr;        // device block holding every argument array of the gang
    size_t d_args_bytes = 0;
};

// The streams that every handle of a process issues its kernels on, one set per GPU.  The runtime spreads ordinary
// streams over four hardware queues in its own order, and streams that meet in a queue run one after the other: two of
// an allocation's streams shared a queue while others stood empty (four streams in a row: two queues).  A stream made with
// a compute-unit mask has a queue of its own; the mask names every unit.  Four of them: the GPU drains four queues
// at once (eight take 1.8 times as long as four for the same work per queue, and many queues of short kernels are slower
// than four), and gangs are dealt to them by estimated time.  Streams of this kind order themselves with the null
// stream, so that a request waits for work that another thread has in flight there.
constexpr int LANES = 4;
// Handles share them, each beginning with another one: a request waits for the lanes that it uses itself, and queues behind another
// handle's work only where the two meet on a lane.
hipError_t acquire_lanes(hipStream_t* lanes);    // LANES streams; every successful call is paired with one of
void release_lanes(const hipStream_t* lanes);    // these; the streams go with the last handle

constexpr int CHAIN_SIZES = 6;               // numbers of images that a chain's tiles are chosen for: up to 1, 2, 4, 8, 16, 32 and more
// The chain of one member, worked out when an allocation is installed.
struct Chain {
    std::vector<ChainStep> steps;
    int phases = 0, cap = 0;                 // images that the worker's arena holds in the chain's layout
    struct Pack { int step, groups, rows, K; size_t at, bytes; };   // weights to be put into operand order, and where among all of them
    std::vector<Pack> packs;
    size_t pack_bytes = 0;
    std::vector<size_t> place;               // of every tensor, for one image
    size_t image_bytes = 0;
    double seconds[CHAIN_SIZES] = {};        // of a program of 1, 2, 4 ... images: its steps added up, by which requests are cut into programs;
    double span[CHAIN_SIZES] = {};           // the estimate proper, with the steps of a phase side by side
};
// A small fp32 member that runs in a compute unit's LDS (resident.h), worked out when an allocation is installed.
struct Resident {
    std::vector<float> fixed;                // what LDS begins with
    int lds_floats = 0;
    int in = 0, in_p = 0, in_r = 0;          // the input tensor in LDS: pixel (0, 0), floats a pixel and a row
    int n_ops = 0;
    double seconds = 0;                      // estimate of an image
};

// A request cut into programs, and its estimate.
struct ChainPlan {
    bool known = false;
    std::vector<ChainProgram> programs;      // the longest first
    double seconds = 1e30;
};

// A request of a size that came before, recorded: per lane every launch of it.
struct RequestGraph {
    int64_t n = 0;
    uint64_t used = 0;             // for giving up the one used longest ago
    int lanes = 0;
    std::vector<int> gangs;        // that it runs: indices into ens_handle::gangs
    std::vector<std::pair<int64_t, int>> last_batch;   // of each of them: first image, images
    hipGraphExec_t exec[LANES] = {nullptr, nullptr, nullptr, nullptr};
};

// A request size that has come and is not recorded (yet).
struct SeenSize {
    int64_t n = 0;
    uint64_t when = 0;             // number of the request that last had it
    bool failed = false;           // its recording did: not tried again
};

struct ProfClass {
    std::string name;
    double ms = 0, flop = 0, bytes = 0;
    int64_t launches = 0;
};

struct ProfRec { int klass; hipEvent_t start, stop; double flop, bytes; };

}  // namespace ens

struct ens_handle {
    std::vector<ens::Member> members;
    std::vector<ens::Worker> workers;
    std::vector<ens::Gang> gangs;                // the copies last
    int own_gangs = 0;                           // without the copies
    bool gangs_enabled = true;                   // false: every worker is a gang of its own
    bool args_stale = false;                     // other logits buffers are in use: argument arrays need rebuilding
    ens_alloc alloc;
    bool have_alloc = false;
    int segment_size = 128;
    int base_h = 0, base_w = 0, classes = 0;
    bool images_on_device = false, probs_on_device = false;
    uint64_t budget = 0;                         // 0: whatever the device has
    int64_t reserve = 0;                         // of the budget for request buffers (ens_plan)
    hipStream_t main_stream = nullptr;           // copies, and the recording of graphs
    hipStream_t lanes[ens::LANES] = {nullptr, nullptr, nullptr, nullptr};
    bool have_lanes = false;
    int lanes_used = 0;                          // by the last request: the first ones of `lanes`
    std::vector<hipEvent_t> copied;              // per piece of a host request: its images are on the device
    ens::RequestSlot* d_slots = nullptr;         // one per lane
    unsigned* d_arrivals = nullptr;              // see CombineArgs; one more for finish_kernel
    uint32_t* flag = nullptr;                    // pinned: number of the last request that is complete (see wait_lanes), then
                                                 // per lane the number of its last batch that is
    bool flagged = false;                        // the request in flight will write it
    // small requests as chains (chain.h): one per member, or none at all; their steps in device memory, and where in it each begins
    std::vector<ens::Chain> chains;
    ens::ChainStep* d_chain = nullptr;           // and behind them weights in operand order
    int64_t chain_bytes = 0;
    std::vector<size_t> chain_at;
    std::vector<ens::ChainPlan> chain_plans;     // by the number of images
    ens::ChainSync* d_chain_sync = nullptr;
    bool chains_off = false;                     // one of them gave up waiting: no more of them with this allocation
    // fp32 members that fit LDS (resident.h): one per member, or none at all; what LDS begins with in device memory, and where each begins
    std::vector<ens::Resident> residents;
    float* d_resident = nullptr;
    unsigned* resident_queue = nullptr;              // in it
    int64_t resident_bytes = 0;
    std::vector<size_t> resident_at;
    std::vector<ens::RequestGraph> graphs;
    std::vector<ens::SeenSize> sizes_seen;
    uint64_t requests = 0, last_recorded = 0;    // requests so far, and the one that was recorded last
    ens_stats stats = {};
    // pinned host memory for small requests: kernels read the images and write the probabilities there themselves
    float* pin_in = nullptr;    size_t pin_in_cap = 0;
    float* pin_out = nullptr;   size_t pin_out_cap = 0;
    // request buffers, grown on demand
    float* d_images = nullptr;  size_t d_images_cap = 0;
    float* d_probs = nullptr;   size_t d_probs_cap = 0;
    // Per-member logits of the request in flight.  d_logits are the buffers in use:
    // either the library's own allocations (d_logits_heap; grown on demand) or, for the
    // allocation-free entry point, slices of the fixed device array.
    std::vector<float*> d_logits; size_t d_logits_rows = 0;      // in use, and the rows they hold
    std::vector<float*> d_logits_heap; size_t d_logits_heap_rows = 0;
    bool logits_static = false;
    int combine_rule = 0;                        // ENS_COMBINE_*
    float* d_weights = nullptr;                  // member weights of the weighted rule (device)
    float* d_calib = nullptr;   size_t d_calib_images = 0;
    int stage_klass = 0;
    int64_t last_n = 0;
    double last_ms = 0;
    // profiling
    bool profiling = false;
    bool keep_tensors = false;                   // debug: no reuse of arena regions
    bool keeps = false;                          // the installed workers were laid out that way
    bool fake_predictor = false;                 // overhead experiment: forward passes replaced by zeros
    bool no_rows = false;                        // test: rows_off() (kernels.h) of its requests
    bool planning = false;                       // the optimizer's benchmarks: launch by launch, and nothing is prepared for other requests
    bool one_stream = false;                     // measurement: every worker issues on the first lane, one kernel at a time
    std::vector<ens::ProfClass> prof;
    std::vector<ens::ProfRec> prof_recs;
    std::vector<hipEvent_t> event_pool;
};

// C boundary and step executor: carves the caller's arena, runs the layer
// list forward and backward for each worker's shard, then the fused
// aggregation + update.  See include/edl.h for the contract of every call.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <vector>

#include "bn_pointwise.h"
#include "graph.h"
#include "kernels.h"
#include "narrow.h"
#include "profiler.h"
#include "thin.h"
#include "tune.h"

using namespace edl;

#define HIP_TRY(expr)                                                                      \
    do {                                                                                   \
        hipError_t e_ = (expr);                                                            \
        if (e_ != hipSuccess) {                                                            \
            set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
            return EDL_EHIP;                                                               \
        }                                                                                  \
    } while (0)

// Scratch for edl_step_static_scratch (callers that cannot bring or allocate a scratch piece): one fixed buffer
// per GPU, held from the time the library's code is loaded on that GPU until the process ends.  In host code
// this name is only a handle for hipGetSymbolAddress; the device address is taken once per device in edl_init
// and kept in g_static_scratch, and that pointer is what kernels and copies are given.
static __device__ __align__(256) unsigned char scratch[EDL_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
void* g_static_scratch[kMaxDevices] = {};     // per device: address of that device's copy of `scratch`

// The library's own pair of side streams is one per job stream, shared by the jobs on that stream and destroyed with
// the last of them.  A process has few hardware queues (four by default) and streams are dealt to them in turn: with
// a pair of its own, the third job's side streams shared a queue with the jobs' main stream and with each other, and
// its weight gradients ran in line with the pass they should run beside (ResNet-50, shard of 32: 4.40 ms per step for
// the first two jobs, 5.75 for the third; three jobs in turn 4.92 -> 4.40 with one pair).  Jobs on one stream follow
// one another there anyway, so sharing orders nothing that was free: a job whose stream is held up, or under capture
// into a graph, holds up or captures the side work of the jobs on that stream only.
struct SharedStreams {
    int device;
    hipStream_t main, side, upd;
    int users;
};
std::vector<SharedStreams> g_side_streams;      // as many as there are job streams in use
std::mutex g_side_streams_mutex;

constexpr int64_t kAlign = 256;
constexpr int kIdxSlots = 4;
constexpr size_t kStageBytes = 256;  // pinned staging of what is read back: the workers' losses, an image's header
constexpr int kReadyEvents = 64;   // ring of "dy is final" events for the second stream
constexpr int kChunkEvents = 64;   // ring of "these weight gradients are final" events for the update stream
constexpr int kBranchEvents = 16;  // ring of event pairs around a shortcut branch on the second side stream

int64_t align_up(int64_t v, int64_t a = kAlign) { return (v + a - 1) / a * a; }

// header of the state image (little endian, packed by construction)
struct SnapshotHeader {
    uint32_t magic, version, model, dtype;
    uint64_t seed;
    int64_t N, B, step, epoch, step_in_epoch;
    float lr, momentum, wd;
    uint32_t optimizer;
    int64_t P, R;
    float beta2, eps;      // Adam only, else 0
};
static_assert(sizeof(SnapshotHeader) == 104, "snapshot header layout");

// The kernels' scratch (partial results that live inside one pass), in one contiguous piece [scratch_lo, scratch_hi).
struct Scratch {
    int scratch_samples = 0, scratch_shards = 0;     // most samples / shards it takes together
    int64_t row_loss = 0, partial = 0, partial_held = 0, coef = 0, wgrad_scratch = 0;
    int64_t partial_side = 0, coef_side = 0, splitk_side = 0;   // the branch stream's own scratch
    int64_t partial_floats = 0;          // of each of the three partial-sum pieces
    int64_t wgrad_scratch_bytes = 0;
    int64_t wgrad_scratch2 = 0;          // for the few weight gradients that run on the main stream beside the second one
    // partial sums of forward / dgrad reductions that are cut; apart from the weight-gradient
    // scratch because weight gradients may run on the second stream meanwhile
    int64_t splitk_scratch = 0, splitk_scratch_bytes = 0;
    int64_t dwpad = 0;                   // float32 gradient of weights on padded images before it is compacted
    int64_t scratch_lo = 0, scratch_hi = 0;
};

struct Layout : Scratch {                // the Scratch is the arena's
    int64_t params = 0, momentum = 0, second = -1, running = 0, shadow = 0, grads = 0, grad_stride = 0;
    int64_t idx = 0, labels = 0, losses = 0;
    int pass_samples = 0, pass_shards = 0;   // most samples / shards that one pass runs together
    int64_t ttable = 0;                  // TransposeEntry[] for the one-launch weight transpose
    InputFold in;                        // how the input images are stored (see input_fold)
    std::vector<int64_t> wpad;           // per op: zero-padded weight copy of a convolution on padded images (-1 if none)
    std::vector<int64_t> act, grad;      // per tensor (storage owners only; -1 otherwise)
    std::vector<int64_t> sign;           // per tensor: (activation > 0) as bits, for outputs of a batch norm with ReLU that a stride-1 convolution reads (bf16)
    std::vector<int64_t> wT;             // per op: transposed weight copy (-1 if not needed)
    std::vector<int64_t> bn_save;        // per op
    std::vector<int64_t> pool_arg;       // per op
    int64_t total = 0;
};

int validate(const edl_config& c) {
    if (c.dtype != EDL_DTYPE_F32 && c.dtype != EDL_DTYPE_BF16) { set_error("unknown dtype %d", c.dtype); return EDL_EINVAL; }
    if (c.N <= 0 || c.B <= 0 || c.p_max <= 0 || c.max_shard <= 0) { set_error("N, B, p_max, max_shard must be positive"); return EDL_EINVAL; }
    if (c.p_max > kMaxP) { set_error("p_max %d exceeds %d", c.p_max, kMaxP); return EDL_EINVAL; }
    if (c.N % c.B) { set_error("N=%lld is not a multiple of B=%lld", (long long)c.N, (long long)c.B); return EDL_EINDIVISIBLE; }
    if (c.max_shard > c.B) { set_error("max_shard exceeds B"); return EDL_EINVAL; }
    if (c.optimizer != EDL_OPT_MOMENTUM && c.optimizer != EDL_OPT_ADAM) { set_error("unknown optimizer %d", c.optimizer); return EDL_EINVAL; }
    if (c.optimizer == EDL_OPT_ADAM &&
        !(c.momentum >= 0.f && c.momentum < 1.f && c.beta2 >= 0.f && c.beta2 < 1.f && c.eps >= 0.f)) {
        set_error("Adam needs 0 <= beta1 (momentum), beta2 < 1 and eps >= 0");
        return EDL_EINVAL;
    }
    return EDL_OK;
}

int storage_of(const Graph& g, int t) { return g.tensors[(size_t)t].alias_of >= 0 ? g.tensors[(size_t)t].alias_of : t; }

ConvGeom geom_of(const Graph& g, const Op& op, int n) {
    const Tensor& tx = g.tensors[(size_t)op.x];
    const Tensor& ty = g.tensors[(size_t)op.y];
    ConvGeom q;
    q.N = n; q.H = tx.H; q.W = tx.W; q.C = tx.C;
    q.K = op.K; q.R = op.R; q.S = op.S; q.stride = op.stride; q.pad = op.pad; q.Ho = ty.H; q.Wo = ty.W;
    return q;
}

// Images whose channel count is not a multiple of the 16-byte vector (RGB) are
// stored with every pixel padded to one vector, so that the first convolution
// runs on the vector path.  Not when a flattened view of the images exists.
// In bf16, under a first convolution of stride 2 or 4, blocks of stride x stride pixels become one pixel of 3 * stride^2
// channels instead (padded to whole vectors), and the convolution one of stride 1 whose taps are blocks: the same products
// and far fewer of the padding's zeros (elements per output: ResNet's 7x7/2 392 -> 256, AlexNet's 11x11/4 968 -> 432), on
// images of half to three eighths of the bytes.  ResNet-50, 8 shards of 32: stem 333 -> 226 us forward, 318 -> 190 us weight
// gradient; AlexNet, 2 shards of 64: 92 -> 42 us and 90 -> 46 us.  In float32 the pixel's vector holds four channels, so a 7x7 has
// 196 elements unfolded and 192 folded: nothing to gain.
InputFold input_fold(const edl_config& c, const Graph& g) {
    const int vec = c.dtype == EDL_DTYPE_BF16 ? 8 : 4;
    InputFold in;
    in.C = g.tensors[0].C;
    in.H = g.tensors[0].H;
    in.W = g.tensors[0].W;
    if (in.C % vec == 0 || in.C > vec) return in;
    for (const Tensor& t : g.tensors)
        if (t.alias_of == 0) return in;
    const int C = in.C;
    in.C = vec;
    const Op* first = nullptr;
    for (const Op& op : g.ops) {
        if (op.x != 0 && op.res != 0) continue;
        if (first != nullptr || op.kind != OP_CONV) return in;
        first = &op;
    }
    if (first == nullptr || c.dtype != EDL_DTYPE_BF16 || C != 3 || (first->stride != 2 && first->stride != 4)) return in;
    const int f = first->stride, wide = (f * f * C + vec - 1) / vec * vec;
    const int taps = ((first->R + f - 1) / f) * ((first->S + f - 1) / f);
    if (taps * wide >= first->R * first->S * vec) return in;
    // output row ho reads image rows ho * f - pad + r; with `lead` zero rows in front, block row ho - pad / f + r / f
    in.f = f;
    in.lead = first->pad % f;
    in.C = wide;
    in.H = (in.H + in.lead + f - 1) / f;
    in.W = (in.W + in.lead + f - 1) / f;
    return in;
}

// The convolution as it is launched: on the stored images, if it reads them.
ConvGeom geom_stored(const Graph& g, const Op& op, int n, const InputFold& in) {
    ConvGeom q = geom_of(g, op, n);
    if (op.x != 0) return q;
    q.H = in.H; q.W = in.W; q.C = in.C;
    q.R = (q.R + in.f - 1) / in.f;
    q.S = (q.S + in.f - 1) / in.f;
    q.stride /= in.f;
    q.pad /= in.f;
    return q;
}
bool stored_apart(const Graph& g, const InputFold& in) { return in.C != g.tensors[0].C; }
// elements of a filter of the first convolution as it is launched
int64_t stored_row(const Op& op, const InputFold& in) {
    return (int64_t)((op.R + in.f - 1) / in.f) * ((op.S + in.f - 1) / in.f) * in.C;
}

// The kernels' scratch from offset `o` on for running up to `samples` samples in up to `shards` shards together, as
// parts of passes of up to L.pass_samples and L.pass_shards (whose tiles and cuts the parts take).  Returns its end.
int64_t plan_scratch(const edl_config& c, const Graph& g, const Layout& L, int samples, int shards, int64_t o, Scratch& X) {
    auto take = [&](int64_t bytes) { const int64_t at = o; o += align_up(bytes); return at; };
    X.scratch_samples = samples;
    X.scratch_shards = shards;
    int cmax = 1;
    int64_t dwpad_bytes = 16;
    X.wgrad_scratch_bytes = X.splitk_scratch_bytes = X.partial_floats = 0;
    std::vector<ConvGeom> seen;          // layers repeat few shapes (a job of ResNet-20 plans its arena in 164 us, before 428)
    for (const Op& op : g.ops) {
        if (op.kind == OP_CONV) {
            const ConvGeom shape = geom_of(g, op, op.x == 0 ? 0 : 1);      // (0: reads the padded images)
            if (std::any_of(seen.begin(), seen.end(), [&](const ConvGeom& o) { return memcmp(&o, &shape, sizeof(shape)) == 0; })) continue;
            seen.push_back(shape);
            cmax = std::max(cmax, op.K);
            const Tensor& ty = g.tensors[(size_t)op.y];
            if (op.x == 0 && stored_apart(g, L.in)) dwpad_bytes = std::max<int64_t>(dwpad_bytes, op.K * stored_row(op, L.in) * 4 * shards);
            // a weight gradient is cut for the largest of the pass's shards
            for (int q = 1; q <= shards && q <= samples; ++q)
                X.wgrad_scratch_bytes = std::max<int64_t>(
                    X.wgrad_scratch_bytes, (int64_t)conv_wgrad_scratch_bytes(c.dtype, geom_stored(g, op, c.max_shard, L.in), q));
            X.splitk_scratch_bytes = std::max<int64_t>(X.splitk_scratch_bytes,
                                                       (int64_t)conv_splitk_scratch_bytes(c.dtype, geom_of(g, op, L.pass_samples), samples));
            X.partial_floats = std::max<int64_t>(X.partial_floats, (int64_t)conv_sums_floats(geom_stored(g, op, samples, L.in), shards));
            X.partial_floats = std::max<int64_t>(X.partial_floats,
                                                 (int64_t)norm_sums_floats(c.dtype, (int64_t)L.pass_samples * ty.H * ty.W, op.K, L.pass_shards));
        } else if (op.kind == OP_BN) {
            cmax = std::max(cmax, op.K);
            const Tensor& tx = g.tensors[(size_t)op.x];
            X.partial_floats = std::max<int64_t>(X.partial_floats,
                                                 (int64_t)norm_sums_floats(c.dtype, (int64_t)L.pass_samples * tx.H * tx.W, op.K, L.pass_shards));
        }
    }
    // (a column reduction's blocks are planned for the whole pass and may be as many for a part of it;
    // room for kRedRowBlocks blocks of the widest layer in any case: what a job needs of the static buffer does not
    // depend on how its launches happen to be cut)
    X.partial_floats = std::max<int64_t>(X.partial_floats, 2 * (int64_t)kRedRowBlocks * cmax);
    X.scratch_lo = o;
    X.row_loss = take(4 * (int64_t)samples);
    X.partial = take(4 * X.partial_floats);
    // a second one for sums that wait while another batch norm runs (a block's last convolution, whose
    // batch norm comes after the projection shortcut's)
    X.partial_held = take(4 * X.partial_floats);
    X.coef = take(4 * 2 * (int64_t)cmax * shards);
    // the same pair for the projection shortcut's batch norm while it runs on the branch stream beside the main one
    X.partial_side = take(4 * X.partial_floats);
    X.coef_side = take(4 * 2 * (int64_t)cmax * shards);
    X.wgrad_scratch = take(std::max<int64_t>(X.wgrad_scratch_bytes, 16));
    X.wgrad_scratch2 = take(std::max<int64_t>(X.wgrad_scratch_bytes, 16));
    X.splitk_scratch = take(std::max<int64_t>(X.splitk_scratch_bytes, 16));
    // the branch stream cuts reductions exactly as the main stream would (same results, bit for bit, whichever
    // stream a layer runs on), in a buffer of its own
    X.splitk_side = take(std::max<int64_t>(X.splitk_scratch_bytes, 16));
    X.dwpad = take(dwpad_bytes);
    X.scratch_hi = o;
    return o;
}

// How many samples and shards one pass runs together.  All of the mini-batch if it fits: a layer of p shards is then
// one launch instead of p, with p times the workgroups (ResNet-50 bf16, aggregate batch 256 as 8 shards of 32:
// 34.5 -> 23.4 ms per step; ResNet-20 float32, 8 shards of 16: 8.3 -> 1.8 ms; MLP, 4 shards of 16: 0.41 -> 0.15 ms).
// Limits, none of which cuts a single shard:
// 32 GB of activations and gradients (a pass of some 250 images of 224x224 gains nothing more from more of them),
// 2 GiB per tensor (the vector kernels' 32-bit offsets), and what every convolution's vector kernel takes (VGG-16 on
// 320x320 images: 95 samples).
void plan_pass(const edl_config& c, const Graph& g, Layout& L) {
    const int64_t esz = c.dtype == EDL_DTYPE_BF16 ? 2 : 4;
    int64_t per_sample = 1, widest = 1;
    for (size_t t = 0; t < g.tensors.size(); ++t) {
        if (g.tensors[t].alias_of >= 0) continue;
        const int64_t bytes = (t == 0 ? (int64_t)L.in.H * L.in.W * L.in.C : g.tensors[t].elems()) * (g.tensors[t].fp32 ? 4 : esz);
        per_sample += 2 * bytes;
        widest = std::max(widest, bytes);
    }
    int64_t samples = std::min<int64_t>(c.B, std::min<int64_t>(32000000000ll / per_sample, 2147483647ll / widest));
    samples = std::min<int64_t>(samples, 65535);
    for (const Op& op : g.ops)
        if (op.kind == OP_CONV)
            samples = std::min<int64_t>(samples, conv_vector_samples(geom_stored(g, op, 1, L.in), storage_of(g, op.x) != 0));
    samples = std::max<int64_t>(samples, c.max_shard);
    L.pass_shards = c.p_max;
    L.pass_samples = c.p_max == 1 ? c.max_shard : (int)samples;
}

// the arena of a job whose passes run up to L.pass_samples samples in up to L.pass_shards shards
void plan_arena(const edl_config& c, const Graph& g, Layout& L) {
    const int64_t esz = c.dtype == EDL_DTYPE_BF16 ? 2 : 4;
    int64_t o = 0;
    auto take = [&](int64_t bytes) { const int64_t at = o; o += align_up(bytes); return at; };
    // The arrays the update kernel walks side by side (w, v, the bf16 copy, the p gradient buffers) start on 4 KB
    // boundaries, alternately even and odd ones (offset bit 12): a workgroup touches the same offset of every
    // array at the same time, and arrays that all start 8 KB-aligned meet in the same half of the memory system
    // (measured: 5.6 -> 6.2 TB/s for the update; the arena itself should start on an 8 KB boundary for this to
    // hold, as torch's large allocations do).
    auto take_page = [&](int64_t bytes, int odd) {
        o = (o + 8191) / 8192 * 8192 + (odd ? 4096 : 0);
        const int64_t at = o;
        o += align_up(bytes);
        return at;
    };
    L.params = take_page(4 * g.P, 0);
    L.momentum = take_page(4 * g.P, 1);
    if (c.optimizer == EDL_OPT_ADAM) L.second = take_page(4 * g.P, 0);
    L.shadow = c.dtype == EDL_DTYPE_BF16 ? take_page(2 * g.P, c.optimizer == EDL_OPT_ADAM ? 1 : 0) : -1;
    // consecutive gradient buffers an odd number of 4 KB pages apart, the first one on an odd page
    L.grad_stride = ((4 * g.P + 8191) / 8192 * 8192 + 4096) / 4;
    L.grads = take_page(4 * L.grad_stride * c.p_max, 1);
    L.running = take(4 * std::max<int64_t>(g.R, 1));
    L.idx = take(8 * c.B);
    L.labels = take(4 * (int64_t)L.pass_samples);
    L.losses = take(4 * kMaxP);
    const size_t nt = g.tensors.size();
    L.act.assign(nt, -1);
    L.grad.assign(nt, -1);
    for (size_t t = 0; t < nt; ++t) {
        if (g.tensors[t].alias_of >= 0) continue;
        int64_t elems = g.tensors[t].elems() * L.pass_samples;
        if (t == 0) elems = (int64_t)L.in.H * L.in.W * L.in.C * L.pass_samples;
        L.act[t] = take(elems * (g.tensors[t].fp32 ? 4 : esz));
        if (t != 0) L.grad[t] = take(elems * esz);
    }
    const size_t no = g.ops.size();
    // What an input gradient needs of the activation before it is its sign: a sixteenth of the bytes, once written by
    // the batch norm, for a third of what the epilogue of most of ResNet-50's input gradients reads.
    L.sign.assign(nt, -1);
    if (c.dtype == EDL_DTYPE_BF16)
        for (const Op& op : g.ops)
            if (op.kind == OP_BN && op.relu && op.K % 8 == 0)
                for (const Op& reader : g.ops)
                    if (reader.kind == OP_CONV && reader.stride == 1 && reader.x == op.y && L.sign[(size_t)op.y] < 0)
                        L.sign[(size_t)op.y] = take(g.tensors[(size_t)op.y].elems() / 8 * L.pass_samples);
    L.wT.assign(no, -1);
    L.wpad.assign(no, -1);
    L.bn_save.assign(no, -1);
    L.pool_arg.assign(no, -1);
    for (size_t i = 0; i < no; ++i) {
        const Op& op = g.ops[i];
        if (op.kind == OP_CONV) {
            const Tensor& tx = g.tensors[(size_t)op.x];
            // none where the input gradient reads the weights themselves: fully connected layers, of whole vectors in bf16, small
            // ones (for passes of this many samples) in either type
            const bool in_place = conv_dgrad_reads_weights(c.dtype, geom_of(g, op, L.pass_samples), op.w_off);
            if (storage_of(g, op.x) != 0 && !in_place) L.wT[i] = take((int64_t)op.K * op.R * op.S * tx.C * esz);
            else if (op.x == 0 && stored_apart(g, L.in)) L.wpad[i] = take(op.K * stored_row(op, L.in) * esz);
        } else if (op.kind == OP_BN) {
            L.bn_save[i] = take(4 * 2 * (int64_t)op.K * L.pass_shards);
        } else if (op.kind == OP_MAXPOOL) {
            L.pool_arg[i] = take(g.tensors[(size_t)op.y].elems() * L.pass_samples);
        }
    }
    o = plan_scratch(c, g, L, L.pass_samples, L.pass_shards, o, L);
    L.ttable = take((int64_t)sizeof(TransposeEntry) * 2 * std::max<size_t>(no, 1));   // element-wise entries, then vector ones
    L.total = o;
}

// The arena, for the largest pass of plan_pass or, if that takes more than arena_bytes, the largest that fits: the
// caller bounds a job's memory by what it gives.  The state arrays lie at the same offsets whatever the pass.  Returns
// false if not even one shard of max_shard samples at a time fits (L is the plan for that then).
bool plan_layout(const edl_config& c, const Graph& g, Layout& L, int64_t arena_bytes = INT64_MAX) {
    L.in = input_fold(c, g);
    plan_pass(c, g, L);
    plan_arena(c, g, L);
    if (L.total <= arena_bytes) return true;
    const int shards = L.pass_shards;
    int lo = c.max_shard, hi = L.pass_samples;      // lo fits (once tried), hi does not
    const auto fits = [&](int samples, int p) {
        L.pass_samples = samples;
        L.pass_shards = p;
        plan_arena(c, g, L);
        return L.total <= arena_bytes;
    };
    if (shards == 1 || !fits(lo, shards)) return fits(c.max_shard, 1);
    while (hi - lo > 1) (fits(lo + (hi - lo) / 2, shards) ? lo : hi) = lo + (hi - lo) / 2;
    return fits(lo, shards);
}

// The scratch of edl_step_static_scratch: a pass in as large parts as the static buffer has room for.  Returns false if
// it has none for a shard of max_shard samples (X is the plan for that then).
bool plan_static_scratch(const edl_config& c, const Graph& g, const Layout& L, Scratch& X) {
    int samples = L.pass_samples, shards = L.pass_shards;
    while (plan_scratch(c, g, L, samples, shards, 0, X) > (int64_t)EDL_STATIC_SCRATCH_BYTES) {
        if (shards == 1 && samples == c.max_shard) return false;
        shards = (shards + 1) / 2;
        samples = shards == 1 ? c.max_shard : std::max(samples / 2, c.max_shard);
    }
    return true;
}

}  // namespace

struct edl_handle {
    edl_config cfg;
    uint64_t seed;
    Graph g;
    Layout L;
    char* arena;
    hipStream_t st;
    const float* data_x = nullptr;
    const int32_t* data_y = nullptr;
    edl_progress prog = {0, 0, 0};
    bool weights_dirty = true;
    // cached permutation of the current epoch
    int64_t perm_epoch = -1;
    std::vector<int64_t> perm;
    int t_entries = 0, t_tiles = 0;      // one-launch weight transpose (element-wise entries)
    double t_bytes = 0;
    int tv_entries = 0, tv_tiles = 0;    // ... and the bf16 layers of vector-friendly shape
    double tv_bytes = 0;
    // pinned staging
    int64_t* idx_host[kIdxSlots] = {nullptr, nullptr, nullptr, nullptr};
    hipEvent_t idx_event[kIdxSlots] = {};
    int idx_slot = 0;
    float* loss_host = nullptr;
    std::vector<int> readers;            // per tensor storage: how many layers read it (as input or as residual)
    std::vector<int> first_reader;       // per tensor storage: the first of them in the layer list (the last to run backward)
    // shard sizes of the last edl_gradients (what edl_apply weighs the gradient buffers by)
    std::vector<int64_t> shard_n;
    bool shards_equal = true;
    bool grads_pending = false;          // edl_gradients has run and edl_apply has not consumed its buffers yet
    // second stream for the weight gradients (null: everything on st); own_streams: the library's (shared by the
    // jobs on this stream), not the caller's
    hipStream_t side = nullptr;
    bool own_streams = false;
    hipEvent_t ev_ready[kReadyEvents] = {};
    hipEvent_t ev_side_done = nullptr;
    int ev_slot = 0;
    // The update of the parameters whose gradients are final starts during the last backward pass of a step,
    // on a stream of its own: `early_p` > 0 asks the backward pass for it (the p of the step), `applied_from`
    // is the first parameter already updated (P = none yet).
    hipStream_t upd = nullptr;
    hipEvent_t ev_chunk[kChunkEvents] = {};
    hipEvent_t ev_upd_done = nullptr;
    int chunk_slot = 0;
    int early_p = 0;
    int64_t applied_from = 0;

    // where the kernels' scratch lives during the current call: the arena piece (null), or the static buffer, whose
    // plan L then holds (exchanged with static_plan)
    char* scratch_base = nullptr;
    Scratch static_plan;
    bool static_fits = false;
    int device = -1;
    std::vector<char> written;           // backward pass: which gradient buffers hold something (per tensor)
    std::vector<size_t> wgrad_waiting;   // a backward pass: layers whose weight gradient is yet to be launched
    std::vector<char> bias_waiting;      // ... of them, those whose bias gradient goes with it (2: from the pool after the layer)
    std::vector<char> dw_in_pieces;      // ... those whose weight gradient is there in pieces that are yet to be added up
    bool has_bn = false;
    std::vector<char> op_done;           // a pass: layers already launched out of list order (on the branch stream)
    // backward pass, per tensor: where the gradient "already there" is to be read from if not from the tensor's
    // own gradient buffer (an identity shortcut's part is the masked gradient of the block's output itself)
    std::vector<const void*> grad_alias;
    // The projection shortcut of a residual block (a convolution and its batch norm) depends only on the block's
    // input (forward) / on the gradient the block's last batch norm leaves for it (backward), so it runs on the
    // second side stream beside the main branch: ev_branch_go releases it, ev_branch_done joins it.
    hipEvent_t ev_branch_go[kBranchEvents] = {}, ev_branch_done[kBranchEvents] = {};
    int branch_slot = 0;
    hipEvent_t ev_tr_go = nullptr, ev_tr_done = nullptr;   // around the weight transposes on the weight-gradient stream
    bool transposes_pending = false;

    template <typename T> T* at(int64_t off) const { return reinterpret_cast<T*>(arena + off); }
    // a piece of the kernels' scratch (off is its arena offset)
    template <typename T> T* sc(int64_t off) const {
        return reinterpret_cast<T*>(scratch_base ? scratch_base + (off - L.scratch_lo) : arena + off);
    }
    float* w() const { return at<float>(L.params); }
    float* v() const { return at<float>(L.momentum); }
    float* s2() const { return at<float>(L.second); }                     // Adam only
    bool adam() const { return cfg.optimizer == EDL_OPT_ADAM; }
    int64_t state_floats() const { return (adam() ? 3 : 2) * g.P + g.R; }   // w, optimizer slots, running
    float* running() const { return at<float>(L.running); }
    float* grad_buf(int k) const { return at<float>(L.grads) + (int64_t)k * L.grad_stride; }
    unsigned char* sign(int t) const { return L.sign[(size_t)t] < 0 ? nullptr : at<unsigned char>(L.sign[(size_t)t]); }
    void* act(int t) const { return arena + L.act[(size_t)storage_of(g, t)]; }
    void* grad(int t) const { return arena + L.grad[(size_t)storage_of(g, t)]; }
};

extern "C" {

const char* edl_last_error(void) { return get_error(); }

int32_t edl_query(const edl_config* cfg, edl_sizes* out) {
    if (!cfg || !out) { set_error("null argument"); return EDL_EINVAL; }
    int rc = validate(*cfg);
    if (rc) return rc;
    Graph g;
    rc = build_graph(*cfg, g);
    if (rc) return rc;
    Layout L;
    plan_layout(*cfg, g, L);       // no limit: all of the mini-batch together if it can be
    out->P = g.P;
    out->R = g.R;
    out->params_off = L.params;
    out->momentum_off = L.momentum;
    out->running_off = L.running;
    out->grads_off = L.grads;
    out->grad_stride = L.grad_stride;
    out->arena_bytes = L.total;
    out->snapshot_bytes = EDL_SNAPSHOT_HEADER_BYTES + 4 * ((cfg->optimizer == EDL_OPT_ADAM ? 3 : 2) * g.P + g.R);
    out->flops_per_sample = g.flops_per_sample();
    out->second_off = L.second;
    out->shadow_off = L.shadow;
    out->scratch_bytes = L.scratch_hi - L.scratch_lo;
    return EDL_OK;
}

int32_t edl_arena_bytes(const edl_config* cfg, int64_t pass_samples, int64_t* out_bytes) {
    if (!cfg || !out_bytes) { set_error("null argument"); return EDL_EINVAL; }
    if (pass_samples < 0) { set_error("negative pass_samples"); return EDL_EINVAL; }
    int rc = validate(*cfg);
    if (rc) return rc;
    Graph g;
    rc = build_graph(*cfg, g);
    if (rc) return rc;
    Layout L;
    if (pass_samples == 0) {
        plan_layout(*cfg, g, L, 0);
    } else {
        plan_layout(*cfg, g, L);
        if (pass_samples < L.pass_samples) {
            L.pass_samples = (int)std::max<int64_t>(pass_samples, cfg->max_shard);
            plan_arena(*cfg, g, L);
        }
    }
    *out_bytes = L.total;
    return EDL_OK;
}

int32_t edl_debug_side_streams(const edl_handle* h, void** wgrad_stream, void** update_stream) {
    if (!h || !wgrad_stream || !update_stream) { set_error("null argument"); return EDL_EINVAL; }
    *wgrad_stream = (void*)h->side;
    *update_stream = (void*)h->upd;
    return EDL_OK;
}

// What a job of this configuration runs, and p shards of these sizes as one pass of it.
static int one_pass(const edl_config* cfg, int32_t p, const int64_t* sizes, Graph& g, Layout& L, ShardSet& S) {
    int rc = validate(*cfg);
    if (rc) return rc;
    if (p <= 0 || p > cfg->p_max) { set_error("p=%d outside [1, p_max=%d]", p, cfg->p_max); return EDL_EINVAL; }
    rc = build_graph(*cfg, g);
    if (rc) return rc;
    plan_layout(*cfg, g, L);
    S = {};
    for (int k = 0; k < p; ++k) {
        if (sizes[k] <= 0 || sizes[k] > cfg->max_shard) { set_error("shard %d outside [1, max_shard]", k); return EDL_EINVAL; }
        S.off[k + 1] = S.off[k] + (int)sizes[k];
        S.k[k] = k;
    }
    S.p = p;
    S.plan_itself();
    if (p > L.pass_shards || S.samples() > L.pass_samples) { set_error("these shards do not run in one pass"); return EDL_ERANGE; }
    return EDL_OK;
}

int32_t edl_debug_wgrad_scratch(const edl_config* cfg, int32_t p, const int64_t* sizes, int64_t* out_needed, int64_t* out_there) {
    if (!cfg || !sizes || !out_needed || !out_there) { set_error("null argument"); return EDL_EINVAL; }
    Graph g;
    Layout L;
    ShardSet S;
    const int rc = one_pass(cfg, p, sizes, g, L, S);
    if (rc) return rc;
    *out_needed = 0;
    *out_there = L.wgrad_scratch_bytes;
    for (const Op& op : g.ops)
        if (op.kind == OP_CONV)
            *out_needed = std::max(*out_needed, (int64_t)conv_wgrad_needs(cfg->dtype, geom_stored(g, op, S.samples(), L.in), S));
    return EDL_OK;
}

int32_t edl_debug_narrow_layers(const edl_config* cfg, int32_t p, const int64_t* sizes, int32_t* out_layers) {
    if (!cfg || !sizes || !out_layers) { set_error("null argument"); return EDL_EINVAL; }
    Graph g;
    Layout L;
    ShardSet S;
    const int rc = one_pass(cfg, p, sizes, g, L, S);
    if (rc) return rc;
    *out_layers = 0;
    for (const Op& op : g.ops)
        if (op.kind == OP_CONV) *out_layers += narrow_takes(cfg->dtype, geom_stored(g, op, S.samples(), L.in), S);
    return EDL_OK;
}

int32_t edl_tensor_count(const edl_config* cfg, int32_t* out_count) {
    if (!cfg || !out_count) { set_error("null argument"); return EDL_EINVAL; }
    Graph g;
    const int rc = build_graph(*cfg, g);
    if (rc) return rc;
    *out_count = (int32_t)g.params.size();
    return EDL_OK;
}

int32_t edl_tensor_info(const edl_config* cfg, int32_t i, char* name_buf, size_t name_cap, int64_t* out_offset,
                        int64_t* out_size, int64_t* out_fan_in) {
    if (!cfg) { set_error("null argument"); return EDL_EINVAL; }
    Graph g;
    const int rc = build_graph(*cfg, g);
    if (rc) return rc;
    if (i < 0 || (size_t)i >= g.params.size()) { set_error("tensor index %d out of range", i); return EDL_ERANGE; }
    const ParamTensor& pt = g.params[(size_t)i];
    if (name_buf && name_cap) snprintf(name_buf, name_cap, "%s", pt.name.c_str());
    if (out_offset) *out_offset = pt.off;
    if (out_size) *out_size = pt.size;
    if (out_fan_in) *out_fan_in = pt.fan_in;
    return EDL_OK;
}

int32_t edl_init_params_host(const edl_config* cfg, uint64_t seed, float* out_params) {
    if (!cfg || !out_params) { set_error("null argument"); return EDL_EINVAL; }
    Graph g;
    const int rc = build_graph(*cfg, g);
    if (rc) return rc;
    he_init(g, seed, out_params);
    return EDL_OK;
}

int32_t edl_shard_host(uint64_t seed, int64_t N, int64_t B, int32_t p, int64_t epoch, int64_t step_in_epoch,
                       int64_t* out_idx, int64_t* out_off) {
    if (!out_idx || !out_off) { set_error("null argument"); return EDL_EINVAL; }
    if (N <= 0 || B <= 0 || p <= 0 || epoch < 0) { set_error("N, B, p must be positive and epoch non-negative"); return EDL_EINVAL; }
    if (B % p || N % B) { set_error("B=%lld must divide by p=%d and N=%lld by B", (long long)B, p, (long long)N); return EDL_EINDIVISIBLE; }
    if (step_in_epoch < 0 || step_in_epoch >= N / B) { set_error("step_in_epoch %lld outside the epoch", (long long)step_in_epoch); return EDL_ERANGE; }
    epoch_permutation_slice(seed, epoch, N, step_in_epoch * B, B, out_idx);
    for (int k = 0; k <= p; ++k) out_off[k] = (int64_t)k * (B / p);
    return EDL_OK;
}

static int refresh_weight_copies(edl_handle* h) {
    // the bf16 copy is written by the update kernel; after init / restore /
    // set_params it is made here.  The transposed copies always are.
    const int dt = h->cfg.dtype;
    if (dt == EDL_DTYPE_BF16) launch_cast_bf16(h->w(), h->at<uint16_t>(h->L.shadow), h->g.P, h->st);
    return EDL_OK;
}

// The transposed weight copies (read by the input-gradient passes only) on stream tst; the zero-padded copy of
// the first convolution's weights (read by the forward pass) on the job's stream.
static void transpose_weights(edl_handle* h, hipStream_t tst) {
    launch_weight_transpose_all(h->cfg.dtype, h->w(), h->arena, h->at<TransposeEntry>(h->L.ttable), h->t_entries,
                                h->t_tiles, h->t_bytes, tst);
    if (h->tv_entries > 0)
        launch_weight_transpose_bf16(h->at<uint16_t>(h->L.shadow), h->arena, h->at<TransposeEntry>(h->L.ttable) + h->g.ops.size(),
                                     h->tv_entries, h->tv_tiles, h->tv_bytes, tst);
    for (size_t i = 0; i < h->g.ops.size(); ++i)
        if (h->L.wpad[i] >= 0) {
            const Op& op = h->g.ops[i];
            launch_pad_weights(h->cfg.dtype, h->w() + op.w_off, h->arena + h->L.wpad[i], op.K, op.R, op.S,
                               h->g.tensors[0].C, h->L.in, h->st);
        }
}

static int init_device_state(edl_handle* h);

// Events that order the side streams against the job's stream (created once, whoever owns the streams).  They order work on
// one GPU only, for which the agent-scope release at the end of every kernel is enough: the write-back to system scope that
// recording does otherwise is left out.  Measured on a chain of 8 us kernels with a record after each: 10.9 -> 9.1 us per
// kernel (a backward pass of ResNet-50 records 70 on the chain of its input gradients).  What the host reads is ordered by
// stream synchronisation or by events of the full kind.
constexpr unsigned kOrderOnly = hipEventDisableTiming | hipEventDisableSystemFence;
static int create_side_events(edl_handle* h) {
    for (int e = 0; e < kReadyEvents; ++e)
        if (!h->ev_ready[e]) HIP_TRY(hipEventCreateWithFlags(&h->ev_ready[e], kOrderOnly));
    if (!h->ev_side_done) HIP_TRY(hipEventCreateWithFlags(&h->ev_side_done, kOrderOnly));
    for (int e = 0; e < kChunkEvents; ++e)
        if (!h->ev_chunk[e]) HIP_TRY(hipEventCreateWithFlags(&h->ev_chunk[e], kOrderOnly));
    if (!h->ev_upd_done) HIP_TRY(hipEventCreateWithFlags(&h->ev_upd_done, kOrderOnly));
    if (!h->ev_tr_go) HIP_TRY(hipEventCreateWithFlags(&h->ev_tr_go, kOrderOnly));
    if (!h->ev_tr_done) HIP_TRY(hipEventCreateWithFlags(&h->ev_tr_done, kOrderOnly));
    for (int e = 0; e < kBranchEvents; ++e) {
        if (!h->ev_branch_go[e]) HIP_TRY(hipEventCreateWithFlags(&h->ev_branch_go[e], kOrderOnly));
        if (!h->ev_branch_done[e]) HIP_TRY(hipEventCreateWithFlags(&h->ev_branch_done[e], kOrderOnly));
    }
    return EDL_OK;
}

// takes the library's pair of side streams for the job's stream into use (created by the first job there)
static int acquire_side_streams(edl_handle* h) {
    std::lock_guard<std::mutex> lock(g_side_streams_mutex);
    SharedStreams* s = nullptr;
    for (SharedStreams& q : g_side_streams)
        if (q.device == h->device && q.main == h->st) s = &q;
    if (s == nullptr) {
        SharedStreams q = {h->device, h->st, nullptr, nullptr, 0};
        HIP_TRY(hipStreamCreateWithFlags(&q.side, hipStreamNonBlocking));
        const hipError_t e = hipStreamCreateWithFlags(&q.upd, hipStreamNonBlocking);
        if (e != hipSuccess) {
            (void)hipStreamDestroy(q.side);
            HIP_TRY(e);
        }
        g_side_streams.push_back(q);
        s = &g_side_streams.back();
    }
    s->users += 1;
    h->side = s->side;
    h->upd = s->upd;
    h->own_streams = true;
    return EDL_OK;
}

// waits for the side streams and lets go of them (the library's own go with their last user)
static void release_side_streams(edl_handle* h) {
    if (h->side) (void)hipStreamSynchronize(h->side);
    if (h->upd) (void)hipStreamSynchronize(h->upd);
    if (h->own_streams) {
        std::lock_guard<std::mutex> lock(g_side_streams_mutex);
        for (size_t i = 0; i < g_side_streams.size(); ++i) {
            if (g_side_streams[i].side != h->side || --g_side_streams[i].users > 0) continue;
            (void)hipStreamDestroy(h->side);
            (void)hipStreamDestroy(h->upd);
            g_side_streams.erase(g_side_streams.begin() + (long)i);
            break;
        }
    }
    h->side = nullptr;
    h->upd = nullptr;
    h->own_streams = false;
}

// frees whatever of the handle's resources exist (also a half-built handle) and the handle
static void destroy_handle(edl_handle* h) {
    (void)hipStreamSynchronize(h->st);
    release_side_streams(h);
    for (int s = 0; s < kIdxSlots; ++s) {
        if (h->idx_host[s]) (void)hipHostFree(h->idx_host[s]);
        if (h->idx_event[s]) (void)hipEventDestroy(h->idx_event[s]);
    }
    if (h->loss_host) (void)hipHostFree(h->loss_host);
    for (int e = 0; e < kReadyEvents; ++e)
        if (h->ev_ready[e]) (void)hipEventDestroy(h->ev_ready[e]);
    for (int e = 0; e < kChunkEvents; ++e)
        if (h->ev_chunk[e]) (void)hipEventDestroy(h->ev_chunk[e]);
    if (h->ev_side_done) (void)hipEventDestroy(h->ev_side_done);
    if (h->ev_upd_done) (void)hipEventDestroy(h->ev_upd_done);
    if (h->ev_tr_go) (void)hipEventDestroy(h->ev_tr_go);
    if (h->ev_tr_done) (void)hipEventDestroy(h->ev_tr_done);
    for (int e = 0; e < kBranchEvents; ++e) {
        if (h->ev_branch_go[e]) (void)hipEventDestroy(h->ev_branch_go[e]);
        if (h->ev_branch_done[e]) (void)hipEventDestroy(h->ev_branch_done[e]);
    }
    delete h;
}

int32_t edl_init(edl_handle** out, const edl_config* cfg, uint64_t seed, void* dev_arena, size_t arena_bytes,
                 void* hip_stream) {
    if (!out || !cfg || !dev_arena) { set_error("null argument"); return EDL_EINVAL; }
    int rc = validate(*cfg);
    if (rc) return rc;
    if (((uintptr_t)dev_arena) % kAlign) { set_error("arena must be 256-byte aligned"); return EDL_EINVAL; }
    edl_handle* h = new edl_handle();
    h->cfg = *cfg;
    h->seed = seed;
    rc = build_graph(*cfg, h->g);
    if (rc) { delete h; return rc; }
    if (!plan_layout(*cfg, h->g, h->L, (int64_t)std::min<size_t>(arena_bytes, INT64_MAX))) {
        set_error("arena of %zu bytes is smaller than the %lld needed", arena_bytes, (long long)h->L.total);
        delete h;
        return EDL_ENOMEM;
    }
    h->static_fits = plan_static_scratch(*cfg, h->g, h->L, h->static_plan);
    // a conv output feeding a batch norm must have no other consumer (its gradient is written, not added)
    h->arena = (char*)dev_arena;
    h->st = (hipStream_t)hip_stream;
    h->readers.assign(h->g.tensors.size(), 0);
    h->written.assign(h->g.tensors.size(), 0);
    h->op_done.assign(h->g.ops.size(), 0);
    h->wgrad_waiting.reserve(h->g.ops.size());
    h->bias_waiting.assign(h->g.ops.size(), 0);
    h->dw_in_pieces.assign(h->g.ops.size(), 0);
    for (const Op& op : h->g.ops) h->has_bn = h->has_bn || op.kind == OP_BN;
    h->grad_alias.assign(h->g.tensors.size(), nullptr);
    h->shard_n.reserve(kMaxP);
    h->perm.reserve((size_t)cfg->N);
    h->first_reader.assign(h->g.tensors.size(), -1);
    for (size_t i = 0; i < h->g.ops.size(); ++i) {
        const Op& op = h->g.ops[i];
        auto reads = [&](int t) {
            const size_t sx = (size_t)storage_of(h->g, t);
            h->readers[sx] += 1;
            if (h->first_reader[sx] < 0) h->first_reader[sx] = (int)i;
        };
        if (op.x >= 0) reads(op.x);
        if (op.kind == OP_BN && op.res >= 0) reads(op.res);
    }
    h->applied_from = h->g.P;
    rc = init_device_state(h);
    if (rc) {                            // whatever was created so far goes again
        destroy_handle(h);
        return rc;
    }
    *out = h;
    return EDL_OK;
}

// Pinned staging, events, the library's own side streams, and the initial model on the device.
static int init_device_state(edl_handle* h) {
    const edl_config* cfg = &h->cfg;
    const uint64_t seed = h->seed;
    for (int s = 0; s < kIdxSlots; ++s) {
        HIP_TRY(hipHostMalloc((void**)&h->idx_host[s], sizeof(int64_t) * (size_t)cfg->B, hipHostMallocDefault));
        HIP_TRY(hipEventCreateWithFlags(&h->idx_event[s], hipEventDisableTiming));
    }
    HIP_TRY(hipHostMalloc((void**)&h->loss_host, kStageBytes, hipHostMallocDefault));
    // this GPU's copy of the static scratch buffer: its address is looked up once, with the device current
    HIP_TRY(hipGetDevice(&h->device));
    if (h->device >= 0 && h->device < kMaxDevices && g_static_scratch[h->device] == nullptr) {
        void* ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        g_static_scratch[h->device] = ptr;
    }
    if (tune().wgrad_stream != 0) {
        int rc = acquire_side_streams(h);
        if (!rc) rc = create_side_events(h);
        if (rc) return rc;
    }
    std::vector<float> init((size_t)h->g.P);
    std::vector<TransposeEntry> tab, tabv;
    // the copies below read these host arrays: whichever way this function is left, the stream is drained first
    struct DrainOnExit { hipStream_t st; ~DrainOnExit() { (void)hipStreamSynchronize(st); } } drain{h->st};
    he_init(h->g, seed, init.data());
    HIP_TRY(hipMemcpyAsync(h->w(), init.data(), sizeof(float) * (size_t)h->g.P, hipMemcpyHostToDevice, h->st));
    launch_fill_f32(h->v(), 0.f, h->g.P, h->st);
    if (h->adam()) launch_fill_f32(h->s2(), 0.f, h->g.P, h->st);
    for (const Op& op : h->g.ops)
        if (op.kind == OP_BN) {
            launch_fill_f32(h->running() + op.run_off, 0.f, op.K, h->st);
            launch_fill_f32(h->running() + op.run_off + op.K, 1.f, op.K, h->st);
        }
    {
        // bf16 layers of vector-friendly shape are transposed from the bf16 copy of the weights in 64x64
        // tiles; the others element by element from the float32 weights
        const double esz = cfg->dtype == EDL_DTYPE_BF16 ? 2.0 : 4.0;
        for (size_t i = 0; i < h->g.ops.size(); ++i) {
            const Op& op = h->g.ops[i];
            if (op.kind != OP_CONV || h->L.wT[i] < 0) continue;
            const Tensor& tx = h->g.tensors[(size_t)op.x];
            TransposeEntry te;
            te.src_off = op.w_off; te.dst_off = h->L.wT[i];
            te.K = op.K; te.RS = op.R * op.S; te.C = tx.C;
            if (cfg->dtype == EDL_DTYPE_BF16 && te.K % 8 == 0 && te.C % 8 == 0 && op.w_off % 8 == 0) {
                te.tile_start = h->tv_tiles;
                h->tv_tiles += ((te.C + 63) / 64) * ((te.K + 63) / 64) * te.RS;
                h->tv_bytes += 4.0 * (double)te.K * te.RS * te.C;
                tabv.push_back(te);
            } else {
                te.tile_start = h->t_tiles;
                h->t_tiles += ((te.C + 31) / 32) * ((te.K + 31) / 32) * te.RS;
                h->t_bytes += (4.0 + esz) * (double)te.K * te.RS * te.C;
                tab.push_back(te);
            }
        }
        h->t_entries = (int)tab.size();
        h->tv_entries = (int)tabv.size();
        if (!tab.empty())
            HIP_TRY(hipMemcpyAsync(h->at<TransposeEntry>(h->L.ttable), tab.data(), sizeof(TransposeEntry) * tab.size(),
                                   hipMemcpyHostToDevice, h->st));
        if (!tabv.empty())
            HIP_TRY(hipMemcpyAsync(h->at<TransposeEntry>(h->L.ttable) + h->g.ops.size(), tabv.data(),
                                   sizeof(TransposeEntry) * tabv.size(), hipMemcpyHostToDevice, h->st));
        HIP_TRY(hipStreamSynchronize(h->st));
    }
    h->weights_dirty = true;
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

int32_t edl_set_side_streams(edl_handle* h, void* wgrad_stream, void* update_stream) {
    if (!h) { set_error("null handle"); return EDL_EINVAL; }
    if ((wgrad_stream == nullptr) != (update_stream == nullptr)) { set_error("give both streams or neither"); return EDL_EINVAL; }
    if (wgrad_stream != nullptr && (wgrad_stream == update_stream || wgrad_stream == (void*)h->st || update_stream == (void*)h->st)) {
        set_error("the two side streams must differ from each other and from the job's stream");
        return EDL_EINVAL;
    }
    HIP_TRY(hipStreamSynchronize(h->st));
    release_side_streams(h);
    if (wgrad_stream == nullptr) return EDL_OK;         // everything on the job's stream from now on
    h->side = (hipStream_t)wgrad_stream;
    h->upd = (hipStream_t)update_stream;
    h->own_streams = false;
    const int rc = create_side_events(h);
    if (rc) { release_side_streams(h); return rc; }
    return EDL_OK;
}

int32_t edl_set_option(const char* name, int64_t value) {
    if (!tune_set(name, value)) { set_error("no option named '%s'", name ? name : "(null)"); return EDL_EINVAL; }
    return EDL_OK;
}

int32_t edl_get_option(const char* name, int64_t* out_value) {
    if (!tune_get(name, out_value)) { set_error("no option named '%s'", name ? name : "(null)"); return EDL_EINVAL; }
    return EDL_OK;
}

int32_t edl_bind_dataset(edl_handle* h, const float* dev_x, const int32_t* dev_y, int64_t N) {
    if (!h || !dev_x || !dev_y) { set_error("null argument"); return EDL_EINVAL; }
    if (N != h->cfg.N) { set_error("data set has %lld samples, the job was created for %lld", (long long)N, (long long)h->cfg.N); return EDL_EINVAL; }
    h->data_x = dev_x;
    h->data_y = dev_y;
    return EDL_OK;
}

int32_t edl_shard(const edl_handle* h, int64_t B, int32_t p, int64_t epoch, int64_t step_in_epoch, int64_t* out_idx,
                  int64_t* out_off) {
    if (!h) { set_error("null handle"); return EDL_EINVAL; }
    return edl_shard_host(h->seed, h->cfg.N, B, p, epoch, step_in_epoch, out_idx, out_off);
}

// Whether the last layer, op i, the loss and their backward pass go in one launch: few outputs over a ReLU layer with a bias that
// nothing else reads.
static bool classifier_together(const edl_handle* h, size_t i, const ShardSet& S, const void* weights) {
    const Graph& g = h->g;
    const Op& op = g.ops[i];
    if (i == 0 || op.kind != OP_CONV || op.relu || !op.bias || g.ops[i + 1].kind != OP_LOSS || g.ops[i + 1].x != op.y) return false;
    const Op& prod = g.ops[i - 1];
    const int sx = storage_of(g, op.x);
    return prod.kind == OP_CONV && prod.relu && prod.bias && storage_of(g, prod.y) == sx && sx != 0 && h->readers[(size_t)sx] == 1 &&
           h->L.wT[i] < 0 && h->L.wpad[i] < 0 && op.K == g.classes && thin_head_takes(h->cfg.dtype, geom_stored(g, op, S.samples(), h->L.in), S, h->act(op.x), weights);
}

// Whether the first layer takes a pass's samples from the data set itself, their numbers in the launch's arguments: no copy of
// the numbers to the GPU and no gather then.
static bool gathers_itself(const edl_handle* h, const ShardSet& S) {
    const Graph& g = h->g;
    const Op& op = g.ops[0];
    return op.kind == OP_CONV && storage_of(g, op.x) == 0 && !stored_apart(g, h->L.in) && h->L.wpad[0] < 0 && h->cfg.dtype != EDL_DTYPE_BF16 &&
           h->cfg.N <= INT32_MAX && conv_fwd_gathers(h->cfg.dtype, geom_stored(g, op, S.samples(), h->L.in), S, h->data_x, h->act(0), h->w() + op.w_off);
}

// Forward pass of a set of shards whose samples' indices start at dev_idx; mean losses into dev_losses[worker].
// op_lo..op_hi: the slice of the layer list to run (the whole list in normal use;
// single layers from the debugging hooks, which then skip the gather)
// host_idx: the samples' numbers where the first layer gathers them itself (gathers_itself), else null.
// train: a backward pass over the same shards follows.  Returns whether the last layer's part of it is done (thin_head_takes).
static bool forward_pass(edl_handle* h, const ShardSet& S, const int64_t* dev_idx, float* dev_losses, bool update_running,
                         size_t op_lo = 0, size_t op_hi = (size_t)-1, const int64_t* host_idx = nullptr, bool train = false) {
    const int n = S.samples();
    const Graph& g = h->g;
    bool head = false;
    const int dt = h->cfg.dtype;
    hipStream_t st = h->st;
    const bool bf = dt == EDL_DTYPE_BF16;
    float* partial = h->sc<float>(h->L.partial);
    const Tensor& tin = g.tensors[0];
    if (dev_idx && !host_idx) {
        if (stored_apart(g, h->L.in))
            launch_gather_pad(dt, h->data_x, h->data_y, dev_idx, n, tin.H, tin.W, tin.C, h->L.in, h->act(0),
                              h->at<int32_t>(h->L.labels), st);
        else
            launch_gather(dt, h->data_x, h->data_y, dev_idx, n, tin.elems(), h->act(0), h->at<int32_t>(h->L.labels), st);
    }
    if (op_hi > g.ops.size()) op_hi = g.ops.size();
    RowCut sums;                // p > 0: the convolution just launched left the next batch norm's partial sums
    const size_t pf = (size_t)h->L.partial_floats;
    // the same for a convolution whose batch norm is not the next op: its sums wait in a buffer of their own
    float* const partial_held = h->sc<float>(h->L.partial_held);
    RowCut held_sums;
    int held_tensor = -1;
    auto weights_of = [&](size_t i) {
        const Op& o = g.ops[i];
        const void* wsrc = bf ? (const void*)(h->at<uint16_t>(h->L.shadow) + o.w_off) : (const void*)(h->w() + o.w_off);
        if (h->L.wpad[i] >= 0) wsrc = h->arena + h->L.wpad[i];
        return wsrc;
    };
    // A residual block's projection shortcut (convolution + batch norm on the block's input) runs on the second
    // side stream while the main branch runs here; the block's last batch norm, which adds the two, waits for it.
    // Only when the whole list runs and nothing is being timed kernel by kernel.
    const bool branch = op_lo == 0 && op_hi == g.ops.size() && h->upd != nullptr && !prof_enabled() && tune().branch_stream != 0;
    std::vector<char>& done = h->op_done;
    std::fill(done.begin(), done.end(), 0);
    int join_tensor = -1;
    hipEvent_t join_event = nullptr;
    for (size_t i = op_lo; i < op_hi; ++i) {
        const Op& op = g.ops[i];
        if (done[i]) continue;
        if (branch && op.kind == OP_CONV && join_tensor < 0) {
            for (size_t j = i + 1; j + 2 < op_hi && j <= i + 8; ++j) {
                const Op& pj = g.ops[j];
                const Op& pb = g.ops[j + 1];
                if (!(pj.kind == OP_CONV && pj.x == op.x && pb.kind == OP_BN && pb.x == pj.y && pb.res < 0)) continue;
                bool joins = false;
                for (size_t k = j + 2; k < op_hi && k <= j + 3; ++k) joins = joins || (g.ops[k].kind == OP_BN && g.ops[k].res == pb.y);
                if (!joins) break;
                hipEvent_t go = h->ev_branch_go[h->branch_slot], dn = h->ev_branch_done[h->branch_slot];
                if (hipEventRecord(go, st) != hipSuccess || hipStreamWaitEvent(h->upd, go, 0) != hipSuccess) break;
                h->branch_slot = (h->branch_slot + 1) % kBranchEvents;
                float* const ps = h->sc<float>(h->L.partial_side);
                // this stream's own split-reduction scratch (the main stream's is in use)
                const RowCut left = launch_conv_fwd(dt, geom_stored(g, pj, n, h->L.in), S, h->act(pj.x), weights_of(j),
                                                    pj.bias ? h->w() + pj.b_off : nullptr, pj.relu, g.tensors[(size_t)pj.y].fp32,
                                                    h->act(pj.y), h->sc<float>(h->L.splitk_side), (size_t)h->L.splitk_scratch_bytes,
                                                    SumsBuf{ps, pf}, h->upd);
                const Tensor& t = g.tensors[(size_t)pb.x];
                launch_bn_forward(dt, h->act(pb.x), nullptr, h->act(pb.y), h->w() + pb.w_off, h->w() + pb.b_off,
                                  h->at<float>(h->L.bn_save[j + 1]), update_running ? h->running() + pb.run_off : nullptr,
                                  S, t.H * t.W, t.C, pb.relu, h->sign(pb.y), ps, left, h->upd);
                (void)hipEventRecord(dn, h->upd);
                done[j] = done[j + 1] = 1;
                join_tensor = pb.y;
                join_event = dn;
                break;
            }
        }
        switch (op.kind) {
            case OP_CONV: {
                const void* wsrc = weights_of(i);
                if (host_idx && i == 0) {
                    const SmallInput in = {h->data_x, h->data_y, host_idx, (float*)h->act(0), h->at<int32_t>(h->L.labels)};
                    launch_small_fc_fwd(geom_stored(g, op, n, h->L.in), S, (const float*)h->act(op.x), (const float*)wsrc, op.bias ? h->w() + op.b_off : nullptr,
                                        op.relu, (float*)h->act(op.y), &in, st);
                    break;
                }
                // The classifier, the loss and what their backward pass leaves: the next op is done then
                if (train && i + 2 == op_hi && op_hi == g.ops.size() && classifier_together(h, i, S, wsrc)) {
                    const Op& prod = g.ops[i - 1];
                    ThinHead t = {};
                    t.x = h->act(op.x); t.w = wsrc; t.bias = h->w() + op.b_off; t.labels = h->at<int32_t>(h->L.labels);
                    t.logits = (float*)h->act(op.y); t.row_loss = h->sc<float>(h->L.row_loss); t.loss = dev_losses;
                    t.dlogits = h->grad(op.y); t.dx = h->grad(op.x);
                    t.dw = GradDst{h->grad_buf(0) + op.w_off, h->L.grad_stride};
                    t.db = GradDst{h->grad_buf(0) + op.b_off, h->L.grad_stride};
                    t.dbias = GradDst{h->grad_buf(0) + prod.b_off, h->L.grad_stride};
                    launch_thin_head(dt, geom_stored(g, op, n, h->L.in), S, t, st);
                    done[i + 1] = 1;
                    head = true;
                    break;
                }
                // the batch norm that follows (in this call) can take its sums from the convolution's epilogue
                const bool bn_next = i + 1 < op_hi && g.ops[i + 1].kind == OP_BN && g.ops[i + 1].x == op.y;
                // ... or a later one of this call, if the held buffer is free
                const bool tune_held = tune().held_stats != 0;
                bool bn_later = false;
                if (!bn_next && tune_held && held_tensor < 0)
                    for (size_t j = i + 2; j < op_hi && j <= i + 4 && !bn_later; ++j)
                        bn_later = g.ops[j].kind == OP_BN && g.ops[j].x == op.y;
                const RowCut left = launch_conv_fwd(dt, geom_stored(g, op, n, h->L.in), S, h->act(op.x), wsrc,
                                                    op.bias ? h->w() + op.b_off : nullptr, op.relu, g.tensors[(size_t)op.y].fp32,
                                                    h->act(op.y), h->sc<float>(h->L.splitk_scratch),
                                                    (size_t)h->L.splitk_scratch_bytes,
                                                    SumsBuf{bn_next ? partial : bn_later ? partial_held : nullptr, pf}, st);
                if (bn_later) {
                    if (left.p > 0) { held_sums = left; held_tensor = op.y; }
                    sums = RowCut();
                } else {
                    sums = left;
                }
                break;
            }
            case OP_BN: {
                const Tensor& t = g.tensors[(size_t)op.x];
                const bool held = held_tensor == op.x && held_sums.p > 0;
                if (op.res >= 0 && op.res == join_tensor) {      // the shortcut's part comes from the other stream
                    (void)hipStreamWaitEvent(st, join_event, 0);
                    join_tensor = -1;
                }
                launch_bn_forward(dt, h->act(op.x), op.res >= 0 ? h->act(op.res) : nullptr, h->act(op.y), h->w() + op.w_off,
                                  h->w() + op.b_off, h->at<float>(h->L.bn_save[i]),
                                  update_running ? h->running() + op.run_off : nullptr, S, t.H * t.W, t.C, op.relu, h->sign(op.y),
                                  held ? partial_held : partial, held ? held_sums : sums, st);
                if (held) { held_sums = RowCut(); held_tensor = -1; }
                sums = RowCut();
                break;
            }
            case OP_MAXPOOL: {
                const Tensor& tx = g.tensors[(size_t)op.x];
                const Tensor& ty = g.tensors[(size_t)op.y];
                launch_maxpool_forward(dt, h->act(op.x), h->act(op.y), h->at<uint8_t>(h->L.pool_arg[i]), n, tx.H, tx.W, tx.C,
                                       op.R, op.stride, op.pad, ty.H, ty.W, st);
                break;
            }
            case OP_GAVGPOOL: {
                const Tensor& tx = g.tensors[(size_t)op.x];
                launch_gavgpool_forward(dt, h->act(op.x), h->act(op.y), n, tx.H * tx.W, tx.C, st);
                break;
            }
            case OP_LOSS:
                launch_softmax_ce(dt, (const float*)h->act(op.x), h->at<int32_t>(h->L.labels), h->grad(op.x),
                                  h->sc<float>(h->L.row_loss), dev_losses, S, g.classes, st);
                break;
        }
    }
    if (join_tensor >= 0) (void)hipStreamWaitEvent(st, join_event, 0);   // a branch nobody joined (cannot happen)
    return head;
}

static int apply_range(edl_handle* h, int32_t p, int64_t lo, int64_t hi, hipStream_t st, int max_blocks = 0);

// What the input gradient of layer i reads: the transposed copy, or the weights (bf16: their copy) where there is none.
static const void* dgrad_weights(const edl_handle* h, size_t i) {
    if (h->L.wT[i] < 0 && h->cfg.dtype != EDL_DTYPE_BF16) return h->w() + h->g.ops[i].w_off;
    return h->L.wT[i] >= 0 ? (const void*)(h->arena + h->L.wT[i]) : (const void*)(h->arena + h->L.shadow + 2 * h->g.ops[i].w_off);
}

// About how long a layer's weight gradient takes: its launches, and the longer of its contraction (250 and 25 TFLOP/s, what
// such short launches reach) and of its bytes at 4 TB/s.  Only for the choice of what is handed over to the second stream together.
static double weight_gradient_us(int dt, const ConvGeom& q, int shards) {
    const double esz = dt == EDL_DTYPE_BF16 ? 2.0 : 4.0, weights = (double)q.K * q.R * q.S * q.C, rows = (double)q.N * q.Ho * q.Wo;
    const double bytes = 4.0 * shards * weights + esz * (rows * q.K + (double)q.N * q.H * q.W * q.C);
    return 4.0 + std::max(2.0 * weights * rows / (dt == EDL_DTYPE_BF16 ? 250e6 : 25e6), bytes / 4e6);
}

// early_p > 0: this is the last backward pass of a step of early_p shards, so gradients that are final may be
// applied while the pass goes on.
// head: the forward pass has done the last layer's part (forward_pass).
// held (debugging hook only): tensors whose gradient buffers already hold a contribution the pass adds to.
// hook: gradients that the pass needs no more are left in their buffers as well (a debugging hook hands them out).
static void backward_pass(edl_handle* h, const ShardSet& S, size_t op_lo = 0, size_t op_hi = (size_t)-1, int early_p = 0,
                          const std::vector<int>* held = nullptr, bool head = false, bool hook = false) {
    const int n = S.samples();
    // the workers' gradients of the parameters from offset `off` of the flat vector on
    auto grads_at = [&](int64_t off) { return GradDst{h->grad_buf(0) + off, h->L.grad_stride}; };
    const GradDst no_grads = {nullptr, 0};
    const Graph& g = h->g;
    const int dt = h->cfg.dtype;
    hipStream_t st = h->st;
    float* partial = h->sc<float>(h->L.partial);
    float* coef = h->sc<float>(h->L.coef);
    if (h->transposes_pending) {          // the transposed weight copies were made on the weight-gradient stream
        (void)hipStreamWaitEvent(st, h->ev_tr_done, 0);
        h->transposes_pending = false;
    }
    std::vector<char>& written = h->written;     // sized at init: no allocation in the pass
    std::fill(written.begin(), written.end(), 0);
    std::fill(h->grad_alias.begin(), h->grad_alias.end(), nullptr);
    if (held)
        for (int t : *held) written[(size_t)storage_of(g, t)] = 1;
    if (op_hi > g.ops.size()) op_hi = g.ops.size();
    // per-kernel timing wants one kernel at a time
    const bool overlap = h->side != nullptr && !prof_enabled();
    bool used_side = false, used_upd = false;
    // the projection shortcut's backward on the second side stream (see forward_pass)
    const bool branch = overlap && op_lo == 0 && op_hi == g.ops.size() && h->upd != nullptr && tune().branch_stream != 0;
    std::vector<char>& done = h->op_done;
    std::fill(done.begin(), done.end(), 0);
    int join_storage = -1;               // gradient buffer the branch stream is still writing
    hipEvent_t join_event = nullptr;
    size_t fused_for = (size_t)-1;   // the layer whose masked gradient and column sums the dgrad after it left
    RowCut fused_sums;
    float* fused_at = partial;       // ... and where the sums are
    size_t premasked_for = (size_t)-1;   // the layer whose gradient the max pool after it left masked by its ReLU
    // If the layer just before in the list produced a convolution's input and ends in a ReLU, and
    // the convolution is the first reader of that tensor in the list (so every other reader, such as
    // the shortcut of a residual block, has already added its part), that layer's backward starts with
    // the masked gradient and its column sums: the dgrad's epilogue can leave both (see DgradMask),
    // and that layer then skips its own reduction pass.
    auto producer_mask = [&](size_t ii, bool acc, float* sums) {
        DgradMask mask = {};
        const Op& op = g.ops[ii];
        const int sx = storage_of(g, op.x);
        const bool fuse_joins = tune().fused_mask_join != 0;
        const bool last_writer = h->first_reader[(size_t)sx] == (int)ii &&
                                 (h->readers[(size_t)sx] == 1 ? !acc : (fuse_joins && acc));
        if (ii > op_lo && last_writer) {
            const Op& prod = g.ops[ii - 1];
            if (prod.relu && storage_of(g, prod.y) == sx && (prod.kind == OP_BN || prod.kind == OP_CONV)) {
                mask.act = h->act(op.x);
                if (prod.kind == OP_BN) mask.sign = h->sign(op.x);
                mask.sums = SumsBuf{sums, (size_t)h->L.partial_floats};
                if (prod.kind == OP_CONV && prod.bias) mask.dbias = grads_at(prod.b_off);
                if (prod.kind == OP_BN) {
                    mask.xin = h->act(prod.x);
                    mask.mean_rstd = h->at<float>(h->L.bn_save[ii - 1]);
                }
            }
        }
        return mask;
    };
    // The convolution whose output batch norm ii normalises, if the two go backward in one launch (k_bn_pointwise.hip): a plain
    // 1x1 convolution of many pixels, the gradient of whose output nothing else wants, the gradient of whose input nothing
    // has been added to, and a batch norm whose own gradient is there masked.  Else ops.size().
    auto conv_behind = [&](size_t ii) {
        const size_t none = g.ops.size();
        const Op& bn = g.ops[ii];
        if (dt != EDL_DTYPE_BF16 || (bn.relu && fused_for != ii) || h->readers[(size_t)storage_of(g, bn.x)] != 1) return none;
        size_t ic = ii;
        while (ic > op_lo && !(g.ops[ic].kind == OP_CONV && g.ops[ic].y == bn.x)) --ic;
        const Op& op = g.ops[ic];
        if (op.kind != OP_CONV || op.y != bn.x || done[ic] || op.bias || op.relu || h->L.wT[ic] < 0 || h->L.wpad[ic] >= 0) return none;
        const int sx = storage_of(g, op.x);
        if (sx == 0 || written[(size_t)sx] != 0 || h->grad_alias[(size_t)sx] != nullptr) return none;
        const DgradMask mask = producer_mask(ic, false, nullptr);
        if (mask.act != nullptr && (mask.xin == nullptr || tune().fused_mask == 0)) return none;
        return bn_pointwise_takes(dt, geom_stored(g, op, n, h->L.in), S) ? ic : none;
    };
    // ... and that launch, behind the batch norm's sums.  The pieces of the weight gradient lie where the gradient of the
    // batch norm's input would; the column sums in a buffer of their own (a block's projection may come before they are read).
    auto backward_through = [&](size_t ii, size_t ic, const void* dy, const float* bn_coef, hipStream_t bs) {
        const Op& bn = g.ops[ii];
        const Op& op = g.ops[ic];
        const DgradMask mask = producer_mask(ic, false, h->sc<float>(h->L.partial_held));
        BnPointwiseTask t = {};
        t.x = h->act(bn.x); t.dy = dy;
        t.gamma = h->w() + bn.w_off; t.save = h->at<float>(h->L.bn_save[ii]); t.coef = bn_coef;
        t.act = h->act(op.x); t.wT = dgrad_weights(h, ic); t.dact = h->grad(op.x);
        t.mask = mask.act != nullptr ? &mask : nullptr;
        t.partial = (float*)h->grad(op.y);
        const RowCut left = launch_bn_pointwise_backward(geom_stored(g, op, n, h->L.in), S, t, bs);
        if (left.p > 0) { fused_for = ic - 1; fused_sums = left; fused_at = h->sc<float>(h->L.partial_held); }
        written[(size_t)storage_of(g, op.x)] = 1;
        h->dw_in_pieces[ic] = 1;
        done[ic] = 1;
    };
    auto bias_gradient = [&](size_t ii, bool premasked, const RowCut& sums, float* part, hipStream_t bs) {
        const Op& op = g.ops[ii];
        const GradDst dst = op.bias ? grads_at(op.b_off) : no_grads;
        if (premasked && sums.p == 0 && op.bias) {       // its sum is that of the pool's gradient where the pooled value is positive
            const int py = g.ops[ii + 1].y;
            const Tensor& tp = g.tensors[(size_t)py];
            launch_pooled_bias_backward(dt, h->act(py), h->grad(py), dst, S, tp.H * tp.W, op.K, part, bs);
            return;
        }
        const Tensor& ty = g.tensors[(size_t)op.y];
        launch_bias_relu_backward(dt, h->act(op.y), h->grad(op.y), dst, S, ty.H * ty.W, op.K, op.relu && !premasked, part, sums, bs);
    };
    auto weight_gradient = [&](size_t ii, hipStream_t ws, float* scratch) {
        const Op& op = g.ops[ii];
        const ConvGeom q = geom_stored(g, op, n, h->L.in);
        if (h->dw_in_pieces[ii] != 0) {       // its contraction went with the batch norm's backward
            launch_bn_pointwise_reduce(q, S, (const float*)h->grad(op.y), grads_at(op.w_off), ws);
            h->dw_in_pieces[ii] = 0;
            return;
        }
        if (h->bias_waiting[ii] != 0) {
            bias_gradient(ii, h->bias_waiting[ii] == 2, RowCut(), ws == h->side ? h->sc<float>(h->L.partial_side) : h->sc<float>(h->L.partial_held), ws);
            h->bias_waiting[ii] = 0;
        }
        if (h->L.wpad[ii] >= 0) {
            // the shards' gradients of the padded weights side by side, then compacted into the flat vectors
            ShardSet slots = S;
            for (int k = 0; k < S.p; ++k) slots.k[k] = k;
            launch_conv_wgrad(dt, q, slots, h->act(op.x), h->grad(op.y), GradDst{h->sc<float>(h->L.dwpad), op.K * stored_row(op, h->L.in)},
                              scratch, (size_t)h->L.wgrad_scratch_bytes, ws);
            launch_unpad_weights(h->sc<float>(h->L.dwpad), grads_at(op.w_off), S, op.K, op.R, op.S, g.tensors[0].C, h->L.in, ws);
        } else {
            launch_conv_wgrad(dt, q, S, h->act(op.x), h->grad(op.y), grads_at(op.w_off), scratch, (size_t)h->L.wgrad_scratch_bytes, ws);
        }
    };
    // weight gradients that wait to be handed over to the second stream
    std::vector<size_t>& waiting = h->wgrad_waiting;
    waiting.clear();
    double waiting_us = 0;
    auto hand_over = [&]() {
        hipEvent_t ev = h->ev_ready[h->ev_slot];
        h->ev_slot = (h->ev_slot + 1) % kReadyEvents;
        const bool ok = hipEventRecord(ev, st) == hipSuccess && hipStreamWaitEvent(h->side, ev, 0) == hipSuccess;
        for (size_t j : waiting) weight_gradient(j, ok ? h->side : st, h->sc<float>(ok ? h->L.wgrad_scratch : h->L.wgrad_scratch2));
        used_side = used_side || ok;
        waiting.clear();
        waiting_us = 0;
        return ok;
    };
    // For a hook: the gradient of the input of batch norm ii, which went backward with convolution ic, in the place of the pieces
    auto instead_of_pieces = [&](size_t ii, size_t ic, const void* dy, const float* bn_coef, hipStream_t bs) {
        const Op& bn = g.ops[ii];
        const Tensor& t = g.tensors[(size_t)bn.x];
        weight_gradient(ic, bs, nullptr);
        launch_bn_backward_apply(h->act(bn.x), dy, h->grad(bn.x), h->w() + bn.w_off, h->at<float>(h->L.bn_save[ii]), bn_coef, S, t.H * t.W, t.C, bs);
    };
    for (size_t ii = op_hi; ii-- > op_lo;) {
        const Op& op = g.ops[ii];
        if (done[ii]) continue;
        if (join_storage >= 0 && op.x >= 0 && storage_of(g, op.x) == join_storage) {
            // this layer adds to the gradient the branch stream has been writing
            (void)hipStreamWaitEvent(st, join_event, 0);
            join_storage = -1;
        }
        switch (op.kind) {
            case OP_LOSS:
                written[(size_t)storage_of(g, op.x)] = 1;
                break;
            case OP_CONV: {
                if (head && ii + 2 == g.ops.size()) {
                    written[(size_t)storage_of(g, op.x)] = 1;
                    fused_for = ii - 1;
                    fused_sums = cut_rows(S, 1, n);
                    fused_sums.stored = true;
                    break;
                }
                const ConvGeom q = geom_stored(g, op, n, h->L.in);
                // The weight gradient needs only dy (final from here on) and the layer's input, and nothing
                // before the update reads it: it runs on the second stream, beside the chain of input
                // gradients, whose short kernels leave part of the chip idle.  Handing work over costs an event (1 us on
                // this chain, some 18 us of host time), so small layers' gradients are handed over together.
                // The first layers' weight gradients are the last of the pass: by then the main stream has nothing
                // else to do, so they stay on it (with a scratch of their own) and run beside the second stream's backlog.
                int conv_ordinal = 0;
                for (size_t j = 0; j < ii; ++j) conv_ordinal += g.ops[j].kind == OP_CONV;
                const bool on_main = !overlap || conv_ordinal < (int)tune().wgrad_tail_main;
                // Bias and ReLU mask come first, except where the chain needs nothing of them: with the gradient masked by the
                // pool after the layer, or without a ReLU, what is left is the bias gradient's sum, which goes with the weight
                // gradient (VGG-16, shard of 32: 21 us a layer on the chain; jobs with batch norms use the second
                // buffer of partial sums on their branch stream).
                // a small layer's weight gradient is left by the launch of its input gradient
                const bool with_dgrad = storage_of(g, op.x) != 0 && h->L.wT[ii] < 0 && h->L.wpad[ii] < 0 && conv_gradients_together(dt, q, S, true);
                const bool aside = op.bias && !on_main && !with_dgrad && !h->has_bn && fused_for != ii && (premasked_for == ii || !op.relu);
                if (!aside) bias_gradient(ii, premasked_for == ii, fused_for == ii ? fused_sums : RowCut(), fused_for == ii ? fused_at : partial, st);
                const int64_t own = (int64_t)op.K * op.R * op.S * g.tensors[(size_t)op.x].C;
                const bool early = early_p > 0 && overlap && !on_main && h->upd != nullptr && tune().early_update > 0 && own >= tune().early_update;
                bool handed_over = false;
                if (on_main && !with_dgrad) {
                    weight_gradient(ii, st, h->sc<float>(overlap ? h->L.wgrad_scratch2 : h->L.wgrad_scratch));
                } else if (!with_dgrad) {
                    waiting.push_back(ii);
                    if (aside) h->bias_waiting[ii] = premasked_for == ii ? 2 : 1;
                    // From 15 us of work on, and a layer of 8 or 10 us at once.  us per step: each layer by itself / from 15 with 10 at
                    // once / 15 and 8 / 20 and 8 / 25 and 8 (MLP, 4 x 16: 116 / 61 to 70 whichever)
                    //   VGG-16 of 64x64 1 x 4 761 / 782 / 771 / 770 / 770     1 x 8 794 / 805 / 793 / 807 / 806
                    //   2 x 8 924 / 943 / 925 / 924 / 925                     1 x 32 1,015 / 1,029 / 1,015 / 1,015 / 1,015
                    //   of 112x112 1 x 4 890 / 897 / 893 / 900 / 906
                    //   AlexNet of 96x96 1 x 16 425 / 450 / 427 / 431 / 431   of 224x224 1 x 16 749 / 764 / 754 / 750 / 755
                    //   ResNet-20 1 x 8 1,228 / 1,079 / 1,039 / 1,003 / 999   3 x 8 1,339 / 1,126 / 1,280
                    //   ResNet-50 of 112x112 1 x 8 2,928 / 2,382 / 2,388 / 2,305 / 2,262
                    // A layer of 8 to 10 us that waits for the next leaves the second stream idle for longer than its event costs on
                    // the chain.  Not so where the event's host time counts (nets with batch norms launch three times as much per layer:
                    // ResNet-20, 3 x 8), or where nothing but the first layer is left to run beside it and the wait at the end of the
                    // pass is for that layer alone (MLP 784-100-300-10, 8 x 256: 104 behind the chain, 114 handed over).
                    const double us = weight_gradient_us(dt, q, S.p), batch = (double)tune().wgrad_batch_us;
                    waiting_us += us;
                    const double at_once = batch * (!h->has_bn && (used_side || conv_ordinal > 1) ? 8 : 10) / 15;
                    if (early || waiting_us >= batch || us >= at_once) handed_over = hand_over();
                }
                // Parameters are laid out in layer order, so everything from this layer's weights on now has its
                // final gradient: the second stream holds the weight gradients, and the event it waited for
                // covers what the main stream has written (bias and batch-norm gradients of the later layers)
                // and read (their batch-norm scales, and the weights of those whose input gradient reads them where
                // they lie).  Nothing of the rest of the pass reads those parameters but this layer's own input
                // gradient, if it is of that kind: the update then waits for it as well.  Other input gradients use
                // transposed copies.  So their update starts now, on a third stream, if
                // the layer is a large one (chunk_min weights or more: the update of a small piece gains less than
                // its launch beside the input-gradient chain costs).  The piece starts at the layer's first weight
                // rounded up to 64, so that the vector accesses stay aligned; the few weights below go with the
                // next piece or with the rest of the update after the pass.
                const bool reads_weights = storage_of(g, op.x) != 0 && h->L.wT[ii] < 0;
                auto wait_for_main = [&]() {
                    hipEvent_t ev = h->ev_chunk[h->chunk_slot];
                    h->chunk_slot = (h->chunk_slot + 1) % kChunkEvents;
                    return hipEventRecord(ev, st) == hipSuccess && hipStreamWaitEvent(h->upd, ev, 0) == hipSuccess;
                };
                auto update_early = [&]() {
                    if (early && handed_over) {
                        const int64_t lo = (op.w_off + 63) / 64 * 64;
                        if (lo > 0 && lo < h->applied_from) {
                            hipEvent_t ev = h->ev_chunk[h->chunk_slot];
                            h->chunk_slot = (h->chunk_slot + 1) % kChunkEvents;
                            if (hipEventRecord(ev, h->side) == hipSuccess && hipStreamWaitEvent(h->upd, ev, 0) == hipSuccess &&
                                (!reads_weights || wait_for_main())) {
                                // held to few workgroups: a full-width launch would take the CUs from the chain of
                                // input gradients for as long as it runs
                                const int early_blocks = (int)tune().early_blocks;
                                apply_range(h, early_p, lo, h->applied_from, h->upd, early_blocks);
                                h->applied_from = lo;
                                used_upd = true;
                            }
                        }
                    }
                };
                if (!reads_weights) update_early();
                const int sx = storage_of(g, op.x);
                if (sx != 0) {
                    const bool acc = written[(size_t)sx] != 0;
                    const DgradMask mask = producer_mask(ii, acc, partial);
                    const BothGradients both = {h->act(op.x), grads_at(op.w_off)};
                    const RowCut left = launch_conv_dgrad(dt, q, S, h->grad(op.y), dgrad_weights(h, ii), acc, h->grad(op.x),
                                                          h->sc<float>(h->L.splitk_scratch), (size_t)h->L.splitk_scratch_bytes,
                                                          mask.act ? &mask : nullptr, st, acc ? h->grad_alias[(size_t)sx] : nullptr, reads_weights,
                                                          with_dgrad ? &both : nullptr);
                    h->grad_alias[(size_t)sx] = nullptr;
                    if (left.p > 0) { fused_for = ii - 1; fused_sums = left; fused_at = partial; }
                    written[(size_t)sx] = 1;
                }
                if (reads_weights) update_early();
                break;
            }
            case OP_BN: {
                const Tensor& t = g.tensors[(size_t)op.x];
                const int sx = storage_of(g, op.x);
                void* dres = nullptr;
                bool dres_acc = false;
                if (op.res >= 0 && storage_of(g, op.res) != 0) {
                    const int sr = storage_of(g, op.res);
                    dres = h->grad(op.res);
                    dres_acc = written[(size_t)sr] != 0;
                    written[(size_t)sr] = 1;
                    // An identity shortcut whose gradient would be a plain copy of this layer's (already masked)
                    // output gradient: nothing is copied; the one other reader of the tensor - a stride-1
                    // convolution later in this pass, which adds its part - reads it from where it lies.
                    const bool dy_is_dres = !dres_acc && (!op.relu || fused_for == ii || premasked_for == ii);
                    const int fr = h->first_reader[(size_t)sr];
                    if (dy_is_dres && tune().alias_shortcut != 0 && h->readers[(size_t)sr] == 2 && fr >= (int)op_lo && fr < (int)ii &&
                        g.ops[(size_t)fr].kind == OP_CONV && g.ops[(size_t)fr].stride == 1 && storage_of(g, g.ops[(size_t)fr].x) == sr) {
                        h->grad_alias[(size_t)sr] = h->grad(op.y);
                        dres = nullptr;
                    }
                    // The same for a projection shortcut: the batch norm listed just before produced the tensor and is
                    // its only other user, and its backward only reads the gradient.
                    if (dy_is_dres && tune().alias_shortcut != 0 && h->readers[(size_t)sr] == 1 && ii >= op_lo + 1 &&
                        g.ops[ii - 1].kind == OP_BN && g.ops[ii - 1].y == op.res && !g.ops[ii - 1].relu) {
                        h->grad_alias[(size_t)sr] = h->grad(op.y);
                        dres = nullptr;
                    }
                }
                const size_t sy = (size_t)storage_of(g, op.y);
                const void* const dy_src = h->grad_alias[sy] ? h->grad_alias[sy] : h->grad(op.y);
                h->grad_alias[sy] = nullptr;
                const size_t behind = dres == nullptr ? conv_behind(ii) : g.ops.size();
                launch_bn_backward(dt, h->act(op.x), h->act(op.y), dy_src, behind < ii ? nullptr : h->grad(op.x), dres, dres_acc,
                                   h->w() + op.w_off, h->at<float>(h->L.bn_save[ii]), grads_at(op.w_off), grads_at(op.b_off),
                                   S, t.H * t.W, t.C, op.relu && premasked_for != ii, fused_for == ii ? fused_at : partial, coef,
                                   fused_for == ii ? fused_sums : RowCut(), st);
                written[(size_t)sx] = 1;
                // The gradient of the shortcut is final now.  If the shortcut is a projection (the convolution and
                // batch norm listed just before), its backward - batch norm, weight gradient, input gradient into
                // the block's input - needs nothing else of the main branch: it goes to the second side stream,
                // with a reduction scratch of its own, while the main branch's chain continues here.  The block's
                // first convolution, which adds to the same input gradient, waits for it.
                if (branch && op.res >= 0 && ii >= op_lo + 2 && join_storage < 0) {
                    const Op& pb = g.ops[ii - 1];
                    const Op& pj = g.ops[ii - 2];
                    const int pj_sx = pj.x >= 0 ? storage_of(g, pj.x) : 0;
                    if (pb.kind == OP_BN && pb.y == op.res && pb.res < 0 && pj.kind == OP_CONV && pj.y == pb.x && pj_sx != 0 &&
                        h->L.wpad[ii - 2] < 0) {
                        hipEvent_t go = h->ev_branch_go[h->branch_slot], dn = h->ev_branch_done[h->branch_slot];
                        hipEvent_t wg = h->ev_ready[h->ev_slot];
                        if (hipEventRecord(go, st) == hipSuccess && hipStreamWaitEvent(h->upd, go, 0) == hipSuccess) {
                            h->branch_slot = (h->branch_slot + 1) % kBranchEvents;
                            h->ev_slot = (h->ev_slot + 1) % kReadyEvents;
                            hipStream_t bs = h->upd;
                            float* const ps = h->sc<float>(h->L.partial_side);
                            const Tensor& tb = g.tensors[(size_t)pb.x];
                            const size_t spy = (size_t)storage_of(g, pb.y);
                            const void* const pdy = h->grad_alias[spy] ? h->grad_alias[spy] : h->grad(pb.y);
                            h->grad_alias[spy] = nullptr;
                            const size_t pbehind = conv_behind(ii - 1);
                            launch_bn_backward(dt, h->act(pb.x), h->act(pb.y), pdy, pbehind < ii ? nullptr : h->grad(pb.x), nullptr, false,
                                               h->w() + pb.w_off, h->at<float>(h->L.bn_save[ii - 1]), grads_at(pb.w_off), grads_at(pb.b_off),
                                               S, tb.H * tb.W, tb.C, pb.relu, ps, h->sc<float>(h->L.coef_side), RowCut(), bs);
                            written[(size_t)storage_of(g, pb.x)] = 1;
                            const ConvGeom qj = geom_stored(g, pj, n, h->L.in);
                            if (pbehind < ii) {
                                backward_through(ii - 1, pbehind, pdy, h->sc<float>(h->L.coef_side), bs);
                                if (hook) instead_of_pieces(ii - 1, pbehind, pdy, h->sc<float>(h->L.coef_side), bs);
                            } else {
                                launch_bias_relu_backward(dt, h->act(pj.y), h->grad(pj.y), pj.bias ? grads_at(pj.b_off) : no_grads, S,
                                                          qj.Ho * qj.Wo, pj.K, pj.relu, ps, RowCut(), bs);
                            }
                            // weight gradient: on the first side stream like every other, behind this stream's work
                            hipStream_t ws = bs;
                            if (hipEventRecord(wg, bs) == hipSuccess && hipStreamWaitEvent(h->side, wg, 0) == hipSuccess) {
                                ws = h->side;
                                used_side = true;
                            }
                            if (pbehind < ii) {
                                if (!hook) weight_gradient(pbehind, ws, nullptr);
                            } else {
                                launch_conv_wgrad(dt, qj, S, h->act(pj.x), h->grad(pj.y), grads_at(pj.w_off),
                                                  ws == h->side ? h->sc<float>(h->L.wgrad_scratch) : nullptr,
                                                  ws == h->side ? (size_t)h->L.wgrad_scratch_bytes : 0, ws);
                                // input gradient, with this stream's own split-reduction scratch; nothing to hand over (the
                                // block's first convolution is the last to add to this gradient)
                                launch_conv_dgrad(dt, qj, S, h->grad(pj.y), dgrad_weights(h, ii - 2), written[(size_t)pj_sx] != 0,
                                                  h->grad(pj.x), h->sc<float>(h->L.splitk_side), (size_t)h->L.splitk_scratch_bytes, nullptr, bs,
                                                  nullptr, h->L.wT[ii - 2] < 0);
                            }
                            written[(size_t)pj_sx] = 1;
                            (void)hipEventRecord(dn, bs);
                            done[ii - 1] = done[ii - 2] = 1;
                            join_storage = pj_sx;
                            join_event = dn;
                            used_upd = true;
                        }
                    }
                }
                if (behind < ii) {
                    backward_through(ii, behind, dy_src, coef, st);
                    if (hook) {
                        instead_of_pieces(ii, behind, dy_src, coef, st);
                    } else if (overlap) {       // the pieces are added up beside the chain, with the next weight gradient handed over
                        waiting.push_back(behind);
                        waiting_us += 8;
                    } else {
                        weight_gradient(behind, st, nullptr);
                    }
                }
                break;
            }
            case OP_MAXPOOL: {
                const Tensor& tx = g.tensors[(size_t)op.x];
                const Tensor& ty = g.tensors[(size_t)op.y];
                const int sx = storage_of(g, op.x);
                if (sx != 0) {
                    // a ReLU layer just before in the list whose output only this pool reads: its gradient can leave
                    // the pool already masked, and with a batch norm's sums
                    const DgradMask mask = h->readers[(size_t)sx] == 1 ? producer_mask(ii, written[(size_t)sx] != 0, tune().fused_mask != 0 ? partial : nullptr) : DgradMask{};
                    RowCut left;
                    if (launch_maxpool_backward(dt, h->grad(op.y), h->at<uint8_t>(h->L.pool_arg[ii]), h->grad(op.x),
                                                written[(size_t)sx] != 0, S, tx.H, tx.W, tx.C, op.R, op.stride, op.pad, ty.H,
                                                ty.W, mask.act != nullptr ? &mask : nullptr, h->act(op.y), &left, st))
                        premasked_for = ii - 1;
                    if (left.p > 0) { fused_for = ii - 1; fused_sums = left; fused_at = partial; }
                    written[(size_t)sx] = 1;
                }
                break;
            }
            case OP_GAVGPOOL: {
                const Tensor& tx = g.tensors[(size_t)op.x];
                const int sx = storage_of(g, op.x);
                if (sx != 0) {
                    launch_gavgpool_backward(dt, h->grad(op.y), h->grad(op.x), written[(size_t)sx] != 0, n, tx.H * tx.W, tx.C, st);
                    written[(size_t)sx] = 1;
                }
                break;
            }
        }
    }
    // too little to hand over: behind the chain (a pass whose weight gradients are all small takes no event at all)
    for (size_t j : waiting) weight_gradient(j, st, h->sc<float>(h->L.wgrad_scratch2));
    waiting.clear();
    // the next forward pass overwrites the activations the weight gradients read, and the update reads G
    if (used_side) {
        (void)hipEventRecord(h->ev_side_done, h->side);
        (void)hipStreamWaitEvent(st, h->ev_side_done, 0);
    }
    if (used_upd) {
        (void)hipEventRecord(h->ev_upd_done, h->upd);
        (void)hipStreamWaitEvent(st, h->ev_upd_done, 0);
    }
}

// how many of p equal shards of n samples one pass runs together
static int shards_per_pass(const edl_handle* h, int64_t n, int p) {
    return (int)std::max<int64_t>(1, std::min<int64_t>(p, std::min<int64_t>(h->L.pass_shards, h->L.pass_samples / n)));
}

static int check_p(const edl_handle* h, int32_t p) {
    if (p <= 0 || p > h->cfg.p_max) { set_error("p=%d outside [1, p_max=%d]", p, h->cfg.p_max); return EDL_EINVAL; }
    if (h->cfg.B % p) { set_error("B=%lld is not a multiple of p=%d", (long long)h->cfg.B, p); return EDL_EINDIVISIBLE; }
    if (h->cfg.B / p > h->cfg.max_shard) { set_error("shard of %lld samples exceeds max_shard=%d", (long long)(h->cfg.B / p), h->cfg.max_shard); return EDL_ENOMEM; }
    return EDL_OK;
}

// The gradient passes of one mini-batch.  alone: every shard in a pass of its own, as the worker that holds only this
// shard would run it, and without touching the running statistics (a measurement; the buffers cannot be applied).
static int gradient_passes(edl_handle* h, int32_t p, const int64_t* idx, const int64_t* off, float* out_loss, bool alone) {
    if (!h) { set_error("null handle"); return EDL_EINVAL; }
    if (!h->data_x) { set_error("no data set bound"); return EDL_EINVAL; }
    if ((idx == nullptr) != (off == nullptr)) { set_error("idx and off must both be given or both be NULL"); return EDL_EINVAL; }
    const int64_t B = h->cfg.B;
    int64_t sizes[kMaxP];
    if (idx) {
        // the caller's cut of the mini-batch: any shard sizes that fit the workspace (equal ones in normal use)
        if (p <= 0 || p > h->cfg.p_max) { set_error("p=%d outside [1, p_max=%d]", p, h->cfg.p_max); return EDL_EINVAL; }
        if (off[0] != 0 || off[p] != B) { set_error("off must run from 0 to B=%lld", (long long)B); return EDL_ERANGE; }
        for (int k = 0; k < p; ++k) {
            const int64_t nk = off[k + 1] - off[k];
            if (nk < 0) { set_error("off[%d] > off[%d]", k, k + 1); return EDL_ERANGE; }
            if (nk > h->cfg.max_shard) { set_error("shard %d of %lld samples exceeds max_shard=%d", k, (long long)nk, h->cfg.max_shard); return EDL_ENOMEM; }
            sizes[k] = nk;
        }
    } else {
        const int rc = check_p(h, p);
        if (rc) return rc;
        for (int k = 0; k < p; ++k) sizes[k] = B / p;
    }
    bool equal = true;
    for (int k = 0; k < p; ++k) equal = equal && sizes[k] == sizes[0];
    const int slot = h->idx_slot;
    h->idx_slot = (slot + 1) % kIdxSlots;
    HIP_TRY(hipEventSynchronize(h->idx_event[slot]));
    int64_t* stage = h->idx_host[slot];
    if (idx) {
        for (int64_t i = 0; i < B; ++i) {
            if (idx[i] < 0 || idx[i] >= h->cfg.N) { set_error("idx[%lld]=%lld outside [0,N)", (long long)i, (long long)idx[i]); return EDL_ERANGE; }
            stage[i] = idx[i];
        }
    } else {
        if (h->perm_epoch != h->prog.epoch) {
            epoch_permutation(h->seed, h->prog.epoch, h->cfg.N, h->perm);
            h->perm_epoch = h->prog.epoch;
        }
        memcpy(stage, h->perm.data() + h->prog.step_in_epoch * B, sizeof(int64_t) * (size_t)B);
    }
    h->shard_n.assign(sizes, sizes + p);
    h->shards_equal = equal;
    int64_t* dev_idx = h->at<int64_t>(h->L.idx);
    // The shards of the pass from shard k on
    auto shards_from = [&](int& k, int last_k) {
        ShardSet S = {};
        for (; k <= last_k; ++k) {
            if (sizes[k] == 0) continue;
            if (S.p > 0 && (alone || S.p == h->L.pass_shards || S.off[S.p] + sizes[k] > h->L.pass_samples)) break;
            S.k[S.p] = k;
            S.off[S.p + 1] = S.off[S.p] + (int)sizes[k];
            S.p += 1;
        }
        if (equal && !alone) S.plan_equal((int)sizes[0], shards_per_pass(h, sizes[0], p));
        else S.plan_itself();
        return S;
    };
    int last_k = -1;
    for (int k = 0; k < p; ++k)
        if (sizes[k] > 0) last_k = k;
    bool in_arguments = false;       // the samples' numbers: where one pass of one part takes the whole mini-batch
    if (last_k >= 0) {
        int k = 0;
        const ShardSet S = shards_from(k, last_k);
        in_arguments = k > last_k && S.p <= h->L.scratch_shards && S.samples() <= h->L.scratch_samples && gathers_itself(h, S);
    }
    if (!in_arguments) {
        HIP_TRY(hipMemcpyAsync(dev_idx, stage, sizeof(int64_t) * (size_t)B, hipMemcpyHostToDevice, h->st));
        HIP_TRY(hipEventRecord(h->idx_event[slot], h->st));
    }
    if (h->weights_dirty) {
        refresh_weight_copies(h);
        h->weights_dirty = false;
    }
    // The transposed copies are first read by the backward pass: they are made on the weight-gradient stream, which
    // is idle during the forward pass, and the first backward pass waits for them.
    h->transposes_pending = false;
    if (h->side != nullptr && !prof_enabled() && tune().transpose_stream != 0 &&
        hipEventRecord(h->ev_tr_go, h->st) == hipSuccess && hipStreamWaitEvent(h->side, h->ev_tr_go, 0) == hipSuccess) {
        transpose_weights(h, h->side);
        h->transposes_pending = hipEventRecord(h->ev_tr_done, h->side) == hipSuccess;
        if (!h->transposes_pending) (void)hipStreamSynchronize(h->side);
    } else {
        transpose_weights(h, h->st);
    }
    float* dev_losses = h->at<float>(h->L.losses);
    int64_t at = 0;
    bool first = true;       // the first worker that has samples keeps the running statistics
    // consecutive shards in passes of as many as the workspace holds
    for (int k = 0; k <= last_k;) {
        const ShardSet S = shards_from(k, last_k);
        // ... and a pass in parts, if its scratch takes no more
        for (int s = 0; s < S.p;) {
            ShardSet part = S;
            for (part.p = 0; s < S.p; ++s) {
                const int n = S.off[s + 1] - S.off[s];
                if (part.p > 0 && (part.p == h->L.scratch_shards || part.off[part.p] + n > h->L.scratch_samples)) break;
                part.k[part.p] = S.k[s];
                part.off[part.p + 1] = part.off[part.p] + n;
                part.p += 1;
            }
            const bool head = forward_pass(h, part, dev_idx + at, dev_losses, first && !alone, 0, (size_t)-1, in_arguments ? stage : nullptr, true);
            backward_pass(h, part, 0, (size_t)-1, k > last_k && s == S.p ? h->early_p : 0, nullptr, head);
            first = false;
            at += part.samples();
        }
    }
    HIP_TRY(hipGetLastError());
    if (out_loss) {
        HIP_TRY(hipMemcpyAsync(h->loss_host, dev_losses, sizeof(float) * (size_t)p, hipMemcpyDeviceToHost, h->st));
        HIP_TRY(hipStreamSynchronize(h->st));
        double s = 0;
        if (equal) {
            for (int k = 0; k < p; ++k) s += h->loss_host[k];
            s /= p;
        } else {   // the mean over the mini-batch: every worker's mean weighs in with its share
            for (int k = 0; k < p; ++k)
                if (sizes[k] > 0) s += (double)h->loss_host[k] * ((double)sizes[k] / (double)B);
        }
        *out_loss = (float)s;
    }
    h->grads_pending = !alone;
    return EDL_OK;
}

int32_t edl_gradients(edl_handle* h, int32_t p, const int64_t* idx, const int64_t* off, float* out_loss) {
    return gradient_passes(h, p, idx, off, out_loss, false);
}

// bias corrections of update number t, formed in double
static void adam_corrections(double beta1, double beta2, int64_t t, float* c1, float* c2) {
    *c1 = (float)(1.0 / (1.0 - std::pow(beta1, (double)t)));
    *c2 = (float)(1.0 / (1.0 - std::pow(beta2, (double)t)));
}

// The update of parameters [lo, hi) from the gradient buffers of the step's p shards (every buffer weighs in
// with its shard's share of the mini-batch if the shards are unequal), on stream st.  lo is a multiple of 4.
static int apply_range(edl_handle* h, int32_t p, int64_t lo, int64_t hi, hipStream_t st, int max_blocks) {
    if (hi <= lo) return EDL_OK;
    uint16_t* shadow = h->cfg.dtype == EDL_DTYPE_BF16 ? h->at<uint16_t>(h->L.shadow) + lo : nullptr;
    const int64_t len = hi - lo;
    GradPtrs gp = {};
    ShardShares sh = {};
    int np = 0;
    if (h->shards_equal) {
        for (int k = 0; k < p; ++k) gp.g[k] = h->grad_buf(k) + lo;
        np = p;
    } else {
        for (int k = 0; k < p; ++k) {
            if (h->shard_n[(size_t)k] == 0) continue;
            gp.g[np] = h->grad_buf(k) + lo;
            sh.share[np] = (float)((double)h->shard_n[(size_t)k] / (double)h->cfg.B);
            ++np;
        }
    }
    if (h->adam()) {
        float c1, c2;
        adam_corrections(h->cfg.momentum, h->cfg.beta2, h->prog.step + 1, &c1, &c2);
        launch_adam_update(np, gp, h->shards_equal ? nullptr : &sh, h->w() + lo, h->v() + lo, h->s2() + lo, shadow, len, h->cfg.lr,
                           h->cfg.momentum, h->cfg.beta2, h->cfg.eps, h->cfg.wd, c1, c2, st, max_blocks);
    } else if (h->shards_equal) {
        launch_average_update(np, gp, h->w() + lo, h->v() + lo, shadow, len, h->cfg.lr, h->cfg.momentum, h->cfg.wd, st, max_blocks);
    } else {
        launch_weighted_update(np, gp, sh, h->w() + lo, h->v() + lo, shadow, len, h->cfg.lr, h->cfg.momentum, h->cfg.wd, st);
    }
    return EDL_OK;
}

int32_t edl_apply(edl_handle* h, int32_t p) {
    if (!h) { set_error("null handle"); return EDL_EINVAL; }
    // the gradient buffers are applied once: a second call, or one without gradients, would move the model by
    // whatever the buffers happen to hold
    if (!h->grads_pending) { set_error("no gradients pending: edl_apply follows one edl_gradients"); return EDL_EINVAL; }
    if ((size_t)p != h->shard_n.size()) {
        set_error("p=%d, but the pending gradients are of %zu shards", p, h->shard_n.size());
        return EDL_EINVAL;
    }
    h->grads_pending = false;
    // what the backward pass has not already updated (all of it, unless this is the second half of edl_step)
    apply_range(h, p, 0, h->applied_from, h->st);
    h->applied_from = h->g.P;
    HIP_TRY(hipGetLastError());
    h->prog.step += 1;
    h->prog.step_in_epoch += 1;
    if (h->prog.step_in_epoch == h->cfg.N / h->cfg.B) {
        h->prog.step_in_epoch = 0;
        h->prog.epoch += 1;
    }
    return EDL_OK;
}

int32_t edl_step(edl_handle* h, int32_t p, const int64_t* idx, const int64_t* off, float* out_loss) {
    if (h) h->early_p = p;      // the last backward pass may start the update
    const int rc = edl_gradients(h, p, idx, off, out_loss);
    if (h) h->early_p = 0;
    if (rc) {
        if (h && h->applied_from != h->g.P) {   // cannot happen after the arguments passed their checks
            set_error("the step failed after part of the update was launched");
            h->applied_from = h->g.P;
        }
        return rc;
    }
    return edl_apply(h, p);
}

int32_t edl_step_static_scratch(edl_handle* h, int32_t p, const int64_t* idx, const int64_t* off, float* out_loss) {
    if (!h) { set_error("null handle"); return EDL_EINVAL; }
    if (!h->static_fits) {
        set_error("the kernels of this job need %lld bytes of scratch; the static buffer holds %lld (use edl_step, whose "
                  "scratch is part of the caller's arena)", (long long)h->static_plan.scratch_hi, (long long)EDL_STATIC_SCRATCH_BYTES);
        return EDL_ENOMEM;
    }
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != h->device || dev < 0 || dev >= kMaxDevices || g_static_scratch[dev] == nullptr) {
        set_error("device %d is current, the job was created on device %d (or its static scratch was never set up)", dev, h->device);
        return EDL_EINVAL;
    }
    // nothing in the buffer has to start at zero: every partial result is written by the launch that precedes its
    // reader (the arena's piece is never cleared either)
    h->scratch_base = (char*)g_static_scratch[dev];
    std::swap(static_cast<Scratch&>(h->L), h->static_plan);
    const int rc = edl_step(h, p, idx, off, out_loss);
    std::swap(static_cast<Scratch&>(h->L), h->static_plan);
    h->scratch_base = nullptr;
    return rc;
}

int32_t edl_profile_parallelism(edl_handle* h, int32_t min_p, int32_t max_p, int32_t steps, edl_parallelism_point* out,
                                int32_t cap, int32_t* out_count) {
    if (!h || !out || !out_count) { set_error("null argument"); return EDL_EINVAL; }
    *out_count = 0;
    if (steps <= 0 || steps > 256) { set_error("steps=%d outside [1, 256]", steps); return EDL_EINVAL; }
    if (!h->data_x) { set_error("no data set bound"); return EDL_EINVAL; }
    std::vector<int32_t> ps;
    for (int32_t p = std::min(max_p, h->cfg.p_max); p >= std::max(min_p, 1); --p)
        if (h->cfg.B % p == 0 && h->cfg.B / p <= h->cfg.max_shard) ps.push_back(p);
    if (ps.empty()) { set_error("no parallelism in [%d, %d] fits B=%lld, p_max=%d, max_shard=%d", min_p, max_p, (long long)h->cfg.B, h->cfg.p_max, h->cfg.max_shard); return EDL_EINVAL; }
    if ((size_t)cap < ps.size()) { set_error("%zu entries needed", ps.size()); return EDL_ENOMEM; }
    // A step runs the shards of a mini-batch together, which no worker with a shard of its own does: what the workers
    // sustain is timed on passes of one shard each.  The step that moves the model runs as ever (where it would run
    // the same passes, those are the timed ones).
    std::vector<hipEvent_t> ev((size_t)steps * 4, nullptr);
    int rc = EDL_OK;
    for (hipEvent_t& e : ev)
        if (rc == EDL_OK && hipEventCreate(&e) != hipSuccess) { set_error("hipEventCreate failed"); rc = EDL_EHIP; }
    auto mark = [&](int t, int which) -> int {
        if (hipEventRecord(ev[(size_t)4 * t + which], h->st) == hipSuccess) return EDL_OK;
        set_error("hipEventRecord failed");
        return EDL_EHIP;
    };
    for (size_t i = 0; i < ps.size() && rc == EDL_OK; ++i) {
        const int32_t p = ps[i];
        const bool together = shards_per_pass(h, h->cfg.B / p, p) > 1;
        // per step: before the workers' passes, after them, before the update, after it
        for (int t = 0; t < steps && rc == EDL_OK; ++t) {
            rc = mark(t, 0);
            if (!rc) rc = gradient_passes(h, p, nullptr, nullptr, nullptr, together);
            if (!rc) rc = mark(t, 1);
            if (!rc && together) rc = edl_gradients(h, p, nullptr, nullptr, nullptr);
            if (!rc) rc = mark(t, 2);
            if (!rc) rc = edl_apply(h, p);
            if (!rc) rc = mark(t, 3);
        }
        if (rc) break;
        if (hipEventSynchronize(ev.back()) != hipSuccess) {
            set_error("timing events failed");
            rc = EDL_EHIP;
            break;
        }
        double grad_ms = 0.0, total_ms = 0.0;
        for (int t = 0; t < steps; ++t) {
            float grad = 0.f, update = 0.f;
            (void)hipEventElapsedTime(&grad, ev[(size_t)4 * t], ev[(size_t)4 * t + 1]);
            (void)hipEventElapsedTime(&update, ev[(size_t)4 * t + 2], ev[(size_t)4 * t + 3]);
            grad_ms += grad;
            total_ms += (double)grad + update;
        }
        edl_parallelism_point& o = out[i];
        o.p = p;
        o.shard = (int32_t)(h->cfg.B / p);
        o.ms_per_step = total_ms / steps;
        o.samples_per_s = (double)h->cfg.B / (o.ms_per_step * 1e-3);
        o.worker_samples_per_s = (double)h->cfg.B / (grad_ms / steps * 1e-3);
        o.efficiency = 0.0;
    }
    for (hipEvent_t e : ev)
        if (e) (void)hipEventDestroy(e);
    if (rc) return rc;
    double best = 0.0;
    for (size_t i = 0; i < ps.size(); ++i) best = std::max(best, out[i].worker_samples_per_s);
    for (size_t i = 0; i < ps.size(); ++i) out[i].efficiency = best > 0 ? out[i].worker_samples_per_s / best : 0.0;
    *out_count = (int32_t)ps.size();
    return EDL_OK;
}

// the arrays of the state image in its order (as the sources of a copy)
static ImageParts state_parts(const edl_handle* h) {
    ImageParts parts = {};
    int q = 0;
    auto add = [&](float* a, int64_t n) { parts.src[q] = a; parts.n[q] = n; ++q; };
    add(h->w(), h->g.P);
    add(h->v(), h->g.P);
    if (h->adam()) add(h->s2(), h->g.P);
    add(h->running(), h->g.R);
    return parts;
}

int32_t edl_snapshot(edl_handle* h, void* dev_dst, size_t cap, size_t* out_written) {
    if (!h || !dev_dst) { set_error("null argument"); return EDL_EINVAL; }
    const int64_t P = h->g.P, R = h->g.R;
    const size_t need = EDL_SNAPSHOT_HEADER_BYTES + 4 * (size_t)h->state_floats();
    if (cap < need) { set_error("snapshot needs %zu bytes, buffer has %zu", need, cap); return EDL_ENOMEM; }
    static_assert(kImageHeaderBytes == EDL_SNAPSHOT_HEADER_BYTES, "state image header");
    ImageHeader hdr = {};
    SnapshotHeader sh = {};
    sh.magic = EDL_SNAPSHOT_MAGIC; sh.version = 1; sh.model = (uint32_t)h->cfg.model; sh.dtype = (uint32_t)h->cfg.dtype;
    sh.seed = h->seed; sh.N = h->cfg.N; sh.B = h->cfg.B;
    sh.step = h->prog.step; sh.epoch = h->prog.epoch; sh.step_in_epoch = h->prog.step_in_epoch;
    sh.lr = h->cfg.lr; sh.momentum = h->cfg.momentum; sh.wd = h->cfg.wd; sh.P = P; sh.R = R;
    sh.optimizer = (uint32_t)h->cfg.optimizer;
    if (h->adam()) { sh.beta2 = h->cfg.beta2; sh.eps = h->cfg.eps; }
    memcpy(&hdr, &sh, sizeof(sh));
    ImageParts parts = state_parts(h);
    float* at = (float*)((char*)dev_dst + EDL_SNAPSHOT_HEADER_BYTES);
    for (int q = 0; q < kImageParts; ++q) { parts.dst[q] = at; at += parts.n[q]; }
    launch_image(parts, hdr, dev_dst, h->st);
    HIP_TRY(hipGetLastError());
    if (out_written) *out_written = need;
    return EDL_OK;
}

int32_t edl_restore(edl_handle* h, const void* dev_src, size_t len) {
    if (!h || !dev_src) { set_error("null argument"); return EDL_EINVAL; }
    const int64_t P = h->g.P, R = h->g.R;
    const size_t need = EDL_SNAPSHOT_HEADER_BYTES + 4 * (size_t)h->state_floats();
    if (len < need) { set_error("snapshot image of %zu bytes is shorter than %zu", len, need); return EDL_ERANGE; }
    // the header is read back through pinned memory (the loss staging, idle between calls)
    SnapshotHeader sh;
    static_assert(sizeof(SnapshotHeader) <= kStageBytes, "header fits the staging");
    HIP_TRY(hipMemcpyAsync(h->loss_host, dev_src, sizeof(sh), hipMemcpyDeviceToHost, h->st));
    HIP_TRY(hipStreamSynchronize(h->st));
    memcpy(&sh, h->loss_host, sizeof(sh));
    if (sh.magic != EDL_SNAPSHOT_MAGIC || sh.version != 1) { set_error("not a snapshot image"); return EDL_EINVAL; }
    if (sh.P != P || sh.R != R || (int32_t)sh.model != h->cfg.model) { set_error("snapshot is of another model (P=%lld, R=%lld)", (long long)sh.P, (long long)sh.R); return EDL_EINVAL; }
    if (sh.N != h->cfg.N || sh.B != h->cfg.B) { set_error("snapshot is of a job with N=%lld B=%lld", (long long)sh.N, (long long)sh.B); return EDL_EINVAL; }
    if ((int32_t)sh.optimizer != h->cfg.optimizer) { set_error("snapshot is of a job with optimizer %u", sh.optimizer); return EDL_EINVAL; }
    if ((int32_t)sh.dtype != h->cfg.dtype) { set_error("snapshot is of a job with dtype %u, this worker was created for %d", sh.dtype, h->cfg.dtype); return EDL_EINVAL; }
    if (!std::isfinite(sh.lr) || !std::isfinite(sh.momentum) || !std::isfinite(sh.wd)) { set_error("snapshot header holds non-finite hyper-parameters"); return EDL_EINVAL; }
    if (h->adam() && !(sh.momentum >= 0.f && sh.momentum < 1.f && sh.beta2 >= 0.f && sh.beta2 < 1.f && sh.eps >= 0.f)) {
        set_error("snapshot header holds Adam coefficients outside their range");
        return EDL_EINVAL;
    }
    ImageParts parts = state_parts(h);
    const float* at = (const float*)((const char*)dev_src + EDL_SNAPSHOT_HEADER_BYTES);
    for (int q = 0; q < kImageParts; ++q) { parts.dst[q] = (float*)parts.src[q]; parts.src[q] = at; at += parts.n[q]; }
    launch_image(parts, ImageHeader(), nullptr, h->st);
    HIP_TRY(hipGetLastError());
    // job meta-data travels with the model (section 4.2): the joiner takes over the seed, the progress and the
    // optimizer's coefficients, whatever it was created with
    h->seed = sh.seed;
    h->cfg.lr = sh.lr; h->cfg.momentum = sh.momentum; h->cfg.wd = sh.wd;
    if (h->adam()) { h->cfg.beta2 = sh.beta2; h->cfg.eps = sh.eps; }
    h->grads_pending = false;               // gradients of the model that was replaced are void
    h->prog.step = sh.step; h->prog.epoch = sh.epoch; h->prog.step_in_epoch = sh.step_in_epoch;
    h->perm_epoch = -1;
    h->weights_dirty = true;
    return EDL_OK;
}

int32_t edl_get_progress(const edl_handle* h, edl_progress* out) {
    if (!h || !out) { set_error("null argument"); return EDL_EINVAL; }
    *out = h->prog;
    return EDL_OK;
}

static int d2h(edl_handle* h, float* dst, const float* src, int64_t n) {
    if (!h || !dst) { set_error("null argument"); return EDL_EINVAL; }
    HIP_TRY(hipMemcpyAsync(dst, src, sizeof(float) * (size_t)n, hipMemcpyDeviceToHost, h->st));
    HIP_TRY(hipStreamSynchronize(h->st));
    return EDL_OK;
}

int32_t edl_get_params(edl_handle* h, float* host_dst) { return h ? d2h(h, host_dst, h->w(), h->g.P) : EDL_EINVAL; }
int32_t edl_get_momentum(edl_handle* h, float* host_dst) { return h ? d2h(h, host_dst, h->v(), h->g.P) : EDL_EINVAL; }
int32_t edl_get_second_moment(edl_handle* h, float* host_dst) {
    if (!h || !h->adam()) { set_error("not an Adam job"); return EDL_EINVAL; }
    return d2h(h, host_dst, h->s2(), h->g.P);
}
int32_t edl_get_running(edl_handle* h, float* host_dst) { return h ? d2h(h, host_dst, h->running(), h->g.R) : EDL_EINVAL; }
int32_t edl_get_grad(edl_handle* h, int32_t k, float* host_dst) {
    if (!h || k < 0 || k >= h->cfg.p_max) { set_error("gradient buffer %d outside [0,p_max)", k); return EDL_EINVAL; }
    return d2h(h, host_dst, h->grad_buf(k), h->g.P);
}
int32_t edl_get_losses(edl_handle* h, int32_t p, float* host_dst) {
    if (!h || p <= 0 || p > kMaxP) { set_error("bad p"); return EDL_EINVAL; }
    return d2h(h, host_dst, h->at<float>(h->L.losses), p);
}

int32_t edl_set_params(edl_handle* h, const float* host_src) {
    if (!h || !host_src) { set_error("null argument"); return EDL_EINVAL; }
    HIP_TRY(hipMemcpyAsync(h->w(), host_src, sizeof(float) * (size_t)h->g.P, hipMemcpyHostToDevice, h->st));
    HIP_TRY(hipStreamSynchronize(h->st));
    h->weights_dirty = true;
    return EDL_OK;
}

// ---------------------------------------------------------------- debugging hooks
static inline float host_bf16_to_f32(uint16_t v) { uint32_t u = (uint32_t)v << 16; float f; memcpy(&f, &u, 4); return f; }
static inline uint16_t host_f32_to_bf16(float f) {
    uint32_t u; memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

int32_t edl_debug_tensor_count(const edl_handle* h, int32_t* out) {
    if (!h || !out) { set_error("null argument"); return EDL_EINVAL; }
    *out = (int32_t)h->g.tensors.size();
    return EDL_OK;
}

int32_t edl_debug_tensor_shape(const edl_handle* h, int32_t t, int32_t* H, int32_t* W, int32_t* C, int32_t* alias_of) {
    if (!h || t < 0 || (size_t)t >= h->g.tensors.size()) { set_error("tensor %d out of range", t); return EDL_ERANGE; }
    const Tensor& x = h->g.tensors[(size_t)t];
    if (H) *H = x.H;
    if (W) *W = x.W;
    if (C) *C = x.C;
    if (alias_of) *alias_of = x.alias_of;
    return EDL_OK;
}

// one shard of n samples, computed as in a step of such shards
static ShardSet one_shard(const edl_handle* h, int n, int k) {
    ShardSet S = {};
    S.p = 1;
    S.off[1] = n;
    S.plan_equal(n, h->cfg.B % n == 0 && h->cfg.B / n <= h->cfg.p_max ? shards_per_pass(h, n, (int)(h->cfg.B / n)) : 1);
    S.k[0] = k;
    return S;
}

static int debug_prepare(edl_handle* h, int32_t n) {
    if (!h) { set_error("null handle"); return EDL_EINVAL; }
    if (n <= 0 || n > h->cfg.max_shard || n > h->cfg.B) { set_error("n=%d outside [1, max_shard]", n); return EDL_EINVAL; }
    if (h->weights_dirty) { refresh_weight_copies(h); h->weights_dirty = false; }
    transpose_weights(h, h->st);
    return EDL_OK;
}

int32_t edl_debug_forward(edl_handle* h, const int64_t* idx, int32_t n) {
    int rc = debug_prepare(h, n);
    if (rc) return rc;
    if (!idx || !h->data_x) { set_error("idx and a bound data set are needed"); return EDL_EINVAL; }
    for (int i = 0; i < n; ++i)
        if (idx[i] < 0 || idx[i] >= h->cfg.N) { set_error("idx[%d] outside [0,N)", i); return EDL_ERANGE; }
    HIP_TRY(hipStreamSynchronize(h->st));
    memcpy(h->idx_host[0], idx, sizeof(int64_t) * (size_t)n);
    HIP_TRY(hipMemcpyAsync(h->at<int64_t>(h->L.idx), h->idx_host[0], sizeof(int64_t) * (size_t)n, hipMemcpyHostToDevice, h->st));
    forward_pass(h, one_shard(h, n, 0), h->at<int64_t>(h->L.idx), h->at<float>(h->L.losses), false);
    HIP_TRY(hipStreamSynchronize(h->st));
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

int32_t edl_debug_backward(edl_handle* h, int32_t n, int32_t k) {
    int rc = debug_prepare(h, n);
    if (rc) return rc;
    if (k < 0 || k >= h->cfg.p_max) { set_error("gradient buffer %d outside [0,p_max)", k); return EDL_EINVAL; }
    const Graph& g = h->g;
    launch_softmax_ce(h->cfg.dtype, (const float*)h->act(g.logits), h->at<int32_t>(h->L.labels), h->grad(g.logits),
                      h->sc<float>(h->L.row_loss), h->at<float>(h->L.losses), one_shard(h, n, 0), g.classes, h->st);
    backward_pass(h, one_shard(h, n, k), 0, (size_t)-1, 0, nullptr, false, true);
    HIP_TRY(hipStreamSynchronize(h->st));
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

int32_t edl_debug_op_count(const edl_handle* h, int32_t* out) {
    if (!h || !out) { set_error("null argument"); return EDL_EINVAL; }
    *out = (int32_t)h->g.ops.size();
    return EDL_OK;
}

int32_t edl_debug_forward_op(edl_handle* h, int32_t op, int32_t n) {
    int rc = debug_prepare(h, n);
    if (rc) return rc;
    if (op < 0 || (size_t)op >= h->g.ops.size()) { set_error("layer %d out of range", op); return EDL_ERANGE; }
    forward_pass(h, one_shard(h, n, 0), nullptr, h->at<float>(h->L.losses), false, (size_t)op, (size_t)op + 1);
    HIP_TRY(hipStreamSynchronize(h->st));
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

int32_t edl_debug_forward_range(edl_handle* h, int32_t op_lo, int32_t op_hi, int32_t n) {
    int rc = debug_prepare(h, n);
    if (rc) return rc;
    if (op_lo < 0 || op_hi < op_lo || (size_t)op_hi > h->g.ops.size()) { set_error("layers [%d, %d) out of range", op_lo, op_hi); return EDL_ERANGE; }
    forward_pass(h, one_shard(h, n, 0), nullptr, h->at<float>(h->L.losses), false, (size_t)op_lo, (size_t)op_hi);
    HIP_TRY(hipStreamSynchronize(h->st));
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

int32_t edl_debug_backward_op(edl_handle* h, int32_t op, int32_t n, int32_t k) {
    int rc = debug_prepare(h, n);
    if (rc) return rc;
    if (op < 0 || (size_t)op >= h->g.ops.size()) { set_error("layer %d out of range", op); return EDL_ERANGE; }
    if (k < 0 || k >= h->cfg.p_max) { set_error("gradient buffer %d outside [0,p_max)", k); return EDL_EINVAL; }
    backward_pass(h, one_shard(h, n, k), (size_t)op, (size_t)op + 1, 0, nullptr, false, true);
    HIP_TRY(hipStreamSynchronize(h->st));
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

int32_t edl_debug_backward_range(edl_handle* h, int32_t op_lo, int32_t op_hi, int32_t n, int32_t k) {
    return edl_debug_backward_range_from(h, op_lo, op_hi, n, k, nullptr, 0);
}

int32_t edl_debug_backward_range_from(edl_handle* h, int32_t op_lo, int32_t op_hi, int32_t n, int32_t k,
                                      const int32_t* held, int32_t n_held) {
    int rc = debug_prepare(h, n);
    if (rc) return rc;
    if (op_lo < 0 || op_hi < op_lo || (size_t)op_hi > h->g.ops.size()) { set_error("layers [%d, %d) out of range", op_lo, op_hi); return EDL_ERANGE; }
    if (k < 0 || k >= h->cfg.p_max) { set_error("gradient buffer %d outside [0,p_max)", k); return EDL_EINVAL; }
    if (n_held < 0 || (n_held > 0 && !held)) { set_error("bad list of held tensors"); return EDL_EINVAL; }
    std::vector<int> hv;
    for (int32_t i = 0; i < n_held; ++i) {
        if (held[i] <= 0 || (size_t)held[i] >= h->g.tensors.size()) { set_error("held tensor %d out of range", held[i]); return EDL_ERANGE; }
        hv.push_back(held[i]);
    }
    backward_pass(h, one_shard(h, n, k), (size_t)op_lo, (size_t)op_hi, 0, &hv, false, true);
    HIP_TRY(hipStreamSynchronize(h->st));
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}


int32_t edl_debug_set_labels(edl_handle* h, const int32_t* labels, int32_t n) {
    if (!h || !labels || n <= 0 || n > h->cfg.max_shard) { set_error("bad argument"); return EDL_EINVAL; }
    HIP_TRY(hipMemcpyAsync(h->at<int32_t>(h->L.labels), labels, sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice, h->st));
    HIP_TRY(hipStreamSynchronize(h->st));
    return EDL_OK;
}

static int debug_tensor_ptr(edl_handle* h, int32_t t, int32_t which, int32_t n, char** ptr, int64_t* elems, bool* is_f32) {
    if (!h) { set_error("null handle"); return EDL_EINVAL; }
    if (t < 0 || (size_t)t >= h->g.tensors.size()) { set_error("tensor %d out of range", t); return EDL_ERANGE; }
    if (n <= 0 || n > h->cfg.max_shard) { set_error("n=%d outside [1, max_shard]", n); return EDL_EINVAL; }
    const int s = storage_of(h->g, t);
    if (which == 1 && s == 0) { set_error("the input image has no gradient buffer"); return EDL_EINVAL; }
    *ptr = which == 0 ? (char*)h->act(t) : (char*)h->grad(t);
    *elems = h->g.tensors[(size_t)t].elems() * n;
    if (s == 0 && stored_apart(h->g, h->L.in)) { set_error("the input batch is stored padded; it is set by edl_debug_forward only"); return EDL_EINVAL; }
    *is_f32 = h->cfg.dtype == EDL_DTYPE_F32 || (which == 0 && h->g.tensors[(size_t)s].fp32);
    return EDL_OK;
}

int32_t edl_debug_get_tensor(edl_handle* h, int32_t t, int32_t which, int32_t n, float* host_dst) {
    char* ptr; int64_t elems; bool f32;
    const int rc = debug_tensor_ptr(h, t, which, n, &ptr, &elems, &f32);
    if (rc) return rc;
    if (!host_dst) { set_error("null argument"); return EDL_EINVAL; }
    if (f32) {
        HIP_TRY(hipMemcpyAsync(host_dst, ptr, 4 * (size_t)elems, hipMemcpyDeviceToHost, h->st));
        HIP_TRY(hipStreamSynchronize(h->st));
    } else {
        std::vector<uint16_t> tmp((size_t)elems);
        HIP_TRY(hipMemcpyAsync(tmp.data(), ptr, 2 * (size_t)elems, hipMemcpyDeviceToHost, h->st));
        HIP_TRY(hipStreamSynchronize(h->st));
        for (int64_t i = 0; i < elems; ++i) host_dst[i] = host_bf16_to_f32(tmp[(size_t)i]);
    }
    return EDL_OK;
}

int32_t edl_debug_set_tensor(edl_handle* h, int32_t t, int32_t which, int32_t n, const float* host_src) {
    char* ptr; int64_t elems; bool f32;
    const int rc = debug_tensor_ptr(h, t, which, n, &ptr, &elems, &f32);
    if (rc) return rc;
    if (!host_src) { set_error("null argument"); return EDL_EINVAL; }
    if (f32) {
        HIP_TRY(hipMemcpyAsync(ptr, host_src, 4 * (size_t)elems, hipMemcpyHostToDevice, h->st));
        HIP_TRY(hipStreamSynchronize(h->st));
    } else {
        std::vector<uint16_t> tmp((size_t)elems);
        for (int64_t i = 0; i < elems; ++i) tmp[(size_t)i] = host_f32_to_bf16(host_src[i]);
        HIP_TRY(hipMemcpyAsync(ptr, tmp.data(), 2 * (size_t)elems, hipMemcpyHostToDevice, h->st));
        if (which == 0 && h->sign(t) != nullptr) launch_signs(ptr, h->sign(t), elems, h->st);    // kept beside the activation
        HIP_TRY(hipStreamSynchronize(h->st));
    }
    return EDL_OK;
}

int32_t edl_set_momentum(edl_handle* h, const float* host_src) {
    if (!h || !host_src) { set_error("null argument"); return EDL_EINVAL; }
    HIP_TRY(hipMemcpyAsync(h->v(), host_src, sizeof(float) * (size_t)h->g.P, hipMemcpyHostToDevice, h->st));
    HIP_TRY(hipStreamSynchronize(h->st));
    return EDL_OK;
}

int32_t edl_set_second_moment(edl_handle* h, const float* host_src) {
    if (!h || !host_src) { set_error("null argument"); return EDL_EINVAL; }
    if (!h->adam()) { set_error("not an Adam job"); return EDL_EINVAL; }
    HIP_TRY(hipMemcpyAsync(h->s2(), host_src, sizeof(float) * (size_t)h->g.P, hipMemcpyHostToDevice, h->st));
    HIP_TRY(hipStreamSynchronize(h->st));
    return EDL_OK;
}

int32_t edl_shutdown(edl_handle* h) {
    if (!h) { set_error("null handle"); return EDL_EINVAL; }
    destroy_handle(h);
    return EDL_OK;
}

int32_t edl_profile(int32_t enable) {
    prof_enable(enable != 0);
    return EDL_OK;
}

int32_t edl_profile_report(char* buf, size_t cap, size_t* out_needed) {
    const long n = prof_report(buf, cap);
    if (n < 0) { set_error("reading the timing events failed"); return EDL_EHIP; }
    if (out_needed) *out_needed = (size_t)n + 1;
    if ((size_t)n + 1 > cap) { set_error("report needs %ld bytes", n + 1); return EDL_ENOMEM; }
    return EDL_OK;
}

int32_t edl_average_update(int32_t p, const float* const* dev_grads, float* dev_w, float* dev_v, uint16_t* dev_w16,
                           int64_t P, float lr, float momentum, float wd, void* hip_stream) {
    if (!dev_grads || !dev_w || !dev_v) { set_error("null argument"); return EDL_EINVAL; }
    if (p <= 0 || p > kMaxP) { set_error("p=%d outside [1,%d]", p, kMaxP); return EDL_EINVAL; }
    if (P < 0) { set_error("negative P"); return EDL_EINVAL; }
    if (P == 0) return EDL_OK;
    GradPtrs gp = {};
    uintptr_t bits = (uintptr_t)dev_w | (uintptr_t)dev_v | (uintptr_t)dev_w16;
    for (int k = 0; k < p; ++k) {
        if (!dev_grads[k]) { set_error("gradient pointer %d is NULL", k); return EDL_EINVAL; }
        gp.g[k] = dev_grads[k];
        bits |= (uintptr_t)dev_grads[k];
    }
    if (bits & 15) { set_error("pointers must be 16-byte aligned"); return EDL_EINVAL; }
    launch_average_update(p, gp, dev_w, dev_v, dev_w16, P, lr, momentum, wd, (hipStream_t)hip_stream);
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

int32_t edl_adam_update(int32_t p, const float* const* dev_grads, const float* shares, float* dev_w, float* dev_m,
                        float* dev_s, uint16_t* dev_w16, int64_t P, float lr, float beta1, float beta2, float eps,
                        float wd, int64_t t, void* hip_stream) {
    if (!dev_grads || !dev_w || !dev_m || !dev_s) { set_error("null argument"); return EDL_EINVAL; }
    if (p <= 0 || p > kMaxP) { set_error("p=%d outside [1,%d]", p, kMaxP); return EDL_EINVAL; }
    if (P < 0 || t < 1) { set_error("negative P or t < 1"); return EDL_EINVAL; }
    if (!(beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f && eps >= 0.f)) { set_error("betas must lie in [0,1), eps >= 0"); return EDL_EINVAL; }
    if (P == 0) return EDL_OK;
    GradPtrs gp = {};
    ShardShares sh = {};
    uintptr_t bits = (uintptr_t)dev_w | (uintptr_t)dev_m | (uintptr_t)dev_s | (uintptr_t)dev_w16;
    for (int k = 0; k < p; ++k) {
        if (!dev_grads[k]) { set_error("gradient pointer %d is NULL", k); return EDL_EINVAL; }
        gp.g[k] = dev_grads[k];
        bits |= (uintptr_t)dev_grads[k];
        if (shares) sh.share[k] = shares[k];
    }
    if (bits & 15) { set_error("pointers must be 16-byte aligned"); return EDL_EINVAL; }
    float c1, c2;
    adam_corrections(beta1, beta2, t, &c1, &c2);
    launch_adam_update(p, gp, shares ? &sh : nullptr, dev_w, dev_m, dev_s, dev_w16, P, lr, beta1, beta2, eps, wd, c1, c2,
                       (hipStream_t)hip_stream);
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

int32_t edl_mfma_rate(int32_t dtype, int32_t blocks, int32_t iters, float* dev_sink, void* hip_stream, double* out_flops) {
    if ((dtype != EDL_DTYPE_F32 && dtype != EDL_DTYPE_BF16) || blocks <= 0 || blocks > (1 << 20) || iters <= 0 || !dev_sink) {
        set_error("bad argument");
        return EDL_EINVAL;
    }
    const double flops = launch_mfma_rate(dtype, blocks, iters, dev_sink, (hipStream_t)hip_stream);
    if (out_flops) *out_flops = flops;
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

int32_t edl_copy(void* dev_dst, const void* dev_src, size_t bytes, void* hip_stream) {
    if (!dev_dst || !dev_src) { set_error("null argument"); return EDL_EINVAL; }
    launch_copy(dev_dst, dev_src, bytes, (hipStream_t)hip_stream);
    HIP_TRY(hipGetLastError());
    return EDL_OK;
}

}  // extern "C"

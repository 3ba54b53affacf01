// Host-callable launchers of the HIP kernels.  `dtype` is EDL_DTYPE_*: the
// element type of activation tensors and of the weight copies the matrix
// cores read.  Every launcher only queues work on `st`.
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

namespace edl {

constexpr int kMaxP = 16;           // gradient buffers one update launch can average
constexpr int kRedRowBlocks = 1024;   // row blocks a separate column reduction aims at, at most (plus one per shard)

struct GradPtrs { const float* g[kMaxP]; };
struct ShardShares { float share[kMaxP]; };   // a shard's part of the mini-batch

// The workers' shards that one pass runs together: their samples lie one after another in the activation buffers
// (none is empty).  A layer is then one launch for all of them; what belongs to a worker alone - batch statistics,
// the gradients of the parameters, the loss - is formed per shard.
struct ShardSet {
    int p;                    // shards in the pass
    int off[kMaxP + 1];       // first sample of each, off[p] = samples of the pass
    int k[kMaxP];             // the worker: which gradient buffer, which loss
    // What tiles and reduction cuts are chosen for: samples, shards and the largest and smallest shard of the pass, or of
    // the pass this one stands for (a step's last pass may hold fewer shards than the others; a debugging hook runs one
    // shard of such a pass; the static scratch buffer may take a pass in parts).  Sums are then formed in the same
    // order for a shard whichever part it is in.
    int plan, plan_p, plan_largest, plan_smallest;
    void plan_itself() { plan = samples(); plan_p = p; plan_largest = largest(); plan_smallest = smallest(); }
    void plan_equal(int n, int shards) { plan = n * shards; plan_p = shards; plan_largest = plan_smallest = n; }
    int samples() const { return off[p]; }
    int largest() const { int m = 0; for (int s = 0; s < p; ++s) if (off[s + 1] - off[s] > m) m = off[s + 1] - off[s]; return m; }
    int smallest() const { int m = off[1]; for (int s = 1; s < p; ++s) if (off[s + 1] - off[s] < m) m = off[s + 1] - off[s]; return m; }
};

// Rows of a [rows][channels] matrix cut into blocks that stay within a shard: how a launch's partial column sums
// are laid out, sums[kind * channels + channel][block].  p == 0: there are none.
struct RowCut {
    int p = 0, rows_per_block = 0;
    int row0[kMaxP + 1] = {};     // first row of each shard
    int blk0[kMaxP + 1] = {};     // first block of each shard, blk0[p] = blocks in all
    int k[kMaxP] = {};            // the shard's worker
    int most = 0;                 // blocks of the largest shard of the plan
    bool stored = false;          // column sums: each shard is one block, and its sums are already where they go (DgradMask::dbias)
    bool block_per_shard() const { return p > 0 && blk0[p] == p; }
};
inline RowCut cut_rows(const ShardSet& S, int rows_per_sample, int rows_per_block) {
    RowCut c;
    c.p = S.p;
    c.rows_per_block = rows_per_block;
    for (int s = 0; s < S.p; ++s) {
        c.row0[s + 1] = S.off[s + 1] * rows_per_sample;
        c.blk0[s + 1] = c.blk0[s] + (c.row0[s + 1] - c.row0[s] + rows_per_block - 1) / rows_per_block;
        c.k[s] = S.k[s];
    }
    c.most = (S.plan_largest * rows_per_sample + rows_per_block - 1) / rows_per_block;
    return c;
}

// The workers' gradients of one parameter tensor: worker k's starts at g + k * stride.
struct GradDst { float* g; int64_t stride; };

// ---- aggregation + update, copies ----------------------------------------
// max_blocks > 0 holds the launch to that many workgroups (a pass that runs in the background of other work).
void launch_average_update(int p, const GradPtrs& grads, float* w, float* v, uint16_t* w16, int64_t P,
                           float lr, float momentum, float wd, hipStream_t st, int max_blocks = 0);
// aggregate = sum_k shares[k] * grads[k] (shards of unequal size)
void launch_weighted_update(int np, const GradPtrs& grads, const ShardShares& shares, float* w, float* v, uint16_t* w16,
                            int64_t P, float lr, float momentum, float wd, hipStream_t st);
// Adam on the aggregated gradient.  shares == nullptr: the mean of the p gradients; otherwise sum_k shares->share[k]*G_k.
// c1 = 1/(1-beta1^t), c2 = 1/(1-beta2^t).
void launch_adam_update(int p, const GradPtrs& grads, const ShardShares* shares, float* w, float* m, float* s, uint16_t* w16,
                        int64_t P, float lr, float beta1, float beta2, float eps, float wd, float c1, float c2, hipStream_t st,
                        int max_blocks = 0);
void launch_copy(void* dst, const void* src, size_t bytes, hipStream_t st);
// The state image: arrays of floats (n = 0: none) copied in one launch, its header written from the arguments
constexpr int kImageParts = 4, kImageHeaderBytes = 256;
struct ImageHeader { uint32_t words[kImageHeaderBytes / 4]; };
struct ImageParts { float* dst[kImageParts]; const float* src[kImageParts]; int64_t n[kImageParts]; int block0[kImageParts]; };
void launch_image(const ImageParts& parts, const ImageHeader& hdr, void* header_dst /* null: none */, hipStream_t st);
void launch_fill_f32(float* dst, float value, int64_t n, hipStream_t st);
// dst[c][r][s][k] = cast(src[k][r][s][c]) (weights for the input-gradient contraction) for every
// layer of a model in one launch, from a table in device memory
struct TransposeEntry {
    int64_t src_off;     // floats from the start of the parameter vector
    int64_t dst_off;     // bytes from the start of the arena
    int K, RS, C;
    int tile_start;      // index of the layer's first 32x32 tile among all layers' tiles
};
void launch_weight_transpose_all(int dtype, const float* w, void* arena, const TransposeEntry* dev_table, int entries,
                                 int total_tiles, double bytes, hipStream_t st);
// bf16 layers with K and C multiples of 8, from the bf16 copy of the weights; tile_start counts 64x64 tiles
void launch_weight_transpose_bf16(const uint16_t* w16, void* arena, const TransposeEntry* dev_table, int entries,
                                  int total_tiles, double bytes, hipStream_t st);
// dst = cast(src) for float32 -> bf16 (weight copy after restore / set_params)
void launch_cast_bf16(const float* src, uint16_t* dst, int64_t n, hipStream_t st);

// ---- input --------------------------------------------------------------
void launch_gather(int dtype, const float* data_x, const int32_t* data_y, const int64_t* idx, int n,
                   int64_t sample_elems, void* out_x, int32_t* out_y, hipStream_t st);

// How the input images are stored: f x f blocks of pixels as one pixel of C channels, (row in the block, column in the
// block, channel) one after another and zeros up to C; `lead` rows and columns of zeros stand before the image's first.
// f = 1: pixels padded to one vector, or as they are.
struct InputFold { int f = 1, lead = 0, H = 0, W = 0, C = 0; };
// images of H x W x C written that way (C less than a vector; f > 1: C = 3)
void launch_gather_pad(int dtype, const float* data_x, const int32_t* data_y, const int64_t* idx, int n, int H, int W, int C,
                       const InputFold& in, void* out_x, int32_t* out_y, hipStream_t st);
// float32 weights [K][R][S][C] of the convolution that reads them as [K][R/f][S/f][in.C] dtype, zero padded; and the way
// back for their gradient (one per shard: src holds the shards' one after another)
void launch_pad_weights(int dtype, const float* src, void* dst, int K, int R, int S, int C, const InputFold& in, hipStream_t st);
void launch_unpad_weights(const float* src, GradDst dst, const ShardSet& set, int K, int R, int S, int C, const InputFold& in, hipStream_t st);

// ---- implicit-GEMM convolution --------------------------------------------
enum ConvMode { CONV_FWD = 0, CONV_DGRAD = 1, CONV_WGRAD = 2 };

struct ConvGeom {
    int N, H, W, C;          // input images
    int K, R, S, stride, pad, Ho, Wo;
};

// Partial column sums: a buffer of `floats` floats (conv_sums_floats / norm_sums_floats say how many are needed).
struct SumsBuf { float* buf; size_t floats; };

// y = conv(x, w) (+bias) (ReLU) over the pass's samples; y is float32 if out_fp32 else dtype.
// stats.buf (may be null): if the launch can, it also leaves there the column sums of y and y*y per block of rows
// and returns how they are cut; p == 0 if it left none.
RowCut launch_conv_fwd(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* w, const float* bias, bool relu,
                       bool out_fp32, void* y, float* scratch, size_t scratch_bytes, SumsBuf stats, hipStream_t st);
// Whether the first layer of a net can take its rows from the data set itself (launch_small_fc_fwd with SmallInput)
bool conv_fwd_gathers(int dtype, const ConvGeom& g, const ShardSet& S, const void* data, const void* x, const void* w);
// The most samples (65535 at most) of which a launch, forward and with dgrad also of the input gradient, keeps to the
// vector kernel: its multiply-shift divisions are exact up to some number of pixels (g.N is ignored).
int conv_vector_samples(const ConvGeom& g, bool dgrad);
// floats the sums of this layer's forward and input-gradient epilogues can take over g.N samples of p shards
size_t conv_sums_floats(const ConvGeom& g, int p);
// What the layer that produced the convolution's input wants from the gradient dx when it ends in a ReLU:
// dx * (act > 0), and per-channel sums of that over the rows (plain, and times (xin - mean) * rstd if xin is
// given: a batch norm's backward sums).
struct DgradMask {
    const void* act;          // the producer's output (= this convolution's input), dtype elements
    const unsigned char* sign;    // (act > 0), one bit per element, eight channels to a byte; null if not kept
    const void* xin;          // the producing batch norm's input, or null
    const float* mean_rstd;   // with xin: mean[C], rstd[C] of each shard
    SumsBuf sums;
    GradDst dbias;            // without xin: the workers' bias gradients, which are these sums; a launch whose row blocks are whole
                              // shards may store them there itself (RowCut::stored).  g may be null
};
struct BothGradients { const void* x; GradDst dw; };
// dx (+)= conv^T(dy, wT); wT is the [C][R][S][K] copy.  mask (may be null): if the launch can (stride 1, one
// launch over all pixels, writing), dx is stored already masked and the sums are left in mask->sums; returns
// how they are cut (what the producer's backward takes), else p == 0 and dx is the plain gradient.
// acc_src (stride 1 with accumulate only; may be null): the gradient that is added to is read from this tensor of
// dx's shape instead of from dx itself (dx is then written, not read).
// w_rows (only where conv_dgrad_reads_weights): wT is not a copy but the weights (bf16: their copy) as they lie, [K][C].
RowCut launch_conv_dgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* dy, const void* wT, bool accumulate, void* dx,
                         float* scratch, size_t scratch_bytes, const DgradMask* mask, hipStream_t st,
                         const void* acc_src = nullptr, bool w_rows = false, const BothGradients* wgrad = nullptr);
// whether that launch can leave the layer's weight gradient too (BothGradients: its input, where the gradient goes)
bool conv_gradients_together(int dtype, const ConvGeom& g, const ShardSet& S, bool w_rows);
// whether the input gradient of a layer whose weights start at element w_off reads them where they lie, in passes of up to
// g.N samples
bool conv_dgrad_reads_weights(int dtype, const ConvGeom& g, int64_t w_off);
// float32 scratch the forward / dgrad launches of passes of up to `samples` samples may use to cut a long reduction of a
// small problem, where cuts are planned for passes of up to g.N
size_t conv_splitk_scratch_bytes(int dtype, const ConvGeom& g, int samples);
// dw = x^T * dy of every shard, float32 [K][R][S][C]; scratch holds split partial sums
void launch_conv_wgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* dy, GradDst dw, float* scratch,
                       size_t scratch_bytes, hipStream_t st);
// what any p shards need of which the largest has up to g.N samples; and what those of one pass do
size_t conv_wgrad_scratch_bytes(int dtype, const ConvGeom& g, int p);
size_t conv_wgrad_needs(int dtype, const ConvGeom& g, const ShardSet& S);
// pixels that the weight gradient of one shard of g.N samples sums in one chain, at most
int conv_wgrad_chain(int dtype, const ConvGeom& g);

// ---- batch norm, bias / ReLU backward --------------------------------------
// floats the column reductions below take as scratch over the given rows of p shards
size_t norm_sums_floats(int dtype, int64_t M, int C, int p);
// save: mean[C], rstd[C] of each shard; running ([2C] or null) follows the first shard; sums.p > 0: partial already
// holds the sums, cut that way; hw: rows per sample.  sign (bf16 with C a multiple of 8, else null): receives the bits
// (y > 0), a sixteenth of y's bytes, for the backward passes that need no more of it
void launch_bn_forward(int dtype, const void* x, const void* res, void* y, const float* gamma, const float* beta,
                       float* save, float* running, const ShardSet& S, int hw, int C, bool relu, unsigned char* sign, float* partial,
                       const RowCut& sums, hipStream_t st);
// sign[i] = bits (act[8i + e] > 0) of n elements (a multiple of 8)
void launch_signs(const void* act_bf16, unsigned char* sign, int64_t n, hipStream_t st);
// sums.p > 0: partial already holds the two backward sums (left there by the dgrad that produced dy, which is then
// also masked already); coef: 2C floats per shard: means over the shard of dy and of dy * xhat.  dx null: these and the
// gradients of the parameters only
void launch_bn_backward(int dtype, const void* x, const void* y, const void* dy, void* dx, void* dres,
                        bool dres_accumulate, const float* gamma, const float* save, GradDst dgamma, GradDst dbeta,
                        const ShardSet& S, int hw, int C, bool relu, float* partial, float* coef, const RowCut& sums,
                        hipStream_t st);
// dx alone, from a gradient that is masked already and its coef (bf16, C a multiple of 8)
void launch_bn_backward_apply(const void* x, const void* dy, void* dx, const float* gamma, const float* save, const float* coef,
                              const ShardSet& S, int hw, int C, hipStream_t st);
// dy <- dy * (y > 0) in place if relu; dbias[c] = sum_rows dy of each shard (if dbias.g).
// sums.p > 0: dy is masked already and partial holds its column sums.
void launch_bias_relu_backward(int dtype, const void* y, void* dy, GradDst dbias, const ShardSet& S, int hw, int C, bool relu,
                               float* partial, const RowCut& sums, hipStream_t st);
// how launch_bias_relu_backward sums C channels that are no whole vectors: rows of a block, channels side by side in one, and
// whether its lanes are added in float64
int bias_sums_rows(int dtype, const ShardSet& S, int hw, int C, int* side_by_side, bool* in_double);
// The same bias gradient of a ReLU layer whose output only a max pool reads, from the pool's output and its gradient: the pool
// hands each of its gradients to one element, whose activation is the pooled value, so that the sum over the layer's masked
// gradient is that of dpooled * (pooled > 0), of fewer elements.  hw: pooled pixels per sample.
void launch_pooled_bias_backward(int dtype, const void* pooled, const void* dpooled, GradDst dbias, const ShardSet& S, int hw, int C,
                                 float* partial, hipStream_t st);

// ---- pooling --------------------------------------------------------------
void launch_maxpool_forward(int dtype, const void* x, void* y, uint8_t* arg, int N, int H, int W, int C, int k,
                            int stride, int pad, int Ho, int Wo, hipStream_t st);
// mask (may be null), relu_pooled: if the pooled tensor is the output of a ReLU layer with no other reader, that layer's part of
// DgradMask and the pool's output; the gradient is then stored multiplied by (act > 0) where the kernel taken supports it.
// Returns whether it was.  sums: how the column sums left in mask->sums are cut, if the producer is a batch norm and the kernel
// leaves them (else p == 0).
bool launch_maxpool_backward(int dtype, const void* dy, const uint8_t* arg, void* dx, bool accumulate, const ShardSet& S, int H,
                             int W, int C, int k, int stride, int pad, int Ho, int Wo, const DgradMask* mask, const void* relu_pooled, RowCut* sums,
                             hipStream_t st);
void launch_gavgpool_forward(int dtype, const void* x, void* y, int N, int HW, int C, hipStream_t st);
void launch_gavgpool_backward(int dtype, const void* dy, void* dx, bool accumulate, int N, int HW, int C,
                              hipStream_t st);

// ---- loss -------------------------------------------------------------------
// logits float32 [samples][C]; dlogits in dtype (of the mean over the sample's shard); loss_out[worker] = mean over
// the worker's shard
void launch_softmax_ce(int dtype, const float* logits, const int32_t* labels, void* dlogits, float* row_loss,
                       float* loss_out, const ShardSet& S, int C, hipStream_t st);

// register-resident MFMA loop (attainable matrix rate); returns the flops the launch issues
double launch_mfma_rate(int dtype, int blocks, int iters, float* sink, hipStream_t st);

}  // namespace edl

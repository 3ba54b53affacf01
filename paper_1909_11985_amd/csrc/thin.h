// Small fully connected layers (k_thin.hip), behind launch_conv_fwd, launch_conv_dgrad and launch_conv_wgrad.  Input gradients
// read the weights as they lie, [K][C] (conv_dgrad_reads_weights).
#pragma once
#include "kernels.h"

namespace edl {

struct SmallWgrad { const float* x; GradDst dw; };

// few, ragged outputs: the forward contraction of a pass planned for `samples` (small: if not, launch_small_fc_fwd takes it), the
// input gradient of passes of up to g.N, the weight gradient of a pass planned as S is
bool thin_fwd_takes(int dtype, const ConvGeom& g, int samples, bool small);
bool thin_dgrad_takes(int dtype, const ConvGeom& g);
bool thin_wgrad_takes(int dtype, const ConvGeom& g, const ShardSet& S);
void launch_thin_fwd(int dtype, const ConvGeom& g, const void* x, const void* w, const float* bias, bool relu, bool out_fp32, void* y, hipStream_t st);
// old (may be null, may be dx): the gradient that is added to.  Returns how the sums of mask are cut, p == 0 if it left none.
RowCut launch_thin_dgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* dy, const void* w, const void* old, void* dx,
                         const DgradMask* mask, hipStream_t st);
void launch_thin_wgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* dy, GradDst dw, hipStream_t st);
// float32, few tiles of 32x32 outputs: the forward or input-gradient contraction of K products for N outputs, over a pass
// planned for `samples`
bool small_fc_takes(int dtype, const ConvGeom& g, int K, int N, int samples);
// in (may be null): x is not there yet, its rows are samples in->idx[] of the data set (up to kSmallGather of them), and the launch leaves
// them and their labels
constexpr int kSmallGather = 256;
struct SmallInput { const float* data; const int32_t* data_y; const int64_t* idx; float* out; int32_t* labels; };
void launch_small_fc_fwd(const ConvGeom& g, const ShardSet& S, const float* x, const float* w, const float* bias, bool relu, float* y, const SmallInput* in,
                         hipStream_t st);
// its weight gradient, where a shard's rows are few
bool small_wgrad_takes(int dtype, const ConvGeom& g, const ShardSet& S);
void launch_small_wgrad(const ConvGeom& g, const ShardSet& S, const float* x, const float* dy, GradDst dw, hipStream_t st);
// wgrad (may be null): the same launch leaves the layer's weight gradient as well
RowCut launch_small_fc_dgrad(const ConvGeom& g, const ShardSet& S, const float* dy, const float* w, const float* old, float* dx,
                             const DgradMask* mask, const SmallWgrad* wgrad, hipStream_t st);
// A classifier that one launch takes forward, through the loss and backward (k_thin.hip), and what that launch leaves
struct ThinHead {
    const void *x, *w;
    const float* bias;
    const int32_t* labels;
    float *logits, *row_loss, *loss;
    void *dlogits, *dx;
    GradDst dw, db, dbias;
};
bool thin_head_takes(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* w);
void launch_thin_head(int dtype, const ConvGeom& g, const ShardSet& S, const ThinHead& t, hipStream_t st);

}  // namespace edl

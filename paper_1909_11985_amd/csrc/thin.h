// Fully connected layers with few, ragged outputs (k_thin.hip), behind launch_conv_fwd, launch_conv_dgrad and launch_conv_wgrad.
#pragma once
#include "kernels.h"

namespace edl {

bool thin_takes(int dtype, const ConvGeom& g);
// ... and, for the weight gradient, shards of this many samples at most
bool thin_takes_shard(int largest);
void launch_thin_fwd(int dtype, const ConvGeom& g, const void* x, const void* w, const float* bias, bool relu, bool out_fp32, void* y, hipStream_t st);
// old (may be null, may be dx): the gradient that is added to.  Returns how the sums of mask are cut, p == 0 if it left none.
RowCut launch_thin_dgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* dy, const void* wT, const void* old, void* dx,
                         const DgradMask* mask, hipStream_t st);
void launch_thin_wgrad(int dtype, const ConvGeom& g, const ShardSet& S, const void* x, const void* dy, GradDst dw, hipStream_t st);

}  // namespace edl

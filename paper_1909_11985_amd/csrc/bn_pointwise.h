// The backward pass of a batch norm and of the expanding 1x1 convolution before it in one launch (k_bn_pointwise.hip).
#pragma once
#include "kernels.h"

namespace edl {

struct BnPointwiseTask {
    // the batch norm: its input (the convolution's output), the gradient of its output (masked already), the coefficients that
    // launch_bn_backward leaves
    const void *x, *dy;
    const float *gamma, *save, *coef;
    // the convolution: its input, its weights transposed [C][K], the gradient of its input (written)
    const void *act, *wT;
    void* dact;
    const DgradMask* mask;           // what the layer before wants of dact (xin given), or null
    float* partial;                  // bn_pointwise_partial_floats: pieces of the weight gradient
};

// Whether a batch norm over this convolution's output is taken, in passes of S.
bool bn_pointwise_takes(int dtype, const ConvGeom& g, const ShardSet& S);
// Returns how the sums of mask->sums are cut (p == 0 without a mask).
RowCut launch_bn_pointwise_backward(const ConvGeom& g, const ShardSet& S, const BnPointwiseTask& t, hipStream_t st);
// the weight gradient out of its pieces
void launch_bn_pointwise_reduce(const ConvGeom& g, const ShardSet& S, const float* partial, GradDst dw, hipStream_t st);

}  // namespace edl

// The streaming kernel of 1x1 convolutions with a short reduction (k_pointwise.hip), behind launch_conv_fwd and
// launch_conv_dgrad.
#pragma once
#include "kernels.h"

namespace edl {

struct PointwiseTask {
    int K, N;                        // reduction, output channels
    const void *A, *B;               // [pixels][K], [N][K]
    void* out;                       // [pixels][N]
    SumsBuf sums;                    // forward: the sums of out and out * out (may be null); join: those of DgradMask
    bool join;                       // an input gradient that is added to `old`, masked by `sign` and summed
    const void* old;
    const unsigned char* sign;
    const void* xin;
    const float* mean_rstd;
};

// Whether a layer's launch over a pass planned for plan_samples samples, with reduction K and N output channels, is taken.
bool pointwise_takes(int dtype, const ConvGeom& g, int plan_samples, int K, int N);
// False: not launched (the sums' buffer is too small).  *left: how the sums are cut, p == 0 if there are none.
bool launch_pointwise(const ConvGeom& g, const ShardSet& S, const PointwiseTask& t, RowCut* left, hipStream_t st);

}  // namespace edl

// 3x3 convolutions of few channels in float32 (k_narrow.hip), behind launch_conv_fwd and launch_conv_dgrad.
#pragma once
#include "kernels.h"

namespace edl {

struct NarrowTask {
    const float *x, *w;              // [pixels][C], [C][3][3][C]
    float* y;                        // [pixels][C]
    bool flip;                       // an input gradient: the taps the other way round
    const float* old;                // added to the output, or null
    SumsBuf sums;                    // forward: of y and y * y (buf may be null); with mask: DgradMask's
    const DgradMask* mask;           // with xin, or null
};

// Whether a layer of a pass planned as S goes there; true only for 3x3 of stride 1 in float32.
bool narrow_takes(int dtype, const ConvGeom& g, const ShardSet& S);
// Returns how the sums are cut, p == 0 if there are none.
RowCut launch_narrow(const ConvGeom& g, const ShardSet& S, const NarrowTask& t, hipStream_t st);

}  // namespace edl

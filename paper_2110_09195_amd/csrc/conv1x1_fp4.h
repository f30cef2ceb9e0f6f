// 1x1 layers on packed channels as a dense FP4 contraction (conv1x1_fp4.hip): host interface.
#pragma once

#include "snn_internal.h"

namespace snn {

// layers the kernel takes (of those subbit_conv1x1_supported allows): 32-bit offsets inside the images that a wave touches
bool conv1x1_fp4_supported(const Geom &g);
size_t conv1x1_fp4_workspace_bytes(const Geom &g);
int launch_conv1x1_fp4(const Geom &g, const void *x, const uint16_t *codebook8, const uint16_t *idx, const float *alpha, float *y, void *ws,
                       hipStream_t s, int phases);

}  // namespace snn

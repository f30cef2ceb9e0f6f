// Sub-bit 3x3 convolution on packed rows as a dense FP4 contraction (rows_fp4.hip): host interface.
#pragma once

#include "snn_internal.h"

namespace snn {

// layers the kernel takes: any subset size; rows narrow enough that the tile of a workgroup fits LDS, 32-bit offsets
bool rows_fp4_supported(const Geom &g);
// whether the one-hot matrix form is the faster one (for layers that it takes)
bool rows_fp4_loses_on_wide_rows(const Geom &g, bool sign);
size_t rows_fp4_workspace_bytes(const Geom &g);

// tau = 0: `idx` is uint16 [C_out][C_in]; else a stream of tau-bit indices (see snn_pack_indices)
int launch_rows_fp4(const Geom &g, const void *x, const uint16_t *codebook, const void *idx, int tau, const float *alpha, float *y,
                    void *ws, hipStream_t s, const SignEpilogue *sign, int phases);
// the 1-bit layer on packed channels (weights: 9-bit kernel codes; alpha is read by the convolution)
bool bnn_rows_form(const Geom &g);
size_t bnn_rows_workspace_bytes(const Geom &g);
int launch_bnn_rows(const Geom &g, const void *x, const uint16_t *w9, const float *alpha, float *y, void *ws, hipStream_t s, int phases);
// Alg. 1 forward of a layer: projection (idx_out) and packing (x -> xr; x == nullptr: xr is the packed input), then the convolution
int launch_rows_fp4_forward(const Geom &g, const float *x, const float *w, const uint16_t *codebook, const float *alpha, uint16_t *idx_out,
                            float *y, uint32_t *xr, void *ws, hipStream_t s, const SignEpilogue *sign);
// several layers: the weights-side work, and the convolutions from prepared workspaces (fp32 output)
int launch_rows_fp4_project_many(int n_layers, const Geom *gs, const float *const *w, const uint16_t *const *codebook,
                                 const float *const *alpha, const float *const *beta, uint16_t *const *idx_out, void *const *ws, hipStream_t s);
// the same with the packing of the layers' activations (x -> xr)
int launch_rows_fp4_front_many(int n_layers, const Geom *gs, const float *const *x, uint32_t *const *xr, const float *const *w,
                               const uint16_t *const *codebook, const float *const *alpha, uint16_t *const *idx_out, void *const *ws,
                               hipStream_t s);
// (projected: the same call has projected the layers' real-valued kernels)
int launch_rows_fp4_many(int n_layers, const Geom *gs, const void *const *x, float *const *y, void *const *ws, bool projected, hipStream_t s);

}  // namespace snn

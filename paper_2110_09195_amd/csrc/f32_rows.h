// Dense form of the fp32-activation layer (subbit_f32.hip): which input value lies at which place of the rows that a block
// of 32 output pixels keeps in LDS.  Also compiled for the host, where the numbering can be checked at any size.
#pragma once

#include "snn_internal.h"

namespace snn {

struct SdRows {
    int pitch;                                 // W + 1: column -1, a zero pixel, is also the right border of the row above
    Divisor div_pitch, div_H1;
};

inline SdRows sd_rows(const Geom &g) { return {g.W + 1, make_divisor((uint32_t)g.W + 1u), make_divisor((uint32_t)g.H + 1u)}; }

// values per channel that the block's rows hold at most (a zero row between images), as the loads of a lane half
inline int64_t sd_loads(const Geom &g)
{
    const int64_t row_changes = (g.Wo - 1 + 31) / g.Wo, image_changes = ((int64_t)g.HoWo - 1 + 31) / g.HoWo;
    return ((g.stride * row_changes + image_changes + 3) * (g.W + 1) + 1 + 31) / 32;
}

// Rows are numbered n (H + 1) + h + 1 from the block's first image on, so that the numbers stay small whatever the batch: over
// the batch they pass 2^31 (N > 2^30 images of one row).
struct SdBlock {
    uint32_t n0;                               // first image
    int row0;                                  // number of the row that position 0 lies in
};

__host__ __device__ inline SdBlock sd_block(const Geom &g, uint32_t blk)
{
    const uint32_t p0 = blk * 32u, n0 = p0 / (uint32_t)g.HoWo;
    return {n0, (int)((p0 - n0 * (uint32_t)g.HoWo) / (uint32_t)g.Wo) * g.stride};
}

// position of tap 0 of output pixel (n, ho, wo); tap t lies (t / 3) pitch + t % 3 further on
__host__ __device__ inline int sd_window(const Geom &g, const SdRows &rows, const SdBlock &b, uint32_t n, int ho, int wo)
{
    return ((int)(n - b.n0) * (g.H + 1) + ho * g.stride - b.row0) * rows.pitch + wo * g.stride;
}

struct SdPixel {
    int image, h, w;                           // image counted from the block's first
    bool in;                                   // else a zero
};

__host__ __device__ inline SdPixel sd_pixel(const Geom &g, const SdRows &rows, const SdBlock &b, int position)
{
    const int row = (int)fast_div((uint32_t)position, rows.div_pitch), R = b.row0 + row;
    const int image = (int)fast_div((uint32_t)R, rows.div_H1);
    SdPixel p = {image, R - image * (g.H + 1) - 1, position - row * rows.pitch - 1, false};
    p.in = p.h >= 0 && p.w >= 0 && image < g.N - (int)b.n0;
    return p;
}

}  // namespace snn

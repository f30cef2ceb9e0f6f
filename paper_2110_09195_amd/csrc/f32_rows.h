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

// Whether a wave of the form on the fp32 unit brings the rows to LDS, and with how many loads per pair of channels (three instances of the
// kernel); 0: its nine taps straight from memory.  (Rows of up to six loads and more than eight channels go in bf16 pieces, subbit_f32.hip;
// sd_looks_up goes by this rule for both.)  Both ways, us, prepared weights, memory -> LDS:
//   three loads        3x5 and 7x7 to 8x8: 64 -> 64 8x8 batch 256 18.2 -> 17.2, 512 -> 512 7x7 batch 64 173 -> 160
//   four               where a chip half full waits for each load, 64 -> 64 16x16 batch 8 7.0 -> 6.9, 512 -> 512 13x13 batch 8 (688
//                      blocks) 79 -> 74, 96 -> 96 13x13 batch 64 (1014) 24.7 -> 24.6; not over more than two rounds of
//                      workgroups, 64 -> 64 14x14 batch 256 (3136) 53.8 -> 57.1, 128 -> 128 13x13 batch 64 (1352) 43.9 -> 44.4.
//                      Blocks of one wave (few channels) at any number: 24 -> 64 13x13 batch 256 20.9 -> 20.4
//   five and six       only over long chains of channels where half the chip has no block at all, 512 -> 64 32x32 batch 1 (64 blocks)
//                      34.0 -> 32.5, 512 -> 512 10x25 batch 1 (128) 34.2 -> 33.0, or (stride 2) on rows of eight pixels, whose taps
//                      from memory are slow, 128 -> 128 8x8 batch 256 20.7 -> 18.0; not 64 -> 64 10x25 batch 256 64.9 -> 73.4, 28x28
//                      189 -> 219, 16 -> 16 28x28 batch 64 (one wave) 10.5 -> 11.1, 512 -> 512 28x28 batch 1 (400) 49.2 -> 49.4,
//                      128 -> 128 1x1 batch 256 11.2 -> 11.6, 33 -> 20 28x28 batch 1 5.7 -> 5.9, 7x7 stride 2 16.7 -> 17.9
// quads: of pairs of input channels; more than three are split over four waves.
inline int sd_staged(const Geom &g, int quads, int64_t n_blocks)
{
    const int64_t loads = sd_loads(g);
    if (loads <= 3) return 3;
    if (loads <= 4 && (quads < 4 || n_blocks <= 1024)) return 4;
    if (loads <= 6 && ((quads >= 16 && n_blocks <= 128 && g.HoWo >= 32) || (g.stride == 2 && (g.W & 7) == 0))) return 6;
    return 0;
}

// Whether a layer given as indices looks its codes up in the convolution, without a launch that prepares its words (2.5 us).  A
// workgroup then waits for indices and codebook before its first pair, and for each quad's indices in turn with its own loads, which
// costs more the more loads it has in flight.  us per call, two launches -> looked up:
//   three loads   64 -> 64 8x8 batch 128 (512 workgroups) 11.3 -> 10.9, batch 256 (1024) 19.37 -> 19.28, 256 -> 256 8x8 batch 64 (1024)
//                 51.2 -> 51.0, 64 -> 512 8x8 batch 64 (2048) 33.3 -> 34.9
//   four, six     128 -> 128 14x14 batch 8 (200) 12.9 -> 11.6, batch 32 (784) 31.1 -> 31.6, 64 -> 64 14x14 batch 64 (784) 20.0 -> 20.3
//   memory        64 -> 64 28x28 batch 8 (392) 12.4 -> 12.0, 128 -> 128 37x53 batch 1 (248) 13.5 -> 12.4, 256 -> 256 32x32 batch 1 (256) 21.0 ->
//                 19.8, 3 -> 64 28x28 batch 128 (1568, one quad) 19.9 -> 19.5, batch 256 32.8 -> 33.4; 64 -> 64 16x16 stride 2 batch 256
//                 (1024) 26.0 -> 27.2, 128 -> 128 32x32 batch 8 (1024) 31.9 -> 32.6, 512 -> 64 28x28 batch 8 (392) 52.2 -> 55.5
inline bool sd_looks_up(int staged, int quads, int64_t n_wgs)
{
    if (staged == 3) return n_wgs <= 1024;
    if (staged) return n_wgs <= (quads <= 8 ? 1024 : 256);
    return quads <= 32 && n_wgs <= 2048 && n_wgs * quads <= (n_wgs <= 512 ? 8192 : 4608);
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

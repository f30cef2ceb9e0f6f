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

// Whether the bf16 pieces (subbit_f32.hip) are the faster way: rows that fit six loads (two workgroups of a compute unit then have their LDS) and
// more channels than half of the sixteen that a step takes.  us, fp32 unit -> pieces, K = 32: 12 -> 12 8x8 batch 256 6.7 -> 5.8, 28x28 batch 200
// 22.6 -> 18.4; 8 -> 32 8x8 batch 256 6.25 -> 5.96, 28x28 batch 200 18.7 -> 19.0, 4 -> 16 14.1 -> 18.3, 1 -> 8 12.4 -> 18.4.  With ten loads (one
// workgroup to a compute unit) 64 -> 64 56x56 batch 32 100 -> 95, 16 -> 16 batch 64 35 -> 49, 14x53 batch 8 12.3 -> 16.6.
inline bool sd_split(const Geom &g) { return g.C_in > 8 && sd_loads(g) <= 6; }

struct SdSplit {
    int loads;                   // instance of the kernel: 3, 4 or 6
    int CB;                      // blocks of 32 output channels of a wave
    bool four;                   // four waves split the channels of a block
    int steps;                   // of sixteen channels, of a wave
    int64_t blocks, n_wgs;
};

// Two blocks of output channels read each piece for two products; one, and the channels split over four waves, where that leaves SIMDs
// without a wave (2 -> 1 blocks, us: 512 -> 21 6x6 batch 231 37.6 -> 27.4, 64 -> 64 8x8 batch 8 7.5 -> 5.7; one wave -> four: 24 -> 64 13x13
// batch 64 11.4 -> 8.6; of few channels and many blocks four waves have nothing to do).
inline SdSplit sd_split_plan(const Geom &g)
{
    const int n_cob = (g.C_out + 31) / 32;
    const int64_t px = (g.P + 31) / 32, octs = (g.C_in + 15) / 16, loads = sd_loads(g);
    SdSplit s;
    s.loads = loads <= 3 ? 3 : loads == 4 ? 4 : 6;
    s.CB = n_cob >= 2 && px * ((n_cob + 1) / 2) * (octs >= 4 ? 4 : 1) >= 1024 ? 2 : 1;
    s.blocks = px * ((n_cob + s.CB - 1) / s.CB);
    s.four = octs >= 4 || (octs >= 2 && s.blocks < 1024);
    s.steps = (int)(s.four ? (octs + 3) / 4 : octs);
    s.n_wgs = s.four ? s.blocks : (s.blocks + 3) / 4;
    return s;
}

// Whether a layer given as indices looks its codes up in the pieces kernel, without a launch that prepares its words (1.3 us in a row of
// calls).  A step then loads sixteen indices a lane, two bytes each from rows C_in apart, which is soon dearer: with the second step, the
// second block of output channels, and the third workgroup of a compute unit.  Rows of indices that are a multiple of 32 bytes are read more
// slowly than others.  us per call, two launches -> looked up:
//   C_in a multiple of 16   64 -> 64 8x8 batch 8 (32 workgroups) 6.6 -> 5.8, batch 64 (256) 6.7 -> 5.9, 32 -> 96 8x8 batch 83 (498) 7.45 -> 7.44, batch 100
//                           (600) 8.2 -> 9.0; two steps: 96 -> 96 8x8 batch 33 (198) 8.6 -> 8.2, 128 -> 128 8x8 batch 8 (64) 8.5 -> 8.6, 14x14 batch 8
//                           (196) 9.9 -> 10.0, 128 -> 64 7x7 batch 97 (298) +9 %; four: 256 -> 256 8x8 batch 1 (16) 12.2 -> 13.6; two blocks: 64 -> 64
//                           8x8 batch 128 (256) 7.9 -> 8.0, batch 256 (512) 9.2 -> 10.2, 256 -> 256 8x8 batch 64 (512) 19.9 -> 29.2
//   not                     40 -> 96 8x8 batch 33 (198) 6.6 -> 5.3, batch 83 (498) 7.6 -> 6.6, batch 133 (798) 10.1 -> 9.0, 9 -> 32 8x8 batch 2000 (1000)
//                           -17 %; two steps: 100 -> 60 8x8 batch 50 (200) -11 %, batch 125 (500) -8 %; three and four, up to 512 workgroups: -6 % to +1 %;
//                           five and more (300 and 500 channels): +2 to +13 %; two blocks: 12 to 60 channels up to 512 workgroups -13 to -1 %, up to
//                           820 -5 to +4 %; two blocks and steps: -1 to +10 %
inline bool sd_pieces_look_up(const Geom &g, const SdSplit &s)
{
    const bool apart = g.C_in % 16 != 0;
    if (s.CB == 2) return apart && s.steps == 1 && s.n_wgs <= 512;
    if (apart) return s.n_wgs <= 512 ? s.steps <= 4 : s.steps == 1 && s.n_wgs <= 1024;
    return s.steps == 1 ? s.n_wgs <= 512 : s.steps == 2 && s.n_wgs <= 256;
}

// The form on the fp32 unit, which has what the pieces do not take, eight channels and fewer or wide rows.  Whether a wave brings the rows to
// LDS, and with how many loads per pair of channels (three instances of the kernel); 0: its nine taps straight from memory.  Only of
// eight channels and fewer: wide rows are more than six loads.  us per call, memory -> LDS:
//   three loads        1 -> 8 8x8 batch 256 4.60 -> 4.39, 3 -> 64 5.39 -> 5.25, 8 -> 32 6.13 -> 5.85, 8 -> 128 3x5 8.7 -> 8.2
//   four               1 -> 8 14x14 batch 256 6.08 -> 6.03, 3 -> 64 12.01 -> 12.11, 8 -> 32 9.52 -> 9.28, 8 -> 128 16x16 27.1 -> 25.9
//   five and six       1 -> 8 28x28 batch 256 15.5 -> 16.6, 3 -> 64 30.5 -> 33.1, 8 -> 128 73.8 -> 80.3; at stride 2 on rows of whole eight
//                      pixels, whose taps from memory are slow, 8x8 batch 256 8 -> 32 6.80 -> 6.25, 8 -> 128 7.03 -> 6.51 (but 3 -> 64 5.29 -> 5.29,
//                      1 -> 8 4.49 -> 4.69), not on others, 7x7 8 -> 32 6.12 -> 6.29
inline int sd_staged(const Geom &g)
{
    const int64_t loads = sd_loads(g);
    if (loads > 6 || g.C_in > 8) return 0;
    return loads <= 3 ? 3 : loads == 4 ? 4 : g.stride == 2 && (g.W & 7) == 0 ? 6 : 0;
}

// The same question for this form; quads: of pairs of input channels.  us per call, two launches -> looked up:
//   three, four loads  1 -> 8 8x8 batch 200 (100 workgroups) 5.7 -> 4.4, 8 -> 128 batch 512 (1024) 14.3 -> 13.7, batch 1024 (2048) 24.7 -> 25.1,
//                      3 -> 64 14x14 batch 334 (1023) 13.8 -> 12.6, 8 -> 32 batch 1337 (2048) 26.1 -> 26.3
//   six                8 -> 32 8x8 stride 2 batch 4096 (512) 9.9 -> 9.1, batch 8192 (1024) 15.5 -> 15.3, batch 16384 28.8 -> 29.7
//   memory             3 -> 64 28x28 batch 41 (503) 8.4 -> 6.8, batch 167 (2046) 21.1 -> 20.2, 8 -> 32 56x56 batch 41 (1005) 14.9 -> 14.4; at stride 2
//                      8 -> 128 16x16 batch 256 (512) 10.6 -> 10.2, batch 512 (1024) 17.3 -> 18.0; two quads and more: 16 -> 64 56x56 batch 5
//                      (245) 9.6 -> 8.4, batch 16 (784) 20.9 -> 21.1, batch 41 (2009) 38.2 -> 40.2; 64 -> 64 37x53 batch 1 (124) 9.5 -> 8.3,
//                      batch 4 (492) 12.5 -> 11.6, 14x100 batch 9 (788) 20.1 -> 19.9, batch 14 (1226) 25.8 -> 26.4; 128 -> 128 37x53 batch 2
//                      (492) 18.4 -> 17.9; at stride 2 32 -> 64 56x56 batch 10 (490) 9.5 -> 9.4, batch 16 (784) 14.5 -> 16.2, 256 -> 256 32x32
//                      batch 4 (256) 21.8 -> 21.2, batch 8 (512) 31.0 -> 32.4
inline bool sd_looks_up(const Geom &g, int staged, int quads, int64_t n_wgs)
{
    if (staged) return n_wgs <= 1024;
    return quads <= 32 && n_wgs <= (g.stride == 2 ? 512 : quads == 1 ? 2048 : 1024) && n_wgs * quads <= (n_wgs <= 512 ? 8192 : 4608);
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

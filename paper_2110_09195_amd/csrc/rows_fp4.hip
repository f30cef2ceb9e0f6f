// The sub-bit 3x3 convolution on packed rows as a dense contraction over (tap, input channel) on the matrix cores:
//
//   S[co][pixel] = sum over taps t and input channels c of  w(co, c, t) * x(pixel, t, c),   w = codebook[idx[co][c]]
//
// with w, x in {+1, -1} (0 for taps outside the image and for padding channels) as FP4 e2m1 operands of
// v_mfma_f32_32x32x64_f8f6f4.  All products are +-1 or 0 and |S| <= 9 C_in < 2^24, so the fp32 accumulator holds S
// exactly and the results are those of the two-stage form bit for bit, for every subset size.
//
// Why not the one-hot form of the two stages (subbit_mfma.hip): gathering one of K responses costs that form K
// contraction slots per input channel on a matrix unit (16, 32 or 64), this one costs nine, whatever K is.  Matrix
// instructions of the ResNet-18 stack at batch 64, K = 32: 5.82 M there, 1.64 M here.  Measured, one-hot form -> this one:
// that stack's convolutions 200 -> 91 us; 256 -> 256 14x14 batch 128 K = 32 32 -> 14.7 us; 512 -> 512 7x7 batch 256
// K = 64 92 -> 29 us; K > 64 (the LDS-gather kernel) 100 -> 150 37x53 stride 2 batch 12 164 -> 12.5 us.
//
// Operands.  A step is 64 contraction slots; lane half h of a wave supplies 32 of them, the 32 channels of one
// channel block at one tap:
//   main steps   step 9 p + t: channel blocks 2 p (h = 0) and 2 p + 1 (h = 1), tap t
//   last steps   (an odd number of channel blocks) the last block alone, taps 2 s (h = 0) and 2 s + 1 (h = 1); for the tap
//                that does not exist the lanes read a zero pixel
// Both operands are FP4 codes 0010 (+1 or -1 by the sign bit, bit 3): a set bit (+1) is stored with the sign bit set on
// both sides, so that the sign bits are the packed bits themselves and the product comes out right.
// A (weights) is kept at one bit per weight, 32 slots in a word whose bit 4 j + r is slot 8 r + j: two instructions make
//   eight codes of it.  (As codes in memory, four times the bytes, the weights were the bound: a wave of 1 x 2 blocks
//   needs 2 KB of codes per 64 clocks of matrix work.)
// B (activations) is read from LDS as it is: a workgroup expands the packed rows its pixels touch into codes once,
//   [channel block of 32][pixel] 16 bytes,
//   on rows of W + 1 pixels (column -1 is a zero pixel and also the right border of the row above; or of W + 2) and images of H + 1
//   rows (a zero row above each image is also the bottom border of the one before): no tap needs a mask, and the
//   window of an output pixel is nine reads at fixed distances.  Channels past C_in are zero here.
// Packed channels (the 1-bit layer: a word holds 32 channels of a pixel, no transposition) run through the same kernel: which
// channel of a block sits in which slot is free as long as both operands agree, so there slot 8 r + j is channel 4 j + r, a
// word of packed channels is expanded as a word of weights is, and weight words are plain bit planes.
#include "fp4_common.h"
#include "front_ops.h"
#include "rows_fp4.h"

#include <algorithm>
#include <type_traits>
#include <vector>

namespace snn {

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const u32x4 lds_cu32x4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef __attribute__((address_space(3))) const f32x4 lds_cf32x4;

// words of a pair of channel blocks and 32 output channels: [lane] 16 bytes (taps 0..3), [lane] 16 bytes (4..7), [lane] 4 (8)
constexpr uint32_t RF_PAIR_BYTES = 2304;
// One layer as the kernel sees it.
struct RfLayer {
    const uint32_t *x;       // packed rows [N][C_in][H][WW]
    const uint32_t *wq;      // weights in operand layout
    const float *scale;      // [2][32 n_cob]: alpha, 0 for padding channels; before the sign epilogue what sign_entry gives
    void *out;               // float y, or packed rows of the signs
    int N, C_in, C_out, H, W, WW, stride;
    int Ho, Wo, HoWo, P;
    int n_cob;               // blocks of 32 output channels
    int ncb;                 // blocks of 32 input channels
    int chunk;               // of which this many are expanded into LDS at a time (even unless all of them)
    int pairs;               // pairs of channel blocks, the last one possibly half empty
    int pitch;               // pixels from one expanded row to the next: W + 1, or W + 2
    int plane;               // bytes of one expanded channel block
    int n_blk;               // blocks of up to 32 pixels
    int n_cotiles, n_wgs;
    int wpx_shift;           // log2 of the waves of a workgroup along pixels; the others share its pixels
    int policy;              // of the output's stores, FP4_STORE_*
    int rows_pb, bpi, wpr;   // sign epilogue: rows per block, blocks per image, blocks per row
    Divisor div_HoWo, div_Wo, div_H1, div_WW, div_cotiles, div_bpi, div_wpr, div_Ho;
    Divisor div_W1;          // packed channels
    const uint16_t *codebook, *idx;      // INDEXED
    int K;
};

// byte p of the four words -> o[p]
__device__ __forceinline__ void bytes4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&o)[4])
{
    const uint32_t ab_lo = __builtin_amdgcn_perm(b, a, 0x05010400u), ab_hi = __builtin_amdgcn_perm(b, a, 0x07030602u);
    const uint32_t cd_lo = __builtin_amdgcn_perm(d, c, 0x05010400u), cd_hi = __builtin_amdgcn_perm(d, c, 0x07030602u);
    o[0] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x07060302u);
}

// ---- weights -> operand layout, device side ----------------------------------------------------------------------
// Codes of up to 8 consecutive channels as three words of nibbles (nibble j: bits 0..3 of channel j's code in `lo`, 4..7 in
// `mid`, bit 8 in `hi`) -> bits 4 j: tap t of channel j (code bit 8 - t).
__device__ __forceinline__ uint32_t tap_bits(uint32_t lo, uint32_t mid, uint32_t hi, int t)
{
    const int bit = 8 - t;
    return ((bit == 8 ? hi : bit >= 4 ? mid : lo) >> (bit & 3)) & 0x11111111u;
}

// Stores the words of (channel co of a block of 32 output channels, input channel block cb) in their pair's RF_PAIR_BYTES (in memory or
// in LDS): w[t] for tap t.
template <class Put16, class Put4>
__device__ __forceinline__ void put_words(Put16 &&put16, Put4 &&put4, int co, int cb, int ncb, const uint32_t (&w)[9])
{
    if ((ncb & 1) && cb == ncb - 1) {
        // the last block of an odd number: word u of lane half h is tap 2 u + h
        put16(co * 16, (u32x4){w[0], w[2], w[4], w[6]});
        put16((co + 32) * 16, (u32x4){w[1], w[3], w[5], w[7]});
        put4(1024 + co * 16, w[8]);
        put4(1024 + (co + 32) * 16, 0u);
        return;
    }
    const int lane = co + 32 * (cb & 1);
    put16(lane * 16, (u32x4){w[0], w[1], w[2], w[3]});
    put16(1024 + lane * 16, (u32x4){w[4], w[5], w[6], w[7]});
    put4(2048 + lane * 4, w[8]);
}

__device__ __forceinline__ void store_words(uint32_t *wq, int cob, int co, int cb, int ncb, const uint32_t (&w)[9])
{
    unsigned char *const at = (unsigned char *)wq + (int64_t)(cob * ((ncb + 1) >> 1) + (cb >> 1)) * RF_PAIR_BYTES;
    put_words([&](int o, u32x4 v) { *(u32x4 *)(at + o) = v; }, [&](int o, uint32_t v) { *(uint32_t *)(at + o) = v; }, co, cb, ncb, w);
}

// The words of eight codes per lane, four lanes side by side (d = lane % 4: channels 8 d .. 8 d + 7 of a block), valid in all four.
__device__ __forceinline__ void words_of_codes(const uint32_t (&code)[8], int d, uint32_t (&w)[9])
{
    uint32_t lo = 0, mid = 0, hi = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        lo |= (code[j] & 15u) << (4 * j);
        mid |= ((code[j] >> 4) & 15u) << (4 * j);
        hi |= (code[j] >> 8) << (4 * j);
    }
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        w[t] = tap_bits(lo, mid, hi, t) << d;
        w[t] |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[t], 0xB1 /* quad_perm [1,0,3,2] */, 0xF, 0xF, true);
        w[t] |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[t], 0x4E /* quad_perm [2,3,0,1] */, 0xF, 0xF, true);
    }
}

// ---- the convolution ----------------------------------------------------------------------------------------
// A workgroup of four waves: 2^wpx_shift of them side by side along pixels, the others on further output channels of
// the same pixels.  A wave owns PB blocks of 32 pixels x CB blocks of 32 output channels.  Pixel blocks: 32 consecutive
// pixels of the flattened (n, ho, wo) order; for the sign epilogue whole output words (whole rows while they fit 32
// pixels, else one word of a row), so that the wave that owns a block owns the words it writes.
// INDEXED: the weight words are made here, from codebook and indices, and kept in LDS behind the expanded pixels.
// PACED (several layers whose outputs are past the last-level cache): a divisor of one is a branch, buffers end with the batch, in 64 bits, and
// stores are non-temporal.  The start of a workgroup's life is a chain of scalar and vector instructions; without those branches and with
// buffers that end with the tile's images, in 32 bits, it is shorter: 1-bit chain of ResNet-18 batch 64 127 -> 123.5 us, 256 -> 256 14x14
// batch 128 13.0 -> 12.6, 100 -> 150 37x53 stride 2 batch 12 9.75 -> 9.3, the 32-layer stack at batch 8 51.3 -> 50.1.  Not so here, and it
// shows on some cards only.  States of rows_fp4_many_kernel, in turn, forward pass of the ResNet-18 stack at batch 64, us on each of five cards, and
// registers that the compiler keeps in scratch memory:
//   branches, 64 bits      180.6 180.4 178.8 179.6 179.8   2 (this)
//   branches, 32 bits      184.3 179.6 179.9 182.6 183.8   none
//   no branches, 64 bits   184.1 179.9                     none
//   no branches, 32 bits   197.5                           4
// At batch 50 the first two are the same (145.6 and 145.5).  With the other policy's store loop beside the non-temporal one 180.3, 178.8, 178.8, 178.9;
// with the last block's values kept from registers (see there; none in scratch) 182.8, 179.8.  Why is not known, no counter was read.
template <int PB, int CB, bool SIGN, bool CHANNELS = false, int TASKS = 4, bool INDEXED = false, bool PACED = false>
__device__ __forceinline__ void rf_tile(const RfLayer &L, uint32_t wg, unsigned char *const smem)
{
    const int tid = threadIdx.x;
    auto div = [](uint32_t n, const Divisor &d) -> uint32_t {      // (PACED: see above)
        if constexpr (PACED) {
            if (d.shift == 0) return n;
        }
        return fast_div(n, d);
    };
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_l = lane & 31, h = lane >> 5;
    // Workgroups go to the eight XCDs in turn: an XCD gets a contiguous run of tiles, so that neighbours in the output
    // planes and the tiles that read the same packed rows share an L2.
    {
        const uint32_t per = (uint32_t)L.n_wgs >> 3, rem = (uint32_t)L.n_wgs & 7u, xcd = wg & 7u;
        wg = xcd * per + min(xcd, rem) + (wg >> 3);
    }
    const uint32_t pxt = div(wg, L.div_cotiles);
    const int cot = (int)(wg - pxt * (uint32_t)L.n_cotiles);
    const int wpx = wave & ((1 << L.wpx_shift) - 1), wco = wave >> L.wpx_shift;
    const int wg_blk0 = (int)pxt * (PB << L.wpx_shift);
    const int blk0 = wg_blk0 + wpx * PB;
    const int cob0 = ((cot << (2 - L.wpx_shift)) + wco) * CB;
    const bool active = cob0 < L.n_cob && blk0 < L.n_blk;       // wave-uniform; idle waves still fill LDS

    // ---- pixels --------------------------------------------------------------------------------------------------
    auto pixel_of = [&](int B, int px, int &n, int &ho, int &wo) -> bool {
        bool ok = B < L.n_blk;
        if (!ok) B = L.n_blk - 1;
        if constexpr (!SIGN) {
            int pp = B * 32 + px;
            if (pp >= L.P) {
                ok = false;
                pp = L.P - 1;
            }
            n = (int)div((uint32_t)pp, L.div_HoWo);
            const int r = pp - n * L.HoWo;
            ho = (int)div((uint32_t)r, L.div_Wo);
            wo = r - ho * L.Wo;
        } else if (L.Wo <= 32) {
            n = (int)div((uint32_t)B, L.div_bpi);
            const int rb = B - n * L.bpi;
            int rl = (int)div((uint32_t)px, L.div_Wo);
            wo = px - rl * L.Wo;
            ho = rb * L.rows_pb + rl;
            if (rl >= L.rows_pb || ho >= L.Ho) {
                ok = false;
                ho = rb * L.rows_pb;
                wo = 0;
            }
        } else {
            const int R = (int)div((uint32_t)B, L.div_wpr);
            n = (int)div((uint32_t)R, L.div_Ho);
            ho = R - n * L.Ho;
            wo = 32 * (B - R * L.wpr) + px;
            if (wo >= L.Wo) {
                ok = false;
                wo = 32 * (B - R * L.wpr);
            }
        }
        return ok;
    };
    // rows (numbered n (H + 1) + h + 1 over the batch) that the workgroup's pixels touch
    const int H1 = L.H + 1, W1 = L.pitch;
    const uint32_t pitch = (uint32_t)W1 * 16u;
    int R0, nrows, n0, n_images;
    {
        int ho, wo, n1, ho1, wo1;
        pixel_of(wg_blk0, 0, n0, ho, wo);
        R0 = n0 * H1 + ho * L.stride;
        const int lastB = min(wg_blk0 + (PB << L.wpx_shift), L.n_blk) - 1;
        if constexpr (!SIGN) {
            pixel_of(lastB, min(31, L.P - 1 - 32 * lastB), n1, ho1, wo1);
        } else {
            pixel_of(lastB, 0, n1, ho1, wo1);
            if (L.Wo <= 32) ho1 = min(ho1 + L.rows_pb, L.Ho) - 1;
        }
        nrows = n1 * H1 + ho1 * L.stride + 3 - R0;
        R0 = __builtin_amdgcn_readfirstlane(R0);
        nrows = __builtin_amdgcn_readfirstlane(nrows);
        n0 = __builtin_amdgcn_readfirstlane(n0);
        n_images = __builtin_amdgcn_readfirstlane(n1) - n0 + 1;
    }

    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const uint32_t plane = (uint32_t)L.plane;
    const uint32_t tile_lds = lds0 + 4u * CB * 32u * (SIGN ? 8u : 4u);      // behind the scales
    // ---- packed rows -> FP4 codes in LDS --------------------------------------------------------------------------
    // A task of a wave is 16 words (a word: 32 pixels of a row) of one channel block: lane (i, g) takes word i of the 8
    // channels of group g - eight loads, a transposition of nibbles, two instructions per pixel - and four lanes side by
    // side write the 16 bytes of a pixel.  A wave loads TASKS tasks at a time, four in the one-layer kernels: a load takes as long to come
    // back as six tasks to expand.  Measured, one task ahead -> four at a time, the last pixels of a row apart from the whole groups
    // of four, and the row pitch of rf_plan: 1-bit chain of ResNet-18 batch 64 156 -> 148 us, 512 -> 512 7x7 batch 256 28.2 -> 26.0, 256 -> 256
    // 14x14 batch 128 14.5 -> 13.6, 100 -> 150 37x53 stride 2 batch 12 12.2 -> 10.0.  Several layers in one launch are bound by memory:
    // two at a time 180.2 us for the ResNet-18 stack's forward pass, four 183.7, one 182.5.
    const uint32_t xplane = (uint32_t)(L.H * L.WW) * 4u;
    // the images from the tile's first on, of C planes each (of those that a tile touches: < 2 GiB)
    auto images = [&](const void *base, int C, uint32_t plane_bytes) {
        if constexpr (PACED) {
            const int64_t image_words = (int64_t)C * (int)(plane_bytes >> 2);
            const int64_t left = (int64_t)(L.N - n0) * image_words * 4;
            return make_rsrc((const uint32_t *)base + (int64_t)n0 * image_words, (uint32_t)min(left, (int64_t)0x7fffffff));
        } else {
            const uint32_t image_bytes = (uint32_t)C * plane_bytes;
            return make_rsrc((const char *)base + (uint64_t)(uint32_t)n0 * image_bytes, (uint32_t)n_images * image_bytes);
        }
    };
    const __amdgpu_buffer_rsrc_t xres = images(L.x, L.C_in, xplane);
    const int RW = nrows * L.WW, nk = (RW + 15) >> 4;
    const int grp = lane & 3;
    struct Task {
        uint32_t w[8];
        uint32_t addr, vmask;
        int npx;                                               // pixels of the word
        bool edge;                                             // the word starts a row
    };
    int my_k = 0, my_cb = 0, at_k = -1, at_npx = 0;            // the wave's next task: words 16 k .. 16 k + 15, channel block
    uint32_t at_off = 0, at_addr = 0;                          // what follows from k
    bool at_ok = false, at_edge = false;
    auto load_task = [&](Task &T, int cb_first) {
        if (my_k != at_k) {                                    // (wave-uniform)
            at_k = my_k;
            const int rw = 16 * my_k + (lane >> 2);
            const bool have = rw < RW;
            const int row = (int)div((uint32_t)rw, L.div_WW), word = rw - row * L.WW;
            const int R = R0 + row;
            const int n = (int)div((uint32_t)R, L.div_H1), hh = R - n * H1;
            at_ok = have && hh > 0 && n < L.N;
            at_off = (uint32_t)((((n - n0) * L.C_in + grp * 8) * L.H + hh - 1) * L.WW + word) * 4u;
            at_addr = tile_lds + (uint32_t)(row * W1 + 1 + 32 * word) * 16u + (uint32_t)grp * 4u;
            at_npx = have ? min(32, L.W - 32 * word) : 0;
            at_edge = have && word == 0;
        }
        const int cb0 = (cb_first + my_cb) * 32, left = L.C_in - cb0 - grp * 8;    // channels of the group that exist
        const bool ok = at_ok && left > 0;
        if ((L.C_in & 7) == 0) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                T.w[j] = __builtin_amdgcn_raw_buffer_load_b32(xres, (int)(ok ? at_off : OFF_NONE), (int)((uint32_t)(cb0 + j) * xplane), 0);
            T.vmask = ok ? 0xffffffffu : 0u;
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                T.w[j] = __builtin_amdgcn_raw_buffer_load_b32(xres, (int)(ok && left > j ? at_off + (uint32_t)j * xplane : OFF_NONE),
                                                              (int)((uint32_t)cb0 * xplane), 0);
            T.vmask = !ok ? 0u : left >= 8 ? 0xffffffffu : (1u << (4 * left)) - 1u;
        }
        T.addr = at_addr + (uint32_t)my_cb * plane;
        T.npx = at_npx;
        T.edge = at_edge;
        my_k += 4;
        while (my_k >= nk) {
            my_k -= nk;
            ++my_cb;
        }
    };
    auto store_task = [&](const Task &T) {
        int W = L.W;                                           // (opaque: a condition per group of pixels, kept in registers, would be
        asm volatile("" : "+s"(W));                            // dozens of them)
        uint32_t ev[4], od[4];
        bytes4(T.w[0], T.w[2], T.w[4], T.w[6], ev);
        bytes4(T.w[1], T.w[3], T.w[5], T.w[7], od);
        const uint32_t m8 = T.vmask & 0x88888888u, m2 = T.vmask & 0x22222222u;
        if (T.edge) {                                          // columns -1 and W
            *(lds_u32 *)(uintptr_t)(T.addr - 16u) = 0u;
            *(lds_u32 *)(uintptr_t)(T.addr + (uint32_t)L.W * 16u) = 0u;
        }
        uint32_t rest = 0;                                     // the last pixels of a row, where they are no whole group of four
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (8 * p >= W) break;                           // (wave-uniform: short rows have no such pixels)
            // D[m]: nibble j = pixels 4 m .. 4 m + 3 of channel j
            const uint32_t D[2] = {(ev[p] & 0x0f0f0f0fu) | ((od[p] << 4) & 0xf0f0f0f0u), ((ev[p] >> 4) & 0x0f0f0f0fu) | (od[p] & 0xf0f0f0f0u)};
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int px = 8 * p + 4 * m;
                if (px + 4 <= T.npx) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) *(lds_u32 *)(uintptr_t)(T.addr + 16u * (px + r)) = ((D[m] << (3 - r)) & m8) | m2;
                }
                if (px == (W & 28)) rest = D[m];
            }
        }
        if ((W & 3) && T.npx == (W & 31)) {
            const uint32_t at = T.addr + 16u * (uint32_t)(W & 28);
#pragma unroll
            for (int r = 0; r < 3; ++r)
                if (r < (W & 3)) *(lds_u32 *)(uintptr_t)(at + 16u * r) = ((rest << (3 - r)) & m8) | m2;
        }
    };
    // Packed channels [N][H][W][ncb]: a thread takes whole pixels of the tile, zero pixels included, two at a time.
    const __amdgpu_buffer_rsrc_t cres = images(L.x, 1, (uint32_t)(L.H * L.W * L.ncb) * 4u);
    auto fill_channels = [&](int cb_first, int ncb) {
        const int n_px = nrows * W1 + 1;
        for (int q0 = tid; q0 < n_px; q0 += 512) {
            uint32_t off[2], at[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int q = q0 + 256 * u;
                const int row = (int)div((uint32_t)q, L.div_W1), col = q - row * W1 - 1;
                const int R = R0 + row;
                const int n = (int)div((uint32_t)R, L.div_H1), hh = R - n * H1;
                const bool ok = row < nrows && col >= 0 && col < L.W && hh > 0 && n < L.N;
                off[u] = ok ? (uint32_t)((((n - n0) * L.H + hh - 1) * L.W + col) * L.ncb + cb_first) * 4u : OFF_NONE;
                at[u] = q < n_px ? tile_lds + (uint32_t)q * 16u : 0u;
            }
            for (int c0 = 0; c0 < ncb; c0 += 4) {
                uint32_t w[2][4];
                // (the scalar offset stays inside the buffer, also for words that do not exist: a lane offset is checked against what
                // the scalar one leaves of the buffer, which for the last pixel of one word would be less than nothing)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        w[u][c] = __builtin_amdgcn_raw_buffer_load_b32(cres, (int)(c0 + c < ncb ? off[u] : OFF_NONE), 4 * min(c0 + c, ncb - 1), 0);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int left = L.C_in - 32 * (cb_first + c0 + c);                    // channels of the block that exist
                        const uint32_t exist = off[u] == OFF_NONE ? 0u : left >= 32 ? 0xffffffffu : (1u << (left & 31)) - 1u;
                        const uint32_t v = w[u][c] & exist;
                        const u32x4 codes = {((v << 3) & 0x88888888u) | ((exist << 1) & 0x22222222u), ((v << 2) & 0x88888888u) | (exist & 0x22222222u),
                                             ((v << 1) & 0x88888888u) | ((exist >> 1) & 0x22222222u), (v & 0x88888888u) | ((exist >> 2) & 0x22222222u)};
                        if (at[u] && c0 + c < ncb) *(lds_u32x4 *)(uintptr_t)(at[u] + (uint32_t)(c0 + c) * plane) = codes;
                    }
            }
        }
    };
    // (of as many tasks at a time as there are in `task`)
    auto load_tasks = [&](auto &task, int cb_first, int ncb) -> int {
        int n = 0;
#pragma unroll
        for (auto &T : task)
            if (my_cb < ncb) {
                load_task(T, cb_first);
                ++n;
            }
        return n;
    };
    auto first_task = [&]() {
        my_k = wave;
        my_cb = 0;
        while (my_k >= nk) {
            my_k -= nk;
            ++my_cb;
        }
    };
    auto fill = [&](auto &task, int n_tasks, int cb_first, int ncb) {
        while (n_tasks > 0) {
            int i = 0;
#pragma unroll
            for (const auto &T : task)
                if (i++ < n_tasks) store_task(T);
            n_tasks = load_tasks(task, cb_first, ncb);
        }
    };
    Task tasks[TASKS];
    const int here0 = min(L.chunk, L.ncb);
    int n_tasks = 0;
    if constexpr (!CHANNELS) {
        first_task();
        n_tasks = load_tasks(tasks, 0, here0);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- weights: the words of the first pair (and of the second, where a pair is too little work to hide a load) ----
    const uint32_t words_lds = tile_lds + (uint32_t)L.ncb * plane;          // (INDEXED: all channel blocks are expanded at once)
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(L.wq, (uint32_t)(L.n_cob * L.pairs) * RF_PAIR_BYTES);
    constexpr bool AHEAD = PB * CB == 2;
    uint32_t A[CB][9], An[AHEAD ? CB : 1][9];
    auto load_words = [&](int pr, int cb, int piece, uint32_t (&a)[9]) {       // (past the last pair or block: the last one, not used)
        if constexpr (INDEXED) {
            const uint32_t at = words_lds + (uint32_t)((wco * CB + cb) * L.pairs + min(pr, L.pairs - 1)) * RF_PAIR_BYTES;
            if (piece < 2) {
                const u32x4 v = *(lds_cu32x4 *)(uintptr_t)(at + 1024u * piece + (uint32_t)lane * 16u);
#pragma unroll
                for (int i = 0; i < 4; ++i) a[4 * piece + i] = v[i];
            } else {
                a[8] = *(lds_u32 *)(uintptr_t)(at + 2048u + (uint32_t)lane * 4u);
            }
            return;
        }
        const uint32_t at = (uint32_t)(min(cob0 + cb, L.n_cob - 1) * L.pairs + min(pr, L.pairs - 1)) * RF_PAIR_BYTES;
        if (piece < 2) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(wres, lane * 16, (int)(at + 1024u * piece), 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) a[4 * piece + i] = v[i];
        } else {
            a[8] = __builtin_amdgcn_raw_buffer_load_b32(wres, lane * 4, (int)(at + 2048u), 0);
        }
    };
    auto first_words = [&]() {
#pragma unroll
        for (int piece = 0; piece < 3; ++piece)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) load_words(0, cb, piece, A[cb]);
        if constexpr (AHEAD) {
#pragma unroll
            for (int piece = 0; piece < 3; ++piece)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) load_words(1, cb, piece, An[cb]);
        }
    };
    if constexpr (INDEXED) {
        // as rows_fp4_prep_kernel: a pass of the 256 threads is 32 output channels x a pair of channel blocks
        const uint32_t codes_lds = words_lds + (uint32_t)((CB << (2 - L.wpx_shift)) * L.pairs) * RF_PAIR_BYTES;
        const __amdgpu_buffer_rsrc_t ires = make_rsrc(L.idx, (uint32_t)(L.C_out * L.C_in) * 2u);
        const int d = tid & 3, co = (tid >> 2) & 31, first_cob = (cot << (2 - L.wpx_shift)) * CB;
        const int n_pass = min(CB << (2 - L.wpx_shift), L.n_cob - first_cob) * L.pairs;
        int c = 0, pr = 0;                                     // block of output channels (of the workgroup's), pair, of the next load
        auto load_idx = [&](uint32_t (&k)[8]) {                // (past the last one: of no use)
            const int oc = (first_cob + c) * 32 + co, c0 = (2 * pr + (tid >> 7)) * 32 + d * 8;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                k[j] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(
                    ires, (int)(oc < L.C_out && c0 + j < L.C_in ? (uint32_t)(oc * L.C_in + c0 + j) * 2u : OFF_NONE), 0, 0);
            if (++pr == L.pairs) {
                pr = 0;
                ++c;
            }
        };
        uint32_t k[8], kn[8];
        load_idx(k);
        for (int i = tid; i < L.K; i += 256) *(lds_u16 *)(uintptr_t)(codes_lds + 2u * (uint32_t)i) = L.codebook[i] & 511u;
        __syncthreads();
        for (int i = 0; i < n_pass; ++i) {
            const int cb = 2 * (i % L.pairs) + (tid >> 7);
            load_idx(kn);
            uint32_t code[8], w[9];
#pragma unroll
            for (int j = 0; j < 8; ++j) code[j] = *(lds_u16 *)(uintptr_t)(codes_lds + 2u * min(k[j], (uint32_t)L.K - 1u));
            words_of_codes(code, d, w);
            const uint32_t at = words_lds + (uint32_t)i * RF_PAIR_BYTES;
            if (d == 0 && cb < L.ncb)
                put_words([&](int o, u32x4 v) { *(lds_u32x4 *)(uintptr_t)(at + (uint32_t)o) = v; },
                          [&](int o, uint32_t v) { *(lds_u32 *)(uintptr_t)(at + (uint32_t)o) = v; }, co, cb, L.ncb, w);
#pragma unroll
            for (int j = 0; j < 8; ++j) k[j] = kn[j];
        }
    } else {
        if (active) first_words();
    }
    // scales of the workgroup's channels (4 CB blocks at most)
    float early_scale[2] = {0.0f, 0.0f};
    const int scale_first = (cot << (2 - L.wpx_shift)) * CB * 32;
    const bool has_scale = tid < (CB * 32 << (2 - L.wpx_shift)) && scale_first + tid < 32 * L.n_cob;
    {
        // (the 1-bit layer's, and of a layer given as indices, are alpha itself: channels past C_out lie beyond the buffer and read 0)
        const __amdgpu_buffer_rsrc_t sres = make_rsrc(L.scale, CHANNELS || INDEXED ? (uint32_t)L.C_out * 4u : (uint32_t)L.n_cob * 256u);
        const uint32_t off = has_scale ? (uint32_t)(scale_first + tid) * 4u : OFF_NONE;
        early_scale[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(sres, (int)off, 0, 0));
        if constexpr (SIGN) early_scale[1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(sres, (int)off, (int)((uint32_t)L.n_cob * 128u), 0));
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- the lane's windows -----------------------------------------------------------------------------------------
    uint32_t top[PB];                                          // LDS address of the window's first pixel, channel block 0
    uint32_t yoff[PB];                                         // byte offset of y[n - n0][4 h][pixel]
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        int n, ho, wo;
        const bool ok = pixel_of(blk0 + pb, n_l, n, ho, wo);
        const bool mine = blk0 + pb < L.n_blk;                 // (a block past the last one: any pixel of the tile)
        top[pb] = tile_lds + (mine ? (uint32_t)((n * H1 + ho * L.stride - R0) * W1 + wo * L.stride) * 16u : 0u);
        yoff[pb] = ok ? (uint32_t)(((n - n0) * L.C_out + 4 * h) * L.HoWo + ho * L.Wo + wo) * 4u : OFF_NONE;
    }
    v16f acc[CB][PB];
    // (the two constants in registers: an instruction of two operations takes no literals)
    uint32_t sign_bits = 0x88888888u, one_bits = 0x22222222u;
    asm("" : "+v"(sign_bits));
    asm("" : "+s"(one_bits));
    auto expand = [&](uint32_t w, u32x4 &a) {
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] = ((w << (3 - r)) & sign_bits) | one_bits;
    };
    auto multiply = [&](const u32x4 &a, const u32x4 &b, v16f &sum) {
        const v8i av = {(int)a[0], (int)a[1], (int)a[2], (int)a[3], 0, 0, 0, 0};
        const v8i bv = {(int)b[0], (int)b[1], (int)b[2], (int)b[3], 0, 0, 0, 0};
        sum = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, sum, 4, 4, 0, 0, 0, 0);
    };

    if constexpr (CHANNELS) fill_channels(0, here0);
    else fill(tasks, n_tasks, 0, here0);
    if (has_scale) {
        *(lds_f32 *)(uintptr_t)(lds0 + (uint32_t)tid * 4u) = early_scale[0];
        if constexpr (SIGN) *(lds_f32 *)(uintptr_t)(lds0 + 4u * CB * 32u * 4u + (uint32_t)tid * 4u) = early_scale[1];
    }
    if constexpr (!SIGN) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[cb][pb][r] = 0.0f;
    }
    const uint32_t scale_lane = lds0 + (uint32_t)(wco * CB * 32 + 4 * h) * 4u;
    int pair = 0;                                              // of the whole layer
    for (int cb_first = 0; cb_first < L.ncb; cb_first += L.chunk) {
        const int here = min(L.chunk, L.ncb - cb_first);
        if (cb_first > 0) {
            __syncthreads();                                   // the previous blocks are no longer read
            if constexpr (CHANNELS) {
                fill_channels(cb_first, here);
            } else {
                // (beside the accumulators there are registers for one task: with the loads of the next in flight the tiles spill 3 to
                // 35, measured 64 -> 512 13x13 43 -> 52 us, 256 -> 256 14x14 batch 128 13.9 -> 18.5, and where it spilled nothing, four
                // pixel blocks alone, 512 -> 512 28x28 batch 64 57.5 -> 58.0)
                Task one[1];
                first_task();
                const int n = load_tasks(one, cb_first, here);
                fill(one, n, cb_first, here);
            }
        }
        __syncthreads();
        if (!active) continue;
        if constexpr (INDEXED) first_words();
        if constexpr (SIGN) {
            if (cb_first == 0) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 c0 = *(lds_cf32x4 *)(uintptr_t)(scale_lane + (uint32_t)(cb * 32 + 8 * q) * 4u);
#pragma unroll
                        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                            for (int i = 0; i < 4; ++i) acc[cb][pb][4 * q + i] = c0[i];
                    }
            }
        }
        // (opaque here: the addresses made of it would be kept in registers through the fill)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) asm volatile("" : "+v"(top[pb]));
        // (the weights have been here since the fill: said so before the loop, its own waits count only what it has in flight)
        __builtin_amdgcn_s_waitcnt(0x0f70 /* vmcnt(0) */);
        const int np = here >> 1;
        // A step is the matrix instructions of a tap.  A wave issues an instruction every four or five clocks whichever unit it
        // is for, so a step of 32 PB CB matrix clocks has room for some 7 PB CB others: 7 per word of weights to expand, a read
        // per pixel block, an address per row.  The reads are issued two steps ahead (three buffers, and nine taps are a multiple
        // of three): one step of two matrix instructions is shorter than a read takes.  Measured against three instructions per four
        // expanded slots, reads one step ahead and, for small grids, two blocks of output channels per wave on one of pixels: ResNet-18's
        // chain of 1-bit layers at batch 64 167 -> 156 us, 512 -> 512 7x7 batch 8 12.2 -> 10.1.
        u32x4 B[3][PB], E[CB];
        // A step of four pixel blocks has matrix work for its reads and additions in any order; its registers are all taken: one
        // address per pixel block there, and the order of the instructions is the compiler's.  (With three and an order laid down it
        // spilled 14, and a wave that has any scratch memory starts later: 64 -> 512 13x13 batch 256 52.4 -> 43.4 us, 100 -> 150 31x31
        // 66 -> 54, 256 -> 256 28x28 73 -> 64; the smaller tiles kept values of the last block alone, below, and spilled two.)
        constexpr int ROWS = PB == 4 ? 1 : 3;
        uint32_t row[ROWS][PB];                                // LDS addresses of the window's rows, or of the first
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            row[0][pb] = top[pb] + (uint32_t)h * plane;
#pragma unroll
            for (int i = 1; i < ROWS; ++i) row[i][pb] = row[i - 1][pb] + pitch;
        }
        auto read = [&](auto tc) {
            constexpr int t = decltype(tc)::value;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
                B[t % 3][pb] = *(lds_cu32x4 *)(uintptr_t)((ROWS == 3 ? row[t / 3 % ROWS][pb] : row[0][pb] + (uint32_t)(t / 3) * pitch) +
                                                          (uint32_t)(t % 3) * 16u);
        };
        if (np > 0) {
            read(std::integral_constant<int, 0>{});
            read(std::integral_constant<int, 1>{});
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) expand(A[cb][0], E[cb]);
        }
        // (W: the words of this pair; V: those of the next where they are kept beside these)
        auto step = [&](auto tc, uint32_t next, auto &W, auto &V) {
            constexpr int t = decltype(tc)::value;
            if constexpr (ROWS == 1 && t == 7) {
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) row[0][pb] += next;
            }
            read(std::integral_constant<int, (t + 2) % 9>{});
            if constexpr (ROWS == 3 && (t == 0 || t == 3)) {   // a row's three taps have been read: on to the next pair
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) row[t / 3][pb] += next;
            }
            if constexpr (ROWS == 3 && t == 6) {
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) row[2][pb] += next;
            }
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) multiply(E[cb], B[t % 3][pb], acc[cb][pb]);
                if constexpr (AHEAD && t == 8) expand(V[cb][0], E[cb]);
                else expand(W[cb][(t + 1) % 9], E[cb]);
            }
            // new words as soon as the old ones have been expanded: those of the next pair, at least five steps ahead, or of the one
            // after it
            if constexpr (!AHEAD && (t == 3 || t == 7 || t == 8)) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) load_words(pair + 1, cb, t == 3 ? 0 : t == 7 ? 1 : 2, W[cb]);
            }
            if constexpr (AHEAD && t == 8) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int piece = 0; piece < 3; ++piece) load_words(pair + 2, cb, piece, W[cb]);
            }
            if constexpr (PB != 4) {
                __builtin_amdgcn_sched_group_barrier(0x100 /* LDS reads */, PB, 0);
#pragma unroll
                for (int i = 0; i < PB * CB; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008 /* matrix */, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002 /* vector */, 7 / PB + 1, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto run_pair = [&](auto &W, auto &V, bool last) {
            const uint32_t next = last ? 0u : 2u * plane;
            step(std::integral_constant<int, 0>{}, next, W, V);
            step(std::integral_constant<int, 1>{}, next, W, V);
            step(std::integral_constant<int, 2>{}, next, W, V);
            step(std::integral_constant<int, 3>{}, next, W, V);
            step(std::integral_constant<int, 4>{}, next, W, V);
            step(std::integral_constant<int, 5>{}, next, W, V);
            step(std::integral_constant<int, 6>{}, next, W, V);
            step(std::integral_constant<int, 7>{}, next, W, V);
            step(std::integral_constant<int, 8>{}, next, W, V);
            ++pair;
        };
        if constexpr (AHEAD) {
            // two pairs per turn: a copy from one set of words to the other waits for loads just issued (512 -> 512 7x7 batch 64: 4.0 us
            // of multiplication, now 3.5)
            int pr = 0;
            for (; pr + 2 <= np; pr += 2) {
                run_pair(A, An, false);
                run_pair(An, A, pr + 2 == np);
            }
            if (pr < np) {
                run_pair(A, An, true);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        const uint32_t w = A[cb][i];
                        A[cb][i] = An[cb][i];
                        An[cb][i] = w;
                    }
            }
        } else {
            for (int pr = 0; pr < np; ++pr) run_pair(A, A, pr + 1 == np);
        }
        if (here & 1) {
            // the last block alone: two taps per step
            const uint32_t last = (uint32_t)(here - 1) * plane;
            // (opaque: what is chosen by it would be kept in registers all along, and the tiles of two blocks of output channels have none
            // left.  Several layers in one launch spill two for it: the ResNet-18 stack's forward pass 181.4 us with them, 183.4 without)
            int second = h;
            if constexpr (CB == 2 && TASKS == 4) asm volatile("" : "+v"(second));
#pragma unroll
            for (int u = 0; u < 5; ++u) {
                const int t0 = 2 * u, t1 = u < 4 ? 2 * u + 1 : 0;
                const uint32_t o0 = (uint32_t)(t0 / 3) * pitch + (uint32_t)(t0 % 3) * 16u;
                const uint32_t o1 = (uint32_t)(t1 / 3) * pitch + (uint32_t)(t1 % 3) * 16u;
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    const uint32_t at = u == 4 && second ? tile_lds : top[pb] + (second ? o1 : o0);      // (the tile's first pixel is zero)
                    B[0][pb] = *(lds_cu32x4 *)(uintptr_t)(at + last);
                }
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    expand(A[cb][u], E[cb]);
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb) multiply(E[cb], B[0][pb], acc[cb][pb]);
                }
            }
        }
    }
    if (!active) return;

    if constexpr (SIGN) {
        // ---- the next layer's sign: bit = (fl(fl(S alpha) + beta) >= 0), packed rows ---------------------------------
        // The accumulators began at the channel's threshold (sign_entry): a bit is a sign bit.  A lane collects those of its pixel,
        // sixteen channels of a block, two blocks to a word, one instruction each; a transposition of 32 x 32 bits over the
        // lanes of a half (fifteen instructions) gives each lane the word of a channel.  (The two roundings, a ballot and its two words
        // written to lanes were five instructions per register, 1.2 to 2.1 us of a layer's 8 to 13: 1-bit chain of ResNet-18 batch 64
        // 148 us, now 132.)
        uint32_t *const out = (uint32_t *)L.out;
        const int WWo = (L.Wo + 31) / 32;
        const uint32_t oplane = (uint32_t)(L.Ho * WWo);
        const bool short_rows = L.Wo <= 32;
        const uint32_t sel16 = lane & 16 ? 0x07060302u : 0x05040100u, sel8 = lane & 8 ? 0x03070105u : 0x06020400u;
        const uint32_t keep4 = lane & 4 ? 0xf0f0f0f0u : 0x0f0f0f0fu, keep2 = lane & 2 ? 0xccccccccu : 0x33333333u,
                       keep1 = lane & 1 ? 0xaaaaaaaau : 0x55555555u;
        const uint32_t turn4 = lane & 4 ? 4u : 28u, turn2 = lane & 2 ? 2u : 30u, turn1 = lane & 1 ? 1u : 31u;
        auto stage = [](uint32_t x, uint32_t y, uint32_t keep, uint32_t turn) {
            const uint32_t r = __builtin_amdgcn_alignbit(y, y, turn);
            return (x & keep) | (r & ~keep);
        };
        auto transpose = [&](uint32_t x) {                     // bit p of lane l: bit l of lane p
            const auto swapped = __builtin_amdgcn_permlane16_swap(x, x, false, false);       // lanes 0..15 twice, lanes 16..31 twice
            x = __builtin_amdgcn_perm(swapped[1], swapped[0], sel16);
            uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128 /* row_ror:8 */, 0xF, 0xF, true);
            x = __builtin_amdgcn_perm(y, x, sel8);
            y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141 /* row_half_mirror */, 0xF, 0xF, true);
            y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y, 0x1B /* quad_perm [3,2,1,0] */, 0xF, 0xF, true);
            x = stage(x, y, keep4, turn4);
            y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E /* quad_perm [2,3,0,1] */, 0xF, 0xF, true);
            x = stage(x, y, keep2, turn2);
            y = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1 /* quad_perm [1,0,3,2] */, 0xF, 0xF, true);
            return stage(x, y, keep1, turn1);
        };
        // lane l of a half: sixteen bits further up come first
        const int late = n_l < 16, r = 15 - (n_l & 15);        // of the two blocks of sixteen registers: which, register
        const int chan = 8 * (r >> 2) + 4 * h + (r & 3);
        const int cb_of = CB == 2 ? late : 0;
        const int co = (cob0 + cb_of) * 32 + chan;
        const uint32_t flip = *(lds_u32 *)(uintptr_t)(lds0 + (uint32_t)(4 * CB * 32 + (wco * CB + cb_of) * 32 + chan) * 4u);
#pragma unroll
        for (int u = 0; u < (CB == 2 ? PB : (PB + 1) / 2); ++u) {
            uint32_t bits = 0;
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                if (CB == 1 && 2 * u + v >= PB) {
                    bits <<= 16;
                    break;
                }
                const v16f &a = CB == 2 ? acc[v][u] : acc[0][2 * u + v];
#pragma unroll
                for (int i = 0; i < 16; ++i) bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(a[i]), 31);
            }
            bits = transpose(bits) ^ flip;
            const int Bk = blk0 + (CB == 2 ? u : 2 * u + late);
            if (Bk >= L.n_blk || (CB == 1 && 2 * u + late >= PB) || co >= L.C_out) continue;
            int bn, bword, bwords;                             // image, first word in a channel plane, words
            if (short_rows) {
                bn = (int)div((uint32_t)Bk, L.div_bpi);
                bword = (Bk - bn * L.bpi) * L.rows_pb;
                bwords = min(L.rows_pb, L.Ho - bword);
            } else {
                const int R = (int)div((uint32_t)Bk, L.div_wpr);
                bn = (int)div((uint32_t)R, L.div_Ho);
                const int word = Bk - R * L.wpr;
                bword = (R - bn * L.Ho) * WWo + word;
                bwords = 1;
                if (32 * (word + 1) > L.Wo) bits &= (1u << (L.Wo & 31)) - 1u;
            }
            uint32_t *const dst = out + (int64_t)(bn * L.C_out + co) * oplane + bword;
            if (!short_rows || L.Wo == 32) {
                dst[0] = bits;
            } else {
                const uint32_t wmask = (1u << L.Wo) - 1u;
                for (int j = 0; j < bwords; ++j, bits >>= L.Wo) dst[j] = bits & wmask;
            }
        }
        return;
    }
    // ---- y = alpha * S -------------------------------------------------------------------------------------------------
    // Lanes 0..31 of a register are 32 consecutive pixels of one channel; register r is channel 8 (r / 4) + 4 h + r % 4.
    const uint32_t chan = (uint32_t)L.HoWo * 4u;
    const __amdgpu_buffer_rsrc_t yres = images(L.out, L.C_out, chan);
    auto store = [&](auto policy) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int co0 = (cob0 + cb) * 32;
            const bool whole = co0 + 32 <= L.C_out;            // (wave-uniform)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 al = *(lds_cf32x4 *)(uintptr_t)(scale_lane + (uint32_t)(cb * 32 + 8 * q) * 4u);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int c = co0 + 8 * q + i;             // wave-uniform part of the channel
                    if (!whole && c + 4 * h >= L.C_out) continue;
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb)
                        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[cb][pb][4 * q + i] * al[i]), yres, (int)yoff[pb],
                                                              (int)((uint32_t)c * chan), decltype(policy)::value);
                }
            }
        }
    };
    if (PACED || L.policy == FP4_STORE_NT) store(std::integral_constant<int, AUX_NT>{});
    else if (TASKS == 4 && L.policy == FP4_STORE_THROUGH) store(std::integral_constant<int, AUX_THROUGH>{});   // (never in a launch of several layers)
    else store(std::integral_constant<int, AUX_CACHED>{});
}

template <int PB, int CB, bool SIGN, bool CHANNELS, bool INDEXED>
__global__ __launch_bounds__(256, PB == 4 ? 2 : PB * CB == 4 ? 3 : 4)
void rows_fp4_kernel(const RfLayer L)
{
    extern __shared__ __align__(16) unsigned char smem[];
    rf_tile<PB, CB, SIGN, CHANNELS, 4, INDEXED>(L, blockIdx.x, smem);
}

// Several layers in one launch (fp32 output): workgroups [first[l], first[l + 1]) run layer l.  The layers share the
// chip: while the workgroups of one layer store their outputs those of another multiply.
// A layer is described in 112 bytes, what follows from those is computed by the workgroup (scalar instructions), so that
// the 4 KB of kernel arguments hold a whole network: with fifteen layers to a launch the sixteenth layer of the ResNet-18
// stack (512 -> 512 7x7, 19 us alone, most of the chip idle) followed in a launch of its own, and a 32-layer stack took three.
struct RfManyLayer {
    const uint32_t *x;
    const uint32_t *wq;                  // the scales lie behind it
    void *y;
    int N, C_in, C_out, H, W, Ho, Wo;
    int plane, n_cotiles, n_wgs;
    uint16_t chunk, pitch;               // (at most 128; rows fit LDS)
    uint8_t PB_CB, wpx_shift, stride, policy;
    Divisor div_HoWo, div_Wo, div_H1, div_WW, div_cotiles;
};
constexpr int RF_MANY_MAX = 34;
struct RfMany {
    int n_layers;
    int fold;                            // groups of eight workgroups come from the two ends of the list in turn
    int first[RF_MANY_MAX + 1];          // multiples of eight (the XCD of a workgroup inside its layer)
    RfManyLayer layer[RF_MANY_MAX];
};
static_assert(sizeof(RfMany) <= 4096, "kernel arguments");

// The layer whose range [first[l], first[l + 1]) block b falls into, n <= 63 layers: the lanes test one bound each.  (A loop over
// the bounds waits for a scalar load per layer.)
__device__ __forceinline__ int layer_of_block(const int *first, int n, int b)
{
    const int lane = threadIdx.x & 63;
    return __builtin_amdgcn_readfirstlane((int)__popcll(__ballot(lane > 0 && lane < n && b >= first[lane < n ? lane : 0])));
}

__host__ __device__ constexpr size_t rf_weight_bytes(int C_out, int C_in)
{
    return ((size_t)((C_out + 31) / 32) * ((C_in + 63) / 64) * RF_PAIR_BYTES + 255) & ~(size_t)255;
}

template <bool PACED>
__global__ __launch_bounds__(256, 3)
void rows_fp4_many_kernel(const RfMany m)
{
    extern __shared__ __align__(16) unsigned char smem[];
    int b = blockIdx.x;
    if (m.fold) {
        const int g = b >> 3, n_g = (int)(gridDim.x >> 3);
        b = ((g & 1 ? n_g - 1 - (g >> 1) : g >> 1) << 3) + (b & 7);
    }
    const int l = layer_of_block(m.first, m.n_layers, b);
    const RfManyLayer &c = m.layer[l];
    const uint32_t wg = (uint32_t)(b - m.first[l]);
    if (wg >= (uint32_t)c.n_wgs) return;                                // padding to a multiple of eight
    RfLayer L = {};
    L.x = c.x;
    L.wq = c.wq;
    L.scale = (const float *)((const char *)c.wq + rf_weight_bytes(c.C_out, c.C_in));
    L.out = c.y;
    L.N = c.N; L.C_in = c.C_in; L.C_out = c.C_out; L.H = c.H; L.W = c.W; L.WW = (c.W + 31) >> 5; L.stride = c.stride;
    L.Ho = c.Ho; L.Wo = c.Wo; L.HoWo = c.Ho * c.Wo; L.P = c.N * L.HoWo;
    L.n_cob = (c.C_out + 31) >> 5; L.ncb = (c.C_in + 31) >> 5; L.chunk = c.chunk; L.pairs = (L.ncb + 1) >> 1; L.pitch = c.pitch; L.plane = c.plane;
    L.n_blk = (L.P + 31) >> 5; L.n_cotiles = c.n_cotiles; L.n_wgs = c.n_wgs; L.wpx_shift = c.wpx_shift;
    L.div_HoWo = c.div_HoWo; L.div_Wo = c.div_Wo; L.div_H1 = c.div_H1; L.div_WW = c.div_WW; L.div_cotiles = c.div_cotiles;
    L.policy = c.policy;
    switch (c.PB_CB) {
    case 22: rf_tile<2, 2, false, false, 2, false, PACED>(L, wg, smem); break;
    case 21: rf_tile<2, 1, false, false, 2, false, PACED>(L, wg, smem); break;
    default: rf_tile<1, 1, false, false, 2, false, PACED>(L, wg, smem); break;
    }
}

// ---- weights -> operand layout ---------------------------------------------------------------------------------------
struct RfWeights {
    uint32_t *wq;
    float *scale;
    int C_in, C_out, n_cob, ncb;
};

// The next layer's sign, fl(fl(S a) + b) >= 0, of the sums S in [-9 C_in, 9 C_in]: monotone in S, so it is a threshold.  Returns the
// accumulator's start, 0.5 - (first sum on the upper side), whose sum with S is never zero and exact, and what the word of
// its sign bits is turned by: the upper side is 1 (a > 0, all ones) or 0 (a < 0).
__device__ inline float2 sign_entry(float a, float b, int C_in)
{
    // (a = 0 or not a number: one bit for every S)
    if (!(a > 0.0f || a < 0.0f)) return make_float2(-1.0e9f, __uint_as_float(mul_then_add(0.0f, a, b) >= 0.0f ? 0u : 0xffffffffu));
    return make_float2(0.5f - (float)sign_threshold(a, b, 9 * C_in), __uint_as_float(a > 0.0f ? 0xffffffffu : 0u));
}

__device__ __forceinline__ void store_scales(const RfWeights &W, int cob, int c, const float *alpha, const float *beta)
{
    const int co = cob * 32 + c;
    const bool real = co < W.C_out;
    const float a = real ? alpha[co] : 0.0f;
    const float2 e = beta ? sign_entry(a, real ? beta[co] : 0.0f, W.C_in) : make_float2(a, 0.0f);
    W.scale[co] = e.x;
    W.scale[32 * W.n_cob + co] = e.y;
}

// From indices (uint16, or tau bits each in a stream): 256 threads = 2 channel blocks x 32 output channels x 4 groups of 8
// input channels (slots 8 d + j of a word are bits 4 j + d: the four groups of a word are four lanes).
__global__ __launch_bounds__(256)
void rows_fp4_prep_kernel(const RfWeights W, const uint16_t *__restrict__ codebook, int K, const void *__restrict__ idx, int tau,
                          const float *__restrict__ alpha, const float *__restrict__ beta)
{
    __shared__ uint16_t codes[512];
    const int tid = threadIdx.x;
    const int d = tid & 3, co = (tid >> 2) & 31;
    const int cob = blockIdx.x, cb = 2 * blockIdx.y + (tid >> 7);
    const int c0 = cb * 32 + d * 8, oc = cob * 32 + co;
    uint32_t k[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) k[j] = oc < W.C_out && c0 + j < W.C_in ? index_at(idx, (int64_t)oc * W.C_in + c0 + j, tau) : 0u;
    for (int i = tid; i < K; i += 256) codes[i] = codebook[i] & 511u;
    __syncthreads();
    if (blockIdx.y == 0 && tid < 32) store_scales(W, cob, tid, alpha, beta);
    if (cb >= W.ncb) return;
    uint32_t code[8], w[9];
#pragma unroll
    for (int j = 0; j < 8; ++j) code[j] = codes[min(k[j], (uint32_t)K - 1u)];
    words_of_codes(code, d, w);
    if (d == 0) store_words(W.wq, cob, co, cb, W.ncb, w);
}

// The 1-bit layer's: bit planes of 9-bit kernel codes.  A wave takes an output channel and a pair of channel blocks.
__global__ __launch_bounds__(256)
void rows_fp4_prep_planes_kernel(const RfWeights W, const uint16_t *__restrict__ w9)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int oc = blockIdx.x * 4 + wave, pr = blockIdx.y;             // (the grid covers whole blocks of output channels)
    const int c = 64 * pr + lane;
    const uint32_t code = oc < W.C_out && c < W.C_in ? w9[(int64_t)oc * W.C_in + c] : 0u;
    uint32_t w[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const unsigned long long m = __ballot((code >> (8 - t)) & 1u);
        w[t] = (uint32_t)(lane & 1 ? m >> 32 : m);
    }
    const int cb = 2 * pr + lane;
    if (lane < 2 && cb < W.ncb) store_words(W.wq, oc >> 5, oc & 31, cb, W.ncb, w);
}

// From real-valued kernels: the projection of Eq. 2 / Eq. 5 (idx_out as snn_project_kernels writes it) and the operand
// layout.  A workgroup takes 32 output channels x 32 input channels; thread (co, e) the four kernels 4 e .. 4 e + 3 of
// its output channel, so that eight threads read 1152 contiguous bytes and make one word per tap.
struct RfProject {
    RfWeights W;
    const float *w;            // [C_out][C_in][9]
    const uint16_t *codebook;
    const float *alpha;
    const float *beta;         // or nullptr
    uint16_t *idx_out;         // [C_out][C_in]
    int K;
};
constexpr int RF_PROJECT_LDS_WORDS = 64 * 12 + 32;

__device__ __forceinline__ void rf_project_block(const RfProject &p, int block, uint32_t *lds)
{
    const RfWeights &W = p.W;
    const int tid = threadIdx.x;
    const int cob = block / W.ncb, cb = block - cob * W.ncb;
    const int co = tid >> 3, e = tid & 7;
    const int oc = cob * 32 + co, c0 = cb * 32 + 4 * e;
    const int have = oc < W.C_out ? max(0, min(4, W.C_in - c0)) : 0;
    const int64_t at = (int64_t)oc * W.C_in + c0;
    float wt[4][9];
    if (have == 4 && (((uintptr_t)(p.w + at * 9)) & 15) == 0) {
        const float4 *src = (const float4 *)(p.w + at * 9);
        float flat[36];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const float4 v = src[i];
            flat[4 * i] = v.x;
            flat[4 * i + 1] = v.y;
            flat[4 * i + 2] = v.z;
            flat[4 * i + 3] = v.w;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < 9; ++t) wt[q][t] = flat[9 * q + t];
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < 9; ++t) wt[q][t] = q < have ? p.w[(at + q) * 9 + t] : 0.0f;
    }
    float *coef = (float *)lds;
    uint16_t *codes = (uint16_t *)(lds + 64 * 12);
    project_fill_coef(coef, p.codebook, p.K, tid, 256);
    for (int i = tid; i < p.K; i += 256) codes[i] = p.codebook[i] & 511u;
    if (cb == 0 && tid < 32) store_scales(W, cob, tid, p.alpha, p.beta);
    __syncthreads();
    int best[4] = {0, 0, 0, 0};
    if (__builtin_amdgcn_readfirstlane(__ballot(have > 0) != 0ull)) project_argmax<4>(wt, coef, p.K, best);
    if (have == 4 && (((uintptr_t)(p.idx_out + at)) & 7) == 0) {
        *(uint2 *)(p.idx_out + at) = make_uint2((uint32_t)best[0] | (uint32_t)best[1] << 16, (uint32_t)best[2] | (uint32_t)best[3] << 16);
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q < have) p.idx_out[at + q] = (uint16_t)best[q];
    }
    uint32_t lo = 0, mid = 0, hi = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t c = codes[best[q]];
        lo |= (c & 15u) << (4 * q);
        mid |= ((c >> 4) & 15u) << (4 * q);
        hi |= (c >> 8) << (4 * q);
    }
    uint32_t words[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) words[t] = or_of_eight_lanes(tap_bits(lo, mid, hi, t) << (16 * (e & 1) + (e >> 1)));
    if (e == 0) store_words(W.wq, cob, co, cb, W.ncb, words);
}

// The weights-side work of up to RF_PROJECT_MAX layers in one launch.
constexpr int RF_PROJECT_MAX = 32;
struct RfProjectMany {
    int n_layers;
    int first[RF_PROJECT_MAX + 1];
    RfProject layer[RF_PROJECT_MAX];
};
static_assert(sizeof(RfProjectMany) <= 4096, "kernel arguments");

__global__ __launch_bounds__(256)
void rows_fp4_project_many_kernel(const RfProjectMany m)
{
    __shared__ __align__(16) uint32_t lds[RF_PROJECT_LDS_WORDS];
    const int b = blockIdx.x;
    int l = 0;
    while (l + 1 < m.n_layers && b >= m.first[l + 1]) ++l;              // block-uniform
    rf_project_block(m.layer[l], b - m.first[l], lds);
}

// The first launch of a layer's forward pass: projection + operand layout, and sign + packing of the activations.
struct RfFront {
    RfProject pr;
    int project_blocks;
    const float *x;            // activations [rows][W]; none when the input is packed already
    uint32_t *xr;
    int64_t rows;
    int W, WW, rows_per_block, vec;
};

__global__ __launch_bounds__(256)
void rows_fp4_front_kernel(const RfFront p)
{
    static_assert(PACK_THREADS == 256 && PACK_LDS_WORDS <= RF_PROJECT_LDS_WORDS, "one block size and buffer for both roles");
    __shared__ __align__(16) uint32_t lds[RF_PROJECT_LDS_WORDS];
    const int b = blockIdx.x;
    if (b >= p.project_blocks) {
        pack_rows_block(p.x, p.xr, p.rows, p.W, p.WW, p.rows_per_block, p.vec, (int64_t)(b - p.project_blocks), lds);
        return;
    }
    rf_project_block(p.pr, b, lds);
}

// The first launch of a stack's forward pass: the same for every layer.  Projection is vector-unit work and packing a stream
// from memory; in one launch, with the projection's workgroups spread over the first seven eighths of the grid, the
// one runs beside the other.  Whole forward call of the ResNet-18 stack, one launch after the other -> together: batch 64 185 -> 180 us,
// batch 16 74 -> 66 us, batch 2 43 -> 39 us; all projections within the first tenth instead: 185 and 70 us (they fill the
// chip and the stream waits).  Six waves per SIMD asked for: at the projection's own 86 registers five fit, too few loads in flight for
// the stream (batch 64 182-190 us).
struct RfFrontLayer {
    uint32_t *wq;                        // the scales lie behind it
    const float *w;
    const uint16_t *codebook;
    const float *alpha;
    uint16_t *idx_out;
    const float *x;
    uint32_t *xr;
    int64_t rows;
    int C_in, C_out, K;
    int W, rows_per_block, vec, pack_blocks;
};
constexpr int RF_FRONT_MAX = 35;
struct RfFrontMany {
    int n_layers, run;                   // a packing workgroup takes `run` blocks of rows
    int project_blocks;                  // every `period`-th workgroup projects until they are through
    Divisor period;
    uint32_t period_value;
    int first_project[RF_FRONT_MAX + 1], first_pack[RF_FRONT_MAX + 1];
    RfFrontLayer layer[RF_FRONT_MAX];
};
static_assert(sizeof(RfFrontMany) <= 4096, "kernel arguments");

__global__ __launch_bounds__(256, 6)
void rows_fp4_front_many_kernel(const RfFrontMany m)
{
    static_assert(PACK_THREADS == 256 && 2 * PACK_LDS_WORDS <= RF_PROJECT_LDS_WORDS, "one block size and buffer for both roles");
    __shared__ __align__(16) uint32_t lds[RF_PROJECT_LDS_WORDS];
    const uint32_t b = blockIdx.x;
    const uint32_t turn = fast_div(b, m.period);
    if (turn * m.period_value == b && turn < (uint32_t)m.project_blocks) {
        const int l = layer_of_block(m.first_project, m.n_layers, (int)turn);
        const RfFrontLayer &c = m.layer[l];
        RfProject p;
        p.W = {c.wq, (float *)((char *)c.wq + rf_weight_bytes(c.C_out, c.C_in)), c.C_in, c.C_out, (c.C_out + 31) >> 5, (c.C_in + 31) >> 5};
        p.w = c.w;
        p.codebook = c.codebook;
        p.alpha = c.alpha;
        p.beta = nullptr;
        p.idx_out = c.idx_out;
        p.K = c.K;
        rf_project_block(p, (int)turn - m.first_project[l], lds);
        return;
    }
    const int q = (int)b - min((int)turn + 1, m.project_blocks);
    const int l = layer_of_block(m.first_pack, m.n_layers, q);
    const RfFrontLayer &c = m.layer[l];
    const int b0 = (q - m.first_pack[l]) * m.run, b1 = min(b0 + m.run, c.pack_blocks);
    const int WW = (c.W + 31) >> 5;
    if (c.vec && c.W <= PACK_CHUNK) {
        pack_rows_stream(c.x, c.xr, c.rows, c.W, WW, c.rows_per_block, (int64_t)b0, (int64_t)b1, lds);
        return;
    }
    for (int i = b0; i < b1; ++i) pack_rows_block(c.x, c.xr, c.rows, c.W, WW, c.rows_per_block, c.vec, (int64_t)i, lds);
}

// ---- host side -----------------------------------------------------------------------------------------------------------

struct RfPlan {
    int PB, CB, wpx_shift;
    int n_cob, ncb, chunk;
    int64_t n_blk, n_cotiles, n_wgs;
    int rows_pb, bpi, wpr;
    int64_t rows;                // padded input rows a workgroup touches at most
    int64_t plane;
    int pitch;
    size_t lds;
    bool ok;
};

constexpr size_t RF_LDS_TARGET = 72 * 1024;      // two workgroups per compute unit
constexpr size_t RF_LDS_MAX = 150 * 1024;
constexpr size_t RF_LDS_CU = 160 * 1024;

size_t rf_weight_bytes(const Geom &g) { return rf_weight_bytes(g.C_out, g.C_in); }

RfPlan rf_plan(const Geom &g, bool sign, bool many = false)
{
    RfPlan pl;
    pl.n_cob = (g.C_out + 31) / 32;
    pl.ncb = (g.C_in + 31) / 32;
    pl.rows_pb = g.Wo <= 32 ? 32 / g.Wo : 1;
    pl.bpi = (g.Ho + pl.rows_pb - 1) / pl.rows_pb;
    pl.wpr = (g.Wo + 31) / 32;
    pl.n_blk = !sign ? (g.P + 31) / 32 : g.Wo <= 32 ? (int64_t)g.N * pl.bpi : (int64_t)g.N * g.Ho * pl.wpr;
    pl.ok = false;
    struct Tile { int PB, CB; };
    for (const Tile &t : pl.n_cob >= 2 ? std::initializer_list<Tile>{{4, 2}, {2, 2}, {2, 1}} : std::initializer_list<Tile>{{2, 1}, {1, 1}}) {
        const int PB = t.PB;
        // waves of a workgroup share its expanded pixels between as many output channels as there are
        const int wpx_shift = t.CB == 2 ? (pl.n_cob >= 3 ? 1 : 2) : pl.n_cob >= 3 ? 0 : pl.n_cob == 2 ? 1 : 2;
        const int cob_wg = t.CB << (2 - wpx_shift);
        const int64_t n_cotiles = (pl.n_cob + cob_wg - 1) / cob_wg;
        const int64_t nb = (int64_t)PB << wpx_shift;           // pixel blocks of a workgroup
        const int64_t wgs = (pl.n_blk + nb - 1) / nb * n_cotiles;
        // four blocks per wave halve the weight traffic; smaller tiles where that leaves compute units without work (half a tile
        // is one block of output channels, not one of pixels: the weights a wave expands are used twice)
        if (PB == 4 && (wgs < 512 || many)) continue;
        if (PB == 2 && wgs < 256 && !many && t.CB == (pl.n_cob >= 2 ? 2 : 1)) continue;
        // rows the workgroup's pixels touch, and their three-row windows
        int64_t row_changes, image_changes;
        if (!sign) {
            row_changes = (g.Wo - 1 + 32 * nb - 1) / g.Wo;
            image_changes = ((int64_t)g.HoWo - 1 + 32 * nb - 1) / g.HoWo;
        } else {
            row_changes = (g.Wo <= 32 ? nb * pl.rows_pb : (pl.wpr - 1 + nb - 1) / pl.wpr + 1) - 1;
            image_changes = (row_changes + g.Ho - 1) / g.Ho;
        }
        int64_t rows = g.stride * row_changes + image_changes + 3;
        if (rows > (int64_t)g.N * (g.H + 1) + 1) rows = (int64_t)g.N * (g.H + 1) + 1;
        const size_t fixed = (size_t)4 * t.CB * 32 * (sign ? 8 : 4);
        auto plane_of = [&](int pitch) { return (rows * pitch + 1) * 16; };
        int chunk = pl.ncb, pitch = g.W + 1;
        while (chunk > 2 && fixed + (size_t)chunk * plane_of(pitch) > RF_LDS_TARGET) chunk = ((chunk + 1) / 2 + 1) & ~1;
        if (fixed + (size_t)chunk * plane_of(pitch) > RF_LDS_MAX) continue;
        // Of an odd pitch the sixteen rows whose pixels a wave writes at a time lie on different banks of LDS (at 8 or 16 pixels they
        // are on two groups of them or one, 16 clocks per write instruction for 3): taken where it leaves as many workgroups beside
        // each other, of more than three only three.  (The registers of the half tiles allow four, and the pitch is worth more than the
        // fourth: 512 -> 512 7x7 stride 2 batch 64 14.2 us, with four 15.0, batch 256 14.8 and 15.8.)
        auto resident = [&](int p) { return std::min<int64_t>(3, (int64_t)RF_LDS_CU / (int64_t)(fixed + (size_t)chunk * plane_of(p))); };
        if (pitch % 2 == 0 && resident(pitch + 1) == resident(pitch) && fixed + (size_t)chunk * plane_of(pitch + 1) <= RF_LDS_TARGET) ++pitch;
        const int64_t plane = plane_of(pitch);
        pl.PB = PB;
        pl.CB = t.CB;
        pl.wpx_shift = wpx_shift;
        pl.n_cotiles = n_cotiles;
        pl.rows = rows;
        pl.plane = plane;
        pl.pitch = pitch;
        pl.chunk = chunk;
        pl.lds = fixed + (size_t)chunk * plane;
        pl.n_wgs = wgs;
        pl.ok = true;
        break;
    }
    if (!pl.ok) return pl;
    // 32-bit offsets: packed rows and outputs of the images a workgroup touches, the weights, pixel and tile numbers
    const int64_t images = (pl.rows + g.H) / (g.H + 1) + 1;
    const int64_t lim = ((int64_t)1 << 31) - 4096;
    if (images * g.C_in * g.H * g.WW * 4 >= lim || images * g.C_out * g.HoWo * 4 >= lim || (int64_t)rf_weight_bytes(g) >= lim ||
        (int64_t)g.N * g.C_out >= lim || g.P >= lim - 65536 || (int64_t)g.N * (g.H + 1) >= lim || pl.n_blk * 32 >= lim || pl.n_wgs >= lim ||
        (int64_t)g.C_out * g.HoWo * 4 >= lim || pl.ncb > 2 * 65535 /* grid of the preparation */)
        pl.ok = false;
    return pl;
}

RfLayer rf_layer(const RfPlan &pl, const Geom &g, const void *x, void *out, void *ws)
{
    RfLayer L = {};
    L.x = (const uint32_t *)x;
    L.wq = (const uint32_t *)ws;
    L.scale = (const float *)((char *)ws + rf_weight_bytes(g));
    L.out = out;
    L.N = g.N; L.C_in = g.C_in; L.C_out = g.C_out; L.H = g.H; L.W = g.W; L.WW = g.WW; L.stride = g.stride;
    L.Ho = g.Ho; L.Wo = g.Wo; L.HoWo = g.HoWo; L.P = (int)g.P;
    L.n_cob = pl.n_cob; L.ncb = pl.ncb; L.chunk = pl.chunk; L.pairs = (pl.ncb + 1) / 2; L.pitch = pl.pitch; L.plane = (int)pl.plane;
    L.n_blk = (int)pl.n_blk; L.n_cotiles = (int)pl.n_cotiles; L.n_wgs = (int)pl.n_wgs;
    L.wpx_shift = pl.wpx_shift;
    L.policy = store_policy(g, out);
    L.rows_pb = pl.rows_pb; L.bpi = pl.bpi; L.wpr = pl.wpr;
    L.div_HoWo = make_divisor((uint32_t)g.HoWo);
    L.div_Wo = make_divisor((uint32_t)g.Wo);
    L.div_H1 = make_divisor((uint32_t)g.H + 1u);
    L.div_WW = make_divisor((uint32_t)g.WW);
    L.div_cotiles = make_divisor((uint32_t)pl.n_cotiles);
    L.div_bpi = make_divisor((uint32_t)pl.bpi);
    L.div_wpr = make_divisor((uint32_t)pl.wpr);
    L.div_Ho = make_divisor((uint32_t)g.Ho);
    L.div_W1 = make_divisor((uint32_t)pl.pitch);
    return L;
}

RfWeights rf_weights(const Geom &g, void *ws)
{
    RfWeights W;
    W.wq = (uint32_t *)ws;
    W.scale = (float *)((char *)ws + rf_weight_bytes(g));
    W.C_in = g.C_in;
    W.C_out = g.C_out;
    W.n_cob = (g.C_out + 31) / 32;
    W.ncb = (g.C_in + 31) / 32;
    return W;
}

template <int PB, int CB, bool SIGN, bool CHANNELS, bool INDEXED = false>
int launch_rf_one(const RfPlan &pl, const RfLayer &L, hipStream_t s)
{
    auto kern = rows_fp4_kernel<PB, CB, SIGN, CHANNELS, INDEXED>;
    static LdsGrant grant;
    if (grant_dynamic_lds((const void *)kern, pl.lds, grant) != SNN_OK) return SNN_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)pl.n_wgs), dim3(256), pl.lds, s, L);
    return check_launch();
}

template <bool SIGN, bool CHANNELS = false>
int launch_rf(const RfPlan &pl, const RfLayer &L, hipStream_t s)
{
    if (pl.CB == 2) {
        if (pl.PB == 4) return launch_rf_one<4, 2, SIGN, CHANNELS>(pl, L, s);
        return launch_rf_one<2, 2, SIGN, CHANNELS>(pl, L, s);
    }
    if (pl.PB == 2) return launch_rf_one<2, 1, SIGN, CHANNELS>(pl, L, s);
    return launch_rf_one<1, 1, SIGN, CHANNELS>(pl, L, s);
}

// One launch for a layer whose weights come as indices: every workgroup makes the words it needs, in passes of 32 output channels x 64
// input channels of about 0.75 us each.  Against a launch of its own (us per call, two launches -> one, K = 32, workgroups in brackets):
//   one pass      16 -> 16 32x32 batch 8 (64) 8.9 -> 6.4, batch 128 (512) 8.9 -> 7.4, batch 256 (1024) 10.0 -> 9.1, batch 384 (1536)
//                 12.6 -> 13.0, batch 512 (2048) 13.6 -> 14.6; 33 -> 20 28x28 batch 384 (1176) 12.7 -> 12.5
//   two           64 -> 64 8x8 batch 256 (128) 9.2 -> 7.8, batch 512 (256) 9.4 -> 8.0, batch 768 (384) 9.4 -> 10.0; 128 -> 32 28x28
//                 batch 32 (196) 9.3 -> 8.0, batch 64 (392) 9.3 -> 10.2
//   four, eight   64 -> 128 28x28 stride 2 batch 8 8.8 -> 9.7; 100 -> 150 37x53 stride 2 batch 12 9.9 -> 13.1
// Both lines lie at half of where the two meet: there the one launch still gains a sixth.
bool rf_indexed(const RfPlan &pl, const Geom &g, size_t &lds)
{
    const int64_t passes = (int64_t)(pl.CB << (2 - pl.wpx_shift)) * ((pl.ncb + 1) / 2);
    lds = pl.lds + (size_t)passes * RF_PAIR_BYTES + align_up((size_t)g.K * 2, 16);
    // (tiles of two blocks of output channels are two passes and more, and taken at 256 workgroups and more)
    return pl.CB == 1 && pl.chunk == pl.ncb && pl.n_wgs <= (passes == 1 ? 512 : passes == 2 ? 128 : 0) && lds <= RF_LDS_TARGET;
}

int launch_rf_indexed(RfPlan pl, RfLayer L, const Geom &g, const uint16_t *codebook, const uint16_t *idx, const float *alpha, size_t lds,
                      hipStream_t s)
{
    L.scale = alpha;
    L.codebook = codebook;
    L.idx = idx;
    L.K = g.K;
    pl.lds = lds;
    if (pl.PB == 2) return launch_rf_one<2, 1, false, false, true>(pl, L, s);
    return launch_rf_one<1, 1, false, false, true>(pl, L, s);
}

RfProject rf_project(const Geom &g, const float *w, const uint16_t *codebook, const float *alpha, const float *beta, uint16_t *idx_out,
                     void *ws)
{
    RfProject p;
    p.W = rf_weights(g, ws);
    p.w = w;
    p.codebook = codebook;
    p.alpha = alpha;
    p.beta = beta;
    p.idx_out = idx_out;
    p.K = g.K;
    return p;
}

}  // namespace

bool rows_fp4_supported(const Geom &g) { return rf_plan(g, false).ok && rf_plan(g, true).ok; }

// Layers with wide rows.  A workgroup expands at least five rows for its one or two, so that from rows of about 600 pixels on the
// expansion is most of the time: pixels expanded per output pixel, times channel blocks, a quarter more where the tile leaves a
// compute unit one workgroup and a seventh more before the sign epilogue.  The one-hot form reads its windows as they are; its time goes
// with the input channels.  One-hot -> here, prepared, 32 rows, batch 64, K = 16, us: 33 -> 20 512 wide 90 -> 75, 640 106 -> 103 (sign
// 95 -> 117), 900 140 -> 190 (134 -> 214); 2 -> 4 K = 8 640 wide 46 -> 35, 900 67 -> 75; 128 -> 128 900 wide batch 32 269 -> 220.
// Launches of fewer than 800 workgroups stay here (batch 8 33 -> 20 768 wide, 768 of them, 24 -> 20; 900 wide, 900, 23.9 -> 28.7).
bool rows_fp4_loses_on_wide_rows(const Geom &g, bool sign)
{
    if (g.K > 64 || g.W <= 320) return false;                   // (the line is never below 320; no plan for the others)
    const RfPlan pl = rf_plan(g, sign);
    if (!pl.ok || pl.n_wgs < 800) return false;
    const int64_t expanded = pl.rows * (g.W + 1) * pl.ncb, pixels = (int64_t)(32 * pl.PB) << pl.wpx_shift;
    const int64_t here = expanded * (pl.lds > RF_LDS_TARGET ? 125 : 100) * (sign ? 115 : 100) / (100 * pixels);
    const int64_t one_hot = 1350 + (g.K > 32 ? 220 * g.C_in : 57 * g.C_in + 23 * std::max(0, g.C_in - 64));
    return here > one_hot;
}

size_t rows_fp4_workspace_bytes(const Geom &g)
{
    return rf_weight_bytes(g) + align_up((size_t)((g.C_out + 31) / 32) * 64 * sizeof(float), 256);
}

int launch_rows_fp4(const Geom &g, const void *x, const uint16_t *codebook, const void *idx, int tau, const float *alpha, float *y,
                    void *ws, hipStream_t s, const SignEpilogue *sign, int phases)
{
    const RfPlan pl = rf_plan(g, sign != nullptr);
    if (!pl.ok) return SNN_ERR_UNSUPPORTED;
    size_t lds;
    if (phases == SNN_PHASE_BOTH && !sign && tau == 0 && rf_indexed(pl, g, lds))
        return launch_rf_indexed(pl, rf_layer(pl, g, x, y, ws), g, codebook, (const uint16_t *)idx, alpha, lds, s);
    if (phases & SNN_PHASE_PREPARE) {
        const RfWeights W = rf_weights(g, ws);
        hipLaunchKernelGGL(rows_fp4_prep_kernel, dim3((unsigned)W.n_cob, (unsigned)((W.ncb + 1) / 2)), dim3(256), 0, s, W, codebook, g.K, idx,
                           tau, alpha, sign ? sign->beta : nullptr);
        const int rc = check_launch();
        if (rc != SNN_OK) return rc;
    }
    if (!(phases & SNN_PHASE_CONVOLVE)) return SNN_OK;
    if (sign) return launch_rf<true>(pl, rf_layer(pl, g, x, sign->out, ws), s);
    return launch_rf<false>(pl, rf_layer(pl, g, x, y, ws), s);
}

// The 1-bit layer: packing and convolution, popcount kernel -> here: 128 -> 128 28x28 batch 64 27.8 -> 16.5 us (packing is 5 of both),
// 64 -> 64 56x56 batch 64 34 -> 24, 512 -> 512 7x7 batch 64 31 -> 17.5; small batches and 16 -> 16 32x32 batch 256 the same 17 (the
// two launches from the host).  The popcount kernels' time goes with the output channels, this one's mostly with the pixels
// that its workgroups expand (rows above and below included, so more per output pixel the wider the rows are, and once per tile of
// output channels): they keep the layers of few output channels.  Up to 512 input channels the line is about five output channels
// per expanded pixel and output pixel, ten where the tile of wide rows leaves a compute unit one workgroup; past those
// the popcount kernel is several times slower and keeps up to eight output channels on wide rows, 32 where a unit has one
// workgroup.  Prepared, popcount -> here, us:
// 56x56 batch 64 (2.0 expanded) 256 -> 1 5.6 -> 16.8, 256 -> 8 13.3 -> 16.9, 256 -> 12 17.4 -> 17.1, 256 -> 32 35.3 -> 18.0,
// 32 -> 8 5.9 -> 6.4; 56x224 batch 16 (5.3) 128 -> 16 13.1 -> 14.7, 128 -> 24 17.3 -> 15.0; 32x512 batch 64 64 -> 32 (10.0)
// 53 -> 89, 64 -> 64 (5.0) 98 -> 77; 32x900 batch 2 (35) 64 -> 64 11.8 -> 19.2; 600 -> 1 56x56 batch 64 87 -> 31, 32x900 batch 2
// 27 -> 133, 600 -> 32 56x448 batch 8 172 -> 92, 32x640 batch 16 156 -> 250.  Layers of fewer than 256 kernels leave most of a
// 32 x 32 block empty (1 -> 1 56x56 batch 256 17.3 there, 19.6 here) and stay with the popcount kernel.  The packed input of the images a workgroup touches takes 32-bit offsets, too.
bool bnn_rows_form(const Geom &g)
{
    if ((int64_t)g.C_in * g.C_out < 256) return false;
    const RfPlan pl = rf_plan(g, false);
    if (!pl.ok || tuning(SNN_TUNE_BNN_REGS) != SNN_TUNE_AUTO) return false;
    const int64_t expanded = pl.rows * (g.W + 1) * pl.n_cotiles, pixels = (int64_t)(32 * pl.PB) << pl.wpx_shift;
    const bool alone = pl.lds > RF_LDS_TARGET;
    if (g.CW > 16 ? (g.C_out <= 8 && expanded > 8 * pixels) || (g.C_out <= 32 && alone) : g.C_out * pixels < (alone ? 10 : 5) * expanded)
        return false;
    const int64_t images = (pl.rows + g.H) / (g.H + 1) + 1;
    return images * g.H * g.W * g.CW * 4 < ((int64_t)1 << 31) - 4096;
}

size_t bnn_rows_workspace_bytes(const Geom &g) { return rf_weight_bytes(g); }

int launch_bnn_rows(const Geom &g, const void *x, const uint16_t *w9, const float *alpha, float *y, void *ws, hipStream_t s, int phases)
{
    const RfPlan pl = rf_plan(g, false);
    if (!pl.ok) return SNN_ERR_UNSUPPORTED;
    if (phases & SNN_PHASE_PREPARE) {
        const RfWeights W = rf_weights(g, ws);
        hipLaunchKernelGGL(rows_fp4_prep_planes_kernel, dim3((unsigned)W.n_cob * 8u, (unsigned)((W.ncb + 1) / 2)), dim3(256), 0, s, W, w9);
        const int rc = check_launch();
        if (rc != SNN_OK) return rc;
    }
    if (!(phases & SNN_PHASE_CONVOLVE)) return SNN_OK;
    RfLayer L = rf_layer(pl, g, x, y, ws);
    L.scale = alpha;
    return launch_rf<false, true>(pl, L, s);
}

int launch_rows_fp4_forward(const Geom &g, const float *x, const float *w, const uint16_t *codebook, const float *alpha, uint16_t *idx_out,
                            float *y, uint32_t *xr, void *ws, hipStream_t s, const SignEpilogue *sign)
{
    const RfPlan pl = rf_plan(g, sign != nullptr);
    if (!pl.ok) return SNN_ERR_UNSUPPORTED;
    RfFront f;
    f.pr = rf_project(g, w, codebook, alpha, sign ? sign->beta : nullptr, idx_out, ws);
    f.project_blocks = f.pr.W.n_cob * f.pr.W.ncb;
    f.x = x;
    f.xr = xr;
    f.rows = (int64_t)g.N * g.C_in * g.H;
    f.W = g.W;
    f.WW = g.WW;
    const PackRowsPlan pk = pack_rows_plan(x, f.rows, g.W);
    f.rows_per_block = pk.rows_per_block;
    f.vec = pk.vec;
    const int64_t blocks = f.project_blocks + (x ? pk.blocks : 0);
    if (blocks > 0x7fffffffLL) return SNN_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(rows_fp4_front_kernel, dim3((unsigned)blocks), dim3(256), 0, s, f);
    const int rc = check_launch();
    if (rc != SNN_OK) return rc;
    if (sign) return launch_rf<true>(pl, rf_layer(pl, g, xr, sign->out, ws), s);
    return launch_rf<false>(pl, rf_layer(pl, g, xr, y, ws), s);
}

int launch_rows_fp4_project_many(int n_layers, const Geom *gs, const float *const *w, const uint16_t *const *codebook,
                                 const float *const *alpha, const float *const *beta, uint16_t *const *idx_out, void *const *ws, hipStream_t s)
{
    for (int l0 = 0; l0 < n_layers; l0 += RF_PROJECT_MAX) {
        RfProjectMany m;
        m.n_layers = n_layers - l0 < RF_PROJECT_MAX ? n_layers - l0 : RF_PROJECT_MAX;
        int64_t blocks = 0;
        for (int i = 0; i < m.n_layers; ++i) {
            const int l = l0 + i;
            m.layer[i] = rf_project(gs[l], w[l], codebook[l], alpha[l], beta[l], idx_out[l], ws[l]);
            m.first[i] = (int)blocks;
            blocks += (int64_t)m.layer[i].W.n_cob * m.layer[i].W.ncb;
            if (blocks > 0x7fffffffLL) return SNN_ERR_UNSUPPORTED;
        }
        for (int i = m.n_layers; i <= RF_PROJECT_MAX; ++i) m.first[i] = (int)blocks;
        hipLaunchKernelGGL(rows_fp4_project_many_kernel, dim3((unsigned)blocks), dim3(256), 0, s, m);
        const int rc = check_launch();
        if (rc != SNN_OK) return rc;
    }
    return SNN_OK;
}

int launch_rows_fp4_front_many(int n_layers, const Geom *gs, const float *const *x, uint32_t *const *xr, const float *const *w,
                               const uint16_t *const *codebook, const float *const *alpha, uint16_t *const *idx_out, void *const *ws,
                               hipStream_t s)
{
    for (int l0 = 0; l0 < n_layers; l0 += RF_FRONT_MAX) {
        RfFrontMany m;
        m.n_layers = std::min(RF_FRONT_MAX, n_layers - l0);
        int64_t row_blocks = 0, project = 0, pack = 0;
        for (int i = 0; i < m.n_layers; ++i) {
            const Geom &g = gs[l0 + i];
            row_blocks += pack_rows_plan(x[l0 + i], (int64_t)g.N * g.C_in * g.H, g.W).blocks;
        }
        m.run = pack_run(row_blocks);
        for (int i = 0; i < m.n_layers; ++i) {
            const int l = l0 + i;
            const Geom &g = gs[l];
            const int64_t rows = (int64_t)g.N * g.C_in * g.H;
            const PackRowsPlan pk = pack_rows_plan(x[l], rows, g.W);
            if (pk.blocks > 0x7fffffffLL) return SNN_ERR_UNSUPPORTED;
            m.layer[i] = {(uint32_t *)ws[l], w[l], codebook[l], alpha[l], idx_out[l], x[l], xr[l], rows, g.C_in, g.C_out, g.K,
                          g.W, pk.rows_per_block, pk.vec, (int)pk.blocks};
            m.first_project[i] = (int)project;
            m.first_pack[i] = (int)pack;
            project += (int64_t)((g.C_out + 31) / 32) * ((g.C_in + 31) / 32);
            pack += (pk.blocks + m.run - 1) / m.run;
            if (project + pack > 0x7fffffffLL) return SNN_ERR_UNSUPPORTED;
        }
        for (int i = m.n_layers; i <= RF_FRONT_MAX; ++i) {
            m.first_project[i] = (int)project;
            m.first_pack[i] = (int)pack;
        }
        m.project_blocks = (int)project;
        // odd: consecutive workgroups go to the eight XCDs in turn, an even period would leave some without projections
        int64_t period = (project + pack) * 7 / 8 / project;
        period = period < 1 ? 1 : period - 1 + (period & 1);
        m.period_value = (uint32_t)period;
        m.period = make_divisor((uint32_t)period);
        hipLaunchKernelGGL(rows_fp4_front_many_kernel, dim3((unsigned)(project + pack)), dim3(256), 0, s, m);
        const int rc = check_launch();
        if (rc != SNN_OK) return rc;
    }
    return SNN_OK;
}

int launch_rows_fp4_many(int n_layers, const Geom *gs, const void *const *x, float *const *y, void *const *ws, bool projected, hipStream_t s)
{
    static LdsGrant grant[2];
    std::vector<RfPlan> plans(n_layers);
    std::vector<int> order(n_layers);
    for (int l = 0; l < n_layers; ++l) {
        plans[l] = rf_plan(gs[l], false, true);
        if (!plans[l].ok) return SNN_ERR_UNSUPPORTED;
        order[l] = l;
    }
    // Order of the layers.  Outputs that the last-level cache (256 MB) takes up: the layers whose workgroups run longest from one end and the
    // shortest, which are mostly stores, from the other in turn, so that stores and matrix work overlap and no long
    // workgroup is left to run alone at the end.  More, or so much beside real-valued kernels that the call has projected, which come through that
    // cache as well: the short ones first, the stores that the cache has taken up drain while the long ones multiply.  Measured, short
    // first / both ends in turn, with the policy below (pack and projection included where they are part of the call; A: the 16-layer stack,
    // 43 MB of kernels, B: the 32-layer stack, 76 MB, C: 18 small layers, 1 MB), MB of output in brackets: A batch 16 (92) 65.8 / 60.4, batch 32 (184)
    // 102 / 96, batch 44 (253) 129 / 125, prepared 63.0 / 59.5, batch 64 (368) 180 / 182; A on 200x200 images batch 45 (212) 160 / 130; B batch 4 (42) 61 / 56,
    // batch 20 (211) 126 / 122, batch 24 (253) 143 / 146 on two cards, 150 / 146 on another, prepared 72 / 63, batch 32 (337) 181 / 189; C batch 256
    // (168) 90 / 86, batch 384 (252) 130 / 125, batch 512 (336) 167 / 162.  The long ones first without the turns: B batch 8 53.8 -> 56.5,
    // A batch 64 193 -> 202; all layers mixed in proportion to their size: 58 and 217 (stores to many tensors at a time).
    // Cache policy: non-temporal, but where the order takes turns the outputs whose runs share lines stay in L2, non-temporal -> in L2: A batch 16
    // 65.0 -> 60.4, batch 32 107 -> 97, prepared 55 -> 46; A on 200x200 images, most of whose planes share lines, batch 12 (56) 55 -> 49, batch 45 150 -> 127,
    // prepared batch 12 28.7 -> 21.8; B prepared batch 10 34.6 -> 30.7, batch 24 73 -> 67; below 48 MB not, B batch 4 (42) 54.4 -> 55.1, prepared
    // 19.27 -> 19.35 (A batch 8 (46) 48.3 -> 47.2, prepared 20.0 -> 19.8).  Beside more than 60 MB of projected kernels up to 176 MB alone: B batch 7 68.7 -> 66.6,
    // batch 10 76.3 -> 73.9, batch 16 (168) 108.5 -> 109.3, 106.6 -> 107.1 and 108.6 -> 106.4 on three cards, batch 20 (211) 122 -> 127; B without its
    // last layer (67 MB of kernels) batch 7 63.6 -> 61.9, batch 12 90 -> 85, batch 16 105 -> 100.  (Where the short ones go first: A batch 64 165 -> 179.)
    auto length = [&](int l) { return (int64_t)plans[l].ncb * plans[l].PB * plans[l].CB; };
    int64_t out_bytes = 0, kernel_bytes = 0;
    for (int l = 0; l < n_layers; ++l) {
        out_bytes += 4 * gs[l].P * gs[l].C_out;
        if (projected) kernel_bytes += (int64_t)36 * gs[l].C_in * gs[l].C_out;
    }
    const bool fold = out_bytes <= (int64_t)256 << 20 && out_bytes + kernel_bytes <= (int64_t)304 << 20;
    const bool cached = fold && out_bytes >= (int64_t)48 << 20 && (kernel_bytes <= (int64_t)60 << 20 || out_bytes <= (int64_t)176 << 20);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return fold ? length(a) > length(b) : length(a) < length(b); });
    for (int at = 0; at < n_layers;) {
        RfMany m;
        int n = 0;
        int64_t blocks = 0;
        size_t lds = 0;
        for (; at < n_layers && n < RF_MANY_MAX; ++at, ++n) {
            const int l = order[at];
            const RfPlan &pl = plans[l];
            const int64_t here = (pl.n_wgs + 7) / 8 * 8;
            if (blocks + here > 0x7fffffffLL) break;
            const RfLayer L = rf_layer(pl, gs[l], x[l], y[l], ws[l]);
            const int policy = cached && (((uintptr_t)y[l] | (uintptr_t)gs[l].HoWo * 4u) & 63) != 0 ? FP4_STORE_CACHED : FP4_STORE_NT;
            m.layer[n] = {L.x, L.wq, L.out, L.N, L.C_in, L.C_out, L.H, L.W, L.Ho, L.Wo, L.plane, L.n_cotiles, L.n_wgs,
                          (uint16_t)L.chunk, (uint16_t)L.pitch, (uint8_t)(10 * pl.PB + pl.CB), (uint8_t)pl.wpx_shift, (uint8_t)gs[l].stride, (uint8_t)policy,
                          L.div_HoWo, L.div_Wo, L.div_H1, L.div_WW, L.div_cotiles};
            m.first[n] = (int)blocks;
            blocks += here;
            lds = std::max(lds, pl.lds);
        }
        m.n_layers = n;
        m.fold = fold;
        for (int i = n; i <= RF_MANY_MAX; ++i) m.first[i] = (int)blocks;
        auto kern = fold ? rows_fp4_many_kernel<false> : rows_fp4_many_kernel<true>;
        if (grant_dynamic_lds((const void *)kern, lds, grant[fold]) != SNN_OK) return SNN_ERR_LAUNCH;
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), lds, s, m);
        const int rc = check_launch();
        if (rc != SNN_OK) return rc;
    }
    return SNN_OK;
}

}  // namespace snn

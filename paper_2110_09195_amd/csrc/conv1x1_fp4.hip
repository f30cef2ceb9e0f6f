// The 1x1 layers (appendix "Extending to Bottleneck with 1x1 Kernels") as a dense contraction over the input channels on the matrix
// cores, from packed channels:
//
//   S[co][pixel] = sum over input channels c of  w(co, c) * x(pixel, c),   w(co, 8 g + j) = element j of codebook8[idx[co][g]]
//
// with w, x in {+1, -1} (0 for channels that do not exist) as FP4 e2m1 operands of v_mfma_f32_32x32x64_f8f6f4; the fp32 accumulator
// holds S exactly and y = fl(S * alpha) is that of the shared form bit for bit.
//
// What bounds it is the output, four bytes per pixel and output channel: 64 -> 256 56x56 batch 64 writes 205 MB.  A gather of one of
// K responses as a one-hot product (subbit_mfma.hip) takes 32 or 64 contraction slots per eight input channels, this takes
// eight.  A wave needs no other's data: no LDS, no barriers.  A word of 32 channels of a pixel, and one of 32 weights of an output channel, is
// a lane's operand; slot 8 r + j of it is bit 4 j + r, two instructions per register.
// Measured, one-hot form -> this one (packing included, us): 64 -> 256 56x56 batch 64 61.2 -> 49.4, of which packing 9 and 205 MB of output at
// 5.1 TB/s; 256 -> 64 65 -> 50; 512 -> 2048 7x7 batch 64 26.9 -> 16.3; 1024 -> 256 14x14 batch 64 35 -> 26; 2048 -> 512 7x7 batch 8 19.8 -> 11.0;
// 72 -> 130 29x31 batch 64 29 -> 15.7; one image 16 -> 10.5.
#include "fp4_common.h"
#include "conv1x1_fp4.h"

#include <algorithm>
#include <type_traits>

namespace snn {

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct C1Layer {
    const uint32_t *x;       // packed channels [N][H][W][CW]
    const uint32_t *wq;      // [block of 32 output channels][pair of words][lane]: bit planes
    const float *scale;      // [32 n_cob]: alpha, 0 for padding channels
    float *y;
    uint32_t x_image, y_image;           // bytes of an image
    int C_in, C_out, H, W, stride, HoWo, Wo, P, CW;
    int pairs, n_cob, n_blk, n_cotiles, n_wgs, wpx_shift, policy;
    Divisor div_HoWo, div_Wo, div_cotiles;
};

__device__ __forceinline__ u32x4 expand(uint32_t w, const u32x4 &ones)
{
    u32x4 a;
#pragma unroll
    for (int r = 0; r < 4; ++r) a[r] = ((w << (3 - r)) & 0x88888888u) | ones[r];
    return a;
}

// A workgroup of four waves, 2^wpx_shift of them side by side along pixels, the others on further output channels; a wave owns PB blocks of 32
// consecutive pixels of the flattened (n, ho, wo) order x CB blocks of 32 output channels.
template <int PB, int CB>
__global__ __launch_bounds__(256, 4)
void conv1x1_fp4_kernel(const C1Layer L)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n_l = lane & 31, h = lane >> 5;
    uint32_t wg = blockIdx.x;
    {                                                          // an XCD gets a contiguous run of tiles
        const uint32_t per = (uint32_t)L.n_wgs >> 3, rem = (uint32_t)L.n_wgs & 7u, xcd = wg & 7u;
        wg = xcd * per + min(xcd, rem) + (wg >> 3);
    }
    const uint32_t pxt = fast_div(wg, L.div_cotiles);
    const int cot = (int)(wg - pxt * (uint32_t)L.n_cotiles);
    const int wpx = wave & ((1 << L.wpx_shift) - 1), wco = wave >> L.wpx_shift;
    const int blk0 = ((int)(pxt << L.wpx_shift) + wpx) * PB;
    const int cob0 = ((cot << (2 - L.wpx_shift)) + wco) * CB;
    if (cob0 >= L.n_cob || blk0 >= L.n_blk) return;
    const int n0 = (int)fast_div((uint32_t)blk0 * 32u, L.div_HoWo);
    const int n_images = (int)fast_div((uint32_t)min((blk0 + PB) * 32, L.P) - 1u, L.div_HoWo) - n0 + 1;

    const __amdgpu_buffer_rsrc_t xres = make_rsrc((const char *)L.x + (uint64_t)(uint32_t)n0 * L.x_image, (uint32_t)n_images * L.x_image);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(L.wq, (uint32_t)(L.n_cob * L.pairs) * 256u);
    uint32_t xoff[PB], yoff[PB];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        const int p = (blk0 + pb) * 32 + n_l;
        const bool ok = p < L.P;
        const int pp = min(p, L.P - 1);
        const int n = (int)fast_div((uint32_t)pp, L.div_HoWo), r = pp - n * L.HoWo;
        int at = r;
        if (L.stride != 1) {                                   // (wave-uniform)
            const int ho = (int)fast_div((uint32_t)r, L.div_Wo);
            at = (ho * L.W + r - ho * L.Wo) * L.stride;
        }
        xoff[pb] = ok ? (uint32_t)(n - n0) * L.x_image + (uint32_t)(at * L.CW + h) * 4u : OFF_NONE;
        yoff[pb] = ok ? (uint32_t)(n - n0) * L.y_image + (uint32_t)(4 * h * L.HoWo + r) * 4u : OFF_NONE;
    }
    // Words of pair pr.  (Of an odd number of words the last pair's second one is some other word of the buffer, or zero: masked.)
    uint32_t X[2][PB], A[2][CB];
    auto load = [&](int pr, uint32_t (&x)[PB], uint32_t (&a)[CB]) {
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) x[pb] = __builtin_amdgcn_raw_buffer_load_b32(xres, (int)xoff[pb], 8 * pr, 0);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
            a[cb] = __builtin_amdgcn_raw_buffer_load_b32(wres, lane * 4, (min(cob0 + cb, L.n_cob - 1) * L.pairs + pr) * 256, 0);
    };
    load(0, X[0], A[0]);
    v16f acc[CB][PB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[cb][pb][r] = 0.0f;

    const u32x4 one = {0x22222222u, 0x22222222u, 0x22222222u, 0x22222222u};
    auto step = [&](int pr, const uint32_t (&x)[PB], const uint32_t (&a)[CB]) {
        u32x4 ones = one;
        uint32_t exist = 0xffffffffu;
        if (64 * (pr + 1) > L.C_in) {                          // (wave-uniform) channels that do not exist are zeros here
            const int left = L.C_in - 64 * pr - 32 * h;
            exist = left >= 32 ? 0xffffffffu : left <= 0 ? 0u : (1u << left) - 1u;
            ones = (u32x4){(exist << 1) & 0x22222222u, exist & 0x22222222u, (exist >> 1) & 0x22222222u, (exist >> 2) & 0x22222222u};
        }
        u32x4 E[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) E[cb] = expand(a[cb], one);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
            const u32x4 b = expand(x[pb] & exist, ones);
            const v8i bv = {(int)b[0], (int)b[1], (int)b[2], (int)b[3], 0, 0, 0, 0};
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const v8i av = {(int)E[cb][0], (int)E[cb][1], (int)E[cb][2], (int)E[cb][3], 0, 0, 0, 0};
                acc[cb][pb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc[cb][pb], 4, 4, 0, 0, 0, 0);
            }
        }
    };
    int pr = 0;
    for (; pr + 2 <= L.pairs; pr += 2) {
        load(pr + 1, X[1], A[1]);
        step(pr, X[0], A[0]);
        if (pr + 2 < L.pairs) load(pr + 2, X[0], A[0]);
        step(pr + 1, X[1], A[1]);
    }
    if (pr < L.pairs) step(pr, X[0], A[0]);

    // (alpha is read here: beside the accumulators and the words it would not fit 128 registers, which four waves per SIMD have)
    f32x4 al[CB][4];                                           // register r of an accumulator is channel 8 (r / 4) + 4 h + r % 4
    const __amdgpu_buffer_rsrc_t sres = make_rsrc(L.scale, (uint32_t)L.n_cob * 128u);
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(sres, 16 * h, (min(cob0 + cb, L.n_cob - 1) * 32 + 8 * q) * 4, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) al[cb][q][i] = __uint_as_float(v[i]);
        }
    // ---- y = alpha * S: lanes 0..31 of a register are 32 consecutive pixels of one channel ------------------------------------
    const uint32_t chan = (uint32_t)L.HoWo * 4u;
    const __amdgpu_buffer_rsrc_t yres = make_rsrc((char *)L.y + (uint64_t)(uint32_t)n0 * L.y_image, (uint32_t)n_images * L.y_image);
    auto store = [&](auto policy, auto whole) {                // whole: all 32 CB channels exist
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int co0 = (cob0 + cb) * 32, left = L.C_out - co0 - 4 * h;
            const uint32_t last = (uint32_t)(L.C_out - 1) * chan;
            uint32_t at = (uint32_t)co0 * chan;                // (wave-uniform)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int pb = 0; pb < PB; ++pb) {
                        const uint32_t v = __float_as_uint(acc[cb][pb][4 * q + i] * al[cb][q][i]);
                        const uint32_t off = decltype(whole)::value || 8 * q + i < left ? yoff[pb] : OFF_NONE;
                        // (the scalar offset stays inside the buffer, also where no lane stores)
                        __builtin_amdgcn_raw_buffer_store_b32(v, yres, (int)off, (int)(decltype(whole)::value ? at : min(at, last)), decltype(policy)::value);
                    }
                    at += i < 3 ? chan : 5u * chan;
                }
        }
    };
    auto store_under = [&](auto policy) {
        if ((cob0 + CB) * 32 <= L.C_out) store(policy, std::true_type{});
        else store(policy, std::false_type{});
    };
    if (L.policy == FP4_STORE_NT) store_under(std::integral_constant<int, AUX_NT>{});
    else if (L.policy == FP4_STORE_THROUGH) store_under(std::integral_constant<int, AUX_THROUGH>{});
    else store_under(std::integral_constant<int, AUX_CACHED>{});
}

// Indices -> bit planes: a thread makes the word of (output channel, 32 input channels), bit i of which is channel i.
__global__ __launch_bounds__(256)
void conv1x1_fp4_prep_kernel(const uint16_t *__restrict__ codebook8, int K, const uint16_t *__restrict__ idx, int G, int C_out, int pairs, int n_cob,
                             const float *__restrict__ alpha, uint32_t *__restrict__ wq, float *__restrict__ scale)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int lane = (int)(t & 63);
    const int64_t unit = t >> 6;                               // (block of output channels, pair)
    if (unit >= (int64_t)n_cob * pairs) return;
    const int cob = (int)(unit / pairs), pr = (int)(unit - (int64_t)cob * pairs);
    const int co = cob * 32 + (lane & 31), g0 = (2 * pr + (lane >> 5)) * 4;
    uint32_t word = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (co < C_out && g0 + j < G) {
            const uint32_t code = codebook8[min((uint32_t)idx[(int64_t)co * G + g0 + j], (uint32_t)K - 1u)] & 255u;
            word |= (__brev(code) >> 24) << (8 * j);           // element j of a vector is bit 7 - j of its code
        }
    wq[t] = word;
    if (pr == 0 && lane < 32) scale[co] = co < C_out ? alpha[co] : 0.0f;
}

struct C1Plan {
    int PB, CB, wpx_shift, pairs;
    int64_t n_cob, n_blk, n_cotiles, n_wgs;
    bool ok;
};

C1Plan c1_plan(const Geom &g)
{
    C1Plan pl;
    pl.pairs = (g.CW + 1) / 2;
    pl.n_cob = (g.C_out + 31) / 32;
    pl.n_blk = (g.P + 31) / 32;
    pl.wpx_shift = pl.n_cob >= 3 ? 1 : 2;
    // Two by two blocks read each word for two products; one where that leaves a SIMD without a wave (1 x 1 -> 2 x 2 blocks, us: 2048 -> 512
    // 7x7 batch 8, 56 waves of 2 x 2, 10.9 -> 14.8, batch 64, 392, 21.3 -> 23.6; 1024 -> 256 14x14 batch 64, 784, 28.1 -> 26.1; 512 -> 2048
    // 7x7 batch 64, 1568, 19.2 -> 16.3).
    pl.PB = pl.CB = (pl.n_blk + 1) / 2 * ((pl.n_cob + 1) / 2) < 512 ? 1 : 2;
    if (pl.PB == 1) pl.wpx_shift = pl.n_cob >= 3 ? 0 : pl.n_cob == 2 ? 1 : 2;
    const int64_t px = (int64_t)pl.PB << pl.wpx_shift, co = (int64_t)pl.CB << (2 - pl.wpx_shift);
    pl.n_cotiles = (pl.n_cob + co - 1) / co;
    pl.n_wgs = (pl.n_blk + px - 1) / px * pl.n_cotiles;
    // 32-bit offsets inside the images that a wave touches, and inside the weights
    const int64_t images = (32 * pl.PB - 1 + g.HoWo - 1) / g.HoWo + 1, lim = ((int64_t)1 << 31) - 4096;
    pl.ok = images * g.H * g.W * g.CW * 4 < lim && images * g.C_out * g.HoWo * 4 < lim && pl.n_cob * pl.pairs * 256 < lim && g.P < lim - 65536 &&
            pl.n_wgs < lim && pl.n_blk * 32 < lim;
    return pl;
}

}  // namespace

bool conv1x1_fp4_supported(const Geom &g) { return c1_plan(g).ok; }

size_t conv1x1_fp4_workspace_bytes(const Geom &g)
{
    const size_t n_cob = (size_t)(g.C_out + 31) / 32, pairs = (size_t)(g.CW + 1) / 2;
    return n_cob * pairs * 256 + n_cob * 128;
}

int launch_conv1x1_fp4(const Geom &g, const void *x, const uint16_t *codebook8, const uint16_t *idx, const float *alpha, float *y, void *ws,
                       hipStream_t s, int phases)
{
    const C1Plan pl = c1_plan(g);
    if (!pl.ok) return SNN_ERR_UNSUPPORTED;
    uint32_t *const wq = (uint32_t *)ws;
    float *const scale = (float *)((char *)ws + pl.n_cob * pl.pairs * 256);
    if (phases & SNN_PHASE_PREPARE) {
        const int64_t blocks = (pl.n_cob * pl.pairs + 3) / 4;
        hipLaunchKernelGGL(conv1x1_fp4_prep_kernel, dim3((unsigned)blocks), dim3(256), 0, s, codebook8, g.K, idx, g.C_in / 8, g.C_out, pl.pairs,
                           (int)pl.n_cob, alpha, wq, scale);
        const int rc = check_launch();
        if (rc != SNN_OK || !(phases & SNN_PHASE_CONVOLVE)) return rc;
    }
    C1Layer L;
    L.x = (const uint32_t *)x;
    L.wq = wq;
    L.scale = scale;
    L.y = y;
    L.x_image = (uint32_t)(g.H * g.W * g.CW) * 4u;
    L.y_image = (uint32_t)(g.C_out * g.HoWo) * 4u;
    L.C_in = g.C_in; L.C_out = g.C_out; L.H = g.H; L.W = g.W; L.stride = g.stride; L.HoWo = g.HoWo; L.Wo = g.Wo; L.P = (int)g.P; L.CW = g.CW;
    L.pairs = pl.pairs; L.n_cob = (int)pl.n_cob; L.n_blk = (int)pl.n_blk; L.n_cotiles = (int)pl.n_cotiles; L.n_wgs = (int)pl.n_wgs;
    L.wpx_shift = pl.wpx_shift;
    L.policy = store_policy(g, y);
    L.div_HoWo = make_divisor((uint32_t)g.HoWo);
    L.div_Wo = make_divisor((uint32_t)g.Wo);
    L.div_cotiles = make_divisor((uint32_t)pl.n_cotiles);
    if (pl.PB == 2) hipLaunchKernelGGL((conv1x1_fp4_kernel<2, 2>), dim3((unsigned)pl.n_wgs), dim3(256), 0, s, L);
    else hipLaunchKernelGGL((conv1x1_fp4_kernel<1, 1>), dim3((unsigned)pl.n_wgs), dim3(256), 0, s, L);
    return check_launch();
}

}  // namespace snn

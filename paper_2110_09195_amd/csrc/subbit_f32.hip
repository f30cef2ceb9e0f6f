// The sub-bit convolution of Sec. 4.5 / Fig. 6 with real-valued activations (SNN_ACT_F32; the
// W/A = x/32 models of Tables 1-2 and the deployment test of Table 4).
//
// Two forms, chosen by subset size and output channels (use_dense); y = alpha * S in both, all sums in fp32.
// Two-stage: per chunk of input channels the workgroup builds T[ci][k][pixel] in LDS (nine add/subtracts of the window's
// values per response, as fma(x, +-1, acc)), then every lane gathers float4 rows T[ci][idx[co][ci]][4 pixels] and adds them.
// Dense: a contraction over taps and input channels on the fp32 matrix unit.
#include "f32_rows.h"
#include "subbit_common.h"

#include <type_traits>

namespace snn {

namespace {

constexpr int SF_TP = 64;    // pixels per tile; a row of T is 64 floats
constexpr int SF_G = 16;     // float4 groups per row
constexpr int SF_CL = 4;     // output channels per wave instruction

// Largest chunk of input channels a workgroup stages at once: one channel per wave and chunk where the registers
// for the chunk's gather offsets allow it.
template <int J, int NW>
struct SfChunk { static constexpr int max = (NW >= 16 && J <= 4) ? 16 : 8; };

template <int J, int NW>
__global__ __launch_bounds__(NW * 64)
void subbit_f32_kernel(const float *__restrict__ x, const float *__restrict__ coef,
                       const uint16_t *__restrict__ offs, const float *__restrict__ alpha,
                       float *__restrict__ y, Geom g, int COP, int CIC)
{
    constexpr int COW = SF_CL * J;
    extern __shared__ __align__(16) unsigned char smem[];
    const int K = g.K;
    float *T = (float *)smem;                               // [CIC][K][TP]
    // coef[K][9] (+-1.0f, window order) stays in memory: its index is wave-uniform, so the nine coefficients of a
    // member arrive through the scalar cache and are scalar operands of the multiply-adds (read from LDS they were
    // 288 broadcast reads per input channel and thread, and the loop waited for every one of them)

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int64_t p_tile = (int64_t)blockIdx.x * SF_TP;

    // stage-1 geometry: this thread always evaluates pixel (tid & 63) of the tile
    int off9[9];
    bool ok9[9];
    int n1;
    {
        int64_t p = p_tile + (tid & 63);
        if (p >= g.P) p = g.P - 1;
        n1 = (int)(p / g.HoWo);
        const int r = (int)(p - (int64_t)n1 * g.HoWo);
        const int ho = r / g.Wo, wo = r - ho * g.Wo;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int h = ho * g.stride + t / 3 - 1, w = wo * g.stride + t % 3 - 1;
            ok9[t] = h >= 0 && h < g.H && w >= 0 && w < g.W;
            off9[t] = ok9[t] ? h * g.W + w : 0;
        }
    }

    float acc[J][4];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int w = 0; w < 4; ++w) acc[j][w] = 0.0f;

    const int g16 = lane & (SF_G - 1);
    const int cl = lane / SF_G;
    const int lane_co = blockIdx.y * (COW * NW) + wave * COW + cl * J;
    const int64_t plane = (int64_t)g.H * g.W;

    __syncthreads();

    // window of the wave's first channel of the first chunk (every later one is requested a chunk ahead)
    float xnext[9];
    {
        const float *src0 = x + ((int64_t)n1 * g.C_in + min(tid >> 6, g.C_in - 1)) * plane;
#pragma unroll
        for (int t = 0; t < 9; ++t) xnext[t] = ok9[t] ? src0[off9[t]] : 0.0f;
    }

    for (int c0 = 0; c0 < g.C_in; c0 += CIC) {
        const int nci = min(CIC, g.C_in - c0);
        // the gather offsets of this chunk are requested before stage 1 and used after it (a dependent global load
        // per gather in stage 2 was most of the kernel's time at one wave per SIMD)
        constexpr int CIC_MAX = SfChunk<J, NW>::max;
        uint16_t ofs[CIC_MAX][J];
        {
            const uint16_t *op = offs + (int64_t)c0 * COP + lane_co;
#pragma unroll
            for (int ci_l = 0; ci_l < CIC_MAX; ++ci_l)
#pragma unroll
                for (int j = 0; j < J; ++j) ofs[ci_l][j] = ci_l < nci ? op[(int64_t)ci_l * COP + j] : (uint16_t)0;
        }
        // stage 1: nine add/subtracts per (pixel, ci, k)
        for (int ci_l = tid >> 6; ci_l < nci; ci_l += NW) {
            float xv[9];
            if (ci_l == (tid >> 6)) {
                // the wave's first channel of the chunk was requested a chunk ahead; now the next chunk's
#pragma unroll
                for (int t = 0; t < 9; ++t) xv[t] = xnext[t];
                const int cn = c0 + CIC + (tid >> 6);
                const float *srcn = x + ((int64_t)n1 * g.C_in + min(cn, g.C_in - 1)) * plane;
#pragma unroll
                for (int t = 0; t < 9; ++t) xnext[t] = ok9[t] ? srcn[off9[t]] : 0.0f;
            } else {
                const float *src = x + ((int64_t)n1 * g.C_in + c0 + ci_l) * plane;
#pragma unroll
                for (int t = 0; t < 9; ++t) xv[t] = ok9[t] ? src[off9[t]] : 0.0f;
            }
            float *Tw = T + (size_t)ci_l * K * SF_TP + (tid & 63);
#pragma unroll 4
            for (int k = 0; k < K; ++k) {
                const float *ck = coef + k * 9;
                float s = 0.0f;
#pragma unroll
                for (int t = 0; t < 9; ++t) s = __builtin_fmaf(xv[t], ck[t], s);
                Tw[k * SF_TP] = s;
            }
        }
        __syncthreads();
        // stage 2
        {
            const float *Tl = T + g16 * 4;
#pragma unroll
            for (int ci_l = 0; ci_l < CIC_MAX; ++ci_l) {
                if (ci_l < nci) {
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        // offs holds idx * 64 (row bytes of the packed kernel); a row here is 64 floats
                        const float4 v = *(const float4 *)(Tl + ofs[ci_l][j]);
                        acc[j][0] += v.x;
                        acc[j][1] += v.y;
                        acc[j][2] += v.z;
                        acc[j][3] += v.w;
                    }
                }
                Tl += (size_t)K * SF_TP;
            }
        }
        __syncthreads();
    }

    const int64_t p0 = p_tile + g16 * 4;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int64_t p = p0 + b;
        if (p >= g.P) break;
        const int n = (int)(p / g.HoWo);
        const int r = (int)(p - (int64_t)n * g.HoWo);
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (lane_co + j < g.C_out)
                store_output(y + ((int64_t)n * g.C_out + lane_co + j) * g.HoWo + r, alpha[lane_co + j] * acc[j][b]);
    }
}

struct F32Cfg { int J, NW, COB, CIC; size_t lds; };

// J output channels per lane, NW waves: a workgroup covers COB = 4 * J * NW output channels, and stage 1 is
// repeated once per group of COB, so COB should reach C_out.  Few pixel tiles (a small image or batch) want many
// waves per workgroup, since a tile is then all a compute unit has to hide its latencies with; many tiles want
// several small workgroups per unit, which overlap each other's barriers.
F32Cfg pick_f32_cfg(const Geom &g)
{
    const int64_t tiles = (g.P + SF_TP - 1) / SF_TP;
    int NW = tiles <= 512 ? 16 : tiles <= 2048 ? 8 : 4;
    const int forced = tuning(SNN_TUNE_F32_WAVES);
    if (forced == 4 || forced == 8 || forced == 16) NW = forced;
    int J = 1;
    while (J < 8 && 4 * J * NW < g.C_out) J <<= 1;
    while (NW > 4 && J == 1 && 4 * (NW / 2) >= g.C_out) NW >>= 1;     // no wave without output channels
    F32Cfg c;
    c.J = J;
    c.NW = NW;
    c.COB = 4 * J * NW;
    const size_t budget = NW >= 16 ? 128 * 1024 : NW >= 8 ? 64 * 1024 : 48 * 1024;
    c.CIC = (NW >= 16 && J <= 4) ? 16 : 8;
    while (c.CIC > 1 && (size_t)c.CIC * g.K * SF_TP * sizeof(float) > budget) c.CIC >>= 1;
    c.lds = (size_t)c.CIC * g.K * SF_TP * sizeof(float);
    return c;
}

// offs[ci][co] = min(idx[co][ci], K-1) * 64 (floats per row of T); codes[k] in window order.
__global__ __launch_bounds__(256)
void subbit_f32_prep_kernel(const uint16_t *__restrict__ codebook, const uint16_t *__restrict__ idx, int C_in,
                            int C_out, int COP, int K, uint32_t *__restrict__ codes, float *__restrict__ coef,
                            uint16_t *__restrict__ offs)
{
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t n_offs = (int64_t)C_in * COP;
    if (gid < n_offs) {
        const int ci = (int)(gid / COP), co = (int)(gid - (int64_t)ci * COP);
        const int k = co < C_out ? min((int)idx[(int64_t)co * C_in + ci], K - 1) : 0;
        offs[gid] = (uint16_t)(k * SF_TP);
    } else if (gid < n_offs + 512) {
        const int k = (int)(gid - n_offs);
        const uint32_t c = k < K ? code_to_window_order(codebook[k] & 511u) : 0u;
        codes[k] = c;
        for (int t = 0; t < 9; ++t) coef[k * 9 + t] = ((c >> t) & 1u) ? 1.0f : -1.0f;    // window order: tap t is bit t
    }
}

// ---- the dense form ----------------------------------------------------------------------------------------------------
// S[co][pixel] = sum over taps and input channels of w x on v_mfma_f32_32x32x2_f32: a wave owns 32 output channels x 32
// pixels, a step is a pair of input channels (one per lane half) at one tap.  The weight operand is +-1.0f made from the
// channel's 9-bit code in two instructions, the activation operand comes from rows in LDS or straight from memory (NL, below).  Each tap
// has an accumulator of its own, so that no chain of roundings is longer than the two-stage form's over the channels.
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr uint32_t SD_NONE = 0x80000000u;              // past every buffer used here

// wq: codes of [32 output channels][4 pairs of input channels]; lane (co, h) has the pairs' channels 2 p + h as four uint16.
//
// S = 4: the four waves of a workgroup share a block and split its channels, their sums meet in LDS (a quarter of the chain, four
// times the waves: 1 x 512 -> 64 7x7 has four blocks); S = 1: a block per wave, for the few channels that are not worth it.
//
// NL > 0: a wave brings the input rows that its pixels touch, zero pixels around the images included, to LDS with NL loads per pair of
// channels and reads its nine taps there (two pairs in LDS, two more in registers on the way; within a wave LDS keeps the order, no
// barrier).  NL = 0: nine loads per pair straight from memory (L1 / L2: 64 x 4 bytes per 64 clocks of matrix work), three pairs of
// channels ahead.  The sums are the same bit for bit; which way, and what both take: sd_staged (f32_rows.h).
//
// INDEXED: the codes are looked up here, in a copy of the codebook in LDS, instead of in words that a launch of their own has made
// (where: sd_looks_up).
struct SdIndexed {
    const uint16_t *codebook, *idx;
    int K;
};

template <int S, int NL, bool INDEXED>
__global__ __launch_bounds__(256, 2)
void subbit_f32_dense_kernel(const float *__restrict__ x, const uint32_t *__restrict__ wq, const float *__restrict__ alpha,
                             float *__restrict__ y, Geom g, int n_cob, int quads, uint32_t n_blocks, SdRows rows, SdIndexed ix)
{
    const int lane = threadIdx.x & 63, n_l = lane & 31, h = lane >> 5;
    const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t my_id = S == 1 ? blockIdx.x * 4u + (uint32_t)wave : blockIdx.x, id = min(my_id, n_blocks - 1u);
    const uint32_t blk = id / (uint32_t)n_cob;
    const int cob = (int)(id - blk * (uint32_t)n_cob);
    const uint32_t P = (uint32_t)g.P, HoWo = (uint32_t)g.HoWo;
    const uint32_t n0 = blk * 32u / HoWo;
    const bool mine = blk * 32u + (uint32_t)n_l < P;
    const uint32_t pp = min(blk * 32u + (uint32_t)n_l, P - 1u);
    const uint32_t n = pp / HoWo, r = pp - n * HoWo;
    const int ho = (int)(r / (uint32_t)g.Wo), wo = (int)r - ho * g.Wo;

    const int64_t x_image = (int64_t)g.C_in * g.H * g.W, y_image = (int64_t)g.C_out * g.HoWo;
    const int64_t lim = 0x7fffffff;
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(x + (int64_t)n0 * x_image), 0, (int)min((int64_t)(g.N - (int)n0) * x_image * 4, lim), 0x00020000);
    const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
        y + (int64_t)n0 * y_image, 0, (int)min((int64_t)(g.N - (int)n0) * y_image * 4, lim), 0x00020000);
    const uint32_t plane = (uint32_t)(g.H * g.W) * 4u;
    uint32_t off[NL > 0 ? NL : 9];
    uint32_t window = 0;                                       // NL > 0: LDS offset of the window's first pixel in a channel's plane
    if constexpr (NL > 0) {
        const SdBlock b = sd_block(g, blk);
        window = (uint32_t)sd_window(g, rows, b, n, ho, wo) * 4u;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const SdPixel p = sd_pixel(g, rows, b, 32 * i + n_l);
            off[i] = p.in ? (uint32_t)p.image * (uint32_t)x_image * 4u + (uint32_t)h * plane + (uint32_t)(p.h * g.W + p.w) * 4u : SD_NONE;
        }
    } else
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int hh = ho * g.stride + t / 3 - 1, ww = wo * g.stride + t % 3 - 1;
        const bool in = hh >= 0 && hh < g.H && ww >= 0 && ww < g.W;
        off[t] = in ? (n - n0) * (uint32_t)x_image * 4u + (uint32_t)h * plane + (uint32_t)(hh * g.W + ww) * 4u : SD_NONE;
    }
    const int pairs = (g.C_in + 1) >> 1;
    float B[NL > 0 ? 2 : 4][9], G[2][NL > 0 ? NL : 1];
    auto load_pair = [&](int p, auto &b) {                     // (past the last channel: zeros, nothing read)
        const bool have = 2 * p + h < g.C_in;
        const uint32_t at = 2u * (uint32_t)min(p, pairs - 1) * plane;
#pragma unroll
        for (int t = 0; t < (NL > 0 ? NL : 9); ++t)
            b[t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xres, (int)(have ? off[t] : SD_NONE), (int)at, 0));
    };
    const u32x2 *codes = (const u32x2 *)wq + (int64_t)cob * quads * 64 + lane;
    const int q0 = S == 1 ? 0 : wave * quads / S, q1 = S == 1 ? quads : (wave + 1) * quads / S;
    const int p_end = min(pairs, 4 * q1);
    // INDEXED: the quad's four channels 8 q + 2 u + h of output channel 32 cob + lane % 32
    const __amdgpu_buffer_rsrc_t ires =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(ix.idx), 0, INDEXED ? g.C_out * g.C_in * 2 : 0, 0x00020000);
    const uint32_t idx_row = (uint32_t)((cob * 32 + n_l) * g.C_in);
    auto load_idx = [&](int q, uint32_t (&k)[4]) {             // (of channels that do not exist: anything, their activations are zeros)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ci = 8 * q + 2 * u + h;
            k[u] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(
                ires, (int)(cob * 32 + n_l < g.C_out && ci < g.C_in ? (idx_row + (uint32_t)ci) * 2u : SD_NONE), 0, 0);
        }
    };
    uint32_t kn[4];
    u32x2 c = {0, 0};
    if constexpr (INDEXED) load_idx(q0, kn);
    else c = codes[(int64_t)min(q0, quads - 1) * 64];
    // [wave][stage][channel of the pair][32 NL positions]
    __shared__ float staged[NL > 0 ? 4 : 1][2][2][NL > 0 ? 32 * NL : 1];
    auto put = [&](int stage, const float (&b)[NL > 0 ? NL : 1]) {
#pragma unroll
        for (int i = 0; i < NL; ++i) staged[wave][stage][h][32 * i + n_l] = b[i];
        __builtin_amdgcn_wave_barrier();                       // (other lanes read them; no instruction)
    };
    auto taps = [&](int stage, float (&b)[9]) {
        const float *const at = &staged[wave][stage][h][0] + (window >> 2);
#pragma unroll
        for (int t = 0; t < 9; ++t) b[t] = at[(t / 3) * rows.pitch + t % 3];
        __builtin_amdgcn_wave_barrier();
    };
    float first[2][NL > 0 ? NL : 1];
    if constexpr (NL > 0) {
        load_pair(4 * q0, first[0]);
        load_pair(4 * q0 + 1, first[1]);
        load_pair(4 * q0 + 2, G[0]);
        load_pair(4 * q0 + 3, G[1]);
    } else {
#pragma unroll
        for (int u = 0; u < 3; ++u) load_pair(4 * q0 + u, B[u]);
    }
    __shared__ uint16_t book[INDEXED ? 512 : 1];               // in window order, bit t: tap t is -1
    if constexpr (INDEXED) {
        for (int k = (int)threadIdx.x; k < ix.K; k += 256) book[k] = (uint16_t)(code_to_window_order(ix.codebook[k] & 511u) ^ 511u);
    }
    // accumulator register i is row 8 (i / 4) + 4 h + i % 4; a wave stores all sixteen, or four of the sums of four waves
    constexpr int NR = 16 / S;
    const int row0 = S == 1 ? 0 : 8 * wave;
    float al[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) al[i] = alpha[min(cob * 32 + row0 + 8 * (i >> 2) + 4 * h + (i & 3), g.C_out - 1)];
    v16f acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.0f;
    auto look_up = [&](const uint32_t (&k)[4]) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = book[min(k[u], (uint32_t)ix.K - 1u)];
        return (u32x2){v[0] | v[1] << 16, v[2] | v[3] << 16};
    };
    if constexpr (INDEXED) __syncthreads();
    if constexpr (NL > 0) {
        put(0, first[0]);
        put(1, first[1]);
        taps(0, B[0]);
    }
    if (my_id >= n_blocks) return;                             // (S = 4: never, the grid is n_blocks)
    for (int q = q0; q < q1; ++q) {
        u32x2 cn;
        if constexpr (INDEXED) {
            c = look_up(kn);
            load_idx(q + 1, kn);
        } else {
            cn = codes[(int64_t)min(q + 1, quads - 1) * 64];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int p = 4 * q + u;
            if (p < p_end) {                                   // (wave-uniform)
                if constexpr (NL > 0) {
                    put(u & 1, G[u & 1]);                      // pair p + 2, over this one, whose taps have been read
                    load_pair(p + 4, G[u & 1]);
                    taps((u & 1) ^ 1, B[(u & 1) ^ 1]);
                } else {
                    if (p + 3 < p_end) load_pair(p + 3, B[(u + 3) & 3]);
                }
                const uint32_t code = c[u >> 1] >> (16 * (u & 1));     // bit t: tap t is -1
#pragma unroll
                for (int t = 0; t < 9; ++t) {
                    const float w = __uint_as_float(((code << (31 - t)) & 0x80000000u) | 0x3f800000u);
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, B[NL > 0 ? u & 1 : u][t], acc[t], 0, 0, 0);
                }
            }
        }
        if constexpr (!INDEXED) c = cn;
    }
    const uint32_t yo = mine ? (((n - n0) * (uint32_t)g.C_out + 4u * (uint32_t)h) * HoWo + r) * 4u : SD_NONE;
    float sum[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
        sum[i] = ((acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i])) + ((acc[4][i] + acc[5][i]) + (acc[6][i] + acc[7][i])) + acc[8][i];
    if constexpr (S > 1) {
        __shared__ float part[S][16][64];
#pragma unroll
        for (int i = 0; i < 16; ++i) part[wave][i][lane] = sum[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int r16 = NR * wave + i;
            sum[i] = (part[0][r16][lane] + part[1][r16][lane]) + (part[2][r16][lane] + part[3][r16][lane]);
        }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int co = cob * 32 + row0 + 8 * (i >> 2) + (i & 3);
        const uint32_t o = co + 4 * h < g.C_out ? yo : SD_NONE;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sum[i] * al[i]), yres, (int)o, (int)((uint32_t)min(co, g.C_out - 1) * HoWo * 4u), 2);
    }
}

// The same sums with the activations as three bf16 pieces, x = hi + mid + lo exactly (eight bits of the significand each), on
// v_mfma_f32_32x32x16_bf16: products with +-1 are exact, sums are fp32, and sixteen channels of a tap take 96 clocks of a SIMD for 512.
// A wave owns 32 pixels x 64 output channels; it brings its rows to LDS sixteen channels at a time, already in pieces, so that
// a tap is three reads for six products, and hi has accumulators apart from mid and lo.  Measured, fp32 unit -> pieces (one call, us): 64 -> 64
// 8x8 batch 256 20.4 -> 11.3, of which the matrix unit's share falls from 7.7 to 1.5 and what is left is one round of workgroups' loads,
// splitting (six instructions a value) and stores; 128 -> 128 14x14 batch 32 33 -> 15, 512 -> 512 7x7 batch 4 30.2 -> 23.2, 16 -> 32 16x16 batch 200
// 12.0 -> 8.7.  Error of the sums against 64 bits: 5.3e-8 for 1.03e-7 at 64 channels, 5.9e-8 for 2.2e-7 at 512 (a rounding per sixteen
// channels of a tap for one per two).
// Values that three pieces do not hold (subnormal remainders, infinities, NaN) send the wave's sixteen channels through the fp32 unit.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int S, int CB, int NL, bool INDEXED>
__global__ __launch_bounds__(256, 2)
void subbit_f32_split_kernel(const float *__restrict__ x, const uint32_t *__restrict__ wq, const float *__restrict__ alpha,
                             float *__restrict__ y, Geom g, int n_cob, int quads, uint32_t n_blocks, SdRows rows, SdIndexed ix)
{
    const int lane = threadIdx.x & 63, n_l = lane & 31, h = lane >> 5;
    const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t my_id = S == 1 ? blockIdx.x * 4u + (uint32_t)wave : blockIdx.x, id = min(my_id, n_blocks - 1u);
    const uint32_t cob_groups = (uint32_t)(n_cob + CB - 1) / CB, blk = id / cob_groups;
    const int cob0 = CB * (int)(id - blk * cob_groups);
    const uint32_t P = (uint32_t)g.P, HoWo = (uint32_t)g.HoWo;
    const uint32_t n0 = blk * 32u / HoWo;
    const bool mine = blk * 32u + (uint32_t)n_l < P;
    const uint32_t pp = min(blk * 32u + (uint32_t)n_l, P - 1u);
    const uint32_t n = pp / HoWo, r = pp - n * HoWo;
    const int ho = (int)(r / (uint32_t)g.Wo), wo = (int)r - ho * g.Wo;

    const int64_t x_image = (int64_t)g.C_in * g.H * g.W, y_image = (int64_t)g.C_out * g.HoWo;
    const int64_t lim = 0x7fffffff;
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(x + (int64_t)n0 * x_image), 0, (int)min((int64_t)(g.N - (int)n0) * x_image * 4, lim), 0x00020000);
    const __amdgpu_buffer_rsrc_t yres = __builtin_amdgcn_make_buffer_rsrc(
        y + (int64_t)n0 * y_image, 0, (int)min((int64_t)(g.N - (int)n0) * y_image * 4, lim), 0x00020000);
    const uint32_t plane = (uint32_t)(g.H * g.W) * 4u;
    const SdBlock b0 = sd_block(g, blk);
    const int window = sd_window(g, rows, b0, n, ho, wo);      // position of the window's first pixel
    uint32_t off[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const SdPixel p = sd_pixel(g, rows, b0, 32 * i + n_l);
        off[i] = p.in ? (uint32_t)p.image * (uint32_t)x_image * 4u + (uint32_t)h * plane + (uint32_t)(p.h * g.W + p.w) * 4u : SD_NONE;
    }
    const int pairs = (g.C_in + 1) >> 1, octs = (quads + 1) >> 1;
    const int o0 = S == 1 ? 0 : wave * octs / S, o1 = S == 1 ? octs : (wave + 1) * octs / S;
    float v[NL][8];                                            // lane half h: channels 16 o + 2 j + h
    auto load_x = [&](int o) {                                 // (past the last channel: zeros, nothing read)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int p = 8 * o + j;
            const bool have = 2 * p + h < g.C_in;
            const uint32_t at = 2u * (uint32_t)min(p, pairs - 1) * plane;
#pragma unroll
            for (int i = 0; i < NL; ++i)
                v[i][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xres, (int)(have ? off[i] : SD_NONE), (int)at, 0));
        }
    };
    // Codes of the channels, two to a word: word m of a block has those of j = 2 m and 2 m + 1.  (Of a quad past the last: any.)
    __shared__ uint16_t book[INDEXED ? 512 : 1];               // in window order, bit t: tap t is -1
    const __amdgpu_buffer_rsrc_t ires =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(ix.idx), 0, INDEXED ? g.C_out * g.C_in * 2 : 0, 0x00020000);
    uint32_t k[CB][8], c[CB][4];
    auto load_w = [&](int o) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const int cob = min(cob0 + cb, n_cob - 1);
            if constexpr (INDEXED) {
                const int co = cob * 32 + n_l;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int ci = 16 * o + 2 * j + h;
                    k[cb][j] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(
                        ires, (int)(co < g.C_out && ci < g.C_in ? (uint32_t)(co * g.C_in + ci) * 2u : SD_NONE), 0, 0);
                }
            } else {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const u32x2 w = *((const u32x2 *)wq + ((int64_t)cob * quads + min(2 * o + q, quads - 1)) * 64 + lane);
                    k[cb][2 * q] = w[0];
                    k[cb][2 * q + 1] = w[1];
                }
            }
        }
    };
    auto take_w = [&]() {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                if constexpr (INDEXED)
                    c[cb][m] = (uint32_t)book[min(k[cb][2 * m], (uint32_t)ix.K - 1u)] | (uint32_t)book[min(k[cb][2 * m + 1], (uint32_t)ix.K - 1u)] << 16;
                else c[cb][m] = k[cb][m];
            }
    };
    load_x(min(o0, octs - 1));
    load_w(min(o0, octs - 1));
    v16f hi[CB], low[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) hi[cb][i] = low[cb][i] = 0.0f;
    // [wave][piece][lane half][position]: eight channels of a half as bf16; as they are, [wave][half of the eight][lane half][position]
    __shared__ u32x4 stage[4][3][2][32 * NL];
    if constexpr (INDEXED) {
        for (int i = (int)threadIdx.x; i < ix.K; i += 256) book[i] = (uint16_t)(code_to_window_order(ix.codebook[i] & 511u) ^ 511u);
        __syncthreads();
    }
    if (my_id >= n_blocks) return;                             // (S = 4: never, the grid is n_blocks)
    for (int o = o0; o < o1; ++o) {
        uint32_t lost = 0;
        float odd = 0.0f;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            u32x4 piece[3];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                uint32_t f[3][2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float a = v[i][2 * m + e];
                    f[0][e] = __float_as_uint(a);
                    const float b = a - __uint_as_float(f[0][e] & 0xffff0000u);
                    f[1][e] = __float_as_uint(b);
                    f[2][e] = __float_as_uint(b - __uint_as_float(f[1][e] & 0xffff0000u));
                    lost |= f[2][e] & 0xffffu;
                    odd = __builtin_fmaf(a, 0.0f, odd);
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) piece[q][m] = __builtin_amdgcn_perm(f[q][1], f[q][0], 0x07060302u);     // the upper halves
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) stage[wave][q][h][32 * i + n_l] = piece[q];
        }
        const bool pieces = __ballot(lost != 0 || odd != odd) == 0;        // (wave-uniform)
        if (!pieces) {
#pragma unroll
            for (int i = 0; i < NL; ++i)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    stage[wave][q][h][32 * i + n_l] = (u32x4){__float_as_uint(v[i][4 * q]), __float_as_uint(v[i][4 * q + 1]),
                                                              __float_as_uint(v[i][4 * q + 2]), __float_as_uint(v[i][4 * q + 3])};
        }
        __builtin_amdgcn_wave_barrier();                       // (other lanes read them; within a wave LDS keeps the order)
        take_w();
        if (o + 1 < o1) {
            load_x(o + 1);
            load_w(o + 1);
        }
        if (pieces) {
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int at = window + (t / 3) * rows.pitch + t % 3;
                u32x4 B[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) B[q] = stage[wave][q][h][at];
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    u32x4 A;
#pragma unroll
                    for (int m = 0; m < 4; ++m) A[m] = ((c[cb][m] << (15 - t)) & 0x80008000u) | 0x3f803f80u;
                    const bf16x8 w = __builtin_bit_cast(bf16x8, A);
                    hi[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, __builtin_bit_cast(bf16x8, B[0]), hi[cb], 0, 0, 0);
                    low[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, __builtin_bit_cast(bf16x8, B[1]), low[cb], 0, 0, 0);
                    low[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, __builtin_bit_cast(bf16x8, B[2]), low[cb], 0, 0, 0);
                }
            }
        } else {
            for (int t = 0; t < 9; ++t) {
                const int at = window + (t / 3) * rows.pitch + t % 3;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const f32x4 B = __builtin_bit_cast(f32x4, stage[wave][q][h][at]);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) {
                            const uint32_t code = c[cb][2 * q + (u >> 1)] >> (16 * (u & 1));
                            const float w = __uint_as_float(((code << (31 - t)) & 0x80000000u) | 0x3f800000u);
                            hi[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, B[u], hi[cb], 0, 0, 0);
                        }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    // accumulator register i is row 8 (i / 4) + 4 h + i % 4; a wave stores all 16 CB, or a quarter of the sums of four waves
    constexpr int NR = 16 * CB / S;
    const int r0 = S == 1 ? 0 : NR * wave;
    float al[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int q = r0 + i;
        al[i] = alpha[min((cob0 + (q >> 4)) * 32 + 8 * ((q & 15) >> 2) + 4 * h + (q & 3), g.C_out - 1)];
    }
    const uint32_t yo = mine ? (((n - n0) * (uint32_t)g.C_out + 4u * (uint32_t)h) * HoWo + r) * 4u : SD_NONE;
    float sum[16 * CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) sum[16 * cb + i] = hi[cb][i] + low[cb][i];
    if constexpr (S > 1) {
        static_assert(sizeof(stage[0]) >= 16 * CB * 64 * sizeof(float), "a wave's sums lie over its own rows");
        float *const part = (float *)&stage[wave][0][0][0];
#pragma unroll
        for (int i = 0; i < 16 * CB; ++i) part[i * 64 + lane] = sum[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            float f[S];
#pragma unroll
            for (int w = 0; w < S; ++w) f[w] = ((const float *)&stage[w][0][0][0])[(r0 + i) * 64 + lane];
            sum[i] = (f[0] + f[1]) + (f[2] + f[3]);
        }
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int q = r0 + i, co = (cob0 + (q >> 4)) * 32 + 8 * ((q & 15) >> 2) + (q & 3);
        const uint32_t o = co + 4 * h < g.C_out ? yo : SD_NONE;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(sum[i] * al[i]), yres, (int)o, (int)((uint32_t)min(co, g.C_out - 1) * HoWo * 4u), 2);
    }
}

__global__ __launch_bounds__(256)
void subbit_f32_dense_prep_kernel(const uint16_t *__restrict__ codebook, const uint16_t *__restrict__ idx, int C_in, int C_out, int K,
                                  int quads, int n, uint16_t *__restrict__ wq)
{
    const int gid = blockIdx.x * 256 + threadIdx.x;            // [cob][quad][lane][pair of the quad]
    if (gid >= n) return;
    const int lane = (gid >> 2) & 63, cq = gid >> 8;
    const int cob = cq / quads, q = cq - cob * quads;
    const int co = cob * 32 + (lane & 31), ci = 8 * q + 2 * (gid & 3) + (lane >> 5);
    uint32_t code = 0;
    if (co < C_out && ci < C_in) code = code_to_window_order(codebook[min((int)idx[(int64_t)co * C_in + ci], K - 1)] & 511u) ^ 511u;
    wq[gid] = (uint16_t)code;
}

struct SdPlan { int n_cob, quads; int64_t n_blocks; };

SdPlan sd_plan(const Geom &g)
{
    SdPlan p;
    p.n_cob = (g.C_out + 31) / 32;
    p.quads = (g.C_in + 7) / 8;
    p.n_blocks = (g.P + 31) / 32 * p.n_cob;
    return p;
}

bool use_dense(const Geom &g)
{
    if (tuning(SNN_TUNE_F32_WAVES) != SNN_TUNE_AUTO) return false;
    // its words lie in the two-stage form's workspace (up to seven padding channels: 14 C_out bytes of the 20 KB before the
    // offsets); 32-bit offsets inside the images of 32 pixels
    const int64_t lim = ((int64_t)1 << 31) - 4096, images = (g.HoWo - 1 + 31) / g.HoWo + 1;
    if (g.C_out > 512 || images * g.C_in * g.H * g.W * 4 >= lim || images * g.C_out * g.HoWo * 4 >= lim || g.P >= lim ||
        sd_plan(g).n_blocks >= lim || (int64_t)sd_plan(g).n_cob * sd_plan(g).quads * 256 >= lim)
        return false;
    // In pieces (sd_split) it is the faster one at every K: K = 4 64 -> 64 8x8 batch 256 19.8 -> 11.7 (one call), 16 -> 16 32x32 batch 128 21.9 -> 15.6,
    // 12 -> 12 28x28 batch 200 20.7 -> 18.3.
    // On the fp32 unit nine multiply-adds per output channel stand against nine per subset member and a gather: the two-stage form is left
    // the small subsets with few output channels.  Measured on layers that the pieces do not take, two-stage (its best workgroup) -> dense, prepared
    // weights, us: 8 -> 8 56x56 batch 32 K = 8 11.1 -> 12.7, K = 15 13.0 -> 12.6, K = 32 18.7 -> 12.6; 16 -> 16 56x56 batch 32 K = 8 16.8 -> 18.9,
    // K = 16 21.5 -> 18.9; 64 -> 64 56x56 batch 32 K = 8 87 -> 99, K = 16 97 -> 99, K = 32 135 -> 99; 512 -> 512 7x7 batch 8 K = 4 217 -> 36 (C_out).
    // (Eight channels and fewer to 32 and more are faster here at every K, 3 -> 64 56x56 batch 32 K = 8 30 -> 18.)
    // Relative error of the sums against 64 bits: 1.0e-7 for 1.6e-7 at 64 channels, 2.2e-7 for 4.1e-7 at 512.  That error is why K >= 16 is the
    // whole rule: where 64 pixels' responses are shared by 33 to 128 output channels and the pixels fill the chip, the two-stage form
    // is the faster one up to K = 32, 64 -> 128 56x56 batch 32 K = 16 145 -> 190, K = 32 169 -> 189, 14x53 batch 64 K = 16 86 -> 95; so it is for
    // 128 -> 200, 56x56 batch 32 K = 16 554 -> 585.
    return g.K >= 16 || g.C_out >= 256 || sd_split(g);
}

}  // namespace

size_t subbit_f32_workspace_bytes(const Geom &g)
{
    // the widest padding of C_out any launch shape uses (the shape may change with the tuning knob between the
    // size query and the call)
    const int COP = (g.C_out + 511) / 512 * 512;
    return align_up(512 * sizeof(uint32_t), 256) + align_up(512 * 9 * sizeof(float), 256) + align_up((size_t)g.C_in * COP * sizeof(uint16_t), 256);
}

int launch_subbit_f32(const Geom &g, const void *x, const uint16_t *codebook, const uint16_t *idx,
                      const float *alpha, float *y, void *ws, hipStream_t s, int phases)
{
    if (use_dense(g)) {
        const SdPlan p = sd_plan(g);
        const bool split = p.quads >= 4, pieces = sd_split(g);
        const int64_t n_wgs = split ? p.n_blocks : (p.n_blocks + 3) / 4;
        const int staged = sd_staged(g);
        const SdSplit sp = sd_split_plan(g);
        const bool look_up = phases == SNN_PHASE_BOTH && (pieces ? sd_pieces_look_up(g, sp) : sd_looks_up(g, staged, p.quads, n_wgs));
        if ((phases & SNN_PHASE_PREPARE) && !look_up) {
            const int words = p.n_cob * p.quads * 256;
            hipLaunchKernelGGL(subbit_f32_dense_prep_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, codebook, idx, g.C_in, g.C_out,
                               g.K, p.quads, words, (uint16_t *)ws);
            const int rc = check_launch();
            if (rc != SNN_OK) return rc;
        }
        if (!(phases & SNN_PHASE_CONVOLVE)) return SNN_OK;
        if (pieces) {
            auto pick_split = [&](auto nl, auto cb) {
                constexpr int NL = decltype(nl)::value, CB = decltype(cb)::value;
                if (look_up) return sp.four ? subbit_f32_split_kernel<4, CB, NL, true> : subbit_f32_split_kernel<1, CB, NL, true>;
                return sp.four ? subbit_f32_split_kernel<4, CB, NL, false> : subbit_f32_split_kernel<1, CB, NL, false>;
            };
            auto pick_loads = [&](auto cb) {
                return sp.loads == 3   ? pick_split(std::integral_constant<int, 3>{}, cb)
                       : sp.loads == 4 ? pick_split(std::integral_constant<int, 4>{}, cb) : pick_split(std::integral_constant<int, 6>{}, cb);
            };
            const auto kern = sp.CB == 2 ? pick_loads(std::integral_constant<int, 2>{}) : pick_loads(std::integral_constant<int, 1>{});
            hipLaunchKernelGGL(kern, dim3((unsigned)sp.n_wgs), dim3(256), 0, s, (const float *)x, (const uint32_t *)ws,
                               alpha, y, g, p.n_cob, p.quads, (uint32_t)sp.blocks, sd_rows(g), SdIndexed{codebook, idx, g.K});
            return check_launch();
        }
        // (rows through LDS: only of eight channels and fewer here, one wave to a block)
        auto pick = [&](auto nl) {
            constexpr int NL = decltype(nl)::value;
            if constexpr (NL == 0) {
                if (split) return look_up ? subbit_f32_dense_kernel<4, NL, true> : subbit_f32_dense_kernel<4, NL, false>;
            }
            return look_up ? subbit_f32_dense_kernel<1, NL, true> : subbit_f32_dense_kernel<1, NL, false>;
        };
        const auto kern = staged == 3   ? pick(std::integral_constant<int, 3>{})
                          : staged == 4 ? pick(std::integral_constant<int, 4>{})
                          : staged == 6 ? pick(std::integral_constant<int, 6>{})
                                        : pick(std::integral_constant<int, 0>{});
        hipLaunchKernelGGL(kern, dim3((unsigned)n_wgs), dim3(256), 0, s, (const float *)x, (const uint32_t *)ws, alpha, y, g, p.n_cob, p.quads,
                           (uint32_t)p.n_blocks, sd_rows(g), SdIndexed{codebook, idx, g.K});
        return check_launch();
    }
    const F32Cfg c = pick_f32_cfg(g);
    const int COP = (g.C_out + c.COB - 1) / c.COB * c.COB;
    uint32_t *codes = (uint32_t *)ws;
    float *coef = (float *)((char *)ws + align_up(512 * sizeof(uint32_t), 256));
    uint16_t *offs = (uint16_t *)((char *)coef + align_up(512 * 9 * sizeof(float), 256));
    const int64_t tiles = (g.P + SF_TP - 1) / SF_TP;
    const int cblocks = COP / c.COB;
    if (tiles > 0x7fffffffLL || cblocks > 65535) return SNN_ERR_UNSUPPORTED;
    const int CIC = c.CIC;
    const size_t lds = c.lds;
    if (lds > 160 * 1024) return SNN_ERR_UNSUPPORTED;
    const int64_t nprep = (int64_t)g.C_in * COP + 512;
    if (phases & SNN_PHASE_PREPARE)
        hipLaunchKernelGGL(subbit_f32_prep_kernel, dim3((unsigned)((nprep + 255) / 256)), dim3(256), 0, s, codebook, idx,
                           g.C_in, g.C_out, COP, g.K, codes, coef, offs);
    if (!(phases & SNN_PHASE_CONVOLVE)) return check_launch();
    const dim3 grid((unsigned)tiles, (unsigned)cblocks);
#define SNN_F32_CASE(J_, NW_)                                                                                  \
    case J_ * 100 + NW_: {                                                                                     \
        auto kern = subbit_f32_kernel<J_, NW_>;                                                                \
        static LdsGrant grant;                                                                                 \
        if (grant_dynamic_lds((const void *)kern, lds, grant) != SNN_OK) return SNN_ERR_LAUNCH;                \
        hipLaunchKernelGGL(kern, grid, dim3(NW_ * 64), lds, s, (const float *)x, coef, offs, alpha, y, g, COP, \
                           CIC);                                                                               \
    } break;
    switch (c.J * 100 + c.NW) {
        SNN_F32_CASE(1, 4)
        SNN_F32_CASE(2, 4)
        SNN_F32_CASE(4, 4)
        SNN_F32_CASE(8, 4)
        SNN_F32_CASE(1, 8)
        SNN_F32_CASE(2, 8)
        SNN_F32_CASE(4, 8)
        SNN_F32_CASE(8, 8)
        SNN_F32_CASE(1, 16)
        SNN_F32_CASE(2, 16)
        SNN_F32_CASE(4, 16)
        SNN_F32_CASE(8, 16)
    default:
        return SNN_ERR_UNSUPPORTED;
    }
#undef SNN_F32_CASE
    return check_launch();
}

}  // namespace snn

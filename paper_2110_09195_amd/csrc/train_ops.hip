// Training-side operations of a sub-bit layer (Alg. 1 backward lines, Sec. 4.2 / 4.3):
//   * the straight-through estimator for the real-valued kernels (Eq. 3) together with the gradient of
//     the subset tensor p, which is the gradient of its sign memory m: per member, the sum of the
//     gradients of the binarised kernels assigned to it (backward of Eq. 5 / Eq. 6);
//   * the update of the sign memory m from p with the hysteresis threshold theta (Eq. 4), the 9-bit
//     codes of the refined subset, and the check for repeated members (Sec. 4.3).
// All of it is memory-bound streaming over [n][9] floats plus a K x 9 reduction.
#include <algorithm>

#include "snn_internal.h"

namespace snn {

namespace {

constexpr int TB_THREADS = 256;
constexpr int TB_UNIT = 112;                         // kernels that one 16-byte load of every thread covers (252 of 256 busy)

// 16-byte loads per thread and tensor: as many as leave enough blocks to fill the chip.  A block's time is a round
// trip to memory and its LDS additions; its K x 9 partial sums are what more blocks cost.
// (4096 kernels 4.1 us, 16384 3.8, 65536 6.0, 262144 11.9.)
constexpr int64_t TB_ONE_MAX = (int64_t)TB_UNIT * 320, TB_TWO_MAX = (int64_t)TB_UNIT * 1280;      // kernels: one load, two loads up to here
inline int tb_units(int64_t n) { return n <= TB_ONE_MAX ? 1 : n <= TB_TWO_MAX ? 2 : 4; }
inline int64_t tb_blocks(int64_t n)
{
    const int64_t per = (int64_t)TB_UNIT * tb_units(n);
    return (n + per - 1) / per;
}

// Copies of the sums by member that a block adds to with atomics: 36 KB of LDS at most
__host__ __device__ constexpr int tb_copies(int K) { return K <= 256 ? 4 : 2; }
inline size_t tb_copies_bytes(int K) { return (size_t)(tb_copies(K) * K * 9 + 3) / 4 * 16; }

__device__ __forceinline__ void clear_copies(float *acc, int n)        // (up to the next multiple of four)
{
    for (int i = 4 * threadIdx.x; i < n; i += 4 * TB_THREADS) *(float4 *)(acc + i) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

__device__ __forceinline__ void store_copies(const float *acc, int copies, int K9, float *__restrict__ dst)
{
    for (int e = threadIdx.x; e < K9; e += TB_THREADS) {
        const float lo = acc[e] + acc[K9 + e];
        dst[e] = copies == 4 ? lo + (acc[2 * K9 + e] + acc[3 * K9 + e]) : lo;
    }
}

// Pass 1: g_w = g_wbar where w in (-1, 1) (element-wise), else 0; per block, the sums of g_wbar by member, written as one
// partial [K][9] per block.
//
// The sums by member are a product [member][kernel] x [kernel][tap] with the indices as a one-hot matrix, on the fp32 matrix
// unit (products with 1 and 0 are exact, sums are fp32; a wave's chain is a sixteenth of the block).  16 M members
// cost 32 M clocks of a SIMD per four kernels, which stays near the 110 bytes per kernel of memory traffic up to
// M = 4 (where the line lies: launch_project_backward).  With LDS float atomics instead, which was the whole kernel's time at any layout of the lanes (290 clocks
// per 64 additions, equal addresses among them or not), 262144 kernels at K = 32 take 17 us, here 11.9 (4096 kernels: 8.6
// with one kernel per thread, here 4.1).
// A zero times an infinity would reach members that it does not belong to: blocks with a value that is not finite add with
// LDS float atomics, and so do (M = 0) the subsets whose one-hot rows are mostly zeros.  Each wave adds to a copy of the sums of its
// own while four copies fit beside other blocks (K <= 256; two beyond), which keeps the chains of roundings as short as the product's.
template <int U, int M, bool WHOLE>
__device__ __forceinline__ void project_backward_block(const float *__restrict__ wb, const float *__restrict__ gb,
                                                       const uint16_t *__restrict__ ib, int cnt, int K, float *__restrict__ ob,
                                                       float *__restrict__ dst, float *lds)
{
    constexpr int PER = TB_UNIT * U;
    constexpr int STAGE = M > 0 ? PER * 9 + 16 : 0;  // (lanes 9..15 of the last kernel read past it)
    __shared__ int member[PER + 1];
    __shared__ int not_finite;
    float *const acc = lds + STAGE;
    const int tid = threadIdx.x;
    const int ne = cnt * 9;
    const int copies = tb_copies(K);
    float wv[U][4], gv[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e = (u * TB_THREADS + tid) * 4;
        if constexpr (WHOLE) {                       // (threads past the end load the last elements again)
            const int at = min(e, PER * 9 - 4);
            const float4 a = *(const float4 *)(wb + at), b = *(const float4 *)(gb + at);
            wv[u][0] = a.x; wv[u][1] = a.y; wv[u][2] = a.z; wv[u][3] = a.w;
            gv[u][0] = b.x; gv[u][1] = b.y; gv[u][2] = b.z; gv[u][3] = b.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int at = min(e + j, ne - 1);
                wv[u][j] = wb[at];
                gv[u][j] = e + j < ne ? gb[at] : 0.0f;
            }
        }
    }
    for (int c = tid; c <= PER; c += TB_THREADS) {
        const int k = min((int)ib[min(c, cnt - 1)], K - 1);
        member[c] = c < cnt ? k : -1;
    }
    if (tid == 0) not_finite = M == 0;
    __syncthreads();
    bool odd = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e = (u * TB_THREADS + tid) * 4;
        if (e >= PER * 9) break;
        float o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] = wv[u][j] > -1.0f && wv[u][j] < 1.0f ? gv[u][j] : 0.0f;
            odd |= !__builtin_isfinite(gv[u][j]);
        }
        if constexpr (WHOLE) {
            *(float4 *)(ob + e) = make_float4(o[0], o[1], o[2], o[3]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (e + j < ne) ob[e + j] = o[j];
        }
        if constexpr (M > 0) *(float4 *)(lds + e) = make_float4(gv[u][0], gv[u][1], gv[u][2], gv[u][3]);
    }
    if (M > 0 && odd) not_finite = 1;
    if constexpr (M > 0) {
        if (tid < 16) lds[PER * 9 + tid] = 0.0f;
    }
    __syncthreads();
    if (not_finite) {                                // (block-uniform)
        clear_copies(acc, copies * K * 9);
        __syncthreads();
        float *const mine = acc + ((tid >> 6) & (copies - 1)) * K * 9;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = (u * TB_THREADS + tid) * 4;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = (e + j) / 9;
                if (e + j < ne) atomicAdd(&mine[member[c] * 9 + e + j - 9 * c], gv[u][j]);
            }
        }
        __syncthreads();
        store_copies(acc, copies, K * 9, dst);
        return;
    }
    if constexpr (M > 0) {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        // v_mfma_f32_16x16x4_f32: lane (i = lane % 16, q = lane / 16) holds A[member i][kernel q], B[kernel q][tap i] and
        // D[members 4 q .. 4 q + 3][tap i]
        const int lane = tid & 63, wave = tid >> 6, i = lane & 15, q = lane >> 4;
        f32x4 sum[M];
#pragma unroll
        for (int m = 0; m < M; ++m) sum[m] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 7
        for (int step = 0; step < PER / 16; ++step) {
            const int c = 16 * step + 4 * wave + q;
            const float g = lds[c * 9 + i];          // taps 9..15: whatever follows, in columns nobody reads
            const int k = member[c] - i;
#pragma unroll
            for (int m = 0; m < M; ++m) sum[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(k == 16 * m ? 1.0f : 0.0f, g, sum[m], 0, 0, 0);
        }
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = 16 * m + 4 * q + r;
                if (i < 9 && k < K) acc[(wave * K + k) * 9 + i] = sum[m][r];
            }
        __syncthreads();
        store_copies(acc, 4, K * 9, dst);
    }
}

template <int U, int M>
__global__ __launch_bounds__(TB_THREADS)
void project_backward_kernel(const float *__restrict__ w, const float *__restrict__ g_wbar,
                             const uint16_t *__restrict__ idx, int64_t n, int K, float *__restrict__ g_w,
                             float *__restrict__ partial, int vec)
{
    constexpr int PER = TB_UNIT * U;                 // a multiple of four: every block starts 16-byte aligned if the tensors do
    extern __shared__ __align__(16) float lds[];
    const int64_t c0 = (int64_t)blockIdx.x * PER;
    const int cnt = (int)min((int64_t)PER, n - c0);
    float *const dst = partial + (int64_t)blockIdx.x * K * 9;
    if (vec && cnt == PER)                           // (block-uniform)
        project_backward_block<U, M, true>(w + c0 * 9, g_wbar + c0 * 9, idx + c0, cnt, K, g_w + c0 * 9, dst, lds);
    else
        project_backward_block<U, M, false>(w + c0 * 9, g_wbar + c0 * 9, idx + c0, cnt, K, g_w + c0 * 9, dst, lds);
}

// The same with the atomics on larger blocks: two kernels per thread.  For many kernels the partial sums, K x 9 per block, are what
// counts, and the product's one-hot rows of large subsets are.
constexpr int TB_LARGE = 2 * TB_THREADS;

__global__ __launch_bounds__(TB_THREADS)
void project_backward_large_kernel(const float *__restrict__ w, const float *__restrict__ g_wbar, const uint16_t *__restrict__ idx,
                                   int64_t n, int K, float *__restrict__ g_w, float *__restrict__ partial)
{
    extern __shared__ __align__(16) float lds[];
    const int tid = threadIdx.x, K9 = K * 9, copies = tb_copies(K);
    constexpr int Q = TB_LARGE / TB_THREADS;
    const int64_t c0 = (int64_t)blockIdx.x * TB_LARGE + tid;
    int k[Q];
    float wv[Q][9], gv[Q][9];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t c = min(c0 + q * TB_THREADS, n - 1);
        k[q] = min((int)idx[c], K - 1);
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            wv[q][t] = w[c * 9 + t];
            gv[q][t] = g_wbar[c * 9 + t];
        }
    }
    clear_copies(lds, copies * K9);
    __syncthreads();
    float *const mine = lds + ((tid >> 6) & (copies - 1)) * K9;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t c = c0 + q * TB_THREADS;
        if (c < n) {
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                g_w[c * 9 + t] = wv[q][t] > -1.0f && wv[q][t] < 1.0f ? gv[q][t] : 0.0f;
                atomicAdd(&mine[k[q] * 9 + t], gv[q][t]);
            }
        }
    }
    __syncthreads();
    store_copies(lds, copies, K9, partial + (int64_t)blockIdx.x * K9);
}

// Both gradients of few kernels in one launch: block k < K sums the gradients of member k's kernels, the blocks behind them write g_w.
// A member's block reads all indices, which is what bounds it (a quarter of a microsecond per 1024); a wave keeps the numbers of those that are
// k in a piece of LDS of its own (in order, so that the sum is the same from run to run) and adds their gradients, seven kernels of
// nine taps at a time.  No partial sums pass through memory, and no second launch waits for them.  Two launches -> one, us, replayed from a
// graph (from Python, call by call), indices even over the members / skewed as in trained layers (Zipf 1.1):
//   K = 4   1024 kernels 4.5 -> 2.5 (6.0 -> 3.4) / the same       4096 4.8 -> 3.9 (6.3 -> 4.1) / 4.8 -> 4.2 (6.2 -> 4.3)
//           5120 4.8 -> 4.3 (6.2 -> 4.4) / 4.9 -> 4.9 (6.2 -> 5.0)   8192 5.0 -> 5.6 (6.3 -> 5.7) / 5.1 -> 6.4 (6.2 -> 6.4)
//   K = 8   4096 4.8 -> 3.4 (6.3 -> 3.6) / 4.8 -> 4.1 (6.3 -> 4.1)   8192 5.1 -> 4.9 (6.3 -> 5.0) / 5.1 -> 6.0 (6.2 -> 6.0)
//   K = 16  8192 5.2 -> 4.1 (6.3 -> 4.2) / 5.2 -> 5.7 (6.2 -> 5.8)   K = 32  8192 5.6 -> 3.9 (6.3 -> 4.0) / 5.6 -> 5.6 (6.1 -> 5.6)
//   K = 512 4096 8.0 -> 3.8 (8.4 -> 3.8) / 8.0 -> 4.1 (8.3 -> 4.1)   8192 10.0 -> 4.5 (10.4 -> 4.5) / 10.0 -> 5.5 (10.4 -> 5.5)
// The block of the most frequent member is the longest.  Hence the lines: 5120 kernels of fewer than eight members, above which
// skewed indices are slower from Python too, and 8192, what the lanes' indices hold, of more: between 8 and 31 members skewed indices are up to a
// sixth slower there in a graph (even ones up to a fifth faster) and both are faster from Python.  (All of 8192 kernels in one of
// 32 members: 5.7 -> 6.5 and 6.3 -> 6.6; 16384 kernels would take 9.9 for 6.3.)  Error of the sums against 64 bits, K = 4 to 32:
// 8.2e-8 to 1.0e-7 -> 7.8e-8 to 9.8e-8.
constexpr int TM_THREADS = 1024, TM_WAVES = TM_THREADS / 64;
constexpr int TM_SCAN = 8;                           // indices that a lane looks at
constexpr int TM_MAX = TM_THREADS * TM_SCAN, TM_MAX_FEW = 5120;      // kernels; of fewer than eight members

__global__ __launch_bounds__(TM_THREADS)
void project_backward_members_kernel(const float *__restrict__ w, const float *__restrict__ g_wbar, const uint16_t *__restrict__ idx, int n, int K,
                                     float *__restrict__ g_w, float *__restrict__ g_p, int vec)
{
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= K) {
        const int e = (((int)blockIdx.x - K) * TM_THREADS + tid) * 4, ne = n * 9;
        auto through = [](float wv, float gv) { return wv > -1.0f && wv < 1.0f ? gv : 0.0f; };
        if (vec && e + 4 <= ne) {
            const float4 a = *(const float4 *)(w + e), b = *(const float4 *)(g_wbar + e);
            *(float4 *)(g_w + e) = make_float4(through(a.x, b.x), through(a.y, b.y), through(a.z, b.z), through(a.w, b.w));
        } else {
            for (int j = 0; j < 4; ++j)
                if (e + j < ne) g_w[e + j] = through(w[e + j], g_wbar[e + j]);
        }
        return;
    }
    __shared__ uint16_t list[TM_WAVES][TM_SCAN * 64];
    __shared__ float sums[TM_WAVES][64];
    const int k = blockIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int entry = lane / 9, tap = lane - 9 * entry;        // (lane 63: no entry)
    uint16_t *const mine = list[wave];
    // (the indices go to the waves in turn, 64 at a time)
    const int rounds = min(TM_SCAN, (n - wave * 64 + TM_THREADS - 1) / TM_THREADS);
    int member[TM_SCAN];
#pragma unroll
    for (int i = 0; i < TM_SCAN; ++i) {
        if (i >= rounds) break;                                // (wave-uniform)
        const int c = i * TM_THREADS + tid;
        member[i] = c < n ? min((int)idx[c], K - 1) : -1;
    }
    int found = 0;                                             // (wave-uniform)
#pragma unroll
    for (int i = 0; i < TM_SCAN; ++i) {
        if (i >= rounds) break;
        const bool hit = member[i] == k;
        const unsigned long long hits = __ballot(hit);
        if (hit) mine[found + (int)__popcll(hits & ((1ull << lane) - 1ull))] = (uint16_t)(i * TM_THREADS + tid);
        found += (int)__popcll(hits);
    }
    // The wave's own piece: LDS gives a wave back in order what it has written.  The compiler knows that of a lane's own words alone.
    __builtin_amdgcn_wave_barrier();
    float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};                   // four chains: a quarter of the roundings in a row
    if (entry < 7) {
        int e = entry;
        for (; e + 49 < found; e += 56) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = g_wbar[(int)mine[e + 7 * u] * 9 + tap];
#pragma unroll
            for (int u = 0; u < 4; ++u) sum[u] += v[u] + v[u + 4];
        }
        float v[7];
#pragma unroll
        for (int u = 0; u < 7; ++u) v[u] = e + 7 * u < found ? g_wbar[(int)mine[e + 7 * u] * 9 + tap] : 0.0f;
#pragma unroll
        for (int u = 0; u < 3; ++u) sum[u] += v[u] + v[u + 4];
        sum[3] += v[3];
    }
    sums[wave][lane] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    __syncthreads();
    // sixteen waves x seven entries of a tap: a thread adds the seven of a wave, sixteen lanes side by side their sums
    if (tid < 9 * TM_WAVES) {
        const int t = tid >> 4, wv = tid & 15;
        float v[7];
#pragma unroll
        for (int e = 0; e < 7; ++e) v[e] = sums[wv][9 * e + t];
        float s = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + v[6]);
#pragma unroll
        for (int d = 8; d >= 1; d >>= 1) s += __shfl_xor(s, d, 16);
        if (wv == 0) g_p[k * 9 + t] = s;
    }
}

// Pass 2: g_p[k][t] = sum of the block partials; one wave per entry: lane l adds the partials of
// blocks l, l + 64, ... in order, then the 64 lane sums are added in a fixed butterfly.
__global__ __launch_bounds__(TB_THREADS)
void reduce_partials_kernel(const float *__restrict__ partial, int64_t blocks, int K9, float *__restrict__ g_p)
{
    const int i = blockIdx.x * (TB_THREADS / 64) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= K9) return;                             // wave-uniform
    float s = 0.0f;
    for (int64_t b = lane; b < blocks; b += 64) s += partial[b * K9 + i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
    if (lane == 0) g_p[i] = s;
}

// One block: m' (Eq. 4), codes, repeated members.
__global__ __launch_bounds__(TB_THREADS)
void subset_update_kernel(const float *__restrict__ p, int8_t *__restrict__ m, float theta, int K,
                          uint16_t *__restrict__ codebook, uint8_t *__restrict__ dup)
{
    __shared__ uint16_t codes[512];
    const int tid = threadIdx.x;
    for (int k = tid; k < K; k += TB_THREADS) {
        uint32_t code = 0;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const float pv = p[k * 9 + t];
            int8_t mv = m[k * 9 + t];
            if (fabsf(pv) > theta) mv = pv > 0.0f ? 1 : -1;      // |p| > theta >= 0: p is not zero
            m[k * 9 + t] = mv;
            code |= (mv > 0 ? 1u : 0u) << (8 - t);
        }
        codes[k] = (uint16_t)code;
        codebook[k] = (uint16_t)code;
    }
    __syncthreads();
    for (int k = tid; k < K; k += TB_THREADS) {
        uint8_t d = 0;
        for (int j = 0; j < k; ++j) d |= codes[j] == codes[k] ? 1 : 0;
        dup[k] = d;
    }
}

}  // namespace

// Room for any number of kernels up to n: the block size jumps, and a workspace of a network's largest layer serves the others.
size_t project_backward_workspace_bytes(int64_t n, int K)
{
    int64_t blocks = tb_blocks(n);
    for (const int64_t end : {TB_ONE_MAX, TB_TWO_MAX})
        if (n > end) blocks = std::max(blocks, tb_blocks(end));
    return align_up((size_t)(blocks > 0 ? blocks : 1) * K * 9 * sizeof(float), 256);
}

int launch_project_backward(const float *w, const float *g_wbar, const uint16_t *idx, int64_t n, int K, float *g_w,
                            float *g_p, void *ws, hipStream_t s)
{
    // The product costs time with K, the atomics do not: up to 64 members it is the faster at any size, up to 128 as long as blocks are
    // small.  The small blocks' partial sums cost more than they save from some 5 M sums on.  Measured, product -> atomics on large
    // blocks, us: 262144 kernels K = 64 19.1 -> 20.1, K = 128 29.4 -> 22.9, K = 256 52.8 -> 28.9; 20000 kernels K = 128
    // 9.3 -> 10.3.  Atomics on small -> large blocks: 5000 kernels K = 512 9.1 -> 11.1, 20000 14.9 -> 12.8.  One copy of the sums
    // instead of four is 4 % faster on large blocks, and its error on skewed indices 1.4 times as large (1.7e-7 for 1.2e-7).
    const bool product = K <= 64 || (K <= 128 && n <= TB_ONE_MAX);
    const bool large = !product && (n > TB_ONE_MAX || n * K > ((int64_t)5 << 20));
    // Blocks of the one launch read what others may have written by then if g_w lies over g_wbar (in place) or g_p over an input: the two
    // launches write g_p when all inputs have been read, and g_w where the same block has read g_wbar.
    auto apart = [](const void *a, size_t a_bytes, const void *b, size_t b_bytes) {
        return (uintptr_t)a + a_bytes <= (uintptr_t)b || (uintptr_t)b + b_bytes <= (uintptr_t)a;
    };
    const size_t bytes = (size_t)n * 36, p_bytes = (size_t)K * 36;
    const bool in_order = apart(g_w, bytes, g_wbar, bytes) && apart(g_w, bytes, idx, (size_t)n * 2) && apart(g_p, p_bytes, w, bytes) &&
                          apart(g_p, p_bytes, g_wbar, bytes) && apart(g_p, p_bytes, idx, (size_t)n * 2);
    if (n > 0 && n <= (K < 8 ? TM_MAX_FEW : TM_MAX) && in_order) {
        const bool vec = ((((uintptr_t)w) | ((uintptr_t)g_wbar) | ((uintptr_t)g_w)) & 15u) == 0;
        const unsigned grid = (unsigned)(K + (n * 9 + 4 * TM_THREADS - 1) / (4 * TM_THREADS));
        hipLaunchKernelGGL(project_backward_members_kernel, dim3(grid), dim3(TM_THREADS), 0, s, w, g_wbar, idx, (int)n, K, g_w, g_p, vec ? 1 : 0);
        return check_launch();
    }
    const int64_t blocks = large ? (n + TB_LARGE - 1) / TB_LARGE : tb_blocks(n);
    if (blocks > 0x7fffffffLL) return SNN_ERR_INVALID_ARG;
    if (large) {
        hipLaunchKernelGGL(project_backward_large_kernel, dim3((unsigned)blocks), dim3(TB_THREADS), tb_copies_bytes(K), s, w,
                           g_wbar, idx, n, K, g_w, (float *)ws);
    } else if (blocks > 0) {
        const bool vec = ((((uintptr_t)w) | ((uintptr_t)g_wbar) | ((uintptr_t)g_w)) & 15u) == 0;
        const int U = tb_units(n), M = !product ? 0 : K <= 16 ? 1 : K <= 32 ? 2 : K <= 64 ? 4 : 8;
        const size_t lds = sizeof(float) * (M > 0 ? TB_UNIT * U * 9 + 16 : 0) + tb_copies_bytes(K);
        auto kern = M == 0 ? project_backward_kernel<1, 0> : project_backward_kernel<1, 8>;      // (n <= TB_ONE_MAX: U = 1)
#define SNN_TB_CASE(M_)                                                                                                      \
    if (M == M_) kern = U == 1 ? project_backward_kernel<1, M_> : U == 2 ? project_backward_kernel<2, M_> : project_backward_kernel<4, M_>;
        SNN_TB_CASE(1)
        SNN_TB_CASE(2)
        SNN_TB_CASE(4)
#undef SNN_TB_CASE
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(TB_THREADS), lds, s, w, g_wbar, idx, n, K, g_w, (float *)ws, vec ? 1 : 0);
    }
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((unsigned)((K * 9 + TB_THREADS / 64 - 1) / (TB_THREADS / 64))), dim3(TB_THREADS), 0, s,
                       (const float *)ws, blocks, K * 9, g_p);
    return check_launch();
}

int launch_subset_update(const float *p, int8_t *m, float theta, int K, uint16_t *codebook, uint8_t *dup, hipStream_t s)
{
    hipLaunchKernelGGL(subset_update_kernel, dim3(1), dim3(TB_THREADS), 0, s, p, m, theta, K, codebook, dup);
    return check_launch();
}

}  // namespace snn

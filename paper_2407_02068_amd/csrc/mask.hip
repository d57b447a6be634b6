// mask.hip -- the block mask of a weight on the GPU: block scores, then the
// top-k blocks (gfx950).
//
// Paper, Sec. 3.1: the blocks of a weight are ranked by the 2-D average pool
// of the first-order Taylor score |W * grad_W f| of their elements, and the
// bottom-ranked ones are dropped; Sec. 3.4: ceil((1 - alpha) R C) blocks
// survive.  Without a gradient the score is the block's sum of squares (it
// ranks like the block's L2 norm).
//
// A score is an integer-deciding quantity (it picks the kept set), so it is
// computed exactly as specified: in float64, the block's elements row by row,
// one addition after the other, with no contraction into fused multiply-adds.
// Every product of two decoded elements is exact in float64 and the average's
// divisor is a power of two, so the value depends only on that order.
//
// Scores are non-negative (+0.0 at least), so their IEEE bit patterns order
// like their values; the selection works on those 64-bit keys.
#include "lpv_device.h"
#include "lpv_internal.h"
#include "lpv_scores.h"

namespace lpv {
namespace {

template <int DT> __device__ inline double load_f64(const char* base, int64_t idx)
{
    if (DT == LPV_F32)
        return (double)((const float*)base)[idx];
    const uint16_t bits = ((const uint16_t*)base)[idx];
    if (DT == LPV_BF16)
        return (double)__uint_as_float((uint32_t)bits << 16);
    return (double)(float)__builtin_bit_cast(_Float16, bits);
}

// One thread per block (r, c) = blockIdx.x * 256 + threadIdx.x (row-major), element by
// element: for weights and gradients that 16-byte loads cannot read (base or row stride
// not a multiple of 16 bytes).
template <int DT, bool TAYLOR>
__global__ __launch_bounds__(256) void k_block_scores(const char* __restrict__ W, int64_t ldw,
                                                      const char* __restrict__ G, int64_t ldg,
                                                      int64_t R, int64_t C, int32_t b_r,
                                                      int32_t b_c, double* __restrict__ scores)
{
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= R * C)
        return;
    const int64_t r = i / C, c = i - r * C;
    double s = 0.0;
    for (int32_t a = 0; a < b_r; ++a) {
        const int64_t n = r * b_r + a;
        for (int32_t b = 0; b < b_c; ++b) {
            const int64_t k = c * b_c + b;
            const double w = load_f64<DT>(W, n * ldw + k);
            if (TAYLOR) {
                const double p = w * load_f64<DT>(G, n * ldg + k);
                s = s + (p < 0.0 ? -p : p);
            } else {
                s = s + w * w;
            }
        }
    }
    scores[i] = TAYLOR ? s / (double)(b_r * b_c) : s;
}

// The same scores through LDS (wg_block_scores): as many blocks of one block row per
// workgroup as fit SC_LDS bytes of float64 terms.
constexpr int SC_THREADS = 256;
constexpr int SC_LDS = 131072;  // bytes of float64 terms per workgroup

template <int DT, bool TAYLOR>
__global__ __launch_bounds__(SC_THREADS) void k_block_scores_lds(const char* __restrict__ W,
                                                                 int64_t ldw,
                                                                 const char* __restrict__ G,
                                                                 int64_t ldg, int64_t C,
                                                                 int32_t b_r, int32_t b_c,
                                                                 int32_t nb,
                                                                 double* __restrict__ scores)
{
    // at most SC_LDS bytes of terms and 16 bytes of padding per block
    // (blocks of at least 256 elements: at most SC_LDS / 2048 blocks)
    __shared__ double2 terms[(SC_LDS + 16 * (SC_LDS / 2048)) / 16];
    wg_block_scores<DT, TAYLOR, SC_THREADS>(W, ldw, G, ldg, C, b_r, b_c, nb, blockIdx.x, terms, scores);
}

// rank[b] = #{b' : score(b') > score(b), or equal and b' < b}: perm[rank[b]] = b
// (perm, if given) and mask[b] = rank[b] < n_keep (mask, if given).  Scores are
// non-negative, so their bit patterns order like their values.  Workgroup: RANK_B
// blocks; thread t takes for block t % RANK_B the keys t / RANK_B, t / RANK_B +
// RANK_PARTS, ... and counts those at or above it up to the block's own place, those
// above it from there on: one compare a key, ties or not.  The keys come through LDS
// (RANK_CHUNK at a time); integer counts, exact in any order.  Bound: the 64-bit
// compares, so few blocks per workgroup and the whole chip (64 blocks per workgroup
// kept 36 CUs busy with 2304 blocks: 12.6 us; this 5.4).  The delta curve of 131072 blocks,
// nearly all of it ranking, 2.89 ms, of 65536 0.78; counting equal keys in a pass of their
// own took 3.31 and 0.88 without ties, 6.53 and 1.72 with them.
constexpr int RANK_B = 8;
constexpr int RANK_NT = 1024;
constexpr int RANK_PARTS = RANK_NT / RANK_B;
constexpr int RANK_CHUNK = 4096;  // 32 KB of keys
// Most blocks for which the selection ranks every block (quadratic work).
constexpr int64_t RANK_MAX = 8192;

__global__ __launch_bounds__(RANK_NT) void k_rank(const double* __restrict__ scores, int64_t nb,
                                                  int64_t n_keep, int32_t* __restrict__ perm,
                                                  uint8_t* __restrict__ mask)
{
    __shared__ uint64_t s_keys[RANK_CHUNK];
    __shared__ int32_t s_cnt[RANK_NT / 64][RANK_B];
    const int tid = threadIdx.x, part = tid / RANK_B;
    const int64_t b = (int64_t)blockIdx.x * RANK_B + tid % RANK_B;
    const uint64_t* keys = (const uint64_t*)scores;
    const uint64_t key = keys[min(b, nb - 1)];
    int32_t ahead = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += RANK_CHUNK) {
        const int n = (int)min((int64_t)RANK_CHUNK, nb - c0);
        __syncthreads();  // the chunk before is counted
        for (int i = tid; i < n; i += RANK_NT)
            s_keys[i] = keys[c0 + i];
        __syncthreads();
        const int own = (int)min(max(b - c0, (int64_t)0), (int64_t)n);  // the block's place in the chunk
        int i = part;
#pragma unroll 4
        for (; i < own; i += RANK_PARTS)
            ahead += s_keys[i] >= key;
#pragma unroll 4
        for (; i < n; i += RANK_PARTS)
            ahead += s_keys[i] > key;
    }
    // the threads' counts of a block, added over the workgroup
#pragma unroll
    for (int o = RANK_B; o < 64; o <<= 1)
        ahead += __shfl_xor(ahead, o, 64);
    if ((tid & 63) < RANK_B)
        s_cnt[tid >> 6][tid & 63] = ahead;
    __syncthreads();
    if (tid < RANK_B && b < nb) {
        int32_t rank = 0;
#pragma unroll
        for (int j = 0; j < RANK_NT / 64; ++j)
            rank += s_cnt[j][tid];
        if (perm)
            perm[rank] = (int32_t)b;
        if (mask)
            mask[b] = rank < n_keep;
    }
}

constexpr int SEL_THREADS = 1024;

__device__ inline uint64_t key_of(double v) { return (uint64_t)__double_as_longlong(v); }

// One workgroup: mask[i] = 1 for the n_keep best-ranked scores (larger first,
// equal scores by lower index).  T, the n_keep-th largest key, is found one
// byte at a time from the top (a radix select): among the keys that match the
// bytes found so far, an LDS histogram of the next byte gives the byte of T
// and how many keys above it drop out.  Then every key > T is kept, and of the
// keys == T the (n_keep - #keys > T) lowest indices (wave ballots give each
// tie its rank in index order).  The keys (more than RANK_MAX) are read from global
// memory in every pass.
__global__ __launch_bounds__(SEL_THREADS) void k_mask_topk(const double* __restrict__ scores,
                                                           int64_t n, int64_t n_keep,
                                                           uint8_t* __restrict__ mask)
{
    __shared__ int64_t s_part[SEL_THREADS / 64];
    __shared__ uint32_t s_hist[256];
    __shared__ uint32_t s_sel[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (n_keep <= 0) {
        for (int64_t i = tid; i < n; i += SEL_THREADS)
            mask[i] = 0;
        return;
    }
    uint64_t prefix = 0, pmask = 0;
    int64_t remaining = n_keep;  // rank of T among the keys matching the prefix
    for (int byte = 7; byte >= 0; --byte) {
        const int sh = 8 * byte;
        for (int i = tid; i < 256; i += SEL_THREADS)
            s_hist[i] = 0;
        __syncthreads();
        for (int64_t i = tid; i < n; i += SEL_THREADS) {
            const uint64_t k = key_of(scores[i]);
            if ((k & pmask) == prefix)
                atomicAdd(&s_hist[(k >> sh) & 255], 1u);
        }
        __syncthreads();
        if (wave == 0) {
            // the byte value v with (# above v) < remaining <= (# at or above
            // v): lane L holds bins 4L .. 4L + 3 and the suffix sum S_L of the
            // bins from 4L up; the lane with S_{L+1} < remaining <= S_L scans
            // its four
            const uint32_t h0 = s_hist[4 * lane], h1 = s_hist[4 * lane + 1],
                           h2 = s_hist[4 * lane + 2], h3 = s_hist[4 * lane + 3];
            uint32_t suf = h0 + h1 + h2 + h3;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = __shfl_down(suf, o, 64);
                if (lane + o < 64)
                    suf += t;
            }
            uint32_t up = __shfl_down(suf, 1, 64);  // S_{L+1}
            if (lane == 63)
                up = 0;
            if (up < (uint64_t)remaining && suf >= (uint64_t)remaining) {
                uint32_t above = up;
                int v = 4 * lane + 3;
                const uint32_t hv[4] = {h0, h1, h2, h3};
                for (int b = 3; b > 0; --b, --v) {
                    if (above + hv[b] >= (uint64_t)remaining)
                        break;
                    above += hv[b];
                }
                s_sel[0] = (uint32_t)v;
                s_sel[1] = above;
            }
        }
        __syncthreads();
        prefix |= (uint64_t)s_sel[0] << sh;
        pmask |= (uint64_t)255 << sh;
        remaining -= s_sel[1];
        __syncthreads();  // s_hist and s_sel are rewritten by the next pass
    }
    const uint64_t T = prefix;
    const int64_t need = remaining;  // >= 1 keys equal to T
    // ties in index order: per chunk of SEL_THREADS indices, each tie's rank
    // from a ballot within its wave and the wave totals before it
    int64_t taken = 0;
    for (int64_t base = 0; base < n; base += SEL_THREADS) {
        const int64_t i = base + tid;
        const uint64_t k = i < n ? key_of(scores[i]) : 0;
        const bool tie = i < n && k == T;
        const uint64_t bal = __ballot(tie);
        const int64_t before_in_wave = __popcll(bal & (((uint64_t)1 << lane) - 1));
        if (lane == 0)
            s_part[wave] = __popcll(bal);
        __syncthreads();
        int64_t before = taken + before_in_wave, total = 0;
        for (int w = 0; w < SEL_THREADS / 64; ++w) {
            if (w < wave)
                before += s_part[w];
            total += s_part[w];
        }
        if (i < n)
            mask[i] = k > T || (tie && before < need);
        taken += total;
        __syncthreads();  // s_part is rewritten by the next chunk
    }
}

hipError_t launch_block_scores(const MaskCall& m, hipStream_t s)
{
    const int64_t R = m.N / m.b_r, C = m.K / m.b_c, nb = R * C;
    const int es = m.dtype == LPV_F32 ? 4 : 2;
    const bool vec = ((uintptr_t)m.W % 16) == 0 && (m.ldw * es) % 16 == 0 &&
                     (!m.G || (((uintptr_t)m.G % 16) == 0 && (m.ldg * es) % 16 == 0));
    if (nb > 0 && vec) {
        // blocks per workgroup: as many as fit SC_LDS bytes of float64 terms
        // (at least one), at most one per thread
        const int bytes = m.b_r * m.b_c * 8;
        const int nbw = (int)min(min((int64_t)max(1, SC_LDS / bytes), (int64_t)SC_THREADS), C);
        const int64_t n_wg = R * ((C + nbw - 1) / nbw);
        const dim3 grid((unsigned)n_wg), block(SC_THREADS);
#define LPV_SCORES2(DT_, TY_)                                                                       \
    hipLaunchKernelGGL((k_block_scores_lds<DT_, TY_>), grid, block, 0, s, (const char*)m.W, m.ldw, \
                       (const char*)m.G, m.ldg, C, m.b_r, m.b_c, nbw, m.scores)
        if (m.dtype == LPV_BF16) {
            if (m.G)
                LPV_SCORES2(LPV_BF16, true);
            else
                LPV_SCORES2(LPV_BF16, false);
        } else if (m.dtype == LPV_F16) {
            if (m.G)
                LPV_SCORES2(LPV_F16, true);
            else
                LPV_SCORES2(LPV_F16, false);
        } else {
            if (m.G)
                LPV_SCORES2(LPV_F32, true);
            else
                LPV_SCORES2(LPV_F32, false);
        }
#undef LPV_SCORES2
        return hipGetLastError();
    }
    if (nb > 0) {
        const dim3 grid((unsigned)((nb + 255) / 256)), block(256);
#define LPV_SCORES(DT_, TY_)                                                                       \
    hipLaunchKernelGGL((k_block_scores<DT_, TY_>), grid, block, 0, s, (const char*)m.W, m.ldw,     \
                       (const char*)m.G, m.ldg, R, C, m.b_r, m.b_c, m.scores)
#define LPV_SCORES_DT(DT_)             \
    do {                               \
        if (m.G)                       \
            LPV_SCORES(DT_, true);     \
        else                           \
            LPV_SCORES(DT_, false);    \
    } while (0)
        if (m.dtype == LPV_BF16)
            LPV_SCORES_DT(LPV_BF16);
        else if (m.dtype == LPV_F16)
            LPV_SCORES_DT(LPV_F16);
        else
            LPV_SCORES_DT(LPV_F32);
#undef LPV_SCORES_DT
#undef LPV_SCORES
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_rank(const double* scores, int64_t nb, int64_t n_keep, int32_t* perm,
                       uint8_t* mask, hipStream_t s)
{
    hipLaunchKernelGGL(k_rank, dim3((unsigned)((nb + RANK_B - 1) / RANK_B)), dim3(RANK_NT), 0, s, scores,
                       nb, n_keep, perm, mask);
    return hipGetLastError();
}

hipError_t launch_mask_topk(const MaskCall& m, hipStream_t s)
{
    const int64_t nb = (m.N / m.b_r) * (m.K / m.b_c);
    const hipError_t e = launch_block_scores(m, s);
    if (e != hipSuccess)
        return e;
    // counting ahead of every block over the whole chip against eight dependent
    // passes of one workgroup: 2304 blocks 5.4 us, 16.1; 8192 equal
    if (nb <= RANK_MAX)
        return launch_rank(m.scores, nb, m.n_keep, nullptr, m.mask, s);
    hipLaunchKernelGGL(k_mask_topk, dim3(1), dim3(SEL_THREADS), 0, s, (const double*)m.scores, nb,
                       m.n_keep, m.mask);
    return hipGetLastError();
}

}  // namespace lpv

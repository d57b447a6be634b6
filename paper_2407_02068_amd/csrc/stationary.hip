// stationary.hip -- the block-sparse product with X held in registers (bf16 /
// fp16, at most 768 reduction columns).
//
// A wave keeps 32 tokens of X, all columns, in registers (KT column tiles x 8
// registers) and its workgroup of 8 waves walks tile rows of W~ past them: one
// run of kept tiles in row-major order (row_vals), staged through an LDS ring in
// chunks that every wave reads.  Against k_linear16, which brings X and W of every
// column pair through LDS, a step costs one tile of LDS traffic and DMA instead of
// the pair's whole X slice, the walk needs no step table (a row's kept columns are
// a bit mask, its tiles follow each other), and a barrier comes once per 16
// tiles.  Persistent: the (token tile, tile row) sequence is cut into one
// contiguous share per workgroup, equal in cost, so at most a few X loads per
// workgroup and no last round.
//
// Bound: with few kept tiles the stores of Y and the read of X (50432 tokens, 768
// -> 3072 at 90% block sparsity: 88 us for 387 MB; k_linear16 102); else the round
// trips of the LDS reads of W, which are waited for right after the two products they
// run beside, and the row epilogues, at two waves per SIMD (50%: 157 us, k_linear16 172;
// 70%: 126 / 150).  No unit is near its rate there: matrix cores 31% busy, LDS 28%, waves
// 32% issuing and 43% waiting (24% at s_waitcnt).  12608 tokens, 384 -> 1536, 50%, GELU:
// 26.5 us (32.4).  The stores were the bound throughout (121 us at any sparsity above
// 70%) while each tile row wrote its own 64-byte halves of Y's 128-byte lines.
// Two waves of 64 tokens per SIMD do not fit the registers, one does and ran no
// faster (158 us): every LDS wait and every epilogue is then exposed.
#include "lpv_device.h"
#include "lpv_internal.h"
#include "lpv_lds.h"

namespace lpv {
namespace {

constexpr int XS_NT = 512;
constexpr int XS_NW = XS_NT / 64;
constexpr int XS_BM = XS_NW * 32;    // tokens per workgroup: 32 per wave
constexpr int XS_CH = 16;            // tiles per chunk of the W ring
constexpr int XS_SLOTS = 4;          // chunks in the ring
constexpr int XS_AGPR = 16;          // column tiles whose X sits in AGPRs

struct XsDims {
    int64_t ldx, M, N, ldy;
    int32_t n_rows, n_cols, n_mt;
    int32_t row_cost;  // cost of a row beside its tiles, in tiles
};

// acc += w x (32x32x16), in place.  Inline assembly with X in an AGPR or a VGPR,
// so that the accumulators never move: past every kept-column branch the
// compiler's own form copied them.  Wait states between other instructions and
// these are the caller's (the compiler does not see the hazards).
template <int DT, bool AG> __device__ inline void mm(f32x16& acc, v4i w, v4i x)
{
    if constexpr (DT == LPV_BF16) {
        if constexpr (AG)
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "a"(x));
        else
            asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(x));
    } else {
        if constexpr (AG)
            asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "a"(x));
        else
            asm volatile("v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(x));
    }
}

__device__ inline void lds_write8(uint32_t addr, uint64_t v)
{
    *(__attribute__((address_space(3))) uint64_t*)(uintptr_t)addr = v;
}

template <int DT, bool GELU, int KT>
__global__ __launch_bounds__(XS_NT, 2) void k_linear16_xs(
    const XsDims d, const char* __restrict__ X, const char* __restrict__ row_vals,
    const int32_t* __restrict__ row_tile0, const uint32_t* __restrict__ row_mask,
    const char* __restrict__ bias, char* __restrict__ Y)
{
    using E = Elem<DT>;
    constexpr int RING = XS_SLOTS * XS_CH * 2048;
    constexpr int WCH = XS_CH / XS_NW;         // tiles of a chunk that a wave loads
    constexpr int PB = RING / XS_NW / 4096;    // column pairs of X staged at a time
    __shared__ uint4 s_ring[RING / 16];
    __shared__ uint4 s_out[XS_NW * 128];       // 2 KB per wave
    __shared__ float s_bias[XS_ROWS * TILE];
    static_assert(RING + XS_NW * 2048 + XS_ROWS * TILE * 4 <= 163840, "LDS budget of one workgroup");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    for (int i = tid; i < d.n_rows * TILE; i += XS_NT)
        s_bias[i] = (bias && i < d.N) ? E::to_f32(((const uint16_t*)bias)[i]) : 0.0f;

    // This workgroup's share of the (token tile, tile row) sequence, cut by cost:
    // row r of a token tile starts at cost row_tile0[r] + r row_cost.  Consecutive
    // shares, which may split a token tile, run on one XCD.
    const int P = (int)gridDim.x;
    const int w = (int)(blockIdx.x & 7) * (P >> 3) + (int)(blockIdx.x >> 3);
    const int64_t per_mt = row_tile0[d.n_rows] + (int64_t)d.n_rows * d.row_cost;
    const int64_t total = per_mt * d.n_mt;
    auto cut = [&](int64_t at, int& mt, int& row) {
        mt = (int)(at / per_mt);
        const int64_t rest = at - mt * per_mt;
        row = 0;  // the first row that starts at or after `at` (past the last: the next tile's)
        for (int r0 = 0; r0 < d.n_rows; r0 += 64) {
            const int r = r0 + lane;
            const int64_t start = row_tile0[min(r, d.n_rows - 1)] + (int64_t)r * d.row_cost;
            row += __popcll(__ballot(r < d.n_rows && start < rest));
        }
        if (row == d.n_rows) {
            row = 0;
            ++mt;
        }
    };
    int mt, row, mt_end, row_end;
    cut(total * w / P, mt, row);
    cut(total * (w + 1) / P, mt_end, row_end);
    __syncthreads();

    const uint32_t ring = lds_addr(s_ring);
    const uint32_t outb = lds_addr(s_out) + (uint32_t)wave * 2048;
    const uint32_t loff = (uint32_t)lane * 16;

    while (mt < mt_end || (mt == mt_end && row < row_end)) {
        const int r_end = mt < mt_end ? d.n_rows : row_end;
        // ---- X of this wave's tokens into registers, through the wave's part of the
        // ring: column pairs of 32 rows x 128 bytes (piece ch of row r at ch ^ xswz(r))
        v4i xf[KT][2];
        const int64_t m0 = (int64_t)mt * XS_BM + wave * 32;
        {
            // (lane made opaque: what only this part needs is not kept in registers
            // through the row loop; the same below)
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int fr = ln & 31, fh = ln >> 5;
            const char* xb0 = X + min(m0, d.M - 1) * d.ldx * 2;
            const int64_t last = max(d.M - 1 - m0, (int64_t)0);  // rows past M repeat the last
            uint32_t xoff[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 8 * i + (ln >> 3);
                xoff[i] = (uint32_t)((min((int64_t)r, last) * d.ldx + 8 * ((ln & 7) ^ xswz(r))) * 2);
            }
            const uint32_t base = ring + (uint32_t)wave * (RING / XS_NW);
            const int n_pairs = d.n_cols / 2;
#pragma unroll
            for (int p0 = 0; p0 < KT / 2; p0 += PB) {
#pragma unroll
                for (int p = p0; p < p0 + PB && p < KT / 2; ++p)
                    if (p < n_pairs) {
                        const char* xb = xb0 + p * 128;
                        const uint32_t at = base + (uint32_t)(p - p0) * 4096;
                        dma16i<0>(xb, xoff[0], at);
                        dma16i<1024>(xb - 1024, xoff[1], at);
                        dma16i<2048>(xb - 2048, xoff[2], at);
                        dma16i<3072>(xb - 3072, xoff[3], at);
                    }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                // (pairs past the weight's columns read stale data that no kept bit uses)
#pragma unroll
                for (int p = p0; p < p0 + PB && p < KT / 2; ++p)
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
                        xf[2 * p + (ks >> 1)][ks & 1] =
                            lds_read16<0>(base + (uint32_t)(p - p0) * 4096 + fr * 128 +
                                          ((2 * ks + fh) ^ xswz(fr)) * 16);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
        }
        __syncthreads();

        // ---- the W tiles of rows [row, r_end), positions 0 .. n - 1 of the row-major
        // run, in chunks through the ring; wave w loads WCH tiles of every chunk
        // (positions past the end repeat the last tile, so that every chunk has the
        // same number of instructions)
        const int t0 = __builtin_amdgcn_readfirstlane(row_tile0[row]);
        const int n = __builtin_amdgcn_readfirstlane(row_tile0[r_end]) - t0;
        const char* wsrc = row_vals + (int64_t)t0 * 2048;
        int dpos = wave * WCH, dslot = 0;
        auto dma_chunk = [&]() __attribute__((always_inline)) {
            const uint32_t at = ring + (uint32_t)(dslot * XS_CH + wave * WCH) * 2048;
#pragma unroll
            for (int i = 0; i < WCH; ++i) {
                const uint32_t off = loff + (uint32_t)min(dpos + i, n - 1) * 2048u;
                dma16i<0>(wsrc, off, at + i * 2048);
                dma16i<1024>(wsrc, off, at + i * 2048);
            }
            dpos += XS_CH;
            dslot = dslot + 1 == XS_SLOTS ? 0 : dslot + 1;
        };
        // the W fragments of the next tile
        v4i w0[2] = {};
        int left = 0;     // tiles left in the chunk being read
        uint32_t rd = 0;  // next tile to read, from the ring's start
        auto read = [&](v4i(&o)[2]) __attribute__((always_inline)) {
            if (__builtin_expect(left == 0, 0)) {
                // a new chunk: it has landed for every wave (at least the DMA of
                // SLOTS - 2 later chunks has been issued after its own), and every
                // wave has read the chunk before it, whose place the next DMA takes
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n s_barrier" ::"i"((XS_SLOTS - 2) * WCH * 2) : "memory");
                dma_chunk();
                left = XS_CH;
                if (rd == RING)
                    rd = 0;
            }
            const uint32_t at = ring + loff + rd;
            o[0] = lds_read16<0>(at);
            o[1] = lds_read16<1024>(at);
            rd = __builtin_amdgcn_readfirstlane(rd + 2048);
            left = __builtin_amdgcn_readfirstlane(left - 1);
        };
        if (n > 0) {
#pragma unroll
            for (int i = 0; i < XS_SLOTS - 1; ++i)
                dma_chunk();
            read(w0);
        }
        uint64_t even[4] = {};  // the rounded outputs of an even row
        uint32_t masks = 0;     // lane l: the row mask of row `row` + l (64 at a time)
        for (int r = row; r < r_end; ++r) {
            if (((r - row) & 63) == 0)
                masks = row_mask[min(r + lane, d.n_rows - 1)];
            uint32_t mask = __builtin_amdgcn_readlane(masks, (r - row) & 63);
            asm volatile("" : "+s"(mask));
            f32x16 acc;  // starts at the bias
            {
                int ln = lane;
                asm volatile("" : "+v"(ln));
                const uint32_t ba = lds_addr(s_bias) + (uint32_t)(r * TILE + 4 * (ln >> 5)) * 4;
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    const v4i v = lds_read16<0>(ba + qq * 32);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[4 * qq + i] = __builtin_bit_cast(float, (int)v[i]);
                }
                asm volatile("s_nop 4" : "+v"(acc));
            }
#pragma unroll
            for (int c = 0; c < KT; ++c) {
                if ((mask >> c) & 1) {
                    v4i w1[2];
                    read(w1);
                    __builtin_amdgcn_sched_barrier(0);
                    // (two wait states between the copy of w0 and its first use)
                    asm volatile("s_nop 1");
                    if (c < XS_AGPR) {
                        mm<DT, true>(acc, w0[0], xf[c][0]);
                        mm<DT, true>(acc, w0[1], xf[c][1]);
                    } else {
                        mm<DT, false>(acc, w0[0], xf[c][0]);
                        mm<DT, false>(acc, w0[1], xf[c][1]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    w0[0] = w1[0];
                    w0[1] = w1[1];
                }
            }
            // ---- epilogue: lane l holds outputs 8 qq + 4 (l / 32) + i of token l % 32.
            // An even row, rounded, waits for the odd one after it, so that whole
            // 128-byte lines of Y leave.  (24 wait states: the last product has been
            // written.)
            asm volatile("s_nop 15\n s_nop 7" : "+v"(acc));
            uint64_t pk[4];
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = acc[4 * qq + i];
                    if (GELU)
                        v[i] = gelu_erf(v[i]);
                }
                pk[qq] = pack2<DT>(v[0], v[1]) | (uint64_t)pack2<DT>(v[2], v[3]) << 32;
            }
            const bool odd = r & 1;
            if (!odd) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq)
                    even[qq] = pk[qq];
                if (r + 1 < r_end)
                    continue;
            }
            // 16 tokens at a time through this wave's 2 KB: 16-byte piece p of token t's
            // 128 bytes (0 .. 3 the even row's outputs) at p ^ (t % 8)
            const bool have_even = !odd || r > row;
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int fr = ln & 31, fh = ln >> 5;
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                if ((fr >> 4) == hf) {
                    const uint32_t at = outb + (fr & 15) * 128 + fh * 8;
#pragma unroll
                    for (int qq = 0; qq < 4; ++qq) {
                        lds_write8(at + ((qq ^ fr) & 7) * 16, even[qq]);
                        lds_write8(at + (((4 + qq) ^ fr) & 7) * 16, pk[qq]);
                    }
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int t = 8 * i + (ln >> 3), pc = ln & 7;
                    const v4i v = lds_read16<0>(outb + t * 128 + ((pc ^ t) & 7) * 16);
                    const int64_t m = m0 + 16 * hf + t, nn = (int64_t)(r & ~1) * TILE + 8 * pc;
                    if (m < d.M && nn < d.N && (pc < 4 ? have_even : odd))
                        __builtin_nontemporal_store(v, (v4i*)(Y + (m * d.ldy + nn) * 2));
                }
            }
        }
        // the ring is X's next
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        row = 0;
        ++mt;
    }
}

}  // namespace

bool use_xs(const lpv_bsr* h, int64_t M, bool gelu, int n_cus)
{
    if (!h->row_vals)
        return false;
    // Rows of 256 tokens per CU: each workgroup pays for its X load first (us at
    // 50%, this / k_linear16: 25 x 48 rows 15.4 / 13.9, 50 x 24 21.2 / 20.5, 50 x 48
    // 20.5 / 23.5, 25 x 96 31.6 / 38.0).
    if ((M + XS_BM - 1) / XS_BM * h->n_tile_rows < 8 * (int64_t)n_cus)
        return false;
    // Kept tiles: the W reads bound it, X's traffic is what it saves (50432 x 768 ->
    // 3072: all kept 246 / 238, 70% 196 / 198, 50% 158 / 172).  With 16-wide block
    // columns k_linear16 skips the dropped halves of a tile; this kernel does not.
    const int64_t tiles = (int64_t)h->n_tile_rows * h->n_tile_cols;
    // Steps: with few column tiles left to a group and whole groups k_linear16's items are
    // short and this kernel's epilogues are the bound (768 x 768, 64 x 64 blocks, 45507
    // tokens, 90%: 36.7 / 30.5; 1536 x 384, 19306: 21.2 / 17.5), unless the epilogue has the
    // GELU, which k_linear16 does not overlap either (1024 x 512, 16611: 24.0 / 32.1), or a group
    // is partial (1152 x 192, 31157, 50%: 24.4 / 40.8).
    if (!gelu && h->n_steps < 10 * (int64_t)h->n_groups && h->n_tile_rows % GROUP_TILES == 0)
        return false;
    return h->n_tiles * 100 <= tiles * (h->b_c == 16 ? 50 : 70);
}

hipError_t launch_xs_linear(const lpv_bsr* h, const LinearCall& c, int n_cus, hipStream_t s)
{
    XsDims d = {c.ldx, c.M, h->N, c.ldy, h->n_tile_rows, h->n_tile_cols};
    d.n_mt = (int32_t)((c.M + XS_BM - 1) / XS_BM);
    // a row's epilogue takes about as long as 9 tiles, its GELU as 5 more
    d.row_cost = c.gelu ? 14 : 9;
    const dim3 grid((unsigned)max(n_cus & ~7, 8)), block(XS_NT);
#define LPV_XS(DT_, GELU_, KT_)                                                                \
    hipLaunchKernelGGL((k_linear16_xs<DT_, GELU_, KT_>), grid, block, 0, s, d,                  \
                       (const char*)c.X, (const char*)h->row_vals, (const int32_t*)h->row_tile0, \
                       (const uint32_t*)h->row_mask, (const char*)c.bias, (char*)c.Y)
#define LPV_XS_KT(DT_, GELU_)           \
    do {                                \
        if (h->n_tile_cols <= 12)       \
            LPV_XS(DT_, GELU_, 12);     \
        else                            \
            LPV_XS(DT_, GELU_, 24);     \
    } while (0)
    if (h->dtype == LPV_BF16) {
        if (c.gelu)
            LPV_XS_KT(LPV_BF16, true);
        else
            LPV_XS_KT(LPV_BF16, false);
    } else {
        if (c.gelu)
            LPV_XS_KT(LPV_F16, true);
        else
            LPV_XS_KT(LPV_F16, false);
    }
#undef LPV_XS_KT
#undef LPV_XS
    return hipGetLastError();
}

}  // namespace lpv

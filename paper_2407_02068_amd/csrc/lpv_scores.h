// lpv_scores.h -- the block scores of a workgroup's blocks, shared by the mask
// generation and the delta curve (gfx950 only).
#pragma once

#include "lpv_device.h"
#include "lpv_internal.h"

namespace lpv {

// 8 consecutive elements (16-byte aligned) decoded to float64, from 16-byte loads.
template <int DT> __device__ inline void load8_f64(const char* base, int64_t idx, double* out)
{
    if (DT == LPV_F32) {
        const float4 a = *(const float4*)(base + idx * 4), b = *(const float4*)(base + idx * 4 + 16);
        out[0] = a.x, out[1] = a.y, out[2] = a.z, out[3] = a.w;
        out[4] = b.x, out[5] = b.y, out[6] = b.z, out[7] = b.w;
    } else {
        const uint4 u = *(const uint4*)(base + idx * 2);
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint16_t lo = (uint16_t)(w[j] & 0xffffu), hi = (uint16_t)(w[j] >> 16);
            if (DT == LPV_BF16) {
                out[2 * j] = (double)__uint_as_float((uint32_t)lo << 16);
                out[2 * j + 1] = (double)__uint_as_float((uint32_t)hi << 16);
            } else {
                out[2 * j] = (double)(float)__builtin_bit_cast(_Float16, lo);
                out[2 * j + 1] = (double)(float)__builtin_bit_cast(_Float16, hi);
            }
        }
    }
}

// The scores of a workgroup's run of blocks with the loads taken off the additions'
// path: the workgroup (number `wg` of those that cover the weight) takes nb
// consecutive blocks of one block row; its NT threads load them with 16-byte reads
// and write every element's term (|w g| or w w, exact in float64) to LDS; then
// thread j adds up block j's terms from LDS, one after the other in row-major order
// (the value of the plain loop bit for bit; the additions, 16 clocks each, are the
// bound).  A block's terms sit at a stride of its size plus 16 bytes, so the adding
// threads' 16-byte reads fall in distinct banks: `terms` holds nb (b_r b_c / 2 + 1)
// entries.
template <int DT, bool TAYLOR, int NT>
__device__ inline void wg_block_scores(const char* __restrict__ W, int64_t ldw,
                                       const char* __restrict__ G, int64_t ldg, int64_t C,
                                       int32_t b_r, int32_t b_c, int32_t nb, int64_t wg,
                                       double2* terms, double* __restrict__ scores)
{
#pragma clang fp contract(off)
    const int64_t n_chunks = (C + nb - 1) / nb;
    const int64_t r = wg / n_chunks, c0 = (wg - r * n_chunks) * nb;
    const int nbk = (int)min((int64_t)nb, C - c0);  // blocks of this workgroup
    const int n_el = b_r * b_c;
    const int stride = n_el / 2 + 1;                  // double2 units per block
    const int u_row = b_c / 8;                        // 8-element units per block row
    const int units = nbk * b_r * u_row;
    for (int i = threadIdx.x; i < units; i += NT) {
        const int q = i % u_row, t = i / u_row, j = t % nbk, a = t / nbk;
        const int64_t n = r * b_r + a, k = (c0 + j) * b_c + 8 * q;
        double w[8], g[8];
        load8_f64<DT>(W, n * ldw + k, w);
        if (TAYLOR)
            load8_f64<DT>(G, n * ldg + k, g);
        double2* dst = terms + j * stride + (a * b_c + 8 * q) / 2;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            double t0, t1;
            if (TAYLOR) {
                const double p0 = w[e] * g[e], p1 = w[e + 1] * g[e + 1];
                t0 = p0 < 0.0 ? -p0 : p0;
                t1 = p1 < 0.0 ? -p1 : p1;
            } else {
                t0 = w[e] * w[e];
                t1 = w[e + 1] * w[e + 1];
            }
            dst[e / 2] = double2{t0, t1};
        }
    }
    __syncthreads();
    const int j = threadIdx.x;
    if (j >= nbk)
        return;
    const double2* src = terms + j * stride;
    double s = 0.0;
    for (int e = 0; e < n_el / 2; e += 4) {  // n_el is a multiple of 8
        const double2 v0 = src[e], v1 = src[e + 1], v2 = src[e + 2], v3 = src[e + 3];
        s = s + v0.x;
        s = s + v0.y;
        s = s + v1.x;
        s = s + v1.y;
        s = s + v2.x;
        s = s + v2.y;
        s = s + v3.x;
        s = s + v3.y;
    }
    scores[r * C + c0 + j] = TAYLOR ? s / (double)n_el : s;
}

}  // namespace lpv

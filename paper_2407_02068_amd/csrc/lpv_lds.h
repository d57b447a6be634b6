// lpv_lds.h -- LDS access and global -> LDS DMA shared by the linear kernels
// (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lpv {

__device__ inline uint32_t lds_addr(const void* p)
{
    return (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) char*)p);
}

// Global -> LDS DMA of 16 bytes per lane to 1 KB at a wave-uniform LDS base.
// Issued from inline assembly: the compiler then neither drains this DMA
// before every LDS read of the wave (as it must for the builtin, which it
// knows writes LDS) nor counts it in its own vmcnt waits.  Every wait for it
// is explicit (the ring protocol: vmcnt wait + barrier per step); the memory
// clobber keeps the compiler's LDS reads in program order around it.
__device__ inline void dma16(const void* src, uint4* lds_wave_base)
{
    asm volatile(
        "s_nop 0\n"
        "global_load_lds_dwordx4 %0, off"
        :
        : "v"(src), "{m0}"(lds_addr(lds_wave_base))
        : "memory");
}

// The same from a wave-uniform base and a 32-bit per-lane byte offset (the
// saddr + voffset form: no 64-bit address per lane is kept live).
__device__ inline void dma16(const char* base, uint32_t off, uint4* lds_wave_base)
{
    asm volatile(
        "s_nop 0\n"
        "global_load_lds_dwordx4 %0, %1"
        :
        : "v"(off), "s"(base), "{m0}"(lds_addr(lds_wave_base))
        : "memory");
}

// The same with the instruction offset IMM, which the hardware adds to both
// the global and the LDS address (global: saddr + voff + IMM; LDS: M0 + IMM +
// 16 * lane).  Two DMAs 1 KB apart in LDS share one M0 value this way.
template <int IMM> __device__ inline void dma16i(const char* saddr, uint32_t voff, uint32_t m0)
{
    asm volatile(
        "s_nop 0\n"
        "global_load_lds_dwordx4 %0, %1 offset:%3"
        :
        : "v"(voff), "s"(saddr), "{m0}"(m0), "i"(IMM)
        : "memory");
}

typedef int v4i __attribute__((ext_vector_type(4)));

// 16-byte LDS read at a byte address (an ordinary load: the compiler places
// the lgkmcnt wait before the first use of the value).
template <int OFF> __device__ inline v4i lds_read16(uint32_t addr)
{
    return *(const __attribute__((address_space(3))) v4i*)(uintptr_t)(addr + OFF);
}

__device__ inline void lds_write16(uint32_t addr, v4i v)
{
    *(__attribute__((address_space(3))) v4i*)(uintptr_t)addr = v;
}

// Pair X (and dense W) layout in LDS: chunk ch (0..7: 16 bytes; 0..3 the first
// step's column tile, 4..7 the second's) of row r at r * 8 + (ch ^ swz(r)).
// A 16-byte read by 16 lanes (rows r .. r + 15 of one chunk) then touches 16
// different 16-byte bank groups (the LDS serves 256 bytes per clock).
__device__ inline int xswz(int r) { return (r >> 1) & 7; }

}  // namespace lpv

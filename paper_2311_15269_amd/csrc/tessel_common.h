// What the scoring kernels share on the device: block records, the order of candidates, bit and LDS helpers.
// (Included by the kernel sources only.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tessel_device.h"

namespace tessel {

struct BlockRec {
    int32_t  period;
    uint32_t n_retried;          // candidates whose first sweeps found no eigenvector (they got more in the same launch)
    uint64_t index;
    uint32_t n_status[kNumStatus];
    uint32_t n_evaluated;
    uint32_t n_sweeps;           // window sweeps spent on period computations
    uint32_t n_blocks;           // blocks placed by the build (fast kernel)
    uint32_t pad;
};

constexpr uint32_t kDrawLeadBase = 0u;
constexpr uint32_t kDrawOrdBase = 128u;

__device__ __forceinline__ uint32_t byte_of(uint32_t packed, uint32_t y) { return (packed >> (8u * y)) & 0xFFu; }

__device__ __forceinline__ bool key_less(int pa, uint64_t ia, int pb, uint64_t ib)
{
    return pa < pb || (pa == pb && ia < ib);
}

__device__ __forceinline__ uint32_t bfi(uint32_t sel, uint32_t a, uint32_t b) { return (sel & a) | (~sel & b); }

// position of the lowest set bit; all ones for 0, which "& 28", shift counts and bit-field offsets (all of them use the
// low five bits) read as 31: no guard bit has to be set first
__device__ __forceinline__ uint32_t low_bit(uint32_t x)
{
    uint32_t r;
    asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// a * b + c for a, b below 2^24, low 32 bits: the full-rate 24-bit multiply-add (b uniform)
__device__ __forceinline__ uint32_t mad24(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t r;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
    return r;
}

// keeps a value in a VGPR at this point, so that the loads above it are issued together instead of
// being sunk into later branches
#define TESSEL_PIN(x) asm volatile("" : "+v"(x))

// LDS accesses by byte address: address arithmetic stays integer arithmetic, and a constant added to an
// address goes into the instruction's offset field.
typedef __attribute__((address_space(3))) uint32_t lds_word;
__device__ __forceinline__ uint32_t lds_address(const void *p) { return (uint32_t)(uintptr_t)(const lds_word *)p; }
__device__ __forceinline__ uint32_t lds_load(uint32_t a) { return *(const lds_word *)(uintptr_t)a; }
__device__ __forceinline__ void lds_store(uint32_t a, uint32_t v) { *(lds_word *)(uintptr_t)a = v; }
__device__ __forceinline__ uint32_t lds_fetch_add(uint32_t a, uint32_t v)
{
    return __hip_atomic_fetch_add((lds_word *)(uintptr_t)a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// even bits of a 32-bit word, compacted (bit 2p -> bit p)
__device__ __forceinline__ uint32_t even_bits32(uint32_t x)
{
    x &= 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    x = (x | (x >> 8)) & 0x0000FFFFu;
    return x;
}

}  // namespace tessel

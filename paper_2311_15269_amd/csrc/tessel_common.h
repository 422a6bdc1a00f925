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
    uint32_t n_high;             // (sums of records) bits of n_sweeps above 32 << 16 | those of n_blocks
};

__device__ __forceinline__ uint32_t byte_of(uint32_t packed, uint32_t y) { return (packed >> (8u * y)) & 0xFFu; }

__device__ __forceinline__ bool key_less(int pa, uint64_t ia, int pb, uint64_t ib)
{
    return pa < pb || (pa == pb && ia < ib);
}

// Rates of this chip, measured with independent chains in all waves of a SIMD (T lane-operations/s of the chip): add, sub, and, or, xor, right
// shifts and bitop3 on vector registers, literals and small constants run at 58 (53 to 69); left shifts, minimum and maximum, compares and
// selects, bit-field and three-operand instructions, multiplies (the 32-bit ones too), and anything that reads a scalar
// register, a part of a word or another lane at 37.7.  (Program and table: profiles/instruction_rates.md.)
__device__ __forceinline__ uint32_t bfi(uint32_t sel, uint32_t a, uint32_t b) { return __builtin_amdgcn_bitop3_b32(sel, a, b, 0xCA); }

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

// The waves of a SIMD issue first in turns of 10 us, by their place on it (bits 0 to 3 of HW_ID) and the clock.  At one priority the oldest
// does: waves with the same work end one after the other, and the last runs alone.  `turns`, a wave's word: among how many it takes turns
// less one (a mask), the highest step of these that it gets << 2, what is added to the step << 4; 0, looked at by the callers: no turns.  (The clock takes a
// wave that is alone on its SIMD some 300 cycles a look, 300 candidates of 72 to 96 blocks 2 to 4 us a call; the callers put the call out of the way,
// which is worth another 0.5.)
__host__ __device__ constexpr uint32_t turns_of(uint32_t mask, uint32_t highest, uint32_t add) { return mask | highest << 2 | add << 4; }
__device__ __forceinline__ void take_turn(uint32_t turns)
{
    const uint32_t clock = ((uint32_t)__builtin_amdgcn_s_memrealtime() >> 10) + __builtin_amdgcn_s_getreg((3 << 11) | 4);
    const uint32_t turn = min(clock & turns & 3u, turns >> 2 & 3u) + (turns >> 4);
    if (turn == 0u) __builtin_amdgcn_s_setprio(0);
    else if (turn == 1u) __builtin_amdgcn_s_setprio(1);
    else if (turn == 2u) __builtin_amdgcn_s_setprio(2);
    else __builtin_amdgcn_s_setprio(3);
}

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

// half words.  (A row that is written by halves is also read by words: its accesses must not be reordered as if types told them apart.)
typedef __attribute__((address_space(3), may_alias)) uint16_t lds_half;
__device__ __forceinline__ uint32_t lds_load16(uint32_t a) { return *(const lds_half *)(uintptr_t)a; }
__device__ __forceinline__ void lds_store16(uint32_t a, uint32_t v) { *(lds_half *)(uintptr_t)a = (uint16_t)v; }

// a device's order while it is decoded: bit p of plane k = bit k of the symbol at position p
template <int NP>
struct Planes {
    uint32_t p0, p1, p2;
    __device__ __forceinline__ void clear() { p0 = p1 = p2 = 0; }
    __device__ __forceinline__ void put(uint32_t y, uint32_t pos)
    {
        p0 |= (y & 1u) << pos;
        if (NP > 1) p1 |= ((y >> 1) & 1u) << pos;
        if (NP > 2) p2 |= (y >> 2) << pos;
    }
};

// blocks of device d in the sampled spaces: a draw picks among the blocks left, types in ascending order
template <int NP>
__device__ __forceinline__ void sampled_order(uint32_t ka, uint32_t kb, int d, uint32_t ntd, uint32_t NR, Planes<NP> &o)
{
    const uint32_t n = ntd * NR;
    o.clear();
    // cumulative counts of the blocks left by type: one (shifted by 16) for two types; else bytes 0x80 - t, so that adding
    // the replicated digit leaves "digit >= t" in bit 7 of every byte (t, digit <= 32)
    uint32_t c = NR << 16, ta = 0, tb = 0, tc = 0;
    if (NP > 1) {
        auto cum = [&](uint32_t k) -> uint32_t { return min(k, ntd) * NR; };
        ta = 0x808080u - (cum(1) | (cum(2) << 8) | (cum(3) << 16));
        if (NP > 2) { tb = 0x808080u - (cum(4) | (cum(5) << 8) | (cum(6) << 16)); tc = 0x80u - cum(7); }
    }
    auto pick = [&](uint32_t draw, uint32_t left, uint32_t pos) {
        if (NP == 1) {
            const uint32_t prod = __umul24(draw, left);
            const uint32_t y = prod >= c ? 1u : 0u;
            c -= y ? 0u : 0x10000u;
            o.p0 |= y << pos;
            return;
        }
        const uint32_t digit = (uint32_t)(((uint64_t)draw * (uint64_t)((left << 16) & 0xFFFFFFu)) >> 32);   // 24-bit high multiply
        const uint32_t ga = mad24(digit, 0x010101u, ta) & 0x808080u;
        ta += (ga >> 7) ^ 0x010101u;                    // a threshold above the digit loses one block
        uint32_t y = (uint32_t)__builtin_popcount(ga);
        if (NP > 2) {
            const uint32_t gb = mad24(digit, 0x010101u, tb) & 0x808080u;
            tb += (gb >> 7) ^ 0x010101u;
            const uint32_t gc = (tc + digit) & 0x80u;
            tc += (gc >> 7) ^ 1u;
            y += (uint32_t)__builtin_popcount(gb) + (gc >> 7);
        }
        o.put(y, pos);
    };
    uint32_t pos = 0;
    // (four draws at a time: the two words' hashes overlap)
    for (; pos + 4 <= n; pos += 4) {
        const uint32_t w0 = stream_word(ka, kb, (kDrawOrdBase + 32u * (uint32_t)d + pos) >> 1);
        const uint32_t w1 = stream_word(ka, kb, ((kDrawOrdBase + 32u * (uint32_t)d + pos) >> 1) + 1u);
        pick(w0 & 0xFFFFu, n - pos, pos);
        pick(w0 >> 16, n - pos - 1u, pos + 1u);
        pick(w1 & 0xFFFFu, n - pos - 2u, pos + 2u);
        pick(w1 >> 16, n - pos - 3u, pos + 3u);
    }
    for (; pos < n; pos += 2) {
        const uint32_t word = stream_word(ka, kb, (kDrawOrdBase + 32u * (uint32_t)d + pos) >> 1);
        pick(word & 0xFFFFu, n - pos, pos);
        if (pos + 1 < n) pick(word >> 16, n - pos - 1u, pos + 1u);
    }
}

}  // namespace tessel

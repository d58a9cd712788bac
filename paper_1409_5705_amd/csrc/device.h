// Device functions that several kernel files share.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace sfb {

// Two fp32 values as bf16, round to nearest even; the first in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    floatx2 f = {a, b};
    bf16x2 h = __builtin_convertvector(f, bf16x2);
    return __builtin_bit_cast(uint32_t, h);
}

// Slot swizzle of the eight 16-byte chunks of a 128-byte LDS row r: chunk c of the row sits in slot c ^ swz(r).
// Chosen by measurement: an MFMA operand read (runs of 16 consecutive rows at one
// chunk, 16 bytes a lane: rows of either parity meet the eight slots once each)
// costs 26.9 cycles with this function, as little as with padded rows, against
// 32.2 with r & 7 or (r >> 1) ^ (r >> 3) and 128 without a swizzle.
// swz(r + 16) = swz(r) ^ 2, swz(r + 32) = swz(r) ^ 4 and swz(r + 64) = swz(r).
__device__ __forceinline__ int swz(int r) { return (r ^ (r >> 3)) & 7; }

// f(integral_constant<int, B>), ..., f(integral_constant<int, E - 1>): a loop that is unrolled by construction (some
// bodies are beyond what the unroller accepts under a pragma, and an index that is not a constant would put
// accumulators in scratch memory).
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// A wave-uniform 64-bit value as the compiler can see it (scalar registers).
__device__ __forceinline__ uint64_t uniform64(uint64_t a)
{
    // (the builtin returns a signed int: narrow to 32 unsigned bits before widening)
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    return ((uint64_t)hi << 32) | (uint64_t)lo;
}

// 16 bytes per lane from global memory straight into LDS: lane l's bytes land at
// LDS address lds_addr + 16 l (lds_addr wave-uniform, in M0); the global address
// is gbase (uniform) + voff (per lane).  Issued as inline assembly so that the
// compiler's wait-count insertion does not tie every later LDS read to it; the
// caller waits (vmcnt) before the barrier that publishes the data.
// NT: non-temporal, for an operand whose lines are used by a few CUs at about the
// same time and never again.
template <bool NT = false>
__device__ __forceinline__ void load_to_lds_16(uint32_t lds_addr, uint64_t gbase, uint32_t voff)
{
    if (NT)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_addr), "v"(voff), "s"(gbase)
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(gbase)
                     : "memory");
}

}  // namespace sfb

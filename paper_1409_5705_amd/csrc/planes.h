// The parameter matrix of the bf16 path as its kernels see it: the blocks of a bf16 operand, the two 16-bit planes.
#pragma once
#include "device.h"
#include "kernels.h"

namespace sfb {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int BK = 64;                   // columns of a block of an operand (BM rows x BK columns)
constexpr int BM = 256, BN = 256;        // rows of such a block; the low plane is stored in tiles of BM x BN
// Cache policy of the accesses of C and of its bf16 copy: non-temporal (each
// line is touched once per launch; left at the default policy they sweep the
// operand panels, which ARE reused, out of the 4 MiB L2 of the XCD).
constexpr int C_POLICY = 2;

// A parameter matrix kept as two 16-bit planes: the halves of word = bits + 0x8000 (modulo 2^32).  hi = word >> 16
// is the value rounded to bf16 (to nearest, ties away from zero), lo = word & 0xffff; bits = ((hi << 16) | lo) -
// 0x8000, exactly.  Two elements a dword in both planes: split_pair / join_pair move between the packed halves and
// the two words with one byte permute each.
__device__ __forceinline__ uint32_t split_word(float v) { return __float_as_uint(v) + 0x8000u; }
__device__ __forceinline__ float split_value(uint32_t word) { return __uint_as_float(word - 0x8000u); }
// words of elements 0 and 1 from their packed high halves h = [h1 : h0] and low halves l = [l1 : l0]
__device__ __forceinline__ uint32_t join_pair0(uint32_t h, uint32_t l) { return __builtin_amdgcn_perm(h, l, 0x05040100u); }
__device__ __forceinline__ uint32_t join_pair1(uint32_t h, uint32_t l) { return __builtin_amdgcn_perm(h, l, 0x07060302u); }
// packed high halves [w1 >> 16 : w0 >> 16] and low halves [w1 & 0xffff : w0 & 0xffff] of two words
__device__ __forceinline__ uint32_t pack_hi(uint32_t w0, uint32_t w1) { return __builtin_amdgcn_perm(w1, w0, 0x07060302u); }
__device__ __forceinline__ uint32_t pack_lo(uint32_t w0, uint32_t w1) { return __builtin_amdgcn_perm(w1, w0, 0x05040100u); }

// Whether any of the LANES neighbouring lanes that write one 128-byte line of the bf16 copy (high plane) has something to
// write there: a line is stored whole or not at all, since one written in part costs the memory a read as well.  Measured:
// apply of 40000 x 10000 with 100 pairs, 2 to 3 % of the values changing, 0.97 -> 0.83 ms with the copy, 0.69 -> 0.57 on
// the planes.  (In the 256 x 256 kernel, with its many pairs, it gains nothing.)
template <int LANES>
__device__ __forceinline__ bool any_in_line(bool mine, int lane)
{
    const uint64_t b = __builtin_amdgcn_ballot_w64(mine);
    return ((b >> (lane & ~(LANES - 1))) & ((1ull << LANES) - 1)) != 0;
}

}  // namespace sfb

// What the two kernels of the column-order search share: the ways of dealing eight columns out as two groups of four.
#pragma once
#include "common.hpp"

namespace sp24 {

// The 35 ways in lexicographic order of (a, b, c), as bit masks of the positions a, b, c (1 .. 7; bit 0 for position 1),
// nine to a word: read with shifts, not from memory.
struct Ways {
    uint64_t word[4];
};
constexpr Ways make_ways()
{
    Ways t{};
    int n = 0;
    for (int a = 1; a < 8; ++a)
        for (int b = a + 1; b < 8; ++b)
            for (int c = b + 1; c < 8; ++c, ++n) t.word[n / 9] |= (uint64_t)((1u << (a - 1)) | (1u << (b - 1)) | (1u << (c - 1))) << (7 * (n % 9));
    return t;
}

// The four positions of way w that share a group with position 0, that one among them, as a bit mask of 0 .. 7
__host__ __device__ constexpr uint32_t way_mask(int w)
{
    constexpr Ways t = make_ways();
    const uint64_t word = w < 9 ? t.word[0] : w < 18 ? t.word[1] : w < 27 ? t.word[2] : t.word[3];
    return 1u | ((uint32_t)(word >> (7 * (w % 9))) & 127u) << 1;
}

// The larger of two sums of magnitudes (never NaN); two rows of int8 at once as 16-bit halves
typedef uint16_t ushort2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int larger(int a, int b) { return a > b ? a : b; }
__device__ __forceinline__ double larger(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ ushort2v larger(ushort2v a, ushort2v b) { return __builtin_elementwise_max(a, b); }

// position of the i-th set bit
__device__ __forceinline__ int nth_bit(uint32_t mask, int i)
{
    for (; i > 0; --i) mask &= mask - 1;
    return __builtin_ctz(mask);
}

} // namespace sp24

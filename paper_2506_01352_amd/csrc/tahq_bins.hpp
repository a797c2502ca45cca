// The orders and bins of entropies that the selection of the widest tiles works with.  Nothing here touches memory or knows of
// lanes, so that a host program can run the same functions on every value that matters.
#pragma once
#include <stdint.h>

namespace tahq {

constexpr uint32_t kLinBins = 2048;       // linear bins of the entropy histogram (selection of large units)
constexpr uint32_t kSubBins = 1024;       // sub-bins of the bin that holds the threshold (k_select_resolve)

// Order-preserving 32-bit key of an entropy (larger entropy -> larger key).
__device__ __forceinline__ uint32_t order_key(float h)
{
    const uint32_t u = __float_as_uint(h);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Linear bin of an entropy, 0 .. kLinBins - 1: non-decreasing in the entropy's order-preserving key (so a higher bin
// means a higher rank), and the same instruction sequence wherever it is evaluated.  Negative values go to bin 0; a NaN
// goes where its key goes: above +infinity with the sign bit clear, below -infinity with it set.
__device__ __forceinline__ uint32_t linear_bin(float h, float scale)
{
    // the median of three takes a NaN for the smallest of the three (bin 0, where a NaN with the sign bit set belongs)
    const uint32_t b = (uint32_t)__builtin_amdgcn_fmed3f(h * scale, 0.0f, (float)(kLinBins - 1));
    return (int32_t)__float_as_uint(h) > 0x7f800000 ? kLinBins - 1 : b;
}

// Sub-bin of an entropy that lies in linear bin `b`, 0 .. kSubBins - 1: non-decreasing in the entropy's key.  h * scale
// is the product linear_bin rounds down; its distance to b is exact in fp32, and so is the multiplication by a power of
// two.
__device__ __forceinline__ uint32_t linear_sub_bin(float h, float scale, uint32_t b)
{
    const uint32_t s = (uint32_t)__builtin_amdgcn_fmed3f((h * scale - (float)b) * (float)kSubBins, 0.0f, (float)(kSubBins - 1));
    return (int32_t)__float_as_uint(h) > 0x7f800000 ? kSubBins - 1 : s;
}

// The same for a bin that many tiles share: most of them may be alike, and the usual ones are all-zero tiles.  In the lowest bin
// their entropy, +0.0f, has sub-bin 1 to itself, with whatever is negative below it.
__device__ __forceinline__ uint32_t crowd_sub_bin(float h, float scale, uint32_t b)
{
    const uint32_t s = linear_sub_bin(h, scale, b);
    if (b != 0) return s;
    const int32_t v = (int32_t)__float_as_uint(h);
    return v == 0 ? 1u : v < 0 ? 0u : s < 2u ? 2u : s;
}

// The entropy an order-preserving key was made from.
__device__ __forceinline__ float key_to_float(uint32_t key)
{
    return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}

// The bit pattern of the smallest entropy in linear bin `b`, 1 .. kLinBins - 1 (a larger b counts as the last).  The division and
// the product in linear_bin round once each, so it lies at most three floats from b / scale: eight steps, whatever the
// arguments are.
__device__ __forceinline__ int linear_bin_edge(uint32_t b, float scale)
{
    const uint32_t bin = b < kLinBins ? b : kLinBins - 1;
    int e = (int)__float_as_uint((float)bin / scale) - 4;
#pragma unroll 1
    for (int step = 0; step < 8; ++step) e += linear_bin(__uint_as_float((uint32_t)e), scale) < bin ? 1 : 0;
    return e;
}

}  // namespace tahq

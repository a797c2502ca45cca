// What the selections and the launch that ranks and quantizes share: scans of a wavefront, the search for a histogram's bin, a ranking
// unit in places.
#pragma once
#include "tahq_common.hpp"
#include "tahq_stream_kernels.hpp"

namespace tahq {

// Inclusive scan over the 64 lanes of a wavefront with data-parallel-primitive moves (all lanes must be
// enabled): shifts by 1, 2, 4, 8 inside each row of 16 lanes, then the last lane of row 0 / 2 is added to
// row 1 / 3, then the last lane of the lower half to the upper half.  A lane without a source adds 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += dpp_or_zero<0x111, 0xF>(v);     // row_shr:1
    v += dpp_or_zero<0x112, 0xF>(v);     // row_shr:2
    v += dpp_or_zero<0x114, 0xF>(v);     // row_shr:4
    v += dpp_or_zero<0x118, 0xF>(v);     // row_shr:8
    v += dpp_or_zero<0x142, 0xA>(v);     // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xC>(v);     // row_bcast:31 into rows 2 and 3
    return v;
}

// The four bits of eight neighbouring lanes as one dword, lowest lane first; in each of the eight.
__device__ __forceinline__ uint32_t nibbles_to_dword(uint32_t four, int lane)
{
    uint32_t d = four << (4 * (lane & 7));
    d |= dpp_or_zero<0xB1, 0xF>(d);              // lane ^ 1
    d |= dpp_or_zero<0x4E, 0xF>(d);              // lane ^ 2
    d |= dpp_or_zero<0x141, 0xF>(d);             // lane ^ 7: the other four
    return d;
}

// The largest a and the largest b of the wavefront, in every lane.
__device__ __forceinline__ void wave_max(uint32_t &a, uint32_t &b)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t oa = (uint32_t)__shfl_xor((int)a, off, 64), ob = (uint32_t)__shfl_xor((int)b, off, 64);
        a = oa > a ? oa : a;
        b = ob > b ? ob : b;
    }
}

// The 16 wavefronts' entries of `totals` that come before mine, added up.
__device__ __forceinline__ uint32_t sum_of_waves_before(const uint32_t *totals, uint32_t wave, int lane)
{
    const uint32_t own = totals[lane & 15];
    uint32_t v = own;
    v += dpp_or_zero<0x111, 0xF>(v);             // a scan over each row of 16 lanes
    v += dpp_or_zero<0x112, 0xF>(v);
    v += dpp_or_zero<0x114, 0xF>(v);
    v += dpp_or_zero<0x118, 0xF>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)(v - own), (int)wave);
}

// hist[bin] += 1 in LDS for every lane that is `active`.  Where many tiles are alike whole wavefronts meet on one address, whose
// additions would follow one another: then it is one addition.  (Adding up the lanes of one bin beforehand in every case cost a
// selection from 7000 different candidates 1.5 us.)
__device__ __forceinline__ void add_one_each(uint32_t *hist, uint32_t bin, bool active)
{
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
    if (__ballot(active && bin == first) == ~0ull) {
        if ((threadIdx.x & 63) == 0) atomicAdd(&hist[first], 64u);
    } else if (active) {
        atomicAdd(&hist[bin], 1u);
    }
}

// Which of BINS bins holds the `want`-th largest value (bins counted from the top), how many values are wanted inside it and how
// many it holds, found by the whole workgroup of 1024 threads: BINS / 1024 bins per thread and a scan.  chosen[0..2] is written
// before the last of its two barriers, and left as it was where there are fewer than `want` values; `totals`: 16 words of LDS.
// (One wavefront with a sixteenth of the bins per lane, its loads as far apart, took 1.5 us longer.)
template <int BINS>
__device__ __forceinline__ void block_pick_bin(const uint32_t *hist, uint32_t want, uint32_t *totals, uint32_t *chosen)
{
    constexpr int PER = BINS / 1024;
    static_assert(PER == 1 || PER == 2 || PER % 4 == 0, "whole loads");
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t low = (uint32_t)(BINS - PER * (tid + 1));                   // my bins: low .. low + PER - 1
    uint32_t c[PER], mine = 0;
    if constexpr (PER == 1) {
        c[0] = hist[low];
    } else if constexpr (PER == 2) {
        const uint2 q = *reinterpret_cast<const uint2 *>(hist + low);
        c[0] = q.x; c[1] = q.y;
    } else {
#pragma unroll
        for (int i = 0; i < PER / 4; ++i) {
            const uint4 q = reinterpret_cast<const uint4 *>(hist + low)[i];
            c[4 * i] = q.x; c[4 * i + 1] = q.y; c[4 * i + 2] = q.z; c[4 * i + 3] = q.w;
        }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) mine += c[i];
    const uint32_t incl = wave_incl_scan(mine);
    if (lane == 63) totals[wave] = incl;
    __syncthreads();
    uint32_t above = sum_of_waves_before(totals, wave, lane) + incl - mine;
    if (above < want && want <= above + mine) {
#pragma unroll
        for (int i = PER; i-- > 0;) {
            if (above < want && want <= above + c[i]) { chosen[0] = low + i; chosen[1] = want - above; chosen[2] = c[i]; }
            above += c[i];
        }
    }
    __syncthreads();
}

#ifndef TAHQ_SMALL_UNIT_MAX
#define TAHQ_SMALL_UNIT_MAX 32768
#endif
// Places (tiles, counted from the 64-tile boundary at or before the unit's first tile) that the LDS of one workgroup holds.
constexpr uint32_t kSmallUnitMaxKeys = TAHQ_SMALL_UNIT_MAX;
constexpr uint32_t kSmallListCap = 256;          // tiles of the threshold bin that are placed directly

// A ranking unit in places: a place is a tile's index counted from the 64-tile boundary at or before the unit's first tile, so
// that 64 places are one word of the bit map, which the unit may share with a neighbour at either end.
struct UnitPlaces {
    uint32_t phase, end, nwords;                 // places of the unit: [phase, end)
    uint64_t word0;                              // its first word in the bit map
    __device__ __forceinline__ UnitPlaces(uint32_t u, uint32_t n)
    {
        const uint64_t j0 = (uint64_t)u * n;
        phase = (uint32_t)(j0 & 63u);
        end = phase + n;
        nwords = (end + 63) / 64;
        word0 = j0 >> 6;
    }
    // places of word g that belong to the unit
    __device__ __forceinline__ uint64_t mask(uint32_t g) const
    {
        uint64_t m = ~0ull;
        if (g == 0) m <<= phase;
        if (end - g * 64u < 64u) m &= (1ull << (end - g * 64u)) - 1ull;
        return m;
    }
};

// Word g of a unit whose selected places are `bits`; a shared word has been cleared by an earlier kernel.
__device__ __forceinline__ void put_word(uint64_t *word, uint64_t mask, uint64_t bits)
{
    if (mask == ~0ull) *word = bits;
    else atomicOr(reinterpret_cast<unsigned long long *>(word), (unsigned long long)bits);
}

}  // namespace tahq

// Selection and quantizer in one launch (Sec. 3.2 top-p%, Sec. 3.3 Eq. 3-4, Sec. 3.4), for tensors that are one round of workgroups: every
// workgroup ranks its tiles' whole unit for itself, while the rows it will quantize are on their way.
#pragma once
#include "tahq_rank_common.hpp"

namespace tahq {

constexpr int kCrewThreads = 1024, kCrewWaves = kCrewThreads / 64;
// Places of a unit whose entropies stay in LDS beside the histogram, and of a unit at all.  Larger units are read from memory for
// every pass, two or three, out of the L2: encode of bf16, against a selection of its own (one launch up to 65536 tiles, two and a
// histogram in the entropy pass above), at 3.8 bits: one unit of 32768 tiles G = 16 14.9 -> 11.2 us, 49152 20.3 -> 13.5,
// 65536 22.6 -> 15.7, 77700 28.5 -> 17.7, 98304 29.3 -> 20.1, 131072 29.1 -> 24.8, 163840 30.4 -> 29.0; G = 64 49152 23.7 -> 16.0, 98304
// 34.2 -> 26.0, 114688 35.5 -> 30.2; [3,777,1600] G = 16 at 2.25 bits 29.0 -> 23.7.  Ends where a threshold among tiles that are alike,
// which takes four passes, costs clearly more than the other way: a fifth of the tokens constant, G = 8, one unit of 90112 tiles 35.3 ->
// 35.7, 98304 36.7 -> 38.2 (ordinary ones 25.7 -> 20.8), two of 86016 37.4 -> 35.3, 90112 34.5 -> 36.2, 98304 35.4 -> 38.6; fp32 G = 16
// two of 98304 ordinary tiles 26.4 -> 27.9.
constexpr uint32_t kCrewPlaces = 28672, kCrewMost = 98304, kCrewMostOfSeveral = 86016;
// Bins of 2048 neighbouring floats, two octaves below ln A: half as wide as k_select_small's, so that half as many tiles have to be
// placed directly.
constexpr uint32_t kCrewBins = 8192;
constexpr int kCrewShift = 11;
constexpr uint32_t kCrewMany = 2048;             // tiles of the threshold's bin that are listed at all

struct CrewLds {
    uint64_t list[kSmallListCap];                // tiles of the threshold bin: key << 32 | ~place
    uint64_t words[kCrewWaves], equal[kCrewWaves];                         // bit map words of the batch, and those that share the threshold
    uint32_t wave_total[kCrewWaves];
    uint32_t chosen[3];                          // threshold bin, wanted inside it, its tiles
    uint32_t listed;
    uint32_t above_zero, zero;                   // the lowest bin's entropies above +0.0f and equal to it
    uint32_t before, equal_before;               // selected places before the batch, and those that share the threshold
};

// Lane i's value becomes the sum of those before it among 16.
__device__ __forceinline__ uint32_t before_in_sixteen(uint32_t own)
{
    uint32_t v = own;
    v += dpp_or_zero<0x111, 0xF>(v);
    v += dpp_or_zero<0x112, 0xF>(v);
    v += dpp_or_zero<0x114, 0xF>(v);
    v += dpp_or_zero<0x118, 0xF>(v);
    return v - own;
}

// The bit patterns of a unit's entropies, four consecutive places per lane and block of 256, places outside the unit as that of -0.0f,
// the lowest of all as a signed integer and no entropy's: from LDS, where they lie by place, or from memory each time.
template <bool RESIDENT>
struct UnitKeys {
    static constexpr bool resident = RESIDENT;
    int *key;                                    // in LDS
    const float *uH;                             // in memory, by place
    uint32_t n, phase, end, top;
    uint32_t lane, wave;
    __device__ __forceinline__ UnitKeys(int *lds, const float *H, const UnitPlaces &at, uint32_t unit)
        : key(lds), uH(H), n(unit), phase(at.phase), end(at.end), top(at.nwords * 64u - 4u), lane(threadIdx.x & 63u),
          wave((uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) {}
    __device__ __forceinline__ uint32_t blocks() const { return (end + 255u) / 256u; }
    // The unit's entropies straight to LDS.  (Whole words of 64 places are read, which may reach into the neighbouring units or up
    // to 63 floats past the entropies, where the workspace goes on; beyond them from a clamped index.)
    __device__ __forceinline__ void request() const
    {
        static_assert(RESIDENT, "in LDS");
#pragma unroll 1
        for (uint32_t b = wave; b * 256u < end; b += kCrewWaves) {
            const uint32_t place = b * 256u + 4u * lane;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(uH + (place < top ? place : top)),
                                             (__attribute__((address_space(3))) void *)&key[b * 256u], 16, 0, 0);
        }
    }
    __device__ __forceinline__ bool edge(uint32_t b) const
    {
        return (b == 0 && phase != 0) || (b == blocks() - 1 && (end & 255u) != 0);
    }
    __device__ __forceinline__ int4 inside(uint32_t b, int4 q) const
    {
        const uint32_t i = b * 256u + 4u * lane - phase;
        q.x = i < n ? q.x : INT32_MIN; q.y = i + 1u < n ? q.y : INT32_MIN;
        q.z = i + 2u < n ? q.z : INT32_MIN; q.w = i + 3u < n ? q.w : INT32_MIN;
        return q;
    }
    // f(block, its four bit patterns) for my wavefront's blocks below `last`; FIRST: the first time
    template <bool FIRST, class F>
    __device__ __forceinline__ void each(uint32_t last, F f) const
    {
        if constexpr (RESIDENT) {
            if (wave >= last) return;
            int4 next = *reinterpret_cast<const int4 *>(&key[wave * 256u + 4u * lane]);
#pragma unroll 1
            for (uint32_t b = wave; b < last; b += kCrewWaves) {
                int4 q = next;
                if (b + kCrewWaves < last) next = *reinterpret_cast<const int4 *>(&key[(b + kCrewWaves) * 256u + 4u * lane]);
                if (FIRST && edge(b)) {
                    q = inside(b, q);
                    *reinterpret_cast<int4 *>(&key[b * 256u + 4u * lane]) = q;
                }
                f(b, q);
            }
        } else {
            constexpr uint32_t AHEAD = 2;        // blocks on their way (4 as fast, 8 slower by 1 us: more code to fetch)
            auto load = [&](uint32_t b) {
                const uint32_t place = b * 256u + 4u * lane;
                return *reinterpret_cast<const int4 *>(uH + (place < top ? place : top));
            };
            int4 q[AHEAD];
#pragma unroll
            for (uint32_t i = 0; i < AHEAD; ++i) q[i] = load(wave + i * kCrewWaves);
#pragma unroll 1
            for (uint32_t b0 = wave; b0 < last; b0 += AHEAD * kCrewWaves) {
#pragma unroll
                for (uint32_t i = 0; i < AHEAD; ++i) {
                    const uint32_t b = b0 + i * kCrewWaves;
                    if (b < last) f(b, edge(b) ? inside(b, q[i]) : q[i]);
                    q[i] = load(b + AHEAD * kCrewWaves);
                }
            }
        }
    }
};

// Median of three integers in one vector instruction.
__device__ __forceinline__ int imed3(int a, int b, int c)
{
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// A unit's entropies counted in bins of 2^kCrewShift neighbouring floats by the whole workgroup, all but the lowest bin's, which the
// caller has filled.  Its usual ones are all-zero tiles, whose additions, a wavefront's at a time, would meet on one counter; they
// go to 64 words in front of the histogram instead, a lane's each.  (Encode of [1,1000,4096] G = 32, a fifth of the tokens all zero,
// 49 us with a counter, 29 so; with those lanes switched off 30, and every other tensor 0.3 us longer.  [3,777,1600] G = 16 with a fifth
// constant 43 us at one addition per tile, 35 as below.)
template <class Keys>
__device__ __forceinline__ void count_places(const Keys &keys, uint32_t *hist, int bin0)
{
    const int mine = -1 - (int)keys.lane;
    keys.template each<true>(keys.blocks(), [&](uint32_t, const int4 &q) {
        const int v[4] = {q.x, q.y, q.z, q.w};
        auto add = [&](int value, uint32_t times) {
            const int bin = (value >> kCrewShift) - bin0;    // as signed integers: negative values and NaN with the sign bit set lowest
            atomicAdd(hist + imed3(bin, mine, (int)kCrewBins - 1), times);
        };
        if (!Keys::resident && __builtin_expect(__ballot(v[0] == v[3]) != 0, 0)) {
            // (tokens that are alike make a crowd of neighbours: one addition for the four.  In small units it takes longer than that)
            if (v[0] == v[1] && v[1] == v[2] && v[2] == v[3]) {
                add(v[0], 4);
                return;
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) add(v[c], 1);
    });
}

// Which of the places [p0, p0 + batch) of a unit are selected, and how many before them, found by the whole workgroup from the unit's
// entropies and their counts.  p0 and batch are multiples of 64.  The result is in L.words and L.before behind the last barrier.
template <class Keys>
__device__ __forceinline__ void rank_batch(const Keys &keys, uint32_t *hist, uint32_t n, uint32_t k, int bin0, uint32_t p0, uint32_t batch,
                                           CrewLds &L)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t nblocks = keys.blocks();
    const uint32_t upto = (p0 + batch + 255u) / 256u < nblocks ? (p0 + batch + 255u) / 256u : nblocks;        // blocks up to the batch's end
    lds_barrier();
    block_pick_bin<(int)kCrewBins>(hist, k, L.wave_total, L.chosen);
    const uint32_t bstar = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[0]);
    uint32_t rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[1]);
    uint32_t crowd = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[2]);
    if (bstar == 0) crowd = n - (k - rem);       // (it was filled with as many as there could be)
    // the bit patterns of that bin, first and last
    int lo = bstar == 0 ? INT32_MIN + 1 : (int)((bstar + (uint32_t)bin0) << kCrewShift);
    int hi = bstar == kCrewBins - 1 ? INT32_MAX : (int)(((bstar + (uint32_t)bin0 + 1u) << kCrewShift) - 1u);
    auto four_bits = [](const int4 &q, auto test) {
        return (test(q.x) ? 1u : 0u) | (test(q.y) ? 2u : 0u) | (test(q.z) ? 4u : 0u) | (test(q.w) ? 8u : 0u);
    };
    // block b's four bits per lane: counted where they lie before the batch, or put into its words
    auto put_bits = [&](uint64_t *out, uint32_t b, uint32_t four) {
        const uint32_t place = b * 256u + 4u * lane, d = nibbles_to_dword(four, lane);
        if ((lane & 7) == 0 && place >= p0 && place < p0 + batch) reinterpret_cast<uint32_t *>(out)[(place - p0) >> 5] = d;
    };
    uint32_t before = 0;
    // Every place that is_above is selected; those others that are not below are listed.
    auto classify = [&](uint64_t *list, uint32_t mask, auto is_above, auto is_not_below, auto any_between) {
        keys.template each<false>(nblocks, [&](uint32_t b, const int4 &q) {
            if (__ballot(any_between(q)) != 0) {
                const int v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (is_not_below(v[c]) && !is_above(v[c]))
                        list[atomicAdd(&L.listed, 1u) & mask] =
                            ((uint64_t)order_key(__uint_as_float((uint32_t)v[c])) << 32) | (uint32_t)~(b * 256u + 4u * lane + c);
                }
            }
            if (b * 256u + 256u <= p0) {
                before += is_above(q.x) ? 1u : 0u; before += is_above(q.y) ? 1u : 0u;
                before += is_above(q.z) ? 1u : 0u; before += is_above(q.w) ? 1u : 0u;
            } else if (b * 256u < p0 + batch) {
                const uint32_t above = four_bits(q, is_above);
                put_bits(L.words, b, above);
                if (b * 256u + 4u * lane < p0) before += (uint32_t)__popc(above);
            }
        });
        lds_barrier();
    };
    auto select = [&](bool selected, uint32_t place) {
        const uint64_t earlier = __ballot(selected && place < p0);
        if (lane == 0 && earlier != 0) atomicAdd(&L.before, (uint32_t)__popcll(earlier));
        if (selected && place >= p0 && place < p0 + batch)
            atomicOr(reinterpret_cast<uint32_t *>(L.words) + ((place - p0) >> 5), 1u << (place & 31u));
    };
    // Of the `crowd` listed tiles the `rem` first by (key descending, tile ascending): four threads per tile count those ahead of it.
    auto place_listed = [&]() {
        before = wave_incl_scan(before);
        if (lane == 63 && before != 0) atomicAdd(&L.before, before);
        if ((uint32_t)tid < 4 * crowd) {
            const uint64_t mine = L.list[tid >> 2];
            uint32_t ahead = 0;
#pragma unroll 4
            for (uint32_t i = (uint32_t)tid & 3u; i < crowd; i += 4) ahead += L.list[i] > mine ? 1u : 0u;
            ahead += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ahead, 0xB1, 0xF, 0xF, true);      // lane ^ 1
            ahead += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ahead, 0x4E, 0xF, 0xF, true);      // lane ^ 2
            select(((uint32_t)tid & 3u) == 0 && ahead < rem, ~(uint32_t)mine);
        }
        lds_barrier();
    };
    const bool few = crowd <= kSmallListCap;
    if (__builtin_expect(few || (bstar != 0 && crowd <= kCrewMany), 1)) {
        // the histogram's first half takes the list of many, its second half the counts of their parts
        uint64_t *many = reinterpret_cast<uint64_t *>(hist);
        uint32_t *parts = hist + kCrewBins / 2;
        static_assert(kCrewMany * 2 <= kCrewBins / 2 && kCrewBins / 2 >= 4096, "they fit");
        if (!few) reinterpret_cast<uint4 *>(parts)[tid] = make_uint4(0, 0, 0, 0);
        classify(few ? L.list : many, few ? kSmallListCap - 1u : kCrewMany - 1u, [&](int v) { return v > hi; },
                 [&](int v) { return v >= lo; }, [&](const int4 &q) {
            const uint32_t a = (uint32_t)q.x - (uint32_t)lo, b = (uint32_t)q.y - (uint32_t)lo, c = (uint32_t)q.z - (uint32_t)lo,
                           d = (uint32_t)q.w - (uint32_t)lo, ab = a < b ? a : b, cd = c < d ? c : d;
            return (ab < cd ? ab : cd) <= (uint32_t)hi - (uint32_t)lo;
        });
        if (few) { place_listed(); return; }
        // Many: the list is cut into 4096 parts, of one float each as a rule, and what is in the threshold's placed directly.  (Units of
        // 65536 tiles and more have hundreds of ordinary tiles in a bin, and a second pass over 128000 entropies took 15 us.)
        const uint32_t key0 = order_key(__uint_as_float((uint32_t)lo)), span = (uint32_t)hi - (uint32_t)lo;
        const int bits = 32 - __builtin_clz(span | 1u), shift = bits > 12 ? bits - 12 : 0;
        for (uint32_t i = (uint32_t)tid; i < crowd; i += kCrewThreads) atomicAdd(&parts[((uint32_t)(many[i] >> 32) - key0) >> shift], 1u);
        if (tid == 0) L.listed = 0;
        lds_barrier();
        block_pick_bin<4096>(parts, rem, L.wave_total, L.chosen);
        const uint32_t part = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[0]), most = crowd;
        rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[1]);
        crowd = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[2]);
        if (crowd <= kSmallListCap) {
            for (uint32_t i = (uint32_t)tid; i < (most + 63u) / 64u * 64u; i += kCrewThreads) {      // (whole wavefronts)
                const uint64_t entry = i < most ? many[i] : 0ull;
                const uint32_t in = i < most ? ((uint32_t)(entry >> 32) - key0) >> shift : 0u;
                if (i < most && in == part) L.list[atomicAdd(&L.listed, 1u) & (kSmallListCap - 1u)] = entry;
                select(i < most && in > part, ~(uint32_t)entry);
            }
            lds_barrier();
            place_listed();
            return;
        }
        // (too many that are nearly alike: the general way, inside that part)
        lo = (int)((uint32_t)lo + (part << shift));
        const uint32_t room = (uint32_t)hi - (uint32_t)lo, whole = (1u << shift) - 1u;
        hi = (int)((uint32_t)lo + (room < whole ? room : whole));
        before = 0;
    }
    // More tiles in the bin than the list takes: it is cut again, 4096 parts at a time, until they fit or all share one
    // entropy.  Bit patterns count in the order of their keys here, as signed integers, in which -0.0f (the places outside
    // the unit) is -1: in none of the ranges below.
    auto ordered = [](int v) { return v ^ ((v >> 31) & INT32_MAX); };
    if (bstar == 0) {
        // The lowest bin's usual crowd are the entropies of all-zero tiles, +0.0f, which counting tells from those above
        // and below.
        uint32_t above = 0, zero = 0;
        keys.template each<false>(nblocks, [&](uint32_t, const int4 &q) {
            above += (uint32_t)__popc(four_bits(q, [&](int v) { return v > 0 && v <= hi; }));
            zero += (uint32_t)__popc(four_bits(q, [](int v) { return v == 0; }));
        });
        above = wave_incl_scan(above);
        zero = wave_incl_scan(zero);
        if (lane == 63) { atomicAdd(&L.above_zero, above); atomicAdd(&L.zero, zero); }
        lds_barrier();
        above = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.above_zero);
        zero = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.zero);
        if (rem <= above) { lo = 1; crowd = above; }
        else if (rem <= above + zero) { lo = hi = 0; rem -= above; crowd = zero; }
        else { lo = INT32_MIN; hi = -2; rem -= above + zero; crowd -= above + zero; }
    }
#pragma unroll 1
    while (crowd > kSmallListCap && lo != hi) {              // three times at most: 32 bits, 12 fewer each time
        const uint32_t span = (uint32_t)hi - (uint32_t)lo;
        const int bits = 32 - __builtin_clz(span), shift = bits > 12 ? bits - 12 : 0;
        static_assert(kCrewBins >= 4096, "the parts' counts");
        reinterpret_cast<uint4 *>(hist)[tid] = make_uint4(0, 0, 0, 0);
        lds_barrier();
        keys.template each<false>(nblocks, [&](uint32_t, const int4 &q) {
            const uint32_t from_lo[4] = {(uint32_t)ordered(q.x) - (uint32_t)lo, (uint32_t)ordered(q.y) - (uint32_t)lo,
                                         (uint32_t)ordered(q.z) - (uint32_t)lo, (uint32_t)ordered(q.w) - (uint32_t)lo};
            // (where a crowd shares one entropy all additions meet on one counter, one after the other; tokens that are
            // alike make a crowd of neighbours: one addition for the four)
            if (q.x == q.y && q.y == q.z && q.z == q.w) {
                if (from_lo[0] <= span) atomicAdd(&hist[from_lo[0] >> shift], 4u);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (from_lo[c] <= span) atomicAdd(&hist[from_lo[c] >> shift], 1u);
            }
        });
        lds_barrier();
        block_pick_bin<4096>(hist, rem, L.wave_total, L.chosen);
        lo = (int)((uint32_t)lo + ((uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[0]) << shift));
        rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[1]);
        crowd = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[2]);
        const uint32_t room = (uint32_t)hi - (uint32_t)lo, part = (1u << shift) - 1u;
        hi = (int)((uint32_t)lo + (room < part ? room : part));
    }
    auto is_above = [&](int v) { return ordered(v) > hi && v != INT32_MIN; };
    if (crowd <= kSmallListCap) {
        classify(L.list, kSmallListCap - 1u, is_above, [&](int v) { return ordered(v) >= lo && v != INT32_MIN; },
                 [](const int4 &) { return true; });
        place_listed();
        return;
    }
    // `crowd` tiles of one entropy: taken in index order until `rem` are used up
    uint32_t equal_before = 0;
    keys.template each<false>(upto, [&](uint32_t b, const int4 &q) {
        const uint32_t above = four_bits(q, is_above), same = four_bits(q, [&](int v) { return ordered(v) == lo; });
        put_bits(L.words, b, above);
        put_bits(L.equal, b, same);
        if (b * 256u + 4u * lane < p0) { before += (uint32_t)__popc(above); equal_before += (uint32_t)__popc(same); }
    });
    before = wave_incl_scan(before);
    equal_before = wave_incl_scan(equal_before);
    if (lane == 63) { atomicAdd(&L.before, before); atomicAdd(&L.equal_before, equal_before); }
    lds_barrier();
    if (wave == 0) {
        uint64_t taken = lane < kCrewWaves ? L.equal[lane] : 0ull;
        const uint32_t count = (uint32_t)__popcll(taken);
        const uint32_t ahead = L.equal_before + wave_incl_scan(count) - count;
        if (ahead >= rem) taken = 0;
        else
            for (uint32_t over = ahead + count; over > rem; --over) taken &= ~(1ull << (63 - __builtin_clzll(taken)));
        if (lane < kCrewWaves) L.words[lane] |= taken;
        if (lane == 0) L.before += L.equal_before < rem ? L.equal_before : rem;
    }
    lds_barrier();
}

// The pivot swap P_d on a tile in registers: element d of the tile and element 0, which is the first part's first.  d = 0 changes nothing.
template <int EPL, int LPT>
__device__ __forceinline__ void swap_across(float *x, uint32_t part, uint32_t d)
{
    const bool holds = d / EPL == part;
    const uint32_t mine = holds ? d % EPL : EPL;
    const float x0 = LPT == 1 ? x[0] : __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(
                                           0, (int)__float_as_uint(x[0]), LPT == 2 ? 0xA0 : 0x00, 0xF, 0xF, true));
    uint32_t xd = 0;
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
        const bool it = mine == (uint32_t)e;
        xd = it ? __float_as_uint(x[e]) : xd;
        x[e] = it ? x0 : x[e];
    }
    if constexpr (LPT >= 2) xd |= lane_xor<1>(xd);           // (the other parts have 0)
    if constexpr (LPT >= 4) xd |= lane_xor<2>(xd);
    if (part == 0) x[0] = __uint_as_float(xd);
}

// A workgroup of 1024 threads takes `batch` places of a unit, counted from the 64-tile boundary at or before its first tile.  All of a
// unit's workgroups find its threshold, each for itself as k_select_small does and with the same result, so that nothing passes
// between them; each then knows which of its own places are selected and how many before them, and that is all its tiles' payload
// needs.  A wavefront quantizes its tiles by itself, in registers but for the payload's way to storage order.
//
// What it replaces, k_select_small and k_quant_pack, are two launches of which the first keeps one compute unit per ranking unit
// busy and the others idle.  A launch is 2.5 us of a chain, and Eq. 3, Eq. 4 and the tiles' ranges are done while the unit's
// entropies are counted.  bf16 [1,1024,1600] G = 64 (25600 tiles, 200 workgroups), by the 100 MHz clock: entropies in LDS after 1.3 us,
// counted, and rows transformed, after 4.2, threshold bin 4.9, its tiles listed 6.5 and placed 6.8, payload written 7.7.  Bound by
// what one compute unit issues for 25600 entropies (LDS additions 1.8 us, comparisons 1.0), the same in every one.
// Encode, two launches -> one: that tensor 14.1 -> 11.7 us; fp32 [4,512,2048] with its decode 22.7 -> 21.1; 256 to 8192 tiles of
// 8 to 64 channels 12.4 -> 9.0; [1,1600,2048] G = 128 16.5 -> 14.7; [10,1638,128] G = 8, 256 workgroups, 16.7 -> 16.3.
// (With the entropies in registers and loops unrolled over them: [1,1024,1600] 13.1.  Rows requested before the entropies have
// arrived: the fp32 tensor 22.5, as those wait behind all workgroups' rows.  Two histograms, by the lanes' parity: no faster.)
template <int G, bool BF16, int LOW, int LPT, bool RESIDENT>
__global__ __launch_bounds__(kCrewThreads)
void k_rank_quant(const float *__restrict__ H, const void *__restrict__ in, uint8_t *__restrict__ packed, uint32_t T, uint32_t n,
                  uint32_t k, uint32_t batch, int bin0, float tau, float eps_ratio)
{
    constexpr int ES = BF16 ? 2 : 4;
    using W = Wave<G, ES, LPT>;
    using U = typename Unit<G>::type;
    constexpr int EPL = W::EPL, WORDS = W::LANE_BYTES / 4;
    constexpr uint32_t WIDE = LOW + 1, PLACES = RESIDENT ? kCrewPlaces : 0u;
    constexpr uint32_t ROWS = kCrewWaves * W::LDS_BYTES, RANK = (PLACES + 64u + kCrewBins) * 4;
    // the unit's entropies and their histogram; later the rows, and the payload
    __shared__ __attribute__((aligned(16))) uint8_t lds[ROWS > RANK ? ROWS : RANK];
    __shared__ CrewLds L;
    static_assert(sizeof(lds) + sizeof(L) <= 163840, "the LDS of a compute unit");
    uint32_t *hist = reinterpret_cast<uint32_t *>(lds) + PLACES + 64;
    const int tid = threadIdx.x;
    const uint32_t lane = (uint32_t)tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t u = blockIdx.y, p0 = blockIdx.x * batch;
    const UnitPlaces at(u, n);
    if (p0 >= at.end) return;                    // (units that start off a boundary reach one batch further)
    const uint64_t first = (uint64_t)u * n - at.phase;       // the tile of place 0
    const UnitKeys<RESIDENT> keys(reinterpret_cast<int *>(lds), H + first, at, n);
    // (cleared first: the compiler has LDS accesses wait for what is on its way to LDS)
#pragma unroll
    for (uint32_t i = 0; i < kCrewBins / 4 / kCrewThreads; ++i)
        reinterpret_cast<uint4 *>(hist)[i * kCrewThreads + tid] = make_uint4(0, 0, 0, 0);
    if (tid < kCrewWaves) { L.words[tid] = 0; L.equal[tid] = 0; }
    if (tid == 0) { L.listed = 0; L.above_zero = 0; L.zero = 0; L.before = 0; L.equal_before = 0; }
    if (tid == 0) hist[0] = n;                   // the lowest bin takes whatever the others leave
    if constexpr (RESIDENT) keys.request();
    // my wavefront's places of the batch, [w0, w1), and of those the unit's, [v0, v1)
    const uint32_t w0 = p0 + wave * W::TILES;
    const uint32_t v0 = w0 > at.phase ? w0 : at.phase, w1 = w0 + W::TILES, v1 = w1 < at.end ? w1 : at.end;
    const bool works = wave * W::TILES < batch && v0 < v1;
    const uint32_t place = w0 + lane / LPT, part = lane % LPT;
    const bool valid = place >= v0 && place < v1;
    // (a wavefront without places takes the unit's first tile, so that the loads are under no condition, behind which the compiler would
    // wait for them)
    const uint64_t j = first + (valid ? place : works ? v0 : at.phase);
    if constexpr (RESIDENT) __builtin_amdgcn_s_waitcnt(0x0f70);            // vmcnt(0): my wavefront's entropies are in LDS
    lds_barrier();
    // (requested only now: the entropies would wait behind all workgroups' rows)
    uint32_t w[WORDS];
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(static_cast<const uint8_t *>(in) + (j * LPT + part) * W::LANE_BYTES);
#pragma unroll
        for (int i = 0; i < WORDS / 4; ++i) {
            const uint4 v = src[i];
            w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
        }
    }
    count_places(keys, hist, bin0);
    // Eq. 3 and 4, and the tile's range, which do not depend on its width, before the barrier behind the counts.
    float x[EPL];
    uint32_t pv = 0;
    TileRange range{};
    if (works) {
        pv = pivot_of<EPL, BF16, LPT>(w, part, tau, eps_ratio);
#pragma unroll
        for (int e = 0; e < EPL; ++e)
            x[e] = BF16 ? __uint_as_float(e & 1 ? w[e >> 1] & 0xffff0000u : w[e >> 1] << 16) : __uint_as_float(w[BF16 ? 0 : e]);
        if (__ballot(pv > 0x80u) != 0) swap_across<EPL, LPT>(x, part, pv & (G - 1u));
        if ((pv & 0x80u) != 0) {                 // the lanes of a tile agree
            butterfly<EPL>(x);
            butterfly_across<EPL, LPT>(x, part);
#pragma unroll
            for (int e = 0; e < EPL; ++e) x[e] = x[e] * TileConst<G>::c;
        }
        range = tile_range<EPL, LPT>(x);
    }
    rank_batch(keys, hist, n, k, bin0, p0, batch, L);

    const Sections lay(T);
    // selected places of the batch before each of its words: lane i of the first 16 has word i's
    const uint32_t words_before = before_in_sixteen((uint32_t)__popcll(L.words[lane & 15u]));
    const uint32_t rank0 = u * k + L.before;     // (every earlier unit holds exactly k)
    if (wave == kCrewWaves - 1 && lane < batch / 64) {
        const uint32_t g = p0 / 64 + lane;
        if (g < at.nwords) {
            put_word(reinterpret_cast<uint64_t *>(packed + lay.bitmap) + at.word0 + g, at.mask(g), L.words[lane]);
            if (g != 0 || at.phase == 0) reinterpret_cast<uint32_t *>(packed + lay.ranks)[at.word0 + g] = rank0 + words_before;
        }
    }
    if (!works) return;
    uint8_t *rows = lds + wave * W::LDS_BYTES;
    // width and rank of my tile, and of the wavefront's first
    const uint32_t g = (wave * W::TILES) / 64;
    const uint64_t word = L.words[g];
    const uint32_t before_word = (uint32_t)__builtin_amdgcn_readlane((int)words_before, (int)g);
    auto below = [&](uint32_t p) { return (uint32_t)__popcll(word & ((1ull << (p & 63u)) - 1ull)); };
    const uint32_t tile = valid ? place : v0;
    const uint32_t width = LOW + (uint32_t)((word >> (tile & 63u)) & 1u);
    const uint32_t below0 = below(v0), at_unit = LOW * (tile - v0) + below(tile) - below0;
    U *pay = reinterpret_cast<U *>(rows);
    uint32_t meta16 = 0;
    if (valid) {
        meta16 = quantize_values<EPL, LOW>(x, range, width, reinterpret_cast<typename Unit<EPL>::type *>(pay + at_unit) + part * width);
        if (part == 0) {
            reinterpret_cast<uint16_t *>(packed + lay.scale)[j] = (uint16_t)meta16;
            reinterpret_cast<uint16_t *>(packed + lay.zero)[j] = (uint16_t)(meta16 >> 16);
            packed[lay.pivot + j] = (uint8_t)pv;
        }
    }
    wave_lds_fence();
    const uint64_t upto = (v1 & 63u) != 0 ? word & ((1ull << (v1 & 63u)) - 1ull) : word;
    const uint32_t units = LOW * (v1 - v0) + (uint32_t)__popcll(upto) - below0;
    U *dst = reinterpret_cast<U *>(packed + lay.payload) + ((uint64_t)LOW * (first + v0) + rank0 + before_word + below0);
#pragma unroll
    for (int i = 0; i < ((int)WIDE + LPT - 1) / LPT; ++i) {
        const uint32_t s = (uint32_t)i * 64 + lane;
        if (s < units) dst[s] = pay[s];
    }
}

}  // namespace tahq

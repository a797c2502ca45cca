// Streaming kernels: entropy (Eq. 1-2), transform + quantize + pack (Eq. 3-4, Sec. 3.4),
// decode (Alg. 1 step 5).
//
// Mapping: A LANE OWNS A TILE, or, of a tile of more than 128 bytes or in a tensor of few tiles, one part of two or four.  The
// codec is bound by vector-ALU issue as much as by HBM, so the per-tile work (reductions, butterflies, quantizer
// parameters) crosses lanes in its last one or two levels only, inside a quad.  In the quantizer of bf16 tiles of 32 and 64 channels a
// workgroup stages TILES consecutive tiles through LDS with coalesced 128-bit global accesses, then every lane pulls its tile into
// registers; LDS rows are padded by 16 bytes so that the lane-per-row 128-bit reads are bank-conflict free.  In the other quantizer,
// the entropy kernels and the decoder every wavefront works by itself on LDS of its own.
#pragma once
#include "tahq_common.hpp"

namespace tahq {

// Lanes per tile.  `usual`: as many as keep a lane at 128 bytes of the tensor or less.  `few`: for tensors of so few tiles that the
// usual lanes do not make a wavefront for every vector unit of the chip; what counts then is how long one lane takes, so a
// tile gets up to four lanes of at least 8 elements.
template <int G, int ESIZE>
struct Lanes {
    static constexpr int usual = G * ESIZE > 128 ? G * ESIZE / 128 : 1;
    static constexpr int few = G >= 32 ? 4 : G / 8;
    static_assert(usual <= few && few <= 4, "quads");
};

// Geometry of one workgroup's batch of tiles for an element type of ESIZE bytes: as many as 256 threads hold at the usual number of
// lanes per tile.
template <int G, int ESIZE>
struct Batch {
    static constexpr int BYTES = G * ESIZE;                                   // one tile
    static constexpr int TILES = 256 / Lanes<G, ESIZE>::usual;                // tiles per workgroup
    static constexpr int STRIDE = BYTES + 16;                                 // padded LDS row
    static constexpr int CHUNKS = BYTES / 16;                                 // 16-byte chunks per tile
    static constexpr int LDS_BYTES = TILES * STRIDE;
};

// A batch's tiles travel global -> registers -> padded LDS rows, in two steps, so that the loads of the
// next batch can be in flight while the current one is being processed.  Thread t moves the 16-byte
// chunks t, t + THREADS, t + 2 THREADS, ... of the batch (coalesced); TILES threads, or more.  FULL: all TILES tiles exist, no
// per-thread conditions (so that the compiler can count outstanding memory operations exactly).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// 16-byte global load; STREAM marks data that will not be read again soon (non-temporal hint).
template <bool STREAM>
__device__ __forceinline__ uint4 load16(const uint8_t *p)
{
    if constexpr (STREAM) {
        const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
        return make_uint4(t.x, t.y, t.z, t.w);
    } else {
        return *reinterpret_cast<const uint4 *>(p);
    }
}

template <class B, bool FULL, bool STREAM = false, int N>
__device__ __forceinline__ void load_batch(const void *__restrict__ in, uint64_t j0, uint32_t nvalid, uint4 (&v)[N],
                                           int tid = (int)threadIdx.x)
{
    constexpr int THREADS = B::TILES * B::CHUNKS / N;        // N chunks per thread
    const uint8_t *src = static_cast<const uint8_t *>(in) + j0 * B::BYTES;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t q = (uint32_t)i * THREADS + tid;
        if constexpr (FULL) {
            v[i] = load16<STREAM>(src + (uint64_t)q * 16);
        } else {
            v[i] = make_uint4(0u, 0u, 0u, 0u);
            if (q / B::CHUNKS < nvalid) v[i] = load16<STREAM>(src + (uint64_t)q * 16);
        }
    }
}

template <class B, bool FULL, int N>
__device__ __forceinline__ void store_batch(const uint4 (&v)[N], uint32_t nvalid, uint8_t *lds, int tid = (int)threadIdx.x)
{
    constexpr int THREADS = B::TILES * B::CHUNKS / N;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t q = (uint32_t)i * THREADS + tid;
        const uint32_t tile = q / B::CHUNKS, sub = q % B::CHUNKS;
        if (FULL || tile < nvalid) *reinterpret_cast<uint4 *>(lds + tile * B::STRIDE + sub * 16) = v[i];
    }
}

// Coalesced copy of `nvalid` tiles from padded LDS rows to global memory.
template <int G, int ESIZE, bool FULL>
__device__ __forceinline__ void stage_out(void *__restrict__ out, uint64_t j0, uint32_t nvalid, const uint8_t *lds)
{
    using B = Batch<G, ESIZE>;
    uint8_t *dst = static_cast<uint8_t *>(out) + j0 * B::BYTES;
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < B::CHUNKS; ++i) {
        const uint32_t q = (uint32_t)i * B::TILES + tid;
        const uint32_t tile = q / B::CHUNKS, sub = q % B::CHUNKS;
        if (FULL || tile < nvalid) {
            // streaming store: the decoded tensor is not read again by this library
            const uint4 val = *reinterpret_cast<const uint4 *>(lds + tile * B::STRIDE + sub * 16);
            const u32x4 vv = {val.x, val.y, val.z, val.w};
            __builtin_nontemporal_store(vv, reinterpret_cast<u32x4 *>(dst + (uint64_t)q * 16));
        }
    }
}

// My tile, from its LDS row into registers, widened to fp32.
template <int G, bool BF16>
__device__ __forceinline__ void read_tile(const uint8_t *row, float *x)
{
    if constexpr (BF16) {
#pragma unroll
        for (int c = 0; c < G / 8; ++c) {
            const uint4 w = *reinterpret_cast<const uint4 *>(row + c * 16);
            const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[8 * c + 2 * i] = __uint_as_float(ws[i] << 16);
                x[8 * c + 2 * i + 1] = __uint_as_float(ws[i] & 0xffff0000u);
            }
        }
    } else {
#pragma unroll
        for (int c = 0; c < G / 4; ++c) {
            const float4 w = *reinterpret_cast<const float4 *>(row + c * 16);
            x[4 * c] = w.x; x[4 * c + 1] = w.y; x[4 * c + 2] = w.z; x[4 * c + 3] = w.w;
        }
    }
}

// Adjacent-pair binary tree over N = 2^m values held in registers: the level-by-level pairing
// z'[k] = z[2k] + z[2k+1] is the same expression tree as "left half + right half", recursively.
template <int N>
__device__ __forceinline__ float tree_sum(const float *z)
{
    if constexpr (N == 1) return z[0];
    else return tree_sum<N / 2>(z) + tree_sum<N / 2>(z + N / 2);
}

// Unnormalised Sylvester butterfly on a whole tile in registers, stages h = 1, 2, ..., G/2.
template <int G>
__device__ __forceinline__ void butterfly(float *x)
{
#pragma unroll
    for (int h = 1; h < G; h <<= 1) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if ((i & h) == 0) {
                const float p = x[i], q = x[i + h];
                x[i] = p + q;
                x[i + h] = p - q;
            }
        }
    }
}

// How tiles spread over lanes in the entropy kernel, the quantizer and the decoder: LPT lanes per tile, EPL consecutive
// elements per lane, at most 128 bytes of the tensor; TILES tiles per wavefront.
template <int G, int ESIZE, int LPT>
struct Wave {
    static constexpr int EPL = G / LPT;                                       // elements per lane
    static constexpr int TILES = 64 / LPT;                                    // tiles per wavefront
    static constexpr int LANE_BYTES = EPL * ESIZE;
    static constexpr int CHUNKS = LANE_BYTES / 16;                            // 16-byte chunks per lane
    static constexpr int LDS_BYTES = 64 * LANE_BYTES;
    static_assert(TILES * LPT == 64 && CHUNKS >= 1 && CHUNKS <= 8, "whole tiles, whole chunks");
    // Lane r's chunks lie in LDS at slots r * CHUNKS + (c ^ swizzle(r)): eight lanes that read the same chunk of their
    // rows, like eight that read consecutive chunks of one row, meet eight different 16-byte columns of the banks.
    static __device__ __forceinline__ uint32_t swizzle(uint32_t r)
    {
        return CHUNKS == 8 ? (r & 7u) : CHUNKS == 4 ? ((r >> 1) & 3u) : CHUNKS == 2 ? ((r >> 2) & 1u) : 0u;
    }
    // byte offset of element e of the tile that starts at lane `row0`
    static __device__ __forceinline__ uint32_t element_at(uint32_t row0, uint32_t e)
    {
        const uint32_t r = row0 + e / EPL, byte = (e % EPL) * ESIZE;
        return r * LANE_BYTES + (((byte >> 4) ^ swizzle(r)) << 4) + (byte & 15u);
    }
};

// The value of lane (mine ^ X), X = 1 or 2.
template <int X>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    static_assert(X == 1 || X == 2, "inside a quad");
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, X == 1 ? 0xB1 : 0x4E, 0xF, 0xF, true);
}
template <int X>
__device__ __forceinline__ float lane_xor(float v)
{
    return __uint_as_float(lane_xor<X>(__float_as_uint(v)));
}

// The butterfly stages that cross lanes: element i of lane part p meets element i of part p ^ (h / EPL).
template <int EPL, int LPT>
__device__ __forceinline__ void butterfly_across(float *x, uint32_t part)
{
    if constexpr (LPT >= 2) {
        const float s1 = (part & 1u) ? -1.0f : 1.0f;
#pragma unroll
        for (int i = 0; i < EPL; ++i) x[i] = __builtin_fmaf(x[i], s1, lane_xor<1>(x[i]));     // p + q, or p - q: one rounding
    }
    if constexpr (LPT >= 4) {
        const float s2 = (part & 2u) ? -1.0f : 1.0f;
#pragma unroll
        for (int i = 0; i < EPL; ++i) x[i] = __builtin_fmaf(x[i], s2, lane_xor<2>(x[i]));
    }
    static_assert(LPT <= 4, "two stages across lanes");
}

// Orders the LDS accesses of one wavefront for the compiler; the hardware performs them in program order.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------- outlier test

// Median of three unsigned integers in one vector instruction.
__device__ __forceinline__ uint32_t umed3(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Eq. 3 on a tile of LPT parts, of which I have the part-th, G elements: the magnitudes of the largest and the second-largest element
// (with multiplicity) and the lowest index of the largest.  Elements come in index order, by pairs, then `finish`.
template <int G, bool BF16, int LPT> struct Top2;

// A bf16 magnitude has 16 free low bits: key = |bits| << 16 | (G-1-k) orders by magnitude, then by
// lower index, under unsigned integer max.  Even and odd elements run in separate chains.
template <int G, int LPT>
struct Top2<G, true, LPT> {
    // (the even chain's keys are shifted left by one, which drops the sign bit for free, and hold (G - 2 - k) / 2 for the index: the
    // constants of both chains fit the instructions)
    uint32_t e1 = 0, e2 = 0, o1 = 0, o2 = 0;
    // the pair of elements k, k + 1 as it lies in memory
    __device__ __forceinline__ void add(uint32_t k, uint32_t pair)
    {
        add_even((pair << 17) | (G - 2 - k));
        add_odd((pair & 0x7fff0000u) | (G - 2 - k));
    }
    __device__ __forceinline__ void finish(uint32_t part, float *a1_out, float *a2_out, uint32_t *d_out)
    {
        e1 = ((e1 >> 1) & 0x7fff0000u) | ((e1 & 0xffffu) + 1u);      // G - 1 - k
        e2 = ((e2 >> 1) & 0x7fff0000u) | ((e2 & 0xffffu) + 1u);
        uint32_t k1 = e1 > o1 ? e1 : o1;
        const uint32_t lo = e1 > o1 ? o1 : e1;
        const uint32_t hi2 = e2 > o2 ? e2 : o2;
        uint32_t k2 = lo > hi2 ? lo : hi2;
        // the other parts of the tile: two pairs become one
        auto merge = [&](uint32_t p1, uint32_t p2) {
            const uint32_t less = k1 < p1 ? k1 : p1, more2 = k2 > p2 ? k2 : p2;
            k1 = k1 > p1 ? k1 : p1;
            k2 = less > more2 ? less : more2;
        };
        if constexpr (LPT >= 2) {
            k1 += (LPT - 1 - part) * G;          // the low bits count indices of the whole tile from its end
            merge(lane_xor<1>(k1), lane_xor<1>(k2));
        }
        if constexpr (LPT >= 4) merge(lane_xor<2>(k1), lane_xor<2>(k2));
        *a1_out = __uint_as_float(k1 & 0x7fff0000u);
        *a2_out = __uint_as_float(k2 & 0x7fff0000u);
        *d_out = (LPT * G - 1) - (k1 & 0x7fu);
    }
private:
    __device__ __forceinline__ void add_even(uint32_t key)
    {
        e2 = umed3(e1, e2, key);                 // second largest of {e1 >= e2, key}
        e1 = e1 > key ? e1 : key;
    }
    __device__ __forceinline__ void add_odd(uint32_t key)
    {
        o2 = umed3(o1, o2, key);
        o1 = o1 > key ? o1 : key;
    }
};

// (fp32 magnitudes leave no room for the index: the two largest first, and where that makes an outlier tile in the wavefront, a second
// look at the elements for the lowest index.  2 or 4 vector slots per element; carrying the index along took 5.5.)
template <int G, int LPT>
struct Top2<G, false, LPT> {
    float a1 = -1.0f, a2 = -1.0f;                // magnitudes are >= 0: the first element always replaces a1
    __device__ __forceinline__ void add(float x)
    {
        // (a signalling NaN made quiet: the median would make a NaN of a2 from it.  The maximum asks for the same instruction.)
        const float a = __builtin_canonicalizef(__builtin_fabsf(x));
        a2 = __builtin_amdgcn_fmed3f(a1, a2, a); // second largest of {a1 >= a2, a}; a NaN counts as the smallest
        a1 = __builtin_fmaxf(a1, a);
    }
    // of the whole tile
    __device__ __forceinline__ void merge()
    {
        auto with = [&](float p1, float p2) {
            a2 = __builtin_fmaxf(__builtin_fminf(a1, p1), __builtin_fmaxf(a2, p2));
            a1 = __builtin_fmaxf(a1, p1);
        };
        if constexpr (LPT >= 2) with(lane_xor<1>(a1), lane_xor<1>(a2));
        if constexpr (LPT >= 4) with(lane_xor<2>(a1), lane_xor<2>(a2));
        a2 = __builtin_fmaxf(a2, 0.0f);
    }
    // the lowest index of an element of magnitude a1, 0 in a tile of NaN only; element(k): the k-th of mine
    template <class Element>
    __device__ __forceinline__ uint32_t index(uint32_t part, Element element) const
    {
        uint32_t d = 0x7fu;
#pragma unroll
        for (int k = G; k-- > 0;) d = __builtin_fabsf(element(k)) == a1 ? part * G + k : d;
        if constexpr (LPT >= 2) { const uint32_t p = lane_xor<1>(d); d = p < d ? p : d; }
        if constexpr (LPT >= 4) { const uint32_t p = lane_xor<2>(d); d = p < d ? p : d; }
        return a1 < 0.0f ? 0u : d;               // (no element has replaced a1, and none equals it)
    }
};

// Outlier flag and pivot index of the tile: the pivot byte (bit 7 = flag, bits 0..6 = d), from the dwords of my part.
template <int EPL, bool BF16, int LPT>
__device__ __forceinline__ uint32_t pivot_of(const uint32_t *w, uint32_t part, float tau, float eps_ratio)
{
    Top2<EPL, BF16, LPT> t;
    if constexpr (BF16) {
#pragma unroll
        for (int k = 0; k < EPL; k += 2) t.add(k, w[k / 2]);
        float a1, a2;
        uint32_t d;
        t.finish(part, &a1, &a2, &d);
        return a1 > tau * (a2 + eps_ratio) ? (0x80u | d) : 0u;
    } else {
#pragma unroll
        for (int k = 0; k < EPL; ++k) t.add(__uint_as_float(w[k]));
        t.merge();
        const bool flag = t.a1 > tau * (t.a2 + eps_ratio);
        if (__ballot(flag) == 0) return 0u;
        const uint32_t d = t.index(part, [&](int k) { return __uint_as_float(w[k]); });
        return flag ? (0x80u | d) : 0u;
    }
}

// ... of a bf16 tile that one lane has, in its LDS row
template <int G>
__device__ __forceinline__ uint32_t pivot_of_row(const uint8_t *row, float tau, float eps_ratio)
{
    uint32_t w[G / 2];
#pragma unroll
    for (int c = 0; c < G / 8; ++c) {
        const uint4 q = *reinterpret_cast<const uint4 *>(row + c * 16);
        w[4 * c] = q.x; w[4 * c + 1] = q.y; w[4 * c + 2] = q.z; w[4 * c + 3] = q.w;
    }
    return pivot_of<G, true, 1>(w, 0, tau, eps_ratio);
}

// The pivot swap P_d on a bf16 tile's LDS row.
__device__ __forceinline__ void swap_pivot(uint8_t *row, uint32_t d)
{
    uint16_t *r16 = reinterpret_cast<uint16_t *>(row);
    const uint16_t v0 = r16[0], vd = r16[d];
    r16[0] = vd; r16[d] = v0;
}

// ------------------------------------------------------------- prologue

// What a stream holds besides the kernels' results: header and zeroed section padding.  And the bit map words that ranking
// units share with a neighbour or with the end of the map, cleared because the selection adds to them.
struct HeaderWords { uint32_t w[16]; };
struct PadList { uint64_t begin[5]; uint32_t len[5]; };
struct Prologue {
    uint8_t *packed;                             // header and padding go here; null: none of them
    uint64_t *bitmap;
    uint32_t edge_units, unit_tiles;             // edge_units != 0: clear the shared words of that many units
    HeaderWords hdr;
    PadList pads;
};

// Thread `gid` of `threads` (at least 64): as many as there are edge units, in whole workgroups (prologue_blocks), so that the others
// need not read these arguments.  The small launches of a call cost more than what they do, so the prologue rides
// along with the call's first kernel, at its end, where nothing waits for it: instead of a launch in front of the entropies
// (encode of 1024 x 1600 channels: 18.8 -> 17.5 us), or of the quantizer where all tiles have one width (fp32 [1,128,512],
// encode and decode: 19.7 -> 16.8).
inline uint32_t prologue_blocks(const Prologue &p, uint32_t threads, uint32_t blocks)
{
    const uint32_t want = (p.edge_units + threads - 1) / threads;
    return want < 1u ? 1u : want < blocks ? want : blocks;
}

__device__ __forceinline__ void write_prologue(const Prologue &p, uint32_t gid, uint32_t threads)
{
    if (p.packed != nullptr && gid < 64) {
        if (gid < 16) reinterpret_cast<uint32_t *>(p.packed)[gid] = p.hdr.w[gid];
#pragma unroll
        for (int s = 0; s < 5; ++s)
            if (gid < p.pads.len[s]) p.packed[p.pads.begin[s] + gid] = 0;            // paddings are shorter than 64 bytes
    }
    for (uint32_t i = gid; i < p.edge_units; i += threads) {
        const uint64_t j = (uint64_t)(i + 1) * p.unit_tiles;   // the first tile after unit i
        if ((j & 63u) != 0) p.bitmap[j >> 6] = 0;
    }
}

// A budget of exactly `lo` or `lo + 1` bits: every tile has the same width.  Bit map word `w`.
__device__ __forceinline__ uint64_t constant_word(uint64_t w, uint32_t T, bool all_wide)
{
    const uint64_t left = (uint64_t)T - w * 64;
    return !all_wide ? 0ull : left >= 64 ? ~0ull : ((1ull << left) - 1ull);
}

// ... and its rank-table entry, both written.
__device__ __forceinline__ void constant_width_word(uint64_t w, uint32_t T, int all_wide, uint64_t *__restrict__ bitmap,
                                                    uint32_t *__restrict__ ranks)
{
    bitmap[w] = constant_word(w, T, all_wide != 0);
    ranks[w] = all_wide ? (uint32_t)(w * 64) : 0u;
}

// -------------------------------------------------------------- K0: entropy

// Wavefronts that read the tensor for its entropies take their rows straight from memory to their own piece of LDS, without
// registers or barriers in between, and request the next ones as soon as the present ones are in registers: what a wavefront
// computes hides its own loads.  Lane r's 128 bytes or less lie as `Wave` says; as consecutive lanes fill consecutive 16 bytes of
// LDS, the swizzle is in the addresses they load from.
//   src: row 0; rows: how many exist (lanes past them load the last one); NG groups of 64 rows
template <class W, int NG, bool MOSTLY_FULL>
__device__ __forceinline__ void request_rows(const uint8_t *__restrict__ src, uint32_t rows, uint8_t *lds, uint32_t lane)
{
    constexpr uint32_t STEP = 64 / W::CHUNKS;                // rows per load: a multiple of the swizzle's period
    const uint32_t r = lane / W::CHUNKS, c = (lane % W::CHUNKS) ^ W::swizzle(r);
    // (2: non-temporal.  The tensor is much larger than any cache, and keeping part of it for the second pass was slower.)
    auto load = [&](const uint8_t *from, uint32_t i) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from,
                                         (__attribute__((address_space(3))) void *)(lds + i * 1024u), 16, 0, 2);
    };
    // (mostly whole groups: without the rows' comparisons on the way to the loads)
    if (MOSTLY_FULL && rows >= 64u * NG) {
        const uint32_t at = r * W::LANE_BYTES + c * 16u;
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)(NG * W::CHUNKS); ++i) load(src + i * 1024u + at, i);
    } else {
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)(NG * W::CHUNKS); ++i) {
            const uint32_t row = r + i * STEP;
            load(src + ((row < rows ? row : rows - 1) * W::LANE_BYTES + c * 16u), i);
        }
    }
}
// ... have arrived
__device__ __forceinline__ void wait_for_rows() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// ... are in registers: their LDS may be written again
__device__ __forceinline__ void rows_are_read()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// A result that a later kernel reads, written through to memory at once.  Left in the L2 until it is evicted or the kernel ends, the
// entropies cost a pass over 512 MB 8 us, so 4.
template <class V>
__device__ __forceinline__ void store_through(V *p, V v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// LDS accesses beside rows that are on their way.  The compiler cannot tell them from the loads' destination and would have each
// of them wait until the rows have arrived; it does not see these.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}
__device__ __forceinline__ void lds_add_one(uint32_t at) { asm volatile("ds_add_u32 %0, %1" ::"v"(at), "v"(1u) : "memory"); }
__device__ __forceinline__ void lds_store(uint32_t at, float v) { asm volatile("ds_write_b32 %0, %1" ::"v"(at), "v"(v) : "memory"); }
__device__ __forceinline__ float lds_load(uint32_t at)
{
    float v;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v) : "v"(at) : "memory");
    return v;
}
// sixteen consecutive values, 16-byte aligned
__device__ __forceinline__ void lds_load(uint32_t at, f32x4 (&v)[4])
{
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:16\n\tds_read_b128 %2, %4 offset:32\n\t"
                 "ds_read_b128 %3, %4 offset:48\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(at) : "memory");
}
// Barrier of the workgroup for accesses to LDS only: the next rows stay on their way.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// My row of group `g`, as it is in memory, and its k-th element, widened to fp32.  Tiles stay packed in registers, and every pass
// over them widens them anew: three quarters of a vector slot per element against 32 registers.
template <class W, bool BF16>
struct Row {
    static constexpr int WORDS = W::LANE_BYTES / 4;
    uint32_t w[WORDS];
    __device__ __forceinline__ void read(const uint8_t *lds, uint32_t g, uint32_t lane)
    {
        const uint8_t *row = lds + g * W::LDS_BYTES + lane * W::LANE_BYTES;
        const uint32_t swz = W::swizzle(lane) << 4;
#pragma unroll
        for (uint32_t c = 0; c < (uint32_t)W::CHUNKS; ++c) {
            const uint4 q = *reinterpret_cast<const uint4 *>(row + ((c << 4) ^ swz));
            w[4 * c] = q.x; w[4 * c + 1] = q.y; w[4 * c + 2] = q.z; w[4 * c + 3] = q.w;
        }
    }
    __device__ __forceinline__ float operator[](int k) const
    {
        if constexpr (BF16) return __uint_as_float(k & 1 ? w[k >> 1] & 0xffff0000u : w[k >> 1] << 16);
        else return __uint_as_float(w[k]);
    }
    // Nothing derived from the words is kept across this point.
    __device__ __forceinline__ void forget()
    {
        if constexpr (BF16) {
#pragma unroll
            for (int i = 0; i < WORDS; ++i) asm volatile("" : "+v"(w[i]));
        }
    }
};

// A tile's row, or my part of it, from the tensor.
template <class W, bool BF16>
struct TensorRow : Row<W, BF16> {
    __device__ __forceinline__ explicit TensorRow(const uint8_t *p)
    {
#pragma unroll
        for (int c = 0; c < W::CHUNKS; ++c) {
            const uint4 q = reinterpret_cast<const uint4 *>(p)[c];
            this->w[4 * c] = q.x; this->w[4 * c + 1] = q.y; this->w[4 * c + 2] = q.z; this->w[4 * c + 3] = q.w;
        }
    }
};

// The sum over a tile from its LPT parts' sums, which meet in pairs: the top of the tile's binary tree.
template <int LPT>
__device__ __forceinline__ float whole_tile(float part)
{
    if constexpr (LPT >= 2) part = part + lane_xor<1>(part);
    if constexpr (LPT >= 4) part = part + lane_xor<2>(part);
    return part;
}

// Sum over my elements of |v| (Eq. 1), and of |v| log(|v| r + varsigma) (Eq. 2 but for its common factor r = 1 / (L1 + eps)).
template <int N, class R>
__device__ __forceinline__ float magnitude_sum(const R &x)
{
    float a[N];
#pragma unroll
    for (int k = 0; k < N; ++k) a[k] = __builtin_fabsf(x[k]);
    return tree_sum<N>(a);
}
template <int N, class R>
__device__ __forceinline__ float weighted_sum(const R &x, float invL, float eps_log)
{
    float a[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        a[k] = __builtin_fabsf(x[k]);
        a[k] = a[k] * log_contract(__builtin_fmaf(a[k], invL, eps_log));
    }
    return tree_sum<N>(a);
}

// Eq. 1-2 for a tile of LPT parts, of which `x` holds mine.
template <int EPL, int LPT, class R>
__device__ __forceinline__ float entropy_of(R &x, float eps_l1, float eps_log)
{
    const float invL = 1.0f / (whole_tile<LPT>(magnitude_sum<EPL>(x)) + eps_l1);
    x.forget();
    return 0.0f - invL * whole_tile<LPT>(weighted_sum<EPL>(x, invL, eps_log));
}

// The same to within kEntropySlack, with the hardware's logarithm, two vector slots instead of nine, and in one pass:
//     H ~ 0 - ln2 (r S + r L1 log2 r),  S = sum of |v| log2 (|v| + 2^-126)
// (what is added keeps a zero's logarithm finite, and is lost in the rounding beside anything that counts).
// How far it is from the sum above, for norms in the range below; r is what either side computed, p = |v| r, u = 2^-24.
//   - The terms here.  In bits, p |log2 |v|| adds up to at most 31, as |log2 L1| <= 24 and p's own entropy is at most 7, and r L1
//     |log2 r| to 24.6 (24 and, for an eps beside which the norm vanishes, x |log2 x| of their ratio x).  Each of the two
//     passes 11 additions, two products and the hardware's logarithm: v_log_f32 is within 2 u of its result, relatively, for
//     every float from 2^-25 to 2^25 (all of them compared with the double logarithm).  Then a sum and two steps by ln2, of at most 7.
//   - r: sums of 11 and 7 levels, the addition of eps and the division, 22 u between the two.  The sum over p log p moves by
//     that times at most ln 128 - 1.
//   - LOG's distance from the logarithm, 1.11e-5 at most over [1e-12, 2), passed on by weights p that add up to 1.
//   - varsigma inside the logarithm, at most 128 times itself (the caller takes this way for varsigma up to 2^-24 only).
//   - The roundings of the sum above: LOG's argument, a product, 7 additions and the factor r, of at most ln 128.
// (Seen: 2.2e-5.)  A tile whose norm is neither zero nor in the range takes the other way, with its wavefront.
constexpr float kApproxLogMax = 0x1p-24f, kApproxLogMin = 1e-12f, kApproxNormMin = 0x1p-24f, kApproxNormMax = 0x1p24f;
constexpr double kApproxError = 0x1p-24 * ((15 * 31 + 15 * 24.6 + 3 * 7) * 0.69315 + 22 * 3.86 + 10 * 4.86) + 1.11e-5 +
                                128.0 * kApproxLogMax;
constexpr float kEntropySlack = 7e-5f;           // (more by far than the rounding of a bin's edge that it is added to twice)
static_assert(kApproxError + 1e-6 < kEntropySlack, "the selection's candidates rest on it");
// k_select_classify looks for candidates no further than the two bins beside the threshold's: the narrowest are ln 8 / kLinBins wide.
static_assert(2.0f * kEntropySlack * kLinBins < 2.07f, "the margin is narrower than a bin");

// `exact` is that other way: it reads the row again, so that nothing has to wait for it in registers.
template <int EPL, int LPT, class R, class Exact>
__device__ __forceinline__ float entropy_approx(const R &x, float eps_l1, Exact exact)
{
    float L1 = 0.0f, S = 0.0f;
    // (eight elements at a time: left to itself the compiler works on all of them at once and runs out of registers)
#pragma unroll
    for (int k0 = 0; k0 < EPL; k0 += 8) {
        float a[8], b[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            a[k] = __builtin_fabsf(x[k0 + k]);
            b[k] = a[k] * __builtin_amdgcn_logf(a[k] + 0x1p-126f);
        }
        L1 = L1 + tree_sum<8>(a);
        S = S + tree_sum<8>(b);
        asm volatile("" : "+v"(L1), "+v"(S));
    }
    L1 = whole_tile<LPT>(L1);
    S = whole_tile<LPT>(S);
    const float r = 1.0f / (L1 + eps_l1);
    // (a difference from +0.0f, as above: never -0.0f, which the selection takes for a place outside the ranking unit.  A single
    // element of magnitude 1 makes both products +0.0f.)
    float h = 0.0f - kLn2 * (r * S + (r * L1) * __builtin_amdgcn_logf(r));
    if (L1 == 0.0f) h = 0.0f;
    if (__ballot(!(L1 == 0.0f || (L1 > kApproxNormMin && L1 < kApproxNormMax))) != 0) h = exact();
    return h;
}

// The entropy of a tile with NaN among its elements: that with the largest payload, made quiet, with the sign turned over.  Which
// payload came through the sums above would be the choice of whoever ordered the instructions' operands, and differ between the
// kernels that compute the same entropies.  (With one kind of NaN in the tile this is what the sums give.)
template <class W, bool BF16, int LPT>
__device__ __forceinline__ float nan_entropy(const Row<W, BF16> &x, float h)
{
    uint32_t most = 0;
#pragma unroll
    for (int i = 0; i < Row<W, BF16>::WORDS; ++i) {
        const uint32_t a = BF16 ? (x.w[i] << 16) & 0x7fff0000u : 0u, b = x.w[i] & (BF16 ? 0x7fff0000u : 0x7fffffffu);
        most = most > a ? most : a;
        most = most > b ? most : b;
    }
    if constexpr (LPT >= 2) { const uint32_t p = lane_xor<1>(most); most = most > p ? most : p; }
    if constexpr (LPT >= 4) { const uint32_t p = lane_xor<2>(most); most = most > p ? most : p; }
    return h != h && most > 0x7f800000u ? __uint_as_float(most | 0x80400000u) : h;
}

constexpr int kDigit0Bits = 10;                  // first radix digit of the selection: key bits 31..22
static_assert((1u << kDigit0Bits) == kDigit0Bins, "digit 0 width");

// Groups of 64 rows that a wavefront takes at a time in tensors of many tiles: 128 bytes per lane whatever the tile.
template <int G, int ESIZE, int LPT>
constexpr int kRowGroups = 128 / (G * ESIZE / LPT);

// A lane usually holds a whole bf16 tile, in which Eq. 3 is two vector slots per element.  Where it does, the entropy kernels can decide
// Eq. 3, into the stream's pivot bytes, which takes a barrier out of the quantizer.  With exact entropies both passes are bound by
// vector issue, and this is what tells them apart: encode of bf16 with Eq. 3 in the entropies, and in the quantizer: [64,64,8192]
// G = 16 54.5 us and 56.8, G = 32 42.3 and 43.4, [16,1024,1600] G = 64 38.3 and 39.0; of tiles that lanes share: [16,512,8192]
// G = 128 73.0 and 68.9, [8,1024,4096] 48.6 and 47.4; and of fp32, where it is three or four slots: [8,2048,4096] G = 64 116.5 and 115.5,
// [6,3000,2048] G = 16 79.9 and 78.3.
template <int G, bool BF16> constexpr bool kWholeTiles = BF16 && Lanes<G, 2>::usual == 1;

// With exact entropies bound by vector issue (twelve and a half slots per element, ten of them the logarithm) and behind it by HBM.
// Without barriers, and with the next rows on their way to LDS while the present ones are in registers, bf16 [8,4096,8192]
// G = 64 108.7 -> 106.1 us, fp32 [4,512,2048] 5.1 -> 4.6.  With approximate ones bound by HBM: 88.8 us against 82 for the loads alone, and
// 98.7 with Eq. 3 and the histogram, where exact entropies and both take 115.
//
// Persistent workgroups of four wavefronts; a step is 4 NG groups of rows, NG for each wavefront, and workgroup w handles a
// contiguous run of steps.  A step's results are stored one step late, just before the next loads, so that no wait for loads ever
// has a younger store in front of it.  The wavefronts of a workgroup meet only where the histogram moves to another unit.
//
// APPROX: entropies to within kEntropySlack, for a selection that makes up for it.
// PIVOTS (below): Eq. 3 is decided here as well, if `pivot` is given: of whole tiles, and with approximate entropies of all, since
// this kernel has vector slots to spare behind HBM then, and k_quant_pack has not.
//
// If HIST, the kernel also builds the first histogram of the selection (Sec. 3.2, top-p%): per
// ranking unit of `unit_tiles` tiles, counts of the keys' top 10 bits (bin_scale == 0) or of the entropies'
// linear bins (bin_scale > 0), `hist_stride` bins per unit, accumulated in LDS and flushed with global atomics
// when the workgroup moves to another unit, in the middle of a step if need be, and at its end.  A step may touch two
// units, not more: `unit_tiles` is at least a step's tiles (the caller checks; otherwise it passes no histogram).
template <int G, bool BF16, int LPT, int NG, bool HIST, bool APPROX>
__global__ __launch_bounds__(256, 4)
void k_entropy(const void *__restrict__ in, float *__restrict__ H, uint8_t *__restrict__ pivot, uint32_t T, uint32_t per,
               float eps_l1, float eps_log, float tau, float eps_ratio, uint32_t pro_blocks, uint32_t *__restrict__ hist0,
               uint32_t unit_tiles, uint32_t hist_stride, float bin_scale, Prologue pro)
{
    using W = Wave<G, BF16 ? 2 : 4, LPT>;
    constexpr bool PIVOTS = APPROX || (kWholeTiles<G, BF16> && LPT == 1);
    constexpr uint32_t WAVE_TILES = W::TILES * NG, STEP_TILES = 4 * WAVE_TILES;
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[4 * NG * W::LDS_BYTES];
    static_assert(kLinBins >= kDigit0Bins, "one LDS histogram serves both kinds of bins");
    __shared__ uint32_t lh[HIST ? kLinBins : 1];
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    uint8_t *lds = lds_all + wave * (NG * W::LDS_BYTES);
    const uint32_t part = lane % LPT, mine = wave * WAVE_TILES + lane / LPT;          // my tile of the step's first group
    const uint32_t steps = (T + STEP_TILES - 1) / STEP_TILES;
    const uint32_t first = blockIdx.x * per;
    const uint32_t last = first + per < steps ? first + per : steps;      // my steps: [first, last)

    auto request = [&](uint32_t step) {
        const uint64_t j0 = (uint64_t)step * STEP_TILES + wave * WAVE_TILES;
        if (j0 >= T) return;                     // (the last step's last wavefronts)
        const uint64_t left = T - j0;
        request_rows<W, NG, true>(static_cast<const uint8_t *>(in) + j0 * (G * (BF16 ? 2 : 4)),
                            left < WAVE_TILES ? (uint32_t)left * LPT : 64u * NG, lds, lane);
    };
    if (first < last) request(first);
    if constexpr (HIST) {
        for (uint32_t i = tid; i < hist_stride; i += 256) lh[i] = 0;
        lds_barrier();
    }
    auto flush = [&](uint32_t unit) {
        lds_barrier();
        for (uint32_t i = tid; i < hist_stride; i += 256) {
            const uint32_t c = lh[i];
            if (c) { atomicAdd(&hist0[(uint64_t)unit * hist_stride + i], c); lh[i] = 0; }
        }
        __syncthreads();
    };
    float h[NG];
    uint32_t pv[NG] = {};
    uint64_t j_prev = 0;                         // the step before, and its tiles
    uint32_t n_prev = 0;
    auto store = [&]() {
#pragma unroll
        for (uint32_t g = 0; g < (uint32_t)NG; ++g) {
            if (part == 0 && mine + g * W::TILES < n_prev) {
                store_through(H + j_prev + (mine + g * W::TILES), h[g]);
                if constexpr (PIVOTS) {
                    if (pivot) store_through(pivot + j_prev + (mine + g * W::TILES), (uint8_t)pv[g]);
                }
            }
        }
    };
    const uint32_t lh_at = lds_address(lh);
    uint32_t cur_unit = HIST && first < last ? (uint32_t)((uint64_t)first * STEP_TILES / unit_tiles) : 0u;
    uint64_t unit_end = (uint64_t)(cur_unit + 1) * unit_tiles;            // the first tile after it
    auto bin_of = [&](float v) {
        return bin_scale > 0.0f ? linear_bin(v, bin_scale) : order_key(v) >> (32 - kDigit0Bits);
    };
    for (uint32_t step = first; step < last; ++step) {
        const uint64_t j0 = (uint64_t)step * STEP_TILES;
        const uint32_t n = T - j0 < STEP_TILES ? (uint32_t)(T - j0) : STEP_TILES;
        if (HIST && j0 >= unit_end) { flush(cur_unit); ++cur_unit; unit_end += unit_tiles; }
        wait_for_rows();
        Row<W, BF16> x[NG];
#pragma unroll
        for (uint32_t g = 0; g < (uint32_t)NG; ++g) x[g].read(lds, g, lane);
        rows_are_read();
        store();
        if (step + 1 < last) request(step + 1);
#pragma unroll
        for (uint32_t g = 0; g < (uint32_t)NG; ++g) {
            if constexpr (PIVOTS) {
                if (pivot) pv[g] = pivot_of<W::EPL, BF16, LPT>(x[g].w, part, tau, eps_ratio);
                x[g].forget();
            }
            auto again = [&]() {                 // my row, from memory
                const uint32_t at = mine + g * W::TILES;
                return TensorRow<W, BF16>(static_cast<const uint8_t *>(in) +
                                          ((j0 + (at < n ? at : n - 1)) * LPT + part) * W::LANE_BYTES);
            };
            if constexpr (APPROX) {
                h[g] = entropy_approx<W::EPL, LPT>(x[g], eps_l1, [&]() {
                    TensorRow<W, BF16> y = again();
                    return entropy_of<W::EPL, LPT>(y, eps_l1, eps_log);
                });
            }
            else h[g] = entropy_of<W::EPL, LPT>(x[g], eps_l1, eps_log);
            if (__ballot(h[g] != h[g]) != 0) h[g] = nan_entropy<W, BF16, LPT>(again(), h[g]);
        }
        j_prev = j0;
        n_prev = n;
        if constexpr (HIST) {                    // (a tile counts in its first lane)
            auto count = [&](uint32_t from, uint32_t to) {
#pragma unroll
                for (uint32_t g = 0; g < (uint32_t)NG; ++g) {
                    const uint32_t j = mine + g * W::TILES;
                    if (part == 0 && j >= from && j < to) lds_add_one(lh_at + 4u * bin_of(h[g]));
                }
            };
            if (unit_end - j0 >= n) {
                count(0, n);
            } else {
                const uint32_t here = (uint32_t)(unit_end - j0);
                count(0, here);
                flush(cur_unit);
                ++cur_unit;
                unit_end += unit_tiles;
                count(here, n);
            }
        }
    }
    if (first < last) store();
    if (HIST && first < last) flush(cur_unit);
    if (blockIdx.x < pro_blocks) write_prologue(pro, blockIdx.x * 256 + tid, pro_blocks * 256);
}

// ---------------------- entropy of allocation tiles wider than a quantization tile

// Sec. 3.2 with A = m*G, m > 1: Eq. 1's norm and Eq. 2's sum run over the A channels of an allocation
// tile.  Both are accumulated per quantization tile by the pairwise tree and then across the m tiles
// from left to right.  In general the work splits into two streaming passes with a small reduction after
// each:
//   WEIGHTED = false: part[j] = sum over tile j of |v|
//   WEIGHTED = true:  part[j] = sum over tile j of |v| log(|v| * r + varsigma), r = inv_norm[j / m] (the common factor r
//                     of Eq. 2's sum is applied once, by the reduction)
// One workgroup per batch of tiles, one lane per tile.
template <int G, bool BF16, bool WEIGHTED>
__global__ __launch_bounds__((Batch<G, BF16 ? 2 : 4>::TILES))
void k_tile_partial(const void *__restrict__ in, const float *__restrict__ inv_norm, float *__restrict__ part,
                    uint32_t T, uint32_t m, float eps_log, uint32_t pro_blocks, Prologue pro)
{
    constexpr int ES = BF16 ? 2 : 4;
    using B = Batch<G, ES>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[B::LDS_BYTES];
    const int tid = threadIdx.x;
    const uint64_t j0 = (uint64_t)blockIdx.x * B::TILES;
    const uint32_t left = T - (uint32_t)j0;
    const uint32_t nvalid = left < (uint32_t)B::TILES ? left : (uint32_t)B::TILES;
    uint4 v[B::CHUNKS];
    if (nvalid == (uint32_t)B::TILES) {
        load_batch<B, true, true>(in, j0, nvalid, v);
        store_batch<B, true>(v, nvalid, lds);
    } else {
        load_batch<B, false>(in, j0, nvalid, v);
        store_batch<B, false>(v, nvalid, lds);
    }
    __syncthreads();
    if ((uint32_t)tid < nvalid) {
        const uint32_t j = (uint32_t)j0 + tid;
        float a[G];
        read_tile<G, BF16>(lds + tid * B::STRIDE, a);
#pragma unroll
        for (int k = 0; k < G; ++k) a[k] = __builtin_fabsf(a[k]);
        if constexpr (WEIGHTED) {
            const float invL = inv_norm[j / m];
#pragma unroll
            for (int k = 0; k < G; ++k) a[k] = a[k] * log_contract(__builtin_fmaf(a[k], invL, eps_log));
        }
        part[j] = tree_sum<G>(a);
    }
    if (blockIdx.x < pro_blocks) write_prologue(pro, blockIdx.x * B::TILES + threadIdx.x, pro_blocks * B::TILES);
}

// The same result in ONE pass over the tensor: a team, a wavefront or a workgroup of four, takes `per` whole allocation tiles at a
// time, as many as its lanes hold (per * m <= SLOTS), and lanes that are left over repeat the last one's work.  The per-tile sums
// meet in LDS, from where every lane adds the m values of its allocation tile from left to right; meanwhile the magnitudes wait in
// registers and the next rows are on their way.  A wavefront by itself needs no barriers.  (Where a workgroup's first lanes added
// up for all and the others waited at barriers, [4,2048,4096] A = 4096, G = 64 took 18.7 us, or 20.7 when its workgroups started
// at once, now 16.6.)
//
// PIVOTS: Eq. 3 is decided here as well, if `pivot` is given: by wavefronts by themselves whose lanes hold whole tiles (encode of
// [4,2048,4096] A = 4096, G = 64: 41.7 us, and 42.5 with Eq. 3 in the quantizer).  Where workgroups meet at barriers or lanes share
// tiles the quantizer has it: [8,2048,5120] A = 5120, G = 32 106.2 us here, 101.0 there; [4,2048,8192] A = 8192, G = 64
// 74.8 and 73.5, G = 128 71.1 and 67.5; fp32 [4,2048,4096] A = 4096, G = 64 57.2 and 56.7.
template <int G, bool BF16, int LPT, bool WAVE_TEAM, bool PIVOTS>
__device__ __forceinline__
void alloc_entropy(const void *__restrict__ in, float *__restrict__ H, uint8_t *__restrict__ pivot, uint32_t n_alloc, uint32_t grid,
                   uint32_t m, uint32_t per, float eps_l1, float eps_log, float tau, float eps_ratio, uint32_t pro_blocks,
                   const Prologue &pro)
{
    using W = Wave<G, BF16 ? 2 : 4, LPT>;
    constexpr uint32_t TEAMS = WAVE_TEAM ? 4 : 1, SLOTS = (WAVE_TEAM ? 64 : 256) / LPT;       // teams per workgroup, tiles per team
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[4 * W::LDS_BYTES];
    __shared__ __attribute__((aligned(16))) float parts[2][TEAMS * SLOTS];
    __shared__ float sums[2][4];             // (at most three allocation tiles of more than 64 tiles)
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    uint8_t *lds = lds_all + wave * W::LDS_BYTES;
    const uint32_t part = lane % LPT, slot = (WAVE_TEAM ? lane : tid) / LPT;
    const uint32_t group = slot / m, q0 = (WAVE_TEAM ? wave * SLOTS : 0u) + group * m;        // my allocation tile, its first slot
    const uint32_t team = WAVE_TEAM ? blockIdx.x * 4 + wave : blockIdx.x, teams = grid * TEAMS;
    const uint32_t wave_row = WAVE_TEAM ? 0u : wave * 64u;                                    // my wavefront's first row of the team's

    auto request = [&](uint32_t a0) {            // allocation tiles [a0, a0 + per)
        const uint32_t have = (n_alloc - a0 < per ? n_alloc - a0 : per) * m * LPT;            // rows
        // (a wavefront without rows of its own repeats the team's last one)
        const uint32_t row0 = wave_row < have ? wave_row : have - 1;
        request_rows<W, 1, false>(static_cast<const uint8_t *>(in) + ((uint64_t)a0 * m * LPT + row0) * W::LANE_BYTES, have - row0,
                                  lds, lane);
    };
    const uint32_t parts_at[2] = {lds_address(parts[0]), lds_address(parts[1])};
    const uint32_t sums_of[2] = {lds_address(sums[0]), lds_address(sums[1])};
    auto meet = [&](uint32_t at, float value) {
        if (part == 0) lds_store(at + 4u * ((WAVE_TEAM ? wave * SLOTS : 0u) + slot), value);
        if constexpr (WAVE_TEAM) wave_lds_fence();
        else lds_barrier();
    };
    // my allocation tile's m values from left to right (lanes left over stay inside the array)
    auto left_to_right = [&](uint32_t at) {
        uint32_t p = at + 4u * (group < per ? q0 : 0u);
        float acc = 0.0f;
        uint32_t q = 0;
        if (m % 4 == 0) {
            for (; q + 16 <= m; q += 16, p += 64) {
                f32x4 v[4];
                lds_load(p, v);
#pragma unroll
                for (int i = 0; i < 16; ++i) acc = acc + v[i / 4][i % 4];
            }
        }
        for (; q < m; ++q, p += 4) acc = acc + lds_load(p);
        return acc;
    };
    // Long sums are the work of one wavefront, in which the allocation tile begins, for all of its lanes: m additions in all four took
    // a third of the vector slots at m = 256 ([4,2048,8192] A = 8192, G = 32: encode 89.5 us, 76.9 so; G = 64, m = 128: 74.8 and 73.9).
    constexpr bool ONE_WAVE = !WAVE_TEAM;
    auto sum_up = [&](uint32_t at, uint32_t sums_at) {
        if constexpr (ONE_WAVE) {
            if (m > 64) {
                const bool begins = group < per && slot == group * m;
                if (__ballot(begins) != 0) {
                    const float acc = left_to_right(at);
                    if (begins && part == 0) lds_store(sums_at + 4u * group, acc);
                }
                lds_barrier();
                return lds_load(sums_at + 4u * (group < per ? group : 0u));
            }
        }
        return left_to_right(at);
    };
    const uint32_t stride = teams * per;
    uint32_t a0 = team * per;
    if (a0 < n_alloc) request(a0);
    float h = 0.0f;
    uint32_t pv = 0, a_prev = n_alloc;           // my allocation tile of the round before
    const bool first = group < per && slot == group * m && part == 0;
    auto store = [&]() {
        if (a_prev >= n_alloc) return;
        if (first) store_through(H + a_prev, h);
        if constexpr (PIVOTS) {
            if (pivot && group < per && part == 0)
                store_through(pivot + ((uint64_t)a_prev * m + (slot - group * m)), (uint8_t)pv);
        }
    };
    for (; a0 < n_alloc; a0 += stride) {
        wait_for_rows();
        Row<W, BF16> x;
        x.read(lds, 0, lane);
        rows_are_read();
        store();
        if (a0 + stride < n_alloc) request(a0 + stride);
        meet(parts_at[0], whole_tile<LPT>(magnitude_sum<W::EPL>(x)));
        x.forget();
        if constexpr (PIVOTS) {
            if (pivot) pv = pivot_of<W::EPL, BF16, LPT>(x.w, part, tau, eps_ratio);
            x.forget();
        }
        const float invL = 1.0f / (sum_up(parts_at[0], sums_of[0]) + eps_l1);
        meet(parts_at[1], whole_tile<LPT>(weighted_sum<W::EPL>(x, invL, eps_log)));
        h = 0.0f - invL * sum_up(parts_at[1], sums_of[1]);
        a_prev = a0 + group;
    }
    store();
    if (blockIdx.x < pro_blocks) write_prologue(pro, blockIdx.x * 256 + tid, pro_blocks * 256);
}

// The usual lanes, wavefronts by themselves.
template <int G, bool BF16>
__global__ __launch_bounds__(256, 4)
void k_alloc_entropy(const void *__restrict__ in, float *__restrict__ H, uint8_t *__restrict__ pivot, uint32_t n_alloc,
                     uint32_t grid, uint32_t m, uint32_t per, float eps_l1, float eps_log, uint32_t pro_blocks, float tau,
                     float eps_ratio, Prologue pro)
{
    alloc_entropy<G, BF16, Lanes<G, BF16 ? 2 : 4>::usual, true, kWholeTiles<G, BF16>>(in, H, pivot, n_alloc, grid, m, per, eps_l1,
                                                                                       eps_log, tau, eps_ratio, pro_blocks, pro);
}

// Any others.
template <int G, bool BF16, int LPT, bool WAVE_TEAM>
__global__ __launch_bounds__(256, 4)
void k_alloc_entropy_by(const void *__restrict__ in, float *__restrict__ H, uint32_t n_alloc, uint32_t grid, uint32_t m, uint32_t per,
                        float eps_l1, float eps_log, uint32_t pro_blocks, Prologue pro)
{
    alloc_entropy<G, BF16, LPT, WAVE_TEAM, false>(in, H, nullptr, n_alloc, grid, m, per, eps_l1, eps_log, 0.0f, 0.0f, pro_blocks, pro);
}

// Left-to-right sum of the m partial sums of every allocation tile.  FINAL = false: the reciprocal norm
// r = 1 / (L1 + eps) of Eq. 1; FINAL = true: the entropy 0 - r * sum of Eq. 2, with r read from `inv_norm`.
template <bool FINAL>
__global__ __launch_bounds__(256) void k_alloc_reduce(const float *__restrict__ part, const float *__restrict__ inv_norm,
                                                      float *__restrict__ out, uint32_t n_alloc, uint32_t m, float eps_l1)
{
    const uint32_t ja = blockIdx.x * 256 + threadIdx.x;
    if (ja >= n_alloc) return;
    const float *p = part + (uint64_t)ja * m;
    float acc = 0.0f;
    for (uint32_t q = 0; q < m; ++q) acc = acc + p[q];
    if constexpr (FINAL) out[ja] = 0.0f - inv_norm[ja] * acc;
    else out[ja] = 1.0f / (acc + eps_l1);
}

// ------------------------------------ K3: transform + quantize + pack

// Payload unit: a tile's payload is b units of G/8 bytes (b = 3 or 4).
template <int G> struct Unit;
template <> struct Unit<8>   { using type = uint8_t; };
template <> struct Unit<16>  { using type = uint16_t; };
template <> struct Unit<32>  { using type = uint32_t; };
template <> struct Unit<64>  { using type = uint2; };
template <> struct Unit<128> { using type = uint4; };

// What a workgroup must know about a batch before it can place payload: the bit map words of the
// batch's 64-tile groups and the rank-table entry of the first one.
template <int TILES>
struct BatchMeta {
    static constexpr int WORDS = (TILES + 63) / 64;
    uint64_t word[WORDS];
    uint32_t rank0;
};

template <int TILES>
__device__ __forceinline__ void load_meta(const uint8_t *__restrict__ packed, const Sections &lay, uint64_t j0, uint32_t T,
                                          BatchMeta<TILES> &m)
{
    const uint64_t *bitmap = reinterpret_cast<const uint64_t *>(packed + lay.bitmap);
    const uint32_t *ranks = reinterpret_cast<const uint32_t *>(packed + lay.ranks);
    const uint64_t last_word = ((uint64_t)T - 1) >> 6;
#pragma unroll
    for (int w = 0; w < BatchMeta<TILES>::WORDS; ++w) {
        const uint64_t jw = (j0 >> 6) + w;
        const uint64_t word = bitmap[jw <= last_word ? jw : last_word];     // clamped index: no load behind a branch
        m.word[w] = jw <= last_word ? word : 0ull;
    }
    m.rank0 = ranks[j0 >> 6];
}

// Number of set bits of `mask` in the lanes below mine (two instructions).
__device__ __forceinline__ uint32_t bits_below_me(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Width of my tile (LOW or LOW + 1 bits), its payload position inside the batch (in units of G/8 bytes), and
// the number of wide tiles in the batch.  A wavefront's tiles are one bit map word.
template <int TILES, int LOW>
__device__ __forceinline__ void tile_pos(const BatchMeta<TILES> &m, int tid, uint32_t *b, uint32_t *rel, uint32_t *total4)
{
    const uint32_t mine_word = (uint32_t)__builtin_amdgcn_readfirstlane(tid / 64);      // the same in every lane
    const uint32_t tile = (uint32_t)tid, at = tile & 63u;
    uint64_t mine = 0;
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < BatchMeta<TILES>::WORDS; ++w) {
        if ((uint32_t)w == mine_word) { mine = m.word[w]; before = tot; }
        tot += (uint32_t)__popcll(m.word[w]);
    }
    const uint32_t half = at < 32u ? (uint32_t)mine : (uint32_t)(mine >> 32);
    *b = (uint32_t)LOW + ((half >> (at & 31u)) & 1u);
    const uint32_t below = bits_below_me(mine);
    *rel = (uint32_t)LOW * tile + before + below;
    *total4 = tot;
}

// Tiles of a batch regrouped by class (0..3; anything else sorts nowhere): the position of my tile when the batch is
// ordered by class and, inside a class, by tile index.  Two steps with a workgroup barrier between them.
// Step 1: my rank among the tiles of my class in my wavefront; lane 0 leaves the wavefront's four counts in
// `counts` (LDS, uint32[4 * WAVES], class-major).
template <int WAVES>
__device__ __forceinline__ uint32_t class_rank_in_wave(uint32_t cls, uint32_t wave, uint32_t lane, uint32_t *counts)
{
    uint32_t rank = 0;
#pragma unroll
    for (uint32_t c = 0; c < 4; ++c) {
        const uint64_t m = __ballot(cls == c);
        if (cls == c) rank = bits_below_me(m);
        if (lane == 0) counts[c * WAVES + wave] = (uint32_t)__popcll(m);
    }
    return rank;
}

// Step 2 (after the barrier): tiles that come before my class-and-wavefront group.  In class-major order that is
// the exclusive prefix sum of the 4 * WAVES counts: lanes 0 .. 4 WAVES - 1 scan them with row shifts, and every
// lane fetches the entry of its own group.  All lanes of the wavefront must be enabled.
template <int WAVES>
__device__ __forceinline__ uint32_t class_group_base(uint32_t cls, uint32_t wave, uint32_t lane, const uint32_t *counts)
{
    static_assert(4 * WAVES <= 16, "the counts must fit one row of 16 lanes");
    const uint32_t own = lane < 4u * WAVES ? counts[lane] : 0u;
    uint32_t v = own;
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);     // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);     // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);     // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);     // row_shr:8
    const uint32_t group = cls < 4u ? cls * WAVES + wave : 0u;
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(group << 2), (int)(v - own));
}

// Three-input float min / max in one instruction each (no NaN canonicalisation around them).
__device__ __forceinline__ float fmin3(float a, float b, float c)
{
    float r;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float fmax3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// The rest of the encoder for one tile, in two steps with a workgroup barrier between them (the payload
// buffer that step 2 writes shares LDS with the rows that step 1 reads).
// Step 1: the row (which already carries P_d) into registers; Eq. 4 on outlier tiles.
template <int G>
__device__ __forceinline__ void transform_row(const uint8_t *row, bool flag, float *x)
{
    read_tile<G, true>(row, x);
    if (flag) {
        butterfly<G>(x);
#pragma unroll
        for (int k = 0; k < G; ++k) x[k] = x[k] * TileConst<G>::c;
    }
}

// Dwords that hold the G W-bit codes of a tile.
template <int G, int W> struct BitString { static constexpr int DWORDS = (G * W + 31) / 32; };

// The tile's LSB-first bit string, as dwords, from groups of four W-bit codes (g4[g] = q0 + 2^W q1 + 2^2W q2
// + 2^3W q3), W <= 4.  Writes the dwords the string occupies; the caller has cleared the rest.
template <int G, int W>
__device__ __forceinline__ void pack_groups(const uint32_t *g4, uint32_t *dw)
{
    static_assert(W >= 1 && W <= 4, "groups of four codes are exact in fp32 up to 4 bits per code");
    if constexpr (G < 32) {
        // at most 64 bits: two or four groups of 4 W bits through one 64-bit accumulator
        uint64_t acc = 0;
#pragma unroll
        for (int g = 0; g < G / 4; ++g) acc |= (uint64_t)g4[g] << (4 * W * g);
        dw[0] = (uint32_t)acc;
        if constexpr (G * W > 32) dw[1] = (uint32_t)(acc >> 32);
    } else if constexpr (W == 4) {
#pragma unroll
        for (int i = 0; i < G / 8; ++i) dw[i] = g4[2 * i] | (g4[2 * i + 1] << 16);
    } else if constexpr (W == 3) {
        // 12-bit groups: eight of them fill three dwords
#pragma unroll
        for (int i = 0; i < G / 32; ++i) {
            const uint32_t *p = g4 + 8 * i;
            dw[3 * i + 0] = p[0] | (p[1] << 12) | (p[2] << 24);
            dw[3 * i + 1] = (p[2] >> 8) | (p[3] << 4) | (p[4] << 16) | (p[5] << 28);
            dw[3 * i + 2] = (p[5] >> 4) | (p[6] << 8) | (p[7] << 20);
        }
    } else if constexpr (W == 2) {
        // 8-bit groups: four of them fill a dword
#pragma unroll
        for (int i = 0; i < G / 16; ++i)
            dw[i] = g4[4 * i] | (g4[4 * i + 1] << 8) | (g4[4 * i + 2] << 16) | (g4[4 * i + 3] << 24);
    } else {
        // 4-bit groups: eight of them fill a dword
#pragma unroll
        for (int i = 0; i < G / 32; ++i) {
            uint32_t t = 0;
#pragma unroll
            for (int g = 0; g < 8; ++g) t |= g4[8 * i + g] << (4 * g);
            dw[i] = t;
        }
    }
}

// The same from the codes themselves, for any width up to 8 bits: code k occupies bits [W k, W k + W).
template <int G, int W>
__device__ __forceinline__ void place_codes(const uint32_t *q, uint32_t *dw)
{
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const int bit = W * k, i = bit >> 5, sh = bit & 31;
        dw[i] |= q[k] << sh;
        if (sh + W > 32) dw[i + 1] |= q[k] >> (32 - sh);
    }
}

// The range of a tile of LPT parts, of which I have G elements.
struct TileRange { float mn, mx; };
template <int G, int LPT>
__device__ __forceinline__ TileRange tile_range(const float *x)
{
    float mn = fmin3(x[0], x[1], x[2]), mx = fmax3(x[0], x[1], x[2]);
#pragma unroll
    for (int k = 3; k + 1 < G; k += 2) { mn = fmin3(mn, x[k], x[k + 1]); mx = fmax3(mx, x[k], x[k + 1]); }
    mn = __builtin_fminf(mn, x[G - 1]);
    mx = __builtin_fmaxf(mx, x[G - 1]);
    if constexpr (LPT >= 2) { mn = __builtin_fminf(mn, lane_xor<1>(mn)); mx = __builtin_fmaxf(mx, lane_xor<1>(mx)); }
    if constexpr (LPT >= 4) { mn = __builtin_fminf(mn, lane_xor<2>(mn)); mx = __builtin_fmaxf(mx, lane_xor<2>(mx)); }
    mn = mn + 0.0f;                              // (as statements: inside the return the compiler orders k_quant_pack<64> otherwise, which
    mx = mx + 0.0f;                              // took 18.2 us instead of 17.7 on bf16 [4,2048,4096] A = 4096)
    return {mn, mx};
}

// Step 2: quantizer parameters of the tile from its range, codes of my G elements of it, and their LSB-first bit string written
// as b units at `dst` (LDS); b is LOW or LOW + 1.  Returns scale | zero << 16.
template <int G, int LOW>
__device__ __forceinline__ uint32_t quantize_values(const float *x, const TileRange &range, uint32_t b, typename Unit<G>::type *dst)
{
    constexpr uint32_t WIDE = LOW + 1;
    const float mn = range.mn, mx = range.mx;

    // asymmetric quantizer, binary16 metadata rounded outwards
    const float Lv = (b == WIDE) ? (float)((1u << WIDE) - 1u) : (float)((1u << LOW) - 1u);
    const uint32_t z16 = f16_down(mn);
    const float mnf = f16_widen(z16);
    const float s = (mx - mnf) / Lv;
    uint32_t s16 = f16_up(s);
    if ((s16 & 0x7fffu) == 0) s16 = 0x3c00u;
    const float sf = f16_widen(s16);
    const float rcp = 1.0f / sf;
    // Every element lies in [mn, mx]; if z <= mn, (x - z) * rcp lies in [0, (mx - z) * rcp], and when that
    // bound rounds to at most L the clamp is the identity and is skipped.  Both conditions can fail only when
    // the binary16 metadata saturated (magnitudes beyond the contract).
    const bool no_clamp = mnf <= mn && (mx - mnf) * rcp <= Lv + 0.25f;

    constexpr int DW = BitString<G, WIDE>::DWORDS > G / 8 ? BitString<G, WIDE>::DWORDS : (G / 8 ? G / 8 : 1);
    uint32_t dw[DW];
#pragma unroll
    for (int i = 0; i < DW; ++i) dw[i] = 0;
    if constexpr (WIDE <= 4) {
        // codes, four at a time: q0 + m q1 + m^2 q2 + m^3 q3 is an exact integer below 2^16 in fp32
        const float m1 = (b == WIDE) ? (float)(1u << WIDE) : (float)(1u << LOW);
        const float m2 = m1 * m1, m3 = m2 * m1;
        uint32_t g4[G / 4];
        if (no_clamp) {
#pragma unroll
            for (int g = 0; g < G / 4; ++g) {
                float q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = __builtin_rintf((x[4 * g + i] - mnf) * rcp);
                const float acc = __builtin_fmaf(q[3], m3, __builtin_fmaf(q[2], m2, __builtin_fmaf(q[1], m1, q[0])));
                g4[g] = (uint32_t)acc;
            }
        } else {
#pragma unroll
            for (int g = 0; g < G / 4; ++g) {
                float q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    q[i] = __builtin_amdgcn_fmed3f(__builtin_rintf((x[4 * g + i] - mnf) * rcp), 0.0f, Lv);
                const float acc = __builtin_fmaf(q[3], m3, __builtin_fmaf(q[2], m2, __builtin_fmaf(q[1], m1, q[0])));
                g4[g] = (uint32_t)acc;
            }
        }
        if (b == WIDE) pack_groups<G, WIDE>(g4, dw);
        else pack_groups<G, LOW>(g4, dw);
    } else {
        // wider codes: one by one (a NaN code becomes 0 in the clamp)
        uint32_t q[G];
#pragma unroll
        for (int k = 0; k < G; ++k)
            q[k] = (uint32_t)__builtin_amdgcn_fmed3f(__builtin_rintf((x[k] - mnf) * rcp), 0.0f, Lv);
        if (b == WIDE) place_codes<G, WIDE>(q, dw);
        else place_codes<G, LOW>(q, dw);
    }
    // the bit string leaves as b units of G/8 bytes
#pragma unroll
    for (int u = 0; u < (int)WIDE; ++u) {
        if (u < LOW || b == WIDE) {
            if constexpr (G == 8) dst[u] = (uint8_t)(dw[u >> 2] >> (8 * (u & 3)));
            else if constexpr (G == 16) dst[u] = (uint16_t)(dw[u >> 1] >> (16 * (u & 1)));
            else if constexpr (G == 32) dst[u] = dw[u];
            else if constexpr (G == 64) dst[u] = make_uint2(dw[2 * u], dw[2 * u + 1]);
            else dst[u] = make_uint4(dw[4 * u], dw[4 * u + 1], dw[4 * u + 2], dw[4 * u + 3]);
        }
    }
    return s16 | (z16 << 16);
}

// Store of a payload unit that passes the caches by.
template <class U>
__device__ __forceinline__ void store_streaming(U *p, const U &v)
{
    if constexpr (sizeof(U) == 16) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), reinterpret_cast<u32x4 *>(p));
    else if constexpr (sizeof(U) == 8) __builtin_nontemporal_store(__builtin_bit_cast(uint64_t, v), reinterpret_cast<uint64_t *>(p));
    else __builtin_nontemporal_store(v, p);
}

// How k_quant_pack goes about it.
enum : uint32_t { QUANT_ALL_WIDE = 1, QUANT_STREAMING = 2 };

// One workgroup per batch of TILES tiles, in two stages.  Stage one: lane i takes tile i's pivot byte, from the entropy pass if
// PIVOTS, from Eq. 3 on the spot otherwise, and swaps its pivot in LDS.  The tiles are regrouped by
// class -- (plain | transformed) x (narrow | wide) -- so that in
// stage two, where lane p takes the p-th tile in class order, most wavefronts hold a single class: the
// Hadamard butterfly runs only in the wavefronts that hold transformed tiles, and the two packing
// paths rarely both run.  The payload buffer reuses the rows' LDS once every lane holds its tile in
// registers, which keeps the workgroup small enough for four to share a compute unit: this kernel
// lives on the loads of its neighbours being in flight while it computes.
// For bf16 tiles of 32 and 64 channels in tensors of many; all others are quantized by wavefronts, below.
template <int G, int LOW, bool RANKED, bool PIVOTS, bool FULL>
__device__ __forceinline__ void quant_pack_batch(const void *__restrict__ in, uint8_t *__restrict__ packed, const Sections &lay,
                                                 uint32_t T, float tau, float eps_ratio, uint32_t batch, uint32_t nvalid,
                                                 bool all_wide, bool streaming, uint8_t *lds, uint32_t *info, uint16_t *order,
                                                 uint32_t *class_count)
{
    using B = Batch<G, 2>;
    using U = typename Unit<G>::type;
    constexpr int THREADS = B::TILES;
    constexpr int WAVES = THREADS / 64;
    constexpr uint32_t WIDE = LOW + 1;           // the two code widths are LOW and WIDE bits
    static_assert(sizeof(U) * WIDE * B::TILES <= (size_t)B::LDS_BYTES, "payload buffer must fit in the rows");
    U *pay = reinterpret_cast<U *>(lds);         // valid only after every lane has left the rows
    // The lane index passes through an empty asm statement, so the optimiser derives every address from
    // it afresh instead of sharing address arithmetic between the phases: measured 3 % faster.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t slot = (uint32_t)tid;
    const uint64_t j0 = (uint64_t)batch * B::TILES;

    uint4 v[B::CHUNKS];
    load_batch<B, FULL, true>(in, j0, nvalid, v, tid);           // second and last read of the tensor
    BatchMeta<B::TILES> meta;
    if constexpr (RANKED) {
        load_meta<B::TILES>(packed, lay, j0, T, meta);
    } else {
        // one width for all tiles: the batch's bit map words and rank-table entries are constants, and written at the end
        const uint64_t w0 = j0 >> 6, words = ((uint64_t)T + 63) >> 6;
#pragma unroll
        for (int w = 0; w < BatchMeta<B::TILES>::WORDS; ++w) meta.word[w] = w0 + w < words ? constant_word(w0 + w, T, all_wide) : 0ull;
        meta.rank0 = all_wide ? (uint32_t)j0 : 0u;
    }
    const bool valid = FULL || slot < nvalid;
    uint32_t pv = 0;                             // pivot byte of the tile of my slot, in storage order
    if constexpr (PIVOTS) {
        pv = packed[lay.pivot + j0 + (valid ? slot : 0u)];
    }
    uint32_t b, rel, total4;
    tile_pos<B::TILES, LOW>(meta, tid, &b, &rel, &total4);
    if constexpr (!PIVOTS) {
        store_batch<B, FULL>(v, nvalid, lds, tid);
        __syncthreads();
        if (valid) pv = pivot_of_row<G>(lds + slot * B::STRIDE, tau, eps_ratio);
    }
    // stage one: my tile's class
    uint32_t cls = 4;                            // tiles past the end sort nowhere
    if (valid) {
        info[slot] = pv | ((b == WIDE) ? 0x100u : 0u) | (rel << 9);
        cls = ((pv >> 7) << 1) | (b == WIDE ? 1u : 0u);
    }
    const uint32_t rank_in_wave = class_rank_in_wave<WAVES>(cls, (uint32_t)wave, (uint32_t)lane, class_count);
    if constexpr (PIVOTS) store_batch<B, FULL>(v, nvalid, lds, tid);
    __syncthreads();
    {
        const uint32_t pos = rank_in_wave + class_group_base<WAVES>(cls, (uint32_t)wave, (uint32_t)lane, class_count);
        if (cls < 4) {
            order[pos] = (uint16_t)slot;
            // an outlier tile with d != 0 (inside the row whatever the stream holds, as in the decoder)
            if (pv > 0x80u) swap_pivot(lds + slot * B::STRIDE, pv & (G - 1u));
        }
    }
    __syncthreads();

    // stage two: the tile of my slot in class order
    float x[G];
    uint32_t t = 0, inf = 0;
    if (valid) {
        t = order[slot];
        inf = info[t];
        transform_row<G>(lds + t * B::STRIDE, (inf & 0x80u) != 0, x);
    }
    __syncthreads();                             // the rows are dead: their LDS becomes the payload buffer
    if (valid) {
        const uint32_t width = (inf & 0x100u) ? WIDE : (uint32_t)LOW;
        const uint32_t meta16 = quantize_values<G, LOW>(x, tile_range<G, 1>(x), width, pay + (inf >> 9));
        const uint64_t j = j0 + t;
        reinterpret_cast<uint16_t *>(packed + lay.scale)[j] = (uint16_t)meta16;
        reinterpret_cast<uint16_t *>(packed + lay.zero)[j] = (uint16_t)(meta16 >> 16);
        if constexpr (!PIVOTS) packed[lay.pivot + j] = (uint8_t)inf;
    }
    __syncthreads();

    // the batch's payload is one contiguous span: copy it out unit by unit, coalesced
    const uint32_t span = (uint32_t)LOW * nvalid + total4;
    U *gdst = reinterpret_cast<U *>(packed + lay.payload) + ((uint64_t)LOW * j0 + meta.rank0);
#pragma unroll
    for (int i = 0; i < (int)WIDE; ++i) {
        const uint32_t q = (uint32_t)i * THREADS + tid;
        if (q < span) {
            if (streaming) store_streaming(gdst + q, pay[q]);
            else gdst[q] = pay[q];
        }
    }
    if constexpr (!RANKED) {
        const uint64_t w = (j0 >> 6) + tid;
        if (tid < BatchMeta<B::TILES>::WORDS && w < ((uint64_t)T + 63) >> 6)
            constant_width_word(w, T, all_wide, reinterpret_cast<uint64_t *>(packed + lay.bitmap),
                                reinterpret_cast<uint32_t *>(packed + lay.ranks));
    }
}

// RANKED: the widths are in the stream's bit map.  Otherwise all tiles have one, and the kernel is the call's only one and
// writes bit map, rank table and prologue as well.  (A variant of its own: the same as a run-time choice delayed the loads of
// the ranked case, 126 -> 136 us on bf16 [8,4096,8192].)
template <int G, int LOW, bool RANKED, bool PIVOTS>
__global__ __launch_bounds__(256, 4)
void k_quant_pack(const void *__restrict__ in, uint8_t *__restrict__ packed, uint32_t T, float tau, float eps_ratio,
                  uint32_t how, Prologue pro)
{
    using B = Batch<G, 2>;
    constexpr int THREADS = B::TILES, WAVES = THREADS / 64;
    __shared__ __attribute__((aligned(16))) uint8_t lds[B::LDS_BYTES];
    __shared__ uint32_t info[B::TILES];          // per tile: pivot byte | (b == WIDE) << 8 | rel << 9
    __shared__ uint16_t order[B::TILES];         // tiles in class order
    __shared__ uint32_t class_count[4 * WAVES];  // tiles per class and wavefront, class-major
    const Sections lay(T);
    const uint32_t nfull = T / B::TILES;        // a workgroup per batch; the last one may be ragged
    if (blockIdx.x < nfull)
        quant_pack_batch<G, LOW, RANKED, PIVOTS, true>(in, packed, lay, T, tau, eps_ratio, blockIdx.x, B::TILES,
                                                                  (how & QUANT_ALL_WIDE) != 0, (how & QUANT_STREAMING) != 0, lds,
                                                                  info, order, class_count);
    else
        quant_pack_batch<G, LOW, RANKED, PIVOTS, false>(in, packed, lay, T, tau, eps_ratio, nfull, T % B::TILES,
                                                                   (how & QUANT_ALL_WIDE) != 0, (how & QUANT_STREAMING) != 0, lds,
                                                                   info, order, class_count);
    if constexpr (!RANKED) {
        if (blockIdx.x == 0) write_prologue(pro, threadIdx.x, THREADS);      // (nothing but header and padding)
    }
}

// The quantizer of a wavefront by itself, for the tiles of its lanes, without barriers, as the decoder is.  The butterfly then runs in every
// wavefront that meets an outlier tile, instead of in those that hold the outlier tiles of a workgroup.  That costs vector slots,
// which are there where tiles have few channels, many bytes or several lanes; what it saves are the barriers, at which most
// of a workgroup waited for its loads and then for the wavefront with the outlier tiles.  RANKED and PIVOTS as in k_quant_pack.
// Encode against k_quant_pack, at 3 bits: bf16 G = 128 [4,1024,4096] 13.3 -> 11.8 us, [8,4096,8192] 131.6 -> 126.2, G = 8 [4,2048,8192]
// 58.5 -> 54.3, G = 16 44.2 -> 42.2; fp32 G = 64 [8,2048,8192] 106.5 -> 102.2, G = 32 [4,2048,8192] 55.0 -> 53.8, G = 8 69.4 -> 65.2; at
// 3.5 bits bf16 G = 128 [8,2048,8192] 133.3 -> 129.6, G = 8 [4,2048,8192] 132.2 -> 124.5, fp32 G = 64 [8,1024,2048] 41.0 -> 39.4.
// bf16 G = 32, a lane per tile: [8,1024,2048] 12.4 -> 11.9, but [4,2048,8192] at 3.5 bits 81.2 -> 82.1 and [16,2048,5120] alike; with
// 64 elements in a lane vector issue is what bounds the quantizer.  Those two stay with k_quant_pack.
template <int G, bool BF16, int LOW, bool RANKED, bool PIVOTS, int LPT>
__global__ __launch_bounds__(256, 4)
void k_quant_by_wave(const void *__restrict__ in, uint8_t *__restrict__ packed, uint32_t T, float tau, float eps_ratio, uint32_t how,
                     Prologue pro)
{
    using W = Wave<G, BF16 ? 2 : 4, LPT>;
    using U = typename Unit<G>::type;
    constexpr int EPL = W::EPL;
    constexpr uint32_t WIDE = LOW + 1;
    static_assert(WIDE * W::TILES * sizeof(U) <= (size_t)W::LDS_BYTES, "the payload lies where the rows were");
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[4 * W::LDS_BYTES];
    const uint32_t lane = threadIdx.x & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t j0 = ((uint64_t)blockIdx.x * 4 + wave) * W::TILES;
    if (j0 < T) {
        uint8_t *lds = lds_all + wave * W::LDS_BYTES;
        const uint32_t left = (uint32_t)(T - j0), tiles = left < (uint32_t)W::TILES ? left : (uint32_t)W::TILES;
        request_rows<W, 1, true>(static_cast<const uint8_t *>(in) + j0 * W::EPL * LPT * (BF16 ? 2 : 4), tiles * LPT, lds, lane);
        const Sections lay(T);
        const uint32_t t = lane / LPT, part = lane % LPT, mine = t < tiles ? t : tiles - 1;      // (lanes past the end: the last tile)
        // my tile's width and, in units of G/8 bytes, its place in the wavefront's payload, which starts at unit `first` and has `units`
        uint32_t b, at;
        uint64_t first;
        uint32_t units;
        if constexpr (RANKED) {
            const uint64_t word = reinterpret_cast<const uint64_t *>(packed + lay.bitmap)[j0 >> 6] >> (j0 & 63u);
            const uint64_t before = reinterpret_cast<const uint64_t *>(packed + lay.bitmap)[j0 >> 6] & ((1ull << (j0 & 63u)) - 1ull);
            const uint32_t rank0 = reinterpret_cast<const uint32_t *>(packed + lay.ranks)[j0 >> 6];
            b = (uint32_t)LOW + ((uint32_t)(word >> mine) & 1u);
            at = (uint32_t)LOW * t + (uint32_t)__popcll(word & ((1ull << mine) - 1ull));
            first = (uint64_t)LOW * j0 + rank0 + (uint32_t)__popcll(before);
            units = (uint32_t)LOW * tiles + (uint32_t)__popcll(tiles < 64 ? word & ((1ull << tiles) - 1ull) : word);
        } else {
            const bool all_wide = (how & QUANT_ALL_WIDE) != 0;
            b = all_wide ? WIDE : (uint32_t)LOW;
            at = b * t;
            first = b * j0;
            units = b * tiles;
            if ((j0 & 63u) == 0 && lane == 0)
                constant_width_word(j0 >> 6, T, all_wide, reinterpret_cast<uint64_t *>(packed + lay.bitmap),
                                    reinterpret_cast<uint32_t *>(packed + lay.ranks));
        }
        uint32_t pv = 0;
        if constexpr (PIVOTS) pv = packed[lay.pivot + j0 + mine];
        wait_for_rows();
        Row<W, BF16> row;
        row.read(lds, 0, lane);
        if constexpr (!PIVOTS) pv = pivot_of<EPL, BF16, LPT>(row.w, part, tau, eps_ratio);
        if (__ballot(pv > 0x80u) != 0) {
            // P_d, on the rows in LDS
            if (pv > 0x80u && part == 0) {
                uint8_t *e0 = lds + W::element_at(lane, 0), *ed = lds + W::element_at(lane, pv & (G - 1u));
                if constexpr (BF16) {
                    const uint16_t v0 = *reinterpret_cast<uint16_t *>(e0), vd = *reinterpret_cast<uint16_t *>(ed);
                    *reinterpret_cast<uint16_t *>(e0) = vd; *reinterpret_cast<uint16_t *>(ed) = v0;
                } else {
                    const float v0 = *reinterpret_cast<float *>(e0), vd = *reinterpret_cast<float *>(ed);
                    *reinterpret_cast<float *>(e0) = vd; *reinterpret_cast<float *>(ed) = v0;
                }
            }
            wave_lds_fence();
            row.read(lds, 0, lane);
        }
        float x[EPL];
#pragma unroll
        for (int k = 0; k < EPL; ++k) x[k] = row[k];
        if ((pv & 0x80u) != 0) {                 // the lanes of a tile agree
            butterfly<EPL>(x);
            butterfly_across<EPL, LPT>(x, part);
#pragma unroll
            for (int k = 0; k < EPL; ++k) x[k] = x[k] * TileConst<G>::c;
        }
        wave_lds_fence();                        // the rows are dead: their LDS becomes the payload buffer
        U *pay = reinterpret_cast<U *>(lds);
        if (t < tiles) {
            const uint32_t meta16 = quantize_values<EPL, LOW>(x, tile_range<EPL, LPT>(x), b,
                                                              reinterpret_cast<typename Unit<EPL>::type *>(pay + at) + part * b);
            if (part == 0) {
                const uint64_t j = j0 + t;
                reinterpret_cast<uint16_t *>(packed + lay.scale)[j] = (uint16_t)meta16;
                reinterpret_cast<uint16_t *>(packed + lay.zero)[j] = (uint16_t)(meta16 >> 16);
                if constexpr (!PIVOTS) packed[lay.pivot + j] = (uint8_t)pv;
            }
        }
        wave_lds_fence();
        U *dst = reinterpret_cast<U *>(packed + lay.payload) + first;
#pragma unroll
        for (int i = 0; i < ((int)WIDE + LPT - 1) / LPT; ++i) {
            const uint32_t q = (uint32_t)i * 64 + lane;
            if (q < units) {
                if (how & QUANT_STREAMING) store_streaming(dst + q, pay[q]);
                else dst[q] = pay[q];
            }
        }
    }
    if constexpr (!RANKED) {
        if (blockIdx.x == 0) write_prologue(pro, threadIdx.x, 256);    // (nothing but header and padding)
    }
}

// ------------------------------------------------------------- K4: decode

// The tile's W-bit codes brought onto nibble boundaries: nib[i] holds codes 8i .. 8i+7, one per nibble.
template <int G, int W>
__device__ __forceinline__ void codes_to_nibbles(const uint32_t *dw, uint32_t *nib)
{
    if constexpr (W == 4) {
#pragma unroll
        for (int i = 0; i < G / 8; ++i) nib[i] = dw[i];
    } else if constexpr (W == 3) {
#pragma unroll
        for (int i = 0; i < G / 8; ++i) {
            // codes 8i .. 8i+7 occupy bits [24i, 24i+24) of the string
            const int lo = (24 * i) >> 5, sh = (24 * i) & 31;
            uint32_t t = dw[lo] >> sh;
            if (sh > 8) t |= dw[lo + 1] << (32 - sh);
            t &= 0x00ffffffu;
            t = (t & 0x00000fffu) | ((t & 0x00fff000u) << 4);
            t = (t & 0x003f003fu) | ((t & 0x0fc00fc0u) << 2);
            t = (t & 0x07070707u) | ((t & 0x38383838u) << 1);
            nib[i] = t;
        }
    } else if constexpr (W == 2) {
#pragma unroll
        for (int i = 0; i < G / 8; ++i) {
            // codes 8i .. 8i+7 occupy bits [16i, 16i+16) of the string
            uint32_t t = (dw[i >> 1] >> (16 * (i & 1))) & 0xffffu;
            t = (t & 0x000000ffu) | ((t & 0x0000ff00u) << 8);
            t = (t & 0x000f000fu) | ((t & 0x00f000f0u) << 4);
            t = (t & 0x03030303u) | ((t & 0x0c0c0c0cu) << 2);
            nib[i] = t;
        }
    } else {
        static_assert(W == 1, "nibbles hold codes of up to 4 bits");
#pragma unroll
        for (int i = 0; i < G / 8; ++i) {
            // codes 8i .. 8i+7 are byte i of the string
            uint32_t t = (dw[i >> 2] >> (8 * (i & 3))) & 0xffu;
            t = (t & 0x0000000fu) | ((t & 0x000000f0u) << 12);
            t = (t & 0x00030003u) | ((t & 0x000c000cu) << 6);
            t = (t & 0x01010101u) | ((t & 0x02020202u) << 3);
            nib[i] = t;
        }
    }
}

// ... and, for any width up to 8 bits, the codes one by one, de-quantized: x[k] = q_k * sf + mnf.
template <int G, int W>
__device__ __forceinline__ void dequantize_codes(const uint32_t *dw, float sf, float mnf, float *x)
{
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const int bit = W * k, i = bit >> 5, sh = bit & 31;
        uint32_t q = dw[i] >> sh;
        if (sh + W > 32) q |= dw[i + 1] << (32 - sh);
        x[k] = __builtin_fmaf((float)(q & ((1u << W) - 1u)), sf, mnf);
    }
}

// My share of a tile's bit string: LOW or LOW + 1 units of UB = EPL / 8 bytes at `p`, as dwords.  `end` is the end of the
// stream.
template <int UB, int LOW>
__device__ __forceinline__ void load_codes(const uint8_t *__restrict__ p, bool wide, const uint8_t *end, uint32_t *dw)
{
    constexpr int WIDE = LOW + 1;
    if constexpr (UB >= 4) {
        const uint8_t *q = static_cast<const uint8_t *>(__builtin_assume_aligned(p, 4));
        __builtin_memcpy(dw, q, LOW * UB);
        // a narrow tile's last unit is its first one again: an address that is in the stream, and ignored
        const uint8_t *last = static_cast<const uint8_t *>(__builtin_assume_aligned(p + (wide ? LOW * UB : 0), 4));
        __builtin_memcpy(dw + LOW * UB / 4, last, UB);
    } else {
        constexpr int BYTES = (WIDE * UB + 3) & ~3;      // one unaligned load of whole dwords, except at the stream's end
        if (p + BYTES <= end) {
            __builtin_memcpy(dw, p, BYTES);
        } else {
#pragma unroll
            for (int i = 0; i < WIDE * UB; ++i)
                if (i < LOW * UB || wide) dw[i >> 2] |= (uint32_t)p[i] << (8 * (i & 3));
        }
    }
}

// Alg. 1 step 5: codes -> q*s + z -> for transformed tiles the butterfly, 1/sqrt(G) and P_d -> output type.
//
// One wavefront per group of tiles, no workgroup barriers: every wavefront finds its payload from the group's bit map word
// and rank-table entry, decodes its tiles in registers and brings them into storage order through its own piece of LDS.
// Bound by HBM, four fifths of the bytes being stores.  Lanes hold at most 128 bytes, so 4 workgroups of 32 KB of LDS and at
// most 128 registers share a compute unit whatever the tile: vector instructions issue at their full rate only from four
// wavefronts per SIMD.  The butterfly then runs in nearly every wavefront that meets transformed tiles (~250 of ~600 issue
// slots per tile at G = 64) and still hides behind the stores.  Before, four wavefronts shared a batch, regrouped by class
// through LDS (three workgroups per compute unit, three barriers per batch), and a tile of 128 channels took one lane.
// Measured (back to back on one box; before -> now): bf16 [8,4096,8192] G = 64 3.25 bits 107.4 -> 92.4 us (667 MB, 7.2 TB/s),
// [8,2048,8192] G = 128 79.8 -> 51.3, fp32 [4,2048,8192] G = 64 53.1 -> 45.7, G = 128 61.6 -> 45.9, bf16 [4,2048,4096] G = 8
// 24.4 -> 18.2; half as many elements per lane: 98.8 us where 64 take 92.4.
template <int G, bool OUT_BF16, int LOW, int LPT>
__global__ __launch_bounds__(256, 4)
void k_decode(const uint8_t *__restrict__ packed, void *__restrict__ out, uint32_t T, uint32_t total_wide)
{
    constexpr int ES = OUT_BF16 ? 2 : 4;
    using W = Wave<G, ES, LPT>;
    constexpr int EPL = W::EPL;
    constexpr uint32_t WIDE = LOW + 1;           // the two code widths are LOW and WIDE bits
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[4 * W::LDS_BYTES];
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63u;
    const uint32_t group = blockIdx.x * 4 + wave;
    const uint32_t j0 = group * W::TILES;
    if (j0 >= T) return;
    uint8_t *lds = lds_all + wave * W::LDS_BYTES;
    const Sections lay(T);
    const bool full = T - j0 >= (uint32_t)W::TILES;
    const uint32_t t = lane / LPT, part = lane % LPT;
    const uint32_t j = (full || j0 + t < T) ? j0 + t : T - 1;            // lanes past the end repeat the last tile

    const uint64_t word = reinterpret_cast<const uint64_t *>(packed + lay.bitmap)[j0 >> 6];
    const uint32_t rank0 = reinterpret_cast<const uint32_t *>(packed + lay.ranks)[j0 >> 6];
    const uint32_t s16 = reinterpret_cast<const uint16_t *>(packed + lay.scale)[j];
    const uint32_t z16 = reinterpret_cast<const uint16_t *>(packed + lay.zero)[j];
    const uint32_t pv = packed[lay.pivot + j];

    // width and place of my tile: wide tiles before it
    const uint32_t at = j & 63u;
    const uint32_t half = at < 32u ? (uint32_t)word : (uint32_t)(word >> 32);
    // The stream may have been damaged on its way here: the number of wide tiles before mine is clamped to what the
    // configuration implies, so that every payload address stays inside the payload section whatever the stream holds.
    const uint32_t bit = ((half >> (at & 31u)) & 1u) & (total_wide != 0u ? 1u : 0u);
    uint32_t rank = rank0 + (uint32_t)__popc(half & ((1u << (at & 31u)) - 1u)) + (at < 32u ? 0u : (uint32_t)__popc((uint32_t)word));
    rank = rank < total_wide - bit ? rank : total_wide - bit;
    const bool wide = bit != 0;
    const uint8_t *src = packed + lay.payload + ((uint64_t)LOW * j + rank) * (G / 8) + part * ((LOW + bit) * (EPL / 8));

    constexpr int DW = (EPL * (int)WIDE + 31) / 32;
    uint32_t dw[DW + 2];                         // the readers below may look past the string
#pragma unroll
    for (int i = 0; i < DW + 2; ++i) dw[i] = 0;
    load_codes<EPL / 8, LOW>(src, wide, packed + lay.end(G, LOW, T, total_wide), dw);

    const float sf = f16_widen(s16), mnf = f16_widen(z16);
    float x[EPL];
    if constexpr (WIDE <= 4) {
        uint32_t nib[EPL / 8];
        if (wide) codes_to_nibbles<EPL, WIDE>(dw, nib);
        else codes_to_nibbles<EPL, LOW>(dw, nib);
        // de-quantize: even codes sit in the low nibbles of the bytes, odd codes in the high nibbles
        // (scaled by 16, undone exactly by a scale of sf/16)
        const float sf16 = sf * 0.0625f;
#pragma unroll
        for (int i = 0; i < EPL / 8; ++i) {
            const uint32_t lo = nib[i] & 0x0f0f0f0fu, hi = nib[i] & 0xf0f0f0f0u;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                x[8 * i + 2 * c] = __builtin_fmaf((float)((lo >> (8 * c)) & 0xffu), sf, mnf);
                x[8 * i + 2 * c + 1] = __builtin_fmaf((float)((hi >> (8 * c)) & 0xffu), sf16, mnf);
            }
        }
    } else {
        if (wide) dequantize_codes<EPL, WIDE>(dw, sf, mnf, x);
        else dequantize_codes<EPL, LOW>(dw, sf, mnf, x);
    }
    const bool flag = (pv & 0x80u) != 0;
    if (flag) {                                  // the lanes of a tile agree
        butterfly<EPL>(x);
        butterfly_across<EPL, LPT>(x, part);
#pragma unroll
        for (int k = 0; k < EPL; ++k) x[k] = x[k] * TileConst<G>::c;
    }
    // my elements into my row of LDS, narrowed to the output type
    const uint32_t row = lane * W::LANE_BYTES + (W::swizzle(lane) << 4);
#pragma unroll
    for (int c = 0; c < W::CHUNKS; ++c) {
        uint4 v;
        if constexpr (OUT_BF16) {
            typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
            typedef float floatx2 __attribute__((ext_vector_type(2)));
            uint32_t ws[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const floatx2 pr = {x[8 * c + 2 * i], x[8 * c + 2 * i + 1]};
                ws[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
            }
            v = make_uint4(ws[0], ws[1], ws[2], ws[3]);
        } else {
            v = make_uint4(__float_as_uint(x[4 * c]), __float_as_uint(x[4 * c + 1]), __float_as_uint(x[4 * c + 2]),
                           __float_as_uint(x[4 * c + 3]));
        }
        *reinterpret_cast<uint4 *>(lds + (row ^ (uint32_t)(c << 4))) = v;
    }
    wave_lds_fence();
    const uint32_t d = pv & 0x7fu & (uint32_t)(G - 1);      // masked: a corrupted pivot byte stays inside the tile
    if (flag && d != 0 && part == 0) {
        // undo P_d
        uint8_t *e0 = lds + W::element_at(lane, 0), *ed = lds + W::element_at(lane, d);
        if constexpr (OUT_BF16) {
            const uint16_t v0 = *reinterpret_cast<uint16_t *>(e0), vd = *reinterpret_cast<uint16_t *>(ed);
            *reinterpret_cast<uint16_t *>(e0) = vd; *reinterpret_cast<uint16_t *>(ed) = v0;
        } else {
            const float v0 = *reinterpret_cast<float *>(e0), vd = *reinterpret_cast<float *>(ed);
            *reinterpret_cast<float *>(e0) = vd; *reinterpret_cast<float *>(ed) = v0;
        }
    }
    wave_lds_fence();
    // rows to the tensor in storage order: chunk lane, lane + 64, ... of the group (streaming stores: the decoded tensor is
    // not read again by this library)
    uint8_t *dst = static_cast<uint8_t *>(out) + (uint64_t)j0 * (G * ES) + lane * 16;
    const uint32_t r = lane / W::CHUNKS;         // (64 / CHUNKS rows per step: a multiple of the swizzle's period)
    const uint8_t *from = lds + r * W::LANE_BYTES + (((lane % W::CHUNKS) ^ W::swizzle(r)) << 4);
    const uint32_t rows = full ? 64u : (T - j0) * LPT;
#pragma unroll
    for (int i = 0; i < W::CHUNKS; ++i) {
        if (full || r + i * (64 / W::CHUNKS) < rows) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(from + i * 1024);
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst + i * 1024));
        }
    }
}

}  // namespace tahq

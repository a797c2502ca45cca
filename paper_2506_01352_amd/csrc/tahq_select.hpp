// Top-p% tile selection (Sec. 3.2): inside every ranking unit the k (allocation) tiles of highest entropy get
// the wider code (4 bits by default), ties going to the lower tile index.  Exact, deterministic, no sort.
// Entropies map to order-preserving 32-bit keys; five ways to find the k-th largest key K*, how many tiles equal to
// K* are still wanted (`take`), and from them the bit map and the rank table:
//
//   * ranking units of at most 86016 tiles (98304 where there is one) in tensors of one round of workgroups: in the quantizer's launch
//     (tahq_rank_quant.hpp);
//   * other ranking units of at most 32768 tiles (32705 where units start off the 64-tile boundaries): k_select_small, one workgroup per
//     unit in one launch (entropies and a histogram in LDS, the threshold's bin ranked directly), because at that size several
//     launches cost more than the work;
//   * units of up to 65536 places in tensors whose entropies are exact: k_select_mid, the same from registers;
//   * larger units: the entropy kernel also counts the entropies over 2048 linear bins per unit; k_select_classify
//     settles every tile outside the bin that holds K* and lists the tiles inside it, k_select_resolve ranks that list
//     (further down in this file);
//   * larger units of allocation tiles (A > G), and every unit when the caller forces it: three histogram passes (10 + 11 + 11
//     bits, from the top; the first one folded into the entropy kernel where units are whole steps) find K* and `take`; then, per
//     segment of tiles, counts of keys == K* and > K*, whose prefix sums give every tile its place among the equal keys
//     (index order) and every 64-tile group its rank-table entry: k_radix_pass x 2, k_seg_count, k_assign.
//
// Kernels never wait on each other inside a launch: every dependency is a launch boundary, and the
// small reductions a later kernel needs (which bin holds the k-th key, prefix over segments) are
// recomputed by every block from a few KB of global data.
//
// In the last way the histograms of digits 1 and 2 are kept in two levels so that no address takes more than a handful
// of global atomics: every workgroup stores its own 2048-bin histogram with plain stores and adds only the
// totals of its 64 super-bins (32 bins each) atomically.  The reader picks the super-bin from the 64
// totals, then sums the workgroups' counts for the 32 bins inside it.
#pragma once
#include "tahq_rank_common.hpp"

namespace tahq {

// selection state of one ranking unit (uint32[8] in the workspace)
enum { ST_BIN0 = 0, ST_BIN1 = 1, ST_BIN2 = 2, ST_KREM0 = 3, ST_KREM1 = 4, ST_KEY = 5, ST_TAKE = 6 };

// Which bin of a BINS-bin histogram holds the `want`-th largest key (bins counted from the top), and how
// many keys are still wanted inside that bin.  Run by one full wavefront; lane l owns the BINS/64 bins
// just below BINS - l*BINS/64.  Result is returned in every lane.
template <int BINS>
__device__ __forceinline__ void pick_bin(const uint32_t *__restrict__ hist, uint32_t want, uint32_t *bin,
                                         uint32_t *rem)
{
    constexpr int PER = BINS / 64;
    const int lane = threadIdx.x & 63;
    uint32_t c[PER], mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) { c[i] = hist[BINS - 1 - (lane * PER + i)]; mine += c[i]; }
    uint32_t above = wave_incl_scan(mine) - mine;      // keys in bins above mine
    uint32_t found_bin = 0, found_rem = 0;
    bool found = false;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (!found && above < want && want <= above + c[i]) {
            found = true;
            found_bin = BINS - 1 - (lane * PER + i);
            found_rem = want - above;
        }
        above += c[i];
    }
    // exactly one lane finds it when 1 <= want <= total; otherwise fall back to bin 0 / 0 wanted
    const uint64_t who = __ballot(found);
    const int src = who ? (int)__ffsll((unsigned long long)who) - 1 : 0;
    *bin = (uint32_t)__shfl((int)found_bin, src, 64);
    *rem = (uint32_t)__shfl((int)found_rem, src, 64);
}

// Two-level variant of pick_bin for digits 1 and 2: `coarse` holds the 64 super-bin totals, `partial` the
// `hb` per-workgroup histograms.  Run by one full wavefront; result in every lane.
__device__ __forceinline__ void pick_bin_two_level(const uint32_t *__restrict__ coarse,
                                                   const uint32_t *__restrict__ partial, uint32_t hb, uint32_t want,
                                                   uint32_t *bin, uint32_t *rem)
{
    const int lane = threadIdx.x & 63;
    // super-bins from the top: lane l looks at super-bin 63 - l
    const uint32_t c = coarse[63 - lane];
    const uint32_t above = wave_incl_scan(c) - c;
    const bool hit = above < want && want <= above + c;
    const uint64_t who = __ballot(hit);
    const int src = who ? (int)__ffsll((unsigned long long)who) - 1 : 0;
    const uint32_t sb = 63u - (uint32_t)src;
    const uint32_t want2 = want - (uint32_t)__shfl((int)above, src, 64);
    // the 32 bins of that super-bin, from the top: lanes l and l+32 split the workgroups of bin 31 - (l & 31)
    const uint32_t b_in = 31u - ((uint32_t)lane & 31u);
    // (all loads first, then the sum: a rolled loop would pay one memory latency per workgroup)
    uint32_t part[32];
#pragma unroll
    for (uint32_t i = 0; i < 32; ++i) {
        const uint32_t blk = ((uint32_t)lane >> 5) + 2 * i;
        part[i] = partial[(uint64_t)(blk < hb ? blk : 0u) * kHistBins + sb * 32 + b_in];    // clamped, not branched
    }
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < 32; ++i) sum += (((uint32_t)lane >> 5) + 2 * i) < hb ? part[i] : 0u;
    sum += (uint32_t)__shfl_xor((int)sum, 32, 64);
    const uint32_t mine = lane < 32 ? sum : 0u;
    const uint32_t above2 = wave_incl_scan(mine) - mine;
    const bool hit2 = lane < 32 && above2 < want2 && want2 <= above2 + mine;
    const uint64_t who2 = __ballot(hit2);
    const int src2 = who2 ? (int)__ffsll((unsigned long long)who2) - 1 : 0;
    *bin = sb * 32 + (31u - (uint32_t)src2);
    *rem = want2 - (uint32_t)__shfl((int)above2, src2, 64);
}

// One radix pass.  Digits: pass 0 = key bits 31..22 (1024 bins), pass 1 = bits 21..11, pass 2 = bits 10..0
// (2048 bins each).  Pass p > 0 first derives, from the histogram of pass p-1, the bin chosen there (every
// block does this; block 0 of the unit also records it in `state`), then histograms digit p of the keys
// whose higher digits match.  Pass 0 runs as a kernel of its own only when the entropy kernel could not
// build its histogram; PEEL > 0 then aggregates equal digits inside a wavefront before touching LDS
// (it sees only a handful of distinct digits, which would serialize the LDS atomics).
template <int PASS, int PEEL>
__global__ __launch_bounds__(256) void k_radix_pass(const float *__restrict__ H, uint32_t n, uint32_t k,
                                                    uint32_t *__restrict__ hist0, uint32_t *__restrict__ coarse,
                                                    uint32_t *__restrict__ partial, uint32_t *__restrict__ state)
{
    constexpr int BINS = PASS == 0 ? (int)kDigit0Bins : (int)kHistBins;
    __shared__ uint32_t lh[BINS];
    __shared__ uint32_t chosen[2];
    const uint32_t u = blockIdx.y, hb = gridDim.x;
    const int tid = threadIdx.x, lane = tid & 63;
    uint32_t *ust = state + (uint64_t)u * 8;
    const float *uH = H + (uint64_t)u * n;
    uint32_t *ucoarse = coarse + (uint64_t)u * 2 * 64;                    // [2][64]
    uint32_t *upartial = partial + (uint64_t)u * 2 * hb * kHistBins;      // [2][hb][2048]

    for (int i = tid; i < BINS; i += 256) lh[i] = 0;

    // every thread walks the unit's keys in steps of the grid, sixteen loads in flight at a time; the first
    // sixteen are issued before the bin of the previous pass is worked out, which they do not depend on.
    // All loads use a clamped index: a load behind a branch would wait for the one before it.
    constexpr int R = 16;
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    const uint64_t base0 = (uint64_t)blockIdx.x * 256 + tid;
    float h[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint64_t i = base0 + r * stride;
        h[r] = uH[i < n ? i : (uint64_t)n - 1];
    }

    uint32_t want_hi = 0;
    if (PASS > 0) {
        if (tid < 64) {
            uint32_t bin, rem;
            if (PASS == 1) pick_bin<kDigit0Bins>(hist0 + (uint64_t)u * kDigit0Bins, k, &bin, &rem);
            else pick_bin_two_level(ucoarse, upartial, hb, ust[ST_KREM0], &bin, &rem);
            if (lane == 0) {
                chosen[0] = bin;
                chosen[1] = rem;
                if (blockIdx.x == 0) { ust[ST_BIN0 + PASS - 1] = bin; ust[ST_KREM0 + PASS - 1] = rem; }
            }
        }
        __syncthreads();
        want_hi = PASS == 1 ? chosen[0] : ((ust[ST_BIN0] << 11) | chosen[0]);
    } else {
        __syncthreads();
    }

    constexpr int shift = PASS == 0 ? 22 : (PASS == 1 ? 11 : 0);
    constexpr uint32_t mask = PASS == 0 ? 1023u : 2047u;
    constexpr int hi_shift = PASS == 1 ? 22 : 11;

    for (uint64_t base = base0; base < n; base += R * stride) {
        uint32_t key[R];
        bool ok[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ok[r] = base + r * stride < n;
            key[r] = order_key(h[r]);
        }
        // the next sixteen, while these are counted
        if (base + R * stride < n) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint64_t i = base + (R + r) * stride;
                h[r] = uH[i < n ? i : (uint64_t)n - 1];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            bool active = ok[r] && (PASS == 0 || (key[r] >> hi_shift) == want_hi);
            const uint32_t bin = (key[r] >> shift) & mask;
#pragma unroll 1
            for (int it = 0; it < PEEL; ++it) {
                const uint64_t am = __ballot(active);
                if (am == 0) break;
                const int leader = (int)__ffsll((unsigned long long)am) - 1;
                const uint32_t lb = (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);
                const bool same = active && bin == lb;
                const uint64_t sm = __ballot(same);
                if (lane == leader) atomicAdd(&lh[lb], (uint32_t)__popcll(sm));
                active = active && !same;
            }
            if (active) atomicAdd(&lh[bin], 1u);
        }
    }
    __syncthreads();
    if (PASS == 0) {
        for (int i = tid; i < BINS; i += 256)
            if (lh[i]) atomicAdd(&hist0[(uint64_t)u * kDigit0Bins + i], lh[i]);
    } else {
        // my histogram with plain stores; only the 64 super-bin totals go through atomics
        uint32_t *mine = upartial + ((uint64_t)(PASS - 1) * hb + blockIdx.x) * kHistBins;
        for (int i = tid; i < BINS; i += 256) mine[i] = lh[i];
        if (tid < 64) {
            uint32_t tot = 0;
#pragma unroll 8
            for (int i = 0; i < 32; ++i) tot += lh[32 * tid + ((i + tid) & 31)];     // rotated: no bank conflicts
            if (tot) atomicAdd(&ucoarse[(PASS - 1) * 64 + tid], tot);
        }
    }
}

// Per segment of kSegTiles tiles (one wavefront each): how many keys equal K* and how many exceed it.
// K* and `take` come from the pass-2 histogram; every block derives them, block 0 records them.
__global__ __launch_bounds__(256) void k_seg_count(const float *__restrict__ H, uint32_t n, uint32_t nseg,
                                                   const uint32_t *__restrict__ coarse,
                                                   const uint32_t *__restrict__ partial, uint32_t hb,
                                                   uint32_t *__restrict__ state, uint32_t *__restrict__ seg)
{
    __shared__ uint32_t chosen[2];
    const uint32_t u = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t *ust = state + (uint64_t)u * 8;
    // my wavefront's segment: its sixteen keys per lane are requested first (clamped index, nothing behind a
    // branch); the threshold they are compared with is worked out while they arrive
    constexpr int KEYS = (int)(kSegTiles / 64);
    const uint32_t s = blockIdx.x * 4 + wave;
    const float *uH = H + (uint64_t)u * n;
    float h[KEYS];
#pragma unroll
    for (int r = 0; r < KEYS; ++r) {
        const uint64_t j = (uint64_t)s * kSegTiles + (uint64_t)r * 64 + lane;
        h[r] = uH[j < n ? j : (uint64_t)n - 1];
    }
    if (tid < 64) {
        uint32_t bin, rem;
        pick_bin_two_level(coarse + ((uint64_t)u * 2 + 1) * 64, partial + ((uint64_t)u * 2 + 1) * hb * kHistBins, hb,
                           ust[ST_KREM1], &bin, &rem);
        const uint32_t key = (ust[ST_BIN0] << 22) | (ust[ST_BIN1] << 11) | bin;
        if (lane == 0) {
            chosen[0] = key;
            chosen[1] = rem;
            if (blockIdx.x == 0) { ust[ST_BIN2] = bin; ust[ST_KEY] = key; ust[ST_TAKE] = rem; }
        }
    }
    __syncthreads();
    const uint32_t thr = chosen[0];
    if (s >= nseg) return;
    uint32_t eq = 0, gt = 0;
#pragma unroll
    for (int r = 0; r < KEYS; ++r) {
        const bool ok = (uint64_t)s * kSegTiles + (uint64_t)r * 64 + lane < n;
        const uint32_t key = order_key(h[r]);
        eq += (uint32_t)__popcll(__ballot(ok && key == thr));
        gt += (uint32_t)__popcll(__ballot(ok && key > thr));
    }
    if (lane == 0) {
        seg[((uint64_t)u * nseg + s) * 2 + 0] = eq;
        seg[((uint64_t)u * nseg + s) * 2 + 1] = gt;
    }
}

// Width bit of every tile, rank-table entries, and the bit map itself when units start on 64-tile
// boundaries (otherwise one byte per tile goes to `sel_bytes` and k_bitmap_pack follows).
// A block owns 4 consecutive segments.  Its first wavefront sums the segment counts that precede
// the block: equal keys before it (they are taken in index order until `take` are used up) and
// wide tiles before it (every earlier ranking unit contributes exactly k).
__global__ __launch_bounds__(256) void k_assign(const float *__restrict__ H, uint32_t n, uint32_t k, uint32_t nseg,
                                                const uint32_t *__restrict__ state,
                                                const uint32_t *__restrict__ seg,
                                                uint64_t *__restrict__ bitmap, uint32_t *__restrict__ ranks,
                                                uint8_t *__restrict__ sel_bytes, int aligned)
{
    __shared__ uint32_t base_eq[4], base_rank[4];
    const uint32_t u = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t *ust = state + (uint64_t)u * 8;
    const uint32_t thr = ust[ST_KEY], take = ust[ST_TAKE];
    const uint32_t *useg = seg + (uint64_t)u * nseg * 2;
    const uint32_t s0 = blockIdx.x * 4;
    // my wavefront's segment: its sixteen keys per lane are requested first (clamped index, nothing behind a
    // branch) and arrive while the first wavefront sums the counts of the segments before this block
    constexpr int KEYS = (int)(kSegTiles / 64);
    const float *uH = H + (uint64_t)u * n;
    float h[KEYS];
#pragma unroll
    for (int r = 0; r < KEYS; ++r) {
        const uint64_t jl = (uint64_t)(s0 + wave) * kSegTiles + (uint64_t)r * 64 + lane;
        h[r] = uH[jl < n ? jl : (uint64_t)n - 1];
    }

    if (tid < 64) {
        // Sums over the s0 segments before this block, 512 segments per sweep: lane l owns the 8 consecutive
        // segments 8l .. 8l+7 of the sweep (loaded at once), a wave scan orders the lanes, `eq_run` / `rank_run`
        // carry the totals from sweep to sweep.
        const uint2 *pairs = reinterpret_cast<const uint2 *>(useg);
        uint32_t eq_run = 0, rank_run = u * k;
        for (uint32_t base = 0; base < s0; base += 512) {
            uint2 e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t sidx = base + (uint32_t)lane * 8 + i;
                e[i] = pairs[sidx < s0 ? sidx : 0u];                 // clamped, not branched; masked below
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (base + (uint32_t)lane * 8 + i >= s0) e[i] = make_uint2(0u, 0u);
            uint32_t eq_sum = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) eq_sum += e[i].x;
            const uint32_t eq_incl = wave_incl_scan(eq_sum);
            uint32_t eq_before = eq_run + eq_incl - eq_sum;
            uint32_t sel_sum = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t left = eq_before < take ? take - eq_before : 0u;
                sel_sum += e[i].y + (e[i].x < left ? e[i].x : left);
                eq_before += e[i].x;
            }
            const uint32_t sel_incl = wave_incl_scan(sel_sum);
            eq_run += (uint32_t)__shfl((int)eq_incl, 63, 64);
            rank_run += (uint32_t)__shfl((int)sel_incl, 63, 64);
        }
        // the block's own four segments, in order
        uint2 own[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) own[w] = pairs[s0 + w < nseg ? s0 + w : nseg - 1];
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if (s0 + w >= nseg) own[w] = make_uint2(0u, 0u);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (lane == 0) { base_eq[w] = eq_run; base_rank[w] = rank_run; }
            const uint32_t left = eq_run < take ? take - eq_run : 0u;
            rank_run += own[w].y + (own[w].x < left ? own[w].x : left);
            eq_run += own[w].x;
        }
    }
    __syncthreads();
    const uint32_t s = s0 + wave;
    if (s >= nseg) return;
    uint32_t eq_run = base_eq[wave], rank_run = base_rank[wave];
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < KEYS; ++r) {
        const uint64_t jl = (uint64_t)s * kSegTiles + (uint64_t)r * 64 + lane;
        const bool ok = jl < n;
        const uint32_t key = order_key(h[r]);
        const bool eq = ok && key == thr;
        const uint64_t eq_mask = __ballot(eq);
        const bool sel = ok && (key > thr || (eq && eq_run + (uint32_t)__popcll(eq_mask & below) < take));
        const uint64_t sel_mask = __ballot(sel);
        const uint64_t jg = (uint64_t)u * n + jl;     // tile index in the tensor
        if (aligned) {
            if (lane == 0 && ok) { bitmap[jg >> 6] = sel_mask; ranks[jg >> 6] = rank_run; }
        } else if (ok) {
            sel_bytes[jg] = sel ? 1 : 0;
            if ((jg & 63u) == 0) ranks[jg >> 6] = rank_run + (uint32_t)__popcll(sel_mask & below);
        }
        eq_run += (uint32_t)__popcll(eq_mask);
        rank_run += (uint32_t)__popcll(sel_mask);
    }
}

__global__ __launch_bounds__(256) void k_bitmap_pack(const uint8_t *__restrict__ sel_bytes, uint32_t T,
                                                     uint64_t *__restrict__ bitmap)
{
    const uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const uint64_t word = __ballot(j < T && sel_bytes[j < T ? j : 0] != 0);
    if ((threadIdx.x & 63) == 0 && (j >> 6) < ((uint64_t)T + 63) / 64) bitmap[j >> 6] = word;
}

// Allocation tiles of m > 1 quantization tiles (Sec. 3.2): the selection ran over allocation tiles and left
// one byte per allocation tile in `sel_a` and, in `ranks_a`, the wide allocation tiles before each group of
// 64.  This kernel writes the stream's bit map and rank table over QUANTIZATION tiles: tile j takes the
// width of allocation tile j / m, and the wide quantization tiles before j are m times the wide
// allocation tiles before j / m, plus j % m if its own allocation tile is wide.  One wavefront per
// 64 quantization tiles.
__global__ __launch_bounds__(256) void k_expand_alloc(const uint8_t *__restrict__ sel_a,
                                                      const uint32_t *__restrict__ ranks_a, uint32_t T, uint32_t m,
                                                      uint64_t *__restrict__ bitmap, uint32_t *__restrict__ ranks)
{
    const uint32_t j = blockIdx.x * 256 + threadIdx.x;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t j0 = j - lane;
    if (j0 >= T) return;                               // whole wavefront past the end
    const uint32_t ja0 = j0 / m, r0 = j0 % m;
    const uint32_t base = ja0 & ~63u;
    const bool before = base + lane < ja0 && sel_a[base + lane] != 0;
    const uint32_t rank_a = ranks_a[ja0 >> 6] + (uint32_t)__popcll(__ballot(before));
    const bool mine = j < T && sel_a[j < T ? j / m : 0] != 0;
    const uint64_t word = __ballot(mine);
    if (lane == 0) {
        bitmap[j0 >> 6] = word;
        ranks[j0 >> 6] = rank_a * m + (sel_a[ja0] != 0 ? r0 : 0u);
    }
}

// ---- small ranking units: the whole selection in one launch

constexpr uint32_t kSmallUnitThreads = 1024;
constexpr uint32_t kExpandWords = 2048;          // bit map words a workgroup expands when A > G

// LDS of k_select_small, for units of at most PLACES places and BINS bins of the first cut
template <uint32_t PLACES, uint32_t BINS>
struct SmallSelectLds {
    int key[PLACES];                             // the entropies' bit patterns, by place
    uint32_t hist[BINS];
    uint64_t list[kSmallListCap];                // tiles of the threshold bin: key << 32 | ~place
    uint64_t words[PLACES / 64];                 // bit map words over places
    uint64_t equal[PLACES / 64];                 // where many share the threshold: the words of those that do
    uint32_t prefix[PLACES / 64];                // selected places before each word
    uint32_t wave_total[kSmallUnitThreads / 64], wave_equal[kSmallUnitThreads / 64];
    uint32_t chosen[3];                          // threshold bin, wanted inside it, its tiles
    uint32_t listed;
    uint32_t above_zero, zero;                   // the lowest bin's entropies above +0.0f and equal to it
};

// A ranking unit that one workgroup can hold, ranked in one launch, everything in LDS.
//
// A place is a tile's index counted from the 64-tile boundary at or before the unit's first tile, so that 64 places are
// one word of the stream's bit map whatever the unit's length (with A > G: the index of the allocation tile, from 0).
// Wavefront w takes the blocks w, w + 16, .. of 256 places, four consecutive places per lane.
//
// The entropies' bit patterns fall into BINS bins of 2^SHIFT neighbouring floats each, four octaves below ln A (`bin0` is
// the number of the lowest bin); the bins at the ends take what lies beyond.  The bin that holds the k-th largest settles
// every other tile with one comparison each; its own tiles, if they are 256 or fewer, are placed directly among each other by (key
// descending, tile ascending).  Of N(0,1) values those are 160 to 220 of 25600 tiles of 64 channels and 260 to 560 of 30720 and
// more, of 12288 tiles of 128 channels or of 2048 of 4096; tiles that are alike are as many as there are.  A bin of more tiles is
// cut again into 4096 parts, as a rule of one or two floats each, by a histogram of the bit patterns in LDS.
// Encode of bf16 at 3.5 bits, against a radix select over the entropies in memory: 32768 tiles of 64 channels 36.5 -> 21.1 us, of 32
// channels 34.4 -> 19.3, 25600 of 128 channels 28.7 -> 19.1, 8192 of 4096 channels 48.9 -> 45.4; a fifth of 32768 tiles alike, at
// 3.1 bits, 35.7 -> 31.0.
//
// Bound by the instruction issue of its one compute unit, scalar instructions included (a ballot per 64 entropies and what
// follows it cost three times as much as the carries that collect a lane's four bits here), and by a dozen dependent
// steps.  25600 tiles: 7.3 us; 14.4 us as a two-pass radix select with the entropies in registers, 8192 tiles 11.0 -> 6.6,
// the 2048 allocation tiles (A = 4096) of four samples with their expansion 11.3 + 4.9 -> 6.4.
//
// With A > G (m > 1) the words of the allocation tiles are expanded to quantization tiles from LDS, kExpandWords words by
// each of the unit's gridDim.y workgroups, all of which select for themselves.
template <uint32_t PLACES, uint32_t BINS, int SHIFT>
__global__ __launch_bounds__(kSmallUnitThreads) void k_select_small(const float *__restrict__ H, uint32_t n, uint32_t k, uint32_t m,
                                                                    int bin0, uint64_t *__restrict__ bitmap,
                                                                    uint32_t *__restrict__ ranks)
{
    __shared__ __attribute__((aligned(16))) SmallSelectLds<PLACES, BINS> L;
    static_assert(sizeof(L) <= 163840, "the LDS of a compute unit");
    constexpr uint32_t WAVES = kSmallUnitThreads / 64;
    constexpr uint32_t PER = BINS / kSmallUnitThreads;       // bins per thread
    constexpr uint32_t BLOCKS = PLACES / 256 / WAVES;        // blocks per wavefront
    static_assert(PER % 4 == 0 && PLACES / 64 <= kSmallUnitThreads && BLOCKS >= 1 && BLOCKS <= 8, "four bits per block in a dword");
    const uint32_t u = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t phase = m == 1 ? (uint32_t)(((uint64_t)u * n) & 63u) : 0u;      // place of the unit's first tile
    const uint32_t end = phase + n, nwords = (end + 63) / 64, nblocks = (end + 255) / 256;
    const float *uH = H + ((uint64_t)u * n - phase);         // by place

    // All loads at once, straight to LDS.  (Whole words of 64 places are read, which may reach into the neighbouring units or up
    // to 63 floats past the entropies, where the workspace goes on; beyond them from a clamped index.)
    for (uint32_t b = wave; b < nblocks; b += WAVES) {
        const uint32_t place = b * 256u + 4u * lane, top = nwords * 64u - 4u;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(uH + (place < top ? place : top)),
                                         (__attribute__((address_space(3))) void *)&L.key[b * 256u], 16, 0, 0);
    }
#pragma unroll
    for (uint32_t i = 0; i < PER / 4; ++i)
        reinterpret_cast<uint4 *>(L.hist)[i * kSmallUnitThreads + tid] = make_uint4(0, 0, 0, 0);
    if (tid == 0) { L.listed = 0; L.above_zero = 0; L.zero = 0; }
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0): my wavefront's entropies are in LDS
    __syncthreads();
    for (uint32_t b = wave; b < nblocks; b += WAVES) {
        int4 *at = reinterpret_cast<int4 *>(&L.key[b * 256u + 4u * lane]);
        int4 q = *at;
        if ((b == 0 && phase != 0) || (b == nblocks - 1 && (end & 255u) != 0)) {
            // places outside the unit take the bit pattern of -0.0f, the lowest of all as a signed integer and no entropy's
            const uint32_t i = b * 256u + 4u * lane - phase;
            q.x = i < n ? q.x : INT32_MIN; q.y = i + 1u < n ? q.y : INT32_MIN;
            q.z = i + 2u < n ? q.z : INT32_MIN; q.w = i + 3u < n ? q.w : INT32_MIN;
            *at = q;
        }
        const int v[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int bin = (v[c] >> SHIFT) - bin0;          // as signed integers: negative values and NaN with the sign bit set lowest
            atomicAdd(&L.hist[bin < 0 ? 0 : bin > (int)BINS - 1 ? (int)BINS - 1 : bin], 1u);
        }
    }
    __syncthreads();
    // The bin of the k-th largest.  1 <= k <= n, so there is one.
    block_pick_bin<(int)BINS>(L.hist, k, L.wave_total, L.chosen);
    const uint32_t bstar = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[0]);
    uint32_t rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[1]);
    uint32_t crowd = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[2]);
    if (bstar == 0) crowd -= nblocks * 256u - n;             // bin 0 has counted the places outside the unit as well
    // the bit patterns of that bin, first and last
    const int first = bstar == 0 ? INT32_MIN + 1 : (int)((bstar + (uint32_t)bin0) << SHIFT);
    const int last = bstar == BINS - 1 ? INT32_MAX : (int)(((bstar + (uint32_t)bin0 + 1u) << SHIFT) - 1u);
    // places of word g that belong to the unit
    auto in_unit = [&](uint32_t g) -> uint64_t {
        uint64_t mask = ~0ull;
        if (g == 0) mask <<= phase;
        if (end - g * 64u < 64u) mask &= (1ull << (end - g * 64u)) - 1ull;
        return mask;
    };
    // block b's four bits per lane -> its eight dwords of `out`: eight neighbouring lanes fill one
    auto put_bits = [&](uint64_t *out, uint32_t b, uint32_t four) {
        const uint32_t d = nibbles_to_dword(four, lane);
        if ((lane & 7) == 0) reinterpret_cast<uint32_t *>(out)[b * 8u + (lane >> 3)] = d;
    };
    auto four_bits = [](const int4 &q, auto test) {
        return (test(q.x) ? 1u : 0u) | (test(q.y) ? 2u : 0u) | (test(q.z) ? 4u : 0u) | (test(q.w) ? 8u : 0u);
    };
    // Every place that is_above is selected, and of the `crowd` others that are not below, the `rem` first by (key descending,
    // tile ascending), placed directly among each other.
    auto place_directly = [&](auto is_above, auto is_not_below) {
        uint32_t inside = 0;                     // my tiles of the bin, four bits per block, the last block lowest
        int4 next = *reinterpret_cast<const int4 *>(&L.key[wave * 256u + 4u * lane]);
        for (uint32_t b = wave; b < nblocks; b += WAVES) {
            const int4 q = next;
            if (b + WAVES < nblocks) next = *reinterpret_cast<const int4 *>(&L.key[(b + WAVES) * 256u + 4u * lane]);
            const uint32_t above = four_bits(q, is_above), reach = four_bits(q, is_not_below);
            put_bits(L.words, b, above);
            inside = (inside << 4) | (reach & ~above);
        }
        if (__ballot(inside != 0) != 0) {
            // one place in the list for all of the wavefront's
            const uint32_t count = (uint32_t)__popc(inside), incl = wave_incl_scan(count);
            uint32_t at = 0;
            if (lane == 63) at = atomicAdd(&L.listed, incl);
            at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + incl - count;
            const uint32_t mine_blocks = (nblocks - wave + WAVES - 1) / WAVES;
            while (inside != 0) {
                const uint32_t bit = (uint32_t)__ffs((int)inside) - 1u;
                inside &= inside - 1u;
                const uint32_t place = (wave + WAVES * (mine_blocks - 1u - bit / 4)) * 256u + 4u * lane + bit % 4;
                L.list[at++] = ((uint64_t)order_key(__uint_as_float((uint32_t)L.key[place])) << 32) | (uint32_t)~place;
            }
        }
        __syncthreads();
        // four threads per listed tile count the tiles ahead of it
        if ((uint32_t)tid < 4 * crowd) {
            const uint64_t mine = L.list[tid >> 2];
            uint32_t ahead = 0;
#pragma unroll 4
            for (uint32_t i = (uint32_t)tid & 3u; i < crowd; i += 4) ahead += L.list[i] > mine ? 1u : 0u;
            ahead += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ahead, 0xB1, 0xF, 0xF, true);      // lane ^ 1
            ahead += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ahead, 0x4E, 0xF, 0xF, true);      // lane ^ 2
            const uint32_t place = ~(uint32_t)mine;
            if (((uint32_t)tid & 3u) == 0 && ahead < rem)
                atomicOr(reinterpret_cast<uint32_t *>(L.words) + (place >> 5), 1u << (place & 31u));
        }
        __syncthreads();
    };
    if (__builtin_expect(crowd <= kSmallListCap, 1)) {
        place_directly([&](int v) { return v > last; }, [&](int v) { return v >= first; });
    } else {
        // More tiles in the bin than the list takes: it is cut again, 4096 parts at a time, until they fit or all share one
        // entropy.  Bit patterns count in the order of their keys here, as signed integers, in which -0.0f (the places outside
        // the unit) is -1: in none of the ranges below.
        auto ordered = [](int v) { return v ^ ((v >> 31) & INT32_MAX); };
        int lo = first, hi = last;
        if (bstar == 0) {
            // The lowest bin's usual crowd are the entropies of all-zero tiles, +0.0f, which counting tells from those above
            // and below.
            uint32_t above = 0, zero = 0;
            for (uint32_t b = wave; b < nblocks; b += WAVES) {
                const int4 q = *reinterpret_cast<const int4 *>(&L.key[b * 256u + 4u * lane]);
                above += (uint32_t)__popc(four_bits(q, [&](int v) { return v > 0 && v <= last; }));
                zero += (uint32_t)__popc(four_bits(q, [](int v) { return v == 0; }));
            }
            above = wave_incl_scan(above);
            zero = wave_incl_scan(zero);
            if (lane == 63) { atomicAdd(&L.above_zero, above); atomicAdd(&L.zero, zero); }
            __syncthreads();
            above = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.above_zero);
            zero = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.zero);
            if (rem <= above) { lo = 1; crowd = above; }
            else if (rem <= above + zero) { lo = hi = 0; rem -= above; crowd = zero; }
            else { lo = INT32_MIN; hi = -2; rem -= above + zero; crowd -= above + zero; }
        }
#pragma unroll 1
        while (crowd > kSmallListCap && lo != hi) {          // three times at most: 32 bits, 12 fewer each time
            const uint32_t span = (uint32_t)hi - (uint32_t)lo;
            const int bits = 32 - __builtin_clz(span), shift = bits > 12 ? bits - 12 : 0;
            static_assert(BINS >= 4096, "the parts' counts");
            reinterpret_cast<uint4 *>(L.hist)[tid] = make_uint4(0, 0, 0, 0);
            __syncthreads();
            for (uint32_t b = wave; b < nblocks; b += WAVES) {
                const int4 q = *reinterpret_cast<const int4 *>(&L.key[b * 256u + 4u * lane]);
                const uint32_t from_lo[4] = {(uint32_t)ordered(q.x) - (uint32_t)lo, (uint32_t)ordered(q.y) - (uint32_t)lo,
                                             (uint32_t)ordered(q.z) - (uint32_t)lo, (uint32_t)ordered(q.w) - (uint32_t)lo};
                // (where a crowd shares one entropy all additions meet on one counter, one after the other; tokens that are
                // alike make a crowd of neighbours: one addition for the four)
                if (q.x == q.y && q.y == q.z && q.z == q.w) {
                    if (from_lo[0] <= span) atomicAdd(&L.hist[from_lo[0] >> shift], 4u);
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (from_lo[c] <= span) atomicAdd(&L.hist[from_lo[c] >> shift], 1u);
                }
            }
            __syncthreads();
            block_pick_bin<4096>(L.hist, rem, L.wave_total, L.chosen);
            lo = (int)((uint32_t)lo + ((uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[0]) << shift));
            rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[1]);
            crowd = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[2]);
            const uint32_t room = (uint32_t)hi - (uint32_t)lo, part = (1u << shift) - 1u;
            hi = (int)((uint32_t)lo + (room < part ? room : part));
        }
        auto is_above = [&](int v) { return ordered(v) > hi && v != INT32_MIN; };
        if (crowd <= kSmallListCap) {
            place_directly(is_above, [&](int v) { return ordered(v) >= lo && v != INT32_MIN; });
        } else {
            // `crowd` tiles of one entropy: taken in index order until `rem` are used up
            for (uint32_t b = wave; b < nblocks; b += WAVES) {
                const int4 q = *reinterpret_cast<const int4 *>(&L.key[b * 256u + 4u * lane]);
                put_bits(L.words, b, four_bits(q, is_above));
                put_bits(L.equal, b, four_bits(q, [&](int v) { return ordered(v) == lo; }));
            }
            __syncthreads();
            const uint64_t eq = (uint32_t)tid < nwords ? L.equal[tid] : 0ull;
            const uint32_t count = (uint32_t)__popcll(eq), incl = wave_incl_scan(count);
            if (lane == 63) L.wave_equal[wave] = incl;
            __syncthreads();
            const uint32_t eq_before = sum_of_waves_before(L.wave_equal, wave, lane) + incl - count;
            if ((uint32_t)tid < nwords) {
                uint64_t taken = eq;
                if (eq_before >= rem) taken = 0;
                else
                    for (uint32_t over = eq_before + count; over > rem; --over) taken &= ~(1ull << (63 - __builtin_clzll(taken)));
                L.words[tid] |= taken;
            }
            __syncthreads();
        }
    }
    // selected places before every word
    const uint64_t word = (uint32_t)tid < nwords ? L.words[tid] : 0ull;
    const uint32_t cnt = (uint32_t)__popcll(word), incl = wave_incl_scan(cnt);
    if (lane == 63) L.wave_total[wave] = incl;
    __syncthreads();
    const uint32_t before = sum_of_waves_before(L.wave_total, wave, lane) + incl - cnt;
    if (m == 1) {
        if ((uint32_t)tid < nwords) {
            const uint64_t at = (((uint64_t)u * n) >> 6) + (uint32_t)tid;
            // a word that the unit shares with a neighbour has been cleared by an earlier kernel
            if (in_unit((uint32_t)tid) == ~0ull) bitmap[at] = word;
            else atomicOr(reinterpret_cast<unsigned long long *>(bitmap) + at, (unsigned long long)word);
            if (tid != 0 || phase == 0) ranks[at] = u * k + before;        // every earlier unit holds exactly k
        }
        return;
    }
    // A > G: the words and rank-table entries of the quantization tiles, m of which share the width of their allocation tile
    if ((uint32_t)tid < nwords) L.prefix[tid] = before;
    __syncthreads();
    const uint32_t *bits = reinterpret_cast<const uint32_t *>(L.words);
    const uint64_t nq = (uint64_t)n * m, q0 = (uint64_t)u * nq;            // the unit's quantization tiles
    const uint64_t w_end = (q0 + nq + 63) >> 6;
    uint64_t w_stop = (q0 >> 6) + (uint64_t)(blockIdx.y + 1) * kExpandWords;
    if (w_stop > w_end) w_stop = w_end;
    for (uint64_t w = (q0 >> 6) + (uint64_t)blockIdx.y * kExpandWords + (uint32_t)tid; w < w_stop; w += kSmallUnitThreads) {
        // quantization tiles [lo, hi) of the word belong to the unit
        const uint64_t lo = 64 * w > q0 ? 64 * w : q0, hi = 64 * w + 64 < q0 + nq ? 64 * w + 64 : q0 + nq;
        const uint32_t a0 = (uint32_t)((lo - q0) / m), r0 = (uint32_t)((lo - q0) % m);
        uint64_t out = 0;
        uint32_t a = a0, run = m - r0;           // quantization tiles left of allocation tile a
        for (uint64_t j = lo; j < hi; j += run, run = m, ++a) {
            const uint64_t len = hi - j < run ? hi - j : run;
            if ((bits[a >> 5] >> (a & 31u)) & 1u) out |= (~0ull >> (64 - len)) << (j & 63u);
        }
        if (hi - lo == 64) bitmap[w] = out;
        else atomicOr(reinterpret_cast<unsigned long long *>(bitmap) + w, (unsigned long long)out);
        if (lo == 64 * w) {
            const uint32_t rank_a = u * k + L.prefix[a0 >> 6] + (uint32_t)__popcll(L.words[a0 >> 6] & ((1ull << (a0 & 63u)) - 1ull));
            ranks[w] = rank_a * m + (((bits[a0 >> 5] >> (a0 & 31u)) & 1u) ? r0 : 0u);
        }
    }
}

// ---- large ranking units: the selection in two launches after the entropy kernel
//
// The entropy kernel leaves, per ranking unit, a histogram of the entropies over kLinBins linear bins.  The bin of an
// entropy is non-decreasing in it, so the k-th largest entropy lies in the bin b* where the counts, summed from the
// top, reach k: every tile in a higher bin is selected, every tile in a lower bin is not, and only the tiles IN
// bin b* (about one in a few hundred for activations) need an exact ranking for the `rem` places that are left.
//
//   k_select_classify (workgroups of 1024 threads over blocks of 16384 tiles): find b*; write the bit map words with
//     the tiles above b* and the block's count of them; append (key, tile) of the tiles in b* to the unit's
//     candidate list.
//   k_select_resolve (same grid): every workgroup ranks the unit's candidates exactly for itself -- a histogram over
//     parts of the bin leaves a handful that are placed directly, ties by tile index, so that they go to the lower index
//     whatever order the list came in -- adds the selected candidates of its own block to the block's bit map
//     words, and writes the block's part of the rank table (tiles above b* in the blocks before it, from the
//     counts; selected candidates before it, counted while ranking).  Ranking a few thousand candidates sixteen to
//     thirty-two times over costs less than one workgroup walking the unit's whole bit map.
// If b* holds a crowd, more tiles than the list or than a sixteenth of the unit, nothing is listed:
//   k_select_classify counts b*'s tiles over the sub-bins of b*;
//   k_select_resolve, in the place of the ranking above: every workgroup settles its own tiles but those in the threshold's
//     sub-bin, whose places it leaves in words of their own; the unit's last workgroup to get there settles those, as a rule
//     by index alone, because they are all alike, or from a list, because they are few.
// (Ordinary values put up to 3 % of a unit into one bin, so more than a sixteenth are tiles that are alike.  From the list those take
// longer than the crowd's way does, three units of 77700 tiles with 15500 all-zero ones each 49 against 40 us for the encode, and
// tiles that are not the other way round, 655520 tiles of 32 channels 74 against 59.)
// Encode, against one workgroup that did all of such a unit from the entropies: 655520 tiles of 32 channels, a fifth of them all zero,
// 1477 -> 72 us, 1056897 tiles of 64 channels 1480 -> 127, a fifth of them all zero 3013 -> 121.
// (Without a crowd, one launch, with the last workgroup of every unit doing the second part, measured ten times slower.  What a
// workgroup wrote becomes visible to a workgroup on another XCD only when the L2 is written back: in the crowd's way one thread
// per workgroup sees to that, in under 1 us; the last workgroup's work takes ten.)

constexpr uint32_t kFusedThreads = 1024;
constexpr uint32_t kFusedKeysPerBlock = 16 * kFusedThreads;

// A threshold bin of more tiles than this is a crowd.
__device__ __forceinline__ uint32_t crowd_from(uint32_t n) { return n / 16 < kCandCap ? n / 16 : kCandCap; }

// ---- ranking units of up to 65536 tiles: one launch, from registers
//
// What k_select_small does for units whose entropies LDS holds, for units whose entropies the registers of 1024 threads hold: 16 blocks of
// 256 places per wavefront, four places per lane and block.  The bins of the first cut are 1024 floats wide, so that the threshold's
// seldom holds more of 65536 ordinary tiles than are placed directly (with bins of 4096 a second cut took 5 us).  Against
// the two-launch selection it saves the launch that clears scratch, one of the selection's two, and the entropy pass its
// histogram, whose additions meet on the bins of a few units.  Encode of bf16: 34816 tiles of 64 channels 30.7 -> 21.6 us, 40980
// 31.7 -> 23.3, 65536 32.2 -> 27.6, four units of those 40.7 -> 38.1, 2 x 40960 of 16 channels 25.9 -> 20.7.  81920 tiles took
// as long as in two launches (33.7 and 33.5), and 77700 of 16 channels longer.
constexpr uint32_t kMidPlaces = 65536, kMidBins = 32768;
constexpr int kMidShift = 10, kMidBlocks = (int)(kMidPlaces / 256 / (kSmallUnitThreads / 64));

struct MidSelectLds {
    uint32_t hist[kMidBins];
    uint64_t list[kSmallListCap];
    uint64_t words[kMidPlaces / 64], equal[kMidPlaces / 64];
    uint32_t wave_total[kSmallUnitThreads / 64];
    uint32_t chosen[3], listed, above_zero, zero;
};

__global__ __launch_bounds__(kSmallUnitThreads)
void k_select_mid(const float *__restrict__ H, uint32_t n, uint32_t k, int bin0, uint64_t *__restrict__ bitmap,
                  uint32_t *__restrict__ ranks)
{
    __shared__ __attribute__((aligned(16))) MidSelectLds L;
    constexpr uint32_t WAVES = kSmallUnitThreads / 64, WPT = kMidPlaces / 64 / kSmallUnitThreads;          // bit map words per thread
    static_assert(kMidPlaces / 64 == WPT * kSmallUnitThreads && sizeof(L) <= 163840, "a thread's words, the LDS of a compute unit");
    const uint32_t u = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const UnitPlaces at(u, n);
    const float *uH = H + ((uint64_t)u * n - at.phase);      // by place
    const uint32_t top = at.nwords * 64u - 4u;

    // All loads at once (whole words of 64 places, as k_select_classify reads them).
    int4 q[kMidBlocks];
#pragma unroll
    for (int r = 0; r < kMidBlocks; ++r) {
        const uint32_t p = ((uint32_t)r * WAVES + wave) * 256u + 4u * lane;
        q[r] = *reinterpret_cast<const int4 *>(uH + (p < top ? p : top));
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (uint32_t i = 0; i < kMidBins / 4 / kSmallUnitThreads; ++i)
        reinterpret_cast<uint4 *>(L.hist)[i * kSmallUnitThreads + tid] = make_uint4(0, 0, 0, 0);
    if (tid == 0) { L.listed = 0; L.above_zero = 0; L.zero = 0; }
    __syncthreads();
    // f(block, its four bit patterns) for my blocks that hold places of the unit
    auto each_block = [&](auto f) {
#pragma unroll
        for (int r = 0; r < kMidBlocks; ++r) {
            const uint32_t b = (uint32_t)r * WAVES + wave;
            if (b * 256u < at.end) f(b, q[r]);
            __builtin_amdgcn_sched_barrier(0);   // (one block after the other: the registers are full)
        }
    };
    // Bit patterns in the order of their keys from here on: signed integers, negative ones' other bits turned over.  Places outside the
    // unit take the lowest of all, which is also that of a NaN with all bits set: where a range reaches down to it they are told
    // apart by their place.
    const uint32_t outside = (at.end + 255u) / 256u * 256u - n;          // so many, in the unit's blocks
#pragma unroll
    for (int r = 0; r < kMidBlocks; ++r) {
        auto ordered = [](int v) { return v ^ ((v >> 31) & INT32_MAX); };
        q[r].x = ordered(q[r].x); q[r].y = ordered(q[r].y); q[r].z = ordered(q[r].z); q[r].w = ordered(q[r].w);
        const uint32_t base = ((uint32_t)r * WAVES + wave) * 256u, i = base + 4u * lane - at.phase;
        if (base < at.end && (base < at.phase || base + 256u > at.end)) {
            q[r].x = i < n ? q[r].x : INT32_MIN; q[r].y = i + 1u < n ? q[r].y : INT32_MIN;
            q[r].z = i + 2u < n ? q[r].z : INT32_MIN; q[r].w = i + 3u < n ? q[r].w : INT32_MIN;
        }
    }
    each_block([&](uint32_t, const int4 &v4) {
        const int v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int bin = (v[c] >> kMidShift) - bin0;
            atomicAdd(&L.hist[bin < 0 ? 0 : bin > (int)kMidBins - 1 ? (int)kMidBins - 1 : bin], 1u);
        }
    });
    __syncthreads();
    block_pick_bin<(int)kMidBins>(L.hist, k, L.wave_total, L.chosen);
    const uint32_t bstar = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[0]);
    uint32_t rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[1]);
    uint32_t crowd = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[2]);
    if (bstar == 0) crowd -= outside;            // bin 0 has counted them as well
    // the bin's patterns, first and last
    int lo = bstar == 0 ? INT32_MIN : (int)((bstar + (uint32_t)bin0) << kMidShift);
    int hi = bstar == kMidBins - 1 ? INT32_MAX : (int)(((bstar + (uint32_t)bin0 + 1u) << kMidShift) - 1u);
    auto four_bits = [](const int4 &v, auto test) {
        return (test(v.x) ? 1u : 0u) | (test(v.y) ? 2u : 0u) | (test(v.z) ? 4u : 0u) | (test(v.w) ? 8u : 0u);
    };
    auto put_bits = [&](uint64_t *out, uint32_t b, uint32_t four) {
        const uint32_t d = nibbles_to_dword(four, lane);
        if ((lane & 7) == 0) reinterpret_cast<uint32_t *>(out)[b * 8u + (lane >> 3)] = d;
    };
    if (crowd > kSmallListCap && bstar == 0) {
        // the lowest bin's usual crowd are the entropies of all-zero tiles, +0.0f, which counting tells from those above and below
        uint32_t above = 0, zero = 0;
        each_block([&](uint32_t, const int4 &v) {
            above += (uint32_t)__popc(four_bits(v, [&](int x) { return x > 0 && x <= hi; }));
            zero += (uint32_t)__popc(four_bits(v, [](int x) { return x == 0; }));
        });
        above = wave_incl_scan(above);
        zero = wave_incl_scan(zero);
        if (lane == 63) { atomicAdd(&L.above_zero, above); atomicAdd(&L.zero, zero); }
        __syncthreads();
        above = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.above_zero);
        zero = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.zero);
        if (rem <= above) { lo = 1; crowd = above; }
        else if (rem <= above + zero) { lo = hi = 0; rem -= above; crowd = zero; }
        else { hi = -1; rem -= above + zero; crowd -= above + zero; }
    }
    // more tiles than the list takes: cut again, 4096 parts at a time, until they fit or all share one entropy (three times at most)
#pragma unroll 1
    while (crowd > kSmallListCap && lo != hi) {
        // (nothing about the entropies is kept from one round to the next: there are no registers for it)
#pragma unroll
        for (int r = 0; r < kMidBlocks; ++r) asm volatile("" : "+v"(q[r].x), "+v"(q[r].y), "+v"(q[r].z), "+v"(q[r].w));
        const uint32_t span = (uint32_t)hi - (uint32_t)lo;
        const int bits = 32 - __builtin_clz(span), shift = bits > 12 ? bits - 12 : 0;
        reinterpret_cast<uint4 *>(L.hist)[tid] = make_uint4(0, 0, 0, 0);
        __syncthreads();
        each_block([&](uint32_t, const int4 &v4) {
            const int v[4] = {v4.x, v4.y, v4.z, v4.w};
            const uint32_t from_lo0 = (uint32_t)v[0] - (uint32_t)lo;
            // (tokens that are alike make a crowd of neighbours: one addition for the four)
            if (v[0] == v[1] && v[1] == v[2] && v[2] == v[3]) {
                if (from_lo0 <= span) atomicAdd(&L.hist[from_lo0 >> shift], 4u);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t from_lo = (uint32_t)v[c] - (uint32_t)lo;
                    if (from_lo <= span) atomicAdd(&L.hist[from_lo >> shift], 1u);
                }
            }
        });
        __syncthreads();
        if (lo == INT32_MIN) {                   // (the first part has counted the places outside the unit as well)
            if (tid == 0) L.hist[0] -= outside;
            __syncthreads();
        }
        block_pick_bin<4096>(L.hist, rem, L.wave_total, L.chosen);
        lo = (int)((uint32_t)lo + ((uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[0]) << shift));
        rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[1]);
        crowd = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[2]);
        const uint32_t room = (uint32_t)hi - (uint32_t)lo, part = (1u << shift) - 1u;
        hi = (int)((uint32_t)lo + (room < part ? room : part));
    }
    const bool by_list = crowd <= kSmallListCap;
    each_block([&](uint32_t b, const int4 &v) {
        const uint32_t above = four_bits(v, [&](int x) { return x > hi; });
        uint32_t inside = four_bits(v, [&](int x) { return x >= lo; }) & ~above;
        if (lo == INT32_MIN) {
            const uint32_t i = b * 256u + 4u * lane - at.phase;
            inside &= (i < n ? 1u : 0u) | (i + 1u < n ? 2u : 0u) | (i + 2u < n ? 4u : 0u) | (i + 3u < n ? 8u : 0u);
        }
        put_bits(L.words, b, above);
        if (!by_list) {
            put_bits(L.equal, b, inside);
        } else if (inside != 0) {
            const int x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if ((inside >> c) & 1u)
                    L.list[atomicAdd(&L.listed, 1u) & (kSmallListCap - 1u)] =
                        ((uint64_t)((uint32_t)x[c] ^ 0x80000000u) << 32) | (uint32_t)~(b * 256u + 4u * lane + c);
            }
        }
    });
    __syncthreads();
    uint64_t word[WPT];
    const uint32_t g0 = WPT * (uint32_t)tid;
    if (by_list) {
        // four threads per listed tile count the tiles ahead of it
        if ((uint32_t)tid < 4 * crowd) {
            const uint64_t mine = L.list[tid >> 2];
            uint32_t ahead = 0;
#pragma unroll 4
            for (uint32_t i = (uint32_t)tid & 3u; i < crowd; i += 4) ahead += L.list[i] > mine ? 1u : 0u;
            ahead += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ahead, 0xB1, 0xF, 0xF, true);      // lane ^ 1
            ahead += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)ahead, 0x4E, 0xF, 0xF, true);      // lane ^ 2
            const uint32_t place = ~(uint32_t)mine;
            if (((uint32_t)tid & 3u) == 0 && ahead < rem)
                atomicOr(reinterpret_cast<uint32_t *>(L.words) + (place >> 5), 1u << (place & 31u));
        }
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < WPT; ++i) word[i] = g0 + i < at.nwords ? L.words[g0 + i] : 0ull;
    } else {
        // `crowd` tiles of one entropy: taken in index order until `rem` are used up
        uint64_t eq[WPT];
        uint32_t count = 0;
#pragma unroll
        for (uint32_t i = 0; i < WPT; ++i) {
            eq[i] = g0 + i < at.nwords ? L.equal[g0 + i] : 0ull;
            count += (uint32_t)__popcll(eq[i]);
        }
        const uint32_t incl = wave_incl_scan(count);
        if (lane == 63) L.wave_total[wave] = incl;
        __syncthreads();
        uint32_t eq_before = sum_of_waves_before(L.wave_total, wave, lane) + incl - count;
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < WPT; ++i) {
            const uint32_t here = (uint32_t)__popcll(eq[i]);
            uint64_t taken = eq_before < rem ? eq[i] : 0ull;
            for (uint32_t over = eq_before + here; taken != 0 && over > rem; --over) taken &= ~(1ull << (63 - __builtin_clzll(taken)));
            word[i] = g0 + i < at.nwords ? L.words[g0 + i] | taken : 0ull;
            eq_before += here;
        }
    }
    // selected places before every word
    uint32_t count = 0;
#pragma unroll
    for (uint32_t i = 0; i < WPT; ++i) count += (uint32_t)__popcll(word[i]);
    const uint32_t incl = wave_incl_scan(count);
    if (lane == 63) L.wave_total[wave] = incl;
    __syncthreads();
    uint32_t rank = u * k + sum_of_waves_before(L.wave_total, wave, lane) + incl - count;    // (every earlier unit holds exactly k)
#pragma unroll
    for (uint32_t i = 0; i < WPT; ++i) {
        const uint32_t g = g0 + i;
        if (g < at.nwords) {
            put_word(&bitmap[at.word0 + g], at.mask(g), word[i]);
            if (g != 0 || at.phase == 0) ranks[at.word0 + g] = rank;
        }
        rank += (uint32_t)__popcll(word[i]);
    }
}

// The edges of the threshold bin as bit patterns, first and last, as signed integers (negative values and NaN with the sign bit set
// lowest), `margin` further apart: tiles between them are the candidates.
struct BinEdges {
    int first, last;
    __device__ __forceinline__ BinEdges(uint32_t bin, float scale, float margin)
    {
        // (a bin is wider than the margin, so the second bin's edge is above it)
        first = bin == 0 ? INT32_MIN + 1 : (int)__float_as_uint(__uint_as_float((uint32_t)linear_bin_edge(bin, scale)) - margin);
        last = bin == kLinBins - 1 ? INT32_MAX
                                   : (int)__float_as_uint(__uint_as_float((uint32_t)linear_bin_edge(bin + 1, scale) - 1u) + margin);
    }
};

// A workgroup takes 16384 places, its wavefront w the blocks w, w + 16, .. of 256, four consecutive places per lane.  The
// threshold bin's edges turn into bit patterns once, so that an entropy costs two comparisons and its two bits; lanes collect
// them in nibbles (a ballot per 64 entropies, and the bin of every entropy, took 2.5 us longer).
//
// APPROX: the entropies in H are within `slack` of the exact ones, and so is the k-th largest of them of the exact threshold.  The
// candidates are then the tiles of the threshold bin and of a margin of 2 slack on either side: whoever is above that has an exact
// entropy above the exact threshold, whoever is below one below it.  The workgroup computes its candidates' exact entropies from
// the tensor (1.3 % of the tiles of [8,4096,8192], G = 64) and lists those.  How many candidates the margins add is not in the
// histogram; where the two bins beside the threshold's could fill the list, the entropies go back into H, for candidates held
// to the margins' ends (who is beyond them is decided), and are counted by sub-bin as for a crowd, in case it came to that.
template <int G, bool BF16, bool APPROX>
__global__ __launch_bounds__(kFusedThreads) void k_select_classify(float *__restrict__ H, uint32_t n, uint32_t k,
                                                                   uint32_t unit0, float bin_scale,
                                                                   const uint32_t *__restrict__ lin_hist,
                                                                   uint32_t *__restrict__ fused,
                                                                   uint2 *__restrict__ cand,
                                                                   uint2 *__restrict__ block_counts,
                                                                   uint32_t *__restrict__ crowd_hist,
                                                                   uint64_t *__restrict__ bitmap, const void *__restrict__ in,
                                                                   float eps_l1, float eps_log, float slack)
{
    constexpr uint32_t WAVES = kFusedThreads / 64, BLOCKS = kFusedKeysPerBlock / 256 / WAVES;
    static_assert(kSubBins == kFusedThreads, "one sub-bin per thread");
    __shared__ uint32_t sub_hist[kSubBins];
    __shared__ uint32_t chosen[4];               // threshold bin, wanted inside it, its tiles; the workgroup's place in the list
    __shared__ uint32_t wave_cand[WAVES], wave_above[WAVES];
    __shared__ uint16_t picked[APPROX ? kFusedKeysPerBlock : 1];         // the candidates, as places of the block
    static_assert(kFusedKeysPerBlock <= 65536, "places of a block in 16 bits");
    const uint32_t u = unit0 + blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const UnitPlaces at(u, n);
    float *uH = H + ((uint64_t)u * n - at.phase);            // by place
    uint2 *ucand = cand + (uint64_t)u * kCandCap;
    uint32_t *ubits = reinterpret_cast<uint32_t *>(bitmap + at.word0);
    const uint32_t *uhist = lin_hist + (uint64_t)u * kLinBins;

    // all loads first.  (Whole words of 64 places, which may reach into the neighbouring units or past the entropies to the end of
    // their padded array; beyond them from a clamped index.)
    const uint32_t place0 = blockIdx.x * kFusedKeysPerBlock + wave * 256u + 4u * lane, top = at.nwords * 64u - 4u;
    int4 q[BLOCKS];
#pragma unroll
    for (uint32_t r = 0; r < BLOCKS; ++r) {
        const uint32_t p = place0 + r * (WAVES * 256u);
        q[r] = *reinterpret_cast<const int4 *>(uH + (p < top ? p : top));
    }
    if (tid == 0) { chosen[0] = 0; chosen[1] = 0; chosen[2] = 0; }           // (for a histogram that does not hold k)
    sub_hist[tid] = 0;
    block_pick_bin<kLinBins>(uhist, k, wave_above, chosen);
    const uint32_t bstar = (uint32_t)__builtin_amdgcn_readfirstlane((int)chosen[0]);
    const uint32_t in_bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)chosen[2]);
    const bool crowd = in_bin > crowd_from(n);               // (the same for all of the unit's workgroups, like `doubt`)
    bool doubt = false;
    if constexpr (APPROX)
        doubt = !crowd &&
                in_bin + (bstar != 0 ? uhist[bstar - 1] : 0u) + (bstar != kLinBins - 1 ? uhist[bstar + 1] : 0u) > kCandCap;
    const BinEdges edge(bstar, bin_scale, APPROX ? 2.0f * slack : 0.0f);
    const int first = edge.first, last = edge.last;

    uint32_t inside = 0, n_above = 0;            // my candidates, four bits per block, the last block lowest
#pragma unroll
    for (uint32_t r = 0; r < BLOCKS; ++r) {
        const uint32_t base = blockIdx.x * kFusedKeysPerBlock + (r * WAVES + wave) * 256u, p = base + 4u * lane;
        if (base < at.phase || base + 256u > at.end) {
            // places outside the unit: the bit pattern of -0.0f, the lowest of all and no entropy's, approximate ones included
            q[r].x = p - at.phase < n ? q[r].x : INT32_MIN; q[r].y = p + 1u - at.phase < n ? q[r].y : INT32_MIN;
            q[r].z = p + 2u - at.phase < n ? q[r].z : INT32_MIN; q[r].w = p + 3u - at.phase < n ? q[r].w : INT32_MIN;
        }
        const uint32_t above =
            (q[r].x > last ? 1u : 0u) | (q[r].y > last ? 2u : 0u) | (q[r].z > last ? 4u : 0u) | (q[r].w > last ? 8u : 0u);
        const uint32_t reach =
            (q[r].x >= first ? 1u : 0u) | (q[r].y >= first ? 2u : 0u) | (q[r].z >= first ? 4u : 0u) | (q[r].w >= first ? 8u : 0u);
        inside = (inside << 4) | (reach & ~above);
        n_above += (uint32_t)__popc(above);
        // eight neighbouring lanes fill a dword of the bit map
        const uint32_t d = nibbles_to_dword(above, lane);
        if ((lane & 7) == 0 && p < at.nwords * 64u) {
            if (p >= at.phase && p + 32u <= at.end) ubits[p >> 5] = d;
            else atomicOr(&ubits[p >> 5], d);    // (a word that units share: cleared by an earlier kernel)
        }
    }
    // one place in the list for the whole workgroup (a unit's workgroups all add to one counter: few, large additions)
    const uint32_t count = (uint32_t)__popc(inside), incl = wave_incl_scan(count), incl_above = wave_incl_scan(n_above);
    __syncthreads();                             // everybody has the threshold bin: `wave_above` is used again
    if (lane == 63) { wave_cand[wave] = incl; wave_above[wave] = incl_above; }
    __syncthreads();
    const uint32_t before = sum_of_waves_before(wave_cand, wave, lane);
    if (wave == WAVES - 1) {
        const uint32_t above_before = sum_of_waves_before(wave_above, wave, lane);
        if (lane == 63) {
            chosen[2] = before + incl;
            chosen[3] = before + incl != 0 && !crowd ? atomicAdd(&fused[(uint64_t)u * 4], before + incl) : 0u;
            block_counts[(uint64_t)u * gridDim.x + blockIdx.x] = make_uint2(above_before + incl_above, before + incl);
        }
    }
    if constexpr (APPROX) {
        uint32_t pos = before + incl - count;
        for (uint32_t left = inside; left != 0; left &= left - 1u) {
            const uint32_t bit = (uint32_t)__ffs((int)left) - 1u;
            picked[pos++] = (uint16_t)((BLOCKS - 1 - bit / 4) * (WAVES * 256u) + wave * 256u + 4u * lane + bit % 4);
        }
        __syncthreads();
        using L = Lanes<G, BF16 ? 2 : 4>;
        using W = Wave<G, BF16 ? 2 : 4, L::few>;
        const uint32_t total = chosen[2], list_at = chosen[3], part = (uint32_t)tid % L::few;
        for (uint32_t i = (uint32_t)tid / L::few; i < total; i += kFusedThreads / L::few) {
            const uint32_t place = blockIdx.x * kFusedKeysPerBlock + picked[i];
            const uint64_t j = (uint64_t)u * n + (place - at.phase);
            TensorRow<W, BF16> x(static_cast<const uint8_t *>(in) + (j * L::few + part) * W::LANE_BYTES);
            float h = entropy_of<W::EPL, L::few>(x, eps_l1, eps_log);
            if (part != 0) continue;
            if (h != h) h = uH[place];           // (no number, and exact as it was)
            const uint32_t pos_in_list = list_at + i;
            if (!crowd && pos_in_list < kCandCap) ucand[pos_in_list] = make_uint2(order_key(h), place);
            if (crowd || doubt) {
                int v = (int)__float_as_uint(h);
                v = v < first ? first : v > last ? last : v;
                uH[place] = __uint_as_float((uint32_t)v);
                // (tiles that are alike meet on one counter: one addition for the wavefront's)
                const uint32_t bin = crowd_sub_bin(__uint_as_float((uint32_t)v), bin_scale, bstar);
                const uint32_t lead = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
                const uint64_t here = __ballot(true), same = __ballot(bin == lead);
                if (here != same) atomicAdd(&sub_hist[bin], 1u);
                else if (bits_below_me(here) == 0) atomicAdd(&sub_hist[lead], (uint32_t)__popcll(here));
            }
        }
    } else if (crowd) {
        if (inside != 0) {
#pragma unroll
            for (uint32_t r = 0; r < BLOCKS; ++r) {
                const uint32_t four = (inside >> (4 * (BLOCKS - 1 - r))) & 15u;
                const int v[4] = {q[r].x, q[r].y, q[r].z, q[r].w};
                auto sub_bin = [&](int bits) { return crowd_sub_bin(__uint_as_float((uint32_t)bits), bin_scale, bstar); };
                // (tiles that are alike meet on one counter; where they are neighbours, with one addition for four)
                if (four == 15u && v[0] == v[1] && v[1] == v[2] && v[2] == v[3]) {
                    atomicAdd(&sub_hist[sub_bin(v[0])], 4u);
                } else {
#pragma unroll
                    for (uint32_t c = 0; c < 4; ++c)
                        if ((four >> c) & 1u) atomicAdd(&sub_hist[sub_bin(v[c])], 1u);
                }
            }
        }
    } else {
        __syncthreads();
        uint32_t pos = chosen[3] + before + incl - count;
        if (__ballot(inside != 0) != 0) {
            // (from registers: a lane may hold sixteen of them, where tiles are all zero)
#pragma unroll
            for (uint32_t r = 0; r < BLOCKS; ++r) {
                const int v[4] = {q[r].x, q[r].y, q[r].z, q[r].w};
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) {
                    if ((inside >> (4 * (BLOCKS - 1 - r) + c)) & 1u) {
                        if (pos < kCandCap)
                            ucand[pos] = make_uint2(order_key(__uint_as_float((uint32_t)v[c])), place0 + r * (WAVES * 256u) + c);
                        ++pos;
                    }
                }
            }
        }
    }
    if (crowd || doubt) {
        __syncthreads();
        if (sub_hist[tid] != 0) atomicAdd(&crowd_hist[(uint64_t)u * kSubBins + tid], sub_hist[tid]);
    }
}

// LDS of k_select_resolve
struct ResolveLds {
    uint32_t hist[4096];
    uint64_t list[kFusedThreads];                // candidates that are placed directly: key << 32 | ~tile
    uint32_t chosen[6];                          // threshold bin, wanted inside it, its tiles; the same of the threshold sub-bin
    uint32_t listed, n_before;
    uint32_t above, candidates;                  // of the unit, by k_select_classify's counts
    uint32_t wave_total[kFusedThreads / 64];
    uint32_t words[2 * (kFusedKeysPerBlock / 64)];           // the block's bit map words, as dwords
};

// The first `rem` of the `count` candidates in L.list, by (key descending, tile ascending), thread t placing the t-th.
template <class TakeIt>
__device__ __forceinline__ void place_listed(uint32_t rem, uint32_t count, TakeIt take_it, const ResolveLds &L)
{
    if (threadIdx.x < count) {
        const uint64_t mine = L.list[threadIdx.x];
        uint32_t ahead = 0;
        for (uint32_t i = 0; i < count; ++i) ahead += L.list[i] > mine ? 1u : 0u;
        if (ahead < rem) take_it(~(uint32_t)mine);
    }
}

// The same for `count` candidates, keys lo .. hi, tiles below `places`, that are too many for the list: each(f) calls f(key, tile)
// for my share of them.  A histogram over 4096 parts of the keys' range narrows them down until they fit the list or share one
// key, and then one over 4096 parts of the tiles.  All 1024 threads.  (Encode of 655520 tiles of 32 channels with 16000 alike at the
// threshold: 89 us when both were radix selects, 69 now.)
template <class Each, class TakeIt>
__device__ __forceinline__ void rank_candidates(uint32_t rem, uint32_t count, uint32_t lo, uint32_t hi, uint32_t places, Each each,
                                                TakeIt take_it, ResolveLds &L)
{
    const int tid = threadIdx.x;
    if (tid == 0) L.listed = 0;
    uint32_t tile0 = 0;                          // of the candidates with one key: tiles from here on
    int tile_bits = 32 - __builtin_clz(places | 1u);         // ... that differ in so many bits
    __syncthreads();
#pragma unroll 1
    while (count > kFusedThreads && (lo != hi || tile_bits != 0)) {          // each part has 12 bits fewer: six times at most
        const bool by_key = lo != hi;
        const uint32_t span = hi - lo;
        const int bits = by_key ? 32 - __builtin_clz(span) : tile_bits, shift = bits > 12 ? bits - 12 : 0;
        reinterpret_cast<uint4 *>(L.hist)[tid] = make_uint4(0, 0, 0, 0);
        __syncthreads();
        each([&](uint32_t key, uint32_t tile) {
            // (the lowest tiles come first: their parts are counted from the top)
            const uint32_t at = by_key ? (key - lo) >> shift : 4095u - ((tile - tile0) >> shift);
            const bool inside = by_key ? key - lo <= span : key == lo && (uint64_t)(tile - tile0) >> tile_bits == 0;
            add_one_each(L.hist, at & 4095u, inside);
        });
        __syncthreads();
        block_pick_bin<4096>(L.hist, rem, L.wave_total, L.chosen);
        const uint32_t part = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[0]);
        rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[1]);
        count = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[2]);
        if (by_key) {
            lo += part << shift;
            const uint32_t width = (1u << shift) - 1u;
            hi = hi - lo < width ? hi : lo + width;
        } else {
            tile0 += (4095u - part) << shift;
            tile_bits = shift;
        }
    }
    each([&](uint32_t key, uint32_t tile) {
        if (key > hi || (key >= lo && tile < tile0)) take_it(tile);
        else if (key >= lo && (uint64_t)(tile - tile0) >> tile_bits == 0) {
            const uint32_t at = atomicAdd(&L.listed, 1u);
            if (at < kFusedThreads) L.list[at] = ((uint64_t)key << 32) | (uint32_t)~tile;
        }
    });
    __syncthreads();
    place_listed(rem, count < kFusedThreads ? count : kFusedThreads, take_it, L);
}

// A unit whose threshold bin holds more tiles than the candidate list: workgroup `blk` of `blocks`, each of 16384 places.
// Every workgroup first settles its own tiles: those above the threshold's sub-bin into the bit map, those in it (`crowd`, of which
// `rem` are selected) into `equal`, words over places that only this unit has; it finds the range of their keys and, where they
// fit, lists them (in a list of their own: `listed_before` is what k_select_classify has listed).  The last of the unit's
// workgroups to finish then knows them all.
__device__ __forceinline__ void resolve_crowd(const float *__restrict__ H, uint32_t n, uint32_t k, uint32_t u, uint32_t blk,
                                              uint32_t blocks, float bin_scale, float margin, uint32_t bstar, uint32_t rem,
                                              uint32_t listed_before,
                                              const uint32_t *crowd_hist, uint32_t *state, uint2 *ucand, uint64_t *equal,
                                              uint64_t *bitmap, uint32_t *ranks, ResolveLds &L)
{
    constexpr uint32_t WAVES = kFusedThreads / 64, BLOCKS = kFusedKeysPerBlock / 256 / WAVES;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const UnitPlaces at(u, n);
    const float *uH = H + ((uint64_t)u * n - at.phase);      // by place
    uint64_t *ubitmap = bitmap + at.word0;
    uint32_t *ubits = reinterpret_cast<uint32_t *>(ubitmap), *equal32 = reinterpret_cast<uint32_t *>(equal);
    const uint32_t top = at.nwords * 64u - 4u;
    // four neighbouring entropies' bit patterns, -0.0f (no entropy's) outside the unit
    auto four_at = [&](uint32_t p) {
        int4 q = *reinterpret_cast<const int4 *>(uH + (p < top ? p : top));
        q.x = p - at.phase < n ? q.x : INT32_MIN; q.y = p + 1u - at.phase < n ? q.y : INT32_MIN;
        q.z = p + 2u - at.phase < n ? q.z : INT32_MIN; q.w = p + 3u - at.phase < n ? q.w : INT32_MIN;
        return q;
    };
    int4 q[BLOCKS];
#pragma unroll
    for (uint32_t r = 0; r < BLOCKS; ++r) q[r] = four_at(blk * kFusedKeysPerBlock + (r * WAVES + wave) * 256u + 4u * lane);
    block_pick_bin<kSubBins>(crowd_hist + (uint64_t)u * kSubBins, rem, L.wave_total, L.chosen + 3);
    const uint32_t sstar = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[3]);
    rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[4]);
    uint32_t crowd = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[5]);
    const bool list_them = crowd <= kCandCap;
    const BinEdges edge(bstar, bin_scale, margin);
    const int first = edge.first, last = edge.last;

    uint32_t inside = 0, key_max = 0, not_key_min = 0;
#pragma unroll
    for (uint32_t r = 0; r < BLOCKS; ++r) {
        const int v[4] = {q[r].x, q[r].y, q[r].z, q[r].w};
        uint32_t above = 0, four = 0;
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c) {
            const float h = __uint_as_float((uint32_t)v[c]);
            const uint32_t s = crowd_sub_bin(h, bin_scale, bstar), key = order_key(h);
            const bool in_bin = v[c] >= first && v[c] <= last, in_sub = in_bin && s == sstar;
            above |= v[c] > last || (in_bin && s > sstar) ? 1u << c : 0u;
            four |= in_sub ? 1u << c : 0u;
            key_max = in_sub && key > key_max ? key : key_max;
            not_key_min = in_sub && ~key > not_key_min ? ~key : not_key_min;
        }
        inside = (inside << 4) | four;
        const uint32_t p = blk * kFusedKeysPerBlock + (r * WAVES + wave) * 256u + 4u * lane;
        const uint32_t d_above = nibbles_to_dword(above, lane), d_equal = nibbles_to_dword(four, lane);
        if ((lane & 7) == 0 && p < at.nwords * 64u) {
            equal32[p >> 5] = d_equal;
            if (p >= at.phase && p + 32u <= at.end) ubits[p >> 5] = d_above;
            else atomicOr(&ubits[p >> 5], d_above);          // (a word that units share)
        }
    }
    wave_max(key_max, not_key_min);
    const uint32_t count = (uint32_t)__popc(inside), incl = wave_incl_scan(count);
    __syncthreads();                             // everybody has the sub-bin: `chosen` and `wave_total` are used again
    if (lane == 63) {
        L.wave_total[wave] = incl;
        if (incl != 0) { atomicMax(&L.n_before, key_max); atomicMax(&L.listed, not_key_min); }       // both start at 0
    }
    __syncthreads();
    const uint32_t before = sum_of_waves_before(L.wave_total, wave, lane);
    if (wave == WAVES - 1 && lane == 63 && before + incl != 0) {
        L.chosen[0] = list_them ? atomicAdd(&state[0], before + incl) - listed_before : 0u;
        atomicMax(&state[2], L.n_before);
        atomicMax(&state[3], L.listed);
    }
    __syncthreads();
    if (list_them) {
        uint32_t pos = L.chosen[0] + before + incl - count;
#pragma unroll
        for (uint32_t r = 0; r < BLOCKS; ++r) {
            const int v[4] = {q[r].x, q[r].y, q[r].z, q[r].w};
#pragma unroll
            for (uint32_t c = 0; c < 4; ++c) {
                if ((inside >> (4 * (BLOCKS - 1 - r) + c)) & 1u) {
                    if (pos < kCandCap)
                        ucand[pos] = make_uint2(order_key(__uint_as_float((uint32_t)v[c])),
                                                blk * kFusedKeysPerBlock + (r * WAVES + wave) * 256u + 4u * lane + c);
                    ++pos;
                }
            }
        }
    }
    // Who is last?  Every wavefront's stores have reached the L2 before the workgroup counts itself, and the one thread that
    // counts writes the L2 back where another XCD could not see it otherwise.
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0)
    __syncthreads();
    if (tid == 0) L.chosen[0] = __hip_atomic_fetch_add(&state[1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (L.chosen[0] != blocks - 1) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");

    // The unit's words in order, 256 consecutive ones per wavefront and sweep, the first of them requested right away.
    constexpr int WPT = 4;
    uint64_t word[WPT], eq[WPT];
    auto load_words = [&](uint32_t sweep, uint64_t (&w)[WPT], uint64_t (&e)[WPT]) {
#pragma unroll
        for (int i = 0; i < WPT; ++i) {
            const uint32_t g = sweep + wave * (64u * WPT) + 64u * i + lane, c = g < at.nwords ? g : at.nwords - 1;
            w[i] = ubitmap[c];                   // (clamped, masked where they are used)
            e[i] = equal[c];
        }
    };
    load_words(0, word, eq);
    uint32_t hi = __hip_atomic_load(&state[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t lo = ~__hip_atomic_load(&state[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool by_index = lo == hi || rem == crowd || !list_them;        // the first `rem` places of `equal` are selected
    auto take_it = [&](uint32_t tile) {
        if (tile < at.nwords * 64u) atomicOr(&ubits[tile >> 5], 1u << (tile & 31u));
    };
    const bool changed = lo != hi && rem != crowd;           // otherwise the words are what has been requested
    if (!by_index) {
        rank_candidates(rem, crowd, lo, hi, at.nwords * 64u, [&](auto f) {
#pragma unroll 1
            for (uint32_t i = tid; i < crowd; i += kFusedThreads) {
                const uint2 c = ucand[i];
                f(c.x, c.y);
            }
        }, take_it, L);
    } else if (changed) {
        // A crowd of several entropies that lie within one sub-bin: the range of their keys is cut into 4096 parts until one
        // entropy is left (three times at most), by passes over the unit.
        const uint32_t largest = hi;
        auto each_four = [&](auto visit) {       // (four loads in flight; every wavefront takes whole blocks of 256 places)
            for (uint32_t b = wave; b * 256u < at.nwords * 64u; b += 4 * WAVES) {
                int4 w[4];
#pragma unroll
                for (uint32_t i = 0; i < 4; ++i) w[i] = four_at((b + i * WAVES) * 256u + 4u * lane);
#pragma unroll
                for (uint32_t i = 0; i < 4; ++i) visit((b + i * WAVES) * 256u + 4u * lane, w[i]);
            }
        };
        auto key_of = [](int v) { return order_key(__uint_as_float((uint32_t)v)); };     // (-0.0f lies in no range: no entropy is)
#pragma unroll 1
        while (lo != hi) {
            const uint32_t span = hi - lo;
            const int bits = 32 - __builtin_clz(span), shift = bits > 12 ? bits - 12 : 0;
            reinterpret_cast<uint4 *>(L.hist)[tid] = make_uint4(0, 0, 0, 0);
            __syncthreads();
            each_four([&](uint32_t, const int4 &w) {
                const int v[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t from_lo = key_of(v[c]) - lo;
                    if (from_lo <= span && v[c] != INT32_MIN) atomicAdd(&L.hist[from_lo >> shift], 1u);
                }
            });
            __syncthreads();
            block_pick_bin<4096>(L.hist, rem, L.wave_total, L.chosen);
            lo += (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[0]) << shift;
            rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.chosen[1]);
            const uint32_t part = (1u << shift) - 1u;
            hi = hi - lo < part ? hi : lo + part;
        }
        each_four([&](uint32_t p, const int4 &w) {
            const int v[4] = {w.x, w.y, w.z, w.w};
            uint32_t above = 0, four = 0;
#pragma unroll
            for (uint32_t c = 0; c < 4; ++c) {
                const uint32_t key = key_of(v[c]);
                above |= key > lo && key <= largest && v[c] != INT32_MIN ? 1u << c : 0u;
                four |= key == lo && v[c] != INT32_MIN ? 1u << c : 0u;
            }
            const uint32_t d_above = nibbles_to_dword(above, lane), d_equal = nibbles_to_dword(four, lane);
            if ((lane & 7) == 0 && p < at.nwords * 64u) {
                equal32[p >> 5] = d_equal;
                if (d_above != 0) atomicOr(&ubits[p >> 5], d_above);
            }
        });
    }
    if (changed) {
        __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0): all wavefronts' words are in the L2
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        load_words(0, word, eq);
    }
    // How many of `equal` come before each word, which of them are taken, and how many selected tiles come before.
    uint32_t equal_run = 0, rank_run = u * k;    // (every earlier unit holds exactly k wide tiles)
    // ahead[i] = the sum of count over all words before my i-th, and `run` moved on by the sum of all
    auto scan_words = [&](const uint32_t (&count)[WPT], uint32_t (&ahead)[WPT], uint32_t *run) {
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < WPT; ++i) {
            const uint32_t upto = wave_incl_scan(count[i]);
            ahead[i] = sum + upto - count[i];
            sum += (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
        }
        __syncthreads();
        if (lane == 0) L.wave_total[wave] = sum;
        __syncthreads();
        const uint32_t before = *run + sum_of_waves_before(L.wave_total, wave, lane);
#pragma unroll
        for (int i = 0; i < WPT; ++i) ahead[i] += before;
        uint32_t total = 0;
#pragma unroll
        for (uint32_t w = 0; w < WAVES; ++w) total += L.wave_total[w];
        *run += total;
    };
    for (uint32_t sweep = 0; sweep < at.nwords; sweep += WPT * kFusedThreads) {
        const uint32_t g0 = sweep + wave * (64u * WPT) + lane;
        uint64_t next_word[WPT], next_eq[WPT];
        load_words(sweep + WPT * kFusedThreads, next_word, next_eq);
        uint32_t count[WPT], ahead[WPT];
#pragma unroll
        for (int i = 0; i < WPT; ++i) {
            const uint32_t g = g0 + 64u * i;
            word[i] = g < at.nwords ? word[i] & at.mask(g) : 0ull;
            eq[i] = g < at.nwords && by_index ? eq[i] : 0ull;
            count[i] = (uint32_t)__popcll(eq[i]);
        }
        scan_words(count, ahead, &equal_run);
#pragma unroll
        for (int i = 0; i < WPT; ++i) {
            uint64_t taken = ahead[i] < rem ? eq[i] : 0ull;
            for (uint32_t over = ahead[i] + count[i]; taken != 0 && over > rem; --over) taken &= ~(1ull << (63 - __builtin_clzll(taken)));
            word[i] |= taken;
            count[i] = (uint32_t)__popcll(word[i]);
        }
        scan_words(count, ahead, &rank_run);
#pragma unroll
        for (int i = 0; i < WPT; ++i) {
            const uint32_t g = g0 + 64u * i;
            if (g < at.nwords) {
                put_word(&ubitmap[g], at.mask(g), word[i]);
                if (g != 0 || at.phase == 0) ranks[at.word0 + g] = ahead[i];
            }
        }
#pragma unroll
        for (int i = 0; i < WPT; ++i) { word[i] = next_word[i]; eq[i] = next_eq[i]; }
    }
}

__global__ __launch_bounds__(kFusedThreads) void k_select_resolve(const float *__restrict__ H, uint32_t n, uint32_t k,
                                                                  uint32_t unit0, float bin_scale, float margin,
                                                                  const uint32_t *__restrict__ lin_hist,
                                                                  uint32_t *__restrict__ fused,
                                                                  uint2 *__restrict__ cand,
                                                                  const uint2 *__restrict__ block_counts,
                                                                  const uint32_t *__restrict__ crowd_hist,
                                                                  uint64_t *__restrict__ equal,
                                                                  uint64_t *__restrict__ bitmap,
                                                                  uint32_t *__restrict__ ranks)
{
    __shared__ ResolveLds L;
    constexpr uint32_t GROUPS = kFusedKeysPerBlock / 64;     // 64-tile groups of a block
    const uint32_t u = unit0 + blockIdx.y, blk = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint2 *ucand = cand + (uint64_t)u * kCandCap;
    const UnitPlaces at(u, n);
    uint64_t *ubitmap = bitmap + at.word0;
    uint32_t *uranks = ranks + at.word0;
    const uint32_t group0 = blk * GROUPS;
    const uint32_t left = group0 < at.nwords ? at.nwords - group0 : 0u, mygroups = left < GROUPS ? left : GROUPS;

    // everything this workgroup reads from global memory, requested at once: the first candidates (the list always has
    // room for them, what lies beyond its end is ignored; the others, where there are more, once their number is known),
    // the block's words, the counts of the blocks before it, the histogram
    constexpr int CPT = (int)(kCandCap / kFusedThreads), AHEAD = 4;
    uint2 c[CPT];
#pragma unroll
    for (int r = 0; r < AHEAD; ++r) c[r] = ucand[(uint32_t)r * kFusedThreads + tid];
    uint64_t my_word = 0;
    if ((uint32_t)tid < mygroups) my_word = ubitmap[group0 + tid] & at.mask(group0 + tid);
    uint32_t above_before = 0, above_all = 0, cand_all = 0;
    for (uint32_t b = tid; b < gridDim.x; b += kFusedThreads) {
        const uint2 counts = block_counts[(uint64_t)u * gridDim.x + b];
        above_before += b < blk ? counts.x : 0u;
        above_all += counts.x;
        cand_all += counts.y;
    }
    if (tid < 6) L.chosen[tid] = 0;              // (for histograms that do not hold as many as are wanted)
    if (tid == 0) { L.n_before = 0; L.listed = 0; L.above = 0; L.candidates = 0; }
    static_assert(kSubBins == kFusedThreads, "one sub-bin per thread");
    uint32_t *sub_hist = L.hist;                 // the threshold bin's candidates by sub-bin
    sub_hist[tid] = 0;
    if ((uint32_t)tid < GROUPS) { L.words[2 * tid] = (uint32_t)my_word; L.words[2 * tid + 1] = (uint32_t)(my_word >> 32); }
    block_pick_bin<kLinBins>(lin_hist + (uint64_t)u * kLinBins, k, L.wave_total, L.chosen);
    {
        const uint32_t a = wave_incl_scan(above_all), c = wave_incl_scan(cand_all);
        if (lane == 63 && a != 0) atomicAdd(&L.above, a);
        if (lane == 63 && c != 0) atomicAdd(&L.candidates, c);
    }
    __syncthreads();
    // wanted among the candidates (where the histogram does not hold k: none)
    const uint32_t bstar = L.chosen[0], rem = L.chosen[1] != 0 ? k - L.above : 0u;
    const bool not_listed = L.chosen[2] > crowd_from(n);
    const uint32_t listed = not_listed ? 0u : L.candidates;

    if (__builtin_expect(not_listed || (rem != 0 && listed > kCandCap), 0)) {          // (the same for all of the unit's workgroups)
        resolve_crowd(H, n, k, u, blk, gridDim.x, bin_scale, margin, bstar, rem, listed, crowd_hist, fused + (uint64_t)u * 4, ucand,
                      equal + (uint64_t)u * (n / 64 + 2), bitmap, ranks, L);
        return;
    }
    // the selected candidates: those of my block go into its words, those before it are counted
    const uint32_t first_tile = group0 * 64u;
    uint32_t before = 0;
    auto take_it = [&](uint32_t tile) {
        if (tile < first_tile) ++before;
        else if (tile - first_tile < kFusedKeysPerBlock) atomicOr(&L.words[(tile - first_tile) >> 5], 1u << (tile & 31u));
    };
    if (rem != 0) {
        // A histogram of the candidates over 1024 sub-bins of their bin narrows the threshold down once more:
        // candidates in a higher sub-bin are selected, those in the threshold's own sub-bin (a handful, as a rule) are
        // ranked directly, thread t placing the t-th of them among all of them by (key descending, tile ascending).
        if (listed > (uint32_t)AHEAD * kFusedThreads) {
#pragma unroll
            for (int r = AHEAD; r < CPT; ++r) c[r] = ucand[(uint32_t)r * kFusedThreads + tid];
        }
        uint32_t sub[CPT];
#pragma unroll
        for (int r = 0; r < CPT; ++r) {
            sub[r] = 0xffffffffu;
            if ((uint32_t)r * kFusedThreads >= listed) continue;         // (the same for all threads)
            if ((uint32_t)r * kFusedThreads + tid < listed) {
                sub[r] = linear_sub_bin(key_to_float(c[r].x), bin_scale, bstar);
            }
            // (many candidates are a crowd of tiles that are alike, as a rule)
            if (listed > (uint32_t)AHEAD * kFusedThreads) add_one_each(sub_hist, sub[r], sub[r] != 0xffffffffu);
            else if (sub[r] != 0xffffffffu) atomicAdd(&sub_hist[sub[r]], 1u);
        }
        __syncthreads();
        block_pick_bin<kSubBins>(sub_hist, rem, L.wave_total, L.chosen + 3);
        const uint32_t sstar = L.chosen[3], rem2 = L.chosen[4], nl = L.chosen[5];
        uint32_t in_sub = 0;                     // bit r: my r-th candidate lies in the threshold's sub-bin
#pragma unroll
        for (int r = 0; r < CPT; ++r) {
            if ((uint32_t)r * kFusedThreads >= listed) continue;
            if (sub[r] != 0xffffffffu) {
                if (sub[r] > sstar) take_it(c[r].y);
                else if (sub[r] == sstar) {
                    in_sub |= 1u << r;
                    if (nl <= kFusedThreads) {
                        const uint32_t at = atomicAdd(&L.listed, 1u);
                        if (at < kFusedThreads) L.list[at] = ((uint64_t)c[r].x << 32) | (uint32_t)~c[r].y;
                    }
                }
            }
        }
        if (nl <= kFusedThreads) {
            __syncthreads();
            place_listed(rem2, nl, take_it, L);
        } else {
            uint32_t key_max = 0, not_key_min = 0;
#pragma unroll
            for (int r = 0; r < CPT; ++r) {
                const bool mine = (in_sub >> r) & 1u;
                key_max = mine && c[r].x > key_max ? c[r].x : key_max;
                not_key_min = mine && ~c[r].x > not_key_min ? ~c[r].x : not_key_min;
            }
            wave_max(key_max, not_key_min);
            __syncthreads();                     // (L.chosen has been read)
            if (tid == 0) { L.chosen[0] = 0; L.chosen[1] = 0; }
            __syncthreads();
            if (lane == 0) { atomicMax(&L.chosen[0], key_max); atomicMax(&L.chosen[1], not_key_min); }
            __syncthreads();
            rank_candidates(rem2, nl, ~L.chosen[1], L.chosen[0], at.nwords * 64u, [&](auto f) {
#pragma unroll
                for (int r = 0; r < CPT; ++r)
                    if ((in_sub >> r) & 1u) f(c[r].x, c[r].y);
            }, take_it, L);
        }
    }
    above_before += before;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) above_before += (uint32_t)__shfl_xor((int)above_before, off, 64);
    if (lane == 0 && above_before != 0) atomicAdd(&L.n_before, above_before);
    __syncthreads();
    // the block's final words and rank-table entries: one group per thread of the first four wavefronts
    uint32_t lo = 0, hi = 0;
    if ((uint32_t)tid < GROUPS) { lo = L.words[2 * tid]; hi = L.words[2 * tid + 1]; }
    const uint32_t cnt = (uint32_t)__popc(lo) + (uint32_t)__popc(hi);
    const uint32_t incl = wave_incl_scan(cnt);
    if (lane == 63) L.wave_total[wave] = incl;
    __syncthreads();
    const uint32_t rank = u * k + L.n_before + sum_of_waves_before(L.wave_total, (uint32_t)wave, lane) + incl - cnt;
    if ((uint32_t)tid < mygroups) {              // (every earlier unit holds exactly k wide tiles)
        put_word(&ubitmap[group0 + tid], at.mask(group0 + tid), ((uint64_t)hi << 32) | lo);
        if (group0 + tid != 0 || at.phase == 0) uranks[group0 + tid] = rank;
    }
}

__global__ __launch_bounds__(256) void k_bitmap_const(uint32_t T, int all_wide, uint64_t *__restrict__ bitmap,
                                                      uint32_t *__restrict__ ranks)
{
    const uint64_t w = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (w < ((uint64_t)T + 63) / 64) constant_width_word(w, T, all_wide, bitmap, ranks);
}

// The prologue in a launch of its own, with the scratch of the large units' selections cleared.
__global__ __launch_bounds__(256) void k_prologue(Prologue pro, uint32_t *__restrict__ zero_base, uint32_t zero_words)
{
    const uint32_t gid = blockIdx.x * 256 + threadIdx.x;
    write_prologue(pro, gid, gridDim.x * 256);
    for (uint32_t i = gid; i < zero_words; i += gridDim.x * 256) zero_base[i] = 0u;
}

}  // namespace tahq

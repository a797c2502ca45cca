// TAH-Quant stage-boundary activation codec for gfx950: launch glue and C ABI.
//
// Paper sections implemented by the kernels this file launches: Sec. 3.1 (tiles of G contiguous
// channels), Sec. 3.2 Eq. 1-2 (entropy) and top-p% selection, Sec. 3.3 Eq. 3-4 (outlier test,
// pivot swap, Hadamard transform, asymmetric quantizer), Sec. 3.4 (byte stream), Alg. 1 step 5
// (dequantize); and, for the backward direction, Sec. 3.5 / Alg. 1 steps 6-7 with the appendix's gradient
// scaling (fixed-point compressor, tahq_naive_*).
//
// Numerics contract (identical results on any mapping of tiles to lanes; a signalling NaN in the input, which no arithmetic
// produces, is the exception: the minimum and maximum of its tile depend on the lanes that share it):
//   * all arithmetic is IEEE binary32, no contraction (-ffp-contract=off); fused multiply-adds
//     only where written (__builtin_fmaf);
//   * sums over a tile use the adjacent-pair binary tree; an allocation tile of several quantization
//     tiles adds their sums from left to right;
//   * the Hadamard butterfly runs its stages h = 1, 2, ..., G/2 in that order;
//   * log(u) = e*ln2 + P(m) with (m, e) = frexp(u) and a fixed degree-5 polynomial;
//   * scale / zero-point are binary16, rounded outwards (up / down).
#include "tahq_common.hpp"
#include "tahq_select.hpp"
#include "tahq_stream_kernels.hpp"
#include "tahq_launch.hpp"
#include "tahq_naive_kernels.hpp"
#include "tahq_naive.h"

#include <atomic>
#include <mutex>
#include <type_traits>

using namespace tahq;

// Built-in scratch of tahq_encode_noalloc: encoder workspace for callers that cannot provide one.  Every GPU
// the library runs on holds its own copy of this array, at its own address, until the process ends.
constexpr size_t kBuiltinScratchBytes = (size_t)TAHQ_NOALLOC_MAX_WORKSPACE;
static __device__ __align__(256) unsigned char scratch[kBuiltinScratchBytes];

namespace {

// Device address of `scratch` on every device that tahq_encode_noalloc has been called on.  In host code the
// array's name is only a handle for hipGetSymbolAddress: kernels are given the address kept here.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];


inline bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

constexpr uint32_t kMaxGridY = 65535;

inline uint32_t blocks_for(uint64_t threads) { return (uint32_t)((threads + 255) / 256); }

// Grid of a persistent kernel: four times the workgroups that fit on the device at once (or fewer, if there
// are fewer batches).  Every workgroup still pipelines a few batches, and the hardware dispatcher evens
// out the load; a grid of exactly the resident count measured up to 30% slower.
// The resident count of a kernel is a property of the kernel and the device; it is looked up once per kernel and
// device (a query of the runtime, no stream operation: also legal while a stream is being captured) and kept
// in `cache`, one slot per device.
struct ResidentCache { std::atomic<uint32_t> per_device[kMaxDevices]; };

inline uint32_t resident_blocks(const void *kernel, int threads, ResidentCache &cache)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) dev = 0;
    const bool cached = dev < kMaxDevices;
    if (cached) {
        const uint32_t known = cache.per_device[dev].load(std::memory_order_relaxed);
        if (known) return known;
    }
    int cus = 256, per_cu = 1;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu <= 0) per_cu = 1;
    const uint32_t res = 4u * (uint32_t)cus * (uint32_t)per_cu;
    if (cached) cache.per_device[dev].store(res, std::memory_order_relaxed);
    return res;
}

// Streams from here on pass the caches by.  Written through them, a large stream is not there any more when the decoder reads it and
// comes out as dirty lines in the middle of the reads of the next kernels.  bf16 [8,S,8192] on three sets of buffers in turn, encode
// and decode in us, through the caches and past them: G = 64 at 3.25 bits: 62 MiB 180 and 183, 125 MiB 363 and 341; at 4 bits:
// 74 MiB 117 and 120, 149 MiB 238 and 231; G = 128 at 3 bits: 106 MiB 233 and 244; G = 32 at 4 bits: 85 MiB 118 and 123,
// 170 MiB 242 and 238.  What it trades: the encode of 125 MiB alone takes 234 us instead of 261, and a decode on the same card
// right after it 120 instead of 97, because the stream is no longer in the Infinity Cache: both on one set of buffers 347
// instead of 338.  A stream that leaves for another card has the gain alone.
constexpr uint64_t kStreamingFrom = 112ull << 20;

// What the entropy pass computes by: Eq. 1-2, and Eq. 3 where it decides that as well.
struct EntropyParams {
    float eps_l1, eps_log, tau, eps_ratio;
    bool approx;                                 // entropies to within kEntropySlack will do (and are to be had)
};

inline EntropyParams entropy_params(const tahq_config *c) { return {c->eps_l1, c->eps_log, c->tau, c->eps_ratio, false}; }

// Whether the two-launch selection works from approximate entropies: for bf16 tensors of 2^25 elements and more, where what
// the entropy pass saves is more than what the selection spends on exact ones, and constants that the bound covers.
inline bool approximate_entropies(const Shape &s, const tahq_config *c)
{
    return s.dtype == TAHQ_BF16 && s.T * s.G >= (1u << 25) && c->eps_log >= kApproxLogMin && c->eps_log <= kApproxLogMax &&
           c->eps_l1 >= 1e-30f && c->eps_l1 <= 1e30f;
}

template <int G, bool BF16>
struct LaunchEntropy {
    template <int LPT, int NG, bool HIST, bool APPROX>
    static void go(const void *d_in, float *d_H, uint8_t *pivot, uint32_t T, const EntropyParams &p, uint32_t *hist,
                   uint32_t bins, float bin_scale, uint64_t n_per_unit, const Prologue &pro, Enqueue *qp)
    {
        Enqueue &q = *qp;
        constexpr uint32_t STEP = 256 / LPT * NG;            // tiles
        const uint32_t nb = (T + STEP - 1) / STEP;
        static ResidentCache cache;
        const uint32_t res = resident_blocks(reinterpret_cast<const void *>(k_entropy<G, BF16, LPT, NG, HIST, APPROX>), 256, cache);
        // Every workgroup adds its histogram to the unit's, and what that costs are the additions that meet on one bin: four
        // steps per workgroup, or four rounds of its lanes where those make no more than two workgroups per compute unit.  Encode of
        // bf16 with four rounds for all, and so: [1,4096,8192] G = 16 106 -> 72 us, G = 8 115 -> 84, [3,4672,2560] G = 16
        // 89.2 -> 63.8, [4,4096,4096] G = 32 83.7 -> 79.8, fp32 [1,5760,5120] G = 8 152 -> 92.  (With four steps for all bf16
        // [8,360,5120] G = 16 40.2 -> 42.8, [4,3028,2048] G = 32 47.9 -> 51; three units of 77700 tiles of 16 channels: 14.1 us with a
        // workgroup per round, 8.4 so.)
        const uint32_t rounds = nb * NG / 4 < 512u ? nb * NG / 4 : 512u;
        const uint32_t some = nb / 4 > rounds ? nb / 4 : rounds, few = some > 256u ? some : 256u;
        const uint32_t most = HIST && few < res ? few : res;
        const uint32_t grid = nb < most ? nb : most;
        q(k_entropy<G, BF16, LPT, NG, HIST, APPROX>, dim3(grid), dim3(256), d_in, d_H, pivot, T, (nb + grid - 1) / grid, p.eps_l1,
          p.eps_log, p.tau, p.eps_ratio, prologue_blocks(pro, 256, grid), hist, (uint32_t)n_per_unit, bins, bin_scale, pro);
    }
    template <int LPT, int NG>
    static void with(const void *d_in, float *d_H, uint8_t *pivot, uint32_t T, const EntropyParams &p, uint32_t *hist,
                     uint32_t bins, float bin_scale, uint64_t n_per_unit, const Prologue &pro, Enqueue *qp)
    {
        if constexpr (BF16 && LPT == Lanes<G, 2>::usual) {
            if (hist && p.approx) { go<LPT, NG, true, true>(d_in, d_H, pivot, T, p, hist, bins, bin_scale, n_per_unit, pro, qp); return; }
        }
        if (hist) go<LPT, NG, true, false>(d_in, d_H, pivot, T, p, hist, bins, bin_scale, n_per_unit, pro, qp);
        else go<LPT, NG, false, false>(d_in, d_H, pivot, T, p, hist, bins, bin_scale, n_per_unit, pro, qp);
    }
    // hist != nullptr: also build the selection's first histogram, `bins` bins per ranking unit (of at least one step): the keys'
    // first radix digit if bin_scale == 0, the entropies' linear bins otherwise
    static void run(const void *d_in, float *d_H, uint8_t *pivot, uint32_t T, const EntropyParams &p, uint32_t *hist,
                    uint32_t bins, float bin_scale, uint64_t n_per_unit, Prologue pro, Enqueue *qp)
    {
        using N = Lanes<G, BF16 ? 2 : 4>;
        constexpr int NG = kRowGroups<G, BF16 ? 2 : 4, N::usual>;
        if (few_tiles<N>(T, 4)) with<N::few, 1>(d_in, d_H, pivot, T, p, hist, bins, bin_scale, n_per_unit, pro, qp);
        else if (NG == 1 || T < (hist ? 128u : 1024u) * 256u * NG)
            with<N::usual, 1>(d_in, d_H, pivot, T, p, hist, bins, bin_scale, n_per_unit, pro, qp);
        else with<N::usual, NG>(d_in, d_H, pivot, T, p, hist, bins, bin_scale, n_per_unit, pro, qp);
    }
    // Whether exact entropies of T tiles are computed by lanes with whole tiles each, and those with Eq. 3.
    static bool pivots(uint32_t T) { return kWholeTiles<G, BF16> && !few_tiles<Lanes<G, 2>>(T, 4); }
    // units are whole steps, whatever those are
    static bool can_fuse_histogram(uint64_t n_per_unit)
    {
        using N = Lanes<G, BF16 ? 2 : 4>;
        return n_per_unit % (256 / N::usual * kRowGroups<G, BF16 ? 2 : 4, N::usual>) == 0;
    }
};

template <int G, bool BF16>
struct CanFuse {
    static void run(uint64_t n_per_unit, bool *out) { *out = LaunchEntropy<G, BF16>::can_fuse_histogram(n_per_unit); }
};

// Where a call's tiles get their widths from: one for all of them, or the stream's bit map, and with that maybe their pivot bytes
// (bf16 at the usual lanes only: the entropies of fewer tiles come without Eq. 3).
enum class Widths { one, ranked, ranked_with_pivots };

// `low`: the narrower of the two code widths, 1..7 (3: INT3/INT4).
template <int G, bool BF16>
struct LaunchQuantPack {
    template <int LOW, int LPT>
    static void with(const void *d_in, uint8_t *packed, uint32_t T, float tau, float eps_ratio, Widths widths,
                   uint32_t how, const Prologue &pro, Enqueue *qp)
    {
        Enqueue &q = *qp;
        // by workgroups where a lane has a bf16 tile of 32 channels or more, by wavefronts otherwise (the figures are at the kernels)
        constexpr bool by_wave = LPT > 1 || !BF16 || G < 32;
        constexpr uint32_t tiles = by_wave ? 4 * (64 / LPT) : Batch<G, 2>::TILES;
        const dim3 grid((T + tiles - 1) / tiles), block(256);
        auto launch = [&](auto ranked, auto pivots) {
            if constexpr (by_wave)
                q(k_quant_by_wave<G, BF16, LOW, ranked.value, pivots.value, LPT>, grid, block, d_in, packed, T, tau, eps_ratio, how, pro);
            else
                q(k_quant_pack<G, LOW, ranked.value, pivots.value>, grid, block, d_in, packed, T, tau, eps_ratio, how, pro);
        };
        if constexpr (BF16 && LPT == Lanes<G, 2>::usual) {
            if (widths == Widths::ranked_with_pivots) { launch(std::true_type{}, std::true_type{}); return; }
        }
        if (widths == Widths::one) launch(std::false_type{}, std::false_type{});
        else launch(std::true_type{}, std::false_type{});
    }
    template <int LOW>
    static void go(const void *d_in, uint8_t *packed, uint32_t T, float tau, float eps_ratio, Widths widths,
                   uint32_t how, const CrewPlan &crew, const Prologue &pro, Enqueue *qp)
    {
        using N = Lanes<G, BF16 ? 2 : 4>;
        // (the tensors that k_rank_quant takes are quantized by as many lanes per tile when the phases are apart)
        if (crew.batch != 0 ? crew.few : few_tiles<N>(T, 2)) with<LOW, N::few>(d_in, packed, T, tau, eps_ratio, widths, how, pro, qp);
        else if (crew.batch != 0) with<LOW, kCrewHalf<G, BF16>>(d_in, packed, T, tau, eps_ratio, widths, how, pro, qp);
        else with<LOW, N::usual>(d_in, packed, T, tau, eps_ratio, widths, how, pro, qp);
    }
    static void run(uint32_t low, const void *d_in, uint8_t *packed, uint32_t T, float tau, float eps_ratio,
                    Widths widths, uint32_t how, CrewPlan crew, Prologue pro, Enqueue *qp)
    {
        switch (low) {
        case 1: go<1>(d_in, packed, T, tau, eps_ratio, widths, how, crew, pro, qp); break;
        case 2: go<2>(d_in, packed, T, tau, eps_ratio, widths, how, crew, pro, qp); break;
        case 3: go<3>(d_in, packed, T, tau, eps_ratio, widths, how, crew, pro, qp); break;
        case 4: go<4>(d_in, packed, T, tau, eps_ratio, widths, how, crew, pro, qp); break;
        case 5: go<5>(d_in, packed, T, tau, eps_ratio, widths, how, crew, pro, qp); break;
        case 6: go<6>(d_in, packed, T, tau, eps_ratio, widths, how, crew, pro, qp); break;
        default: go<7>(d_in, packed, T, tau, eps_ratio, widths, how, crew, pro, qp); break;
        }
    }
};

template <int G, bool BF16>
struct LaunchDecode {
    template <int LOW>
    static void go(const uint8_t *packed, void *d_out, uint32_t T, uint32_t total_wide, Enqueue *qp)
    {
        using N = Lanes<G, BF16 ? 2 : 4>;
        if (few_tiles<N>(T, 4)) with<LOW, N::few>(packed, d_out, T, total_wide, qp);
        else with<LOW, N::usual>(packed, d_out, T, total_wide, qp);
    }
    template <int LOW, int LPT>
    static void with(const uint8_t *packed, void *d_out, uint32_t T, uint32_t total_wide, Enqueue *qp)
    {
        Enqueue &q = *qp;
        using W = Wave<G, BF16 ? 2 : 4, LPT>;
        const uint32_t groups = (T + W::TILES - 1) / W::TILES;
        q(k_decode<G, BF16, LOW, LPT>, dim3((groups + 3) / 4), dim3(256), packed, d_out, T, total_wide);
    }
    static void run(uint32_t low, const uint8_t *packed, void *d_out, uint32_t T, uint32_t total_wide,
                    Enqueue *qp)
    {
        switch (low) {
        case 1: go<1>(packed, d_out, T, total_wide, qp); break;
        case 2: go<2>(packed, d_out, T, total_wide, qp); break;
        case 3: go<3>(packed, d_out, T, total_wide, qp); break;
        case 4: go<4>(packed, d_out, T, total_wide, qp); break;
        case 5: go<5>(packed, d_out, T, total_wide, qp); break;
        case 6: go<6>(packed, d_out, T, total_wide, qp); break;
        default: go<7>(packed, d_out, T, total_wide, qp); break;
        }
    }
};

template <int G, bool BF16>
struct LaunchAllocEntropy {
    using N = Lanes<G, BF16 ? 2 : 4>;
    template <int LPT, bool WAVE_TEAM>
    static void go(const void *d_in, float *d_H, uint8_t *pivot, uint32_t n_alloc, uint32_t m, const EntropyParams &p,
                   const Prologue &pro, Enqueue *qp)
    {
        Enqueue &q = *qp;
        constexpr uint32_t SLOTS = (WAVE_TEAM ? 64 : 256) / LPT, TEAMS = WAVE_TEAM ? 4 : 1;
        const uint32_t per = SLOTS / m, nb = (n_alloc + per * TEAMS - 1) / (per * TEAMS);
        static ResidentCache cache;
        auto launch = [&](auto kernel, auto... params) {
            const uint32_t res = resident_blocks(reinterpret_cast<const void *>(kernel), 256, cache);
            const uint32_t grid = nb < res ? nb : res, pro_blocks = prologue_blocks(pro, 256, grid);
            if constexpr (sizeof...(params) != 0)
                q(kernel, dim3(grid), dim3(256), d_in, d_H, pivot, n_alloc, grid, m, per, p.eps_l1, p.eps_log, pro_blocks, params..., pro);
            else q(kernel, dim3(grid), dim3(256), d_in, d_H, n_alloc, grid, m, per, p.eps_l1, p.eps_log, pro_blocks, pro);
        };
        if constexpr (LPT == N::usual && WAVE_TEAM) launch(k_alloc_entropy<G, BF16>, p.tau, p.eps_ratio);
        else launch(k_alloc_entropy_by<G, BF16, LPT, WAVE_TEAM>);
    }
    // A wavefront by itself where it wastes no more lanes than a workgroup would: as many allocation tiles per workgroup.
    template <int LPT>
    static bool by_wave(uint32_t m) { return 4 * (64 / LPT / m) >= 256 / LPT / m; }
    template <int LPT>
    static void one_pass(const void *d_in, float *d_H, uint8_t *pivot, uint32_t n_alloc, uint32_t m, const EntropyParams &p,
                         const Prologue &pro, Enqueue *qp)
    {
        if (by_wave<LPT>(m)) go<LPT, true>(d_in, d_H, pivot, n_alloc, m, p, pro, qp);
        else go<LPT, false>(d_in, d_H, pivot, n_alloc, m, p, pro, qp);
    }
    // Whether it is k_alloc_entropy that a call of T tiles takes, and that with Eq. 3.
    static bool pivots(uint32_t T, uint32_t m)
    {
        const bool few = few_tiles<N>(T, 4) && m <= 256 / N::few;
        return kWholeTiles<G, BF16> && !few && m <= 256 / N::usual && by_wave<N::usual>(m);
    }
    // Entropies of allocation tiles of m > 1 quantization tiles: one pass if a workgroup's lanes hold whole
    // allocation tiles, otherwise two streaming passes over the tensor.
    static void run(const void *d_in, float *d_H, float *part, float *inv_norm, uint8_t *pivot, uint32_t T, uint32_t m, EntropyParams p,
                    Prologue pro, Enqueue *qp)
    {
        Enqueue &q = *qp;
        const uint32_t n_alloc = T / m;
        if (few_tiles<N>(T, 4) && m <= 256 / N::few) { one_pass<N::few>(d_in, d_H, pivot, n_alloc, m, p, pro, qp); return; }
        if (m <= 256 / N::usual) { one_pass<N::usual>(d_in, d_H, pivot, n_alloc, m, p, pro, qp); return; }
        using B = Batch<G, BF16 ? 2 : 4>;
        const uint32_t nb = (T + B::TILES - 1) / B::TILES;
        q(k_tile_partial<G, BF16, false>, dim3(nb), dim3(B::TILES), d_in,
                           (const float *)nullptr, part, T, m, p.eps_log, prologue_blocks(pro, B::TILES, nb), pro);
        q(k_alloc_reduce<false>, dim3(blocks_for(n_alloc)), dim3(256), (const float *)part, (const float *)nullptr,
                           inv_norm, n_alloc, m, p.eps_l1);
        q(k_tile_partial<G, BF16, true>, dim3(nb), dim3(B::TILES), d_in,
                           (const float *)inv_norm, part, T, m, p.eps_log, 0u, Prologue{});
        q(k_alloc_reduce<true>, dim3(blocks_for(n_alloc)), dim3(256), (const float *)part, (const float *)inv_norm,
                           d_H, n_alloc, m, p.eps_l1);
    }
};

// Whether the entropies of a call come with Eq. 3.
template <int G, bool BF16>
struct EntropyPivots {
    static void run(uint32_t T, uint32_t m, bool *pivots)
    {
        *pivots = m == 1 ? LaunchEntropy<G, BF16>::pivots(T) : LaunchAllocEntropy<G, BF16>::pivots(T, m);
    }
};

// Entropy of every quantization tile; with `pivot`, also Eq. 3; with `hist`, also the selection's first histogram (the caller has
// checked that the ranking units are whole steps).
void launch_entropy(const Shape &s, const tahq_config *cfg, const void *d_in, float *d_H, uint8_t *pivot, bool approx, uint32_t *hist,
                    uint32_t bins, float bin_scale, const Prologue &pro, Enqueue *qp)
{
    EntropyParams p = entropy_params(cfg);
    p.approx = approx;
    dispatch<LaunchEntropy>(s.G, s.dtype == TAHQ_BF16, d_in, d_H, pivot, (uint32_t)s.T, p, hist, bins, bin_scale, s.n, pro, qp);
}

// The first launch of the two-launch selection, with approximate entropies (bf16).
template <int G, bool BF16>
struct LaunchClassify {
    static void run(dim3 grid, float *H, const Shape &s, uint32_t u0, float bin_scale, const uint32_t *lin_hist, uint32_t *fused,
                    uint2 *cand, uint2 *block_counts, uint32_t *crowd_hist, uint64_t *bitmap, const void *d_in, EntropyParams p,
                    Enqueue *qp)
    {
        (*qp)(k_select_classify<G, true, true>, grid, dim3(kFusedThreads), H, (uint32_t)s.n, (uint32_t)s.k, u0, bin_scale, lin_hist, fused,
              cand, block_counts, crowd_hist, bitmap, d_in, p.eps_l1, p.eps_log, kEntropySlack);
    }
};

template <uint32_t PLACES, uint32_t BINS, int SHIFT>
void launch_select_small(dim3 grid, const float *H, uint32_t n, uint32_t k, const Shape &s, uint64_t *bitmap, uint32_t *ranks,
                         Enqueue *qp)
{
    (*qp)(k_select_small<PLACES, BINS, SHIFT>, grid, dim3(kSmallUnitThreads), H, n, k, s.m, lowest_bin<BINS, SHIFT>(s), bitmap, ranks);
}

// ---- backward-pass fixed-point compressor

struct NaiveShape {
    uint64_t N;          // elements
    uint32_t nchunks;    // chunks of 32 elements
    uint32_t bits, dtype;
    uint64_t total;      // stream bytes
};

tahq_status make_naive_shape(const tahq_naive_config *c, NaiveShape *s)
{
    if (!c) return TAHQ_ERR_NULL;
    if (c->struct_size != sizeof(tahq_naive_config)) return TAHQ_ERR_INVALID_ARG;
    if (c->batch == 0 || c->seq == 0 || c->hidden == 0 || c->hidden % kNaiveChunk != 0) return TAHQ_ERR_INVALID_ARG;
    if (c->dtype > TAHQ_BF16 || c->bits < 2 || c->bits > 16) return TAHQ_ERR_INVALID_ARG;
    if (!(c->scale > 0.0f) || c->scale > 3.4028234663852886e38f) return TAHQ_ERR_INVALID_ARG;
    const uint64_t N = (uint64_t)c->batch * c->seq * c->hidden;
    if (N > (1ull << 36)) return TAHQ_ERR_INVALID_ARG;
    s->N = N;
    s->nchunks = (uint32_t)(N / kNaiveChunk);
    s->bits = c->bits;
    s->dtype = c->dtype;
    s->total = 64 + N * c->bits / 8;
    return TAHQ_OK;
}

template <int BITS>
void launch_naive_encode(bool bf16, const void *d_in, uint8_t *packed, const NaiveHeader &hdr, uint32_t nchunks,
                         float scale, Enqueue *qp)
{
    Enqueue &q = *qp;
    const dim3 grid((nchunks + kNaiveChunks - 1) / kNaiveChunks), block(kNaiveChunks);
    if (bf16) q(k_naive_encode<BITS, true>, grid, block, d_in, packed, nchunks, scale, hdr);
    else q(k_naive_encode<BITS, false>, grid, block, d_in, packed, nchunks, scale, hdr);
}

template <int BITS>
void launch_naive_decode(bool out_bf16, const uint8_t *packed, void *d_out, uint32_t nchunks, float inv_scale,
                         Enqueue *qp)
{
    Enqueue &q = *qp;
    const dim3 grid((nchunks + kNaiveChunks - 1) / kNaiveChunks), block(kNaiveChunks);
    if (out_bf16) q(k_naive_decode<BITS, true>, grid, block, packed, d_out, nchunks, inv_scale);
    else q(k_naive_decode<BITS, false>, grid, block, packed, d_out, nchunks, inv_scale);
}

// Every supported code width, for the switch over the run-time width.
#define TAHQ_NAIVE_WIDTHS(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

}  // namespace

// ------------------------------------------------------------------ C ABI

extern "C" {

void tahq_config_default(tahq_config *cfg)
{
    if (!cfg) return;
    memset(cfg, 0, sizeof *cfg);
    cfg->struct_size = (uint32_t)sizeof *cfg;
    cfg->tile = 64;
    cfg->dtype = TAHQ_BF16;
    cfg->scope = 0;
    cfg->budget_bits = 3.8f;
    cfg->tau = 2.0f;
    cfg->eps_l1 = 1e-8f;
    cfg->eps_log = 1e-8f;
    cfg->eps_ratio = 1e-8f;
}

uint64_t tahq_k_per_unit(const tahq_config *cfg)
{
    Shape s;
    if (make_shape(cfg, &s) != TAHQ_OK) return 0;
    return s.kA;
}

size_t tahq_packed_size(const tahq_config *cfg)
{
    Shape s;
    if (make_shape(cfg, &s) != TAHQ_OK) return 0;
    return (size_t)stream_bytes(s);
}

size_t tahq_workspace_size(const tahq_config *cfg)
{
    Shape s;
    if (make_shape(cfg, &s) != TAHQ_OK) return 0;
    Workspace w;
    make_workspace(s, &w);
    return (size_t)w.total;
}

tahq_status tahq_tile_entropy(const tahq_config *cfg, const void *d_in, float *d_entropy, tahq_stream stream)
{
    Shape s;
    tahq_status rc = make_shape(cfg, &s);
    if (rc != TAHQ_OK) return rc;
    if (!d_in || !d_entropy) return TAHQ_ERR_NULL;
    if (misaligned(d_in) || misaligned(d_entropy)) return TAHQ_ERR_MISALIGNED;
    Enqueue q{(hipStream_t)stream};
    launch_entropy(s, cfg, d_in, d_entropy, nullptr, false, nullptr, 0u, 0.0f, Prologue{}, &q);
    return q.result();
}

tahq_status tahq_alloc_tile_entropy(const tahq_config *cfg, const void *d_in, float *d_entropy, void *d_workspace,
                                    size_t workspace_capacity, tahq_stream stream)
{
    Shape s;
    tahq_status rc = make_shape(cfg, &s);
    if (rc != TAHQ_OK) return rc;
    if (!d_in || !d_entropy) return TAHQ_ERR_NULL;
    if (misaligned(d_in) || misaligned(d_entropy)) return TAHQ_ERR_MISALIGNED;
    Enqueue q{(hipStream_t)stream};
    if (s.m == 1) {
        launch_entropy(s, cfg, d_in, d_entropy, nullptr, false, nullptr, 0u, 0.0f, Prologue{}, &q);
    } else {
        if (!d_workspace) return TAHQ_ERR_NULL;
        Workspace ws;
        make_workspace(s, &ws);
        if (workspace_capacity < ws.total) return TAHQ_ERR_WORKSPACE_TOO_SMALL;
        if (misaligned(d_workspace)) return TAHQ_ERR_MISALIGNED;
        uint8_t *wsb = static_cast<uint8_t *>(d_workspace);
        dispatch<LaunchAllocEntropy>(s.G, s.dtype == TAHQ_BF16, d_in, d_entropy,
                                     reinterpret_cast<float *>(wsb + ws.part),
                                     reinterpret_cast<float *>(wsb + ws.inv_norm), (uint8_t *)nullptr, (uint32_t)s.T, s.m,
                                     entropy_params(cfg), Prologue{}, &q);
    }
    return q.result();
}

tahq_status tahq_encode_phases(const tahq_config *cfg, const void *d_in, void *d_packed, size_t packed_capacity,
                               void *d_workspace, size_t workspace_capacity, uint32_t phases, tahq_stream stream)
{
    const bool multi_launch = (phases & TAHQ_SELECT_MULTI_LAUNCH) != 0;
    phases &= ~(uint32_t)TAHQ_SELECT_MULTI_LAUNCH;
    if (phases == 0 || (phases & ~(uint32_t)TAHQ_PHASE_ALL)) return TAHQ_ERR_INVALID_ARG;
    Shape s;
    tahq_status rc = make_shape(cfg, &s);
    if (rc != TAHQ_OK) return rc;
    if (!d_in || !d_packed || !d_workspace) return TAHQ_ERR_NULL;
    const Sections lay((uint32_t)s.T);
    Workspace ws;
    make_workspace(s, &ws);
    if (packed_capacity < stream_bytes(s)) return TAHQ_ERR_BUFFER_TOO_SMALL;
    if (workspace_capacity < ws.total) return TAHQ_ERR_WORKSPACE_TOO_SMALL;
    if (misaligned(d_in) || misaligned(d_packed) || misaligned(d_workspace)) return TAHQ_ERR_MISALIGNED;

    Enqueue q{(hipStream_t)stream};
    uint8_t *packed = static_cast<uint8_t *>(d_packed);
    uint8_t *wsb = static_cast<uint8_t *>(d_workspace);
    uint64_t *bitmap = reinterpret_cast<uint64_t *>(packed + lay.bitmap);
    uint32_t *ranks = reinterpret_cast<uint32_t *>(packed + lay.ranks);
    const bool select = s.kA != 0 && s.kA != s.nA;
    const bool wide = s.m > 1;     // allocation tiles of several quantization tiles
    // Tensors of one round of workgroups are ranked where they are quantized, unless the caller has the phases apart.
    const uint64_t places = s.nA + (!wide && s.n % 64 != 0 ? 63u : 0u);       // counted from a 64-tile boundary
    CrewPlan crew = {0, false, false};
    if (select && !wide && !approximate_entropies(s, cfg))
        crew = plan_rank_quant(s, places);
    constexpr uint32_t together = TAHQ_PHASE_ENTROPY | TAHQ_PHASE_SELECT | TAHQ_PHASE_QUANT;
    const bool ranked_in_quant = crew.batch != 0 && !multi_launch && (phases & together) == together;
    // Otherwise ranking units that one workgroup can hold are ranked in a single launch, from LDS or from registers.  (Not where the
    // two-launch selection's approximate entropies save more: [16,1024,4096] 77.8 us so, 80.5 with exact ones; and as long as every
    // unit has a compute unit.)
    const bool mid_units = select && !wide && !multi_launch && places > kSmallUnitMaxKeys && places <= kMidPlaces && s.U <= 256 &&
                           !approximate_entropies(s, cfg);
    const bool small_units = (select && places <= kSmallUnitMaxKeys && !multi_launch) || mid_units || ranked_in_quant;
    // Large units are ranked in two launches from a histogram of linear bins that the entropy kernel builds; allocation
    // tiles, and every unit when the caller forces it, by the multi-launch radix select, whose first digit the entropy
    // kernel counts where units are whole batches.
    const bool fused_select = select && !wide && !small_units && !multi_launch;
    const bool approx = fused_select && approximate_entropies(s, cfg);
    // Eq. 3 rides in the entropy pass with approximate entropies, and where it is the better place for it with exact ones.
    bool pivots = approx;
    if (select && !approx && crew.batch == 0) dispatch<EntropyPivots>(s.G, s.dtype == TAHQ_BF16, (uint32_t)s.T, s.m, &pivots);

    // The multi-launch selection puts the unit into the grid's second dimension.  (The two-launch selection does so too, in
    // slices: 65536 units and more of 32706 to 32767 tiles each are a tensor of fewer than 2^31.)
    if (select && multi_launch && s.U > kMaxGridY) return TAHQ_ERR_UNSUPPORTED;

    // header and section padding
    Prologue pro;
    memset(&pro, 0, sizeof pro);
    uint32_t *hdr = pro.hdr.w;
    hdr[0] = 0x51484154u;   // "TAHQ"
    hdr[1] = 1;
    hdr[2] = s.dtype; hdr[3] = s.B; hdr[4] = s.S; hdr[5] = s.C; hdr[6] = s.G; hdr[7] = s.scope;
    hdr[8] = (uint32_t)s.kA;
    hdr[14] = s.A;
    hdr[15] = s.low;
    memcpy(&hdr[9], &cfg->budget_bits, 4);
    memcpy(&hdr[10], &cfg->tau, 4);
    memcpy(&hdr[11], &cfg->eps_l1, 4);
    memcpy(&hdr[12], &cfg->eps_log, 4);
    memcpy(&hdr[13], &cfg->eps_ratio, 4);
    const uint64_t words64 = (s.T + 63) / 64;
    const uint64_t sec_begin[5] = {lay.bitmap + words64 * 8, lay.ranks + words64 * 4, lay.pivot + s.T,
                                   lay.scale + 2 * s.T, lay.zero + 2 * s.T};
    const uint64_t sec_end[5] = {lay.ranks, lay.pivot, lay.scale, lay.zero, lay.payload};
    for (int i = 0; i < 5; ++i) { pro.pads.begin[i] = sec_begin[i]; pro.pads.len[i] = (uint32_t)(sec_end[i] - sec_begin[i]); }
    pro.bitmap = bitmap;
    pro.unit_tiles = (uint32_t)s.n;
    // The prologue is part of the call's first kernel: of the quantizer where there is nothing to rank, of the entropies where the
    // selection has no scratch to clear.  Where it has, that must have happened before the entropies are counted.
    const bool histograms = select && !small_units;
    const bool all_in_quant = !select && (phases & (uint32_t)TAHQ_PHASE_QUANT) && (phases & (uint32_t)TAHQ_PHASE_PROLOGUE) &&
                              (phases & (uint32_t)TAHQ_PHASE_SELECT);
    const bool with_entropy = select && !histograms && (phases & (uint32_t)TAHQ_PHASE_PROLOGUE) && (phases & (uint32_t)TAHQ_PHASE_ENTROPY);
    if (phases & TAHQ_PHASE_PROLOGUE) pro.packed = packed;
    if ((phases & TAHQ_PHASE_PROLOGUE) && !all_in_quant && !with_entropy) {
        const uint64_t zero_from = multi_launch || wide ? ws.coarse : ws.hist0;          // what this selection counts in
        const uint32_t zero_words = histograms ? (uint32_t)((ws.zero_bytes - zero_from) / 4) : 0u;
        const uint32_t zero_blocks = blocks_for(zero_words) < 256u ? blocks_for(zero_words) : 256u;
        q(k_prologue, dim3(zero_blocks ? zero_blocks : 1u), dim3(256), pro, reinterpret_cast<uint32_t *>(wsb + zero_from), zero_words);
        pro.packed = nullptr;
    }
    // words of the bit map that units share are cleared with the entropies, for the selection that follows them
    if (select && !multi_launch && (small_units || !wide) && s.n % 64 != 0) pro.edge_units = s.U;

    if (select) {
        float *H = reinterpret_cast<float *>(wsb + ws.keys);
        uint32_t *hist0 = reinterpret_cast<uint32_t *>(wsb + ws.hist0);
        uint32_t *coarse = reinterpret_cast<uint32_t *>(wsb + ws.coarse);
        uint32_t *partial = reinterpret_cast<uint32_t *>(wsb + ws.partial);
        uint32_t *state = reinterpret_cast<uint32_t *>(wsb + ws.state);
        uint32_t *seg = reinterpret_cast<uint32_t *>(wsb + ws.seg);
        uint8_t *sel = wsb + ws.sel;
        bool fused = false;
        if (!wide && multi_launch) dispatch<CanFuse>(s.G, s.dtype == TAHQ_BF16, s.n, &fused);
        uint32_t *lin_hist = reinterpret_cast<uint32_t *>(wsb + ws.lin_hist);
        // bins of width ln(A) / kLinBins: the entropy of A channels lies in [0, ln A]
        const float bin_scale = (float)((double)kLinBins / __builtin_log((double)s.A));
        uint8_t *pivot = pivots ? packed + lay.pivot : nullptr;
        if (phases & TAHQ_PHASE_ENTROPY) {
            if (wide)
                dispatch<LaunchAllocEntropy>(s.G, s.dtype == TAHQ_BF16, d_in, H, reinterpret_cast<float *>(wsb + ws.part),
                                             reinterpret_cast<float *>(wsb + ws.inv_norm), pivot, (uint32_t)s.T,
                                             s.m, entropy_params(cfg), pro, &q);
            else if (fused_select)
                launch_entropy(s, cfg, d_in, H, pivot, approx, lin_hist, kLinBins, bin_scale, pro, &q);
            else
                launch_entropy(s, cfg, d_in, H, pivot, false, fused ? hist0 : (uint32_t *)nullptr, kDigit0Bins, 0.0f, pro, &q);
        }
        if ((phases & TAHQ_PHASE_SELECT) && fused_select) {
            uint32_t *fused_state = reinterpret_cast<uint32_t *>(wsb + ws.fused);
            uint2 *cand = reinterpret_cast<uint2 *>(wsb + ws.cand);
            uint2 *block_counts = reinterpret_cast<uint2 *>(seg);          // fewer entries than the segments it was made for
            for (uint32_t u0 = 0; u0 < s.U; u0 += kMaxGridY) {
                const dim3 grid((uint32_t)((places + kFusedKeysPerBlock - 1) / kFusedKeysPerBlock),
                                s.U - u0 < kMaxGridY ? s.U - u0 : kMaxGridY);
                if (approx)
                    dispatch<LaunchClassify>(s.G, true, grid, H, s, u0, bin_scale, (const uint32_t *)lin_hist, fused_state, cand,
                                             block_counts, hist0, bitmap, d_in, entropy_params(cfg), &q);
                else
                    q(k_select_classify<64, true, false>, grid, dim3(kFusedThreads), H, (uint32_t)s.n, (uint32_t)s.k, u0, bin_scale,
                      (const uint32_t *)lin_hist, fused_state, cand, block_counts, hist0, bitmap, d_in, 0.0f, 0.0f, 0.0f);
                q(k_select_resolve, grid, dim3(kFusedThreads), (const float *)H, (uint32_t)s.n,
                                   (uint32_t)s.k, u0, bin_scale, approx ? 2.0f * kEntropySlack : 0.0f, (const uint32_t *)lin_hist,
                                   fused_state, cand, (const uint2 *)block_counts, (const uint32_t *)hist0,
                                   reinterpret_cast<uint64_t *>(sel), bitmap, ranks);
            }
        } else if (ranked_in_quant) {
            launch_rank_quant(H, d_in, packed, s, places, crew, cfg->tau, cfg->eps_ratio, &q);
        } else if ((phases & TAHQ_PHASE_SELECT) && small_units) {
            const uint32_t n32 = (uint32_t)s.nA, k32 = (uint32_t)s.kA;
            // with A > G every workgroup expands a part of the unit's bit map (a unit may start inside a word)
            const uint64_t unit_words = s.n / 64 + 2;
            const dim3 grid(s.U, wide ? (uint32_t)((unit_words + kExpandWords - 1) / kExpandWords) : 1u);
            // as little LDS as will do; the largest units leave room for half as many bins
            if (mid_units)
                q(k_select_mid, grid, dim3(kSmallUnitThreads), (const float *)H, n32, k32, lowest_bin<kMidBins, kMidShift>(s), bitmap,
                  ranks);
            else if (places <= 4096) launch_select_small<4096, 8192, 12>(grid, H, n32, k32, s, bitmap, ranks, &q);
            else if (places <= 16384) launch_select_small<16384, 8192, 12>(grid, H, n32, k32, s, bitmap, ranks, &q);
            else if (places <= 28672) launch_select_small<28672, 8192, 12>(grid, H, n32, k32, s, bitmap, ranks, &q);
            else launch_select_small<kSmallUnitMaxKeys, 4096, 13>(grid, H, n32, k32, s, bitmap, ranks, &q);
        } else if (phases & TAHQ_PHASE_SELECT) {
            // the selection ranks allocation tiles; with A = G they are the stream's tiles
            const uint32_t n32 = (uint32_t)s.nA, k32 = (uint32_t)s.kA;
            const dim3 rgrid(ws.hb, s.U);
            if (!fused)
                q(k_radix_pass<0, 8>, rgrid, dim3(256), (const float *)H, n32, k32, hist0, coarse, partial, state);
            q(k_radix_pass<1, 0>, rgrid, dim3(256), (const float *)H, n32, k32, hist0, coarse, partial, state);
            q(k_radix_pass<2, 0>, rgrid, dim3(256), (const float *)H, n32, k32, hist0, coarse, partial, state);
            const uint32_t sb = (ws.nseg + 3) / 4;
            q(k_seg_count, dim3(sb, s.U), dim3(256), (const float *)H, n32, ws.nseg,
                               (const uint32_t *)coarse, (const uint32_t *)partial, ws.hb, state, seg);
            const int aligned = (!wide && s.n % 64 == 0) ? 1 : 0;
            uint32_t *ranks_a = reinterpret_cast<uint32_t *>(wsb + ws.ranks_a);
            q(k_assign, dim3(sb, s.U), dim3(256), (const float *)H, n32, k32, ws.nseg,
                               (const uint32_t *)state, (const uint32_t *)seg, bitmap, wide ? ranks_a : ranks, sel,
                               aligned);
            if (wide)
                q(k_expand_alloc, dim3(blocks_for(words64 * 64)), dim3(256),
                                   (const uint8_t *)sel, (const uint32_t *)ranks_a, (uint32_t)s.T, s.m, bitmap, ranks);
            else if (!aligned)
                q(k_bitmap_pack, dim3(blocks_for(words64 * 64)), dim3(256),
                                   (const uint8_t *)sel, (uint32_t)s.T, bitmap);
        }
    } else if ((phases & TAHQ_PHASE_SELECT) && !all_in_quant) {
        q(k_bitmap_const, dim3(blocks_for(words64)), dim3(256), (uint32_t)s.T,
                           s.kA == s.nA ? 1 : 0, bitmap, ranks);
    }

    if ((phases & TAHQ_PHASE_QUANT) && !ranked_in_quant) {
        dispatch<LaunchQuantPack>(s.G, s.dtype == TAHQ_BF16, s.low, d_in, packed, (uint32_t)s.T, cfg->tau,
                                  cfg->eps_ratio, !select ? Widths::one : pivots ? Widths::ranked_with_pivots : Widths::ranked,
                                  (s.kA == s.nA ? QUANT_ALL_WIDE : 0u) | (stream_bytes(s) >= kStreamingFrom ? QUANT_STREAMING : 0u),
                                  crew, pro, &q);
    }
    return q.result();
}

tahq_status tahq_encode(const tahq_config *cfg, const void *d_in, void *d_packed, size_t packed_capacity,
                        void *d_workspace, size_t workspace_capacity, tahq_stream stream)
{
    return tahq_encode_phases(cfg, d_in, d_packed, packed_capacity, d_workspace, workspace_capacity,
                              TAHQ_PHASE_ALL, stream);
}

tahq_status tahq_encode_noalloc(const tahq_config *cfg, const void *d_in, void *d_packed, size_t packed_capacity,
                                tahq_stream stream)
{
    Shape s;
    tahq_status rc = make_shape(cfg, &s);
    if (rc != TAHQ_OK) return rc;
    Workspace ws;
    make_workspace(s, &ws);
    if (ws.total > kBuiltinScratchBytes) return TAHQ_ERR_TOO_LARGE;
    if (!d_in || !d_packed) return TAHQ_ERR_NULL;
    if (packed_capacity < stream_bytes(s)) return TAHQ_ERR_BUFFER_TOO_SMALL;
    if (misaligned(d_in) || misaligned(d_packed)) return TAHQ_ERR_MISALIGNED;
    // the current device's copy of the built-in scratch: looked up once per device, with that device current
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TAHQ_ERR_HIP;
    void *ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        ptr = g_scratch_ptr[dev];
        if (!ptr) {
            if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return TAHQ_ERR_HIP;
            g_scratch_ptr[dev] = ptr;
        }
    }
    // what must start at zero in there (the selection's histograms and state) is cleared by the encoder's
    // first kernel, as it is in a caller's workspace
    return tahq_encode_phases(cfg, d_in, d_packed, packed_capacity, ptr, kBuiltinScratchBytes, TAHQ_PHASE_ALL, stream);
}

tahq_status tahq_decode(const tahq_config *cfg, const void *d_packed, size_t packed_bytes, void *d_out,
                        uint32_t out_dtype, void *d_workspace, size_t workspace_capacity, tahq_stream stream)
{
    (void)d_workspace;
    (void)workspace_capacity;
    Shape s;
    tahq_status rc = make_shape(cfg, &s);
    if (rc != TAHQ_OK) return rc;
    if (out_dtype > TAHQ_BF16) return TAHQ_ERR_INVALID_ARG;
    if (!d_packed || !d_out) return TAHQ_ERR_NULL;
    if (packed_bytes < stream_bytes(s)) return TAHQ_ERR_BUFFER_TOO_SMALL;
    if (misaligned(d_packed) || misaligned(d_out)) return TAHQ_ERR_MISALIGNED;
    Enqueue q{(hipStream_t)stream};
    dispatch<LaunchDecode>(s.G, out_dtype == TAHQ_BF16, s.low, static_cast<const uint8_t *>(d_packed), d_out,
                           (uint32_t)s.T, (uint32_t)(s.U * s.k), &q);
    return q.result();
}

// ---- sample-wise use: a run of samples as a tensor of its own

namespace {
// The configuration of samples [first, first + count) taken as a tensor [count, seq, hidden], and the byte offset
// of the first of them in the whole tensor (element size `esize`).
tahq_status samples_config(const tahq_config *cfg, uint32_t first, uint32_t count, uint32_t esize, tahq_config *sub,
                           uint64_t *offset)
{
    Shape s;
    tahq_status rc = make_shape(cfg, &s);
    if (rc != TAHQ_OK) return rc;
    if (s.scope != 0 || count == 0 || first >= s.B || count > s.B - first) return TAHQ_ERR_INVALID_ARG;
    memset(sub, 0, sizeof *sub);
    memcpy(sub, cfg, cfg->struct_size);          // older, shorter layouts: the missing fields stay 0
    sub->batch = count;
    *offset = (uint64_t)first * s.S * s.C * esize;
    return TAHQ_OK;
}
}  // namespace

size_t tahq_samples_packed_size(const tahq_config *cfg, uint32_t count)
{
    tahq_config sub;
    uint64_t off;
    if (samples_config(cfg, 0, count, 1, &sub, &off) != TAHQ_OK) return 0;
    return tahq_packed_size(&sub);
}

size_t tahq_samples_workspace_size(const tahq_config *cfg, uint32_t count)
{
    tahq_config sub;
    uint64_t off;
    if (samples_config(cfg, 0, count, 1, &sub, &off) != TAHQ_OK) return 0;
    return tahq_workspace_size(&sub);
}

tahq_status tahq_encode_samples(const tahq_config *cfg, uint32_t first, uint32_t count, const void *d_in, void *d_packed,
                                size_t packed_capacity, void *d_workspace, size_t workspace_capacity, tahq_stream stream)
{
    if (!cfg) return TAHQ_ERR_NULL;
    tahq_config sub;
    uint64_t off;
    tahq_status rc = samples_config(cfg, first, count, cfg->dtype == TAHQ_BF16 ? 2u : 4u, &sub, &off);
    if (rc != TAHQ_OK) return rc;
    if (!d_in) return TAHQ_ERR_NULL;
    return tahq_encode(&sub, static_cast<const uint8_t *>(d_in) + off, d_packed, packed_capacity, d_workspace,
                       workspace_capacity, stream);
}

tahq_status tahq_decode_samples(const tahq_config *cfg, uint32_t first, uint32_t count, const void *d_packed,
                                size_t packed_bytes, void *d_out, uint32_t out_dtype, tahq_stream stream)
{
    if (!cfg) return TAHQ_ERR_NULL;
    if (out_dtype > TAHQ_BF16) return TAHQ_ERR_INVALID_ARG;
    tahq_config sub;
    uint64_t off;
    tahq_status rc = samples_config(cfg, first, count, out_dtype == TAHQ_BF16 ? 2u : 4u, &sub, &off);
    if (rc != TAHQ_OK) return rc;
    if (!d_out) return TAHQ_ERR_NULL;
    return tahq_decode(&sub, d_packed, packed_bytes, static_cast<uint8_t *>(d_out) + off, out_dtype, nullptr, 0, stream);
}

tahq_status tahq_parse_header(const void *header64, tahq_config *cfg)
{
    if (!header64 || !cfg) return TAHQ_ERR_NULL;
    uint32_t w[16];
    memcpy(w, header64, 64);
    if (w[0] != 0x51484154u || w[1] != 1u) return TAHQ_ERR_INVALID_ARG;
    tahq_config_default(cfg);
    cfg->dtype = w[2]; cfg->batch = w[3]; cfg->seq = w[4]; cfg->hidden = w[5]; cfg->tile = w[6]; cfg->scope = w[7];
    memcpy(&cfg->budget_bits, &w[9], 4);
    memcpy(&cfg->tau, &w[10], 4);
    memcpy(&cfg->eps_l1, &w[11], 4);
    memcpy(&cfg->eps_log, &w[12], 4);
    memcpy(&cfg->eps_ratio, &w[13], 4);
    cfg->alloc_tile = w[14];
    cfg->low_bits = w[15];
    Shape s;
    tahq_status rc = make_shape(cfg, &s);
    if (rc != TAHQ_OK) return rc;
    return s.kA == w[8] ? TAHQ_OK : TAHQ_ERR_INVALID_ARG;
}

const char *tahq_status_string(tahq_status s)
{
    switch (s) {
    case TAHQ_OK: return "ok";
    case TAHQ_ERR_NULL: return "a required pointer is NULL";
    case TAHQ_ERR_INVALID_ARG: return "invalid argument";
    case TAHQ_ERR_UNSUPPORTED: return "unsupported tile width or tensor too large";
    case TAHQ_ERR_BUFFER_TOO_SMALL: return "packed buffer too small";
    case TAHQ_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
    case TAHQ_ERR_MISALIGNED: return "device pointer not 16-byte aligned";
    case TAHQ_ERR_HIP: return "kernel launch failed";
    case TAHQ_ERR_TOO_LARGE: return "configuration needs more scratch than the built-in buffer of tahq_encode_noalloc holds";
    }
    return "unknown status";
}

uint32_t tahq_version(void) { return (1u << 16) | 1u; }

void tahq_naive_config_default(tahq_naive_config *cfg)
{
    if (!cfg) return;
    memset(cfg, 0, sizeof *cfg);
    cfg->struct_size = (uint32_t)sizeof *cfg;
    cfg->dtype = TAHQ_BF16;
    cfg->bits = 8;
    cfg->scale = 1.0f;
}

size_t tahq_naive_packed_size(const tahq_naive_config *cfg)
{
    NaiveShape s;
    if (make_naive_shape(cfg, &s) != TAHQ_OK) return 0;
    return (size_t)s.total;
}

tahq_status tahq_naive_encode(const tahq_naive_config *cfg, const void *d_in, void *d_packed, size_t packed_capacity,
                              tahq_stream stream)
{
    NaiveShape s;
    tahq_status rc = make_naive_shape(cfg, &s);
    if (rc != TAHQ_OK) return rc;
    if (!d_in || !d_packed) return TAHQ_ERR_NULL;
    if (packed_capacity < s.total) return TAHQ_ERR_BUFFER_TOO_SMALL;
    if (misaligned(d_in) || misaligned(d_packed)) return TAHQ_ERR_MISALIGNED;
    NaiveHeader hdr;
    memset(&hdr, 0, sizeof hdr);
    hdr.w[0] = 0x4e484154u;   // "TAHN"
    hdr.w[1] = 1;
    hdr.w[2] = cfg->dtype; hdr.w[3] = cfg->batch; hdr.w[4] = cfg->seq; hdr.w[5] = cfg->hidden; hdr.w[6] = cfg->bits;
    memcpy(&hdr.w[7], &cfg->scale, 4);
    uint8_t *packed = static_cast<uint8_t *>(d_packed);
    const bool bf16 = cfg->dtype == TAHQ_BF16;
    Enqueue q{(hipStream_t)stream};
    switch (cfg->bits) {
#define X(B) case B: launch_naive_encode<B>(bf16, d_in, packed, hdr, s.nchunks, cfg->scale, &q); break;
        TAHQ_NAIVE_WIDTHS(X)
#undef X
    default: return TAHQ_ERR_INVALID_ARG;
    }
    return q.result();
}

tahq_status tahq_naive_decode(const tahq_naive_config *cfg, const void *d_packed, size_t packed_bytes, void *d_out,
                              uint32_t out_dtype, tahq_stream stream)
{
    NaiveShape s;
    tahq_status rc = make_naive_shape(cfg, &s);
    if (rc != TAHQ_OK) return rc;
    if (out_dtype > TAHQ_BF16) return TAHQ_ERR_INVALID_ARG;
    if (!d_packed || !d_out) return TAHQ_ERR_NULL;
    if (packed_bytes < s.total) return TAHQ_ERR_BUFFER_TOO_SMALL;
    if (misaligned(d_packed) || misaligned(d_out)) return TAHQ_ERR_MISALIGNED;
    const float inv_scale = 1.0f / cfg->scale;      // rounded once, on the host
    const uint8_t *packed = static_cast<const uint8_t *>(d_packed);
    Enqueue q{(hipStream_t)stream};
    switch (cfg->bits) {
#define X(B) case B: launch_naive_decode<B>(out_dtype == TAHQ_BF16, packed, d_out, s.nchunks, inv_scale, &q); break;
        TAHQ_NAIVE_WIDTHS(X)
#undef X
    default: return TAHQ_ERR_INVALID_ARG;
    }
    return q.result();
}

}  // extern "C"


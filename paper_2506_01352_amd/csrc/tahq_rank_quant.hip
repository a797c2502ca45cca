// TAH-Quant activation codec for gfx950: the launch that ranks and quantizes small tensors (Sec. 3.2 top-p%, Sec. 3.3, Sec. 3.4).
#include "tahq_launch.hpp"

namespace tahq {
namespace {

// How k_rank_quant takes U units of up to `places` places: as few places per workgroup as keep its workgroups, each of which fills a
// compute unit, to one round of the 256, so that as many of them work as can.  (In a second round everything would be ranked
// once more: 7 us, for the 3 that a launch less gives.)  With half of the lanes per tile that few tiles get, if they then hold
// at most 32 elements, twice as many tiles fit: bf16 [4,6400,256] G = 64 (102400 tiles) 20.4 -> 18.4 us, G = 32 16.1 -> 15.1.
// Lanes of 128 bytes (fp32, G = 128 and more than 65536 tiles of 64) read their rows in 64 pieces per load, which takes longer than a
// launch less saves unless the ranking is long and the rows are few: up to three units of 12288 places and more, in up to 160
// workgroups, not between kCrewPlaces and what k_select_small ranks.  Selection and quantizer apart -> here, replayed graphs, N(0,1)
// at 3.5 bits and with 5 % of the tokens U[-8,8] at 3.8: taken: G = 128, units x tiles, 1 x 12288 15.2 -> 15.1 and 13.5 -> 12.9,
// 1 x 24576 20.3 -> 19.1 and 17.8 -> 16.0, 2 x 20480 20.6 -> 20.8 and 19.0 -> 18.8 (2 x 16384 18.4 -> 19.4 and 16.8 -> 16.4), 1 x
// 40960 27.6 -> 26.6 and 25.5 -> 24.0; G = 64 3 x 24576 20.3 -> 19.8 and 19.0 -> 18.5, 2 x 40960 26.4 -> 26.0 and 25.0 -> 24.0; refused:
// G = 128 1 x 512 10.2 -> 11.9, 4 x 4096 12.9 -> 13.5, 1 x 8192 with a fifth of the tokens alike 15.2 -> 16.5, 64 x 1024 16.8 -> 20.1,
// 4 x 16384 21.5 -> 24.3, 1 x 65536 33.7 -> 36.4; G = 64 8 x 12288 17.7 -> 19.4, 4 x 24576 20.8 -> 21.7, 1 x 98304 alike 44.2 -> 47.2.
// (Of 64 bytes a lane, full rounds of small units are as fast either way: bf16 G = 64 128 x 1024 16.1 -> 15.6 and 16.3 -> 16.9.)
template <int G, bool BF16>
struct LaunchRankQuant {
    using N = Lanes<G, BF16 ? 2 : 4>;
    static constexpr int half = kCrewHalf<G, BF16>;
    static CrewPlan plan(uint64_t places, uint32_t U)
    {
        for (uint32_t b = 64; b <= (uint32_t)(kCrewThreads / half); b += 64) {
            if ((uint64_t)U * ((places + b - 1) / b) > 256) continue;
            const bool few = b <= (uint32_t)(kCrewThreads / N::few), resident = places <= kCrewPlaces;
            const uint32_t lanes = few ? N::few : half, most = kCrewThreads / lanes;
            if (G / lanes * (BF16 ? 2 : 4) > 64 && (U > 3 || places < 12288 || (!resident && places <= kSmallUnitMaxKeys) ||
                                                    U * ((places + most - 1) / most) > 160))
                break;
            return {b, few, resident};
        }
        return {0, false, false};
    }
    template <int LOW, int LPT>
    static void with(const float *H, const void *d_in, uint8_t *packed, const Shape &s, uint64_t places, const CrewPlan &p, int bin0,
                     float tau, float eps_ratio, Enqueue *qp)
    {
        Enqueue &q = *qp;
        const dim3 grid((uint32_t)((places + p.batch - 1) / p.batch), s.U);
        if (p.resident)
            q(k_rank_quant<G, BF16, LOW, LPT, true>, grid, dim3(kCrewThreads), H, d_in, packed, (uint32_t)s.T, (uint32_t)s.n, (uint32_t)s.k,
              p.batch, bin0, tau, eps_ratio);
        else
            q(k_rank_quant<G, BF16, LOW, LPT, false>, grid, dim3(kCrewThreads), H, d_in, packed, (uint32_t)s.T, (uint32_t)s.n, (uint32_t)s.k,
              p.batch, bin0, tau, eps_ratio);
    }
    template <int LOW>
    static void go(const float *H, const void *d_in, uint8_t *packed, const Shape &s, uint64_t places, const CrewPlan &p, int bin0,
                   float tau, float eps_ratio, Enqueue *qp)
    {
        if (p.few) with<LOW, N::few>(H, d_in, packed, s, places, p, bin0, tau, eps_ratio, qp);
        else with<LOW, half>(H, d_in, packed, s, places, p, bin0, tau, eps_ratio, qp);
    }
    static void run(const float *H, const void *d_in, uint8_t *packed, const Shape &s, uint64_t places, const CrewPlan &p, int bin0,
                    float tau, float eps_ratio, Enqueue *qp)
    {
        switch (s.low) {
        case 1: go<1>(H, d_in, packed, s, places, p, bin0, tau, eps_ratio, qp); break;
        case 2: go<2>(H, d_in, packed, s, places, p, bin0, tau, eps_ratio, qp); break;
        case 3: go<3>(H, d_in, packed, s, places, p, bin0, tau, eps_ratio, qp); break;
        case 4: go<4>(H, d_in, packed, s, places, p, bin0, tau, eps_ratio, qp); break;
        case 5: go<5>(H, d_in, packed, s, places, p, bin0, tau, eps_ratio, qp); break;
        case 6: go<6>(H, d_in, packed, s, places, p, bin0, tau, eps_ratio, qp); break;
        default: go<7>(H, d_in, packed, s, places, p, bin0, tau, eps_ratio, qp); break;
        }
    }
};

template <int G, bool BF16>
struct RankQuantPlan {
    static void run(uint64_t places, uint32_t U, CrewPlan *p) { *p = LaunchRankQuant<G, BF16>::plan(places, U); }
};

}  // namespace

CrewPlan plan_rank_quant(const Shape &s, uint64_t places)
{
    CrewPlan plan = {0, false, false};
    if (places <= (s.U == 1 ? kCrewMost : kCrewMostOfSeveral)) dispatch<RankQuantPlan>(s.G, s.dtype == TAHQ_BF16, places, s.U, &plan);
    return plan;
}

void launch_rank_quant(const float *H, const void *d_in, uint8_t *packed, const Shape &s, uint64_t places, const CrewPlan &plan,
                       float tau, float eps_ratio, Enqueue *q)
{
    dispatch<LaunchRankQuant>(s.G, s.dtype == TAHQ_BF16, H, d_in, packed, s, places, plan, lowest_bin<kCrewBins, kCrewShift>(s), tau,
                              eps_ratio, q);
}

}  // namespace tahq

// What the translation units of the library share on the host: launches, dispatch, the plan of the small tensors' launch.
#pragma once
#include "tahq_rank_quant.hpp"

#include <tuple>
#include <utility>

namespace tahq {

// Dispatch on the tile width G and on a dtype flag (bf16 or not) to a functor template.
template <template <int, bool> class F, typename... Args>
inline void dispatch(uint32_t G, bool bf16, Args... args)
{
    if (G == 8) { if (bf16) F<8, true>::run(args...); else F<8, false>::run(args...); }
    else if (G == 16) { if (bf16) F<16, true>::run(args...); else F<16, false>::run(args...); }
    else if (G == 32) { if (bf16) F<32, true>::run(args...); else F<32, false>::run(args...); }
    else if (G == 64) { if (bf16) F<64, true>::run(args...); else F<64, false>::run(args...); }
    else { if (bf16) F<128, true>::run(args...); else F<128, false>::run(args...); }
}

// Kernel launches of one call: each launch returns its own status (the thread's sticky "last error", which may
// belong to the caller's earlier work, is neither read nor cleared), and after a failure nothing more is enqueued.
struct Enqueue {
    hipStream_t stream;
    hipError_t status = hipSuccess;

    template <typename... P, typename... A>
    void operator()(void (*kernel)(P...), dim3 grid, dim3 block, A... args)
    {
        static_assert(sizeof...(P) == sizeof...(A), "one argument per kernel parameter");
        if (status != hipSuccess) return;
        std::tuple<P...> values(static_cast<P>(args)...);
        status = launch(kernel, grid, block, values, std::index_sequence_for<P...>{});
    }
    tahq_status result() const { return status == hipSuccess ? TAHQ_OK : TAHQ_ERR_HIP; }

private:
    template <typename... P, size_t... I>
    hipError_t launch(void (*kernel)(P...), dim3 grid, dim3 block, std::tuple<P...> &values, std::index_sequence<I...>)
    {
        void *ptrs[] = {static_cast<void *>(&std::get<I>(values))...};
        return hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, ptrs, 0, stream);
    }
};

// Fewer wavefronts than the chip has vector units (256 compute units of four), at the usual number of lanes per tile: the launch
// takes as long as one lane does, and tiles are spread over more lanes, as long as those make no more wavefronts per vector
// unit than `deep`: 4, all that run at once, or 2 in the quantizer.  Above that the usual lanes have less to issue.  bf16, G = 64,
// usual -> few: 25600 tiles: entropies 4.2 -> 3.1 us, decoder 4.5 -> 3.6; 51200: 4.3 -> 3.9, 4.7 -> 4.2; 64512: 4.4 -> 4.0, 4.8 -> 4.4.
// Encode at one width, the quantizer alone: 25600 tiles 6.2 -> 4.5, G = 128 5.8 -> 5.5.  (Its 2 is from when several lanes per tile
// worked by workgroups, where 51200 tiles took 5.7 and 5.8.  By wavefronts they take less above it, too: 51200 tiles 6.3 -> 5.5, G = 32
// 5.1 -> 4.6, G = 128 alike.)
template <class N>
inline bool few_tiles(uint64_t T, uint32_t deep) { return T * N::usual < 65536u && T * N::few < deep * 65536u; }

// k_select_small's and k_select_mid's lowest bin: the topmost bin but one holds ln A, the largest an entropy can be
template <uint32_t BINS, int SHIFT>
inline int lowest_bin(const Shape &s)
{
    const float ln_a = (float)__builtin_log((double)s.A);
    int bits;
    memcpy(&bits, &ln_a, 4);
    return (bits >> SHIFT) - (int)(BINS - 2);
}

// How k_rank_quant takes a tensor, see plan_rank_quant.
struct CrewPlan {
    uint32_t batch;                              // places per workgroup; 0: not this way
    bool few;                                    // lanes per tile: as many as tensors of few tiles get, or half of them
    bool resident;                               // whether the unit's entropies stay in LDS
};
template <int G, bool BF16>
constexpr int kCrewHalf = Lanes<G, BF16 ? 2 : 4>::few / 2 > 0 && G / (Lanes<G, BF16 ? 2 : 4>::few / 2) <= 32
                              ? Lanes<G, BF16 ? 2 : 4>::few / 2 : Lanes<G, BF16 ? 2 : 4>::few;

// How k_rank_quant takes U units of up to `places` places, if it does, and its launch; in a translation unit of their own, which compiles
// beside the others.
CrewPlan plan_rank_quant(const Shape &s, uint64_t places);
void launch_rank_quant(const float *H, const void *d_in, uint8_t *packed, const Shape &s, uint64_t places, const CrewPlan &plan,
                       float tau, float eps_ratio, Enqueue *q);

}  // namespace tahq

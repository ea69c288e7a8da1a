// ra_split.hpp — split forward for few work items: one workgroup per item,
// whose first wavefront steps the chain while the others draw its noise
// (ra_fwd_split.hip, and two contexts in one launch, ra_fwd_split_dual.hip).
//
// A batch with fewer work items than the chip has SIMDs leaves most of them idle and
// is bound by the length of one wavefront's step, of which the noise (Philox,
// Box-Muller) is two thirds in FP32 and nearly all in FP64, and independent of
// the chain. The noise comes through LDS (NoiseRing) as the same radii and sines,
// so the trajectories are the same to the bit as the one-wavefront kernels'.
// Bound by the consumer's step up to one item per CU (about 250 cycles in FP32, of
// them the twelve dependent instructions from |Q|^2 to the new bond 85), by the
// issue of all wavefronts above. 1000 steps of 50 beads, FP32 noise map 1: 50
// replicas 233 -> 137 us, 512 240 -> 165, 1024 245 -> 210; FP64 map 0: 50 replicas
// 821 -> 259 us, 512 836 -> 472.
#pragma once
#include "ra_forward.hpp"

namespace ra {

// Producing wavefronts: noise is 1.5-2 times the update in FP32, five in FP64. FP64 with
// 6 / 9 / 12, us: 64 replicas of 10 beads, 5000 steps 1125 1061 994; 256 of 50 beads,
// 400 steps 135 131 139, 768 321 327 352; 256 of 100 beads 229 216 235. With more than
// two beads per lane nine leave 168 registers, and noise map 1 spills 470-2265 of
// them (six 110-700; three none, but 10% slower). Against the one-wavefront kernel, N = 129-256,
// time at 256 / 512 / 768 items with six: map 0 0.34 0.61 0.91, map 1 0.29 0.56 0.83, with
// TSF 0.93 (nine 1.04); in a cycle 0.34 0.55 0.77, map 1 0.34 0.54 0.74 (nine 0.37 0.58 0.79).
template <typename T, int MAX_M> struct SplitWaves {
    static constexpr int PRODUCERS = sizeof(T) == 4 ? 3 : MAX_M == 4 ? 6 : 9;
};

// Producer p of PRODUCERS: blocks p, p + PRODUCERS, .. of every chunk, one
// barrier after each chunk. Blocks past the last step are drawn and not used.
template <typename T, int M, bool UNIFORM_K, int NMAP, int PRODUCERS>
__device__ __forceinline__ void produce(const FwdArgs& a, const GroupDev& G, int k_first, int64_t n0_64, int p,
                                        const NoiseRing<T, M, NMAP>& ring) {
    using Ring = NoiseRing<T, M, NMAP>;
    const TileGeom tg = tile_geom<UNIFORM_K>(G, k_first, M);
    const RoundKeys keys = round_keys(a.key0, a.key1);
    const LaneCounters<M, UNIFORM_K> lc =
        lane_counters<M, UNIFORM_K>((uint32_t)tg.j0, (uint32_t)tg.k, G.stream, a.key0, a.key1);
    const uint32_t n0 = (uint32_t)n0_64;
    const uint32_t head = NMAP == 1 ? steps_to_group(n0) : 0u;   // steps that draw their own noise
    const int left = (int)a.n_steps - (int)head;
    uint32_t n = n0 + head;
    int buf = 0;
    for (int done = 0; done < left; done += Ring::STEPS) {
        for (int b = p; b < Ring::BLOCKS; b += PRODUCERS) {
            const StepWords sw = lc.words(n + (uint32_t)(NMAP == 1 ? b + b / 3 : b));
#pragma unroll
            for (int m = 0; m < M; ++m) {
                Polar<T> x, y, z, d;
                polars4_paced(lc.draw(m, sw, keys), noise_amp<T>(G), x, y, z, d);
                ring.put(buf, b, m, x, y, z, d);
            }
        }
        __syncthreads();
        n += (uint32_t)Ring::STEPS;
        buf ^= 1;
    }
}

// TSFK as in dispatch_spring.
template <typename T, int M, int NMAP, int TSFK, int PRODUCERS>
__device__ __forceinline__ void split_tile(const FwdArgs& a, const GroupDev& Gm, int k_first, int64_t n0, int wave,
                                           T* lds) {
    const int gidx = (int)(&Gm - a.groups);
    const GroupDev G = Gm;
    const NoiseRing<T, M, NMAP> ring{lds};
    auto run = [&](auto Uk) {
        constexpr bool UK = decltype(Uk)::value;
        auto consume = [&](auto Tsf) {
            constexpr bool TSF = decltype(Tsf)::value;
            if (G.spring == 1) run_forward_impl<T, M, true, UK, TSF, NMAP, TSFK == 3>(a, G, gidx, k_first, n0, ring);
            else run_forward_impl<T, M, false, UK, TSF, NMAP, TSFK == 3>(a, G, gidx, k_first, n0, ring);
        };
        if (wave > 0) {
            produce<T, M, UK, NMAP, PRODUCERS>(a, G, k_first, n0, wave - 1, ring);
        } else if constexpr (TSFK == 2) {
            if (a.tsf) consume(Bool<true>{});
            else consume(Bool<false>{});
        } else {
            consume(Bool<TSFK == 1>{});
        }
    };
    if (sizeof(T) == 4 && G.P == 1) run(Bool<sizeof(T) == 4>{});   // FP64: fewer variants
    else run(Bool<false>{});
}

// MAX_M: the most beads per lane of the batch's groups (1, 2 or 4): a kernel that
// holds the wider tiles too takes their registers, and fewer workgroups fit a
// CU (1024 items of 50 beads: 260 against 210 us).
template <typename T, int NMAP, int TSFK, int MAX_M>
__device__ __forceinline__ void split_item(const FwdArgs& a, int item, T* lds) {
    if (*(const volatile int*)a.status & 1) return;   // invalid parent: no work (whole block)
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Item it = a.items[item];
    const GroupDev& G = a.groups[it.g];
    const int64_t n0 = *a.step0;
    if (MAX_M == 1 || G.M == 1) {
        split_tile<T, 1, NMAP, TSFK, SplitWaves<T, MAX_M>::PRODUCERS>(a, G, it.k0, n0, wave, lds);
    } else if (MAX_M == 2 || G.M == 2) {
        if constexpr (MAX_M >= 2) split_tile<T, 2, NMAP, TSFK, SplitWaves<T, MAX_M>::PRODUCERS>(a, G, it.k0, n0, wave, lds);
    } else if constexpr (MAX_M == 4) {
        if (G.M == 3) split_tile<T, 3, NMAP, TSFK, SplitWaves<T, MAX_M>::PRODUCERS>(a, G, it.k0, n0, wave, lds);
        else split_tile<T, 4, NMAP, TSFK, SplitWaves<T, MAX_M>::PRODUCERS>(a, G, it.k0, n0, wave, lds);
    }
}

template <typename T, int MAX_M> constexpr int split_threads() { return WAVE * (1 + SplitWaves<T, MAX_M>::PRODUCERS); }

template <typename T, int NMAP, int MAX_M> constexpr int split_lds_bytes() {
    int lds = NoiseRing<T, 1, NMAP>::BYTES;
    if (MAX_M >= 2) lds = std::max(lds, NoiseRing<T, 2, NMAP>::BYTES);
    if (MAX_M == 4) lds = std::max({lds, NoiseRing<T, 3, NMAP>::BYTES, NoiseRing<T, 4, NMAP>::BYTES});
    return lds;
}

}  // namespace ra

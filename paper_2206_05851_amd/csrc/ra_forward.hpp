// ra_forward.hpp — the fused forward kernels of the chain model, compiled by
// ra_fwd_lane.hip (FP32, 1-4 beads per lane), ra_fwd_wide.hip (FP32, 6-16) and
// ra_fwd_f64.hip (each with its one- and two-context launches).
//
// Fused forward path (one launch per ra_step):
//   one wavefront per work item = P replicas of one group; a replica occupies
//   L = ceil(N/M) consecutive lanes, lane t holding beads/springs
//   [t*M, t*M + M). The chain lives in VGPRs as bond vectors Q_j = r_{j+1} - r_j
//   for the whole time loop; neighbour springs and neighbour-bead noise come
//   from the adjacent lane by DPP wave shifts. Every slot past the last spring
//   of a replica holds Q = 0 (so its force is 0), which makes the chain ends
//   and the seams between packed replicas need no extra masking.
// The step itself (bond form of Eq. (1) with Eq. (2)) is in ra_chain.hpp.
#pragma once
#include "ra_chain.hpp"
#include "ra_launch.hpp"

namespace ra {

// ---------------------------------------------------------------------------
// Fused persistent forward: all n_steps of one work item in registers.
// ---------------------------------------------------------------------------
// Noise from other wavefronts of the workgroup (split forward, fwd_split_kernel):
// a ring of two chunks of BLOCKS Philox blocks in LDS, transformed (radius and
// sines as polars4 gives them) by the producing wavefronts. Each chunk starts
// with one barrier of the workgroup.
template <typename T, int M, int NMAP> struct NoiseRing {
    static constexpr bool on = true;
    static constexpr int BLOCKS = M * (int)sizeof(T) <= 16 ? 12 : 6;
    static constexpr int STEPS = NMAP == 1 ? BLOCKS / 3 * 4 : BLOCKS;   // steps of a chunk
    static constexpr int BYTES = 2 * BLOCKS * M * 6 * WAVE * (int)sizeof(T);
    typedef T V2 __attribute__((ext_vector_type(2)));
    typedef T V4 __attribute__((ext_vector_type(4)));
    T* base;                                       // [2][BLOCKS][M][6 WAVE]

    // one lane's six values: 16-byte accesses in FP32 (four and two), FP64 (two each)
    __device__ __forceinline__ T* row(int buf, int block, int m) const {
        return base + ((buf * BLOCKS + block) * M + m) * (6 * WAVE);
    }
    __device__ __forceinline__ void put(int buf, int block, int m, const Polar<T>& a, const Polar<T>& b,
                                        const Polar<T>& c, const Polar<T>& d) const {
        const int lane = threadIdx.x & (WAVE - 1);
        T* r = row(buf, block, m);
        if constexpr (sizeof(T) == 4) {
            ((V4*)r)[lane] = V4{a.r, a.t, b.t, c.r};
            ((V2*)(r + 4 * WAVE))[lane] = V2{c.t, d.t};
        } else {
            ((V2*)r)[lane] = V2{a.r, a.t};
            ((V2*)(r + 2 * WAVE))[lane] = V2{b.t, c.r};
            ((V2*)(r + 4 * WAVE))[lane] = V2{c.t, d.t};
        }
    }
    __device__ __forceinline__ void get(int buf, int block, int m, Polar<T>& a, Polar<T>& b, Polar<T>& c,
                                        Polar<T>& d) const {
        const int lane = threadIdx.x & (WAVE - 1);
        const T* r = row(buf, block, m);
        V2 p, q;
        if constexpr (sizeof(T) == 4) {
            const V4 v = ((const V4*)r)[lane];
            p = V2{v.x, v.y};
            q = V2{v.z, v.w};
        } else {
            p = ((const V2*)r)[lane];
            q = ((const V2*)(r + 2 * WAVE))[lane];
        }
        const V2 h = ((const V2*)(r + 4 * WAVE))[lane];
        a = Polar<T>{p.x, p.y};
        b = Polar<T>{p.x, q.x};
        c = Polar<T>{q.y, h.x};
        d = Polar<T>{q.y, h.y};
    }
};
struct OwnNoise {
    static constexpr bool on = false;
    static constexpr int STEPS = 1;
    template <typename... A> __device__ void get(A&&...) const {}
};

// Noise run-ahead per beads-per-lane: with one bead per lane the wave has
// little independent work per step, so U steps of noise (U independent Philox
// chains per lane) are generated before the U physics steps consume them.
template <int M> struct RunAhead { static constexpr int U = M == 1 ? 4 : (M == 2 ? 2 : 1); };

// Fused persistent forward over all n_steps of one work item. The step loop is
// cut into segments between events (window end, checkpoint), so the inner
// loop holds nothing but noise generation and the bond update (plus the
// per-step tension sum when TSF is on).
template <typename T, int M, bool FENE, bool UNIFORM_K, bool TSF, int NMAP, bool EVERY, typename Ring = OwnNoise>
__device__ __forceinline__ void run_forward_impl(const FwdArgs& a, const GroupDev& G, int gidx, int k_first,
                                                 int64_t n0_64, const Ring& ring = Ring{}) {
    constexpr int U = RunAhead<M>::U;
    // Kernel arguments are read once into locals: the step lambdas below must
    // not take the address of the by-value argument block (that would copy it
    // to scratch memory).
    const int S = a.S, K = a.K;
    const int64_t smp_total = a.smp_total, state_total = a.state_total;
    T* const state = (T*)a.state;
    int32_t* const status = a.status;
    unsigned long long* const clamp_ctr = a.clamps + gidx;
    const int n_steps = (int)a.n_steps;
    const TileGeom tg = tile_geom<UNIFORM_K>(G, k_first, M);
    const RoundKeys keys = round_keys(a.key0, a.key1);
    Lane<T, M> s;
    bool valid[M];
    load_lane<T, M>(s, valid, state, G, tg);
    const SlotMask<T, M> mask = slot_mask<T, M>(valid);
    const int nm1 = G.N - 1;
    const uint32_t n0 = (uint32_t)n0_64;       // total steps stay below 2^32
    using Blocks = LaneBlocks<M, NMAP>;
    const LaneCounters<Blocks::value, UNIFORM_K> lc = lane_counters<Blocks::value, UNIFORM_K>(
        Blocks::first((uint32_t)tg.j0), (uint32_t)tg.k, G.stream, a.key0, a.key1);
    // per-lane output cursors, bumped once per window / checkpoint
    const int64_t lane_off = G.smp_off + (int64_t)tg.k * nm1 + tg.j0;
    T* smp_w = (T*)a.samples + (int64_t)(n0 / (uint32_t)S) * smp_total + lane_off;
    T* tsf_w = TSF ? (T*)a.tsf + (int64_t)(n0 / (uint32_t)S) * smp_total + lane_off : nullptr;
    const int64_t ckpt_total = a.ckpt_total;
    T* ck_w = K > 0 ? ckpt_item<T, M>((T*)a.ckpt, G, k_first) + (int64_t)((n0 + (uint32_t)K - 1) / (uint32_t)K) * ckpt_total
                    : nullptr;
    double* const tacc_g = TSF ? a.tsf_acc + lane_off : nullptr;
    int to_smp = S - (int)(n0 % (uint32_t)S);                              // steps to the next window end
    int to_ck = K > 0 ? (int)((K - (int)(n0 % (uint32_t)K)) % K) : INT32_MAX;  // steps to the next checkpoint
    // TSF: each step's force evaluation adds the tension of the state it
    // starts from (slot_force), so a window's states n+1 .. n+S are the
    // evaluations of steps n+1 .. n+S-1 plus the window-end state, which the
    // sample computes anyway; the evaluation of step n (the previous window's
    // last state) is cancelled by starting the sum at minus that tension.
    // The sums stay in registers over at most TSF_FLUSH steps and are folded
    // into the FP64 window sum in global memory only when a window is longer
    // or continues in a later launch. Tensions are nonnegative, so a register
    // sum of at most 512 terms (and the one cancelled term) carries a relative
    // error of a few hundred ulp at most (below 3.1e-5).
    constexpr int TSF_FLUSH = 512;
    // 6-16 beads per lane under noise map 0 keep the separate tension pass after
    // each step: their register budget (two wavefronts per SIMD) has no room for
    // the fused sums beside sixteen Philox chains. Under map 2 (twelve chains)
    // the fused sums fit; the spills they cause sit outside the step loop, and
    // the 16-bead kernel is 4% faster than with the separate pass.
    constexpr bool FUSED = TSF && (M <= 4 || NMAP == 2);
    T tpart[M];
    T* const tsum = FUSED ? tpart : nullptr;
#pragma unroll
    for (int m = 0; m < M; ++m) tpart[m] = (T)0;
    if constexpr (FUSED) {
        if (n0_64 % S == 0) {                // the launch starts a window
            T u[M];
            tsf_terms<T, M, FENE>(s, G, u);
#pragma unroll
            for (int m = 0; m < M; ++m) tpart[m] = -u[m];
        }
    }
    // the window sum in global memory holds part of the current window: true
    // when the launch starts inside a window, and after every mid-window fold
    bool acc_live = (n0_64 % S) != 0;
    const double to_f = FUSED ? (sizeof(T) == 4 ? G.uH : G.uH_d) : 1.0;   // a fused term is cF g |Q|
    // at a window's end the terms of its last state close the sum and start
    // the next window's
    auto flush_tsf = [&](bool window_end) {
        if constexpr (TSF) {
            T u[M] = {};
            if (FUSED && window_end) tsf_terms<T, M, FENE>(s, G, u);
#pragma unroll
            for (int m = 0; m < M; ++m) {
                if (valid[m]) {
                    const double acc = (acc_live ? tacc_g[m] : 0.0) + to_f * ((double)tpart[m] + (double)u[m]);
                    if (window_end) tsf_w[m] = (T)(acc / (double)S);
                    else tacc_g[m] = acc;
                }
                tpart[m] = (FUSED && window_end) ? -u[m] : (T)0;
            }
            acc_live = !window_end;
        }
    };
    auto keep = [&]() {                        // every state, before its step
        if constexpr (EVERY) {
            Rows<M>(G).store(s, ck_w);
            ck_w += ckpt_total;
        }
    };
    int clamps = 0;
    // the separate pass: the tensions of the state after each step
    auto accumulate_tsf = [&]() {
        if constexpr (TSF && !FUSED) {
            T f[M];
            tensions<T, M, FENE>(s, G, f);
#pragma unroll
            for (int m = 0; m < M; ++m) tpart[m] += f[m];
        }
    };
    // noise map 1: with one or two beads per lane the steps run in aligned
    // groups of four. The next group's three Philox blocks per slot are drawn
    // at the top of each group (integer work independent of the steps), and
    // each step transforms the blocks it uses just before it, which spreads
    // the transcendentals over the group (against transforming the next
    // group's blocks along with their draw, 3.5% faster on fene50; against
    // the carry, 5% faster on two beads per lane). A run's unaligned head and
    // its tail, and wider lanes, take the carry step by step. The carry lives
    // for the whole launch (built once for its first step): segments follow
    // each other in step order, an aligned group neither needs nor changes
    // it, and a partial group is always stepped through the carry, so it
    // holds the current group's fourth normals.
    [[maybe_unused]] Carry<T, M> cy;
    if constexpr (NMAP == 1) init_carry<T, M, UNIFORM_K>(cy, lc, G, n0, keys);
    auto run_steps_map1 = [&](auto n, int len) {   // generic: instantiated where it is called
        int i = 0;
        if constexpr (M <= 2) {
            for (; i < len && ((n + (uint32_t)i) & 3u) != 0u; ++i) {
                keep();
                em_step_map1<T, M, FENE, FUSED, UNIFORM_K>(s, cy, lc, G, valid, mask, n + (uint32_t)i, keys, clamps, tsum);
                accumulate_tsf();
            }
            if (i + 4 <= len) {
                Words w[3][M];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const StepWords sw = lc.words(n + (uint32_t)(i + q));
#pragma unroll
                    for (int m = 0; m < M; ++m) w[q][m] = lc.draw(m, sw, keys);
                }
                for (; i + 4 <= len; i += 4) {
                    asm volatile(".p2align 6");
                    Words nw[3][M];
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const StepWords sw = lc.words(n + (uint32_t)(i + 4 + q));
#pragma unroll
                        for (int m = 0; m < M; ++m) nw[q][m] = lc.draw(m, sw, keys);
                    }
                    Noise<T, M> e3;
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        Noise<T, M> e;
#pragma unroll
                        for (int m = 0; m < M; ++m) {
                            Polar<T> d;
                            polars4(w[u][m], noise_amp<T>(G), e.x[m], e.y[m], e.z[m], d);
                            if (u == 0) e3.x[m] = d;
                            if (u == 1) e3.y[m] = d;
                            if (u == 2) e3.z[m] = d;
                        }
                        keep();
                        physics_step<T, M, FENE, FUSED>(s, e, G, valid, mask, clamps, tsum);
                        accumulate_tsf();
                    }
                    keep();
                    physics_step<T, M, FENE, FUSED>(s, e3, G, valid, mask, clamps, tsum);
                    accumulate_tsf();
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int m = 0; m < M; ++m) w[q][m] = nw[q][m];
                }
            }
        }
        // the rest: with one or two beads per lane a tail of at most three
        // steps that starts aligned (the carry is refilled before it is read);
        // wider lanes step through the carry from the start
        for (; i < len; ++i) {
            keep();
            em_step_map1<T, M, FENE, FUSED, UNIFORM_K>(s, cy, lc, G, valid, mask, n + (uint32_t)i, keys, clamps, tsum);
            accumulate_tsf();
        }
    };
    auto run_steps_map0 = [&](auto n, int len) {
        int i = 0;
        if constexpr (U > 1) {
            // software pipeline: the noise of block b+1 is generated in the same
            // basic block as the updates of block b, so the scheduler can fill the
            // update chain's latencies with independent Philox work (one spare
            // block of noise is generated past the end and discarded)
            if constexpr (M == 1) {
                // one bead per lane: the next U steps' blocks are drawn ahead and
                // each step transforms its own block just before it (6% faster
                // on fene50 than transforming along with the draw; with two beads
                // per lane the draw-and-transform pipeline below is 2% faster)
                if (U <= len) {
                    Words w[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) w[u] = lc.draw(0, lc.words(n + (uint32_t)u), keys);
                    for (; i + U <= len; i += U) {
                        asm volatile(".p2align 6");
                        Words nw[U];
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            nw[u] = lc.draw(0, lc.words(n + (uint32_t)(i + U + u)), keys);
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            Noise<T, M> e;
                            Polar<T> d;
                            polars4(w[u], noise_amp<T>(G), e.x[0], e.y[0], e.z[0], d);
                            keep();
                            physics_step<T, M, FENE, FUSED>(s, e, G, valid, mask, clamps, tsum);
                            accumulate_tsf();
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u) w[u] = nw[u];
                    }
                }
            } else if (U <= len) {
                Noise<T, M> e[U];
#pragma unroll
                for (int u = 0; u < U; ++u) gen_noise<T, M, UNIFORM_K>(e[u], lc, G, n + (uint32_t)u, keys);
                for (; i + U <= len; i += U) {
                    // start the loop body on a 64-byte boundary: its speed depends on
                    // where its 4- and 8-byte instructions fall in the fetch lines
                    // (measured: unaligned placements cost up to 10%)
                    asm volatile(".p2align 6");
                    Noise<T, M> f[U];
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        gen_noise<T, M, UNIFORM_K>(f[u], lc, G, n + (uint32_t)(i + U + u), keys);
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        keep();
                        physics_step<T, M, FENE, FUSED>(s, e[u], G, valid, mask, clamps, tsum);
                        accumulate_tsf();
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) e[u] = f[u];
                }
            }
        }
        for (; i < len; ++i) {
            keep();
            em_step<T, M, FENE, FUSED, UNIFORM_K>(s, lc, G, valid, mask, n + (uint32_t)i, keys, clamps, tsum);
            accumulate_tsf();
        }
    };
    // split forward: steps from the ring, the next step's entries read during a
    // step. Under noise map 1 the ring starts at a multiple of 4 and the steps
    // before it, three at most, draw their own noise.
    int at = 0, buf = 0;   // steps taken of the current chunk, its half of the ring
    [[maybe_unused]] int head = NMAP == 1 ? (int)steps_to_group(n0) : 0;
    auto run_steps_ring = [&](auto n, int len) {
        int i = 0;
        if constexpr (NMAP == 1) {
            for (; i < len && head > 0; ++i, --head) {
                keep();
                em_step_map1<T, M, FENE, FUSED, UNIFORM_K>(s, cy, lc, G, valid, mask, n + (uint32_t)i, keys, clamps, tsum);
                accumulate_tsf();
            }
        }
        // noise of step `st` of the chunk; its fourth normals into the carry (map 1)
        auto fetch = [&](Noise<T, M>& e, int st) {
            if constexpr (NMAP == 1) {
                const int r = st & 3;
                if (r == 3) {
#pragma unroll
                    for (int m = 0; m < M; ++m) { e.x[m] = cy.c0[m]; e.y[m] = cy.c1[m]; e.z[m] = cy.c2[m]; }
                    return;
                }
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    Polar<T> d;
                    ring.get(buf, (st >> 2) * 3 + r, m, e.x[m], e.y[m], e.z[m], d);
                    carry_slot((uint32_t)r, d, cy.c0[m], cy.c1[m], cy.c2[m]);
                }
            } else {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    Polar<T> d;
                    ring.get(buf, st, m, e.x[m], e.y[m], e.z[m], d);
                }
            }
        };
        while (i < len) {
            if (at == 0) __syncthreads();          // the chunk is written
            const int cnt = min(len - i, Ring::STEPS - at);
            int j = 0;
            if constexpr (NMAP == 1) {
                // whole groups of four: three blocks, all reads at the top
                if ((at & 3) == 0)
                    for (; j + 4 <= cnt; j += 4) {
                        Noise<T, M> e[3], e3;
#pragma unroll
                        for (int u = 0; u < 3; ++u)
#pragma unroll
                            for (int m = 0; m < M; ++m) {
                                Polar<T>& d = u == 0 ? e3.x[m] : u == 1 ? e3.y[m] : e3.z[m];
                                ring.get(buf, ((at + j) >> 2) * 3 + u, m, e[u].x[m], e[u].y[m], e[u].z[m], d);
                            }
#pragma unroll
                        for (int u = 0; u < 3; ++u) {
                            keep();
                            physics_step<T, M, FENE, FUSED>(s, e[u], G, valid, mask, clamps, tsum);
                            accumulate_tsf();
                        }
                        keep();
                        physics_step<T, M, FENE, FUSED>(s, e3, G, valid, mask, clamps, tsum);
                        accumulate_tsf();
                    }
                for (; j < cnt; ++j) {
                    Noise<T, M> e;
                    fetch(e, at + j);
                    keep();
                    physics_step<T, M, FENE, FUSED>(s, e, G, valid, mask, clamps, tsum);
                    accumulate_tsf();
                }
            } else {
                Noise<T, M> e, f;
                fetch(e, at);
                for (; j + 2 <= cnt; j += 2) {
                    fetch(f, at + j + 1);
                    keep();
                    physics_step<T, M, FENE, FUSED>(s, e, G, valid, mask, clamps, tsum);
                    accumulate_tsf();
                    fetch(e, j + 2 < cnt ? at + j + 2 : at);
                    keep();
                    physics_step<T, M, FENE, FUSED>(s, f, G, valid, mask, clamps, tsum);
                    accumulate_tsf();
                }
                if (j < cnt) {
                    keep();
                    physics_step<T, M, FENE, FUSED>(s, e, G, valid, mask, clamps, tsum);
                    accumulate_tsf();
                }
            }
            i += cnt;
            at += cnt;
            if (at == Ring::STEPS) {
                at = 0;
                buf ^= 1;
            }
        }
    };
    auto run_steps = [&](uint32_t n, int len) {   // len steps starting at global step n
        if constexpr (Ring::on) {
            run_steps_ring(n, len);
        } else if constexpr (NMAP == 1) {
            run_steps_map1(n, len);
        } else if constexpr (NMAP == 2) {
            for (int i = 0; i < len; ++i) {
                em_step_map2<T, M, FENE, FUSED, UNIFORM_K>(s, lc, G, valid, mask, n + (uint32_t)i, keys, clamps, tsum);
                accumulate_tsf();
            }
        } else {
            run_steps_map0(n, len);
        }
    };

    int left = n_steps;
    int to_flush = TSF_FLUSH;
    uint32_t n = n0;
    while (left > 0) {
        if (!EVERY && to_ck == 0) {            // checkpoint before step n
            // by the registers it leaves (1000 beads 77.2 against 75.1 ms with Rows, a mixed
            // batch of 1-4 beads per lane 5.77 against 5.88)
            if constexpr (sizeof(T) == 4 && M <= 4 && !Ring::on) Rows<M>(G).store(s, ck_w);
            else store_ckpt<T, M>(s, ck_w, G);
            ck_w += ckpt_total;
            to_ck = K;
        }
        int len = min(left, EVERY ? to_smp : min(to_smp, to_ck));
        if constexpr (TSF) len = min(len, to_flush);
        run_steps(n, len);
        n += (uint32_t)len;
        left -= len;
        to_ck -= EVERY ? 0 : len;
        to_smp -= len;
        to_flush -= len;
        if (to_smp == 0) {                     // window end after step n - 1
            T f[M];
            tensions<T, M, FENE>(s, G, f);
            bool bad = false;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                if (valid[m]) {
                    smp_w[m] = f[m];
                    bad |= !__builtin_isfinite(f[m]);
                }
            }
            flush_tsf(true);
            to_flush = TSF_FLUSH;
            smp_w += smp_total;
            if constexpr (TSF) tsf_w += smp_total;
            if (bad) atomicOr(status, 2);
            to_smp = S;
        } else if (TSF && (to_flush == 0 || left == 0)) {
            flush_tsf(false);
            to_flush = TSF_FLUSH;
        }
    }
    store_lane<T, M>(s, valid, state, G, tg);
    flush_clamps(clamps, clamp_ctr);
}

// With 1-4 beads per lane the group's constants are copied into a local value
// once: read through the reference, the step loop re-loads them from memory
// every iteration (measured: one extra vector load per step). Wider lanes keep
// the reference, as the copy would not fit their register budget.
// Noise map 1 is compiled for 1-4 beads per lane only (the host rejects it
// for wider lanes, whose register budget has no room for the carry), noise
// map 2 for 8, 12 and 16 beads per lane only, each in kernels of its own, so
// each map gets its own register allocation.
template <typename T, int M, bool FENE, bool UNIFORM_K, bool TSF, int NMAP, bool EVERY>
__device__ __forceinline__ void run_forward(const FwdArgs& a, const GroupDev& Gm, int k_first, int64_t n0_64) {
    const int gidx = (int)(&Gm - a.groups);
    if constexpr (M <= 4) {
        const GroupDev G = Gm;
        run_forward_impl<T, M, FENE, UNIFORM_K, TSF, NMAP, EVERY>(a, G, gidx, k_first, n0_64);
    } else {
        static_assert(NMAP != 1, "noise map 1 is compiled for 1-4 beads per lane");
        run_forward_impl<T, M, FENE, UNIFORM_K, TSF, NMAP, EVERY>(a, Gm, gidx, k_first, n0_64);
    }
}

// TSFK: 0 compiles the variants without TSF, 1 those with TSF (kernels of
// their own, so the time-average sums do not raise the register budget of
// runs without them), 2 both, chosen per context at run time (the RSF
// cycle's dual launch: the parent keeps TSF, the replicas do not). 3: no TSF, and a
// state kept before every step (K = 1), stored inside the step loops: as segments
// of one step between checkpoints the loops lose their run-ahead (1000 items of
// 40-77 beads, 500 steps: 488 us, and 381 with it). In kernels of its own, as it
// raises the registers of the others (a mixed batch: 5.87 ms, with it 6.28).
template <typename T, int M, int NMAP, int TSFK>
__device__ __forceinline__ void dispatch_spring(const FwdArgs& a, const GroupDev& G, int k_first, int64_t n0) {
    const bool tsf = a.tsf != nullptr;
#define RA_FWD(FENE_, UK_, TSF_) run_forward<T, M, FENE_, UK_, TSF_, NMAP, TSFK == 3>(a, G, k_first, n0)
#define RA_TSF(FENE_, UK_)                                        \
    do {                                                          \
        if constexpr (TSFK == 0 || TSFK == 3) RA_FWD(FENE_, UK_, false);       \
        else if constexpr (TSFK == 1) RA_FWD(FENE_, UK_, true);   \
        else if (tsf) RA_FWD(FENE_, UK_, true);                   \
        else RA_FWD(FENE_, UK_, false);                           \
    } while (0)
    if constexpr (sizeof(T) == 8) {           // FP64 correctness path: fewer variants
        if (G.spring == 1) RA_TSF(true, false);
        else RA_TSF(false, false);
    } else {
        const bool uk = G.P == 1;
        if (G.spring == 1) {
            if (uk) RA_TSF(true, true);
            else RA_TSF(true, false);
        } else {
            if (uk) RA_TSF(false, true);
            else RA_TSF(false, false);
        }
    }
#undef RA_TSF
#undef RA_FWD
    (void)tsf;
}

// WAVES_PER_EU is a register budget hint: family 4 needs none (about 100
// VGPRs); family 16 is held to 2 resident waves per SIMD (256 registers), which
// it fits without spilling — left alone the scheduler hoists all 16 Philox
// chains and falls to 1 wave, and asking for 3-4 waves makes it spill.
template <typename T, int FAMILY, int NMAP, int TSFK>
__device__ __forceinline__ void fwd_item(const FwdArgs& a, int item) {
    if (item >= a.n_items) return;
    if (*(const volatile int*)a.status & 1) return;   // invalid parent: no work
    const Item it = a.items[item];
    const GroupDev& G = a.groups[it.g];
    const int64_t n0 = *a.step0;
    if constexpr (FAMILY == 4) {
        switch (G.M) {
        case 1: dispatch_spring<T, 1, NMAP, TSFK>(a, G, it.k0, n0); break;
        case 2: dispatch_spring<T, 2, NMAP, TSFK>(a, G, it.k0, n0); break;
        case 3: dispatch_spring<T, 3, NMAP, TSFK>(a, G, it.k0, n0); break;
        case 4: dispatch_spring<T, 4, NMAP, TSFK>(a, G, it.k0, n0); break;
        default: break;
        }
    } else if constexpr (NMAP == 2) {   // the host picks 8, 12 or 16 beads per lane under map 2
        switch (G.M) {
        case 8: dispatch_spring<T, 8, 2, TSFK>(a, G, it.k0, n0); break;
        case 12: dispatch_spring<T, 12, 2, TSFK>(a, G, it.k0, n0); break;
        case 16: dispatch_spring<T, 16, 2, TSFK>(a, G, it.k0, n0); break;
        default: break;
        }
    } else {
        switch (G.M) {
        case 6: dispatch_spring<T, 6, 0, TSFK>(a, G, it.k0, n0); break;
        case 8: dispatch_spring<T, 8, 0, TSFK>(a, G, it.k0, n0); break;
        case 12: dispatch_spring<T, 12, 0, TSFK>(a, G, it.k0, n0); break;
        case 16: dispatch_spring<T, 16, 0, TSFK>(a, G, it.k0, n0); break;
        default: break;
        }
    }
}

template <typename T, int FAMILY, int WAVES_PER_EU, int NMAP, int TSFK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES_PER_EU)))
void fwd_kernel(FwdArgs a) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    fwd_item<T, FAMILY, NMAP, TSFK>(a, (int)blockIdx.x * (int)(blockDim.x >> 6) + wave);
}

// Two contexts in one launch (the RSF cycle's replicas of window w and the
// parent's next segment): blocks [0, blocks_a) run a's work list, the rest b's.
// One launch keeps the two concurrent whatever hardware queues the streams
// map to, and the parent's few waves get SIMDs of their own.
template <typename T, int FAMILY, int WAVES_PER_EU, int NMAP = 0>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES_PER_EU)))
void fwd_dual_kernel(FwdArgs a, FwdArgs b, int blocks_a) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wpb = (int)(blockDim.x >> 6);
    if ((int)blockIdx.x < blocks_a) fwd_item<T, FAMILY, NMAP, 2>(a, (int)blockIdx.x * wpb + wave);
    else fwd_item<T, FAMILY, NMAP, 2>(b, ((int)blockIdx.x - blocks_a) * wpb + wave);
}

// ---------------------------------------------------------------------------
// Launchers of one kernel family and noise map.
// ---------------------------------------------------------------------------
template <typename T, int FAMILY, int WPE, int NMAP>
static void launch_fwd_tsf(const FwdArgs& a, dim3 grid, dim3 block, hipStream_t st) {
    if (a.tsf) {
        hipLaunchKernelGGL((fwd_kernel<T, FAMILY, WPE, NMAP, 1>), grid, block, 0, st, a);
        return;
    }
    if constexpr (FAMILY == 4 && sizeof(T) == 4) {
        if (a.K == 1) {
            hipLaunchKernelGGL((fwd_kernel<T, FAMILY, WPE, NMAP, 3>), grid, block, 0, st, a);
            return;
        }
    }
    hipLaunchKernelGGL((fwd_kernel<T, FAMILY, WPE, NMAP, 0>), grid, block, 0, st, a);
}

template <typename T, int FAMILY, int WPE, int NMAP>
static void launch_fwd_two(const FwdArgs& a, const FwdArgs& b, int blocks_a, dim3 grid, dim3 block, hipStream_t st) {
    hipLaunchKernelGGL((fwd_dual_kernel<T, FAMILY, WPE, NMAP>), grid, block, 0, st, a, b, blocks_a);
}

}  // namespace ra

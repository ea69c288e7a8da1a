// ra_chain.hpp — per-lane chain state and the bond-form Euler-Maruyama step,
// shared by the forward kernels and the adjoint's segment recompute (which
// must reproduce the forward trajectory bit for bit).
//
// Bond form of Eq. (1) with the free-draining tensor Eq. (2):
//   Y_i  = G_i - G_{i-1} + sigma xi_i,   G_j = cF g_j Q_j,  cF = H dt/zeta,
//   Q_j' = Q_j + dt kappa Q_j + (Y_{j+1} - Y_j),  sigma = sqrt(2 kT dt/zeta)
// which is the difference of the bead update r_i' = r_i + dt (kappa r_i +
// Fnet_i/zeta) + sigma xi_i for beads j+1 and j: Y_i is bead i's displacement
// without the flow, formed once per bead and used by both its bonds. The
// increment is formed first and added once, so FP32 keeps the small flow term
// dt*rate*Q exactly as accurate as the other terms.
//
// The step is bound by VALU issue, so its form is the one with the fewest
// instructions. Against the same update written per bond (Laplacian of G, noise
// difference and sigma on each bond): 24 instructions of bond update per bead
// instead of 31 with cF in the spring's reciprocal, the noise product in the
// displacement's FMA and sigma in the Box-Muller radius; 4.5 more in the
// transform; 8 of 40 per Philox block (philox_block). 1000 beads (16 per lane, map
// 2, TSF, 8192 replicas, 5000 steps): 86.8 -> 75.4 ms; 512 chains of 20-200 beads,
// 500 steps: 6.42 -> 5.88 ms. One wavefront per SIMD (50 beads, 1024 replicas)
// is bound by latency as well: 1.86 -> 1.82 ms.
#pragma once
#include "ra_device.hpp"
#include "ra_types.hpp"

namespace ra {

__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <bool V> struct Bool { static constexpr bool value = V; };

template <typename T> struct Co;
template <> struct Co<float> {
    const GroupDev& G;
    __device__ float kx() const { return G.kx; }
    __device__ float ky() const { return G.ky; }
    __device__ float kz() const { return G.kz; }
    __device__ float kxz() const { return G.kxz; }
    __device__ float cF() const { return G.cF; }
    __device__ float sigma() const { return G.sigma; }
    __device__ float H() const { return G.H; }
    __device__ float iq() const { return G.inv_q0sq; }
};
template <> struct Co<double> {
    const GroupDev& G;
    __device__ double kx() const { return G.kx_d; }
    __device__ double ky() const { return G.ky_d; }
    __device__ double kz() const { return G.kz_d; }
    __device__ double kxz() const { return G.kxz_d; }
    __device__ double cF() const { return G.cF_d; }
    __device__ double sigma() const { return G.sigma_d; }
    __device__ double H() const { return G.H_d; }
    __device__ double iq() const { return G.inv_q0sq_d; }
};

// State of one lane: M bond slots.
template <typename T, int M> struct Lane {
    T qx[M], qy[M], qz[M];
};

// g_j for every slot (1 for Hookean), clamp count accumulated.
template <typename T, int M, bool FENE>
__device__ __forceinline__ void spring_factors(const Lane<T, M>& s, const GroupDev& G, T (&g)[M],
                                               int& clamps) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
        if constexpr (FENE) {
            const T q2 = fmadd(s.qx[m], s.qx[m], fmadd(s.qy[m], s.qy[m], s.qz[m] * s.qz[m]));
            g[m] = fene_g(s.qx[m], s.qy[m], s.qz[m], q2, (T)G.inv_q0sq, G.inv_q0sq_d, clamps);
        } else {
            g[m] = (T)1;
        }
    }
}

// Noise of the M beads of the lane at one step (bead j uses the counter
// (step, bead j, replica, tag|group)); independent of the chain state, so the
// forward kernel generates several steps ahead for instruction-level parallelism.
template <typename T, int M> struct Noise {
    Polar<T> x[M], y[M], z[M];
};

template <typename T> __device__ __forceinline__ T noise_amp(const GroupDev& G) {
    if constexpr (sizeof(T) == 4) return G.cN;
    else return G.cN_d;
}

// The lane's part of its counters: NB blocks (of the lane's beads, or of its
// groups of four beads under noise map 2) of one replica.
template <int NB, bool UNI> struct LaneCounters {
    BlockLane blk[NB];
    uint32_t rl;            // lo(M1 replica) (several replicas per wavefront)
    uint32_t replica, key0, key1, stream;

    __device__ __forceinline__ StepWords words(uint32_t n) const {
        return step_words<UNI>(n, UNI ? replica : 0u, stream, key0, key1);
    }
    __device__ __forceinline__ Words draw(int b, const StepWords& w, const RoundKeys& k) const {
        return philox_block<UNI>(blk[b], w, rl, k);
    }
};

template <int NB, bool UNI>
__device__ __forceinline__ LaneCounters<NB, UNI> lane_counters(uint32_t first, uint32_t replica, uint32_t stream,
                                                               uint32_t key0, uint32_t key1) {
    LaneCounters<NB, UNI> c;
#pragma unroll
    for (int b = 0; b < NB; ++b) c.blk[b] = block_lane(first + (uint32_t)b, replica, key0);
    c.rl = 0xCD9E8D57u * replica;
    c.replica = replica;
    c.key0 = key0;
    c.key1 = key1;
    c.stream = stream;
    return c;
}

// Blocks of a lane and the first block word, by noise map.
template <int M, int NMAP> struct LaneBlocks {
    static constexpr int value = NMAP == 2 ? 3 * M / 4 : M;
    static __device__ __forceinline__ uint32_t first(uint32_t bead0) { return NMAP == 2 ? 3u * (bead0 >> 2) : bead0; }
};

template <typename T, int M, bool UNI>
__device__ __forceinline__ void gen_noise(Noise<T, M>& e, const LaneCounters<M, UNI>& lc, const GroupDev& G,
                                          uint32_t n, const RoundKeys& keys) {
    const StepWords w = lc.words(n);
#pragma unroll
    for (int m = 0; m < M; ++m) {
        Polar<T> d;
        polars4(lc.draw(m, w, keys), noise_amp<T>(G), e.x[m], e.y[m], e.z[m], d);
    }
}

// Noise map 1: the block of step n gives four normals; steps 4m..4m+2 use the
// first three of their own block, step 4m+3 the fourth normals of the blocks
// of steps 4m, 4m+1, 4m+2 (as x, y, z). Three blocks serve four steps, and
// every step still gets three independent standard normals. The fourth
// normals wait in a per-slot carry until step 4m+3.
template <typename T, int M> struct Carry {
    Polar<T> c0[M], c1[M], c2[M];
};

template <typename T>
__device__ __forceinline__ void carry_slot(uint32_t r, const Polar<T>& d, Polar<T>& c0, Polar<T>& c1, Polar<T>& c2) {
    c0.r = r == 0u ? d.r : c0.r;
    c0.t = r == 0u ? d.t : c0.t;
    c1.r = r == 1u ? d.r : c1.r;
    c1.t = r == 1u ? d.t : c1.t;
    c2.r = r == 2u ? d.r : c2.r;
    c2.t = r == 2u ? d.t : c2.t;
}

// Noise of step n under map 1, updating the carry (r = n mod 4 is
// wave-uniform, so the branch is uniform and the carry slot a select).
template <typename T, int M, bool UNI>
__device__ __forceinline__ void gen_noise_map1(Noise<T, M>& e, Carry<T, M>& cy, const LaneCounters<M, UNI>& lc,
                                               const GroupDev& G, uint32_t n, const RoundKeys& keys) {
    const uint32_t r = n & 3u;
    if (r == 3u) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            e.x[m] = cy.c0[m];
            e.y[m] = cy.c1[m];
            e.z[m] = cy.c2[m];
        }
        return;
    }
    const StepWords w = lc.words(n);
#pragma unroll
    for (int m = 0; m < M; ++m) {
        Polar<T> d;
        polars4(lc.draw(m, w, keys), noise_amp<T>(G), e.x[m], e.y[m], e.z[m], d);
        carry_slot(r, d, cy.c0[m], cy.c1[m], cy.c2[m]);
    }
}

// Carry for a run that starts at step n: the fourth normals of the blocks of
// steps 4m .. n-1 of n's group of four (none when n is a multiple of 4).
template <typename T, int M, bool UNI>
__device__ __forceinline__ void init_carry(Carry<T, M>& cy, const LaneCounters<M, UNI>& lc, const GroupDev& G,
                                           uint32_t n, const RoundKeys& keys) {
    const uint32_t r = n & 3u;
#pragma unroll
    for (int m = 0; m < M; ++m) cy.c0[m] = cy.c1[m] = cy.c2[m] = Polar<T>{(T)0, (T)0};
    for (uint32_t q = 0; q < r; ++q) {
        const StepWords w = lc.words(n - r + q);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            Polar<T> a, b, c, d;
            polars4(lc.draw(m, w, keys), noise_amp<T>(G), a, b, c, d);
            carry_slot(q, d, cy.c0[m], cy.c1[m], cy.c2[m]);
        }
    }
}

// G_j = cF g_j Q_j of slot m (spring factor evaluated once per slot and step).
// With TSF the slot's cF g |Q| of the same state is added to tsum[m]: times
// uH = H / cF it is the tension f = H g |Q| (Eq. 4, zero rest length), so the
// step's force evaluation is the TSF sample of the state it starts from, and no
// second spring-law evaluation is needed for the time average.
template <typename T, int M, bool FENE>
__device__ __forceinline__ T slot_factor(const Lane<T, M>& s, const GroupDev& G, int m, T q2, int& clamps) {
    if constexpr (!FENE) return Co<T>{G}.cF();
    else if constexpr (sizeof(T) == 4)
        return fene_force(s.qx[m], s.qy[m], s.qz[m], q2, G.fA, G.fB, G.fT, G.fC_d, G.inv_q0sq_d, clamps);
    else return fene_force(s.qx[m], s.qy[m], s.qz[m], q2, G.cF_d, G.inv_q0sq_d, clamps);
}

template <typename T, int M, bool FENE, bool TSF = false>
__device__ __forceinline__ void slot_force(const Lane<T, M>& s, const GroupDev& G, int m, T& fx, T& fy, T& fz,
                                           int& clamps, T* tsum = nullptr) {
    T q2 = (T)0;
    if constexpr (FENE || TSF) q2 = fmadd(s.qx[m], s.qx[m], fmadd(s.qy[m], s.qy[m], s.qz[m] * s.qz[m]));
    const T h = slot_factor<T, M, FENE>(s, G, m, q2, clamps);
    if constexpr (TSF) tsum[m] = fmadd(h, fast_sqrt(q2), tsum[m]);
    fx = h * s.qx[m];
    fy = h * s.qy[m];
    fz = h * s.qz[m];
}

// cF g |Q| of every slot, the term that slot_force adds to a TSF sum.
template <typename T, int M, bool FENE>
__device__ __forceinline__ void tsf_terms(const Lane<T, M>& s, const GroupDev& G, T (&u)[M]) {
    int dummy = 0;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const T q2 = fmadd(s.qx[m], s.qx[m], fmadd(s.qy[m], s.qy[m], s.qz[m] * s.qz[m]));
        u[m] = slot_factor<T, M, FENE>(s, G, m, q2, dummy) * fast_sqrt(q2);
    }
}

// 1 on slots that are a spring of an active replica, 0 on the others: the
// update is Q + mask * increment in one FMA (exactly Q + increment where the
// mask is 1), so a slot that holds Q = 0 and is no spring stays 0 without a
// select. Used for up to 4 slots per lane; wider lanes have no registers for it
// and select instead.
template <typename T, int M> struct SlotMask {
    T v[M];
};

template <typename T, int M>
__device__ __forceinline__ SlotMask<T, M> slot_mask(const bool (&valid)[M]) {
    SlotMask<T, M> k;
#pragma unroll
    for (int m = 0; m < M; ++m) k.v[m] = valid[m] ? (T)1 : (T)0;
    return k;
}

template <int M> struct MaskedSlots { static constexpr bool value = M <= 4; };

// One Euler-Maruyama step of every slot of the lane. xi(m, x, y, z) yields
// the noise of bead j0 + m (precomputed or generated on demand — the value
// is the same). The update of slot m needs the displacements of beads m and
// m+1, hence G of slots m-1..m+1: both roll through the slots. The lane's first
// bead needs the previous lane's last G, its last slot the next lane's first
// displacement, by DPP. valid[m] and mask hold the slots that are a spring of an
// active replica.
template <typename T, int M, bool FENE, bool TSF = false, typename NoiseFn>
__device__ __forceinline__ void physics_step_fn(Lane<T, M>& s, NoiseFn&& xi, const GroupDev& G,
                                                const bool (&valid)[M], const SlotMask<T, M>& mask, int& clamps,
                                                T* tsum = nullptr) {
    const Co<T> c{G};
    T f0x, f0y, f0z, flx, fly, flz;
    slot_force<T, M, FENE, TSF>(s, G, 0, f0x, f0y, f0z, clamps, tsum);
    if constexpr (M > 1) {
        slot_force<T, M, FENE, TSF>(s, G, M - 1, flx, fly, flz, clamps, tsum);
    } else {
        flx = f0x; fly = f0y; flz = f0z;
    }
    const T kx = c.kx(), ky = c.ky(), kz = c.kz(), kxz = c.kxz();
    Polar<T> ex, ey, ez;
    xi(0, ex, ey, ez);
    T Cx = f0x, Cy = f0y, Cz = f0z;   // G of slot m
    // displacement of bead m
    T Yx = fmadd(ex.r, ex.t, f0x - from_prev_lane(flx));
    T Yy = fmadd(ey.r, ey.t, f0y - from_prev_lane(fly));
    T Yz = fmadd(ez.r, ez.t, f0z - from_prev_lane(flz));
    const T Lx = from_next_lane(Yx), Ly = from_next_lane(Yy), Lz = from_next_lane(Yz);
#pragma unroll
    for (int m = 0; m < M; ++m) {
        T Nx, Ny, Nz, Zx, Zy, Zz;     // G of slot m+1, displacement of bead m+1
        if (m + 1 < M) {
            if (m + 1 == M - 1) { Nx = flx; Ny = fly; Nz = flz; }
            else slot_force<T, M, FENE, TSF>(s, G, m + 1 < M ? m + 1 : m, Nx, Ny, Nz, clamps, tsum);
            xi(m + 1, ex, ey, ez);
            Zx = fmadd(ex.r, ex.t, Nx - Cx);
            Zy = fmadd(ey.r, ey.t, Ny - Cy);
            Zz = fmadd(ez.r, ez.t, Nz - Cz);
        } else {
            Nx = Ny = Nz = (T)0;
            Zx = Lx; Zy = Ly; Zz = Lz;
        }
        const T ix = fmadd(kx, s.qx[m], fmadd(kxz, s.qz[m], Zx - Yx));
        const T iy = fmadd(ky, s.qy[m], Zy - Yy);
        const T iz = fmadd(kz, s.qz[m], Zz - Yz);
        if constexpr (MaskedSlots<M>::value) {
            s.qx[m] = fmadd(ix, mask.v[m], s.qx[m]);
            s.qy[m] = fmadd(iy, mask.v[m], s.qy[m]);
            s.qz[m] = fmadd(iz, mask.v[m], s.qz[m]);
        } else {
            s.qx[m] = valid[m] ? s.qx[m] + ix : (T)0;
            s.qy[m] = valid[m] ? s.qy[m] + iy : (T)0;
            s.qz[m] = valid[m] ? s.qz[m] + iz : (T)0;
        }
        Cx = Nx; Cy = Ny; Cz = Nz;
        Yx = Zx; Yy = Zy; Yz = Zz;
    }
}

template <typename T, int M, bool FENE, bool TSF = false>
__device__ __forceinline__ void physics_step(Lane<T, M>& s, const Noise<T, M>& e, const GroupDev& G,
                                             const bool (&valid)[M], const SlotMask<T, M>& mask, int& clamps,
                                             T* tsum = nullptr) {
    physics_step_fn<T, M, FENE, TSF>(
        s, [&](int m, Polar<T>& x, Polar<T>& y, Polar<T>& z) { x = e.x[m]; y = e.y[m]; z = e.z[m]; }, G, valid, mask,
        clamps, tsum);
}

// One full Euler-Maruyama step at global step n (noise + update).
template <typename T, int M, bool FENE, bool TSF = false, bool UNI = false>
__device__ __forceinline__ void em_step(Lane<T, M>& s, const LaneCounters<M, UNI>& lc, const GroupDev& G,
                                        const bool (&valid)[M], const SlotMask<T, M>& mask, uint32_t n,
                                        const RoundKeys& keys, int& clamps, T* tsum = nullptr) {
    const StepWords w = lc.words(n);
    physics_step_fn<T, M, FENE, TSF>(
        s,
        [&](int m, Polar<T>& x, Polar<T>& y, Polar<T>& z) {
            Polar<T> d;
            polars4(lc.draw(m, w, keys), noise_amp<T>(G), x, y, z, d);
        },
        G, valid, mask, clamps, tsum);
}

// One step at global step n under map 1 (noise from and into the carry).
template <typename T, int M, bool FENE, bool TSF = false, bool UNI = false>
__device__ __forceinline__ void em_step_map1(Lane<T, M>& s, Carry<T, M>& cy, const LaneCounters<M, UNI>& lc,
                                             const GroupDev& G, const bool (&valid)[M], const SlotMask<T, M>& mask,
                                             uint32_t n, const RoundKeys& keys, int& clamps, T* tsum = nullptr) {
    Noise<T, M> e;
    gen_noise_map1<T, M, UNI>(e, cy, lc, G, n, keys);
    physics_step<T, M, FENE, TSF>(s, e, G, valid, mask, clamps, tsum);
}

// Noise map 2, for lanes of a multiple of four beads (the lane's first bead
// is then a multiple of four too): the beads are taken in groups of four,
// j = 4q + r, and the three blocks of counters (step, 3q + c, replica,
// tag|group), c = 0, 1, 2, give four normals each; bead 4q + r takes normal r
// of block c as its component c. Three blocks serve four bead-steps, as under
// map 1, but with no carry from step to step. The step's Philox blocks are
// drawn first (integer work with twelve independent chains at 16 beads per
// lane) and each group's Box-Muller transform runs when the update reaches
// the group's first bead, which spreads the transcendentals over the step
// (measured on 16 beads per lane: 2% faster than transforming all twelve
// blocks up front, 4% faster than drawing and transforming each group at its
// first bead).
template <typename T, int M, bool FENE, bool TSF = false, bool UNI = false>
__device__ __forceinline__ void em_step_map2(Lane<T, M>& s, const LaneCounters<3 * M / 4, UNI>& lc, const GroupDev& G,
                                             const bool (&valid)[M], const SlotMask<T, M>& mask, uint32_t n,
                                             const RoundKeys& keys, int& clamps, T* tsum = nullptr) {
    static_assert(M % 4 == 0, "noise map 2 takes the beads of a lane in groups of four");
    const StepWords sw = lc.words(n);
    Words w[3 * M / 4];
#pragma unroll
    for (int b = 0; b < 3 * M / 4; ++b) w[b] = lc.draw(b, sw, keys);
    Polar<T> gx[4], gy[4], gz[4];
    physics_step_fn<T, M, FENE, TSF>(
        s,
        [&](int m, Polar<T>& x, Polar<T>& y, Polar<T>& z) {
            if ((m & 3) == 0) {
                const T cn = noise_amp<T>(G);
                const int b = 3 * (m >> 2);
                polars4(w[b], cn, gx[0], gx[1], gx[2], gx[3]);
                polars4(w[b + 1], cn, gy[0], gy[1], gy[2], gy[3]);
                polars4(w[b + 2], cn, gz[0], gz[1], gz[2], gz[3]);
            }
            x = gx[m & 3];
            y = gy[m & 3];
            z = gz[m & 3];
        },
        G, valid, mask, clamps, tsum);
}

// Tension f_j = H g_j |Q_j| (Eq. 4, zero rest length) of every slot.
template <typename T, int M, bool FENE>
__device__ __forceinline__ void tensions(const Lane<T, M>& s, const GroupDev& G, T (&f)[M]) {
    int dummy = 0;
    T g[M];
    spring_factors<T, M, FENE>(s, G, g, dummy);
    const T H = Co<T>{G}.H();
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const T q2 = fmadd(s.qx[m], s.qx[m], fmadd(s.qy[m], s.qy[m], s.qz[m] * s.qz[m]));
        f[m] = H * g[m] * fast_sqrt(q2);
    }
}

struct TileGeom {
    int t, k;          // lane position in its replica, replica index
    bool rep_ok;       // lane belongs to an existing replica
    int j0;            // first bead/spring of the lane
};

// With UNIFORM_K (one replica per wavefront, P = 1) every lane carries the
// wave-uniform replica index, so the replica word of the Philox counter stays
// in a scalar register and part of the first rounds runs on the scalar unit.
template <bool UNIFORM_K = false>
__device__ __forceinline__ TileGeom tile_geom(const GroupDev& G, int k_first, int M) {
    const int lane = threadIdx.x & (WAVE - 1);
    TileGeom tg;
    if constexpr (UNIFORM_K) {
        tg.t = lane;
        tg.k = k_first;
        tg.rep_ok = (lane < G.L) && (k_first < G.R);
    } else {
        const int seg = lane / G.L;
        tg.t = lane - seg * G.L;
        tg.k = k_first + seg;
        tg.rep_ok = (seg < G.P) && (tg.k < G.R);
    }
    tg.j0 = tg.t * M;
    return tg;
}

template <typename T, int M>
__device__ __forceinline__ void load_lane(Lane<T, M>& s, bool (&valid)[M], const T* __restrict__ src,
                                          const GroupDev& G, const TileGeom& tg) {
    const int nm1 = G.N - 1;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int j = tg.j0 + m;
        valid[m] = tg.rep_ok && j < nm1;
        T x = (T)0, y = (T)0, z = (T)0;
        if (valid[m]) {
            const int64_t o = G.state_off + ((int64_t)tg.k * nm1 + j) * 3;
            x = src[o];
            y = src[o + 1];
            z = src[o + 2];
        }
        s.qx[m] = x;
        s.qy[m] = y;
        s.qz[m] = z;
    }
}

template <typename T, int M>
__device__ __forceinline__ void store_lane(const Lane<T, M>& s, const bool (&valid)[M], T* __restrict__ dst,
                                           const GroupDev& G, const TileGeom& tg) {
    const int nm1 = G.N - 1;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        if (valid[m]) {
            const int64_t o = G.state_off + ((int64_t)tg.k * nm1 + tg.j0 + m) * 3;
            dst[o] = s.qx[m];
            dst[o + 1] = s.qy[m];
            dst[o + 2] = s.qz[m];
        }
    }
}

// Checkpoint rows of one work item: [slot m][xyz][lane], U = P L lanes per
// row, so each store or load instruction covers U consecutive values. Slots
// that are not a spring of a replica hold 0.
template <typename T, int M>
__device__ __forceinline__ T* ckpt_item(T* base, const GroupDev& G, int k_first) {
    return base + G.ck_off + (int64_t)(k_first / G.P) * (M * 3 * G.P * G.L);
}

template <typename T, int M>
__device__ __forceinline__ void store_ckpt(const Lane<T, M>& s, T* __restrict__ dst, const GroupDev& G) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int U = G.P * G.L;
    if (lane < U) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            dst[(3 * m) * U + lane] = s.qx[m];
            dst[(3 * m + 1) * U + lane] = s.qy[m];
            dst[(3 * m + 2) * U + lane] = s.qz[m];
        }
    }
}

// The same in FP32 through a buffer resource of exactly the rows' size: the lanes past
// U get an offset out of it, so their stores are dropped and their loads give 0
// without a branch in the step loops.
template <int M> struct Rows {
    int offset, row;                // bytes: this lane's first value, one row
    __device__ __forceinline__ explicit Rows(const GroupDev& G) {
        const int lane = threadIdx.x & (WAVE - 1), U = G.P * G.L;
        row = 4 * U;
        offset = lane < U ? 4 * lane : 3 * M * row;
    }
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const float* p) const {
        return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, 3 * M * row, 0x00020000);
    }
    __device__ __forceinline__ void store(const Lane<float, M>& s, float* p) const {
        const auto r = rsrc(p);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s.qx[m]), r, offset, 3 * m * row, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s.qy[m]), r, offset, (3 * m + 1) * row, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s.qz[m]), r, offset, (3 * m + 2) * row, 0);
        }
    }
    __device__ __forceinline__ void load(Lane<float, M>& s, const float* p) const {
        const auto r = rsrc(p);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            s.qx[m] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, offset, 3 * m * row, 0));
            s.qy[m] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, offset, (3 * m + 1) * row, 0));
            s.qz[m] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, offset, (3 * m + 2) * row, 0));
        }
    }
};

template <typename T, int M>
__device__ __forceinline__ void load_ckpt(Lane<T, M>& s, bool (&valid)[M], const T* __restrict__ src,
                                          const GroupDev& G, const TileGeom& tg) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int U = G.P * G.L;
    const int nm1 = G.N - 1;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        valid[m] = tg.rep_ok && tg.j0 + m < nm1;
        T x = (T)0, y = (T)0, z = (T)0;
        if (valid[m] && lane < U) {
            x = src[(3 * m) * U + lane];
            y = src[(3 * m + 1) * U + lane];
            z = src[(3 * m + 2) * U + lane];
        }
        s.qx[m] = x;
        s.qy[m] = y;
        s.qz[m] = z;
    }
}

__device__ __forceinline__ void flush_clamps(int clamps, unsigned long long* counter) {
    if (clamps) atomicAdd(counter, (unsigned long long)clamps);
}

}  // namespace ra

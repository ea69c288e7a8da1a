// ra_pair.hip — forward kernel of the collapsed-polymer force field (Sec. II):
// backbone springs (rest-length harmonic kappa/2 (r - r0)^2, or the Hookean
// and FENE laws) plus Lennard-Jones self-association between non-adjacent
// beads, free-draining (Eq. 1 with the self term Eq. 2 only).
//
// Bound by the issue of the pair loop (13 instructions and a reciprocal per pair and
// lane), and with few items by its latency in a single wavefront: up to four
// wavefronts step one item together (fwd_pair_shared_kernel), one run of the
// partners each. 50 beads, FP32, us a step: 50 replicas 2.31 -> 1.18, 512 2.30 -> 1.38,
// 1000 2.31 -> 2.12, 2048 3.24 -> 3.2 (four sums in place of one, so that the bits
// stay the same for any number of wavefronts); FP64: 50 replicas 4.74 -> 2.16, 1024
// 4.95 -> 4.90, 2048 9.55 -> 8.08.
//
// One bead per lane, P = floor(64/N) replicas per wavefront (N <= 64). The
// state stays the bond vectors Q_j (as in the chain kernels, so FP32 keeps
// bond-scale precision however far the chain drifts in the flow); the bead
// positions relative to bead 0 are rebuilt every step by a wave scan of the
// bonds (DPP with one replica per wavefront, lane shuffles per segment with
// several) and shared through LDS for the O(N^2) pair forces. The
// bond update is the difference of the bead updates of beads j+1 and j:
//   Q_j' = Q_j + dt kappa Q_j + (dt/zeta) (F_{j+1} - F_j) + sigma (xi_{j+1} - xi_j)
// with F_i the total force on bead i (springs + LJ).
#include "ra_chain.hpp"
#include "ra_dpp.hpp"
#include "ra_launch.hpp"

namespace ra {

template <typename T> struct PairCo;
template <> struct PairCo<float> {
    const GroupDev& G;
    __device__ float dtz() const { return G.dtz; }
    __device__ float r0() const { return G.r0; }
};
template <> struct PairCo<double> {
    const GroupDev& G;
    __device__ double dtz() const { return G.dtz_d; }
    __device__ double r0() const { return G.r0_d; }
};

// Force of the spring on bond Q acting on its first bead (toward the second).
template <typename T, int SPRING>
__device__ __forceinline__ void pair_spring_force(T qx, T qy, T qz, const GroupDev& G, T& fx, T& fy, T& fz,
                                                  int& clamps) {
    const T H = Co<T>{G}.H();
    const T q2 = fmadd(qx, qx, fmadd(qy, qy, qz * qz));
    T g;
    if constexpr (SPRING == 0) {
        g = (T)1;
    } else if constexpr (SPRING == 1) {
        g = fene_g(qx, qy, qz, q2, (T)G.inv_q0sq, G.inv_q0sq_d, clamps);
    } else {
        const T q = fast_sqrt(q2);
        g = q > (T)0 ? (T)1 - PairCo<T>{G}.r0() * fast_rcp(q) : (T)0;
    }
    const T Hg = H * g;
    fx = Hg * qx;
    fy = Hg * qy;
    fz = Hg * qz;
}

// Spring tension of Eq. 4: signed H (|Q| - r0) for the rest-length spring,
// H g |Q| for the zero-rest-length laws.
template <typename T, int SPRING>
__device__ __forceinline__ T pair_tension(T qx, T qy, T qz, const GroupDev& G) {
    const T H = Co<T>{G}.H();
    const T q2 = fmadd(qx, qx, fmadd(qy, qy, qz * qz));
    const T q = fast_sqrt(q2);
    if constexpr (SPRING == 2) {
        return H * (q - PairCo<T>{G}.r0());
    } else if constexpr (SPRING == 1) {
        int dummy = 0;
        return H * fene_g(qx, qy, qz, q2, (T)G.inv_q0sq, G.inv_q0sq_d, dummy) * q;
    } else {
        return H * q;
    }
}

// Inclusive scan of v over the lanes of each replica segment (bead index i
// within the segment): after it, lane i holds the sum over beads 0..i.
template <typename T>
__device__ __forceinline__ T segment_scan(T v, int i) {
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const T u = __shfl_up(v, (unsigned)off, WAVE);
        if (i >= off) v += u;
    }
    return v;
}

// LJ sums of one bead, in units of rmin: s = rmin^2 / r^2 is the reciprocal of the
// scaled r^2, and the pair term is s (s^6 - s^3) dx'. `row` is the bead's own row of
// the doubled table: partner i + t is row t.
// The reciprocal is paced (see paced()) where wavefronts share an item or hold one
// replica each; several short replicas per wavefront are 1-6% faster without (8000 replicas of
// 12 beads, 100 steps, 178 against 173 us; 50 beads, 4000 replicas, 551 against 561 with).
template <typename T, bool PACED> struct PairSum {
    T x, y, z;
    __device__ __forceinline__ static float rcp(float v) {
        if constexpr (PACED) return paced<'r'>(v);
        else return fast_rcp(v);
    }
    __device__ __forceinline__ static double rcp(double v) { return fast_rcp(v); }
    __device__ __forceinline__ void add(T px, T py, T pz, const T* r, bool use) {
        const T dx = px - r[0], dy = py - r[1], dz = pz - r[2];
        const T s = rcp(fmadd(dx, dx, fmadd(dy, dy, dz * dz)));
        const T s3 = s * s * s;
        // a select, not a product: drops the Inf/NaN of a coincident bonded neighbour
        const T h = use ? s * fmadd(s3, s3, -s3) : (T)0;
        x = fmadd(h, dx, x);
        y = fmadd(h, dy, y);
        z = fmadd(h, dz, z);
    }
    __device__ __forceinline__ PairSum operator+(const PairSum& o) const { return {x + o.x, y + o.y, z + o.z}; }
};

// The partners t = 2 .. N - 2 (never the bead itself or a bonded neighbour) are cut
// into blocks of four, independent reciprocal chains, and the blocks into PARTS
// runs; the last run also takes the wrap-around pair of beads 0 and N - 1 (N >= 3),
// which the bead table meets at t = 1 and t = N - 1. A bead's force is the sum over
// the runs in fixed order, whichever wavefronts take them.
constexpr int PARTS = 4;

template <typename T, bool PACED>
__device__ __forceinline__ PairSum<T, PACED> pair_part(int part, T px, T py, T pz, const T* row, int i, int N) {
    PairSum<T, PACED> l{(T)0, (T)0, (T)0};
    const int nm1 = N - 1;
    const int blocks = N > 3 ? N / 4 : 0;                // ceil((N - 3) / 4)
    if (part == PARTS - 1 && N >= 3) l.add(px, py, pz, row + 4 * (i == 0 ? nm1 : 1), i == 0 || i == nm1);
    int t = 2 + 4 * (blocks * part / PARTS);
    const int end = 2 + 4 * (blocks * (part + 1) / PARTS);
    const int whole = min(end, 2 + ((nm1 - 2) & ~3));
    if constexpr (sizeof(T) == 4) {
        for (; t < whole; t += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) l.add(px, py, pz, row + 4 * (t + u), true);
        }
    } else if (t < whole) {
        // FP64: the next block's rows are read before this one's arithmetic, where the
        // reciprocal is a division (1000 replicas of 50 beads, one wavefront each: 4.82
        // against 5.86 us a step; FP32, slower: 3.23 against 2.65)
        T r[2][4][3];
        auto load = [&](T (&q)[4][3], int t4) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int d = 0; d < 3; ++d) q[u][d] = row[4 * (t4 + u) + d];
        };
        auto sum = [&](const T (&q)[4][3]) {
#pragma unroll
            for (int u = 0; u < 4; ++u) l.add(px, py, pz, q[u], true);
        };
        load(r[0], t);
        for (;;) {
            if (t + 4 < whole) load(r[1], t + 4);
            sum(r[0]);
            t += 4;
            if (t >= whole) break;
            if (t + 4 < whole) load(r[0], t + 4);
            sum(r[1]);
            t += 4;
            if (t >= whole) break;
        }
    }
    if (t < end) {
#pragma unroll
        for (int u = 0; u < 4; ++u) l.add(px, py, pz, row + 4 * (t + u < nm1 ? t + u : t), t + u < nm1);
    }
    return l;
}

// LDS of a workgroup whose PARTS wavefronts step one work item together.
template <typename T> struct PairShare {
    alignas(16) T part[2][PARTS][WAVE][4];      // sums of each wavefront's partners, by step parity
    alignas(16) T noise[2 * PARTS][WAVE][4];    // normals of the coming steps, one step per wavefront
};

// WAVES = 1: one wavefront per work item. WAVES = PARTS: all wavefronts hold the
// state and step it alike; each sums one run of the partners and draws every fourth
// step's noise. One barrier a step: the sums are written before and read after it,
// the noise of a step is read before it.
template <typename T, int SPRING, bool LJ, int WAVES, bool ONE_SEG>
__device__ __forceinline__ void run_pair(const FwdArgs& a, const GroupDev& Gm, int k_first, T (*xs)[4], int wave,
                                         PairShare<T>* sh) {
    // the group's constants as a local value: read through the reference,
    // the step loop re-loads them from memory every iteration
    const GroupDev G = Gm;
    const int gidx = (int)(&Gm - a.groups);
    const int lane = threadIdx.x & (WAVE - 1);
    const int N = G.N, nm1 = N - 1;
    const int seg = lane / N;
    const int i = lane - seg * N;
    const int k = k_first + seg;
    const bool rep_ok = seg < G.P && k < G.R;
    const bool bond_ok = rep_ok && i < nm1;
    T* const state = (T*)a.state;
    const int64_t sidx = ((int64_t)k * nm1 + i);
    T qx = (T)0, qy = (T)0, qz = (T)0;
    if (bond_ok) {
        const int64_t o = G.state_off + sidx * 3;
        qx = state[o];
        qy = state[o + 1];
        qz = state[o + 2];
    }
    const Co<T> c{G};
    const PairCo<T> pc{G};
    // coefficients are zero on lanes without a bond
    const T kx = bond_ok ? c.kx() : (T)0, ky = bond_ok ? c.ky() : (T)0, kz = bond_ok ? c.kz() : (T)0;
    const T kxz = bond_ok ? c.kxz() : (T)0;
    const T dtz = bond_ok ? pc.dtz() : (T)0, sg = bond_ok ? c.sigma() : (T)0;
    // LJ in units of rmin: positions scaled by 1/rmin, the pair sum scaled
    // back by 12 u / rmin at the end
    const T irm = (T)(1.0 / sqrt(G.ljr2_d)), ljf = (T)(G.lj12u_d / sqrt(G.ljr2_d));
    // LDS rows of this lane's replica: its positions twice over (rows
    // tb .. tb + 2N - 1), so that partner i + t is row tb + i + t for every
    // t < N; lanes past the last segment read segment 0 and write nothing
    const bool seg_ok = seg < G.P;
    const int tb = seg_ok ? 2 * N * seg : 0;
    const RoundKeys keys = round_keys(a.key0, a.key1);
    const uint32_t n0 = (uint32_t)*a.step0;
    const int S = a.S;
    const int64_t smp_total = a.smp_total;
    const bool tsf = a.tsf != nullptr;
    double acc = 0.0;
    if (tsf && bond_ok) acc = a.tsf_acc[G.smp_off + sidx];
    int to_smp = S - (int)(n0 % (uint32_t)S);
    int64_t w = (int64_t)(n0 / (uint32_t)S);
    int clamps = 0;
    const int n_steps = (int)a.n_steps;
    auto draw = [&](uint32_t n, T& x, T& y, T& z) {
        normals3(philox10(n, (uint32_t)i, (uint32_t)k, G.stream, keys), x, y, z);
    };
    // this wavefront's share of the PARTS steps from st
    auto share_noise = [&](int st) {
        T* e = sh->noise[(st + wave) & (2 * WAVES - 1)][lane];
        draw(n0 + (uint32_t)(st + wave), e[0], e[1], e[2]);
    };
    if constexpr (WAVES > 1) {
        share_noise(0);
        __syncthreads();
    }
    const bool writes = WAVES == 1 || wave == 0;
    for (int st = 0; st < n_steps; ++st) {
        const uint32_t n = n0 + (uint32_t)st;
        T ex, ey, ez;
        if constexpr (WAVES > 1) {
            if ((st & (WAVES - 1)) == 0) share_noise(st + WAVES);
            const T* e = sh->noise[st & (2 * WAVES - 1)][lane];
            ex = e[0];
            ey = e[1];
            ez = e[2];
        }
        T gx, gy, gz;
        pair_spring_force<T, SPRING>(qx, qy, qz, G, gx, gy, gz, clamps);
        // net force on bead i: spring i pulls toward i+1, spring i-1 pulls back
        // (the previous lane of bead 0 is the bondless last bead of the
        // previous replica, or lane -1, and contributes 0)
        T Fx = gx - from_prev_lane(gx), Fy = gy - from_prev_lane(gy), Fz = gz - from_prev_lane(gz);
        if constexpr (LJ) {
            // one replica per wavefront (N > 32): the whole-wave DPP scan;
            // else the segmented scan by lane shuffles
            T sx, sy, sz;
            if constexpr (ONE_SEG) {
                sx = qx;
                sy = qy;
                sz = qz;
                wave_scan_incl(sx, sy, sz);
            } else {
                sx = segment_scan(qx, i);
                sy = segment_scan(qy, i);
                sz = segment_scan(qz, i);
            }
            const T px = (sx - qx) * irm, py = (sy - qy) * irm, pz = (sz - qz) * irm;
            if (seg_ok) {
                xs[tb + i][0] = px;
                xs[tb + i][1] = py;
                xs[tb + i][2] = pz;
                xs[tb + i + N][0] = px;
                xs[tb + i + N][1] = py;
                xs[tb + i + N][2] = pz;
            }
            // this wave alone uses its LDS rows: make the writes visible to
            // its own reads (and keep the next step's writes after them)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const T* row = xs[tb + i];
            constexpr bool PACED = WAVES > 1 || ONE_SEG;
            using Sum = PairSum<T, PACED>;
            auto part_sum = [&](int p) { return pair_part<T, PACED>(p, px, py, pz, row, i, N); };
            Sum l;
            if constexpr (WAVES == 1) {
                const Sum a0 = part_sum(0), a1 = part_sum(1), a2 = part_sum(2), a3 = part_sum(3);
                l = (a0 + a1) + (a2 + a3);
            } else {
                T(*part)[WAVE][4] = sh->part[st & 1];
#pragma unroll
                for (int q = 0; q < PARTS / WAVES; ++q) {
                    const int w = wave * (PARTS / WAVES) + q;
                    const Sum own = part_sum(w);
                    part[w][lane][0] = own.x;
                    part[w][lane][1] = own.y;
                    part[w][lane][2] = own.z;
                }
                __syncthreads();
                auto get = [&](int w) { return Sum{part[w][lane][0], part[w][lane][1], part[w][lane][2]}; };
                l = (get(0) + get(1)) + (get(2) + get(3));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            Fx += l.x * ljf;
            Fy += l.y * ljf;
            Fz += l.z * ljf;
        }
        if constexpr (WAVES == 1) draw(n, ex, ey, ez);
        const T Fnx = from_next_lane(Fx), Fny = from_next_lane(Fy), Fnz = from_next_lane(Fz);
        const T enx = from_next_lane(ex), eny = from_next_lane(ey), enz = from_next_lane(ez);
        const T ix = fmadd(kx, qx, fmadd(kxz, qz, fmadd(dtz, Fnx - Fx, sg * (enx - ex))));
        const T iy = fmadd(ky, qy, fmadd(dtz, Fny - Fy, sg * (eny - ey)));
        const T iz = fmadd(kz, qz, fmadd(dtz, Fnz - Fz, sg * (enz - ez)));
        // lanes without a bond keep Q = 0 whatever their neighbours hold
        qx = bond_ok ? qx + ix : (T)0;
        qy = bond_ok ? qy + iy : (T)0;
        qz = bond_ok ? qz + iz : (T)0;
        const bool window_end = --to_smp == 0;
        if (tsf || window_end) {
            const T f = pair_tension<T, SPRING>(qx, qy, qz, G);
            if (tsf) acc += (double)f;
            if (window_end) {
                bool bad = false;
                if (bond_ok && writes) {
                    const int64_t o = w * smp_total + G.smp_off + sidx;
                    ((T*)a.samples)[o] = f;
                    bad = !__builtin_isfinite((double)f);
                    if (tsf) ((T*)a.tsf)[o] = (T)(acc / (double)S);
                }
                acc = 0.0;
                if (bad) atomicOr(a.status, 2);
                to_smp = S;
                ++w;
            }
        }
    }
    if (!writes) return;
    if (bond_ok) {
        const int64_t o = G.state_off + sidx * 3;
        state[o] = qx;
        state[o + 1] = qy;
        state[o + 2] = qz;
        if (tsf) a.tsf_acc[G.smp_off + sidx] = acc;
    }
    flush_clamps(clamps, a.clamps + gidx);
}

template <typename T, int WAVES>
__device__ __forceinline__ void pair_item(const FwdArgs& a, int item, T (*xs)[4], int wave, PairShare<T>* sh) {
    if (item >= a.n_items) return;
    if (*(const volatile int*)a.status & 1) return;   // invalid parent: no work (whole block)
    const Item it = a.items[item];
    const GroupDev& G = a.groups[it.g];
    if (G.lj12u_d > 0.0 && G.N > 2) {                 // two beads have no pair that is not bonded
        auto run = [&](auto One) {
            constexpr bool ONE = decltype(One)::value;
            if (G.spring == 0) run_pair<T, 0, true, WAVES, ONE>(a, G, it.k0, xs, wave, sh);
            else if (G.spring == 1) run_pair<T, 1, true, WAVES, ONE>(a, G, it.k0, xs, wave, sh);
            else run_pair<T, 2, true, WAVES, ONE>(a, G, it.k0, xs, wave, sh);
        };
        if (G.P == 1) run(Bool<true>{});
        else run(Bool<false>{});
    } else if (wave == 0 || WAVES == 1) {             // springs alone: nothing to share
        if (G.spring == 0) run_pair<T, 0, false, 1, false>(a, G, it.k0, xs, wave, sh);
        else if (G.spring == 1) run_pair<T, 1, false, 1, false>(a, G, it.k0, xs, wave, sh);
        else run_pair<T, 2, false, 1, false>(a, G, it.k0, xs, wave, sh);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void fwd_pair_kernel(FwdArgs a) {
    __shared__ T xs[4][2 * WAVE][4];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    pair_item<T, 1>(a, (int)blockIdx.x * (int)(blockDim.x >> 6) + wave, xs[wave], wave, nullptr);
}

// Two contexts in one launch (see fwd_dual_kernel): blocks [0, blocks_a) run a.
template <typename T>
__global__ __launch_bounds__(256) void fwd_pair_dual_kernel(FwdArgs a, FwdArgs b, int blocks_a) {
    __shared__ T xs[4][2 * WAVE][4];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wpb = (int)(blockDim.x >> 6);
    const bool first = (int)blockIdx.x < blocks_a;
    const int block = first ? (int)blockIdx.x : (int)blockIdx.x - blocks_a;
    pair_item<T, 1>(first ? a : b, block * wpb + wave, xs[wave], wave, nullptr);
}

// Few work items: one workgroup each; items [0, a.n_items) are a's, the rest b's.
template <typename T, int WAVES>
__global__ __launch_bounds__(WAVE * WAVES) void fwd_pair_shared_kernel(FwdArgs a, FwdArgs b) {
    __shared__ T xs[WAVES][2 * WAVE][4];
    __shared__ PairShare<T> sh;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool first = (int)blockIdx.x < a.n_items;
    pair_item<T, WAVES>(first ? a : b, first ? (int)blockIdx.x : (int)blockIdx.x - a.n_items, xs[wave], wave, &sh);
}

// Wavefronts per work item. Measured, us a step at 512 / 768 / 1024 / 1280 / 1536
// items with four, two and one: FP32, 50 beads 1.40 1.76 2.16 2.78 3.11, 1.91 1.94 2.15
// 2.63 3.14, 2.54 2.58 2.68 3.32 3.33; 24 beads 1.41 1.73 2.08, 1.50 1.60 1.74 2.04 2.32,
// 1.93 1.97 2.01 2.37 2.37; FP64, 50 beads 3.20 4.87 6.11, 4.48 4.62 5.10 7.18,
// 4.77 4.91 4.97 7.93. Four share the work best while a CU holds two items; from
// there the state that each steps for itself costs more than their overlap gives, the
// earlier the fewer partners there are to share (100 steps, us, at 800 / 1250 items with two
// and one: 6 beads 123 145, 110 123; 9 beads 128 150, 121 145; 12 beads 143 167, 134 165;
// 16 beads 144 171, 149 184).
static int pair_waves(int n_items, int precision, int max_beads) {
    if (n_items <= 512) return 4;
    return n_items <= (precision == 64 || max_beads <= 12 ? 768 : 1280) ? 2 : 1;
}

template <typename T> static void launch_shared(const FwdArgs& a, const FwdArgs& b, int waves, hipStream_t st) {
    const dim3 grid((unsigned)(a.n_items + b.n_items)), block(WAVE * waves);
    if (waves == 4) hipLaunchKernelGGL((fwd_pair_shared_kernel<T, 4>), grid, block, 0, st, a, b);
    else hipLaunchKernelGGL((fwd_pair_shared_kernel<T, 2>), grid, block, 0, st, a, b);
}

static hipError_t launch_pair_shared(const FwdArgs& a, const FwdArgs& b, int precision, int waves, hipStream_t st) {
    if (precision == 64) launch_shared<double>(a, b, waves, st);
    else launch_shared<float>(a, b, waves, st);
    return hipGetLastError();
}

hipError_t launch_forward_pair(const FwdArgs& a, int precision, int waves_per_block, int max_beads, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (a.n_items <= 0 || a.n_steps <= 0) return hipSuccess;
    const int shared = pair_waves(a.n_items, precision, max_beads);
    if (shared > 1) {
        FwdArgs none = a;
        none.n_items = 0;
        return launch_pair_shared(a, none, precision, shared, st);
    }
    const int wpb = waves_per_block;
    dim3 grid((a.n_items + wpb - 1) / wpb), block(WAVE * wpb);
    if (precision == 64) hipLaunchKernelGGL(fwd_pair_kernel<double>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(fwd_pair_kernel<float>, grid, block, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_forward_pair_dual(const FwdArgs& a, const FwdArgs& b, int precision, int waves_per_block,
                                    int max_beads, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    const int wpb = waves_per_block;
    const int ba = (a.n_items + wpb - 1) / wpb, bb = (b.n_items + wpb - 1) / wpb;
    if (ba + bb == 0) return hipSuccess;
    const int shared = pair_waves(a.n_items + b.n_items, precision, max_beads);
    if (shared > 1) return launch_pair_shared(a, b, precision, shared, st);
    dim3 grid((unsigned)(ba + bb)), block(WAVE * wpb);
    if (precision == 64) hipLaunchKernelGGL(fwd_pair_dual_kernel<double>, grid, block, 0, st, a, b, ba);
    else hipLaunchKernelGGL(fwd_pair_dual_kernel<float>, grid, block, 0, st, a, b, ba);
    return hipGetLastError();
}

}  // namespace ra

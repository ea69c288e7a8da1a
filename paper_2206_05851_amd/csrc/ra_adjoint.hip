// ra_adjoint.hip — pathwise adjoint of the fused forward path (FP32 state).
//
// Objective J = sum_{w,j} lam_mu[w][j] * mean_k f_j^{w,k}, where lam_mu is
// dJ/d(replica-mean tension) (Bell-rate cotangents are folded into it first).
// With the noise held fixed, every EM step Q^{n+1} = Phi(Q^n; rate, H, b) is
// a smooth map, and reverse mode runs
//   lambda^n = (dPhi/dQ)^T lambda^{n+1} + dJ/dQ^n (sample injections),
//   dJ/dtheta += lambda^{n+1} . dPhi/dtheta + direct dJ/dtheta at samples.
// The forward stored Q every K steps; each K-step segment is recomputed
// from its checkpoint with the same step function (bitwise-identical
// trajectory) into a per-wavefront HBM buffer, then swept backwards. Many
// wavefronts are bound by that buffer's traffic, so there its rows hold the tile's
// lanes only (4096 replicas of 100 beads, 50 of 64 lanes, 2000 steps, segments of 100:
// 25.2 GB in 4.98 ms with whole rows, 19.7 GB in 4.43 ms). Few are bound by the
// issue of one wavefront, and wide lanes by their registers: their rows are whole,
// at fixed distances from one address (300 replicas of 100 beads, 200 steps, segments
// of 5, noise map 1: packed 183 us, whole 172).
//
// Bond form: Phi_j = Q_j + dt kappa Q_j + cF [G_{j+1} - 2 G_j + G_{j-1}] + noise,
// G_j = g_j Q_j. The Laplacian is symmetric, so
//   (dPhi/dQ)^T lambda at j = lambda_j + (dt kappa)^T lambda_j + cF J_j mu_j,
//   mu_j = lambda_{j+1} - 2 lambda_j + lambda_{j-1},
//   J_j = dG_j/dQ_j = g I + 2 g^2 / Q0^2 Q Q^T (FENE off the guard), g I on it.
#include "ra_chain.hpp"
#include "ra_launch.hpp"

namespace ra {

// g, s and the guard flag by the forward's law and FP64 guard. The forward folds cF into its
// reciprocal (fene_force), so the two round differently by a few ulp / (1 - s), and
// bonds within that of s = 0.9 may take the FP64 branch in one only.
template <bool FENE>
__device__ __forceinline__ void factor_gs(float qx, float qy, float qz, const GroupDev& G, float& g, float& s,
                                          bool& smooth) {
    if constexpr (!FENE) {
        g = 1.0f; s = 0.0f; smooth = false;
        return;
    } else {
        const float q2 = fmadd(qx, qx, fmadd(qy, qy, qz * qz));
        const float sf = q2 * G.inv_q0sq;
        g = fast_rcp(1.0f - sf);
        s = sf;
        smooth = true;
        // wave vote, as in the forward step: the FP64 recomputation runs only
        // in wavefronts where some lane is near full extension
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(sf > FENE_FP64_BAND) != 0, 0)) {
            if (sf > FENE_FP64_BAND) {
                const double dx = qx, dy = qy, dz = qz;
                double sd = (dx * dx + dy * dy + dz * dz) * G.inv_q0sq_d;
                smooth = !(sd > 1.0 - FENE_DELTA);
                if (!smooth) sd = 1.0 - FENE_DELTA;
                g = (float)(1.0 / (1.0 - sd));
                s = (float)sd;
            }
        }
    }
}

// A state as rows of the whole wavefront, [slot][xyz][64].
template <bool STORE, int M>
__device__ __forceinline__ void wave_rows(Lane<float, M>& s, float* p) {
    p += threadIdx.x & (WAVE - 1);
    auto move = [](float& v, float& at) {
        if constexpr (STORE) at = v;
        else v = at;
    };
#pragma unroll
    for (int m = 0; m < M; ++m) {
        move(s.qx[m], p[3 * m * WAVE]);
        move(s.qy[m], p[(3 * m + 1) * WAVE]);
        move(s.qz[m], p[(3 * m + 2) * WAVE]);
    }
}

// dJ/dQ and direct dJ/dtheta of the sampled tension f = H g |Q| at window w.
template <int M, bool FENE>
__device__ __forceinline__ void inject(const Lane<float, M>& q, const bool (&valid)[M], const GroupDev& G,
                                       const AdjArgs& a, const TileGeom& tg, int64_t w, float (&lx)[M],
                                       float (&ly)[M], float (&lz)[M], double& gH, double& gb) {
    const float H = G.H;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const float c = valid[m] ? (float)(a.lam_mu[w * a.spr_total + G.spr_off + tg.j0 + m] / (double)G.R)
                                 : 0.0f;
        float g, s;
        bool smooth;
        factor_gs<FENE>(q.qx[m], q.qy[m], q.qz[m], G, g, s, smooth);
        const float q2 = fmadd(q.qx[m], q.qx[m], fmadd(q.qy[m], q.qy[m], q.qz[m] * q.qz[m]));
        const float len = fast_sqrt(q2);
        // df/dQ = H (g + 2 g^2 s) Q/|Q| off the guard, H g Q/|Q| on it (Hookean: s = 0)
        const float coef = len > 0.0f ? H * (smooth ? fmadd(2.0f * g * g, s, g) : g) / len : 0.0f;
        lx[m] = fmadd(c * coef, q.qx[m], lx[m]);
        ly[m] = fmadd(c * coef, q.qy[m], ly[m]);
        lz[m] = fmadd(c * coef, q.qz[m], lz[m]);
        // df/dH = g |Q| (1 + g s), df/db = -H g^2 (s/b) |Q| off the guard
        const float dH = smooth ? g * len * fmadd(g, s, 1.0f) : g * len;
        const float db = (FENE && smooth) ? -H * g * g * (s / (float)G.b) * len : 0.0f;
        gH += (double)(c * dH);
        gb += (double)(c * db);
    }
}

// FP32 partial sums of at most 128 steps of a reverse sweep, turned into the (rate, H, b) gradient terms by rev_flush:
//   rate: lambda . d(dt kappa Q)/d rate = dt (fx Sxx + fy Syy + fz Szz + fxz Sxz)
//         with (fx, fy, fz, fxz) the flow pattern and S_ab = sum lambda_a Q_b;
//   H:    dtz (S1 + S2), b: -cF S2 / b, with S1 = sum g mu.Q and
//         S2 = sum g^2 s mu.Q (s and the 2/Q0^2 term are 0 on the guard and
//         for Hookean springs).
struct RevSums {
    float sxx, syy, szz, sxz, s1, s2;
};

__device__ __forceinline__ void rev_flush(const RevSums& r, const GroupDev& G, double& gr, double& gH, double& gb) {
    const double dt = G.dt;
    double pr = 0.0;
    if (G.flow == 1) pr = dt * ((double)r.sxx - 0.5 * ((double)r.syy + (double)r.szz));
    else if (G.flow == 2) pr = dt * ((double)r.sxx - (double)r.syy);
    else if (G.flow == 3) pr = dt * (double)r.sxz;
    gr += pr;
    gH += (G.dt / G.zeta) * ((double)r.s1 + (double)r.s2);
    if (G.spring == 1) gb += -(double)G.cF * (double)r.s2 / G.b;
}

// Reverse step through Phi at the state q = Q^n; lambda holds lambda^{n+1}.
// cF is H dt/zeta, 0 on slots that are not a spring of an active replica: their
// lambda starts at 0, gets no injection, and with a zero coefficient on the
// neighbour term stays 0 without a per-step select (their Q is 0, so they add
// nothing to the theta sums either).
template <int M, bool FENE>
__device__ __forceinline__ void reverse_step(const Lane<float, M>& q, const float (&cF)[M], const GroupDev& G,
                                             float (&lx)[M], float (&ly)[M], float (&lz)[M], RevSums& r) {
    const float kx = G.kx, ky = G.ky, kz = G.kz, kxz = G.kxz;
    const float plx = from_prev_lane(lx[M - 1]), ply = from_prev_lane(ly[M - 1]), plz = from_prev_lane(lz[M - 1]);
    const float nlx = from_next_lane(lx[0]), nly = from_next_lane(ly[0]), nlz = from_next_lane(lz[0]);
    float ux[M], uy[M], uz[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const float nx = (m + 1 < M) ? lx[m + 1 < M ? m + 1 : m] : nlx;
        const float ny = (m + 1 < M) ? ly[m + 1 < M ? m + 1 : m] : nly;
        const float nz = (m + 1 < M) ? lz[m + 1 < M ? m + 1 : m] : nlz;
        const float qx = (m > 0) ? lx[m > 0 ? m - 1 : 0] : plx;
        const float qy = (m > 0) ? ly[m > 0 ? m - 1 : 0] : ply;
        const float qz = (m > 0) ? lz[m > 0 ? m - 1 : 0] : plz;
        ux[m] = fmadd(-2.0f, lx[m], nx + qx);
        uy[m] = fmadd(-2.0f, ly[m], ny + qy);
        uz[m] = fmadd(-2.0f, lz[m], nz + qz);
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
        float g, s;
        bool smooth;
        factor_gs<FENE>(q.qx[m], q.qy[m], q.qz[m], G, g, s, smooth);
        const float Qx = q.qx[m], Qy = q.qy[m], Qz = q.qz[m];
        // rate terms with lambda^{n+1}
        r.sxx = fmadd(lx[m], Qx, r.sxx);
        r.syy = fmadd(ly[m], Qy, r.syy);
        r.szz = fmadd(lz[m], Qz, r.szz);
        r.sxz = fmadd(lx[m], Qz, r.sxz);
        const float muQ = fmadd(ux[m], Qx, fmadd(uy[m], Qy, uz[m] * Qz));
        // lambda^n = lambda + (dt kappa)^T lambda + cF J mu with
        // J mu = g mu + (2 g^2 / Q0^2) (Q.mu) Q off the guard, g mu on it
        const float cg = cF[m] * g;
        const float t = g * muQ;
        r.s1 += t;
        float ce = 0.0f;
        if constexpr (FENE) {
            const float ge = g * t;
            r.s2 = fmadd(ge, smooth ? s : 0.0f, r.s2);
            ce = cF[m] * (smooth ? ge * (2.0f * G.inv_q0sq) : 0.0f);
        }
        const float nx = lx[m] + fmadd(kx, lx[m], fmadd(cg, ux[m], ce * Qx));
        const float ny = ly[m] + fmadd(ky, ly[m], fmadd(cg, uy[m], ce * Qy));
        const float nz = lz[m] + fmadd(kz, lz[m], fmadd(kxz, lx[m], fmadd(cg, uz[m], ce * Qz)));
        lx[m] = nx;
        ly[m] = ny;
        lz[m] = nz;
    }
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, WAVE);
    return v;
}

template <int M, bool FENE, int NMAP, bool MANY>
__device__ __forceinline__ void run_adjoint(const AdjArgs& a, const GroupDev& G, int item, int k_first) {
    // kernel arguments into locals (the loops must not address the argument block)
    const int S = a.S, K = a.K;
    const int64_t n_end = a.n_end, ckpt_total = a.ckpt_total;
    const float* const ckpt = ckpt_item<const float, M>((const float*)a.ckpt, G, k_first);
    float* const seg = a.segbuf + a.seg_off[item];
    double* const partial = a.partial + 3 * item;
    const TileGeom tg = tile_geom(G, k_first, M);
    const Rows<M> rows(G);
    Lane<float, M> s;
    bool valid[M];
    float lx[M], ly[M], lz[M];
#pragma unroll
    for (int m = 0; m < M; ++m) lx[m] = ly[m] = lz[m] = 0.0f;
    double gr = 0.0, gH = 0.0, gb = 0.0;      // FP64 totals
    int dummy = 0;
    const RoundKeys keys = round_keys<false>(a.key0, a.key1);
    using Blocks = LaneBlocks<M, NMAP>;
    const LaneCounters<Blocks::value, false> lc = lane_counters<Blocks::value, false>(
        Blocks::first((uint32_t)tg.j0), (uint32_t)tg.k, G.stream, a.key0, a.key1);
    SlotMask<float, M> mask;
    float cF[M];
    auto set_slots = [&]() {
        mask = slot_mask<float, M>(valid);
#pragma unroll
        for (int m = 0; m < M; ++m) cF[m] = valid[m] ? G.cF : 0.0f;
    };
    // Rows of a stored state: of the tile's lanes, or of the whole wavefront, which then
    // sit at fixed distances from one address.
    constexpr bool PACKED = M <= 4 && MANY;
    const int STRIDE = PACKED ? 3 * M * G.P * G.L : 3 * M * WAVE;
    const AdjArgs* ap = &a;                   // for inject(); not touched in the step loops
    auto sampled = [&](const Lane<float, M>& q, int w) {
        double dH = 0.0, db = 0.0;
        inject<M, FENE>(q, valid, G, *ap, tg, w, lx, ly, lz, dH, db);
        gH += dH;
        gb += db;
    };
    // Reverse over the steps hi .. lo: the states Q^lo .. Q^hi at base, base + stride,
    // ..., read by `read`, and s = Q^{hi + 1}; rs: FP32 partials of at most 128 steps.
    // States are read ahead: with one step the loads' latency bounds a sweep of few
    // wavefronts (1000 items of 40-77 beads, 500 kept states: the widest tile's launch
    // 340 us, all of them 269).
    // CUT: between the sampled states and the 128-step sums the loops hold the steps and
    // nothing else. 200 steps, us, both looked for at each step / cut: 100 replicas of 50
    // beads, noise map 1, every state kept 49 / 41, recomputed in segments of 100 88 / 76.
    // Wide lanes take one step per turn, as unrolled steps do not fit the instruction
    // cache: 4 replicas of 1000 beads, every state kept, three steps unrolled 800, one
    // 455, segments of 20 1204 / 980. Two to four beads per lane spill registers in the
    // cut's loops, and many wavefronts hide what the cut saves and lose by its registers
    // (5000 replicas of 50 beads, every state kept: 127, cut 149).
    auto sweep = [&](const float* base, int64_t stride, int lo, int hi, auto read) {
        constexpr bool CUT = (M == 1 && !MANY) || M > 4;
        constexpr int AHEAD = M <= 2 ? 4 : M <= 4 ? 3 : 1;
        Lane<float, M> ring[AHEAD];
        const float* p = base + (hi - lo) * stride;
        int at = hi;
        auto load = [&](Lane<float, M>& q) {          // past the lowest state: that one again, or none
            if (M <= 4 || at >= lo) read(q, p);
            if (M > 4 || at > lo) p -= stride;
            --at;
        };
        RevSums rs{0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (CUT) {                          // ring: Q^n, Q^{n - 1}, ..
#pragma unroll
            for (int d = 0; d < AHEAD; ++d) load(ring[d]);
            int to_sample = (hi + 1) % S, w = (hi + 1) / S - 1;   // steps to the next sampled state, its window
            for (int n = hi; n >= lo;) {
                if (to_sample == 0) {
                    sampled(s, w--);
                    to_sample = S;
                }
                int len = min(min(to_sample, n - lo + 1), (n & 127) + 1);
                to_sample -= len;
                n -= len;
                if constexpr (AHEAD > 1) {
                    for (; len >= AHEAD; len -= AHEAD) {
#pragma unroll
                        for (int d = 0; d < AHEAD; ++d) {
                            reverse_step<M, FENE>(ring[d], cF, G, lx, ly, lz, rs);
                            if (d == AHEAD - 1) s = ring[d];
                            load(ring[d]);
                        }
                    }
                }
                for (; len > 0; --len) {
                    s = ring[0];
#pragma unroll
                    for (int d = 0; d + 1 < AHEAD; ++d) ring[d] = ring[d + 1];
                    load(ring[AHEAD - 1]);
                    reverse_step<M, FENE>(s, cF, G, lx, ly, lz, rs);
                }
                if (((n + 1) & 127) == 0) {
                    rev_flush(rs, G, gr, gH, gb);
                    rs = RevSums{0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                }
            }
        } else {                                      // ring: Q^n, Q^{n - 1}, .. and last Q^{n + 1}
            ring[AHEAD - 1] = s;
#pragma unroll
            for (int d = 0; d < AHEAD - 1; ++d) load(ring[d]);
            // rr = (n + 1) mod S, w = window of state n + 1 when rr == 0
            int rr = (hi + 1) % S, w = (hi + 1) / S - 1;
            for (int n0 = hi; n0 >= lo; n0 -= AHEAD) {
#pragma unroll
                for (int d = 0; d < AHEAD; ++d) {
                    const int n = n0 - d;
                    if (n < lo) break;
                    Lane<float, M>& after = ring[(d + AHEAD - 1) % AHEAD];   // Q^{n+1}
                    if (rr == 0) sampled(after, w--);
                    load(after);
                    reverse_step<M, FENE>(ring[d], cF, G, lx, ly, lz, rs);
                    if ((n & 127) == 0) {
                        rev_flush(rs, G, gr, gH, gb);
                        rs = RevSums{0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                    }
                    rr = rr == 0 ? S - 1 : rr - 1;
                }
            }
        }
        rev_flush(rs, G, gr, gH, gb);
    };
    auto read_ckpt = [&](Lane<float, M>& q, const float* p) {
        if constexpr (M <= 4) rows.load(q, p);
        else load_ckpt<float, M>(q, valid, p, G, tg);
    };
    auto read_seg = [&](Lane<float, M>& q, const float* p) {
        if constexpr (PACKED) rows.load(q, p);
        else wave_rows<false>(q, (float*)p);
    };
    float* wp = seg;                          // next state of the segment
    auto keep = [&]() {
        if constexpr (PACKED) rows.store(s, wp);
        else wave_rows<true>(s, wp);
        wp += STRIDE;
    };
    const int n_seg = (int)((n_end + K - 1) / K);
    if (K == 1 && n_end > 0) {
        // Every state is a checkpoint: no recompute. The state after the last
        // step is rebuilt by one step from the last checkpoint.
        load_ckpt<float, M>(s, valid, ckpt + (n_end - 1) * ckpt_total, G, tg);
        set_slots();
        if constexpr (NMAP == 1) {
            Carry<float, M> cy;
            init_carry<float, M, false>(cy, lc, G, (uint32_t)(n_end - 1), keys);
            em_step_map1<float, M, FENE>(s, cy, lc, G, valid, mask, (uint32_t)(n_end - 1), keys, dummy);
        } else if constexpr (NMAP == 2) {
            em_step_map2<float, M, FENE>(s, lc, G, valid, mask, (uint32_t)(n_end - 1), keys, dummy);
        } else {
            em_step<float, M, FENE>(s, lc, G, valid, mask, (uint32_t)(n_end - 1), keys, dummy);
        }
        sweep(ckpt, ckpt_total, 0, (int)n_end - 1, read_ckpt);
    }
    for (int sgi = (K == 1 && n_end > 0) ? -1 : n_seg - 1; sgi >= 0; --sgi) {
        const int s0 = sgi * K;
        const int s1 = (int)min(n_end, (int64_t)s0 + K);
        load_ckpt<float, M>(s, valid, ckpt + (int64_t)sgi * ckpt_total, G, tg);
        set_slots();
        wp = seg;
        if constexpr (NMAP == 1) {
            Carry<float, M> cy;
            init_carry<float, M, false>(cy, lc, G, (uint32_t)s0, keys);
            int n = s0;
            if constexpr (M <= 2) {
                // aligned groups of four steps as in the forward: the group's
                // three blocks per slot drawn first, each step's transform just
                // before the step (the same normals as the carry gives)
                for (; n < s1 && (n & 3) != 0; ++n) {
                    keep();
                    em_step_map1<float, M, FENE>(s, cy, lc, G, valid, mask, (uint32_t)n, keys, dummy);
                }
                for (; n + 4 <= s1; n += 4) {
                    Words w[3][M];
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const StepWords sw = lc.words((uint32_t)(n + q));
#pragma unroll
                        for (int m = 0; m < M; ++m) w[q][m] = lc.draw(m, sw, keys);
                    }
                    Noise<float, M> e3;
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        Noise<float, M> e;
#pragma unroll
                        for (int m = 0; m < M; ++m) {
                            Polar<float> d;
                            polars4(w[u][m], G.cN, e.x[m], e.y[m], e.z[m], d);
                            if (u == 0) e3.x[m] = d;
                            if (u == 1) e3.y[m] = d;
                            if (u == 2) e3.z[m] = d;
                        }
                        keep();
                        physics_step<float, M, FENE>(s, e, G, valid, mask, dummy);
                    }
                    keep();
                    physics_step<float, M, FENE>(s, e3, G, valid, mask, dummy);
                }
            }
            for (; n < s1; ++n) {
                keep();
                em_step_map1<float, M, FENE>(s, cy, lc, G, valid, mask, (uint32_t)n, keys, dummy);
            }
        } else if constexpr (NMAP == 2) {
            for (int n = s0; n < s1; ++n) {
                keep();
                em_step_map2<float, M, FENE>(s, lc, G, valid, mask, (uint32_t)n, keys, dummy);
            }
        } else {
            for (int n = s0; n < s1; ++n) {
                keep();
                em_step<float, M, FENE>(s, lc, G, valid, mask, (uint32_t)n, keys, dummy);
            }
        }
        sweep(seg, STRIDE, s0, s1 - 1, read_seg);
    }
    gr = wave_sum(gr);
    gH = wave_sum(gH);
    gb = wave_sum(gb);
    if ((threadIdx.x & (WAVE - 1)) == 0) {
        partial[0] = gr;
        partial[1] = gH;
        partial[2] = gb;
    }
}

template <int M, int NMAP, bool MANY>
__device__ __forceinline__ void adjoint_item(const AdjArgs& a, const GroupDev& G, int item, int k_first) {
    if constexpr (M <= 4) {
        // the group's constants as a local value: read through the reference,
        // the recompute loop re-loads them from memory every step
        const GroupDev Gl = G;
        if (Gl.spring == 1) run_adjoint<M, true, NMAP, MANY>(a, Gl, item, k_first);
        else run_adjoint<M, false, NMAP, MANY>(a, Gl, item, k_first);
    } else {   // noise map 1 is not compiled for wider lanes (rejected on the host)
        static_assert(NMAP != 1, "noise map 1 is compiled for 1-4 beads per lane");
        if (G.spring == 1) run_adjoint<M, true, NMAP, MANY>(a, G, item, k_first);
        else run_adjoint<M, false, NMAP, MANY>(a, G, item, k_first);
    }
}

// A contiguous range of the work list (sorted by beads per lane, the most first).
// MAX_M 2 holds the tiles of one and two beads per lane, 4 those of one to four, any
// other MAX_M that width alone, each with a register budget of its own. MANY: the
// segments' rows are packed (adjoint_packed).
template <int MAX_M, int NMAP, bool MANY>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MAX_M <= 2 ? 4 : MAX_M == 8 ? 2 : 1)))
void adjoint_kernel(AdjArgs a, int item_begin, int item_end) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int item = item_begin + (int)blockIdx.x * (int)(blockDim.x >> 6) + wave;
    if (item >= item_end) return;
    const Item it = a.items[item];
    const GroupDev& G = a.groups[it.g];
    if constexpr (MAX_M == 2 || MAX_M == 4) {
        if (G.M == 1) adjoint_item<1, NMAP, MANY>(a, G, item, it.k0);
        else if (G.M == 2) adjoint_item<2, NMAP, MANY>(a, G, item, it.k0);
        else if constexpr (MAX_M == 4) {
            if (G.M == 3) adjoint_item<3, NMAP, MANY>(a, G, item, it.k0);
            else adjoint_item<4, NMAP, MANY>(a, G, item, it.k0);
        }
    } else {
        adjoint_item<MAX_M, NMAP, MANY>(a, G, item, it.k0);
    }
}

// lam_mu[w][s] = grad_mean + grad_rates * dk/dmean, dk/dmean = k * x_dagger / kT.
__global__ __launch_bounds__(64) void lam_mu_kernel(const GroupDev* __restrict__ groups, const double* __restrict__ mean,
                                                    const double* __restrict__ gm, const double* __restrict__ grt,
                                                    double k0, double xd, int64_t spr_total, double* __restrict__ out) {
    const GroupDev& G = groups[blockIdx.x];
    const int64_t w = blockIdx.y;
    for (int j = threadIdx.x; j < G.N - 1; j += WAVE) {
        const int64_t o = w * spr_total + G.spr_off + j;
        double v = gm ? gm[o] : 0.0;
        if (grt) v += grt[o] * k0 * exp(xd * mean[o] / G.kT) * xd / G.kT;
        out[o] = v;
    }
}

// grad[g][p] = sum over the group's work items, one block per group in a
// fixed order: thread t sums items t, t + GR_THREADS, ... in order, then the
// threads' sums combine by a fixed-shape tree.
constexpr int GR_THREADS = 256;

__global__ __launch_bounds__(GR_THREADS) void grad_reduce_kernel(const int32_t* __restrict__ begin_count,
                                                                const double* __restrict__ partial,
                                                                double* __restrict__ grad) {
    __shared__ double sh[3][GR_THREADS];
    const int g = blockIdx.x;
    const int t = threadIdx.x;
    const int b = begin_count[2 * g], n = begin_count[2 * g + 1];
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int i = t; i < n; i += GR_THREADS) {
        const double* q = partial + 3 * (int64_t)(b + i);
        a0 += q[0];
        a1 += q[1];
        a2 += q[2];
    }
    sh[0][t] = a0;
    sh[1][t] = a1;
    sh[2][t] = a2;
    __syncthreads();
    for (int h = GR_THREADS / 2; h >= 1; h >>= 1) {
        if (t < h) {
            sh[0][t] += sh[0][t + h];
            sh[1][t] += sh[1][t + h];
            sh[2][t] += sh[2][t + h];
        }
        __syncthreads();
    }
    if (t < 3) grad[3 * g + t] = sh[t][0];
}

template <int MAX_M, int NMAP>
static void launch_adj(const AdjArgs& a, int item_begin, int item_end, dim3 grid, dim3 block, hipStream_t st) {
    if constexpr (MAX_M <= 4) {
        if (adjoint_packed(MAX_M, a.n_items)) {
            hipLaunchKernelGGL((adjoint_kernel<MAX_M, NMAP, true>), grid, block, 0, st, a, item_begin, item_end);
            return;
        }
    }
    hipLaunchKernelGGL((adjoint_kernel<MAX_M, NMAP, false>), grid, block, 0, st, a, item_begin, item_end);
}

hipError_t launch_adjoint(const AdjArgs& a, int max_m, int item_begin, int item_end, int waves_per_block, int nmap,
                          hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    const int n = item_end - item_begin;
    if (n <= 0) return hipSuccess;
    const int wpb = waves_per_block;
    dim3 grid((n + wpb - 1) / wpb), block(WAVE * wpb);
#define RA_ADJ(M_, NMAP_)                                                 \
    launch_adj<M_, NMAP_>(a, item_begin, item_end, grid, block, st);      \
    break
    if (nmap == 1) {
        switch (max_m) {
        case 1: RA_ADJ(1, 1);
        case 2: RA_ADJ(2, 1);
        case 3:
        case 4: RA_ADJ(4, 1);
        default: return hipErrorInvalidValue;
        }
    } else if (nmap == 2) {   // whole groups of four beads per lane: 8, 12 or 16
        switch (max_m) {
        case 8: RA_ADJ(8, 2);
        case 12: RA_ADJ(12, 2);
        case 16: RA_ADJ(16, 2);
        default: return hipErrorInvalidValue;
        }
    } else {
        switch (max_m) {
        case 1: RA_ADJ(1, 0);
        case 2: RA_ADJ(2, 0);
        case 3:
        case 4: RA_ADJ(4, 0);
        case 6: RA_ADJ(6, 0);
        case 8: RA_ADJ(8, 0);
        case 12: RA_ADJ(12, 0);
        case 16: RA_ADJ(16, 0);
        default: return hipErrorInvalidValue;
        }
    }
#undef RA_ADJ
    return hipGetLastError();
}

hipError_t launch_lam_mu(const GroupDev* groups, int n_groups, int64_t n_windows, const double* mean,
                         const double* grad_mean, const double* grad_rates, double k0, double xd,
                         int64_t spr_total, double* lam_mu, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (n_windows == 0) return hipSuccess;
    hipLaunchKernelGGL(lam_mu_kernel, dim3((unsigned)n_groups, (unsigned)n_windows), dim3(64), 0, st, groups,
                       mean, grad_mean, grad_rates, k0, xd, spr_total, lam_mu);
    return hipGetLastError();
}

hipError_t launch_grad_reduce(const int32_t* item_begin, int n_groups, const double* partial,
                              double* grad_params, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (n_groups == 0) return hipSuccess;
    hipLaunchKernelGGL(grad_reduce_kernel, dim3((unsigned)n_groups), dim3(GR_THREADS), 0, st, item_begin,
                       partial, grad_params);
    return hipGetLastError();
}

}  // namespace ra

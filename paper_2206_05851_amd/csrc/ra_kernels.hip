// ra_kernels.hip — gfx950 kernels of the replica-averaged BD library outside
// the fused step loops: clone, plain path, replica reduction, Bell rates,
// inspection; and the launchers that pick a forward kernel (ra_forward.hpp).
#include "ra_clone.hpp"
#include "ra_chain.hpp"
#include "ra_launch.hpp"

namespace ra {

__global__ void advance_kernel(int64_t* step, int64_t n) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *step += n;
}

// Clears the status word, the per-group guard counters and the device step
// counter: a kernel rather than memset nodes, so a caller may capture the
// clone sequence in a graph.
__global__ void reset_kernel(int32_t* status, unsigned long long* clamps, int n_groups, int64_t* step) {
    const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t == 0) {
        *status = 0;
        *step = 0;
    }
    for (int g = t; g < n_groups; g += (int)(gridDim.x * blockDim.x)) clamps[g] = 0ull;
}

// ---------------------------------------------------------------------------
// Clone (RSF, Sec. II): Q_j = parent_{j+1} - parent_j in FP64, then rounded to
// the state precision, for every replica; the parent is validated here.
// In the same launch the first wavefront of block (0, g) writes group g's clone source,
// and with one group, where no other block needs the status word, block 0 also
// does reset_kernel's work (a launch in a row costs 2-5 us each: a window of 50
// replicas 110.3 -> 108.7 us).
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void clone_kernel(const GroupDev* __restrict__ groups,
                                                    const double* __restrict__ parent,
                                                    const int64_t* __restrict__ par_off, T* __restrict__ state,
                                                    double* __restrict__ tsf_acc, int32_t* status,
                                                    unsigned long long* clamps, int64_t* step,
                                                    double* __restrict__ src) {
    const GroupDev& G = groups[blockIdx.y];
    const int nm1 = G.N - 1;
    const int64_t total = (int64_t)G.R * nm1;
    const double* p = parent + par_off[blockIdx.y];
    if (blockIdx.x == 0) {
        bool bad = false;
        for (int j = threadIdx.x; j < nm1; j += blockDim.x) bad |= !clone_bond(p, j, G).ok;
        bad = __syncthreads_or(bad);
        if (threadIdx.x == 0) {
            if (gridDim.y == 1) {
                *status = bad ? 1 : 0;
                *step = 0;
                *clamps = 0ull;
            } else if (bad) {
                atomicOr(status, 1);
            }
        }
        if (threadIdx.x < WAVE) clone_source(p, src + par_off[blockIdx.y], G.N);
    }
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const CloneBond q = clone_bond(p, (int)(e % nm1), G);
        const int64_t o = G.state_off + e * 3;
        state[o] = (T)q.x;
        state[o + 1] = (T)q.y;
        state[o + 2] = (T)q.z;
        if (tsf_acc) tsf_acc[G.smp_off + e] = 0.0;
    }
}

// Plain path clone: bead positions of every replica = parent.
template <typename T>
__global__ void clone_pos_kernel(const GroupDev* __restrict__ groups, const double* __restrict__ parent,
                                 const int64_t* __restrict__ par_off, T* __restrict__ pos,
                                 double* __restrict__ tsf_acc, int32_t* status) {
    const GroupDev& G = groups[blockIdx.y];
    const int64_t per = (int64_t)G.N * 3;
    const int64_t total = (int64_t)G.R * per;
    const double* p = parent + par_off[blockIdx.y];
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = e % per;
        pos[G.pos_off + e] = (T)p[c];
        if (e < per) {
            bool bad = !__builtin_isfinite(p[c]);
            if (G.spring == 1 && c % 3 == 0 && c + 3 < per) {
                const double qx = p[c + 3] - p[c], qy = p[c + 4] - p[c + 1], qz = p[c + 5] - p[c + 2];
                if (!((qx * qx + qy * qy + qz * qz) * G.inv_q0sq_d < 1.0)) bad = true;
            }
            if (bad) atomicOr(status, 1);
        }
    }
    if (tsf_acc) {
        const int64_t ns = (int64_t)G.R * (G.N - 1);
        for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < ns;
             e += (int64_t)gridDim.x * blockDim.x)
            tsf_acc[G.smp_off + e] = 0.0;
    }
}

// ---------------------------------------------------------------------------
// Plain path: one launch per step per group, bead positions in HBM, one
// thread per (replica, bead), bead form of Eq. (1) with the same counters.
// ---------------------------------------------------------------------------
template <typename T, bool FENE>
__device__ __forceinline__ void bond_force(const T* r0, const T* r1, const GroupDev& G, T& fx, T& fy,
                                           T& fz, int& clamps) {
    const T qx = r1[0] - r0[0], qy = r1[1] - r0[1], qz = r1[2] - r0[2];
    T g = (T)1;
    if constexpr (FENE) {
        const T q2 = fmadd(qx, qx, fmadd(qy, qy, qz * qz));
        g = fene_g(qx, qy, qz, q2, (T)G.inv_q0sq, G.inv_q0sq_d, clamps);
    }
    fx = g * qx;
    fy = g * qy;
    fz = g * qz;
}

template <typename T, bool FENE>
__global__ __launch_bounds__(256) void plain_step_kernel(const GroupDev* __restrict__ groups, int g,
                                                         const T* __restrict__ rin, T* __restrict__ rout,
                                                         const int32_t* status, uint32_t n, uint32_t key0,
                                                         uint32_t key1, unsigned long long* clamp_ctr) {
    const GroupDev& G = groups[g];
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)G.R * G.N) return;
    if (*status & 1) return;
    const int64_t k = e / G.N;
    const int i = (int)(e - k * G.N);
    const T* r = rin + G.pos_off + k * G.N * 3;
    const Co<T> c{G};
    int clamps = 0;
    T fx = 0, fy = 0, fz = 0;
    if (i <= G.N - 2) {
        T ax, ay, az;
        bond_force<T, FENE>(r + 3 * i, r + 3 * (i + 1), G, ax, ay, az, clamps);
        fx += ax; fy += ay; fz += az;
    }
    if (i >= 1) {
        T bx, by, bz;
        int dummy = 0;
        bond_force<T, FENE>(r + 3 * (i - 1), r + 3 * i, G, bx, by, bz, dummy);
        fx -= bx; fy -= by; fz -= bz;
    }
    T ex, ey, ez;
    if (G.nmap == 1 && (n & 3u) == 3u) {   // map 1: fourth normals of steps n-3 .. n-1
        T a_, b_, c_;
        normals4(philox10(n - 3u, (uint32_t)i, (uint32_t)k, G.stream, key0, key1), a_, b_, c_, ex);
        normals4(philox10(n - 2u, (uint32_t)i, (uint32_t)k, G.stream, key0, key1), a_, b_, c_, ey);
        normals4(philox10(n - 1u, (uint32_t)i, (uint32_t)k, G.stream, key0, key1), a_, b_, c_, ez);
    } else if (G.nmap == 2) {              // map 2: normal i mod 4 of the blocks 3 (i / 4) + c
        const uint32_t b = 3u * ((uint32_t)i >> 2);
        const int r = i & 3;
        T v[4];
        normals4(philox10(n, b, (uint32_t)k, G.stream, key0, key1), v[0], v[1], v[2], v[3]);
        ex = r == 0 ? v[0] : r == 1 ? v[1] : r == 2 ? v[2] : v[3];
        normals4(philox10(n, b + 1u, (uint32_t)k, G.stream, key0, key1), v[0], v[1], v[2], v[3]);
        ey = r == 0 ? v[0] : r == 1 ? v[1] : r == 2 ? v[2] : v[3];
        normals4(philox10(n, b + 2u, (uint32_t)k, G.stream, key0, key1), v[0], v[1], v[2], v[3]);
        ez = r == 0 ? v[0] : r == 1 ? v[1] : r == 2 ? v[2] : v[3];
    } else {
        normals3(philox10(n, (uint32_t)i, (uint32_t)k, G.stream, key0, key1), ex, ey, ez);
    }
    const T x = r[3 * i], y = r[3 * i + 1], z = r[3 * i + 2];
    const T ix = fmadd(c.kx(), x, fmadd(c.kxz(), z, fmadd(c.cF(), fx, c.sigma() * ex)));
    const T iy = fmadd(c.ky(), y, fmadd(c.cF(), fy, c.sigma() * ey));
    const T iz = fmadd(c.kz(), z, fmadd(c.cF(), fz, c.sigma() * ez));
    T* o = rout + G.pos_off + k * G.N * 3 + 3 * i;
    o[0] = x + ix;
    o[1] = y + iy;
    o[2] = z + iz;
    if (clamps) atomicAdd(clamp_ctr + g, (unsigned long long)clamps);
}

template <typename T, bool FENE>
__global__ __launch_bounds__(256) void plain_sample_kernel(const GroupDev* __restrict__ groups, int g,
                                                           const T* __restrict__ pos, T* __restrict__ samples,
                                                           T* __restrict__ tsfo, double* __restrict__ tsf_acc,
                                                           int window_end, int S, int32_t* status) {
    const GroupDev& G = groups[g];
    const int nm1 = G.N - 1;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)G.R * nm1) return;
    const int64_t k = e / nm1;
    const int j = (int)(e - k * nm1);
    const T* r = pos + G.pos_off + k * G.N * 3 + 3 * j;
    int dummy = 0;
    T fx, fy, fz;
    bond_force<T, FENE>(r, r + 3, G, fx, fy, fz, dummy);
    const T f = Co<T>{G}.H() * fast_sqrt(fmadd(fx, fx, fmadd(fy, fy, fz * fz)));
    const int64_t o = G.smp_off + e;
    if (tsf_acc) {
        const double acc = tsf_acc[o] + (double)f;
        if (window_end) {
            tsfo[o] = (T)(acc / (double)S);
            tsf_acc[o] = 0.0;
        } else {
            tsf_acc[o] = acc;
        }
    }
    if (window_end) {
        samples[o] = f;
        if (!__builtin_isfinite(f)) atomicOr(status, 2);
    }
}

// ---------------------------------------------------------------------------
// Replica reduction (RSF estimate, Sec. II): per (window, spring) the replica
// mean and the R-1 standard deviation, FP64, two passes, fixed order:
// wave v of RED_WAVES sums replicas [v*c, (v+1)*c) (c = ceil(R/RED_WAVES)) in
// order, the waves' sums combine in wave order. Loads are unrolled so each
// lane keeps several rows in flight; the second pass re-reads the block's
// rows, which are still in L2.
// ---------------------------------------------------------------------------
constexpr int RED_WAVES = 16;

template <typename T>
__global__ __launch_bounds__(WAVE * RED_WAVES) void reduce_kernel(const GroupDev* __restrict__ groups,
                                                               const ColTile* __restrict__ tiles,
                                                               const T* __restrict__ smp, int64_t smp_total,
                                                               int64_t spr_total, double* __restrict__ mean,
                                                               double* __restrict__ stdv,
                                                               const int32_t* __restrict__ nan_if) {
    __shared__ double part[RED_WAVES][WAVE];
    const ColTile tile = tiles[blockIdx.x];
    const int64_t w = blockIdx.y;
    const GroupDev& G = groups[tile.g];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = threadIdx.x >> 6;
    const int nm1 = G.N - 1;
    const int j = tile.j0 + lane;
    const bool ok = j < nm1;
    const int chunk = (G.R + RED_WAVES - 1) / RED_WAVES;
    const int kb = min(G.R, wv * chunk);
    const int ke = min(G.R, kb + chunk);
    const T* base = smp + w * smp_total + G.smp_off + (ok ? j : 0);
    double acc = 0.0;
    if (ok) {
#pragma unroll 8
        for (int k = kb; k < ke; ++k) acc += (double)base[(int64_t)k * nm1];
    }
    part[wv][lane] = acc;
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int v = 0; v < RED_WAVES; ++v) tot += part[v][lane];
    const double mu = tot / (double)G.R;
    __syncthreads();
    double ss = 0.0;
    if (ok) {
#pragma unroll 8
        for (int k = kb; k < ke; ++k) {
            const double d = (double)base[(int64_t)k * nm1] - mu;
            ss = fmadd(d, d, ss);
        }
    }
    part[wv][lane] = ss;
    __syncthreads();
    if (wv == 0 && ok) {
        double sst = 0.0;
#pragma unroll
        for (int v = 0; v < RED_WAVES; ++v) sst += part[v][lane];
        const int64_t o = w * spr_total + G.spr_off + j;
        const bool nan = nan_if && *nan_if != 0;
        if (mean) mean[o] = nan ? __builtin_nan("") : mu;
        if (stdv) stdv[o] = nan ? __builtin_nan("") : G.R > 1 ? sqrt(sst / (double)(G.R - 1)) : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Bell-type rates (Sec. III) and event draws, one wavefront per (group, window).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void bell_kernel(const GroupDev* __restrict__ groups, int n_groups,
                                                  const double* __restrict__ mean, int64_t spr_total,
                                                  double k0, double xd, double* __restrict__ rates,
                                                  double* __restrict__ rate_sum, uint8_t* __restrict__ events,
                                                  int S, uint32_t key0, uint32_t key1) {
    const int g = blockIdx.x;
    const int64_t w = blockIdx.y;
    const GroupDev& G = groups[g];
    const int lane = threadIdx.x;
    double acc = 0.0;
    for (int j = lane; j < G.N - 1; j += WAVE) {
        const int64_t o = w * spr_total + G.spr_off + j;
        const double k = k0 * exp(xd * mean[o] / G.kT);
        if (rates) rates[o] = k;
        acc += k;
        if (events) {
            const Words u = philox10((uint32_t)w, (uint32_t)j, 0u, (2u << 24) | (G.stream & 0xFFFFFFu), key0, key1);
            const double p = -expm1(-k * (double)S * G.dt);
            events[o] = u01_f64_53(u.x, u.y) < p ? 1 : 0;
        }
    }
    // fixed-order butterfly over the 64 lanes
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, WAVE);
    if (lane == 0 && rate_sum) rate_sum[w * n_groups + g] = acc;
}

// ---------------------------------------------------------------------------
// Inspection helpers.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void to_f64_kernel(const T* __restrict__ src, double* __restrict__ dst, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        dst[e] = (double)src[e];
}

template <typename T>
__global__ void pos_to_bonds_kernel(const GroupDev* __restrict__ groups, const T* __restrict__ pos,
                                    double* __restrict__ out) {
    const GroupDev& G = groups[blockIdx.y];
    const int nm1 = G.N - 1;
    const int64_t total = (int64_t)G.R * nm1;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = e / nm1;
        const int j = (int)(e - k * nm1);
        const T* r = pos + G.pos_off + k * G.N * 3 + 3 * j;
        for (int a = 0; a < 3; ++a) out[G.state_off + e * 3 + a] = (double)r[3 + a] - (double)r[a];
    }
}

__global__ void debug_noise_kernel(const uint32_t* __restrict__ ctr, int64_t n, uint32_t key0, uint32_t key1,
                                   uint32_t* __restrict__ words, float* __restrict__ n32,
                                   double* __restrict__ n64) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const Words w = philox10(ctr[4 * e], ctr[4 * e + 1], ctr[4 * e + 2], ctr[4 * e + 3], key0, key1);
    if (words) {
        words[4 * e] = w.x;
        words[4 * e + 1] = w.y;
        words[4 * e + 2] = w.z;
        words[4 * e + 3] = w.w;
    }
    if (n32) {
        float a, b, c;
        normals3(w, a, b, c);
        n32[3 * e] = a;
        n32[3 * e + 1] = b;
        n32[3 * e + 2] = c;
    }
    if (n64) {
        double a, b, c;
        normals3(w, a, b, c);
        n64[3 * e] = a;
        n64[3 * e + 1] = b;
        n64[3 * e + 2] = c;
    }
}

// ---------------------------------------------------------------------------
// Host launchers.
// ---------------------------------------------------------------------------
static dim3 grid1d(int64_t n, int block) {
    int64_t b = (n + block - 1) / block;
    if (b < 1) b = 1;
    if (b > 65535) b = 65535;
    return dim3((unsigned)b);
}

// Whether n_items work items take the split forward (ra_split.hpp): few enough that
// the chip has issue slots left beside one wavefront per item. Measured
// against the one-wavefront kernels, 500 steps, time ratio (above 1: split faster)
// at 256 / 512 / 768 / 1024 / 1536 items: FP32 one bead per lane 1.36 / 1.19 / 1.10 /
// 1.02 / 1.02 (noise map 1: 1.31 / 1.33 / 1.18 / 1.10 / 1.14; at 2048 0.95), two
// 1.58 / 1.35 / 0.95, three and four 1.78 / 1.03 / 0.75 (two workgroups fit a CU beside the
// rings of two beads per lane, one beside those of four); FP64 2.7-3.2 / 1.6-1.7 / 1.1-1.3
// / 0.83-1.02, three and four beads per lane see SplitWaves.
static bool split_forward(int n_items, int precision, int family, int max_m) {
    return family == 4 && n_items <= (precision == 64 ? 768 : max_m == 1 ? 1536 : 512);
}

hipError_t launch_forward(const FwdArgs& a, int precision, int family, int waves_per_block, int max_m, int nmap,
                          hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (split_forward(a.n_items, precision, family, max_m)) {
        launch_forward_split(a, precision, max_m, nmap, st);
        return hipGetLastError();
    }
    const int wpb = waves_per_block;
    dim3 grid((a.n_items + wpb - 1) / wpb), block(WAVE * wpb);
    if (precision == 64) launch_forward_f64(a, nmap, grid, block, st);
    else if (family == 4) launch_forward_lane(a, nmap, grid, block, st);
    else launch_forward_wide(a, nmap, grid, block, st);
    return hipGetLastError();
}

hipError_t launch_forward_dual(const FwdArgs& a, const FwdArgs& b, int precision, int family, int waves_per_block,
                               int max_m, int nmap, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (a.n_items + b.n_items > 0 && split_forward(a.n_items + b.n_items, precision, family, max_m)) {
        launch_forward_split_dual(a, b, precision, max_m, nmap, st);
        return hipGetLastError();
    }
    const int wpb = waves_per_block;
    const int ba = (a.n_items + wpb - 1) / wpb, bb = (b.n_items + wpb - 1) / wpb;
    if (ba + bb == 0) return hipSuccess;
    dim3 grid((unsigned)(ba + bb)), block(WAVE * wpb);
    if (precision == 64) launch_forward_dual_f64(a, b, ba, nmap, grid, block, st);
    else if (family == 4) launch_forward_dual_lane(a, b, ba, nmap, grid, block, st);
    else launch_forward_dual_wide(a, b, ba, nmap, grid, block, st);
    return hipGetLastError();
}

hipError_t launch_advance(int64_t* step, int64_t n, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(64), 0, st, step, n);
    return hipGetLastError();
}

hipError_t launch_reset(int32_t* status, unsigned long long* clamps, int n_groups, int64_t* step, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    hipLaunchKernelGGL(reset_kernel, dim3(1), dim3(256), 0, st, status, clamps, n_groups, step);
    return hipGetLastError();
}

constexpr int64_t INIT_BLOCKS = 4096;

// Fused path: everything that starts a run, in one launch or, with several groups,
// after a reset.
hipError_t launch_init(const GroupDev* groups, int n_groups, int64_t max_elems, const double* parent,
                       const int64_t* par_off, void* state, double* tsf_acc, int32_t* status,
                       unsigned long long* clamps, int64_t* step, double* src, int precision, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (n_groups > 1) {
        const hipError_t e = launch_reset(status, clamps, n_groups, step, st);
        if (e != hipSuccess) return e;
    }
    // one thread per bond of the largest group (max_elems counts its bead coordinates), with
    // many groups a loop over them: 512 groups of 100 replicas of 100 beads, a thread per
    // coordinate 36.9 us, per bond 27.1, with the limit 21.3; 2000 groups 124, 89, 64
    const int64_t most = std::max<int64_t>(8, INIT_BLOCKS / n_groups);
    const int64_t blocks = std::min<int64_t>({(max_elems / 3 + 255) / 256, most, 4096});
    dim3 grid((unsigned)std::max<int64_t>(1, blocks), (unsigned)n_groups), block(256);
    if (precision == 64)
        hipLaunchKernelGGL(clone_kernel<double>, grid, block, 0, st, groups, parent, par_off, (double*)state, tsf_acc,
                           status, clamps, step, src);
    else
        hipLaunchKernelGGL(clone_kernel<float>, grid, block, 0, st, groups, parent, par_off, (float*)state, tsf_acc,
                           status, clamps, step, src);
    return hipGetLastError();
}

hipError_t launch_clone_plain(const GroupDev* groups, int n_groups, int64_t max_elems, const double* parent,
                              const int64_t* par_off, void* pos, double* tsf_acc, int32_t* status, int precision,
                              hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    dim3 grid((unsigned)std::min<int64_t>((max_elems + 255) / 256, 4096), (unsigned)n_groups), block(256);
    if (precision == 64)
        hipLaunchKernelGGL(clone_pos_kernel<double>, grid, block, 0, st, groups, parent, par_off, (double*)pos,
                           tsf_acc, status);
    else
        hipLaunchKernelGGL(clone_pos_kernel<float>, grid, block, 0, st, groups, parent, par_off, (float*)pos, tsf_acc,
                           status);
    return hipGetLastError();
}

hipError_t launch_plain_step(const GroupDev* groups, int g, int64_t n_threads, bool fene, const void* rin,
                             void* rout, const int32_t* status, uint32_t n, uint32_t key0, uint32_t key1,
                             unsigned long long* clamps, int precision, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    dim3 grid((unsigned)((n_threads + 255) / 256)), block(256);
    if (precision == 64) {
        if (fene) hipLaunchKernelGGL((plain_step_kernel<double, true>), grid, block, 0, st, groups, g,
                                     (const double*)rin, (double*)rout, status, n, key0, key1, clamps);
        else hipLaunchKernelGGL((plain_step_kernel<double, false>), grid, block, 0, st, groups, g,
                                (const double*)rin, (double*)rout, status, n, key0, key1, clamps);
    } else {
        if (fene) hipLaunchKernelGGL((plain_step_kernel<float, true>), grid, block, 0, st, groups, g,
                                     (const float*)rin, (float*)rout, status, n, key0, key1, clamps);
        else hipLaunchKernelGGL((plain_step_kernel<float, false>), grid, block, 0, st, groups, g,
                                (const float*)rin, (float*)rout, status, n, key0, key1, clamps);
    }
    return hipGetLastError();
}

hipError_t launch_plain_sample(const GroupDev* groups, int g, int64_t n_threads, bool fene, const void* pos,
                               void* samples_w, void* tsf_w, double* tsf_acc, int window_end, int S,
                               int32_t* status, int precision, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    dim3 grid((unsigned)((n_threads + 255) / 256)), block(256);
    if (precision == 64) {
        if (fene) hipLaunchKernelGGL((plain_sample_kernel<double, true>), grid, block, 0, st, groups, g,
                                     (const double*)pos, (double*)samples_w, (double*)tsf_w, tsf_acc,
                                     window_end, S, status);
        else hipLaunchKernelGGL((plain_sample_kernel<double, false>), grid, block, 0, st, groups, g,
                                (const double*)pos, (double*)samples_w, (double*)tsf_w, tsf_acc,
                                window_end, S, status);
    } else {
        if (fene) hipLaunchKernelGGL((plain_sample_kernel<float, true>), grid, block, 0, st, groups, g,
                                     (const float*)pos, (float*)samples_w, (float*)tsf_w, tsf_acc,
                                     window_end, S, status);
        else hipLaunchKernelGGL((plain_sample_kernel<float, false>), grid, block, 0, st, groups, g,
                                (const float*)pos, (float*)samples_w, (float*)tsf_w, tsf_acc,
                                window_end, S, status);
    }
    return hipGetLastError();
}

hipError_t launch_reduce(const GroupDev* groups, const ColTile* tiles, int n_tiles, int64_t n_windows,
                         const void* smp, int64_t smp_total, int64_t spr_total, double* mean, double* stdv,
                         int precision, const int32_t* nan_if, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (n_tiles == 0 || n_windows == 0) return hipSuccess;
    dim3 grid((unsigned)n_tiles, (unsigned)n_windows), block(WAVE * RED_WAVES);
    if (precision == 64)
        hipLaunchKernelGGL(reduce_kernel<double>, grid, block, 0, st, groups, tiles, (const double*)smp,
                           smp_total, spr_total, mean, stdv, nan_if);
    else
        hipLaunchKernelGGL(reduce_kernel<float>, grid, block, 0, st, groups, tiles, (const float*)smp,
                           smp_total, spr_total, mean, stdv, nan_if);
    return hipGetLastError();
}

hipError_t launch_bell(const GroupDev* groups, int n_groups, int64_t n_windows, const double* mean,
                       int64_t spr_total, double k0, double xd, double* rates, double* rate_sum,
                       uint8_t* events, int S, uint32_t key0, uint32_t key1, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (n_windows == 0) return hipSuccess;
    dim3 grid((unsigned)n_groups, (unsigned)n_windows), block(64);
    hipLaunchKernelGGL(bell_kernel, grid, block, 0, st, groups, n_groups, mean, spr_total, k0, xd, rates,
                       rate_sum, events, S, key0, key1);
    return hipGetLastError();
}

hipError_t launch_to_f64(const void* src, double* dst, int64_t n, int precision, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (n == 0) return hipSuccess;
    if (precision == 64)
        hipLaunchKernelGGL(to_f64_kernel<double>, grid1d(n, 256), dim3(256), 0, st, (const double*)src, dst, n);
    else
        hipLaunchKernelGGL(to_f64_kernel<float>, grid1d(n, 256), dim3(256), 0, st, (const float*)src, dst, n);
    return hipGetLastError();
}

hipError_t launch_pos_to_bonds(const GroupDev* groups, int n_groups, int64_t max_elems, const void* pos,
                               double* out, int precision, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    dim3 grid((unsigned)std::min<int64_t>((max_elems + 255) / 256, 4096), (unsigned)n_groups), block(256);
    if (precision == 64)
        hipLaunchKernelGGL(pos_to_bonds_kernel<double>, grid, block, 0, st, groups, (const double*)pos, out);
    else
        hipLaunchKernelGGL(pos_to_bonds_kernel<float>, grid, block, 0, st, groups, (const float*)pos, out);
    return hipGetLastError();
}

hipError_t launch_debug_noise(const uint32_t* ctr, int64_t n, uint32_t key0, uint32_t key1, uint32_t* words,
                              float* n32, double* n64, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(debug_noise_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, ctr, n, key0,
                       key1, words, n32, n64);
    return hipGetLastError();
}

}  // namespace ra

// ra_rsf.hip — device work of the RSF sampling cycle and of the estimators
// built on it:
//   - re-clone (Sec. II): every replica restarts from the current state of a
//     parent chain that runs its own trajectory in another context;
//   - the centre-of-mass-frame conformation each replica set was cloned from;
//   - the spread sigma(N_R) of the RSF estimate over blocks of N_R replicas
//     (Figs. 2 and 5);
//   - the mean first-passage time to any event of a chain (MFTU, Sec. III),
//     from the mean total rate and by sampling unfolding events;
//   - replica fidelity D-bar (Eq. 5) and radius-of-gyration components
//     (R_Gz, Sec. IV).
// None of these is on the per-step path; they run once per window or per
// analysis call, with fixed summation orders so results are reproducible.
#include "ra_clone.hpp"
#include "ra_device.hpp"
#include "ra_launch.hpp"

namespace ra {

// ---------------------------------------------------------------------------
// Wave helpers (FP64): fixed-shape butterfly sum and an inclusive Hillis-Steele
// scan over the 64 lanes.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_incl_scan_d(double v, int lane) {
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const double u = __shfl_up(v, off, WAVE);
        if (lane >= off) v += u;
    }
    return v;
}

// Lane l of a wave owns beads [l*c, min(N, (l+1)*c)), c = ceil(N/64), and the
// bonds with the same indices (bond m joins beads m and m+1). base = position
// of the lane's first bead relative to bead 0: the exclusive scan of the
// lanes' bond sums.
template <typename T>
struct ChainScan {
    const T* q;          // bonds [N-1][3]
    int N, c, i0, i1;
    double bx, by, bz;   // position of bead i0

    __device__ ChainScan(const T* bonds, int n, int lane) : q(bonds), N(n) {
        c = (N + WAVE - 1) / WAVE;
        i0 = min(N, lane * c);
        i1 = min(N, i0 + c);
        double tx = 0.0, ty = 0.0, tz = 0.0;
        for (int m = i0; m < min(i1, N - 1); ++m) {
            tx += (double)q[3 * m];
            ty += (double)q[3 * m + 1];
            tz += (double)q[3 * m + 2];
        }
        bx = wave_incl_scan_d(tx, lane) - tx;
        by = wave_incl_scan_d(ty, lane) - ty;
        bz = wave_incl_scan_d(tz, lane) - tz;
    }
};

// Centre-of-mass-frame positions of a chain given by its bonds, written to
// out[N][3] (FP64). One wave.
template <typename T>
__device__ void com_frame_from_bonds(const T* bonds, int N, double* out, int lane) {
    ChainScan<T> cs(bonds, N, lane);
    double x = cs.bx, y = cs.by, z = cs.bz, sx = 0.0, sy = 0.0, sz = 0.0;
    for (int i = cs.i0; i < cs.i1; ++i) {
        sx += x; sy += y; sz += z;
        if (i < N - 1) { x += (double)bonds[3 * i]; y += (double)bonds[3 * i + 1]; z += (double)bonds[3 * i + 2]; }
    }
    const double cx = wave_sum_d(sx) / N, cy = wave_sum_d(sy) / N, cz = wave_sum_d(sz) / N;
    x = cs.bx; y = cs.by; z = cs.bz;
    for (int i = cs.i0; i < cs.i1; ++i) {
        out[3 * i] = x - cx;
        out[3 * i + 1] = y - cy;
        out[3 * i + 2] = z - cz;
        if (i < N - 1) { x += (double)bonds[3 * i]; y += (double)bonds[3 * i + 1]; z += (double)bonds[3 * i + 2]; }
    }
}

// ---------------------------------------------------------------------------
// Re-clone: state of every replica of group g := replica 0 of the parent
// context's group g. A FENE bond at or past full extension (or non-finite)
// marks the parent invalid (status bit 1), as at the first clone. In the same
// launch: the first wave of block (0, g) writes group g's clone source (the
// parent's beads in its centre-of-mass frame, for Eq. 5), and one thread sets
// the replicas' device step counter to the window start and adds parent_steps, those
// of the launch before that has left it to this one, to the parent's (a window of
// 1000 replicas for 750 steps: 160.4 -> 158.6 us with the launch of its own gone).
// ---------------------------------------------------------------------------
template <typename T>
__global__ void reclone_kernel(const GroupDev* __restrict__ groups, const GroupDev* __restrict__ pgroups,
                               const T* __restrict__ pstate, T* __restrict__ state,
                               double* __restrict__ tsf_acc, int32_t* status, const int64_t* __restrict__ par_off,
                               double* __restrict__ src, int64_t* step, int64_t step_value, int64_t* parent_step,
                               int64_t parent_steps) {
    const GroupDev& G = groups[blockIdx.y];
    const GroupDev& PG = pgroups[blockIdx.y];
    const int nm1 = G.N - 1;
    const int64_t total = (int64_t)G.R * nm1;
    const T* p = pstate + PG.state_off;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = e / nm1;
        const int j = (int)(e - k * nm1);
        const T qx = p[3 * j], qy = p[3 * j + 1], qz = p[3 * j + 2];
        if (k == 0) {
            const double x = qx, y = qy, z = qz;
            bool bad = !(__builtin_isfinite(x) && __builtin_isfinite(y) && __builtin_isfinite(z));
            if (G.spring == 1 && !((x * x + y * y + z * z) * G.inv_q0sq_d < 1.0)) bad = true;
            if (bad) atomicOr(status, 1);
        }
        const int64_t o = G.state_off + e * 3;
        state[o] = qx;
        state[o + 1] = qy;
        state[o + 2] = qz;
        if (tsf_acc) tsf_acc[G.smp_off + e] = 0.0;
    }
    if (blockIdx.x == 0 && threadIdx.x < WAVE)
        com_frame_from_bonds<T>(p, G.N, src + par_off[blockIdx.y], (int)threadIdx.x);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        step[0] = step_value;
        if (parent_steps > 0) parent_step[0] += parent_steps;
    }
}

// ---------------------------------------------------------------------------
// Replica fidelity (Eq. 5) and radius of gyration, one wave per replica.
// rep_off[g] = first replica of group g in the outputs (n_groups + 1 entries).
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void conformation_kernel(const GroupDev* __restrict__ groups, int n_groups,
                                                           const int64_t* __restrict__ rep_off,
                                                           const T* __restrict__ state,
                                                           const int64_t* __restrict__ par_off,
                                                           const double* __restrict__ src,
                                                           double* __restrict__ dbar, double* __restrict__ d_bead,
                                                           double* __restrict__ rg2) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t q = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (q >= rep_off[n_groups]) return;
    int lo = 0, hi = n_groups - 1;   // group with rep_off[g] <= q < rep_off[g + 1]
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (rep_off[mid] <= q) lo = mid;
        else hi = mid - 1;
    }
    const int g = lo;
    const GroupDev& G = groups[g];
    const int64_t k = q - rep_off[g];
    const int N = G.N;
    const T* bonds = state + G.state_off + k * (int64_t)(N - 1) * 3;
    const double* s = src + par_off[g];
    ChainScan<T> cs(bonds, N, lane);
    double x = cs.bx, y = cs.by, z = cs.bz, sx = 0.0, sy = 0.0, sz = 0.0;
    for (int i = cs.i0; i < cs.i1; ++i) {
        sx += x; sy += y; sz += z;
        if (i < N - 1) { x += (double)bonds[3 * i]; y += (double)bonds[3 * i + 1]; z += (double)bonds[3 * i + 2]; }
    }
    const double cx = wave_sum_d(sx) / N, cy = wave_sum_d(sy) / N, cz = wave_sum_d(sz) / N;
    double dx = 0.0, dy = 0.0, dz = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
    double* db = d_bead ? d_bead + (G.pos_off / 3 + k * N) * 3 : nullptr;
    x = cs.bx; y = cs.by; z = cs.bz;
    for (int i = cs.i0; i < cs.i1; ++i) {
        const double hx = x - cx, hy = y - cy, hz = z - cz;
        const double ex = fabs(hx - s[3 * i]), ey = fabs(hy - s[3 * i + 1]), ez = fabs(hz - s[3 * i + 2]);
        dx += ex; dy += ey; dz += ez;
        gx += hx * hx; gy += hy * hy; gz += hz * hz;
        if (db) { db[3 * i] = ex; db[3 * i + 1] = ey; db[3 * i + 2] = ez; }
        if (i < N - 1) { x += (double)bonds[3 * i]; y += (double)bonds[3 * i + 1]; z += (double)bonds[3 * i + 2]; }
    }
    dx = wave_sum_d(dx); dy = wave_sum_d(dy); dz = wave_sum_d(dz);
    gx = wave_sum_d(gx); gy = wave_sum_d(gy); gz = wave_sum_d(gz);
    const int64_t o = (rep_off[g] + k) * 3;
    if (lane == 0) {
        if (dbar) { dbar[o] = dx / N; dbar[o + 1] = dy / N; dbar[o + 2] = dz / N; }
        if (rg2) { rg2[o] = gx / N; rg2[o + 1] = gy / N; rg2[o + 2] = gz / N; }
    }
}

// Radius-of-gyration components of each group's clone source.
__global__ __launch_bounds__(64) void src_rg2_kernel(const GroupDev* __restrict__ groups,
                                                     const int64_t* __restrict__ par_off,
                                                     const double* __restrict__ src, double* __restrict__ out) {
    const GroupDev& G = groups[blockIdx.x];
    const double* s = src + par_off[blockIdx.x];
    double gx = 0.0, gy = 0.0, gz = 0.0;
    for (int i = threadIdx.x; i < G.N; i += WAVE) {
        gx += s[3 * i] * s[3 * i];
        gy += s[3 * i + 1] * s[3 * i + 1];
        gz += s[3 * i + 2] * s[3 * i + 2];
    }
    gx = wave_sum_d(gx); gy = wave_sum_d(gy); gz = wave_sum_d(gz);
    if (threadIdx.x == 0) {
        out[3 * blockIdx.x] = gx / G.N;
        out[3 * blockIdx.x + 1] = gy / G.N;
        out[3 * blockIdx.x + 2] = gz / G.N;
    }
}

// ---------------------------------------------------------------------------
// sigma(N_R): per (window, spring), B = floor(R/block) consecutive blocks;
// each block's mean tension is one RSF estimate; sigma = their standard
// deviation (B - 1). Wave v of 16 takes a contiguous sixteenth of the blocks
// in order; the sixteenths combine in order; two passes (mean, then deviations).
// ---------------------------------------------------------------------------
constexpr int BSIG_WAVES = 16;

template <typename T>
__global__ __launch_bounds__(1024) void block_sigma_kernel(const GroupDev* __restrict__ groups,
                                                           const ColTile* __restrict__ tiles,
                                                           const T* __restrict__ smp, int64_t smp_total,
                                                           int64_t spr_total, int block,
                                                           double* __restrict__ sigma) {
    constexpr int NW = BSIG_WAVES;
    __shared__ double part[NW][WAVE];
    const ColTile tile = tiles[blockIdx.x];
    const int64_t w = blockIdx.y;
    const GroupDev& G = groups[tile.g];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = threadIdx.x >> 6;
    const int nm1 = G.N - 1;
    const int j = tile.j0 + lane;
    const bool ok = j < nm1;
    const int B = G.R / block;
    const int cb = (B + NW - 1) / NW;
    const int b0 = min(B, wv * cb), b1 = min(B, b0 + cb);
    const T* base = smp + w * smp_total + G.smp_off + (ok ? j : 0);
    auto block_mean = [&](int b) {
        double m = 0.0;
#pragma unroll 8   // loads in flight (1000 replicas, 20 windows, blocks of 10-50: 20 -> 13 us)
        for (int q = 0; q < block; ++q) m += (double)base[(int64_t)(b * block + q) * nm1];
        return m / block;
    };
    auto combine = [&]() {   // the wavefronts' partials in wavefront order
        double t = 0.0;
#pragma unroll
        for (int v = 0; v < NW; ++v) t += part[v][lane];
        return t;
    };
    double acc = 0.0;
    if (ok)
        for (int b = b0; b < b1; ++b) acc += block_mean(b);
    part[wv][lane] = acc;
    __syncthreads();
    const double mu = B > 0 ? combine() / B : 0.0;
    __syncthreads();
    double ss = 0.0;
    if (ok)
        for (int b = b0; b < b1; ++b) {
            const double e = block_mean(b) - mu;
            ss = fma(e, e, ss);
        }
    part[wv][lane] = ss;
    __syncthreads();
    if (wv == 0 && ok) {
        const double tot = combine();
        sigma[w * spr_total + G.spr_off + j] = B > 1 ? sqrt(tot / (double)(B - 1)) : 0.0;
    }
}

// mftu[g] = 1 / (mean over windows of rate_sum[w][g]); one wave per group.
__global__ __launch_bounds__(64) void mftu_kernel(const double* __restrict__ rate_sum, int64_t n_windows,
                                                  int n_groups, double* __restrict__ mftu) {
    const int g = blockIdx.x;
    double acc = 0.0;
    for (int64_t w = threadIdx.x; w < n_windows; w += WAVE) acc += rate_sum[w * n_groups + g];
    acc = wave_sum_d(acc);
    if (threadIdx.x == 0) mftu[g] = 1.0 / (acc / (double)n_windows);
}

// MFTU by sampling unfolding events. Window v carries the rates of sampled
// window v mod n_windows, and spring j unfolds there when the tag-2 53-bit
// uniform of counter (v, j, trial, 2<<24 | stream) is below 1 - exp(-k S dt)
// (trial 0 over the sampled windows draws exactly ra_bell_rates's events).
// The first window with any unfolding, or -1 after max_windows, is the trial's
// first passage.
//
// The uniform is u = (2m + 1) 2^-53 with m the top 52 bits of its two words,
// so u < p holds exactly when m is below the count of such m, ceil((p 2^53 - 1) / 2)
// (0 when p 2^53 <= 1, 2^52 when p >= 1): p 2^53 is exact, and for
// 1 < p 2^53 < 2^53 so are the subtraction and the halving. The per-draw test is
// one 64-bit integer compare against a threshold computed once per (window,
// spring) from the same FP64 expression.
__device__ __forceinline__ uint64_t event_threshold(double p) {
    const double x = p * 0x1p53;
    if (!(x > 1.0)) return 0;   // no m, also for NaN
    if (x >= 0x1p53) return (uint64_t)1 << 52;
    return (uint64_t)ceil((x - 1.0) * 0.5);
}

// Thresholds in LDS, in three launches (two with one group):
//  1. first_event_head_kernel: the first EVENT_HEAD windows of every trial, a few
//     trials to a workgroup and no queue: short trials end here;
//  2. event_live_kernel: the trials of each group that have an event, into its queue;
//  3. first_event_queue_kernel: the rest. The windows of a trial are cut into segments,
//     and workgroups take (segment, trial) tickets from a group's queue, segment-major,
//     so that all live trials advance together and the last ones are shared by the whole
//     chip (trials last exponentially long: with one workgroup per trial the longest of
//     1024 kept a few SIMDs busy for most of the call). A workgroup stays with a
//     group until its queue is done and goes on to the next live one: rates are
//     exponential in the tension, so one group of many can hold nearly all the work.
// A ticket whose trial already has an event in an earlier window is dead. Tickets
// come in segment order, so once every trial has an event all further tickets are dead
// and the group is done (an event counted by then came from an earlier ticket). A claim
// is an atomic on one address that the chip takes in turn, about 50 ns each, so it
// takes enough tickets that one of them is live on average, more live ones where
// they outnumber the workgroups, and more of few springs. first[] holds the
// least window found so far (atomicMin: the result does not depend on the order).
// Measured, us, with one workgroup per trial / with a queue of single tickets and a fixed
// share of the workgroups per group / now, trials of 49 springs unless said:
//   512 groups, 128 trials, one group of mean 1e5 windows, others 100  3450 / 53000 / 2450
//   64 groups, 1024 trials, means over three decades                   52300 / 86300 / 39200
//   1024 trials, mean 300 windows                                      85 / 227 / 76
//   8192 trials of one spring, mean 3e4                                922 / 7160 / 940
//   8192 trials of nine springs, mean 1e6                              105000 / 125000 / 91000
//
// A thread draws all springs of its windows. Of the Philox block only
// the first word is computed: m < t needs word 0 = m >> 20 <= (t - 1) >> 20, which
// a draw meets about as rarely as it unfolds (1e-7 here); a wavefront where some
// lane meets it recomputes the block and compares all 52 bits. With the spring
// and the trial uniform, rounds 1-3 cost four VALU instructions: what depends
// on the window alone is computed once per window, what depends on the spring
// alone once per spring for all windows.
// Bound by VALU issue: 34.5 instructions per draw. 1024 trials of up to 2^20
// windows of 49 springs, 1.06e10 draws: 38.8 ms with a workgroup per trial and
// whole blocks, 9.35 ms now.
constexpr int EVENT_THREADS = 256;
constexpr int EVENT_HEAD = 16 * EVENT_THREADS;     // windows of the first launch
constexpr int EVENT_WPT = 2;                       // windows per thread and round of the queue kernel
constexpr int EVENT_ROUND = EVENT_THREADS * EVENT_WPT;
constexpr int EVENT_MOST_ROUNDS = 4;               // most rounds of a ticket
constexpr int EVENT_MOST_LIVE = 8;                 // most live tickets of a claim, on average
constexpr int EVENT_SHARE = 16;                    // workgroups per live trial at most
constexpr int EVENT_CLAIM_DRAWS = 256;             // least spring-rounds of a claim
constexpr size_t EVENT_LDS_MAX = 32 << 10;   // table of 64-bit thresholds up to this size, else the kernel below
constexpr unsigned long long EVENT_NONE = ~0ull;   // no event found
constexpr uint32_t EVENT_NEVER = 0x80000000u;      // the threshold 0: no draw unfolds
constexpr int EVENT_BLOCKS = 2048;                 // workgroups of a launch: 8 on each of 256 CUs

// The queue of group g is one word, the trials that have an event above the next
// ticket (tickets stay below 2^39: 2^23 segments of 2^16 trials). It lies in the
// caller's mftu[g], which the result overwrites: calls that overlap on one context
// (host threads, replays of captured calls) share nothing.
constexpr int EVENT_SHIFT = 44;
constexpr unsigned long long EVENT_TICKETS = (1ull << EVENT_SHIFT) - 1;

// What of the block (v, j, trial, ctr3) depends on the window v alone.
struct EventWindow {
    uint32_t a, b, c, d;   // lo(p0), lo(p1) ^ k0[2], hi and lo(p2): the window's products of rounds 1-3
};

__device__ __forceinline__ EventWindow event_window(uint32_t v, uint32_t trial, uint32_t ctr3, const RoundKeys& k) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * v, q1 = (uint64_t)0xCD9E8D57u * trial;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ ctr3 ^ k.k1[0];           // round 1
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * n2;                      // round 2
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ (uint32_t)q1 ^ k.k0[1];
    const uint64_t p2 = (uint64_t)0xD2511F53u * n0;                      // round 3
    return EventWindow{(uint32_t)p0, (uint32_t)p1 ^ k.k0[2], (uint32_t)(p2 >> 32), (uint32_t)p2};
}

// Word 0 of the block: sa = hi(M0 n0) ^ k1[1] and sb = lo(M0 n0) ^ k1[2] of the
// spring, with n0 = hi(M1 trial) ^ j ^ k0[0] its first word after round 1.
__device__ __forceinline__ uint32_t event_word0(const EventWindow& w, uint32_t sa, uint32_t sb, const RoundKeys& k) {
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (w.a ^ sa);              // rounds 2 and 3
    uint32_t c0 = (uint32_t)(p1 >> 32) ^ w.b, c1 = (uint32_t)p1, c2 = w.c ^ sb, c3 = w.d;
#pragma unroll
    for (int r = 3; r < 10; ++r) {
        const uint64_t a = (uint64_t)0xD2511F53u * c0, b = (uint64_t)0xCD9E8D57u * c2;
        c0 = xor3((uint32_t)(b >> 32), c1, k.k0[r]);
        c2 = xor3((uint32_t)(a >> 32), c3, k.k1[r]);
        c1 = (uint32_t)b;
        c3 = (uint32_t)a;
    }
    return c0;
}

struct EventArgs {
    const GroupDev* groups;
    const double* rates;
    int64_t n_windows, spr_total, max_windows;
    int n_groups, n_trials, S;
    uint32_t key0, key1;
    unsigned long long* first;   // [n_trials][n_groups]
    unsigned long long* queue;   // [n_groups]
};

// One group's thresholds, [2][n_windows][N - 1] in LDS: upper 32 and lower 20 bits of
// t - 1, and the scan of a trial's windows against them.
struct EventTable {
    uint32_t* thr;
    int nm1, n_thr;
    uint32_t nw, ctr3, key0, key1;

    __device__ EventTable(const EventArgs& a, int g, uint32_t* lds) : thr(lds) {
        const GroupDev& G = a.groups[g];
        nm1 = G.N - 1;
        n_thr = (int)a.n_windows * nm1;
        nw = (uint32_t)a.n_windows;
        ctr3 = (2u << 24) | (G.stream & 0xFFFFFFu);
        key0 = a.key0;
        key1 = a.key1;
        const double window_time = (double)a.S * G.dt;
        for (int i = threadIdx.x; i < n_thr; i += EVENT_THREADS) {
            const int w = i / nm1, j = i - w * nm1;
            const double k = a.rates[w * a.spr_total + G.spr_off + j];
            const uint64_t t = event_threshold(-expm1(-k * window_time));
            thr[i] = t ? (uint32_t)((t - 1) >> 20) : 0u;
            thr[n_thr + i] = t ? (uint32_t)(t - 1) & 0xFFFFFu : EVENT_NEVER;
        }
    }

    // Least window with an unfolding among this thread's of the round at `base`: base
    // + thread + 256 q; EVENT_NONE without one.
    template <int WPT>
    __device__ __forceinline__ unsigned long long scan(int64_t base, uint32_t trial, int64_t max_windows,
                                                       const RoundKeys& keys) const {
        EventWindow win[WPT];
        int row[WPT];
#pragma unroll
        for (int q = 0; q < WPT; ++q) {
            const uint32_t v = (uint32_t)(base + q * EVENT_THREADS + threadIdx.x);
            win[q] = event_window(v, trial, ctr3, keys);
            row[q] = (int)(v % nw) * nm1;
        }
        const uint32_t n0_trial = (uint32_t)(((uint64_t)0xCD9E8D57u * trial) >> 32) ^ key0;
        unsigned long long hit = EVENT_NONE;
        for (int j = 0; j < nm1; ++j) {
            const uint64_t p = (uint64_t)0xD2511F53u * (n0_trial ^ (uint32_t)j);
            const uint32_t sa = (uint32_t)(p >> 32) ^ (key1 + 0xBB67AE85u);
            const uint32_t sb = (uint32_t)p ^ (key1 + 2u * 0xBB67AE85u);
#pragma unroll
            for (int q = 0; q < WPT; ++q) {
                const uint32_t x = event_word0(win[q], sa, sb, keys);
                const bool near = x <= thr[row[q] + j];
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(near) != 0, 0)) {
                    const int64_t v = base + q * EVENT_THREADS + threadIdx.x;
                    const Words u = philox10((uint32_t)v, (uint32_t)j, trial, ctr3, keys);
                    const uint64_t m = ((uint64_t)u.x << 20) | (uint64_t)(u.y >> 12);
                    const uint32_t lo = thr[n_thr + row[q] + j];
                    const uint64_t last = ((uint64_t)thr[row[q] + j] << 20) | lo;
                    if (lo != EVENT_NEVER && m <= last && v < max_windows) hit = min(hit, (unsigned long long)v);
                }
            }
        }
        return hit;
    }
};

__global__ __launch_bounds__(EVENT_THREADS) void first_event_head_kernel(EventArgs a, int trials_per_block) {
    extern __shared__ uint32_t event_thr[];
    __shared__ unsigned long long best;
    const int g = blockIdx.y;
    const EventTable tab(a, g, event_thr);
    const RoundKeys keys = round_keys(a.key0, a.key1);
    const int64_t head = min((int64_t)EVENT_HEAD, a.max_windows);
    const int t0 = (int)blockIdx.x * trials_per_block, t1 = min(a.n_trials, t0 + trials_per_block);
    for (int trial = t0; trial < t1; ++trial) {
        if (threadIdx.x == 0) best = EVENT_NONE;
        __syncthreads();   // and, the first time, the table is written
        for (int64_t base = 0; base < head; base += EVENT_THREADS) {
            const unsigned long long hit = tab.scan<1>(base, (uint32_t)trial, a.max_windows, keys);
            if (hit != EVENT_NONE)
                __hip_atomic_fetch_min(&best, hit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __syncthreads();
            // the same answer in every wavefront: one that is ahead adds later windows only
            if (__hip_atomic_load(&best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <
                (unsigned long long)(base + EVENT_THREADS))
                break;
        }
        __syncthreads();
        if (threadIdx.x == 0) a.first[(int64_t)trial * a.n_groups + g] = best;
    }
    if (a.n_groups == 1 && blockIdx.x == 0 && threadIdx.x == 0) a.queue[0] = 0;
}

__global__ __launch_bounds__(EVENT_THREADS) void event_live_kernel(EventArgs a) {
    __shared__ int events;
    const int g = blockIdx.x;
    if (threadIdx.x == 0) events = 0;
    __syncthreads();
    int n = 0;
    for (int t = threadIdx.x; t < a.n_trials; t += EVENT_THREADS) n += a.first[(int64_t)t * a.n_groups + g] != EVENT_NONE;
    if (n) atomicAdd(&events, n);
    __syncthreads();
    if (threadIdx.x == 0) a.queue[g] = (unsigned long long)events << EVENT_SHIFT;
}

__global__ __launch_bounds__(EVENT_THREADS) void first_event_queue_kernel(EventArgs a, int rounds) {
    extern __shared__ uint32_t event_thr[];
    __shared__ unsigned long long ticket, claim, alive[EVENT_THREADS / WAVE];
    __shared__ uint32_t trial_of[EVENT_THREADS], segment_of[EVENT_THREADS];
    __shared__ unsigned long long live;
    __shared__ int next, found;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const RoundKeys keys = round_keys(a.key0, a.key1);
    const uint64_t n_trials = (uint64_t)a.n_trials;
    const uint64_t seg = (uint64_t)rounds * EVENT_ROUND;
    const uint64_t n_tickets = ((uint64_t)a.max_windows - EVENT_HEAD + seg - 1) / seg * n_trials;
    auto queue_word = [&](int g) { return __hip_atomic_load(a.queue + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    // one group: counted here, the trials that the head has left (their windows, if any by
    // now, lie behind it), and its queue counts from there
    uint64_t trials = n_trials;
    auto unfinished = [&](unsigned long long w) {   // trials without an event, 0 when no ticket is left either
        return (w & EVENT_TICKETS) < n_tickets ? trials - (w >> EVENT_SHIFT) : 0;
    };
    auto sum = [&](unsigned long long mine) {
        __syncthreads();
        if (tid == 0) live = 0;
        __syncthreads();
        if (mine) atomicAdd(&live, mine);
        __syncthreads();
        return live;
    };
    unsigned long long mine = 0;
    if (a.n_groups == 1) {
        for (int t = tid; t < a.n_trials; t += EVENT_THREADS)
            mine += __hip_atomic_load(a.first + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= EVENT_HEAD;
        trials = sum(mine);
        mine = tid == 0 ? unfinished(queue_word(0)) : 0;
    } else {
        for (int g = tid; g < a.n_groups; g += EVENT_THREADS) mine += unfinished(queue_word(g));
    }
    // few live trials: no more workgroups than share them usefully, as each claim waits for the others'
    if (blockIdx.x >= EVENT_SHARE * sum(mine)) return;
    int g = (int)(blockIdx.x % (unsigned)a.n_groups);
    for (;;) {
        // the next live group from g on
        if (tid == 0) next = INT32_MAX;
        __syncthreads();
        int ahead = INT32_MAX;
        for (int o = 0; o < a.n_groups && ahead == INT32_MAX; o += EVENT_THREADS) {
            if (o + tid < a.n_groups) {
                const int c = (int)(((int64_t)g + o + tid) % a.n_groups);
                if (unfinished(queue_word(c))) atomicMin(&next, o + tid);
            }
            __syncthreads();
            ahead = next;
            __syncthreads();   // every thread has read it
        }
        if (ahead == INT32_MAX) return;
        g = (int)(((int64_t)g + ahead) % a.n_groups);
        const EventTable tab(a, g, event_thr);
        const int stride = max(1, 32 / tab.nm1);   // rounds between looks at first[]
        const uint64_t least = (uint64_t)max(1, EVENT_CLAIM_DRAWS / (rounds * tab.nm1));
        if (tid == 0) found = 0;
        for (;;) {
            __syncthreads();   // the table is written; `found` is complete, every thread has read the last claim
            if (tid == 0) {
                const unsigned long long add = (unsigned long long)found << EVENT_SHIFT;
                unsigned long long w = queue_word(g);
                const uint64_t left = unfinished(w + add);
                // more live ones a claim where they outnumber the workgroups
                const uint64_t many = min((uint64_t)EVENT_MOST_LIVE, max((uint64_t)1, left * a.n_groups / gridDim.x));
                claim = left ? max(many * n_trials / left, least) : 0;
                if (left || found) w = atomicAdd(a.queue + g, add + claim);
                ticket = w & EVENT_TICKETS;
                found = 0;
                if (left && !unfinished(w + add)) claim = 0;
            }
            __syncthreads();
            const uint64_t t0 = ticket, t1 = min(ticket + claim, n_tickets);
            if (claim == 0 || t0 >= n_tickets) break;
            for (uint64_t c = t0; c < t1; c += EVENT_THREADS) {
                const uint32_t segment = (uint32_t)((c + tid) / n_trials);
                const uint32_t trial = (uint32_t)(c + tid - segment * n_trials);
                trial_of[tid] = trial;
                segment_of[tid] = segment;
                const bool on = c + tid < t1 && __hip_atomic_load(a.first + (int64_t)trial * a.n_groups + g, __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_AGENT) >= EVENT_HEAD + segment * seg;
                const uint64_t b = __builtin_amdgcn_ballot_w64(on);
                if ((tid & (WAVE - 1)) == 0) alive[wave] = b;
                __syncthreads();
                for (int i = 0; i < EVENT_THREADS; ++i) {
                    if (!(alive[i >> 6] >> (i & 63) & 1)) {
                        if (alive[i >> 6] >> (i & 63) == 0) i |= 63;
                        continue;
                    }
                    const uint32_t trial = __builtin_amdgcn_readfirstlane(trial_of[i]);
                    int64_t base = EVENT_HEAD + (int64_t)(__builtin_amdgcn_readfirstlane(segment_of[i]) * seg);
                    unsigned long long* const best = a.first + (int64_t)trial * a.n_groups + g;
                    for (int round = 0; round < rounds; ++round, base += EVENT_ROUND) {
                        // an event in an earlier window, found here or by another
                        // workgroup, leaves nothing to find in the rest
                        if (base >= a.max_windows ||
                            (round % stride == 0 && __hip_atomic_load(best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                                                        (unsigned long long)base))
                            break;
                        const unsigned long long hit = tab.scan<EVENT_WPT>(base, trial, a.max_windows, keys);
                        if (hit != EVENT_NONE && atomicMin(best, hit) == EVENT_NONE) atomicAdd(&found, 1);
                        if (__builtin_amdgcn_ballot_w64(hit != EVENT_NONE)) break;
                    }
                }
                __syncthreads();   // alive[] is rewritten
            }
        }
        __syncthreads();   // the table is rewritten
    }
}

// The same without the LDS table (chains whose thresholds do not fit): one
// wavefront per (trial, group), the lanes cover the springs and the wave walks
// the windows in order, the rate read and the FP64 test per draw.
__global__ __launch_bounds__(64) void first_event_kernel(const GroupDev* __restrict__ groups,
                                                         const double* __restrict__ rates, int64_t n_windows,
                                                         int64_t spr_total, int64_t max_windows, int S,
                                                         uint32_t key0, uint32_t key1,
                                                         unsigned long long* __restrict__ first_window,
                                                         int n_groups) {
    const int trial = blockIdx.x;
    const int g = blockIdx.y;
    const GroupDev& G = groups[g];
    const int lane = threadIdx.x;
    const int nm1 = G.N - 1;
    const double window_time = (double)S * G.dt;
    const uint32_t ctr3 = (2u << 24) | (G.stream & 0xFFFFFFu);
    const RoundKeys keys = round_keys<false>(key0, key1);
    unsigned long long first = EVENT_NONE;
    int64_t w = 0;
    for (int64_t v = 0; v < max_windows; ++v) {
        bool hit = false;
        for (int j = lane; j < nm1; j += WAVE) {
            const double k = rates[w * spr_total + G.spr_off + j];
            const Words u = philox10((uint32_t)v, (uint32_t)j, (uint32_t)trial, ctr3, keys);
            hit |= u01_f64_53(u.x, u.y) < -expm1(-k * window_time);
        }
        if (__builtin_amdgcn_ballot_w64(hit) != 0) {
            first = (unsigned long long)v;
            break;
        }
        if (++w == n_windows) w = 0;
    }
    if (lane == 0) first_window[(int64_t)trial * n_groups + g] = first;
}

// The censored maximum-likelihood mean of the first-passage times: all
// trials' times (first-passage or censoring) over the number of events; one
// wavefront per group, trials summed in fixed order.
__global__ __launch_bounds__(64) void mftu_events_kernel(const GroupDev* __restrict__ groups,
                                                         unsigned long long* __restrict__ first, int n_trials,
                                                         int64_t max_windows, int S, int n_groups,
                                                         double* __restrict__ mftu) {
    const int g = blockIdx.x;
    const double window_time = (double)S * groups[g].dt;
    double total = 0.0, events = 0.0;
    for (int t = threadIdx.x; t < n_trials; t += WAVE) {
        const unsigned long long f = first[(int64_t)t * n_groups + g];
        const bool hit = f != EVENT_NONE;   // EVENT_NONE is the -1 of a censored trial
        total += (double)(hit ? (int64_t)f + 1 : max_windows) * window_time;
        events += hit ? 1.0 : 0.0;
    }
    total = wave_sum_d(total);
    events = wave_sum_d(events);
    if (threadIdx.x == 0) mftu[g] = events > 0.0 ? total / events : __builtin_inf();
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
hipError_t launch_reclone(const GroupDev* groups, const GroupDev* pgroups, int n_groups, int64_t max_elems,
                          const void* pstate, void* state, double* tsf_acc, int32_t* status, const int64_t* par_off,
                          double* src, int64_t* step, int64_t step_value, int64_t* parent_step, int64_t parent_steps,
                          int precision, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    const int64_t blocks = std::min<int64_t>(1024, (max_elems + 255) / 256);
    dim3 grid((unsigned)std::max<int64_t>(1, blocks), (unsigned)n_groups), block(256);
    if (precision == 64)
        hipLaunchKernelGGL(reclone_kernel<double>, grid, block, 0, st, groups, pgroups, (const double*)pstate,
                           (double*)state, tsf_acc, status, par_off, src, step, step_value, parent_step, parent_steps);
    else
        hipLaunchKernelGGL(reclone_kernel<float>, grid, block, 0, st, groups, pgroups, (const float*)pstate,
                           (float*)state, tsf_acc, status, par_off, src, step, step_value, parent_step, parent_steps);
    return hipGetLastError();
}

hipError_t launch_conformation(const GroupDev* groups, int n_groups, const int64_t* rep_off, int64_t n_reps,
                               const void* state, const int64_t* par_off, const double* src, double* dbar,
                               double* d_bead, double* rg2, double* src_rg2, int precision, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (n_reps > 0 && (dbar || d_bead || rg2)) {
        dim3 grid((unsigned)((n_reps + 3) / 4)), block(256);
        if (precision == 64)
            hipLaunchKernelGGL(conformation_kernel<double>, grid, block, 0, st, groups, n_groups, rep_off,
                               (const double*)state, par_off, src, dbar, d_bead, rg2);
        else
            hipLaunchKernelGGL(conformation_kernel<float>, grid, block, 0, st, groups, n_groups, rep_off,
                               (const float*)state, par_off, src, dbar, d_bead, rg2);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (src_rg2) hipLaunchKernelGGL(src_rg2_kernel, dim3((unsigned)n_groups), dim3(64), 0, st, groups, par_off, src,
                                    src_rg2);
    return hipGetLastError();
}

hipError_t launch_block_sigma(const GroupDev* groups, const ColTile* tiles, int n_tiles, int64_t n_windows,
                              const void* smp, int64_t smp_total, int64_t spr_total, int block, double* sigma,
                              int precision, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (n_tiles == 0 || n_windows == 0) return hipSuccess;
    dim3 grid((unsigned)n_tiles, (unsigned)n_windows), blk(WAVE * BSIG_WAVES);
    if (precision == 64)
        hipLaunchKernelGGL(block_sigma_kernel<double>, grid, blk, 0, st, groups, tiles, (const double*)smp, smp_total,
                           spr_total, block, sigma);
    else
        hipLaunchKernelGGL(block_sigma_kernel<float>, grid, blk, 0, st, groups, tiles, (const float*)smp, smp_total,
                           spr_total, block, sigma);
    return hipGetLastError();
}

hipError_t launch_mftu_events(const GroupDev* groups, int n_groups, const double* rates, int64_t n_windows,
                              int64_t spr_total, int n_trials, int64_t max_windows, int S, uint32_t key0,
                              uint32_t key1, int max_springs, int64_t* first_window, double* mftu, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    const size_t lds = (size_t)n_windows * (size_t)std::max(max_springs, 1) * sizeof(uint64_t);
    unsigned long long* first = (unsigned long long*)first_window;   // -1 is EVENT_NONE
    if (n_windows <= 0xFFFFFFFFll && lds <= EVENT_LDS_MAX) {
        const EventArgs a{groups, rates, n_windows, spr_total, max_windows, n_groups, n_trials, S, key0, key1, first,
                          (unsigned long long*)mftu};
        const int64_t trials = (int64_t)n_trials * n_groups;
        const int per_block = (int)std::min<int64_t>(16, std::max<int64_t>(1, trials / (2 * EVENT_BLOCKS)));
        hipLaunchKernelGGL(first_event_head_kernel, dim3((unsigned)((n_trials + per_block - 1) / per_block), (unsigned)n_groups),
                           dim3(EVENT_THREADS), lds, st, a, per_block);
        if (max_windows > EVENT_HEAD) {
            if (n_groups > 1)
                hipLaunchKernelGGL(event_live_kernel, dim3((unsigned)n_groups), dim3(EVENT_THREADS), 0, st, a);
            // 64 segments per trial or more, of 1 to 4 rounds
            const int rounds = (int)std::min<int64_t>(EVENT_MOST_ROUNDS, std::max<int64_t>(1, max_windows / (64 * EVENT_ROUND)));
            const int64_t seg = (int64_t)rounds * EVENT_ROUND;
            const int64_t tickets = (max_windows - EVENT_HEAD + seg - 1) / seg * trials;
            hipLaunchKernelGGL(first_event_queue_kernel, dim3((unsigned)std::min<int64_t>(tickets, EVENT_BLOCKS)),
                               dim3(EVENT_THREADS), lds, st, a, rounds);
        }
    } else {
        hipLaunchKernelGGL(first_event_kernel, dim3((unsigned)n_trials, (unsigned)n_groups), dim3(64), 0, st, groups,
                           rates, n_windows, spr_total, max_windows, S, key0, key1, first, n_groups);
    }
    hipLaunchKernelGGL(mftu_events_kernel, dim3((unsigned)n_groups), dim3(64), 0, st, groups, first, n_trials,
                       max_windows, S, n_groups, mftu);
    return hipGetLastError();
}

hipError_t launch_mftu(const double* rate_sum, int64_t n_windows, int n_groups, double* mftu, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    hipLaunchKernelGGL(mftu_kernel, dim3((unsigned)n_groups), dim3(64), 0, st, rate_sum, n_windows, n_groups, mftu);
    return hipGetLastError();
}

}  // namespace ra

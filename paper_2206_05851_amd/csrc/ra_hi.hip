// ra_hi.hip — forward kernel with hydrodynamic interaction (Eqs. 1-3).
//
// Per step and replica: the 3N x 3N Rotne-Prager-Yamakawa diffusion tensor D
// (Eq. 2 on the diagonal, Eq. 3 off it) from the current positions, the drift
// dt D F / kT, and the random displacement sqrt(2 dt) L xi with D = L L^T
// (Cholesky), xi the per-bead normals of the replica counter. Forces F are the
// springs (Hookean, FENE or rest-length harmonic) plus optional LJ between
// non-adjacent beads, as in the pair kernel.
//
// One workgroup (256 threads) per replica. Wave 0 keeps the bond state in
// registers (lane i = bond i), rebuilds positions by a wave scan and forms the
// spring forces, while wave 1 draws the noise; D is assembled in LDS as a packed
// lower triangle (n = 3N <= 192: at most 18528 elements) and loaded into the
// matrix-instruction layout, from which the drift D F is taken and which the
// factorization updates in place (see factor_apply). Wave 0 then applies the
// bond-form update Q_j += dt kappa Q_j + (Y_{j+1} - Y_j), Y the bead
// displacements without the flow term.
#include "ra_chain.hpp"
#include "ra_dpp.hpp"
#include "ra_launch.hpp"

namespace ra {

constexpr int HI_THREADS = 256;
constexpr int HI_LD = 20;   // LDS row of 16 panel entries: 16-byte rows, no bank conflict in either use

template <int V> struct Int { static constexpr int value = V; };

// LDS elements of the packed triangle of n rows, whose space then takes two
// panels and the drift's column parts of 16 nb rows.
__host__ __device__ constexpr int hi_matrix_elems(int n, int nb) {
    const int t = n * (n + 1) / 2, p = 16 * nb * (2 * HI_LD + 4 * nb);
    return ((t > p ? t : p) + 3) & ~3;
}

template <typename T> struct HiCo;
template <> struct HiCo<float> {
    const GroupDev& G;
    __device__ float r0() const { return G.r0; }
    __device__ float lj12u() const { return G.lj12u; }
    __device__ float ljr2() const { return G.ljr2; }
};
template <> struct HiCo<double> {
    const GroupDev& G;
    __device__ double r0() const { return G.r0_d; }
    __device__ double lj12u() const { return G.lj12u_d; }
    __device__ double ljr2() const { return G.ljr2_d; }
};

__device__ __forceinline__ int tri(int i) { return (i * (i + 1)) >> 1; }

// Lane force of the spring on bond Q (on its first bead, toward the second).
template <typename T>
__device__ __forceinline__ void hi_spring(T qx, T qy, T qz, const GroupDev& G, T& fx, T& fy, T& fz, int& clamps) {
    const T H = Co<T>{G}.H();
    const T q2 = fmadd(qx, qx, fmadd(qy, qy, qz * qz));
    T g = (T)1;
    if (G.spring == 1) {
        g = fene_g(qx, qy, qz, q2, (T)G.inv_q0sq, G.inv_q0sq_d, clamps);
    } else if (G.spring == 2) {
        const T q = fast_sqrt(q2);
        g = q > (T)0 ? (T)1 - HiCo<T>{G}.r0() * fast_rcp(q) : (T)0;
    }
    fx = H * g * qx;
    fy = H * g * qy;
    fz = H * g * qz;
}

template <typename T>
__device__ __forceinline__ T hi_tension(T qx, T qy, T qz, const GroupDev& G) {
    const T H = Co<T>{G}.H();
    const T q2 = fmadd(qx, qx, fmadd(qy, qy, qz * qz));
    const T q = fast_sqrt(q2);
    if (G.spring == 2) return H * (q - HiCo<T>{G}.r0());
    if (G.spring == 1) {
        int dummy = 0;
        return H * fene_g(qx, qy, qz, q2, (T)G.inv_q0sq, G.inv_q0sq_d, dummy) * q;
    }
    return H * q;
}

// Matrix instructions of the two precisions: D(16x16) = A(16x4) B(4x16) + C.
// Lane l gives A[l % 16][l / 16] and B[l / 16][l % 16]; register r of C and D is
// column l % 16 of row acc_row(l, r).
template <typename T> struct Acc;
template <> struct Acc<float> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct Acc<double> { typedef double type __attribute__((ext_vector_type(4))); };

__device__ __forceinline__ Acc<float>::type mfma16(float a, float b, Acc<float>::type c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ Acc<double>::type mfma16(double a, double b, Acc<double>::type c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
template <typename T> __device__ __forceinline__ int acc_row(int lane, int r) {
    return sizeof(T) == 4 ? 4 * (lane >> 4) + r : (lane >> 4) + 4 * r;
}

// A column C of the factorization. For j > C: d[j] -= l[j] l (the diagonal block's
// rows) and a[j] -= l[j] m (the own row), l[j] the value of l in lane j of the
// 16-lane row (DPP row_newbcast inside the FMA); the next pivot p = d[C + 1] of lane
// C + 1 and its 1 / sqrt r as soon as that column is done; yd += x[C] e, ya += x[C] m.
// One asm block, because a DPP operand needs two wait states after its write and
// the compiler sees no DPP in asm: the block starts with them, and nothing (no
// register copy either) comes between it and the last use of l or x.
// HI_P k: the pair of column C + 1 + k.
#define HI_ROW " row_mask:0xf bank_mask:0xf\n\t"
#define HI_PAIR(OP, D, M, J) \
    OP " %" #D ", -%[l], %[l] row_newbcast:%[j" #J "]" HI_ROW OP " %" #M ", -%[l], %[m] row_newbcast:%[j" #J "]" HI_ROW
#define HI_PIVOT(MOV) MOV " %[p], %0 row_newbcast:%[j0]" HI_ROW
#define HI_NOISE(OP) OP " %[yd], %[x], %[e] row_newbcast:%[c]" HI_ROW OP " %[ya], %[x], %[m] row_newbcast:%[c]" HI_ROW
#define HI_T1(OP, MOV, RSQ) HI_PAIR(OP, 0, 1, 0) "s_nop 0\n\t" HI_PIVOT(MOV) RSQ
#define HI_T2(OP, MOV, RSQ) HI_PAIR(OP, 0, 1, 0) HI_PAIR(OP, 2, 3, 1) HI_PIVOT(MOV) RSQ
#define HI_T3(OP, MOV, RSQ) HI_PAIR(OP, 0, 1, 0) HI_PAIR(OP, 2, 3, 1) HI_PIVOT(MOV) HI_PAIR(OP, 4, 5, 2) RSQ
#define HI_T4(OP, MOV, RSQ) HI_T3(OP, MOV, RSQ) HI_PAIR(OP, 6, 7, 3)
#define HI_T5(OP, MOV, RSQ) HI_T4(OP, MOV, RSQ) HI_PAIR(OP, 8, 9, 4)
#define HI_T6(OP, MOV, RSQ) HI_T5(OP, MOV, RSQ) HI_PAIR(OP, 10, 11, 5)
#define HI_T7(OP, MOV, RSQ) HI_T6(OP, MOV, RSQ) HI_PAIR(OP, 12, 13, 6)
#define HI_T8(OP, MOV, RSQ) HI_T7(OP, MOV, RSQ) HI_PAIR(OP, 14, 15, 7)
#define HI_T9(OP, MOV, RSQ) HI_T8(OP, MOV, RSQ) HI_PAIR(OP, 16, 17, 8)
#define HI_T10(OP, MOV, RSQ) HI_T9(OP, MOV, RSQ) HI_PAIR(OP, 18, 19, 9)
#define HI_T11(OP, MOV, RSQ) HI_T10(OP, MOV, RSQ) HI_PAIR(OP, 20, 21, 10)
#define HI_T12(OP, MOV, RSQ) HI_T11(OP, MOV, RSQ) HI_PAIR(OP, 22, 23, 11)
#define HI_T13(OP, MOV, RSQ) HI_T12(OP, MOV, RSQ) HI_PAIR(OP, 24, 25, 12)
#define HI_T14(OP, MOV, RSQ) HI_T13(OP, MOV, RSQ) HI_PAIR(OP, 26, 27, 13)
#define HI_T15(OP, MOV, RSQ) HI_T14(OP, MOV, RSQ) HI_PAIR(OP, 28, 29, 14)
#define HI_O1 "+v"(d[C + 1]), "+v"(a[C + 1])
#define HI_O2 HI_O1, "+v"(d[C + 2]), "+v"(a[C + 2])
#define HI_O3 HI_O2, "+v"(d[C + 3]), "+v"(a[C + 3])
#define HI_O4 HI_O3, "+v"(d[C + 4]), "+v"(a[C + 4])
#define HI_O5 HI_O4, "+v"(d[C + 5]), "+v"(a[C + 5])
#define HI_O6 HI_O5, "+v"(d[C + 6]), "+v"(a[C + 6])
#define HI_O7 HI_O6, "+v"(d[C + 7]), "+v"(a[C + 7])
#define HI_O8 HI_O7, "+v"(d[C + 8]), "+v"(a[C + 8])
#define HI_O9 HI_O8, "+v"(d[C + 9]), "+v"(a[C + 9])
#define HI_O10 HI_O9, "+v"(d[C + 10]), "+v"(a[C + 10])
#define HI_O11 HI_O10, "+v"(d[C + 11]), "+v"(a[C + 11])
#define HI_O12 HI_O11, "+v"(d[C + 12]), "+v"(a[C + 12])
#define HI_O13 HI_O12, "+v"(d[C + 13]), "+v"(a[C + 13])
#define HI_O14 HI_O13, "+v"(d[C + 14]), "+v"(a[C + 14])
#define HI_O15 HI_O14, "+v"(d[C + 15]), "+v"(a[C + 15])
#define HI_I1 [j0] "n"(C + 1)
#define HI_I2 HI_I1, [j1] "n"(C + 2)
#define HI_I3 HI_I2, [j2] "n"(C + 3)
#define HI_I4 HI_I3, [j3] "n"(C + 4)
#define HI_I5 HI_I4, [j4] "n"(C + 5)
#define HI_I6 HI_I5, [j5] "n"(C + 6)
#define HI_I7 HI_I6, [j6] "n"(C + 7)
#define HI_I8 HI_I7, [j7] "n"(C + 8)
#define HI_I9 HI_I8, [j8] "n"(C + 9)
#define HI_I10 HI_I9, [j9] "n"(C + 10)
#define HI_I11 HI_I10, [j10] "n"(C + 11)
#define HI_I12 HI_I11, [j11] "n"(C + 12)
#define HI_I13 HI_I12, [j12] "n"(C + 13)
#define HI_I14 HI_I13, [j13] "n"(C + 14)
#define HI_I15 HI_I14, [j14] "n"(C + 15)
#define HI_COL(n, OP, MOV, RSQ)                                                                               \
    asm volatile("s_nop 1\n\t" HI_T##n(OP, MOV, RSQ) HI_NOISE(OP)                                             \
                 : HI_O##n, [yd] "+v"(yd), [ya] "+v"(ya), [p] "=&v"(p), [r] "=&v"(r)                          \
                 : [l] "v"(l), [m] "v"(m), [e] "v"(e), [x] "v"(x), [c] "n"(C), HI_I##n)
#define HI_COLUMN(T, OP, MOV, RSQ)                                                                            \
    template <int C>                                                                                          \
    __device__ __forceinline__ void column_update(T (&d)[16], T (&a)[16], T l, T m, T e, T x, T& yd, T& ya, T& p, T& r) { \
        if constexpr (C == 14) HI_COL(1, OP, MOV, RSQ); \
        else if constexpr (C == 13) HI_COL(2, OP, MOV, RSQ); \
        else if constexpr (C == 12) HI_COL(3, OP, MOV, RSQ); \
        else if constexpr (C == 11) HI_COL(4, OP, MOV, RSQ); \
        else if constexpr (C == 10) HI_COL(5, OP, MOV, RSQ); \
        else if constexpr (C == 9) HI_COL(6, OP, MOV, RSQ); \
        else if constexpr (C == 8) HI_COL(7, OP, MOV, RSQ); \
        else if constexpr (C == 7) HI_COL(8, OP, MOV, RSQ); \
        else if constexpr (C == 6) HI_COL(9, OP, MOV, RSQ); \
        else if constexpr (C == 5) HI_COL(10, OP, MOV, RSQ); \
        else if constexpr (C == 4) HI_COL(11, OP, MOV, RSQ); \
        else if constexpr (C == 3) HI_COL(12, OP, MOV, RSQ); \
        else if constexpr (C == 2) HI_COL(13, OP, MOV, RSQ); \
        else if constexpr (C == 1) HI_COL(14, OP, MOV, RSQ); \
        else if constexpr (C == 0) HI_COL(15, OP, MOV, RSQ); \
        else                                                                                                  \
            asm volatile("s_nop 1\n\t" HI_NOISE(OP) : [yd] "+v"(yd), [ya] "+v"(ya)                            \
                         : [m] "v"(m), [e] "v"(e), [x] "v"(x), [c] "n"(C));                                   \
    }                                                                                                         \
    __device__ __forceinline__ T first_pivot(T v) {                                                           \
        T p;                                                                                                  \
        asm volatile("s_nop 1\n\t" MOV " %0, %1 row_newbcast:0" HI_ROW : "=v"(p) : "v"(v));                   \
        return p;                                                                                             \
    }
HI_COLUMN(float, "v_fmac_f32_dpp", "v_mov_b32_dpp", "v_rsq_f32 %[r], %[p]\n\t")
HI_COLUMN(double, "v_fmac_f64_dpp", "v_mov_b64_dpp", "v_rsq_f64 %[r], %[p]\n\t")

// 1 / sqrt(x): the hardware's in FP32; in FP64 its estimate y and two Newton steps.
__device__ __forceinline__ float inv_sqrt(float, float y) { return y; }
__device__ __forceinline__ double inv_sqrt(double x, double y) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double e = __builtin_fma(-x * y, y, 1.0);
        y = __builtin_fma(0.5 * e, y, y);
    }
    return y;
}
__device__ __forceinline__ float inv_sqrt(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double inv_sqrt(double x) { return inv_sqrt(x, __builtin_amdgcn_rsq(x)); }

// RPY block of Eq. 3 over D0 = kT/zeta for the pair separation (dx, dy, dz):
// D_ab = D0 (ci delta_ab + cr rhat_a rhat_b); ia = 1 / a. Both branches are
// computed and one is selected: neighbouring pairs take different ones.
template <typename T>
__device__ __forceinline__ void rpy_coeffs(T dx, T dy, T dz, T a, T ia, T& ci, T& cr, T& ux, T& uy, T& uz) {
    const T r2 = fmadd(dx, dx, fmadd(dy, dy, dz * dz));
    const T iq = r2 > (T)0 ? inv_sqrt(r2) : (T)0;
    const T q = r2 * iq;
    ux = dx * iq;
    uy = dy * iq;
    uz = dz * iq;
    const T aq = a * iq;
    const T s = (T)0.75 * aq, a2r2 = aq * aq;
    const T t = q * ia;
    const bool apart = q >= (T)2 * a;
    ci = apart ? s * fmadd((T)2 / (T)3, a2r2, (T)1) : fmadd((T)(-9.0 / 32.0), t, (T)1);
    cr = apart ? s * fmadd((T)-2, a2r2, (T)1) : (T)(3.0 / 32.0) * t;
}

// Drift, Cholesky factor and displacement for the packed tensor A (n = 3N rows,
// padded to 16 nb with the identity).
//
// The lower triangle is held as 16 x 16 blocks (I, J), J <= I, in the layout of
// the matrix instructions, negated; wavefront w owns block rows NB-1-w, NB-8+w
// and NB-9-w (where not negative), which keeps the four within one block of
// each other while rows retire.
//
// Drift D F: from the registers, as row sums (reduced over the 16 lanes of a
// column group) plus the transposed contribution of each block below the
// diagonal, summed over the block rows in order by wavefront 3, which has no
// rows to factor: the same sum whichever NB the context's longest chain asks for.
//
// Factorization D = L L^T by block columns k of 16:
//  1. the owners of block column k write it to LDS, one barrier;
//  2. wavefronts 0 .. (n - 1) / 64 factor the diagonal block and, in the same
//     sequence, solve for the block column below it: a lane holds its own row
//     of the matrix (row 64 w + lane) and, in every 16 lanes anew, a row of the
//     diagonal block, 16 entries each in registers. Column c takes the pivot and
//     the diagonal block's column by DPP row broadcasts inside the FMAs, so there is
//     no exchange between wavefronts within a block column. The rows' share of
//     y = L xi is summed on the way;
//  3. the rows below the diagonal block go back to LDS as L, one barrier;
//  4. each wavefront updates its blocks right of column k with matrix
//     instructions, C += L_I L_J^T, and writes block column k + 1 first.
// A non-positive pivot sets status bit 4 after the loop.
//
// The step is bound by the chain of block columns at one wavefront per SIMD: step 2
// is 240 FMAs and about 190 other instructions, step 4 128 cycles per block in
// FP32 (matrix instructions and VALU FMAs did not overlap, not from two
// wavefronts of a SIMD either: updating behind the next factor gained nothing).
// The elimination in panels of four columns, exchanged through LDS between all
// threads, took 38 barriers and 70k of the step's 91k cycles at N = 50. Per 40
// steps: FP32 N = 50, 50 replicas 1566 -> 904 us, 512 replicas 3102 -> 1301 us,
// N = 64 2232 -> 1167 us, N = 12 356 -> 283 us; FP64 N = 50 2189 -> 1308 us, N = 64
// 3071 -> 1690 us. The block column's entries by v_readlane instead of DPP: 10%
// slower; eight wavefronts instead of four: 1% faster at 50 replicas, but one
// workgroup per CU instead of two.
template <typename T, int NB>
__device__ __forceinline__ void factor_apply(T* A, int n, int tid, const T* X, T* F, const T* FL, T* DF, T* Y,
                                             T drift, T nsc, int32_t* status) {
    constexpr int NP = 16 * NB;
    constexpr int S0 = NB, S1 = NB > 4 ? NB - 4 : 0, S2 = NB > 8 ? NB - 8 : 0;   // blocks of the owned rows, at most
    constexpr int LD = HI_LD;
    using V = typename Acc<T>::type;
    const int lane = tid & (WAVE - 1), wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lx = lane & 15, lg = lane >> 4;
    const int I0 = NB - 1 - wv, I1 = S1 > 0 ? NB - 8 + wv : -1, I2 = S2 > 0 ? NB - 9 - wv : -1;
    V c0[S0], c1[S1 + 1], c2[S2 + 1];
    // Rows of block row I, negated and padded with the identity. The columns of a
    // lane's row are at a fixed distance, so a block costs its reads; blocks right
    // of the diagonal are read with them (in the LDS, never used). Only the
    // diagonal block needs the transposed part; I is one of the last four of cnt.
    auto load_row = [&](auto& c, int I, auto Count) {
        constexpr int cnt = decltype(Count)::value;
        if (I < 0) return;
        int base[4];
        bool in[4];
        T dg[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * I + acc_row<T>(lane, r), col = 16 * I + lx;
            const int hi = row > col ? row : col, lo = row > col ? col : row;
            in[r] = row < n;
            base[r] = tri(in[r] ? row : 0) + lx;
            const T v = A[hi < n ? tri(hi) + lo : 0];
            dg[r] = hi < n ? v : row == col ? (T)1 : (T)0;
        }
#pragma unroll
        for (int J = 0; J < cnt; ++J) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const T v = A[base[r] + 16 * J];
                const T e = in[r] ? v : (T)0;
                c[J][r] = -(J >= cnt - 4 && J == I ? dg[r] : e);
            }
        }
    };
    load_row(c0, I0, Int<S0>{});
    load_row(c1, I1, Int<S1>{});
    load_row(c2, I2, Int<S2>{});
    // total force: springs + the four LJ partial sums in fixed order
    if (FL != nullptr && tid < n) F[tid] += ((FL[tid] + FL[n + tid]) + FL[2 * n + tid]) + FL[3 * n + tid];
    __syncthreads();   // A has been read: its space takes the panels and the drift's column parts
    T* const panel = A;                    // 2 x [NP][LD]
    T* const colp = A + 2 * NP * LD;       // [4 NB][NP]: per block row and lane group
    {
        T fc[NB];
#pragma unroll
        for (int J = 0; J < NB; ++J) fc[J] = F[16 * J + lx];
        auto drift_row = [&](const auto& c, int I, auto Count) {
            constexpr int cnt = decltype(Count)::value;
            if (I < 0) return;
            T fr[4], p[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                fr[r] = F[16 * I + acc_row<T>(lane, r)];
                p[r] = (T)0;
            }
#pragma unroll
            for (int J = 0; J < cnt; ++J) {
                if (J < cnt - 4 || J <= I) {
                    T q = (T)0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        p[r] = fmadd(c[J][r], fc[J], p[r]);
                        q = fmadd(c[J][r], fr[r], q);
                    }
                    colp[(4 * I + lg) * NP + 16 * J + lx] = q;   // (J == I is not read)
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[r] = row16_sum(p[r]);
                if (lx == 0) DF[16 * I + acc_row<T>(lane, r)] = p[r];
            }
        };
        drift_row(c0, I0, Int<S0>{});
        if constexpr (S1 > 0) drift_row(c1, I1, Int<S1>{});
        if constexpr (S2 > 0) drift_row(c2, I2, Int<S2>{});
    }
    const int nb = (n + 15) >> 4;
    auto publish = [&](const V& c, int I, T* buf) {
#pragma unroll
        for (int r = 0; r < 4; ++r) buf[(16 * I + acc_row<T>(lane, r)) * LD + lx] = -c[r];
    };
    if (I0 >= 0) publish(c0[0], I0, panel);   // block column 0
    if (S1 > 0 && I1 >= 0) publish(c1[0], I1, panel);
    if (S2 > 0 && I2 >= 0) publish(c2[0], I2, panel);
    const int myrow = WAVE * wv + lane;
    T yrow = (T)0;
    bool bad = false;
    int k = 0;
#pragma clang loop unroll(disable)
    for (;;) {
        asm volatile("" : "+s"(k));   // one copy of the body: the compiler peels the switch's cases off otherwise
        T* const buf = panel + (k & 1) * (NP * LD);
        __syncthreads();
        // the diagonal block's rows (row lane % 16 in each 16-lane row) and this
        // lane's row below it
        const bool below = myrow >= 16 * (k + 1) && myrow < 16 * nb;
        if (WAVE * wv < 16 * nb) {
            const T* dsrc = (const T*)__builtin_assume_aligned(buf + (16 * k + lx) * LD, 16);
            T* const src = (T*)__builtin_assume_aligned(buf + (below ? myrow : 16 * k) * LD, 16);
            T d[16], a[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                d[c] = dsrc[c];
                a[c] = src[c];
            }
            const T xv = X[16 * k + lx];
            T yd = (T)0, ya = (T)0;
            T is = inv_sqrt(first_pivot(d[0]));
            auto column = [&](auto Cc) {
                constexpr int c = decltype(Cc)::value;
                const T ld = d[c] * is, la = a[c] * is;
                a[c] = la;
                T p, r;
                column_update<c>(d, a, ld, la, lx >= c ? ld : (T)0, xv, yd, ya, p, r);   // rows above the pivot are done
                if constexpr (c < 15) is = inv_sqrt(p, r);
            };
            column(Int<0>{}); column(Int<1>{}); column(Int<2>{}); column(Int<3>{});
            column(Int<4>{}); column(Int<5>{}); column(Int<6>{}); column(Int<7>{});
            column(Int<8>{}); column(Int<9>{}); column(Int<10>{}); column(Int<11>{});
            column(Int<12>{}); column(Int<13>{}); column(Int<14>{}); column(Int<15>{});
            // a pivot that is not positive makes its own row's l, and so y, not a number
            bad |= !(yd == yd);
            yrow += below ? ya : myrow >= 16 * k && myrow < 16 * k + 16 ? yd : (T)0;
            if (below && k + 1 < nb) {
#pragma unroll
                for (int c = 0; c < 16; ++c) src[c] = a[c];
            }
        }
        if (wv == 3 && k == 0) {
            // the last wavefront has no rows (n <= 192): it adds the drift's column parts
            for (int row = lane; row < n; row += WAVE) {
                T df = DF[row];
#pragma unroll 2
                for (int I = 1; I < nb; ++I) {
                    const T* v = colp + 4 * I * NP + row;
                    const T t = (v[0] + v[NP]) + (v[2 * NP] + v[3 * NP]);
                    df += I > (row >> 4) ? t : (T)0;
                }
                DF[row] = df;
            }
        }
        if (k + 1 == nb) break;
        __syncthreads();
        // C += L_I L_J^T for the owned blocks right of column k; the next block
        // column is published as soon as it is done
        T* const next = panel + ((k + 1) & 1) * (NP * LD);
        // K index of product q in lane group lg: column 4 lg + q, so that a lane's
        // operands are 16 (32) consecutive bytes
        T a0[4], a1[4], a2[4], b[NB][4];
        auto operand = [&](T (&o)[4], int I) {
            const T* r = (const T*)__builtin_assume_aligned(buf + (16 * I + lx) * LD + 4 * lg, 16);
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = r[q];
        };
        operand(a0, I0 > k ? I0 : k);
        if constexpr (S1 > 0) operand(a1, I1 > k ? I1 : k);
        if constexpr (S2 > 0) operand(a2, I2 > k ? I2 : k);
#pragma unroll
        for (int J = 1; J < NB; ++J) operand(b[J], J);   // all in flight at once (those left of k + 1 unused)
        auto update = [&](auto Jc) {
            constexpr int J = decltype(Jc)::value;
            if constexpr (J < NB) {
                auto block = [&](V& c, const T (&o)[4], int I) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) c = mfma16(o[q], b[J][q], c);
                    if (J == k + 1) publish(c, I, next);
                };
                // row I of a slot is one of four: the lowest decides at compile time
                if (J <= S0 - 4 || I0 >= J) block(c0[J], a0, I0);
                if constexpr (J < S1)
                    if (J <= S1 - 4 || I1 >= J) block(c1[J], a1, I1);
                if constexpr (J < S2)
                    if (J <= S2 - 4 || I2 >= J) block(c2[J], a2, I2);
            }
        };
        switch (k) {
        case 0: update(Int<1>{}); [[fallthrough]];
        case 1: update(Int<2>{}); [[fallthrough]];
        case 2: update(Int<3>{}); [[fallthrough]];
        case 3: update(Int<4>{}); [[fallthrough]];
        case 4: update(Int<5>{}); [[fallthrough]];
        case 5: update(Int<6>{}); [[fallthrough]];
        case 6: update(Int<7>{}); [[fallthrough]];
        case 7: update(Int<8>{}); [[fallthrough]];
        case 8: update(Int<9>{}); [[fallthrough]];
        case 9: update(Int<10>{}); [[fallthrough]];
        default: update(Int<11>{}); break;
        }
        ++k;
    }
    if (tid < 16 && bad) atomicOr(status, 4);
    if (myrow < n) {
        Y[myrow] = fmadd(-drift, DF[myrow], nsc * yrow);
    }
}

template <typename T, int NB>
__device__ __forceinline__ void run_hi(const FwdArgs& a, const GroupDev& G, int k, T* lds) {
    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool w0 = wv == 0;
    const int N = G.N, nm1 = N - 1, n = 3 * N;
    T* A = lds;                       // packed lower triangle; then panels and drift parts
    // region offsets are multiples of 4 elements (16-byte aligned panel rows)
    T* P = A + hi_matrix_elems(n, NB);   // positions [N][4]
    T* F = P + 4 * WAVE;              // forces [n], 0 up to 16 NB
    T* X = F + 3 * WAVE;              // normals [n], 0 up to 16 NB
    T* DF = X + 3 * WAVE;             // row part of D F
    T* Y = DF + 3 * WAVE;             // bead displacement without flow [n]
    T* C = Y + 3 * WAVE;              // LJ partial forces [4][n]
    const bool bond_ok = w0 && lane < nm1;
    const bool bead_ok = lane < N;
    T* const state = (T*)a.state;
    const int64_t sidx = (int64_t)k * nm1 + lane;
    T qx = (T)0, qy = (T)0, qz = (T)0;
    if (bond_ok) {
        const int64_t o = G.state_off + sidx * 3;
        qx = state[o];
        qy = state[o + 1];
        qz = state[o + 2];
    }
    const Co<T> c{G};
    const HiCo<T> hc{G};
    const T kx = c.kx(), ky = c.ky(), kz = c.kz(), kxz = c.kxz();
    const T D0 = (T)(G.kT / G.zeta);
    const T drift = (T)(G.dt / G.kT);                                 // dt / kT
    const T nsc = (T)(G.sigma_d * sqrt(G.zeta / G.kT));               // noise_scale sqrt(2 dt)
    const T ahi = (T)G.hi_a_d, iahi = (T)(1.0 / G.hi_a_d);
    const bool lj = G.lj12u_d > 0.0;
    const T lj12u = hc.lj12u(), ljr2 = hc.ljr2();
    const RoundKeys keys = round_keys(a.key0, a.key1);
    const uint32_t n0 = (uint32_t)*a.step0;
    const int S = a.S;
    const bool tsf = a.tsf != nullptr;
    double acc = 0.0;
    if (tsf && bond_ok) acc = a.tsf_acc[G.smp_off + sidx];
    int to_smp = S - (int)(n0 % (uint32_t)S);
    int64_t w = (int64_t)(n0 / (uint32_t)S);
    int clamps = 0;
    const int n_steps = (int)a.n_steps;
    if (tid < 3 * WAVE) F[tid] = X[tid] = (T)0;
    // this thread's bead pairs i > j, the same in every step (i in the upper half)
    constexpr int PAIRS = ((16 * NB / 3 + 1) * (16 * NB / 3) / 2 + HI_THREADS - 1) / HI_THREADS;
    uint32_t pair[PAIRS];
    const int n_pairs = (N * nm1) >> 1;
#pragma unroll
    for (int u = 0; u < PAIRS; ++u) {
        const int p = tid + u * HI_THREADS;
        int i = (int)((fast_sqrt(8.0f * (float)p + 1.0f) + 1.0f) * 0.5f);
        while ((i * (i - 1)) >> 1 > p) --i;
        while ((i * (i + 1)) >> 1 <= p) ++i;
        pair[u] = ((uint32_t)i << 16) | (uint32_t)(p - ((i * (i - 1)) >> 1));
    }
    __syncthreads();
    for (int st = 0; st < n_steps; ++st) {
        const uint32_t nstep = n0 + (uint32_t)st;
        // 1. positions and spring forces (wave 0), noise (wave 1)
        if (w0) {
            const T px = wave_scan_incl(qx) - qx;
            const T py = wave_scan_incl(qy) - qy;
            const T pz = wave_scan_incl(qz) - qz;
            P[4 * lane] = px;
            P[4 * lane + 1] = py;
            P[4 * lane + 2] = pz;
            T gx, gy, gz;
            hi_spring(qx, qy, qz, G, gx, gy, gz, clamps);
            const T bx = gx - from_prev_lane(gx), by = gy - from_prev_lane(gy), bz = gz - from_prev_lane(gz);
            if (bead_ok) {
                F[3 * lane] = bx;
                F[3 * lane + 1] = by;
                F[3 * lane + 2] = bz;
            }
        } else if (wv == 1) {
            T ex, ey, ez;
            normals3(philox10(nstep, (uint32_t)lane, (uint32_t)k, G.stream, keys), ex, ey, ez);
            if (bead_ok) {
                X[3 * lane] = ex;
                X[3 * lane + 1] = ey;
                X[3 * lane + 2] = ez;
            }
        }
        __syncthreads();
        // LJ between non-adjacent beads: wavefront v sums over the beads j of
        // its quarter of the chain for every bead i (lane), into its own rows
        if (lj) {
            const int q = (N + 3) >> 2;
            const int j0 = wv * q, j1 = j0 + q < N ? j0 + q : N;
            const T px = P[4 * lane], py = P[4 * lane + 1], pz = P[4 * lane + 2];
            T fx = (T)0, fy = (T)0, fz = (T)0;
#pragma unroll 4
            for (int j = j0; j < j1; ++j) {
                const T dx = px - P[4 * j], dy = py - P[4 * j + 1], dz = pz - P[4 * j + 2];
                const int dj = j - lane;
                const bool use = dj >= 2 || dj <= -2;
                // excluded pairs get a zero coefficient below (the select also
                // drops the self pair's Inf/NaN from 1/r^2 at r = 0)
                const T r2 = fmadd(dx, dx, fmadd(dy, dy, dz * dz));
                const T inv = fast_rcp(r2);
                const T s1 = ljr2 * inv;
                const T s3 = s1 * s1 * s1;
                const T cc = use ? lj12u * inv * fmadd(s3, s3, -s3) : (T)0;
                fx = fmadd(cc, dx, fx);
                fy = fmadd(cc, dy, fy);
                fz = fmadd(cc, dz, fz);
            }
            if (bead_ok) {
                T* fl = C + wv * n + 3 * lane;
                fl[0] = fx;
                fl[1] = fy;
                fl[2] = fz;
            }
        }
        // 2. D: the 3x3 block of each pair i > j, and the diagonal blocks
#pragma unroll
        for (int u = 0; u < PAIRS; ++u) {
            if (tid + u * HI_THREADS < n_pairs) {
                const int i = (int)(pair[u] >> 16), j = (int)(pair[u] & 0xFFFFu);
                T ci, cr, ux, uy, uz;
                rpy_coeffs(P[4 * j] - P[4 * i], P[4 * j + 1] - P[4 * i + 1], P[4 * j + 2] - P[4 * i + 2], ahi, iahi,
                           ci, cr, ux, uy, uz);
                const T uu[3] = {ux, uy, uz};
                T* row = A + tri(3 * i) + 3 * j;
#pragma unroll
                for (int x = 0; x < 3; ++x) {
#pragma unroll
                    for (int y = 0; y < 3; ++y) row[y] = D0 * fmadd(cr, uu[x] * uu[y], x == y ? ci : (T)0);
                    row += 3 * i + x + 1;
                }
            }
        }
        if (tid < n) {
            const int x = tid % 3;
            T* d = A + tri(tid) + tid;
            d[0] = D0;
            if (x > 0) d[-1] = (T)0;
            if (x > 1) d[-2] = (T)0;
        }
        __syncthreads();
        // 3-5. drift, Cholesky factor and the displacement Y = dt D F / kT + sqrt(2 dt) L xi
        factor_apply<T, NB>(A, n, tid, X, F, lj ? C : nullptr, DF, Y, drift, nsc, a.status);
        __syncthreads();
        // 6. bond update and sampling (wave 0)
        if (w0) {
            if (bond_ok) {
                const T ix = fmadd(kx, qx, fmadd(kxz, qz, Y[3 * lane + 3] - Y[3 * lane]));
                const T iy = fmadd(ky, qy, Y[3 * lane + 4] - Y[3 * lane + 1]);
                const T iz = fmadd(kz, qz, Y[3 * lane + 5] - Y[3 * lane + 2]);
                qx += ix;
                qy += iy;
                qz += iz;
            }
            const bool window_end = --to_smp == 0;
            if (tsf || window_end) {
                const T f = hi_tension(qx, qy, qz, G);
                if (tsf) acc += (double)f;
                if (window_end) {
                    bool bad = false;
                    if (bond_ok) {
                        const int64_t o = w * a.smp_total + G.smp_off + sidx;
                        ((T*)a.samples)[o] = f;
                        bad = !__builtin_isfinite((double)f);
                        if (tsf) {
                            ((T*)a.tsf)[o] = (T)(acc / (double)S);
                            acc = 0.0;
                        }
                    }
                    if (bad) atomicOr(a.status, 2);
                    to_smp = S;
                    ++w;
                }
            }
        }
    }
    if (bond_ok) {
        const int64_t o = G.state_off + sidx * 3;
        state[o] = qx;
        state[o + 1] = qy;
        state[o + 2] = qz;
        if (tsf) a.tsf_acc[G.smp_off + sidx] = acc;
    }
    if (w0) flush_clamps(clamps, a.clamps + (&G - a.groups));
}

// Wavefronts per SIMD that the registers leave room for. FP64 up to 10 beads: 188 registers
// held a CU to two replicas, 168 (three spilled) to three: 600 replicas of 2 beads, 40
// steps, 298 -> 178 us, 5000 1579 -> 1126.
template <typename T, int NB> struct HiWaves { static constexpr int value = sizeof(T) == 4 ? 2 : NB == 2 ? 3 : 1; };

// One kernel per register tile NB (16-row blocks of the tensor): the host
// picks the smallest NB with 16 NB >= 3 N_max, so each instance gets its own
// register allocation.
template <typename T, int NB>
__device__ __forceinline__ void hi_item(const FwdArgs& a, int item, T* lds) {
    if (item >= a.n_items) return;
    if (*(const volatile int*)a.status & 1) return;   // invalid parent: no work (whole block)
    const Item it = a.items[item];
    const GroupDev& G = a.groups[it.g];
    if (it.k0 >= G.R) return;
    run_hi<T, NB>(a, G, it.k0, lds);
}

template <typename T, int NB>
__global__ __launch_bounds__(HI_THREADS) __attribute__((amdgpu_waves_per_eu(HiWaves<T, NB>::value)))
void fwd_hi_kernel(FwdArgs a) {
    extern __shared__ __align__(16) unsigned char hi_lds[];
    hi_item<T, NB>(a, (int)blockIdx.x, (T*)hi_lds);
}

// Two contexts in one launch (see fwd_dual_kernel): blocks [0, n_items of a) run a. One
// body for both: with a copy each, NB = 12 in FP64 had every register taken, and the
// compiler saved one of b's addresses where the threads with tid >= n were masked off:
// parents of two block rows or more became NaN.
template <typename T, int NB>
__global__ __launch_bounds__(HI_THREADS) __attribute__((amdgpu_waves_per_eu(HiWaves<T, NB>::value)))
void fwd_hi_dual_kernel(FwdArgs a, FwdArgs b) {
    extern __shared__ __align__(16) unsigned char hi_lds[];
    const bool first = (int)blockIdx.x < a.n_items;
    hi_item<T, NB>(first ? a : b, (int)blockIdx.x - (first ? 0 : a.n_items), (T*)hi_lds);
}

// Register tile of the kernel instance launched for nb = ceil(3 N_max / 16).
static int hi_nb_instance(int nb) { return nb <= 2 ? 2 : nb <= 4 ? 4 : nb <= 6 ? 6 : nb <= 8 ? 8 : nb <= 10 ? 10 : 12; }

size_t hi_lds_bytes(int max_beads, int precision) {
    const int n = 3 * max_beads;
    const size_t elems = (size_t)hi_matrix_elems(n, hi_nb_instance((n + 15) / 16)) + 4 * WAVE + 12 * WAVE +
                         (size_t)std::max(4 * n, 3 * WAVE);
    return elems * (precision == 64 ? 8 : 4);
}

template <typename T>
static void launch_hi_nb(const FwdArgs& a, int nb, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    if (nb <= 2) hipLaunchKernelGGL((fwd_hi_kernel<T, 2>), grid, block, lds, st, a);
    else if (nb <= 4) hipLaunchKernelGGL((fwd_hi_kernel<T, 4>), grid, block, lds, st, a);
    else if (nb <= 6) hipLaunchKernelGGL((fwd_hi_kernel<T, 6>), grid, block, lds, st, a);
    else if (nb <= 8) hipLaunchKernelGGL((fwd_hi_kernel<T, 8>), grid, block, lds, st, a);
    else if (nb <= 10) hipLaunchKernelGGL((fwd_hi_kernel<T, 10>), grid, block, lds, st, a);
    else hipLaunchKernelGGL((fwd_hi_kernel<T, 12>), grid, block, lds, st, a);
}

hipError_t launch_forward_hi(const FwdArgs& a, int precision, int max_beads, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (a.n_items <= 0 || a.n_steps <= 0) return hipSuccess;
    if (max_beads < 2 || max_beads > WAVE) return hipErrorInvalidValue;
    const size_t lds = hi_lds_bytes(max_beads, precision);   // checked against the device limit by the host
    const int nb = (3 * max_beads + 15) / 16;
    dim3 grid((unsigned)a.n_items), block(HI_THREADS);
    if (precision == 64) launch_hi_nb<double>(a, nb, grid, block, lds, st);
    else launch_hi_nb<float>(a, nb, grid, block, lds, st);
    return hipGetLastError();
}

template <typename T>
static void launch_hi_dual_nb(const FwdArgs& a, const FwdArgs& b, int nb, dim3 grid, dim3 block, size_t lds,
                              hipStream_t st) {
    if (nb <= 2) hipLaunchKernelGGL((fwd_hi_dual_kernel<T, 2>), grid, block, lds, st, a, b);
    else if (nb <= 4) hipLaunchKernelGGL((fwd_hi_dual_kernel<T, 4>), grid, block, lds, st, a, b);
    else if (nb <= 6) hipLaunchKernelGGL((fwd_hi_dual_kernel<T, 6>), grid, block, lds, st, a, b);
    else if (nb <= 8) hipLaunchKernelGGL((fwd_hi_dual_kernel<T, 8>), grid, block, lds, st, a, b);
    else if (nb <= 10) hipLaunchKernelGGL((fwd_hi_dual_kernel<T, 10>), grid, block, lds, st, a, b);
    else hipLaunchKernelGGL((fwd_hi_dual_kernel<T, 12>), grid, block, lds, st, a, b);
}

hipError_t launch_forward_hi_dual(const FwdArgs& a, const FwdArgs& b, int precision, int max_beads, hipStream_t st) {
    (void)hipGetLastError();   // report only this launch's own error
    if (a.n_items + b.n_items <= 0) return hipSuccess;
    if (max_beads < 2 || max_beads > WAVE) return hipErrorInvalidValue;
    const size_t lds = hi_lds_bytes(max_beads, precision);
    const int nb = (3 * max_beads + 15) / 16;
    dim3 grid((unsigned)(a.n_items + b.n_items)), block(HI_THREADS);
    if (precision == 64) launch_hi_dual_nb<double>(a, b, nb, grid, block, lds, st);
    else launch_hi_dual_nb<float>(a, b, nb, grid, block, lds, st);
    return hipGetLastError();
}

}  // namespace ra

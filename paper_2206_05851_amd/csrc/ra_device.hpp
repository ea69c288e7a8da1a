// ra_device.hpp — gfx950 device building blocks: counter-based noise,
// lane-neighbour exchange, spring law. Shared by every kernel of the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ra {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11). The paper fixes only
// zero mean and covariance 2 D dt for the random displacement (Eq. 1 text);
// a counter-based generator gives every (step, bead, replica, group) its own
// draw with no stored state, so any tile layout and any replay (adjoint
// recompute, graph replay) reproduces the same noise.
// Counter words c0 (step) and c3 (tag|group) are wave-uniform and stay in
// SGPRs; the compiler then keeps the first round's c0 product on the scalar
// unit.
// ---------------------------------------------------------------------------
struct Words {
    uint32_t x, y, z, w;
};

// Round keys of one seed: key + r * (Weyl increments), r = 0..9. Built once
// per kernel so the step loop does not redo the key schedule. They are pinned
// to VGPRs (the empty asm only constrains the register class): with a scalar
// key the compiler splits each three-way XOR back into two v_xor_b32, with
// vector keys it selects one v_bitop3_b32, and the per-step scalar work of
// the first rounds disappears from the single instruction stream.
struct RoundKeys {
    uint32_t k0[10], k1[10];
};

// PIN_VGPR = false keeps the keys in scalar registers (20 fewer VGPRs, two
// v_xor_b32 per three-way XOR): for kernels where occupancy matters more.
template <bool PIN_VGPR = true>
__device__ __forceinline__ RoundKeys round_keys(uint32_t key0, uint32_t key1) {
    RoundKeys k;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        k.k0[r] = key0 + (uint32_t)r * 0x9E3779B9u;
        k.k1[r] = key1 + (uint32_t)r * 0xBB67AE85u;
        if constexpr (PIN_VGPR) {
            asm volatile("" : "+v"(k.k0[r]));
            asm volatile("" : "+v"(k.k1[r]));
        }
    }
    return k;
}

// Three-input XOR as one gfx950 v_bitop3_b32 (truth table 0x96 = a ^ b ^ c).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ Words philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                          const RoundKeys& k) {
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k.k0[round]);
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k.k1[round]);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
    return Words{c0, c1, c2, c3};
}

__device__ __forceinline__ Words philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                          uint32_t key0, uint32_t key1) {
    return philox10(c0, c1, c2, c3, round_keys(key0, key1));
}

// The chain kernels' blocks. Their step word c0 and stream word c3 are
// wave-uniform, their bead word c1 and replica word c2 stay with the lane, so of
// rounds 1-3 little is left for each block: what depends on the lane alone
// (BlockLane, once per launch) and what depends on the step alone (StepWords,
// once per step for all blocks of the wavefront) meet in 4 VALU instructions
// with one replica per wavefront (UNI: the replica word uniform too), 6 with
// several, against 12; rounds 4-10 are the 28 they were. The same words.
struct BlockLane {
    uint32_t h, l;     // M0 n0, n0 the block's first word after round 1
};
struct StepWords {
    uint32_t a, b, c, d;
};

template <bool UNI>
__device__ __forceinline__ StepWords step_words(uint32_t n, uint32_t replica, uint32_t stream, uint32_t key0,
                                                uint32_t key1) {
    constexpr uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
    const uint64_t p0 = (uint64_t)0xD2511F53u * n;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * ((uint32_t)(p0 >> 32) ^ stream ^ key1);
    StepWords w;
    w.a = (uint32_t)p0 ^ (key1 + W1);
    w.b = (uint32_t)p1 ^ (key0 + 2u * W0);
    w.c = (uint32_t)(p1 >> 32) ^ (key0 + W0);
    w.d = 0u;
    if constexpr (UNI) {
        const uint64_t q = (uint64_t)0xD2511F53u * (w.c ^ (uint32_t)((uint64_t)0xCD9E8D57u * replica));
        w.c = (uint32_t)(q >> 32) ^ (key1 + 2u * W1);
        w.d = (uint32_t)q ^ (key1 + 3u * W1);
    }
    return w;
}

__device__ __forceinline__ BlockLane block_lane(uint32_t bead, uint32_t replica, uint32_t key0) {
    const uint32_t n0 = (uint32_t)(((uint64_t)0xCD9E8D57u * replica) >> 32) ^ bead ^ key0;
    const uint64_t p = (uint64_t)0xD2511F53u * n0;
    return BlockLane{(uint32_t)(p >> 32), (uint32_t)p};
}

// rl: lo(M1 replica), used with several replicas per wavefront only.
template <bool UNI>
__device__ __forceinline__ Words philox_block(const BlockLane& L, const StepWords& w, uint32_t rl, const RoundKeys& k) {
    uint32_t c0, c1, c2, c3;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (L.h ^ w.a);           // rounds 2 and 3
    c0 = (uint32_t)(p1 >> 32) ^ w.b;
    c1 = (uint32_t)p1;
    if constexpr (UNI) {
        c2 = L.l ^ w.c;
        const uint64_t a = (uint64_t)0xD2511F53u * c0, b = (uint64_t)0xCD9E8D57u * c2;   // round 4
        c0 = xor3((uint32_t)(b >> 32), c1, k.k0[3]);
        c2 = (uint32_t)(a >> 32) ^ w.d;
        c1 = (uint32_t)b;
        c3 = (uint32_t)a;
    } else {
        const uint64_t p0 = (uint64_t)0xD2511F53u * (w.c ^ rl);
        c2 = xor3((uint32_t)(p0 >> 32), L.l, k.k1[2]);
        c3 = (uint32_t)p0;
    }
#pragma unroll
    for (int r = UNI ? 4 : 3; r < 10; ++r) {
        const uint64_t a = (uint64_t)0xD2511F53u * c0, b = (uint64_t)0xCD9E8D57u * c2;
        c0 = xor3((uint32_t)(b >> 32), c1, k.k0[r]);
        c2 = xor3((uint32_t)(a >> 32), c3, k.k1[r]);
        c1 = (uint32_t)b;
        c3 = (uint32_t)a;
    }
    return Words{c0, c1, c2, c3};
}

// Uniform in (0,1): the top 23 bits j of a word give (2j + 1) 2^-24 — an odd
// integer below 2^24 times a power of two, hence exact in binary32 and binary64.
// FP32: one v_alignbit_b32 forms the binary32 word of 1 + j 2^-23 (exponent
// bits 0x7F above the top 23 bits of x); subtracting 1 - 2^-24 is exact
// (Sterbenz) and leaves (2j + 1) 2^-24.
__device__ __forceinline__ float u01_f32(uint32_t x) {
    const uint32_t one_plus = __builtin_amdgcn_alignbit(0x7Fu, x, 9u);
    return __builtin_bit_cast(float, one_plus) - 0x1.fffffep-1f;
}
__device__ __forceinline__ double u01_f64(uint32_t x) {
    return (double)((x >> 8) | 1u) * 0x1p-24;
}
// Unfolding-event uniform from two words: the top 52 bits m of hi:lo give
// (2m + 1) 2^-53, exact in binary64; event probabilities per window reach
// 1e-7 and below, under the 2^-24 grid of the one-word map.
__device__ __forceinline__ double u01_f64_53(uint32_t hi, uint32_t lo) {
    const uint64_t m = ((uint64_t)hi << 20) | (uint64_t)(lo >> 12);
    return (double)(2 * m + 1) * 0x1p-53;
}

// Box-Muller, three normals from one Philox block: (r0 cos 2pi u1, r0 sin 2pi u1,
// r1 cos 2pi u3), r = sqrt(-2 ln u). FP32 uses the hardware transcendentals:
// v_log_f32 is log2, so -2 ln u = (-2 ln 2) log2 u; v_sin_f32/v_cos_f32 take
// their argument in revolutions, so sin(2 pi u) is one instruction on u.
__device__ __forceinline__ void normals3(const Words& w, float& a, float& b, float& c) {
    const float m2ln2 = -1.3862943611198906f;
    const float u0 = u01_f32(w.x), u1 = u01_f32(w.y), u2 = u01_f32(w.z), u3 = u01_f32(w.w);
    const float r0 = __builtin_amdgcn_sqrtf(m2ln2 * __builtin_amdgcn_logf(u0));
    const float r1 = __builtin_amdgcn_sqrtf(m2ln2 * __builtin_amdgcn_logf(u2));
    a = r0 * __builtin_amdgcn_cosf(u1);
    b = r0 * __builtin_amdgcn_sinf(u1);
    c = r1 * __builtin_amdgcn_cosf(u3);
}
// The same with the second pair's other output, d = r1 sin 2 pi u3 (noise map 1).
__device__ __forceinline__ void normals4(const Words& w, float& a, float& b, float& c, float& d) {
    const float m2ln2 = -1.3862943611198906f;
    const float u0 = u01_f32(w.x), u1 = u01_f32(w.y), u2 = u01_f32(w.z), u3 = u01_f32(w.w);
    const float r0 = __builtin_amdgcn_sqrtf(m2ln2 * __builtin_amdgcn_logf(u0));
    const float r1 = __builtin_amdgcn_sqrtf(m2ln2 * __builtin_amdgcn_logf(u2));
    a = r0 * __builtin_amdgcn_cosf(u1);
    b = r0 * __builtin_amdgcn_sinf(u1);
    c = r1 * __builtin_amdgcn_cosf(u3);
    d = r1 * __builtin_amdgcn_sinf(u3);
}
__device__ __forceinline__ void normals4(const Words& w, double& a, double& b, double& c, double& d) {
    const double u0 = u01_f64(w.x), u1 = u01_f64(w.y), u2 = u01_f64(w.z), u3 = u01_f64(w.w);
    const double r0 = sqrt(-2.0 * log(u0));
    const double r1 = sqrt(-2.0 * log(u2));
    double s1, c1, s3, c3;
    sincospi(2.0 * u1, &s1, &c1);
    sincospi(2.0 * u3, &s3, &c3);
    a = r0 * c1;
    b = r0 * s1;
    c = r1 * c3;
    d = r1 * s3;
}

__device__ __forceinline__ void normals3(const Words& w, double& a, double& b, double& c) {
    const double u0 = u01_f64(w.x), u1 = u01_f64(w.y), u2 = u01_f64(w.z), u3 = u01_f64(w.w);
    const double r0 = sqrt(-2.0 * log(u0));
    const double r1 = sqrt(-2.0 * log(u2));
    double s1, c1, s3, c3;
    sincospi(2.0 * u1, &s1, &c1);
    sincospi(2.0 * u3, &s3, &c3);
    (void)s3;
    a = r0 * c1;
    b = r0 * s1;
    c = r1 * c3;
}

// A normal times the step's noise amplitude, as a radius and a sine or cosine:
// the update multiplies them into its sum (one FMA), and the amplitude rides in
// the radius, r = sqrt(cn ln u) with cn = -2 sigma^2.
template <typename T> struct Polar {
    T r, t;
};

__device__ __forceinline__ void polars4(const Words& w, float cn, Polar<float>& a, Polar<float>& b, Polar<float>& c,
                                        Polar<float>& d) {
    const float u0 = u01_f32(w.x), u1 = u01_f32(w.y), u2 = u01_f32(w.z), u3 = u01_f32(w.w);
    const float r0 = __builtin_amdgcn_sqrtf(cn * __builtin_amdgcn_logf(u0));
    const float r1 = __builtin_amdgcn_sqrtf(cn * __builtin_amdgcn_logf(u2));
    a = Polar<float>{r0, __builtin_amdgcn_cosf(u1)};
    b = Polar<float>{r0, __builtin_amdgcn_sinf(u1)};
    c = Polar<float>{r1, __builtin_amdgcn_cosf(u3)};
    d = Polar<float>{r1, __builtin_amdgcn_sinf(u3)};
}
// The same between two s_nop 0 each, for wavefronts that share their SIMD: two
// wavefronts of a SIMD issue FP32, logic and shift instructions in the same
// cycles, and a transcendental breaks that for the next dozen or so unless an idle
// slot stands before and after it (56 adds and one sine per wavefront, two
// wavefronts: 220 cycles without, 150 with; one wavefront alone: 265 and 278).
template <char OP> __device__ __forceinline__ float paced(float x) {
    float r;
    if constexpr (OP == 'l') asm("s_nop 0\n\tv_log_f32 %0, %1\n\ts_nop 0" : "=v"(r) : "v"(x));
    else if constexpr (OP == 'q') asm("s_nop 0\n\tv_sqrt_f32 %0, %1\n\ts_nop 0" : "=v"(r) : "v"(x));
    else if constexpr (OP == 's') asm("s_nop 0\n\tv_sin_f32 %0, %1\n\ts_nop 0" : "=v"(r) : "v"(x));
    else if constexpr (OP == 'r') asm("s_nop 0\n\tv_rcp_f32 %0, %1\n\ts_nop 0" : "=v"(r) : "v"(x));
    else asm("s_nop 0\n\tv_cos_f32 %0, %1\n\ts_nop 0" : "=v"(r) : "v"(x));
    return r;
}
__device__ __forceinline__ void polars4_paced(const Words& w, float cn, Polar<float>& a, Polar<float>& b,
                                              Polar<float>& c, Polar<float>& d) {
    const float u0 = u01_f32(w.x), u1 = u01_f32(w.y), u2 = u01_f32(w.z), u3 = u01_f32(w.w);
    const float r0 = paced<'q'>(cn * paced<'l'>(u0));
    const float r1 = paced<'q'>(cn * paced<'l'>(u2));
    a = Polar<float>{r0, paced<'c'>(u1)};
    b = Polar<float>{r0, paced<'s'>(u1)};
    c = Polar<float>{r1, paced<'c'>(u3)};
    d = Polar<float>{r1, paced<'s'>(u3)};
}
__device__ __forceinline__ void polars4(const Words& w, double cn, Polar<double>& a, Polar<double>& b,
                                        Polar<double>& c, Polar<double>& d) {
    const double u0 = u01_f64(w.x), u1 = u01_f64(w.y), u2 = u01_f64(w.z), u3 = u01_f64(w.w);
    const double r0 = sqrt(cn * log(u0));
    const double r1 = sqrt(cn * log(u2));
    double s1, c1, s3, c3;
    sincospi(2.0 * u1, &s1, &c1);
    sincospi(2.0 * u3, &s3, &c3);
    a = Polar<double>{r0, c1};
    b = Polar<double>{r0, s1};
    c = Polar<double>{r1, c3};
    d = Polar<double>{r1, s3};
}

// ---------------------------------------------------------------------------
// Whole-wavefront lane shifts by DPP (GFX9 wave_shr:1 / wave_shl:1). Lanes
// whose source is outside the wave read 0 (bound_ctrl).
// ---------------------------------------------------------------------------
constexpr int DPP_WAVE_SHL1 = 0x130;   // lane l reads lane l+1
constexpr int DPP_WAVE_SHR1 = 0x138;   // lane l reads lane l-1

// mov_dpp with bound_ctrl writes 0 where the source lane is outside the wave
// and leaves the old value undefined, which lets the compiler fold the shift
// into the consuming VOP2 instruction.
template <int CTRL>
__device__ __forceinline__ float dpp_shift(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_shift(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
template <typename T> __device__ __forceinline__ T from_prev_lane(T v) { return dpp_shift<DPP_WAVE_SHR1>(v); }
template <typename T> __device__ __forceinline__ T from_next_lane(T v) { return dpp_shift<DPP_WAVE_SHL1>(v); }

// ---------------------------------------------------------------------------
// Numeric helpers per precision.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double fast_rcp(double x) { return 1.0 / x; }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double fast_sqrt(double x) { return sqrt(x); }

constexpr double FENE_DELTA = 1.0e-3;   // guard: s = |Q|^2/Q0^2 is clamped at 1 - delta
constexpr float FENE_FP64_BAND = 0.9f;  // FP32 path recomputes s and 1/(1-s) in FP64 above this

// FENE factor g = 1/(1 - min(s, 1 - delta)) from a bond of squared length q2.
// The FP32 path keeps g in FP32 except near full extension, where 1 - s loses
// digits: there s is recomputed in FP64 from the FP32 components (their
// products are exact in FP64). Returns the clamp flag through `clamped`.
__device__ __forceinline__ float fene_g(float qx, float qy, float qz, float q2, float inv_q0sq,
                                        double inv_q0sq_d, int& clamped) {
    const float s = q2 * inv_q0sq;
    float g = fast_rcp(1.0f - s);
    // wave vote: the common case (no lane near full extension) costs one
    // compare and a scalar branch instead of an exec-mask save/restore
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(s > FENE_FP64_BAND) != 0, 0)) {
        if (s > FENE_FP64_BAND) {
            const double dx = qx, dy = qy, dz = qz;
            double sd = (dx * dx + dy * dy + dz * dz) * inv_q0sq_d;
            if (sd > 1.0 - FENE_DELTA) { sd = 1.0 - FENE_DELTA; clamped += 1; }
            g = (float)(1.0 / (1.0 - sd));
        }
    }
    return g;
}
__device__ __forceinline__ double fene_g(double qx, double qy, double qz, double q2, double,
                                         double inv_q0sq_d, int& clamped) {
    (void)qx; (void)qy; (void)qz;
    double s = q2 * inv_q0sq_d;
    if (s > 1.0 - FENE_DELTA) { s = 1.0 - FENE_DELTA; clamped += 1; }
    return 1.0 / (1.0 - s);
}

__device__ __forceinline__ void polars4_paced(const Words& w, double cn, Polar<double>& a, Polar<double>& b,
                                              Polar<double>& c, Polar<double>& d) {
    polars4(w, cn, a, b, c, d);
}

// cF g of the same law for the forward step: fB - |Q|^2 fA = (1 - s) / cF in one
// FMA, and its reciprocal is the bond's force coefficient. The FP64 branch is
// taken where s > 0.9, the same band.
__device__ __forceinline__ float fene_force(float qx, float qy, float qz, float q2, float fA, float fB, float fT,
                                            double fC_d, double inv_q0sq_d, int& clamped) {
    const float t = __builtin_fmaf(-q2, fA, fB);
    float h = fast_rcp(t);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(t < fT) != 0, 0)) {
        if (t < fT) {
            const double dx = qx, dy = qy, dz = qz;
            double sd = (dx * dx + dy * dy + dz * dz) * inv_q0sq_d;
            if (sd > 1.0 - FENE_DELTA) { sd = 1.0 - FENE_DELTA; clamped += 1; }
            h = (float)(fC_d / (1.0 - sd));
        }
    }
    return h;
}
__device__ __forceinline__ double fene_force(double, double, double, double q2, double cF, double inv_q0sq_d,
                                             int& clamped) {
    double s = q2 * inv_q0sq_d;
    if (s > 1.0 - FENE_DELTA) { s = 1.0 - FENE_DELTA; clamped += 1; }
    return cF / (1.0 - s);
}

}  // namespace ra

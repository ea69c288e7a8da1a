// ra_clone.hpp — starting state of a run from a parent's FP64 bead positions.
#pragma once
#include "ra_device.hpp"
#include "ra_types.hpp"

namespace ra {

// Bond j of the parent in FP64; ok: finite, and inside full extension (FENE).
struct CloneBond {
    double x, y, z;
    bool ok;
};
__device__ __forceinline__ CloneBond clone_bond(const double* __restrict__ p, int j, const GroupDev& G) {
    CloneBond q;
    q.x = p[3 * (j + 1)] - p[3 * j];
    q.y = p[3 * (j + 1) + 1] - p[3 * j + 1];
    q.z = p[3 * (j + 1) + 2] - p[3 * j + 2];
    q.ok = __builtin_isfinite(q.x) && __builtin_isfinite(q.y) && __builtin_isfinite(q.z) &&
           (G.spring != 1 || (q.x * q.x + q.y * q.y + q.z * q.z) * G.inv_q0sq_d < 1.0);
    return q;
}

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, WAVE);
    return v;
}

// Clone source, by one wavefront: the parent less its centre of mass.
__device__ __forceinline__ void clone_source(const double* __restrict__ p, double* __restrict__ o, int N) {
    const int lane = threadIdx.x & (WAVE - 1);
    double sx = 0.0, sy = 0.0, sz = 0.0;
    for (int i = lane; i < N; i += WAVE) { sx += p[3 * i]; sy += p[3 * i + 1]; sz += p[3 * i + 2]; }
    const double cx = wave_sum_d(sx) / N, cy = wave_sum_d(sy) / N, cz = wave_sum_d(sz) / N;
    for (int i = lane; i < N; i += WAVE) {
        o[3 * i] = p[3 * i] - cx;
        o[3 * i + 1] = p[3 * i + 1] - cy;
        o[3 * i + 2] = p[3 * i + 2] - cz;
    }
}

}  // namespace ra

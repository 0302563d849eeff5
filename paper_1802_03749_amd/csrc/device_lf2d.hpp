// Device helpers of the 2D finite-volume loops: the edge flux (formula in
// umesh.h, UM_K_EDGE_FLUX_LF2D) and element loads/stores of dim-2 and dim-4
// dats in AoS or SoA layout.  Included by the HIP kernel files only.
#pragma once

#include <hip/hip_runtime.h>

#include "umesh.h"

namespace um {
namespace dev {

// Flux through an edge from cell L into cell R (formula in umesh.h),
// evaluated in type Real.
#define UM_LF2D_FLUX_BODY                                                      \
    const Real half = Real(0.5), one = Real(1);                                \
    const Real nx = xb1 - xa1;                                                 \
    const Real ny = xa0 - xb0;                                                 \
    Real FL[4], FR[4];                                                         \
    {                                                                          \
        const Real ri = one / qL[0];                                           \
        const Real u = qL[1] * ri;                                             \
        const Real v = qL[2] * ri;                                             \
        const Real p = gm1 * (qL[3] - half * (qL[1] * u + qL[2] * v));         \
        const Real U = u * nx + v * ny;                                        \
        FL[0] = qL[0] * U;                                                     \
        FL[1] = qL[1] * U + p * nx;                                            \
        FL[2] = qL[2] * U + p * ny;                                            \
        FL[3] = (qL[3] + p) * U;                                               \
    }                                                                          \
    {                                                                          \
        const Real ri = one / qR[0];                                           \
        const Real u = qR[1] * ri;                                             \
        const Real v = qR[2] * ri;                                             \
        const Real p = gm1 * (qR[3] - half * (qR[1] * u + qR[2] * v));         \
        const Real U = u * nx + v * ny;                                        \
        FR[0] = qR[0] * U;                                                     \
        FR[1] = qR[1] * U + p * nx;                                            \
        FR[2] = qR[2] * U + p * ny;                                            \
        FR[3] = (qR[3] + p) * U;                                               \
    }                                                                          \
    const Real mu = eps * half * (adtL + adtR);                                \
    _Pragma("unroll") for (int k = 0; k < 4; ++k)                              \
        f[k] = half * (FL[k] + FR[k]) + half * mu * (qL[k] - qR[k]);

template <typename Real>
__device__ __forceinline__ void lf2d_flux(Real xa0, Real xa1, Real xb0, Real xb1,
                                          const Real qL[4], const Real qR[4], Real adtL,
                                          Real adtR, Real gm1, Real eps, Real f[4]) {
    UM_LF2D_FLUX_BODY
}

template <typename Real>
__device__ __forceinline__ void lf2d_flux_nocontract(Real xa0, Real xa1, Real xb0, Real xb1,
                                                     const Real qL[4], const Real qR[4],
                                                     Real adtL, Real adtR, Real gm1, Real eps,
                                                     Real f[4]) {
#pragma clang fp contract(off)
    UM_LF2D_FLUX_BODY
}

// Velocity, pressure and (binary32) energy plus pressure of a state.  The
// roundings here and in lf2d_flux_out are written out: in binary32 they are
// those that lf2d_flux gets from the compiler's contractions.
template <typename Real>
struct Flow {
    Real u, v, p, h;
};

template <typename Real>
__device__ __forceinline__ Flow<Real> flow_of(const Real q[4], Real gm1) {
#pragma clang fp contract(off)
    const Real ri = Real(1) / q[0];
    Flow<Real> s;
    s.u = q[1] * ri;
    s.v = q[2] * ri;
    const Real e = fma(Real(-0.5), fma(q[1], s.u, q[2] * s.v), q[3]);
    s.p = e * gm1;
    s.h = fma(e, gm1, q[3]);
    return s;
}

// lf2d_flux as it leaves the cell with state q and flow s into the one with
// state r and flow t; the normal of (a, b) points that way, and `second` says
// that the cell left is the edge's second one.  Seen from the other side
// (states swapped, a and b swapped, second inverted) it is exactly the
// negative: every value rounded only changes its sign.
template <bool DISS, typename Real>
__device__ __forceinline__ void lf2d_flux_out(Real xa0, Real xa1, Real xb0, Real xb1,
                                              const Real q[4], const Flow<Real> &s,
                                              const Real r[4], const Flow<Real> &t, Real aq,
                                              Real ar, Real eps, bool second, Real f[4]) {
#pragma clang fp contract(off)
    const Real half = Real(0.5);
    const Real nx = xb1 - xa1;
    const Real ny = xa0 - xb0;
    const Real U = fma(s.v, ny, s.u * nx);
    const Real V = fma(t.v, ny, t.u * nx);
    const Real hm = half * (eps * half * (aq + ar));
    Real F[4];
    if constexpr (sizeof(Real) == 8) {
        F[0] = q[0] * U + r[0] * V;
        F[3] = (q[3] + s.p) * U + (r[3] + t.p) * V;
    } else {
        // binary32: bit for bit lf2d_flux, which rounds cell 1's product only
        F[0] = second ? fma(r[0], V, q[0] * U) : fma(q[0], U, r[0] * V);
        F[3] = second ? fma(t.h, V, s.h * U) : fma(s.h, U, t.h * V);
    }
    F[1] = fma(s.p, nx, q[1] * U) + fma(t.p, nx, r[1] * V);
    F[2] = fma(s.p, ny, q[2] * U) + fma(t.p, ny, r[2] * V);
#pragma unroll
    for (int k = 0; k < 4; ++k) f[k] = fma(q[k] - r[k], hm, half * F[k]);
    if constexpr (DISS && sizeof(Real) == 4) {
        // in hier_kernel, and in hier_flow_kernel on SoA data at two edges per
        // lane, the compiler rounds the dissipation of these two components
        // first
        f[0] = fma(half, F[0], (q[0] - r[0]) * hm);
        f[3] = fma(half, F[3], (q[3] - r[3]) * hm);
    }
}

// Element g of a dim-4 / dim-2 dat in AoS ([n][dim]) or SoA ([dim][n])
// layout; AoS uses 16-byte vector loads.
template <int LAYOUT, typename Real>
__device__ __forceinline__ void load4(const Real *__restrict__ a, int64_t n, int64_t g,
                                      Real v[4]) {
    if constexpr (LAYOUT == UM_AOS) {
        if constexpr (sizeof(Real) == 8) {
            const double2 *p = reinterpret_cast<const double2 *>(a + 4 * g);
            const double2 lo = p[0], hi = p[1];
            v[0] = lo.x; v[1] = lo.y; v[2] = hi.x; v[3] = hi.y;
        } else {
            const float4 t = reinterpret_cast<const float4 *>(a)[g];
            v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
        }
    } else {
        v[0] = a[g]; v[1] = a[n + g]; v[2] = a[2 * n + g]; v[3] = a[3 * n + g];
    }
}

template <int LAYOUT>
__device__ __forceinline__ void store4(double *__restrict__ a, int64_t n, int64_t g,
                                       const double v[4]) {
    if constexpr (LAYOUT == UM_AOS) {
        double2 *p = reinterpret_cast<double2 *>(a + 4 * g);
        p[0] = make_double2(v[0], v[1]);
        p[1] = make_double2(v[2], v[3]);
    } else {
        a[g] = v[0]; a[n + g] = v[1]; a[2 * n + g] = v[2]; a[3 * n + g] = v[3];
    }
}

template <int LAYOUT, typename Real>
__device__ __forceinline__ void load2(const Real *__restrict__ a, int64_t n, int64_t g, Real &v0,
                                      Real &v1) {
    if constexpr (LAYOUT == UM_AOS) {
        if constexpr (sizeof(Real) == 8) {
            const double2 t = reinterpret_cast<const double2 *>(a)[g];
            v0 = t.x; v1 = t.y;
        } else {
            const float2 t = reinterpret_cast<const float2 *>(a)[g];
            v0 = t.x; v1 = t.y;
        }
    } else {
        v0 = a[g]; v1 = a[n + g];
    }
}

// Sum over the 64 lanes of a wave in a fixed butterfly; every lane ends
// with the same value.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Fixed-order sum over the workgroup (waves in order); valid in lane 0 of
// wave 0.  blockDim.x is a multiple of 64, at most 1024.
__device__ __forceinline__ double block_sum(double v) {
    __shared__ double wsum[16];
    v = wave_sum(v);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) wsum[wave] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < int(blockDim.x >> 6); ++w) t += wsum[w];
    return t;
}

// Lane t's share of a sum of non-negative terms: terms t, t + T, t + 2T, ...
// of T lanes, added in that order; the loads of U terms are issued before their
// additions (a zero past the end leaves the sum unchanged).
template <int U>
__device__ __forceinline__ double lane_sum(const double *__restrict__ v, int32_t n) {
    const int32_t T = int32_t(blockDim.x);
    double acc = 0.0;
    for (int32_t i0 = threadIdx.x; i0 < n; i0 += U * T) {
        double u[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int32_t i = i0 + j * T;
            u[j] = i < n ? v[i] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < U; ++j) acc += u[j];
    }
    return acc;
}

// The time-step scalar of a cell side by side, its sides in order: velocity and
// sound speed of its state, then what one side adds, with the contractions
// that the compiler gives cell_adt written out.
template <typename Real>
struct Wave {
    Real u, v, c;
};

template <typename Real>
__device__ __forceinline__ Wave<Real> wave_of(const Real q[4], Real gm1) {
#pragma clang fp contract(off)
    const Real ri = Real(1) / q[0];
    Wave<Real> s;
    s.u = q[1] * ri;
    s.v = q[2] * ri;
    const Real p = gm1 * fma(Real(-0.5), fma(q[1], s.u, q[2] * s.v), q[3]);
    s.c = sqrt((Real(1) + gm1) * p * ri);
    return s;
}

template <typename Real>
__device__ __forceinline__ Real adt_side(Real xa0, Real xa1, Real xb0, Real xb1,
                                         const Wave<Real> &s) {
#pragma clang fp contract(off)
    const Real mx = xb1 - xa1;
    const Real my = xa0 - xb0;
    return fma(s.c, sqrt(fma(my, my, mx * mx)), fabs(fma(s.v, my, s.u * mx)));
}

}  // namespace dev
}  // namespace um

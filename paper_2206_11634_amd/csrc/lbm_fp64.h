// FP64 device arithmetic shared by the DEM kernels and their adjoint.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <limits>

namespace mdlbm {

// |d| < tol as d.d < step_tol2(tol): never for a tol that is not positive, and
// for one whose square underflows still where d.d is zero.
inline double step_tol2(double tol)
{
    return tol > 0.0 ? std::max(tol * tol, std::numeric_limits<double>::denorm_min()) : 0.0;
}

// 1/x and 1/sqrt(x): the hardware's estimate and two Newton steps, about half an
// ulp (a third of the instructions of a division).  The root's last step takes
// the rounding of x y into its residual.  Not a number at 0.
//
// What the DEM with them, the series below and angular velocities kept in the body
// frame is off its exact values (80-bit arithmetic; in brackets with the library's
// division, root and sincos and a frame change a half kick), rms over 30 substeps
// of 1 to 400 bodies in contact: quaternions 1.7e-16 (2.0e-16) for spheres, 2.1e-16
// (2.1e-16) for three to nine points, angular velocities 5e-17 (8e-17), positions
// and velocities the same to 1 %; of 40 and 100 bodies spinning at up to 1 rad a
// step: quaternions 1.4e-15 (5.3e-15), angular velocities 2.4e-15 (8.7e-15).  dJ/domega
// of 120 substeps in 12 coupled steps, against 113-bit differences: 2.7e-15 and
// 1.6e-15 (1.0e-14 and 5.2e-15) of the largest component for two runs.
__device__ __forceinline__ double fast_rcp(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double fast_rsqrt(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    y = fma(fma(-x * y, y, 1.0), 0.5 * y, y);
    const double p = x * y, e = fma(x, y, -p);  // x y = p + e
    return fma(fma(-e, y, fma(-p, y, 1.0)), 0.5 * y, y);
}

// cos t, sin t / t and the derivative of the latter by z = t^2, from their
// series, for z < 2^-6 (truncated under 1e-19).  The derivative of cos t by z
// is -(sin t / t) / 2.
constexpr double kSmallAngle2 = 0x1p-6;
__device__ __forceinline__ double cos_series(double z)
{
    return 1.0 + z * (-1.0 / 2 + z * (1.0 / 24 + z * (-1.0 / 720 + z * (1.0 / 40320 - z * (1.0 / 3628800)))));
}
__device__ __forceinline__ double sinc_series(double z)
{
    return 1.0 + z * (-1.0 / 6 + z * (1.0 / 120 + z * (-1.0 / 5040 + z * (1.0 / 362880 - z * (1.0 / 39916800)))));
}
__device__ __forceinline__ double sinc_slope(double z)
{
    return -1.0 / 6 + z * (2.0 / 120 + z * (-3.0 / 5040 + z * (4.0 / 362880 - z * (5.0 / 39916800))));
}

// How far the body with control points i0 .. i1 - 1 may reach from its centre:
// the largest distance of a point plus sqrt(sum K).  Four points' loads at once.
__device__ __forceinline__ double reach_of(const double* __restrict__ body, const double* __restrict__ K,
                                           int i0, int i1)
{
    double sk = 0.0, r2 = 0.0;
    for (int i = i0; i < i1; i += 4) {
        double b[4][3], k[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t at = i + j < i1 ? i + j : i1 - 1;
            for (int a = 0; a < 3; ++a) b[j][a] = body[3 * at + a];
            k[j] = K[at];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i + j < i1) {
                r2 = fmax(r2, b[j][0] * b[j][0] + b[j][1] * b[j][1] + b[j][2] * b[j][2]);
                sk += k[j];
            }
    }
    return sqrt(r2) + sqrt(sk);
}

}  // namespace mdlbm

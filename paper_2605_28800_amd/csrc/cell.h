// Per-cell parts of the method shared by the update kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace tdgl {

template <typename T>
__device__ __forceinline__ T landau_dfdp(const T p[3], const T sq[3], const T *cf, int i)
{
    const int j = i == 0 ? 1 : 0;
    const int k = i == 2 ? 1 : 2;
    const T sj = sq[j] + sq[k];
    const T s4 = sq[j] * sq[j] + sq[k] * sq[k];
    // d/dP_i of eq 3 (cf: a1x a1y a1z a11 a12 a111 a112 a123)
    return p[i] * (T(2) * cf[i] + T(4) * cf[3] * sq[i] + T(2) * cf[4] * sj +
                   T(6) * cf[5] * sq[i] * sq[i] + cf[6] * (T(4) * sq[i] * sj + T(2) * s4) +
                   T(2) * cf[7] * sq[j] * sq[k]);
}

template <typename T>
__device__ __forceinline__ T landau_f(const T sq[3], const T *cf)
{
    const T x = sq[0], y = sq[1], z = sq[2];
    return cf[0] * x + cf[1] * y + cf[2] * z + cf[3] * (x * x + y * y + z * z) +
           cf[4] * (x * y + y * z + z * x) + cf[5] * (x * x * x + y * y * y + z * z * z) +
           cf[6] * (x * x * (y + z) + y * y * (x + z) + z * z * (x + y)) + cf[7] * x * y * z;
}

// One component's part of the RK45 error measure: |err| over the tolerance scale.
// An error that is not a number counts as infinite, so that the maxima over
// cells and groups, which drop NaN, keep it and the attempt fails; no error at
// all counts as zero whatever the scale (vacuum cells with an absolute
// tolerance of 0).
template <typename T>
__device__ __forceinline__ T rk_scaled(T err, T scale)
{
    const T r = fabs(err) / scale;
    return err == T(0) ? T(0) : (r == r ? r : T(INFINITY));
}

// Dormand-Prince 5(4) tableau (Dormand & Prince 1980): row s of RK_A gives
// the weights of k_1..k_s for the stage point s + 1 (row 6 is the
// fifth-order solution); RK_E = fifth- minus fourth-order weights.
static __constant__ double RK_A[6][6] = {
    {1.0 / 5, 0, 0, 0, 0, 0},
    {3.0 / 40, 9.0 / 40, 0, 0, 0, 0},
    {44.0 / 45, -56.0 / 15, 32.0 / 9, 0, 0, 0},
    {19372.0 / 6561, -25360.0 / 2187, 64448.0 / 6561, -212.0 / 729, 0, 0},
    {9017.0 / 3168, -355.0 / 33, 46732.0 / 5247, 49.0 / 176, -5103.0 / 18656, 0},
    {35.0 / 384, 0, 500.0 / 1113, 125.0 / 192, -2187.0 / 6784, 11.0 / 84}};
static __constant__ double RK_E[7] = {35.0 / 384 - 5179.0 / 57600, 0, 500.0 / 1113 - 7571.0 / 16695,
                               125.0 / 192 - 393.0 / 640, -2187.0 / 6784 + 92097.0 / 339200,
                               11.0 / 84 - 187.0 / 2100, -1.0 / 40};

}  // namespace tdgl

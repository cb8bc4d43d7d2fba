// Scalar rules of the fused BiCGSTAB iteration, shared by its separate kernels (linalg.hip)
// and the one-kernel solve (krylov_resident.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace fem {

// Finite-precision safeguards of the fused BiCGSTAB, for FP32 vectors.  Omega limit:
// when t and s are nearly orthogonal (|(t, s)| < Omega |t| |s|), omega = (t, s) / (t, t)
// is scaled up by Omega / cos(t, s), which keeps the BiCG coefficients of the next
// steps accurate (Sleijpen and van der Vorst's 'limited omega', Omega = 0.7).  Restart
// floor: see bicg_rho_floor.  Measured on the 5-step 100^3 and 200x100x100 neo-Hookean
// solves: FP32 sweeps without the floor diverged on the larger one; the limit cut its
// FP32 iterations by a third (27,704 against 41,951) but cost the FP64 vectors 48% more
// (23,236 against 15,705), so FP64 runs plain BiCGSTAB.
constexpr double kOmegaLimitF32 = 0.7;
constexpr double kRhoFloorF32 = 1e-5;

template <typename T>
__device__ __forceinline__ double bicg_omega_limit() { return sizeof(T) == 4 ? kOmegaLimitF32 : 0.0; }

struct BicgStart {
    double rho, r2, rh2, rmin2;
    bool nan, conv, div, restart;
};

// Restart floor of |(rhat, r)| / (|rhat| |r|): below it the shadow inner product has
// lost its meaning.  In FP32 the vectors carry relative errors near 1e-7 that grow over
// long solves, so the floor sits well above that noise; FP64 keeps the classic 1e-9.
template <typename T>
__device__ __forceinline__ double bicg_rho_floor() { return sizeof(T) == 4 ? kRhoFloorF32 : 1e-9; }

// Tests at the start of an iteration from the sums tot = ((rhat, r), |r|^2), the shadow
// residual's |rhat|^2, the smallest |r|^2 so far and omega of the iteration before: the
// same rules as the unfused finalize.
__device__ __forceinline__ BicgStart bicg_start(const double tot[2], double tol2, double bnorm2, double rh2,
                                                double rmin2, double omega, double rho_floor) {
    BicgStart b;
    b.r2 = tot[1];
    b.nan = !isfinite(tot[0]) || !isfinite(tot[1]);
    b.conv = !b.nan && tot[1] <= tol2;
    b.div = !b.nan && !b.conv && tot[1] > 1e12 * bnorm2;
    // (rhat, r) lost its size relative to |rhat||r|, omega vanished, or the residual
    // grew 1000x above its best value: restart from the current r
    b.restart = !(fabs(tot[0]) > rho_floor * sqrt(rh2 * tot[1])) || omega == 0.0 || tot[1] > 1e6 * rmin2;
    b.rho = b.restart ? tot[1] : tot[0];
    b.rh2 = b.restart ? tot[1] : rh2;
    b.rmin2 = fmin(rmin2, tot[1]);
    return b;
}

// omega from the sums (t, s), (t, t), (s, s)
template <typename T>
__device__ __forceinline__ double bicg_omega(const double tot[3]) {
    double omega = (tot[1] > 0.0 && isfinite(tot[1])) ? tot[0] / tot[1] : 0.0;
    const double om_lim = bicg_omega_limit<T>();
    if (om_lim > 0.0 && omega != 0.0 && tot[2] > 0.0) {
        const double c = fabs(tot[0]) / sqrt(tot[1] * tot[2]);
        if (c < om_lim) omega *= om_lim / c;
    }
    return omega;
}

}  // namespace fem

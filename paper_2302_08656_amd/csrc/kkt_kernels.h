// Device-side types shared by the kernels and the runtime of the KKT library.
#pragma once

#include <cmath>
#include <cstdint>

#include "kkt_internal.h"

namespace kkt {

constexpr int kFlagNonfinite = 1;
constexpr int kFlagInternal = 2;    // a schedule invariant failed on the device
constexpr int kCountSlots = 1024;   // spread counter for replaced pivots

// Scalars written by the kernels and read back by the host.
struct DevStatus {
    double anorm_scaled;          // ||R A C||_inf of the last refactorization
    double anorm;                 // ||A||_inf of the last refactorization (same order)
    unsigned long long perturbed; // pivots replaced by the last refactorization
    int flags;                    // kFlagNonfinite
    int abort;                    // a persistent solve timed out waiting (sticky until refactor)
};

// Infinity norms of the last residual evaluation, read back by the host.
struct ResNorms {
    double rnorm, xnorm, bnorm;
};

// What one recorded step reports to the host.
struct StepReport {
    DevStatus st;
    ResNorms rn;
};

// ||b - A x|| / (||A|| ||x|| + ||b||) from the norms read back; *den: its denominator
inline double backward_error(const DevStatus &st, const ResNorms &rn, double *den) {
    *den = st.anorm * rn.xnorm + rn.bnorm;
    if (*den == 0.0) return rn.rnorm == 0.0 ? 0.0 : INFINITY;
    return rn.rnorm / *den;
}

// What info says of a system that ended with the error rc, unless it says so already.
inline void info_error(int rc, int64_t perturbed, kkt_info *info) {
    if (info->status >= 0) *info = kkt_info{0, rc, INFINITY, perturbed};
}

// info after the first solve of a system, from its status and residual norms; returns KKT_OK
// when x has reached the target, KKT_WARN_NOT_CONVERGED when FGMRES steps are to follow, and
// KKT_ERR_DEVICE when a wait of the solve timed out (x is then invalid).
inline int first_info(const DevStatus &st, const ResNorms &rn, double berr_tol, kkt_info *info) {
    const int64_t perturbed = (int64_t)st.perturbed;
    *info = kkt_info{0, KKT_OK, 0.0, perturbed};
    if (st.abort) {
        info_error(KKT_ERR_DEVICE, perturbed, info);
        return KKT_ERR_DEVICE;
    }
    double den;
    info->berr = backward_error(st, rn, &den);
    return info->berr <= berr_tol ? KKT_OK : KKT_WARN_NOT_CONVERGED;
}

}  // namespace kkt

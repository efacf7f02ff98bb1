// Host-only driver: what kkt_info says after the first solve of a system (kkt_kernels.h).
// Reads "abort anorm rnorm xnorm bnorm perturbed tol" lines and prints
// "return iters status berr perturbed".
#include <cstdio>

#include "../paper_2302_08656_amd/csrc/kkt_kernels.h"

int main() {
    int abort_flag;
    double anorm, rnorm, xnorm, bnorm, tol;
    long long perturbed;
    while (std::scanf("%d %lf %lf %lf %lf %lld %lf", &abort_flag, &anorm, &rnorm, &xnorm, &bnorm, &perturbed, &tol) == 7) {
        kkt::DevStatus st{1.0, anorm, (unsigned long long)perturbed, 0, abort_flag};
        kkt_info info{7, 7, 7.0, 7};
        const int rc = kkt::first_info(st, kkt::ResNorms{rnorm, xnorm, bnorm}, tol, &info);
        std::printf("%d %d %d %.17g %lld\n", rc, info.iters, info.status, info.berr, (long long)info.perturbed_pivots);
        // an error of a later step stands in info, one that stands there already is kept
        kkt::info_error(KKT_ERR_DEVICE, 3, &info);
        kkt::info_error(KKT_ERR_STATE, 4, &info);
        std::printf("%d %.17g %lld\n", info.status, info.berr, (long long)info.perturbed_pivots);
    }
    return 0;
}

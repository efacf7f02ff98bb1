// Host-only driver: the levels of the refactorization schedule of one matrix (binary file as for
// sanitize_driver.cpp).  Prints a line per level: wide items, medium ones among them, narrow
// items, tiny ones among them, whether medium items run on wavefronts, most rows of a source or
// factored panel of the wide items.
#include <algorithm>
#include <cstdio>
#include <cstdint>
#include <vector>

#include "../paper_2302_08656_amd/csrc/kkt_internal.h"

int main(int argc, char **argv) {
    if (argc != 2) return 2;
    FILE *f = std::fopen(argv[1], "rb");
    if (!f) return 2;
    int32_t n = 0;
    int64_t nnz = 0;
    kkt_opts o{};
    bool ok = std::fread(&n, 4, 1, f) == 1 && std::fread(&nnz, 8, 1, f) == 1 && std::fread(&o.pivot_tau, 8, 1, f) == 1;
    if (!ok || n < 0 || nnz < 0) return 2;
    std::vector<int64_t> rowptr(n + 1);
    std::vector<int32_t> colind(nnz);
    std::vector<double> vals(nnz);
    ok = std::fread(rowptr.data(), 8, n + 1, f) == (size_t)(n + 1) &&
         std::fread(colind.data(), 4, nnz, f) == (size_t)nnz && std::fread(vals.data(), 8, nnz, f) == (size_t)nnz;
    std::fclose(f);
    if (!ok) return 2;
    o.equilibrate = 1;
    o.gmres_restart = 30;
    o.sn_max_width = 256;
    kkt::Symbolic s;
    kkt::Schedule g;
    if (kkt::analyze_symbolic(n, rowptr.data(), colind.data(), vals.data(), o, s) != KKT_OK ||
        kkt::build_schedule(s, kkt::SchedParams{}, g) != KKT_OK)
        return 1;
    for (size_t l = 0; l + 1 < g.f_lvl.size(); ++l) {
        int32_t rows = 0;
        for (int32_t it = g.f_lvl[l]; it < g.f_lvl[l] + g.f_nlarge[l]; ++it) {
            const int32_t P = g.f_item_panel[it];
            if (P >= 0) rows = std::max(rows, g.pan_start[P + 1] - g.pan_start[P] + g.pan_r[P]);
            for (int32_t q = g.f_item_pair[it]; q < g.f_item_pair[it + 1]; ++q)
                rows = std::max(rows, g.pan_r[g.f_pair_src[q]]);
        }
        std::printf("%d %d %d %d %d %d\n", g.f_nlarge[l], g.f_nmed[l], g.f_lvl[l + 1] - g.f_lvl[l] - g.f_nlarge[l],
                    g.f_ntiny[l], g.f_wave[l], rows);
    }
    return 0;
}

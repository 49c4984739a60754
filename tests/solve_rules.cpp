// The rules that choose a 2D launch's kernel, for a host-only plan: prints the
// wavefronts per 16-row tile of the M problems, the R and L problems and the map
// chains.  Arguments: n b gamma precision sequential.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "asp_internal.h"

int main(int, char** v) {
    const int n = std::atoi(v[1]);
    std::vector<double> c((size_t)n * n, 1.0);
    asp_opts o;
    asp_default_opts(&o);
    o.host_only = 1;
    o.prec = std::atoi(v[4]);
    o.sweep2d = std::atoi(v[5]) ? ASP_SWEEP2D_SEQUENTIAL : ASP_SWEEP2D_MAPS;
    asp_plan* P = nullptr;
    if (asp_setup(&P, 2, c.data(), 1.0, n, std::atoi(v[2]), std::atoi(v[3]), &o) != ASP_OK) return 1;
    std::printf("%d %d %d\n", solve_wavefronts(P, IN_GRID), solve_wavefronts(P, IN_BOUNDARY),
                solve_wavefronts(P, IN_TWIST));
    asp_destroy(P);
    return 0;
}

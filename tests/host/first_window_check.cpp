// Host-side check of first_residual_window.  Reads "lx ly lz lt t0 one have_x" lines, prints the
// window's first site and number of sites (0: every site).
#include <cstdio>

#include "../../paper_2510_26313_amd/csrc/laph_internal.h"

int main() {
    int lx, ly, lz, lt, t0, one, have_x;
    while (std::scanf("%d %d %d %d %d %d %d", &lx, &ly, &lz, &lt, &t0, &one, &have_x) == 7) {
        laph::Geom g{};
        g.lx = lx;
        g.ly = ly;
        g.lz = lz;
        g.lt = lt;
        g.lxh = lx / 2;
        g.vs_h = lx * ly * lz / 2;
        g.vh = g.vs_h * lt;
        const laph::SiteWindow w = laph::first_residual_window(g, one, t0, have_x);
        std::printf("%d %d\n", w.lo, w.n);
    }
    return 0;
}

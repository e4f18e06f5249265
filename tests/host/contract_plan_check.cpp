// Reads "lx ly lz lt nev n herm n_left" lines, prints whether the doublets of n momenta of one
// (px, py) go by planes.
#include <cstdio>

#include "../../paper_2510_26313_amd/csrc/contract_plan.h"

int main() {
    int lx, ly, lz, lt, nev, n, herm, left;
    while (std::scanf("%d %d %d %d %d %d %d %d", &lx, &ly, &lz, &lt, &nev, &n, &herm, &left) == 8)
        std::printf("%d\n", (int)laph::DoubletPlan{lx, ly, lz, lt, nev}.by_planes(n, herm != 0, left));
    return 0;
}

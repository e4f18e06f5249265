// Reads "lx ly lz lt nev groups", then "momenta herm" of each group; prints how many groups of doublets
// go by planes.
#include <cstdio>

#include "../../paper_2510_26313_amd/csrc/contract_plan.h"

int main() {
    int lx, ly, lz, lt, nev, n;
    while (std::scanf("%d %d %d %d %d %d", &lx, &ly, &lz, &lt, &nev, &n) == 6) {
        std::vector<std::pair<int, bool>> groups;
        for (int k = 0; k < n; ++k) {
            int m, h;
            if (std::scanf("%d %d", &m, &h) != 2) return 1;
            groups.push_back({m, h != 0});
        }
        int by = 0;
        for (char c : laph::DoubletPlan{lx, ly, lz, lt, nev}.by_planes(groups)) by += c;
        std::printf("%d\n", by);
    }
    return 0;
}

// Host-side check of window_blocks: for every window of a lattice of vh sites, the blocks it
// names are exactly those block_outside does not rule out.  Reads "vh size" lines, prints the
// number of (window, block) pairs that disagree.
#include <cstdio>

#include "../../paper_2510_26313_amd/csrc/laph_internal.h"

int main() {
    int vh, size;
    while (std::scanf("%d %d", &vh, &size) == 2) {
        const int nb = (vh + size - 1) / size;
        long bad = 0;
        for (int lo = 0; lo < vh; ++lo)
            for (int n = 0; n <= vh; ++n) {
                laph::SiteWindow w;
                w.lo = lo;
                w.n = n;
                int first = -1;
                const int cnt = laph::window_blocks(w, size, nb, vh, &first);
                for (int b = 0; b < nb; ++b) {
                    const int h0 = b * size, len = vh - h0 < size ? vh - h0 : size;
                    int d = b - first;
                    if (d < 0) d += nb;
                    bad += (d < cnt) == laph::block_outside(w, h0, len, vh);
                }
            }
        std::printf("%ld\n", bad);
    }
    return 0;
}

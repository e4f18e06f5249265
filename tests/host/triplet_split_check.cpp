// Reads "base nchunk" lines, prints the K slices of a launch of triplets.
#include <cstdio>

#include "../../paper_2510_26313_amd/csrc/contract_plan.h"

int main() {
    int base, nchunk;
    while (std::scanf("%d %d", &base, &nchunk) == 2) std::printf("%d\n", laph::triplet_split(base, nchunk));
    return 0;
}

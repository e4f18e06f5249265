// How the doublets' momenta are launched: estimates of both ways, in seconds, for the rule that
// chooses between them (host code without HIP, so a test can hold it against measurements).
#pragma once

#include <algorithm>

namespace laph {

constexpr int kPlanSites = 8;       // sites per K chunk
constexpr int kPlanMaxMom = 16;     // momenta per launch of the full-phase products
constexpr int kPlanTarget = 2048;   // workgroups aimed for by their K split
constexpr int kPlanMaxSplit = 64;
constexpr int kPlanPlaneMom = 8;    // momenta per launch that sums planes

// K slices of a launch whose (t, column tile, momentum) workgroups number `base`
inline int plan_split(int base, int nchunk) {
    return std::max(1, std::min({(kPlanTarget + base - 1) / base, nchunk, kPlanMaxSplit}));
}

// The same for triplets, with at least 4 chunks a slice (and 4 slices where there are chunks): a
// slice's entry is written once and read for six orderings, which takes about what the products
// of 4 chunks on it take.  8^4 (64 chunks), 33 and 48 vectors, two and one momenta: 262 and 352 us with
// a chunk a slice, 116 and 156 now; 4^4 (8 chunks) is fastest with 4 slices, 12^3 x 24 and above as before.
inline int triplet_split(int base, int nchunk) {
    return plan_split(base, std::max(std::min(nchunk, 4), nchunk / 4));
}

// Products at 50 TFLOP/s, slices or planes written and read at 5 TB/s, 20 us a launch: with these
// no group of 1 to 8 momenta on 40 lattices from 8^4 to 32^3 x 64, nev 4 to 64, was sent the way that
// was more than 3 % slower than the whole phase.
struct DoubletPlan {
    int lx, ly, lz, lt, nev;
    static constexpr double kRate = 50e12, kBytes = 5e12, kLaunch = 20e-6;
    static constexpr int kCUs = 256;

    // flops of the products on `sites` sites of one timeslice: a workgroup has a wave for every 16
    // columns, so up to 64 columns take the time of 64
    double flops(double sites) const { return 8.0 * 3 * sites * 64 * 16 * ((nev + 15) / 16); }
    // the matrices of n K slices, written and read
    double slices(double n) const { return n * nev * nev * 32 / kBytes; }

    // n momenta with the whole phase in their products
    double whole(int n) const {
        const int vs = lx * ly * lz;
        double s = 0;
        for (; n > 0; n -= kPlanMaxMom) {
            const int base = lt * std::min(n, kPlanMaxMom);
            s += kLaunch + base * flops(vs) / kRate +
                 slices((double)base * plan_split(base, (vs + kPlanSites - 1) / kPlanSites));
        }
        return s;
    }
    // n momenta of one (px, py) by planes: a workgroup for each z and t, so that the time goes in
    // whole workgroups of the fullest CU (one alone takes 1.2 times its share) and a lattice with few
    // planes leaves CUs idle (48^2 x 4 x 4, two momenta, nev 64: 1344 us on 16 workgroups, 184 with the
    // whole phase).  A Hermitian S(z) has 10 of 16 blocks, but one of a workgroup's waves runs all
    // four rows: it gains where a CU holds several workgroups, and then 15 %.
    double planes(int n, bool herm) const {
        const int wgs = lz * lt, per_cu = (wgs + kCUs - 1) / kCUs;
        const int chunks = (lx * ly + kPlanSites - 1) / kPlanSites;
        const double unit = flops((double)chunks * kPlanSites) / (kRate / kCUs);
        return kLaunch * (1 + (n + kPlanPlaneMom - 1) / kPlanPlaneMom) +
               unit * (wgs <= kCUs ? 1.2 : herm ? 0.85 * per_cu : per_cu) + slices(wgs);
    }
    // whether n of the n_left momenta still to be launched go by planes.  Planes below 64 sites cost
    // less than writing and reading their S(z) five times: not considered.
    bool by_planes(int n, bool herm, int n_left) const {
        return lx * ly >= 64 && planes(n, herm) + whole(n_left - n) < whole(n_left);
    }
};

}  // namespace laph

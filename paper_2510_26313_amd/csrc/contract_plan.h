// How the doublets' momenta are launched: estimates of both ways, in seconds, for the rule that
// chooses between them (host code without HIP, so a test can hold it against measurements).
#pragma once

#include <algorithm>
#include <numeric>
#include <utility>
#include <vector>

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

// The figures are fits to times on 40 lattices from 8^4 to 32^3 x 64, nev 4 to 64, 1 to 8 momenta of one
// (px, py), both ways: the estimates are within 10 %, and none of 1409 groups was sent the way that was
// more than 3 % slower than the whole phase.
struct DoubletPlan {
    int lx, ly, lz, lt, nev;
    static constexpr int kCUs = 256;

    // seconds of wgs workgroups of `chunks` chunks.  A workgroup has a wave for each 16 columns, which
    // runs all 16-blocks of rows, so a chunk takes a time that grows with the number of blocks; alone on a
    // CU it also waits for its loads.  The time goes in whole workgroups of the fullest CU.  A Hermitian
    // product of several blocks has 10 of 16 (nev 64), but one of its waves runs all rows: 12 % less
    // where a CU holds several workgroups.  Then the matrices are written and read at 6 TB/s.
    double products(int wgs, int chunks, bool herm) const {
        const int blocks = (nev + 15) / 16, per_cu = (wgs + kCUs - 1) / kCUs;
        const double us = per_cu == 1 ? 1.45 + 0.8 * blocks
                                      : per_cu * (0.3 + 0.9 * blocks) * (herm && blocks > 1 ? 0.88 : 1.0);
        return chunks * us * 1e-6 + (double)wgs * nev * nev * 32 / 6e12;
    }
    static constexpr double kLaunch = 13e-6;
    // n momenta with the whole phase in their products
    double whole(int n) const {
        const int nchunk = (lx * ly * lz + kPlanSites - 1) / kPlanSites;
        double s = 0;
        for (; n > 0; n -= kPlanMaxMom) {
            const int base = lt * std::min(n, kPlanMaxMom), split = plan_split(base, nchunk);
            s += kLaunch + products(base * split, (nchunk + split - 1) / split, false);
        }
        return s;
    }
    // n momenta of one (px, py) by planes: a workgroup for each z and t, so a lattice with few
    // planes leaves CUs idle (48^2 x 4 x 4, two momenta, nev 64: 1344 us on 16 workgroups, 184 with the
    // whole phase)
    double planes(int n, bool herm) const {
        return kLaunch * (1 + (n + kPlanPlaneMom - 1) / kPlanPlaneMom) +
               products(lz * lt, (lx * ly + kPlanSites - 1) / kPlanSites, herm);
    }
    // which groups (momenta, Hermitian) go by planes: the cheapest per momentum first, as many as make
    // the total least.  Planes below 64 sites cost less than writing and reading their S(z) five times: not
    // considered.
    std::vector<char> by_planes(const std::vector<std::pair<int, bool>> &groups) const {
        std::vector<char> by(groups.size(), 0);
        if (lx * ly < 64) return by;
        std::vector<double> cost;
        int left = 0;
        for (const auto &g : groups) {
            cost.push_back(planes(g.first, g.second));
            left += g.first;
        }
        std::vector<size_t> order(groups.size());
        std::iota(order.begin(), order.end(), size_t(0));
        std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) {
            return cost[a] * groups[b].first < cost[b] * groups[a].first;
        });
        double spent = 0, best = whole(left);
        size_t take = 0;
        for (size_t k = 0; k < order.size(); ++k) {
            spent += cost[order[k]];
            left -= groups[order[k]].first;
            if (spent + whole(left) < best) {
                best = spent + whole(left);
                take = k + 1;
            }
        }
        for (size_t k = 0; k < take; ++k) by[order[k]] = 1;
        return by;
    }
};

}  // namespace laph

// Meson doublets and baryon triplets of the LapH vectors (Sec. "QUDA": besides
// sourcing the solves and projecting the propagators, the LapH vectors form the
// quark-antiquark doublets and three-quark triplets that enter the Wick
// contractions of meson and baryon correlators).  Per timeslice t and momentum
// p = 2 pi (nx / Lx, ny / Ly, nz / Lz):
//
//   Phi_p[t][l][m]   = sum_x e^{-i p.x} sum_a conj(V_l(x, t)_a) V_m(x, t)_a
//   B_p[t][l][m][n]  = sum_x e^{-i p.x} eps_abc V_l(x, t)_a V_m(x, t)_b V_n(x, t)_c
//
// Both are complex FP64 GEMMs per (t, p) over K = (site, colour), 3 Lx Ly Lz long:
//   doublets  A[l][(x, a)] = e^{-i p.x} conj(V_l(x)_a),  B[(x, a)][m]      = V_m(x)_a
//   triplets  A[l][(x, a)] = e^{-i p.x} V_l(x)_a,        B[(x, a)][(m, n)] = (V_m(x) x V_n(x))_a
// where the triplet's B column is the colour cross product of a pair m < n.  A
// workgroup stages the V of a chunk of sites (all nev vectors) in LDS with the
// direct global-to-LDS loads, two chunks deep, so the next chunk arrives while the
// matrix cores work on the current one; each wave forms its A and B fragments from
// LDS (the cross products are never stored).  B_p is antisymmetric in every index pair, so
// each set of three indices is accumulated once (see PairTable), and the reduction writes
// all six orderings with their signs and zeros where an index repeats.  K is split over
// workgroups for occupancy; the reduction sums the slices in a fixed order.
//
// Doublets of several momenta share their products: with p.x = (px x + py y) + pz z the
// momenta of one (px, py) -- up to an overall sign, which conjugates and transposes --
// need one product per z plane, S(z)[l][m] = sum_xy e^{-i (px x + py y)} conj(V_l) V_m,
// and differ only in the phases their planes are summed with.  For (px, py) = -(px, py)
// S(z) is Hermitian and only the 16x16 blocks on and above its diagonal are formed.
#include <algorithm>
#include <cmath>
#include <vector>

#include "contract_plan.h"
#include "laph_solver.h"

namespace laph {

namespace {

constexpr int kCB = 256;          // threads per workgroup (4 waves)
constexpr int kCS = kPlanSites;   // sites per K chunk
constexpr int kCK = 3 * kCS;      // K (site, colour) per chunk
constexpr int kRS = kCK + 1;      // LDS row stride in complex (odd: conflict-free fragment reads)
constexpr int kSlots = 64 * kRS;  // complex slots of one staged chunk (64 rows)
constexpr int kCRows = 64;        // l rows: nev <= 64
constexpr int kCMaxMom = kPlanMaxMom;   // momenta per launch

typedef double d4 __attribute__((ext_vector_type(4)));

struct ContractArgs {
    int lx, ly, lz, lt, vs;
    int nev;
    int ncol;             // doublets: nev; triplets: columns of the PairTable
    int ntile;            // column tiles per (t, p)
    int nsplit;           // K slices
    int nchunk;           // K chunks of kCS sites
    int nmom;
    int mom[3 * kCMaxMom];
    int out[kCMaxMom];    // index of each momentum in the result
    int plane;            // > 0: K slice = z plane of this many sites (doublets by planes), 0: even slices
    int herm;             // doublets: only the 16x16 blocks on and above the diagonal
    const double2 *V;     // [lt][nev][vs][3]
    double2 *scratch;     // [nsplit][nmom][lt][nev][ncol]
};

// Columns of the triplets.  With the indices in blocks of 16, a sorted triple a < b < c in
// blocks A <= B <= C is the product of
//   row c with the pair (a, b)  if A == B        (cyclic orders: all with sign +)
//   row a with the pair (b, c)  otherwise,
// so the pairs inside a block need every row block, the pairs of two blocks i < j the row
// blocks below i, and pairs with i = 0 are not needed at all.  Columns are listed by falling
// row count (pairs inside blocks 0, 1, ...; then pairs (i, j > i), i = nblk - 2 .. 1), so a wave runs a
// prefix of the row blocks.  Against all pairs m < n with the rows below m, as the list
// was before: nev 64 47 104 products of 16 issued for 41 664 triples instead of 58 300, and
// 1248 cross products instead of 2016.
struct PairTable {
    int nev, nblk;
    __host__ __device__ explicit PairTable(int n) : nev(n), nblk((n + 15) / 16) {}
    __host__ __device__ int width(int i) const { return i + 1 < nblk ? 16 : nev - 16 * i; }
    __host__ __device__ int inside(int i) const { return 120 * i; }   // first column of block i's pairs
    __host__ __device__ int n_inside() const { return inside(nblk - 1) + width(nblk - 1) * (width(nblk - 1) - 1) / 2; }
    // first column of the pairs (block i, later blocks)
    __host__ __device__ int across(int i) const {
        int c = n_inside();
        for (int k = nblk - 2; k > i; --k) c += 16 * (nev - 16 * (k + 1));
        return c;
    }
    __host__ __device__ int ncol() const { return across(0); }
    __host__ __device__ int col(int m, int n) const {   // m < n
        const int i = m >> 4, u = m & 15, w = width(i);
        if (i == n >> 4) return inside(i) + u * w - u * (u + 1) / 2 + (n & 15) - u - 1;
        return across(i) + u * (nev - 16 * (i + 1)) + n - 16 * (i + 1);
    }
    // the pair of a column and the row blocks it needs
    __host__ __device__ void pair(int q, int &m, int &n, int &rows) const {
        if (q < n_inside()) {
            const int i = q / 120 < nblk - 1 ? q / 120 : nblk - 1, w = width(i);
            int e = q - inside(i), u = 0;
            while (e >= w - 1 - u) e -= w - 1 - u++;
            m = 16 * i + u;
            n = m + 1 + e;
            rows = nblk;
            return;
        }
        int i = nblk - 2, e = q - n_inside();
        while (e >= 16 * (nev - 16 * (i + 1))) e -= 16 * (nev - 16 * (i-- + 1));
        const int w = nev - 16 * (i + 1);
        m = 16 * i + e / w;
        n = 16 * (i + 1) + e % w;
        rows = i;
    }
};

// One staged chunk: the wave's A fragments (R row blocks) and B fragments (NCB column
// blocks) per group of 4 K, then the R x NCB x 4 real products as straight-line code,
// each product's accumulator written by the previous group's product of the same kind
// only (independent accumulators back to back).  A row of the chunk holds K colour-major
// (colour a of site s at a kCS + s), so with the 6 groups unrolled each group's colour
// and its cross-product partners are compile-time offsets from one per-lane address.
template <int MODE, int NCB, int R>
__device__ __forceinline__ void chunk_products(const double2 *buf, const double2 *ph, int lane, const int *cm,
                                               const int *cn, d4 (*cre)[NCB], d4 (*cim)[NCB]) {
    const int q = lane >> 4;   // K within a group of 4
    const double2 *arow = buf + (lane & 15) * kRS + q;
    const double2 *bm[NCB], *bn[NCB];
#pragma unroll
    for (int j = 0; j < NCB; ++j) {
        bm[j] = buf + cm[j] * kRS + q;
        bn[j] = buf + cn[j] * kRS + q;
    }
    // the phases of the two sites this lane meets (groups start at site 0 or 4)
    const double2 f0 = ph[q], f1 = ph[q + 4];
#pragma unroll
    for (int k4 = 0; k4 < kCK; k4 += 4) {
        const int a = k4 / kCS, so = k4 % kCS;   // colour and site offset of the group
        const double2 f = so ? f1 : f0;
        double ar[R], ai[R], nai[R], br[NCB], bi[NCB];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const double2 v = arow[16 * i * kRS + k4];
            const double vi = MODE == 0 ? -v.y : v.y;
            ar[i] = f.x * v.x - f.y * vi;
            ai[i] = f.x * vi + f.y * v.x;
            nai[i] = -ai[i];
        }
#pragma unroll
        for (int j = 0; j < NCB; ++j) {
            if (MODE == 0) {
                const double2 v = bm[j][k4];
                br[j] = v.x;
                bi[j] = v.y;
            } else {
                // (V_m x V_n)_a = V_m,b V_n,c - V_m,c V_n,b with (a, b, c) cyclic
                const int ob = (a == 2 ? 0 : a + 1) * kCS + so, oc = (a == 0 ? 2 : a - 1) * kCS + so;
                const double2 ub = bm[j][ob], uc = bm[j][oc];
                const double2 wb = bn[j][ob], wc = bn[j][oc];
                br[j] = (ub.x * wc.x - ub.y * wc.y) - (uc.x * wb.x - uc.y * wb.y);
                bi[j] = (ub.x * wc.y + ub.y * wc.x) - (uc.x * wb.y + uc.y * wb.x);
            }
        }
        // Re += Ar Br - Ai Bi;  Im += Ar Bi + Ai Br
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < NCB; ++j) {
                cre[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[i], br[j], cre[i][j], 0, 0, 0);
                cim[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[i], bi[j], cim[i][j], 0, 0, 0);
            }
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < NCB; ++j) {
                cre[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(nai[i], bi[j], cre[i][j], 0, 0, 0);
                cim[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai[i], br[j], cim[i][j], 0, 0, 0);
            }
        // keep each group's LDS reads with its products (hoisting them all costs occupancy)
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int MODE, int NCB>
__device__ __forceinline__ void chunk_dispatch(int nact, const double2 *buf, const double2 *ph, int lane,
                                               const int *cm, const int *cn, d4 (*cre)[NCB], d4 (*cim)[NCB]) {
    switch (nact) {
        case 4: chunk_products<MODE, NCB, 4>(buf, ph, lane, cm, cn, cre, cim); break;
        case 3: chunk_products<MODE, NCB, 3>(buf, ph, lane, cm, cn, cre, cim); break;
        case 2: chunk_products<MODE, NCB, 2>(buf, ph, lane, cm, cn, cre, cim); break;
        case 1: chunk_products<MODE, NCB, 1>(buf, ph, lane, cm, cn, cre, cim); break;
        default: break;
    }
}

// Copy chunk s0 of every vector (64 rows, nev real) into LDS with the direct
// global-to-LDS loads: lane i of load q fills slot 64 q + i of the buffer, so each
// lane fetches the element that lands in its slot (which also reorders a row's K to
// colour-major).  Pad slots and rows or sites
// outside the data load the timeslice's first element (finite; the zero phase of a
// site outside the lattice cancels it, and pad slots and rows past nev are not read
// into any kept product).
__device__ __forceinline__ void stage_chunk(double2 *buf, const double2 *Vt, int nev, int n3, int s0, int wave,
                                            int lane) {
    for (int q = wave; q < kSlots / 64; q += 4) {
        const int e = 64 * q + lane;
        const int row = e / kRS, col = e - row * kRS;
        const int a = col / kCS, sl = col - a * kCS;   // colour-major within the row
        const double2 *src = Vt;
        if (col < kCK && row < nev && 3 * (s0 + sl) < n3) src = Vt + (size_t)row * n3 + 3 * (s0 + sl) + a;
        __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)(buf + 64 * q), 16, 0, 0);
    }
}

// NCB column blocks of 16 per wave: 4 NCB 16 columns per workgroup
template <int MODE, int NCB>
__global__ __launch_bounds__(kCB) void contract_kernel(ContractArgs A) {
    // two staged chunks: the next one is in flight while the products run on the other
    __shared__ double2 bufA[kSlots], bufB[kSlots];
    __shared__ double2 phA[kCS], phB[kCS];
    // workgroups that share a K slice of one timeslice run on one XCD (consecutive
    // workgroup ids go round-robin over the 8 XCDs)
    const int nb = gridDim.x;
    int bid = blockIdx.x;
    if (nb % 8 == 0) bid = (bid % 8) * (nb / 8) + bid / 8;
    const int inner = A.ntile * A.nmom;
    const int tile = bid % A.ntile;
    const int p = (bid / A.ntile) % A.nmom;
    const int outer = bid / inner;
    const int split = outer % A.nsplit;
    const int t = outer / A.nsplit;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int kCols = 4 * NCB * 16;
    const int nev = A.nev;

    // this lane's column per block, the pair behind it, and the number of 16-row
    // blocks the wave needs (wave-uniform)
    int col[NCB], cm[NCB], cn[NCB];
    int nact = 0;
    // with half of a Hermitian block row to do, the waves take the columns in turn, so that
    // the workgroups sharing a CU load its SIMDs evenly
    const int wcol = MODE == 0 && A.herm ? (wave + bid) & 3 : wave;
#pragma unroll
    for (int j = 0; j < NCB; ++j) {
        const int c0 = tile * kCols + (wcol * NCB + j) * 16;
        col[j] = c0 + (lane & 15);
        cm[j] = 0;
        cn[j] = 0;
        if (c0 >= A.ncol) continue;   // a block past the last column: zero B (V_0 x V_0, or column 0 unread)
        if (MODE == 1) {
            const PairTable pt(nev);
            int rows;
            if (col[j] < A.ncol) pt.pair(col[j], cm[j], cn[j], rows);
            int m0, n0;
            pt.pair(c0, m0, n0, rows);   // the block's first column needs the most rows
            nact = max(nact, rows);
        } else {
            cm[j] = col[j] < A.ncol ? col[j] : 0;
            nact = A.herm ? wcol + 1 : (nev + 15) / 16;
        }
    }

    d4 cre[4][NCB], cim[4][NCB];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NCB; ++j) {
            cre[i][j] = d4{0, 0, 0, 0};
            cim[i][j] = d4{0, 0, 0, 0};
        }
    const int mx = A.mom[3 * p], my = A.mom[3 * p + 1], mz = A.mom[3 * p + 2];
    const int ch0 = A.plane ? 0 : (int)((long)A.nchunk * split / A.nsplit);
    const int ch1 = A.plane ? A.nchunk : (int)((long)A.nchunk * (split + 1) / A.nsplit);
    const int first = A.plane * split, end = A.plane ? first + A.plane : A.vs;   // sites of this slice
    const double2 *Vt = A.V + (size_t)t * nev * A.vs * 3;
    const int n3 = 3 * A.vs;
    // e^{-2 pi i (nx x / Lx + ny y / Ly + nz z / Lz)} of the chunk's sites, integer parts
    // reduced first; zero for sites past the slice
    auto phases = [&](double2 *ph, int s0) {
        if (tid < kCS) {
            const int s = s0 + tid;
            double2 v = make_double2(0.0, 0.0);
            if (s < end) {
                const int x = s % A.lx, y = (s / A.lx) % A.ly, z = s / (A.lx * A.ly);
                const int qx = ((mx * x) % A.lx + A.lx) % A.lx;
                const int qy = ((my * y) % A.ly + A.ly) % A.ly;
                const int qz = ((mz * z) % A.lz + A.lz) % A.lz;
                const double f = (double)qx / A.lx + (double)qy / A.ly + (double)qz / A.lz;
                sincospi(-2.0 * f, &v.y, &v.x);
            }
            ph[tid] = v;
        }
    };
    if (ch0 < ch1) {
        stage_chunk(bufA, Vt, nev, n3, first + ch0 * kCS, wave, lane);
        phases(phA, first + ch0 * kCS);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    for (int ch = ch0; ch < ch1; ch += 2) {
        if (ch + 1 < ch1) {
            stage_chunk(bufB, Vt, nev, n3, first + (ch + 1) * kCS, wave, lane);
            phases(phB, first + (ch + 1) * kCS);
        }
        chunk_dispatch<MODE, NCB>(nact, bufA, phA, lane, cm, cn, cre, cim);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (ch + 1 >= ch1) break;
        if (ch + 2 < ch1) {
            stage_chunk(bufA, Vt, nev, n3, first + (ch + 2) * kCS, wave, lane);
            phases(phA, first + (ch + 2) * kCS);
        }
        chunk_dispatch<MODE, NCB>(nact, bufB, phB, lane, cm, cn, cre, cim);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }
    // v_mfma_f64_16x16x4f64 leaves C[row][col] of a 16 x 16 block in lane col + 16 (row % 4),
    // register row / 4 (a lane holds rows lane / 16 + 4 r of column lane % 16)
    double2 *out = A.scratch + (((size_t)split * A.nmom + p) * A.lt + t) * (size_t)nev * A.ncol;
#pragma unroll
    for (int j = 0; j < NCB; ++j) {
        if (col[j] >= A.ncol) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * i + (lane >> 4) + 4 * r;
                if (row < nev) out[(size_t)row * A.ncol + col[j]] = make_double2(cre[i][j][r], cim[i][j][r]);
            }
    }
}

// Phi[p][t][l][m] = sum over K slices
__global__ void doublet_reduce_kernel(ContractArgs A, double2 *phi) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    const long per = (long)A.lt * A.nev * A.nev;
    if (idx >= per * A.nmom) return;
    const int p = (int)(idx / per);
    const long r = idx - p * per;
    double2 s = make_double2(0.0, 0.0);
    for (int sp = 0; sp < A.nsplit; ++sp) {
        const double2 v = A.scratch[((size_t)sp * A.nmom + p) * per + r];
        s.x += v.x;
        s.y += v.y;
    }
    phi[(size_t)A.out[p] * per + r] = s;
}

// B[p][t][l][m][n]: the sum over K slices of the sorted triple's entry, with the
// sign of the permutation that sorts (l, m, n); zero when two indices coincide
__global__ void triplet_reduce_kernel(ContractArgs A, double2 *B) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    const int nev = A.nev;
    const long per = (long)A.lt * nev * nev * nev;
    if (idx >= per * A.nmom) return;
    const int p = (int)(idx / per);
    long r = idx - p * per;
    const int n = (int)(r % nev);
    const int m = (int)((r / nev) % nev);
    const int l = (int)((r / ((long)nev * nev)) % nev);
    const int t = (int)(r / ((long)nev * nev * nev));
    double2 s = make_double2(0.0, 0.0);
    if (l != m && m != n && l != n) {
        int a = l, b = m, c = n;
        double sg = 1.0;
        if (a > b) { int q = a; a = b; b = q; sg = -sg; }
        if (b > c) { int q = b; b = c; c = q; sg = -sg; }
        if (a > b) { int q = a; a = b; b = q; sg = -sg; }
        const PairTable pt(nev);
        const bool low = a >> 4 == b >> 4;   // (a, b) in one block: row c, else row a
        const int q = low ? pt.col(a, b) : pt.col(b, c), row = low ? c : a;
        for (int sp = 0; sp < A.nsplit; ++sp) {
            const double2 v = A.scratch[((((size_t)sp * A.nmom + p) * A.lt + t) * nev + row) * A.ncol + q];
            s.x += v.x;
            s.y += v.y;
        }
        s.x *= sg;
        s.y *= sg;
    }
    B[(size_t)A.out[p] * per + r] = s;
}

// Doublets by planes: Phi of up to kPlaneMom momenta of one (px, py) from S(z).  A member with
// flip has the opposite (px, py): Phi_p[m][l] = conj(sum_z e^{+i pz z} S(z)[l][m]).  herm: S(z)
// holds the blocks on and above the diagonal and its other half follows the same way.
constexpr int kPlaneMom = kPlanPlaneMom;
constexpr int kPlaneZ = 128;   // phases kept in LDS

struct PlaneArgs {
    int lt, lz, nev, n, herm;
    int mz[kPlaneMom], flip[kPlaneMom], out[kPlaneMom];
    const double2 *S;     // [lz][lt][nev][nev]
    double2 *phi;         // [momenta][lt][nev][nev]
};

template <int NM>
__global__ __launch_bounds__(256) void doublet_planes_kernel(PlaneArgs A) {
    __shared__ double2 ph[NM][kPlaneZ];
    const int nev = A.nev;
    const long per = (long)A.lt * nev * nev;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    const int m = (int)(idx % nev), l = (int)((idx / nev) % nev);
    const bool live = idx < per && !(A.herm && (l >> 4) > (m >> 4));
    double2 s[NM], d[NM];   // sums with e^{-i pz z} and e^{+i pz z}
#pragma unroll
    for (int k = 0; k < NM; ++k) s[k] = d[k] = make_double2(0.0, 0.0);
    for (int z0 = 0; z0 < A.lz; z0 += kPlaneZ) {
        const int nz = min(kPlaneZ, A.lz - z0);
        __syncthreads();
        for (int e = threadIdx.x; e < NM * nz; e += 256) {
            const int k = e / nz, z = e - k * nz;
            const long q = k < A.n ? ((long)A.mz[k] * (z0 + z)) % A.lz : 0;
            sincospi(-2.0 * (double)((q + A.lz) % A.lz) / A.lz, &ph[k][z].y, &ph[k][z].x);
        }
        __syncthreads();
        if (!live) continue;
#pragma unroll 2
        for (int z = 0; z < nz; ++z) {
            const double2 v = A.S[(size_t)(z0 + z) * per + idx];
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                const double2 f = ph[k][z];
                const double a = f.x * v.x, b = f.y * v.y, c = f.x * v.y, e = f.y * v.x;
                s[k].x += a - b;
                s[k].y += c + e;
                d[k].x += a + b;
                d[k].y += c - e;
            }
        }
    }
    if (!live) return;
    const long mirror = idx + (long)(m - l) * (nev - 1);   // (t, m, l)
#pragma unroll
    for (int k = 0; k < NM; ++k) {
        if (k >= A.n) break;
        double2 *o = A.phi + (size_t)A.out[k] * per;
        if (!A.flip[k]) o[idx] = s[k];
        if (A.flip[k] || (A.herm && (l >> 4) < (m >> 4))) o[mirror] = make_double2(d[k].x, -d[k].y);
    }
}

void contract_shape(const Ctx &c, int kind, int nev, int nmom, ContractArgs &a) {
    a.lx = c.g.lx;
    a.ly = c.g.ly;
    a.lz = c.g.lz;
    a.lt = c.g.lt;
    a.vs = c.g.lx * c.g.ly * c.g.lz;
    a.nev = nev;
    a.ncol = kind == 0 ? nev : PairTable(nev).ncol();
    a.plane = a.herm = 0;
    const int cols = kind == 0 ? 64 : 128;
    a.ntile = std::max(1, (a.ncol + cols - 1) / cols);
    a.nmom = nmom;
    a.nchunk = (a.vs + kCS - 1) / kCS;
    const int base = a.lt * a.ntile * nmom;
    a.nsplit = kind == 0 ? plan_split(base, a.nchunk) : triplet_split(base, a.nchunk);
}

}  // namespace

// K-slice partials of one launch group of nmom momenta
static size_t group_bytes(const Ctx &c, int kind, int nev, int nmom) {
    ContractArgs a;
    contract_shape(c, kind, nev, nmom, a);
    return round256((size_t)a.nsplit * a.nmom * a.lt * nev * a.ncol * 16);
}

// S(z) of one group of doublets
static size_t planes_bytes(const Ctx &c, int nev) { return round256((size_t)c.g.lz * c.g.lt * nev * nev * 16); }

size_t contract_workspace_bytes(const Ctx &c, int kind, int nev, int n_mom) {
    if (nev < 1 || nev > kCRows || n_mom < 1 || (kind != 0 && kind != 1)) return 0;
    // the largest launch group: a full one, or the last (its K split may be finer)
    size_t b = group_bytes(c, kind, nev, std::min(n_mom, kCMaxMom));
    if (n_mom > kCMaxMom && n_mom % kCMaxMom) b = std::max(b, group_bytes(c, kind, nev, n_mom % kCMaxMom));
    if (kind == 0) {
        b = std::max(b, planes_bytes(c, nev));
        // what is left after some momenta went by planes may be split finer
        for (int n = 1; n < std::min(n_mom, kCMaxMom); ++n) b = std::max(b, group_bytes(c, kind, nev, n));
    }
    return b;
}

// The momenta of one (px, py), up to an overall sign.
struct PlaneGroup {
    int px, py, herm;
    std::vector<int> members, flip;
};

static std::vector<PlaneGroup> plane_groups(const Ctx &c, int n_mom, const int *mom) {
    std::vector<PlaneGroup> gs;
    auto red = [](int v, int l) { return (v % l + l) % l; };
    const int lx = c.g.lx, ly = c.g.ly;
    for (int q = 0; q < n_mom; ++q) {
        const int px = red(mom[3 * q], lx), py = red(mom[3 * q + 1], ly);
        const int nx = red(-px, lx), ny = red(-py, ly);
        size_t k = 0;
        int flip = 0;
        for (; k < gs.size(); ++k) {
            if (gs[k].px == px && gs[k].py == py) break;
            if (gs[k].px == nx && gs[k].py == ny) {
                flip = 1;
                break;
            }
        }
        if (k == gs.size()) gs.push_back({px, py, px == nx && py == ny ? 1 : 0, {}, {}});
        gs[k].members.push_back(q);
        gs[k].flip.push_back(flip);
    }
    return gs;
}

// Phi of one group's momenta through its S(z)
static laph_status doublet_planes(const Ctx &c, const PlaneGroup &g, double *out, const double *V, int nev,
                                  const int *mom, char *work) {
    ContractArgs a;
    contract_shape(c, 0, nev, 1, a);
    a.plane = a.lx * a.ly;
    a.herm = g.herm;
    a.nsplit = a.lz;
    a.nchunk = (a.plane + kCS - 1) / kCS;
    a.mom[0] = g.px;
    a.mom[1] = g.py;
    a.mom[2] = 0;
    a.V = reinterpret_cast<const double2 *>(V);
    a.scratch = reinterpret_cast<double2 *>(work);
    hipLaunchKernelGGL((contract_kernel<0, 1>), dim3((unsigned)(a.lt * a.lz)), dim3(kCB), 0, c.stream, a);
    LAPH_TRY(check_launch("contract_kernel"));
    for (size_t m0 = 0; m0 < g.members.size(); m0 += kPlaneMom) {
        PlaneArgs p;
        p.lt = a.lt;
        p.lz = a.lz;
        p.nev = nev;
        p.herm = g.herm;
        p.n = (int)std::min<size_t>(kPlaneMom, g.members.size() - m0);
        for (int k = 0; k < kPlaneMom; ++k) {
            const bool on = k < p.n;
            p.mz[k] = on ? mom[3 * g.members[m0 + k] + 2] % a.lz : 0;
            p.flip[k] = on ? g.flip[m0 + k] : 0;
            p.out[k] = on ? g.members[m0 + k] : 0;
        }
        p.S = a.scratch;
        p.phi = reinterpret_cast<double2 *>(out);
        const unsigned nb = (unsigned)(((long)a.lt * nev * nev + 255) / 256);
        if (p.n <= 2)
            hipLaunchKernelGGL(doublet_planes_kernel<2>, dim3(nb), dim3(256), 0, c.stream, p);
        else
            hipLaunchKernelGGL(doublet_planes_kernel<kPlaneMom>, dim3(nb), dim3(256), 0, c.stream, p);
        LAPH_TRY(check_launch("doublet_planes_kernel"));
    }
    return LAPH_OK;
}

laph_status contract(const Ctx &c, int kind, double *out, const double *V, int nev, int n_mom, const int *mom_host,
                     char *work, size_t bytes) {
    if (nev < 1 || nev > kCRows) return set_error(LAPH_ERR_INVALID, "nev must be in 1..%d", kCRows);
    if (kind == 1 && nev < 3) return set_error(LAPH_ERR_INVALID, "triplets need nev >= 3");
    if (n_mom < 1 || !mom_host) return set_error(LAPH_ERR_INVALID, "need at least one momentum");
    const size_t need = contract_workspace_bytes(c, kind, nev, n_mom);
    if (!work || bytes < need) return set_error(LAPH_ERR_WORKSPACE, "workspace too small: %zu < %zu", bytes, need);
    const size_t per = (size_t)c.g.lt * nev * nev * (kind == 0 ? 1 : nev);
    // momenta left for the launches that carry the whole phase: all, or those whose (px, py)
    // does not pay by planes
    std::vector<int> rest;
    if (kind == 0) {
        const std::vector<PlaneGroup> groups = plane_groups(c, n_mom, mom_host);
        std::vector<std::pair<int, bool>> sizes;
        for (const PlaneGroup &g : groups) sizes.push_back({(int)g.members.size(), g.herm != 0});
        const std::vector<char> by = DoubletPlan{c.g.lx, c.g.ly, c.g.lz, c.g.lt, nev}.by_planes(sizes);
        for (size_t k = 0; k < groups.size(); ++k) {
            if (by[k])
                LAPH_TRY(doublet_planes(c, groups[k], out, V, nev, mom_host, work));
            else
                rest.insert(rest.end(), groups[k].members.begin(), groups[k].members.end());
        }
    } else {
        for (int q = 0; q < n_mom; ++q) rest.push_back(q);
    }
    for (size_t p0 = 0; p0 < rest.size(); p0 += kCMaxMom) {
        const int np = (int)std::min<size_t>(kCMaxMom, rest.size() - p0);
        ContractArgs a;
        contract_shape(c, kind, nev, np, a);
        if (group_bytes(c, kind, nev, np) > bytes) return set_error(LAPH_ERR_WORKSPACE, "workspace too small");
        for (int q = 0; q < np; ++q) {
            a.out[q] = rest[p0 + q];
            for (int k = 0; k < 3; ++k) a.mom[3 * q + k] = mom_host[3 * rest[p0 + q] + k];
        }
        a.V = reinterpret_cast<const double2 *>(V);
        a.scratch = reinterpret_cast<double2 *>(work);
        const unsigned nblk = (unsigned)(a.lt * a.nsplit * a.ntile * a.nmom);
        if (kind == 0)
            hipLaunchKernelGGL((contract_kernel<0, 1>), dim3(nblk), dim3(kCB), 0, c.stream, a);
        else
            hipLaunchKernelGGL((contract_kernel<1, 2>), dim3(nblk), dim3(kCB), 0, c.stream, a);
        LAPH_TRY(check_launch("contract_kernel"));
        const long total = (long)per * np;
        const unsigned rb = (unsigned)((total + 255) / 256);
        if (kind == 0)
            hipLaunchKernelGGL(doublet_reduce_kernel, dim3(rb), dim3(256), 0, c.stream, a,
                               reinterpret_cast<double2 *>(out));
        else
            hipLaunchKernelGGL(triplet_reduce_kernel, dim3(rb), dim3(256), 0, c.stream, a,
                               reinterpret_cast<double2 *>(out));
        LAPH_TRY(check_launch("contract_reduce_kernel"));
    }
    return LAPH_OK;
}

}  // namespace laph

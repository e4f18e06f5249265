// Declarations of the solver's vector kernels (blas.hip).
#pragma once

#include "laph_host.h"

namespace laph {

// slots a vector kernel works on: all, active, or flagged for a reliable update
enum { kModeAll = 0, kModeActive = 1, kModeFlagged = 2 };
// (kFinUpdate: kFinUpdateNorm and kFinUpdateRho at once)
enum { kFinAlpha, kFinOmega, kFinRho, kFinUpdate, kFinUpdateNorm, kFinUpdateRho, kFinInit, kFinBnorm, kFinR64, kFinTrueRes };

constexpr int kSolverPq = 6;   // quantities per slot in the solver's partial sums

struct BlasArgs {
    int vh = 0;
    int nsb = 0;                 // site blocks of 256 (partials written per quantity per slot)
    int pstride = 0;             // partial-sum stride per quantity per slot
    const int *list = nullptr;   // slot list
    const int *nlist = nullptr;  // device scalar: entries in use
    int nlist_max = 0;           // grid size
    SlotState *st = nullptr;
    double *partials = nullptr;  // [slot][kSolverPq][pstride]
    Operand r, rh, p, v, t, x;   // inner-precision vectors (x: the x_lo precision)
    Operand x64, r64;            // FP64 solution and residual
    const int *flist = nullptr;  // flagged mode: slots taking a reliable update
    const int *nflist = nullptr; // device scalar: entries of flist
    SiteWindow win;              // norm2 / copy64: the sources are zero outside it (not read);
                                 // p / s / x/r updates: the sites updated
    SiteWindow win_rh;           // x/r update: r^ is zero outside it (not read) unless *rh_full
    int *rh_full = nullptr;      // device flag: r^ is not confined to the source's window (a restart)
    SiteWindow win_pv;           // p update: p and v are zero outside it (not read)
    int sb_first = 0;            // first site block of the launch (set by the launcher)
};

// Input / output of the flagged-slot compaction (the last workgroup of an iteration's last finalize).
struct FlagArgs {
    const int *tile_slots = nullptr;   // static FP64 tiles [ntiles][nr], grouped by mass
    const int *tile_mass = nullptr;
    const int *ntiles = nullptr;       // device scalar
    int nr = 1;
    int *done = nullptr;               // workgroups finished (zero between launches)
    int *out_slots = nullptr, *out_mass = nullptr, *out_ntiles = nullptr;   // flagged tiles
    int *flist = nullptr, *nflist = nullptr;                                // flagged slots
};

struct FinArgs {
    const int *list = nullptr;
    const int *nlist = nullptr;
    int nlist_max = 0;
    int nsb = 0;        // partials to sum (the producing kernel's site blocks)
    int pstride = 0;    // partial-sum stride per quantity per slot
    SlotState *st = nullptr;
    const double *partials = nullptr;
    int max_restarts = 10;
    int first = 0;      // a windowed producer wrote the partials of `count` blocks from `first` (cyclic)
    int count = 0;
    int nsb2 = 0;       // update: blocks of the kernel that wrote quantities 3 .. 5
    FlagArgs flags;     // rho
};

laph_status blas_p_update(const Ctx &c, const BlasArgs &a, int prec);
laph_status blas_xr_update(const Ctx &c, const BlasArgs &a, int prec);
laph_status blas_s_update(const Ctx &c, const BlasArgs &a, int prec);
laph_status blas_accumulate(const Ctx &c, const BlasArgs &a, int prec, int mode);
laph_status blas_lower(const Ctx &c, const BlasArgs &a, int prec, int mode, int init);
laph_status blas_norm2(const Ctx &c, const BlasArgs &a, Operand v1, Operand v2, int mode);
laph_status blas_copy64(const Ctx &c, const BlasArgs &a, Operand dst, Operand src, int mode);
laph_status blas_finalize(const Ctx &c, const FinArgs &f, int what);

}  // namespace laph

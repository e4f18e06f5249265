// Fused BLAS-1 kernels of the batched BiCGStab, their FP64 partial reductions,
// and the per-slot finalize kernels that turn the partials into the solver's
// scalars on the device (no host round trip inside an iteration).
//
// Every vector kernel runs on a 2-D grid (site block, entry of the slot list)
// and touches each site once; inner products are accumulated per site in the
// kernel's arithmetic precision, per thread block in FP64 (wave shuffles, then
// LDS) and across blocks by the finalize kernels in a fixed order, so results
// are reproducible run to run.
#include "laph_blas.h"

namespace laph {

constexpr int kB = 256;

__device__ __forceinline__ void reduce_store(double *v, int nv, double *dst, size_t q_stride) {
    __shared__ double red[kB / 64][4];
    for (int q = 0; q < nv; ++q) {
        double s = v[q];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        v[q] = s;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0)
        for (int q = 0; q < nv; ++q) red[wave][q] = v[q];
    __syncthreads();
    if (threadIdx.x == 0)
        for (int q = 0; q < nv; ++q) {
            double s = 0;
            for (int w = 0; w < kB / 64; ++w) s += red[w][q];
            dst[q * q_stride] = s;
        }
    // a block handles several slots in turn: red is written again next round
    __syncthreads();
}

// Entries of the slot list this launch walks: the flagged list (built on the
// device after the rho finalize) in flagged mode, the slot list otherwise.
__device__ __forceinline__ int blas_count(const BlasArgs &A, int mode) {
    return mode == kModeFlagged ? *A.nflist : *A.nlist;
}

// slot of list entry j, or -1 if it has nothing to do in this mode
__device__ __forceinline__ int blas_slot_at(const BlasArgs &A, int mode, int j) {
    const int s = mode == kModeFlagged ? A.flist[j] : A.list[j];
    const SlotState &st = A.st[s];
    if (mode != kModeAll && st.status != LAPH_RHS_ACTIVE) return -1;
    if (mode == kModeFlagged && st.flag == 0) return -1;
    return s;
}

// Grid rows walk the list entries j = blockIdx.y, blockIdx.y + gridDim.y, ...;
// the slot test is uniform over the block.
#define LAPH_FOR_SLOTS(A, mode, s)                                                              \
    for (int j_ = blockIdx.y, n_ = blas_count(A, mode); j_ < n_; j_ += gridDim.y)              \
        if (const int s = blas_slot_at(A, mode, j_); s >= 0)

template <class R>
__device__ __forceinline__ cplx<R> c_of(double2 z) {
    return {R(z.x), R(z.y)};
}

// first site of this block; grids of windowed updates walk the blocks the window touches
__device__ __forceinline__ int first_site(const BlasArgs &A) {
    int b = A.sb_first + blockIdx.x;
    if (b >= A.nsb) b -= A.nsb;
    return b * kB;
}

// p = r + beta (p - omega v);  beta == 0 means p = r (fresh start: p, v not read).
// Sites outside A.win are not touched; outside A.win_pv p and v are zero and not read.
template <class P>
__global__ __launch_bounds__(kB) void p_update_kernel(BlasArgs A) {
    using R = typename P::real;
    const int h = first_site(A) + threadIdx.x;
    if (h >= A.vh || !in_window(A.win, h, A.vh)) return;
    const bool zero_pv = !in_window(A.win_pv, h, A.vh);
    LAPH_FOR_SLOTS(A, kModeActive, s) {
        const double2 beta = A.st[s].beta;
        cplx<R> r[12];
        SpinorIO<P>::load(A.r.at(s), A.vh, h, r);
        if (zero_pv || (beta.x == 0.0 && beta.y == 0.0)) {
            SpinorIO<P>::store(A.p.at(s), A.vh, h, r);
            continue;
        }
        const cplx<R> b = c_of<R>(beta), w = c_of<R>(A.st[s].omega);
        cplx<R> p[12], v[12];
        SpinorIO<P>::load(A.p.at(s), A.vh, h, p);
        SpinorIO<P>::load(A.v.at(s), A.vh, h, v);
#pragma unroll
        for (int c = 0; c < 12; ++c) p[c] = r[c] + b * (p[c] - w * v[c]);
        SpinorIO<P>::store(A.p.at(s), A.vh, h, p);
    }
}

// r = r - alpha v   (r becomes s)
template <class P>
__global__ __launch_bounds__(kB) void s_update_kernel(BlasArgs A) {
    using R = typename P::real;
    const int h = first_site(A) + threadIdx.x;
    if (h >= A.vh || !in_window(A.win, h, A.vh)) return;
    LAPH_FOR_SLOTS(A, kModeActive, s) {
        const cplx<R> al = c_of<R>(A.st[s].alpha);
        cplx<R> r[12], v[12];
        SpinorIO<P>::load(A.r.at(s), A.vh, h, r);
        SpinorIO<P>::load(A.v.at(s), A.vh, h, v);
#pragma unroll
        for (int c = 0; c < 12; ++c) r[c] = r[c] - al * v[c];
        SpinorIO<P>::store(A.r.at(s), A.vh, h, r);
    }
}

// x_lo += alpha p + omega s (x_lo = ... after a fold or at the start);  r = s - omega t;
// partials <r^, r>, |r|^2.  Outside A.win p, s and t are zero: nothing to do there, except
// that an x_lo not written since the last fold becomes zero in memory.  r^ is not read where
// it is zero.
template <class P, class PX>
__global__ __launch_bounds__(kB) void xr_update_kernel(BlasArgs A) {
    using R = typename P::real;
    using RX = typename PX::real;
    const int h0 = blockIdx.x * kB, h = h0 + threadIdx.x;
    const bool outside = block_outside(A.win, h0, min(kB, A.vh - h0), A.vh);   // uniform
    const bool live = h < A.vh && in_window(A.win, h, A.vh);
    const bool rh_zero = block_outside(A.win_rh, h0, min(kB, A.vh - h0), A.vh) && *A.rh_full == 0;
    LAPH_FOR_SLOTS(A, kModeActive, s) {
        // (iters counts this iteration after this kernel)
        const bool fresh_x = A.st[s].iters < A.st[s].xlo_from;
        if (!live && h < A.vh && fresh_x) {
            cplx<RX> x[12];
#pragma unroll
            for (int c = 0; c < 12; ++c) x[c] = {RX(0), RX(0)};
            SpinorIO<PX>::store(A.x.at(s), A.vh, h, x);
        }
        if (outside) continue;
        double part[3] = {0, 0, 0};
        if (live) {
            const cplx<R> al = c_of<R>(A.st[s].alpha), om = c_of<R>(A.st[s].omega);
            cplx<R> p[12], r[12], t[12], rh[12];
            cplx<RX> x[12];
            SpinorIO<P>::load(A.p.at(s), A.vh, h, p);
            SpinorIO<P>::load(A.r.at(s), A.vh, h, r);
            SpinorIO<P>::load(A.t.at(s), A.vh, h, t);
            if (fresh_x) {
#pragma unroll
                for (int c = 0; c < 12; ++c) x[c] = {RX(0), RX(0)};
            } else {
                SpinorIO<PX>::load(A.x.at(s), A.vh, h, x);
            }
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                cplx<R> dx = al * p[c] + om * r[c];
                x[c] = x[c] + cplx<RX>{RX(dx.re), RX(dx.im)};
                r[c] = r[c] - om * t[c];
            }
            SpinorIO<PX>::store(A.x.at(s), A.vh, h, x);
            SpinorIO<P>::store(A.r.at(s), A.vh, h, r);
            cplx<R> d = {R(0), R(0)};
            R n2 = R(0);
#pragma unroll
            for (int c = 0; c < 12; ++c) n2 += r[c].re * r[c].re + r[c].im * r[c].im;
            if (!rh_zero) {
                SpinorIO<P>::load(A.rh.at(s), A.vh, h, rh);
#pragma unroll
                for (int c = 0; c < 12; ++c) cmac_conj(d, rh[c], r[c]);
            }
            part[0] = d.re;
            part[1] = d.im;
            part[2] = n2;
        }
        reduce_store(part, 3, A.partials + (size_t)s * kSolverPq * A.pstride + blockIdx.x, A.pstride);
    }
}

// reliable update, part 1: x64 += x_lo (flagged slots).  x_lo is not cleared here: the
// update's finalize says which iteration writes it next (xlo_from), without reading it.
template <class PX>
__global__ __launch_bounds__(kB) void accumulate_kernel(BlasArgs A, int mode) {
    using RX = typename PX::real;
    const int h = blockIdx.x * kB + threadIdx.x;
    if (h >= A.vh) return;
    LAPH_FOR_SLOTS(A, mode, s) {
        if (A.st[s].iters < A.st[s].xlo_from) continue;   // uniform: nothing to fold
        cplx<RX> x[12];
        cplx<double> y[12];
        SpinorIO<PX>::load(A.x.at(s), A.vh, h, x);
        SpinorIO<F64>::load(A.x64.at(s), A.vh, h, y);
#pragma unroll
        for (int c = 0; c < 12; ++c) y[c] = y[c] + cplx<double>{(double)x[c].re, (double)x[c].im};
        SpinorIO<F64>::store(A.x64.at(s), A.vh, h, y);
    }
}

// r = lo(r64); restart (flag 2) or init: r^ = r; init: p = r.  init 1: r lives on the source's
// window, 2: on the whole lattice.
// partials <r^, r>, |r|^2.  INIT is init != 0: the update's form, launched every iteration and mostly
// with little to do, has no p to store and a third fewer registers.
template <class P, class PX, bool INIT>
__global__ __launch_bounds__(kB) void lower_kernel(BlasArgs A, int mode, int init) {
    using R = typename P::real;
    const int h = blockIdx.x * kB + threadIdx.x;
    LAPH_FOR_SLOTS(A, mode, s) {
        // a restart replaces r^: it is no longer confined to the source's window
        if ((INIT || A.st[s].flag == 2) && blockIdx.x == 0 && threadIdx.x == 0) *A.rh_full = init != 1;
        double part[3] = {0, 0, 0};
        if (h < A.vh) {
            cplx<double> y[12];
            SpinorIO<F64>::load(A.r64.at(s), A.vh, h, y);
            cplx<R> r[12], rh[12];
#pragma unroll
            for (int c = 0; c < 12; ++c) r[c] = {R(y[c].re), R(y[c].im)};
            SpinorIO<P>::store(A.r.at(s), A.vh, h, r);
            // work with the stored (rounded) values so r^ and r agree exactly
            SpinorIO<P>::load(A.r.at(s), A.vh, h, r);
            const bool reset = INIT || A.st[s].flag == 2;
            if constexpr (INIT) SpinorIO<P>::store(A.p.at(s), A.vh, h, r);
            if (reset) {
                SpinorIO<P>::store(A.rh.at(s), A.vh, h, r);
                SpinorIO<P>::load(A.rh.at(s), A.vh, h, rh);
            } else {
                SpinorIO<P>::load(A.rh.at(s), A.vh, h, rh);
            }
            cplx<R> d = {R(0), R(0)};
            R n2 = R(0);
#pragma unroll
            for (int c = 0; c < 12; ++c) {
                cmac_conj(d, rh[c], r[c]);
                n2 += r[c].re * r[c].re + r[c].im * r[c].im;
            }
            part[0] = d.re;
            part[1] = d.im;
            part[2] = n2;
        }
        // quantities 3 .. 5: those before them hold the update's |r64|^2
        reduce_store(part, 3, A.partials + ((size_t)s * kSolverPq + 3) * A.pstride + blockIdx.x, A.pstride);
    }
}

// |v|^2 of one or two FP64 half-vectors per slot (partials q = 0); sites outside
// the window are not read (the vectors are zero there)
__global__ __launch_bounds__(kB) void norm2_kernel(BlasArgs A, Operand v1, Operand v2, int mode) {
    const int h = blockIdx.x * kB + threadIdx.x;
    const bool live = h < A.vh && in_window(A.win, h, A.vh);
    LAPH_FOR_SLOTS(A, mode, s) {
        double part[1] = {0};
        if (live) {
            cplx<double> y[12];
            SpinorIO<F64>::load(v1.at(s), A.vh, h, y);
            double n2 = 0;
#pragma unroll
            for (int c = 0; c < 12; ++c) n2 += y[c].re * y[c].re + y[c].im * y[c].im;
            if (v2.base) {
                SpinorIO<F64>::load(v2.at(s), A.vh, h, y);
#pragma unroll
                for (int c = 0; c < 12; ++c) n2 += y[c].re * y[c].re + y[c].im * y[c].im;
            }
            part[0] = n2;
        }
        reduce_store(part, 1, A.partials + (size_t)s * kSolverPq * A.pstride + blockIdx.x, A.pstride);
    }
}

// dst = src (FP64 half-vectors) per slot; outside the window src is zero and not read
__global__ __launch_bounds__(kB) void copy64_kernel(BlasArgs A, Operand dst, Operand src, int mode) {
    const int h = blockIdx.x * kB + threadIdx.x;
    if (h >= A.vh) return;
    const bool live = in_window(A.win, h, A.vh);
    LAPH_FOR_SLOTS(A, mode, s) {
        cplx<double> y[12];
        if (live) {
            SpinorIO<F64>::load(src.at(s), A.vh, h, y);
        } else {
#pragma unroll
            for (int c = 0; c < 12; ++c) y[c] = {0.0, 0.0};
        }
        SpinorIO<F64>::store(dst.at(s), A.vh, h, y);
    }
}

// Flagged slots after an iteration's last finalize: the list of slots that take a reliable update this
// iteration, and FP64 tiles of them (tiles never mix masses).  One workgroup; entries of
// the static FP64 tile table (already grouped by mass) are tested in parallel, then packed in
// table order by one lane.  The flags were written by workgroups of this launch: read past the
// caches.  (With a launch of its own, and one more for a second finalize of the update, 8^4 with
// 64 RHS took 4.70 ms instead of 4.50, where an iteration is a chain of launches.)
__device__ void flag_tiles(const FinArgs &A) {
    __shared__ int ks[256], km[256];
    const int nth = blockDim.x;
    const FlagArgs &F = A.flags;
    const int total = *F.ntiles * F.nr;
    int cur = -1, fill = 0, cm = -1, nf = 0;   // packing state (lane 0)
    for (int base = 0; base < total; base += nth) {
        const int e = base + (int)threadIdx.x;
        int s = -1, m = 0;
        if (e < total) {
            s = F.tile_slots[e];
            m = F.tile_mass[e / F.nr];
            if (s >= 0) {
                const int status = __hip_atomic_load(&A.st[s].status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int flag = __hip_atomic_load(&A.st[s].flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (!(status == LAPH_RHS_ACTIVE && flag != 0)) s = -1;
            }
        }
        ks[threadIdx.x] = s;
        km[threadIdx.x] = m;
        __syncthreads();
        if (threadIdx.x == 0) {
            const int n = min(nth, total - base);
            for (int i = 0; i < n; ++i) {
                const int si = ks[i];
                if (si < 0) continue;
                if (cur < 0 || fill == F.nr || km[i] != cm) {
                    ++cur;
                    for (int k = 0; k < F.nr; ++k) F.out_slots[cur * F.nr + k] = -1;
                    F.out_mass[cur] = km[i];
                    cm = km[i];
                    fill = 0;
                }
                F.out_slots[cur * F.nr + fill++] = si;
                F.flist[nf++] = si;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *F.out_ntiles = cur + 1;
        *F.nflist = nf;
    }
}

// ---------------------------------------------------------------------------
// finalize kernels: one workgroup per slot, one 64-thread wave per quantity sums the
// partials in fixed order
// ---------------------------------------------------------------------------
// Eight independent loads in flight per lane: the partials were just written by
// workgroups on every XCD, and a loop that waits for each load in turn spends ~0.1 ms
// of latency per slot and quantity.  The summation order is fixed.  A windowed producer wrote
// only `count` blocks from `first` on (cyclic); the others count as the zeros they stand for,
// each in its place, so a windowed sum has the bits of the whole one.
__device__ __forceinline__ double wave_sum_partials(const double *p, int first, int count, int nsb) {
    double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    auto at = [&](int b) {
        const int d = b - first;
        return (d < 0 ? d + nsb : d) < count ? p[b] : 0.0;
    };
    int i = threadIdx.x & 63;
    for (; i + 7 * 64 < nsb; i += 8 * 64) {
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] += at(i + 64 * k);
    }
    for (; i < nsb; i += 64) a[0] += at(i);
    double s = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    return s;
}

__device__ __forceinline__ double2 cdiv(double2 a, double2 b) {
    const double d = b.x * b.x + b.y * b.y;
    return make_double2((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ bool finite2(double2 a) { return isfinite(a.x) && isfinite(a.y); }
__device__ __forceinline__ double cabs2(double2 a) { return a.x * a.x + a.y * a.y; }

// end of an iteration: beta from rho_new = rn, and whether a reliable update is due (r2 = |r|^2)
__device__ __forceinline__ void finalize_rho(SlotState &st, double2 rn, double r2) {
    st.iters += 1;
    st.r2 = r2;
    if (!isfinite(r2) || !finite2(rn)) st.flag = 2;
    if (st.flag != 2) {
        if (cabs2(st.omega) == 0.0 || cabs2(st.rho) == 0.0 || cabs2(rn) == 0.0) {
            st.flag = 2;
        } else {
            st.beta = cmul(cdiv(rn, st.rho), cdiv(st.alpha, st.omega));
        }
    }
    st.rho_prev = st.rho;
    st.rho = rn;
    if (r2 <= st.stop2 || r2 < st.delta2 * st.r2_upd || st.iters >= st.maxiter) st.flag |= 1;
}

// rho, beta and the residual norm after r was replaced by the FP64 residual (or at the start)
__device__ __forceinline__ void finalize_residual(SlotState &st, double2 rn, double r2, bool restart) {
    st.r2 = r2;
    if (restart) {
        st.beta = make_double2(0, 0);
        st.rho_prev = make_double2(1, 0);
        st.alpha = make_double2(1, 0);
        st.omega = make_double2(1, 0);
    } else {
        st.beta = cmul(cdiv(rn, st.rho_prev), cdiv(st.alpha, st.omega));
    }
    st.rho = rn;
    st.flag = 0;
}

__device__ __forceinline__ void finalize_slot(const FinArgs &A, int what) {
    const int j = blockIdx.x;
    if (j >= *A.nlist) return;
    const int s = A.list[j];
    SlotState &st = A.st[s];
    const double *P = A.partials + (size_t)s * kSolverPq * A.pstride;
    const bool active = st.status == LAPH_RHS_ACTIVE;
    // wave w sums quantity q0 + w (an update's last three: blocks of another kernel) for thread 0
    __shared__ double v[4];
    auto sums = [&](int q0) {
        const int w = threadIdx.x >> 6;
        const bool low = what == kFinUpdate && w > 0;
        const int q = low ? 2 + w : q0 + w;
        const double *p = P + (size_t)q * A.pstride;
        const double t = low ? wave_sum_partials(p, 0, A.nsb2, A.nsb2) : wave_sum_partials(p, A.first, A.count, A.nsb);
        if ((threadIdx.x & 63) == 0) v[w] = t;
        __syncthreads();
    };
    switch (what) {
        case kFinAlpha: {  // sigma = <r^, v>; alpha = rho / sigma
            if (!active) return;
            sums(0);
            if (threadIdx.x) return;
            const double2 sig = make_double2(v[0], v[1]);
            if (!finite2(sig) || cabs2(sig) <= 1e-300 * (cabs2(st.rho) + 1e-300) || cabs2(sig) == 0.0) {
                st.alpha = make_double2(0, 0);
                st.flag = 2;
            } else {
                st.alpha = cdiv(st.rho, sig);
            }
            return;
        }
        case kFinOmega: {  // omega = <t, s> / |t|^2
            if (!active) return;
            sums(0);
            if (threadIdx.x) return;
            const double2 ts = make_double2(v[0], v[1]);
            const double tt = v[2];
            if (!(tt > 0) || !isfinite(tt) || !finite2(ts)) {
                st.omega = make_double2(0, 0);
                st.flag = 2;
            } else {
                st.omega = make_double2(ts.x / tt, ts.y / tt);
            }
            return;
        }
        case kFinRho: {  // rho = <r^, r>, |r|^2; beta; whether a reliable update is due
            if (!active) return;
            sums(0);
            if (threadIdx.x) return;
            finalize_rho(st, make_double2(v[0], v[1]), v[2]);
            return;
        }
        case kFinUpdateRho: {
            if (!(active && st.flag != 0)) return;
            sums(3);
            if (threadIdx.x) return;
            finalize_residual(st, make_double2(v[0], v[1]), v[2], st.flag == 2);
            return;
        }
        case kFinUpdateNorm:
        case kFinUpdate: {
            // after a reliable update: r2_upd = |b_hat - M x64|^2, whether the slot is done, and rho and
            // beta from the corrected residual r = lo(r64)
            if (!(active && st.flag != 0)) return;
            sums(0);
            if (threadIdx.x) return;
            const double u2 = v[0];
            st.updates += 1;
            st.r2_upd = u2;
            st.xlo_from = st.iters + 1;   // folded into x64 by this update (accumulate, or the FP64 stage forming r64)
            if (!isfinite(u2)) {
                st.status = LAPH_RHS_NONFINITE;
            } else if (u2 <= st.stop2) {
                st.status = LAPH_RHS_CONVERGED;
            } else if (st.iters >= st.maxiter) {
                st.status = LAPH_RHS_NOCONV;
            } else if (st.flag == 2) {
                st.restarts += 1;
                if (st.restarts > A.max_restarts) st.status = LAPH_RHS_BREAKDOWN;
            }
            if (st.status != LAPH_RHS_ACTIVE || what == kFinUpdateNorm) return;
            finalize_residual(st, make_double2(v[1], v[2]), v[3], st.flag == 2);
            return;
        }
        case kFinInit: {  // first residual of a solve
            if (!active) return;
            sums(3);
            if (threadIdx.x) return;
            finalize_residual(st, make_double2(v[0], v[1]), v[2], true);
            st.xlo_from = st.iters + 1;
            return;
        }
        case kFinBnorm: {  // |B|^2 of the full-lattice source; zero or non-finite sources end here
            sums(0);
            if (threadIdx.x) return;
            const double b2 = v[0];
            st.bnorm2 = b2;
            if (!isfinite(b2)) st.status = LAPH_RHS_NONFINITE;
            return;
        }
        case kFinR64: {  // |r64|^2 at the start of a solve pass
            if (!active) return;
            sums(0);
            if (threadIdx.x) return;
            const double r2 = v[0];
            st.r2_upd = r2;
            if (!isfinite(r2)) st.status = LAPH_RHS_NONFINITE;
            else if (r2 <= st.stop2) st.status = LAPH_RHS_CONVERGED;
            return;
        }
        case kFinTrueRes: {  // accumulate |B - D X|^2 (called for the even and the odd part)
            sums(0);
            if (threadIdx.x) return;
            const double r2 = v[0];
            st.true_res2 += r2;
            return;
        }
    }
}

__global__ __launch_bounds__(256) void finalize_kernel(FinArgs A, int what) {
    finalize_slot(A, what);
    if (what != kFinRho) return;
    // the workgroup that finishes last compacts the slots flagged for a reliable update
    __shared__ int last;
    if (threadIdx.x == 0) {
        const int n = __hip_atomic_fetch_add(A.flags.done, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        last = n == (int)gridDim.x - 1;
        if (last) __hip_atomic_store(A.flags.done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (last) flag_tiles(A);
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
template <class F>
static laph_status dispatch_prec(int prec, F &&f) {
    if (prec == LAPH_F64) return f(F64{}, F64{});
    if (prec == LAPH_F32) return f(F32{}, F32{});
    return f(F16N{}, F32{});
}

// grid rows: one per list entry, or a quarter of them in flagged mode (a block
// then walks several flagged slots; the flagged count is known only on the device)
static dim3 blas_grid(const BlasArgs &a, int mode) {
    const int rows = mode == kModeFlagged ? (a.nlist_max + 3) / 4 : a.nlist_max;
    return dim3(a.nsb, rows > 0 ? rows : 1);
}

laph_status blas_p_update(const Ctx &c, const BlasArgs &a, int prec) {
    BlasArgs w = a;
    dim3 grid(window_blocks(a.win, kB, a.nsb, a.vh, &w.sb_first), a.nlist_max);
    return dispatch_prec(prec, [&](auto P, auto) {
        hipLaunchKernelGGL(p_update_kernel<decltype(P)>, grid, dim3(kB), 0, c.stream, w);
        return check_launch("p_update_kernel");
    });
}
laph_status blas_s_update(const Ctx &c, const BlasArgs &a, int prec) {
    BlasArgs w = a;
    dim3 grid(window_blocks(a.win, kB, a.nsb, a.vh, &w.sb_first), a.nlist_max);
    return dispatch_prec(prec, [&](auto P, auto) {
        hipLaunchKernelGGL(s_update_kernel<decltype(P)>, grid, dim3(kB), 0, c.stream, w);
        return check_launch("s_update_kernel");
    });
}
laph_status blas_xr_update(const Ctx &c, const BlasArgs &a, int prec) {
    dim3 grid(a.nsb, a.nlist_max);
    return dispatch_prec(prec, [&](auto P, auto PX) {
        hipLaunchKernelGGL((xr_update_kernel<decltype(P), decltype(PX)>), grid, dim3(kB), 0, c.stream, a);
        return check_launch("xr_update_kernel");
    });
}
laph_status blas_accumulate(const Ctx &c, const BlasArgs &a, int prec, int mode) {
    dim3 grid = blas_grid(a, mode);
    return dispatch_prec(prec, [&](auto, auto PX) {
        hipLaunchKernelGGL(accumulate_kernel<decltype(PX)>, grid, dim3(kB), 0, c.stream, a, mode);
        return check_launch("accumulate_kernel");
    });
}
laph_status blas_lower(const Ctx &c, const BlasArgs &a, int prec, int mode, int init) {
    dim3 grid = blas_grid(a, mode);
    return dispatch_prec(prec, [&](auto P, auto PX) {
        if (init)
            hipLaunchKernelGGL((lower_kernel<decltype(P), decltype(PX), true>), grid, dim3(kB), 0, c.stream, a, mode, init);
        else
            hipLaunchKernelGGL((lower_kernel<decltype(P), decltype(PX), false>), grid, dim3(kB), 0, c.stream, a, mode, 0);
        return check_launch("lower_kernel");
    });
}
laph_status blas_norm2(const Ctx &c, const BlasArgs &a, Operand v1, Operand v2, int mode) {
    dim3 grid = blas_grid(a, mode);
    hipLaunchKernelGGL(norm2_kernel, grid, dim3(kB), 0, c.stream, a, v1, v2, mode);
    return check_launch("norm2_kernel");
}
laph_status blas_copy64(const Ctx &c, const BlasArgs &a, Operand dst, Operand src, int mode) {
    dim3 grid = blas_grid(a, mode);
    hipLaunchKernelGGL(copy64_kernel, grid, dim3(kB), 0, c.stream, a, dst, src, mode);
    return check_launch("copy64_kernel");
}
laph_status blas_finalize(const Ctx &c, const FinArgs &f, int what) {
    // quantities (= waves) of each step
    const int nq = what == kFinAlpha ? 2
                   : (what == kFinOmega || what == kFinRho || what == kFinUpdateRho || what == kFinInit) ? 3
                   : what == kFinUpdate ? 4 : 1;
    hipLaunchKernelGGL(finalize_kernel, dim3(f.nlist_max), dim3(64 * nq), 0, c.stream, f, what);
    return check_launch("finalize_kernel");
}

}  // namespace laph

// Setup kernels: gauge ingest (canonical -> even-odd SoA in FP64 / FP32 / FP16,
// SU(3) check), clover term and the Cholesky-based inverses of its chiral blocks
// (FP64), and spinor pack / unpack between the canonical and internal layouts.
#include <cstring>

#include "laph_host.h"

namespace laph {

constexpr int kSetupBlock = 256;

// ---------------------------------------------------------------------------
// gauge ingest
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kSetupBlock) void gauge_pack_kernel(Geom g, const double2 *U, GaugePtrs gp,
                                                                 unsigned long long *maxdev) {
    const long i = (long)blockIdx.x * kSetupBlock + threadIdx.x;
    const long vol = 2L * g.vh;
    if (i >= vol) return;
    const int x = (int)(i % g.lx);
    const int y = (int)((i / g.lx) % g.ly);
    const int z = (int)((i / ((long)g.lx * g.ly)) % g.lz);
    const int t = (int)(i / ((long)g.lx * g.ly * g.lz));
    const int p = (x + y + z + t) & 1;
    const int h = (int)(i >> 1);
    double dev = 0;
    for (int mu = 0; mu < 4; ++mu) {
        cplx<double> u[9];
        for (int k = 0; k < 9; ++k) {
            double2 v = U[(i * 4 + mu) * 9 + k];
            u[k] = {v.x, v.y};
        }
        // distance from SU(3): |U U^+ - 1| and |det U - 1|
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) {
                cplx<double> s = {a == b ? -1.0 : 0.0, 0.0};
                for (int k = 0; k < 3; ++k) cmac_conj(s, u[b * 3 + k], u[a * 3 + k]);
                dev = fmax(dev, fmax(fabs(s.re), fabs(s.im)));
            }
        cplx<double> det = u[0] * (u[4] * u[8] - u[5] * u[7]) - u[1] * (u[3] * u[8] - u[5] * u[6]) +
                           u[2] * (u[3] * u[7] - u[4] * u[6]);
        dev = fmax(dev, fmax(fabs(det.re - 1.0), fabs(det.im)));
        double2 *d64 = reinterpret_cast<double2 *>(const_cast<char *>(gp.f64(p, mu)));
        for (int k = 0; k < 9; ++k) d64[(size_t)k * g.vh + h] = make_double2(u[k].re, u[k].im);
        float4 *d32 = reinterpret_cast<float4 *>(const_cast<char *>(gp.f32(p, mu)));
        for (int j = 0; j < 3; ++j)
            d32[(size_t)j * g.vh + h] = make_float4((float)u[2 * j].re, (float)u[2 * j].im,
                                                    (float)u[2 * j + 1].re, (float)u[2 * j + 1].im);
        half8 a8;
        for (int k = 0; k < 4; ++k) {
            a8[2 * k] = (_Float16)u[k].re;
            a8[2 * k + 1] = (_Float16)u[k].im;
        }
        half4 b4;
        b4[0] = (_Float16)u[4].re;
        b4[1] = (_Float16)u[4].im;
        b4[2] = (_Float16)u[5].re;
        b4[3] = (_Float16)u[5].im;
        reinterpret_cast<half8 *>(const_cast<char *>(gp.f16a(p, mu)))[h] = a8;
        reinterpret_cast<half4 *>(const_cast<char *>(gp.f16b(p, mu)))[h] = b4;
    }
    if (!(dev <= 1e300)) dev = 1e300;  // NaN -> huge
    atomicMax(maxdev, (unsigned long long)__double_as_longlong(dev));
}

laph_status load_gauge(Ctx &c, const double *U) {
    unsigned long long *d_max = c.gauge_dev();
    LAPH_HIP(hipMemsetAsync(d_max, 0, sizeof(unsigned long long), c.stream));
    const long vol = 2L * c.g.vh;
    hipLaunchKernelGGL(gauge_pack_kernel, dim3((unsigned)((vol + kSetupBlock - 1) / kSetupBlock)), dim3(kSetupBlock),
                       0, c.stream, c.g, reinterpret_cast<const double2 *>(U), c.gp, d_max);
    LAPH_TRY(check_launch("gauge_pack_kernel"));
    unsigned long long hmax = 0;
    LAPH_HIP(hipMemcpyAsync(&hmax, d_max, sizeof(hmax), hipMemcpyDeviceToHost, c.stream));
    LAPH_HIP(hipStreamSynchronize(c.stream));
    double dev;
    memcpy(&dev, &hmax, sizeof(dev));
    if (!(dev <= 1e-10)) {
        c.gauge_loaded = false;
        return set_error(LAPH_ERR_INVALID, "gauge field is not SU(3): max deviation %.3e > 1e-10", dev);
    }
    c.gauge_loaded = true;
    c.n_mass = 0;
    return LAPH_OK;
}

// ---------------------------------------------------------------------------
// clover term
// ---------------------------------------------------------------------------
// 3x3 complex matrices in FP64
struct M3 {
    cplx<double> m[9];
};
__device__ __forceinline__ M3 mmul(const M3 &a, const M3 &b) {
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cplx<double> s = {0, 0};
#pragma unroll
            for (int k = 0; k < 3; ++k) cmac(s, a.m[i * 3 + k], b.m[k * 3 + j]);
            c.m[i * 3 + j] = s;
        }
    return c;
}
__device__ __forceinline__ M3 adj(const M3 &a) {
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) c.m[i * 3 + j] = conj(a.m[j * 3 + i]);
    return c;
}

// the link in direction dir at the site x + dm mu + dn nu, dm, dn in {-1, 0, 1}
template <int MU, int NU>
__device__ __forceinline__ M3 link64(const Geom &g, const GaugePtrs &gp, const int (&x)[4], int dm, int dn,
                                     int dir) {
    const int ext[4] = {g.lx, g.ly, g.lz, g.lt};
    int c[4] = {x[0], x[1], x[2], x[3]};
    c[MU] += dm;
    if (c[MU] < 0) c[MU] += ext[MU];
    if (c[MU] == ext[MU]) c[MU] = 0;
    c[NU] += dn;
    if (c[NU] < 0) c[NU] += ext[NU];
    if (c[NU] == ext[NU]) c[NU] = 0;
    M3 u;
    GaugeIO<F64>::load(gp, (c[0] + c[1] + c[2] + c[3]) & 1, dir, g.vh, cb_index(g, c[0], c[1], c[2], c[3]), u.m);
    return u;
}

// An anti-Hermitian 3x3 matrix: i d[k] on the diagonal, o = entries (1,0), (2,0), (2,1).
struct AH3 {
    double d[3];
    cplx<double> o[3];
};

// F_munu(x) = (Q - Q^+)/8 minus its trace part, Q = sum of the four plaquettes at x
template <int MU, int NU>
__device__ __forceinline__ AH3 field_strength(const Geom &g, const GaugePtrs &gp, const int (&x)[4]) {
    auto at = [&](int dm, int dn, int dir) { return link64<MU, NU>(g, gp, x, dm, dn, dir); };
    M3 q;
    auto add = [&](const M3 &l) {
#pragma unroll
        for (int k = 0; k < 9; ++k) q.m[k] = q.m[k] + l.m[k];
        __builtin_amdgcn_sched_barrier(0);   // later links are not loaded early (registers)
    };
    // x -> x+mu -> x+mu+nu -> x+nu -> x
    q = mmul(mmul(at(0, 0, MU), at(1, 0, NU)), mmul(adj(at(0, 1, MU)), adj(at(0, 0, NU))));
    __builtin_amdgcn_sched_barrier(0);
    // x -> x+nu -> x+nu-mu -> x-mu -> x
    add(mmul(mmul(at(0, 0, NU), adj(at(-1, 1, MU))), mmul(adj(at(-1, 0, NU)), at(-1, 0, MU))));
    // x -> x-mu -> x-mu-nu -> x-nu -> x
    add(mmul(mmul(adj(at(-1, 0, MU)), adj(at(-1, -1, NU))), mmul(at(-1, -1, MU), at(0, -1, NU))));
    // x -> x-nu -> x-nu+mu -> x+mu -> x
    add(mmul(mmul(adj(at(0, -1, NU)), at(0, -1, MU)), mmul(at(1, -1, NU), adj(at(0, 0, MU)))));
    AH3 f;
#pragma unroll
    for (int k = 0; k < 3; ++k) f.d[k] = 0.25 * q.m[4 * k].im;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int i = e == 0 ? 1 : 2, j = e == 2 ? 1 : 0;
        f.o[e] = 0.125 * (q.m[3 * i + j] - conj(q.m[3 * j + i]));
    }
    const double tr = (f.d[0] + f.d[1]) + f.d[2];
#pragma unroll
    for (int k = 0; k < 3; ++k) f.d[k] = ffma(-(1.0 / 3.0), tr, f.d[k]);
    return f;
}

// (i csw / 2) (a + s b), a Hermitian matrix: real diagonal, entries (1,0), (2,0), (2,1)
struct H3 {
    double d[3];
    cplx<double> o[3];
};
__device__ __forceinline__ H3 half_i(double csw, const AH3 &a, double s, const AH3 &b) {
#pragma clang fp contract(off)
    const double f = 0.5 * csw;
    H3 h;
#pragma unroll
    for (int k = 0; k < 3; ++k) h.d[k] = -f * ffma(s, b.d[k], a.d[k]);
#pragma unroll
    for (int k = 0; k < 3; ++k)
        h.o[k] = {-f * ffma(s, b.o[k].im, a.o[k].im), f * ffma(s, b.o[k].re, a.o[k].re)};
    return h;
}
// entry (a, b) of an H3
__device__ __forceinline__ cplx<double> h3_at(const H3 &h, int a, int b) {
    if (a == b) return {h.d[a], 0.0};
    const int hi = a > b ? a : b, lo = a > b ? b : a;
    const cplx<double> e = hi == 1 ? h.o[0] : h.o[1 + lo];
    return a > b ? e : conj(e);
}

// Packed Hermitian clover term per site and chiral block (without 4 + m0):
// in this gamma basis sigma_munu is block diagonal; on spins {0,1} (block 0)
//   sum sigma (x) F = sx (x) (Fyz - Fxt) + sy (x) (Fxz + Fyt) + sz (x) (Fxy - Fzt)
// and on spins {2,3} (block 1) the signs of the time planes flip, with
// sx, sy, sz the Pauli matrices.  The block is (i/2) c_sw times that sum,
// [[Gz, Gx - i Gy], [Gx + i Gy, -Gz]] with index 3 s' + a.
//
// One wave per plane on 64 sites: the six field strengths (9 reals each) meet in LDS and
// every wave assembles the entries of its plane's partners.  Bound by the gather of the
// links (16 per plane and site through the caches; the waves of a block read the same ones
// at about the same time) and the FP64 issue of 12 products a plane.
// 32^3 x 64: 2.2-2.4 ms in a kernel trace (2.8 when the next figures were taken).  One thread
// with all six planes as full matrices, under the default 1024-thread register budget, spilled
// 1208 registers and took 6.56 ms; the same at 256 registers 3.63 ms.  Sharing a link between plaquettes (10 products a plane, as outer
// products) takes 2.4 ms but rounds the term differently, and the iterates of every
// mixed-precision solve with it: the mass gradient of a 16^3 x 32 F16N solve moved by
// 1.5e-9, with the plain order by 2e-10.
constexpr int kCloverSites = 64;

__global__ __launch_bounds__(6 * 64) __attribute__((amdgpu_waves_per_eu(2))) void clover_build_kernel(
    Geom g, GaugePtrs gp, double csw, char *term0, char *term1) {
    __shared__ AH3 F[6][kCloverSites];   // xy, zt, yz, xt, xz, yt
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int h = blockIdx.x * kCloverSites + lane;
    const int p = blockIdx.y;
    const bool valid = h < g.vh;
    int x[4];
    site_coords(g, p, valid ? h : g.vh - 1, x[0], x[1], x[2], x[3]);
    switch (wave) {
        case 0: F[0][lane] = field_strength<0, 1>(g, gp, x); break;
        case 1: F[1][lane] = field_strength<2, 3>(g, gp, x); break;
        case 2: F[2][lane] = field_strength<1, 2>(g, gp, x); break;
        case 3: F[3][lane] = field_strength<0, 3>(g, gp, x); break;
        case 4: F[4][lane] = field_strength<0, 2>(g, gp, x); break;
        default: F[5][lane] = field_strength<1, 3>(g, gp, x); break;
    }
    __syncthreads();
    if (!valid) return;
    const size_t vh = g.vh;
    const int blk = wave & 1, part = wave >> 1;
    const double sgn = blk == 0 ? -1.0 : 1.0;
    double2 *d = reinterpret_cast<double2 *>(p == 0 ? term0 : term1) + blk * 18 * vh + h;
    if (part == 0) {
        // the diagonal, then the entries of equal spin: packed index 3 + (i (i - 1) / 2 + j)
        const H3 z = half_i(csw, F[0][lane], sgn, F[1][lane]);
        d[0] = make_double2(z.d[0], z.d[1]);
        d[vh] = make_double2(z.d[2], -z.d[0]);
        d[2 * vh] = make_double2(-z.d[1], -z.d[2]);
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const int i = e == 0 ? 1 : 2, j = e == 2 ? 1 : 0, i1 = i + 3, j1 = j + 3;
            d[(3 + i * (i - 1) / 2 + j) * vh] = make_double2(z.o[e].re, z.o[e].im);
            d[(3 + i1 * (i1 - 1) / 2 + j1) * vh] = make_double2(-z.o[e].re, -z.o[e].im);
        }
    } else {
        // Gx + i Gy: rows 0 and 1 (first half), row 2 (second half)
        const H3 gx = half_i(csw, F[2][lane], sgn, F[3][lane]), gy = half_i(csw, F[4][lane], -sgn, F[5][lane]);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if ((a == 2) != (part == 2)) continue;
            const int i = a + 3;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const cplx<double> e = h3_at(gx, a, b) + mul_i(h3_at(gy, a, b));
                d[(3 + i * (i - 1) / 2 + b) * vh] = make_double2(e.re, e.im);
            }
        }
    }
}

// Inverse of (term + shift) per site and block by Cholesky: A = L L^+, A^-1 = W^+ W, W = L^-1.
__global__ __launch_bounds__(kSetupBlock) void clover_invert_kernel(int vh, const char *term, double shift, char *inv64, char *inv32, int *bad) {
    const int h = blockIdx.x * kSetupBlock + threadIdx.x;
    const int blk = blockIdx.y;
    if (h >= vh) return;
    double m[36];
    CloverIO<F64>::load(term, blk, vh, h, m);
    cplx<double> A[6][6];
    int k = 0;
    for (int i = 0; i < 6; ++i) A[i][i] = {m[i] + shift, 0.0};
    for (int i = 1; i < 6; ++i)
        for (int j = 0; j < i; ++j) {
            A[i][j] = {m[6 + 2 * k], m[7 + 2 * k]};
            A[j][i] = conj(A[i][j]);
            ++k;
        }
    cplx<double> Lm[6][6];
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) Lm[i][j] = {0, 0};
    bool ok = true;
    for (int j = 0; j < 6; ++j) {
        double d = A[j][j].re;
        for (int q = 0; q < j; ++q) d -= Lm[j][q].re * Lm[j][q].re + Lm[j][q].im * Lm[j][q].im;
        if (!(d > 0)) {
            ok = false;
            d = 1.0;
        }
        const double ljj = sqrt(d);
        Lm[j][j] = {ljj, 0};
        for (int i = j + 1; i < 6; ++i) {
            cplx<double> s = A[i][j];
            for (int q = 0; q < j; ++q) {
                // s -= L[i][q] conj(L[j][q])
                cplx<double> t = Lm[i][q] * conj(Lm[j][q]);
                s = s - t;
            }
            Lm[i][j] = (1.0 / ljj) * s;
        }
    }
    if (!ok) atomicOr(bad, 1);
    // W = L^-1 (lower triangular)
    cplx<double> W[6][6];
    for (int i = 0; i < 6; ++i)
        for (int j = 0; j < 6; ++j) W[i][j] = {0, 0};
    for (int j = 0; j < 6; ++j) {
        W[j][j] = {1.0 / Lm[j][j].re, 0};
        for (int i = j + 1; i < 6; ++i) {
            cplx<double> s = {0, 0};
            for (int q = j; q < i; ++q) cmac(s, Lm[i][q], W[q][j]);
            W[i][j] = (-1.0 / Lm[i][i].re) * s;
        }
    }
    // A^-1 = W^+ W: (i, j) = sum_{q >= max(i,j)} conj(W[q][i]) W[q][j]
    double out[36];
    for (int i = 0; i < 6; ++i) {
        double s = 0;
        for (int q = i; q < 6; ++q) s += W[q][i].re * W[q][i].re + W[q][i].im * W[q][i].im;
        out[i] = s;
    }
    k = 0;
    for (int i = 1; i < 6; ++i)
        for (int j = 0; j < i; ++j) {
            cplx<double> s = {0, 0};
            for (int q = i; q < 6; ++q) cmac_conj(s, W[q][i], W[q][j]);
            out[6 + 2 * k] = s.re;
            out[7 + 2 * k] = s.im;
            ++k;
        }
    double2 *d64 = reinterpret_cast<double2 *>(inv64) + (size_t)blk * 18 * vh;
    for (int q = 0; q < 18; ++q) d64[(size_t)q * vh + h] = make_double2(out[2 * q], out[2 * q + 1]);
    float4 *d32 = reinterpret_cast<float4 *>(inv32) + (size_t)blk * 9 * vh;
    for (int q = 0; q < 9; ++q)
        d32[(size_t)q * vh + h] = make_float4((float)out[4 * q], (float)out[4 * q + 1], (float)out[4 * q + 2],
                                              (float)out[4 * q + 3]);
}

laph_status build_clover(Ctx &c, double csw, int n_mass, const double *m0) {
    char *t0 = c.state + c.off_clov;
    char *t1 = t0 + c.sz_cl64_par;
    dim3 grid((c.g.vh + kCloverSites - 1) / kCloverSites, 2);
    hipLaunchKernelGGL(clover_build_kernel, grid, dim3(6 * 64), 0, c.stream, c.g, c.gp, csw, t0, t1);
    LAPH_TRY(check_launch("clover_build_kernel"));
    double *diag = c.mass_diag();
    int *d_bad = c.bad_flag();
    LAPH_HIP(hipMemsetAsync(d_bad, 0, sizeof(int), c.stream));
    std::vector<double> hdiag(n_mass);
    for (int m = 0; m < n_mass; ++m) {
        hdiag[m] = 4.0 + m0[m];
        for (int p = 0; p < 2; ++p) {
            dim3 gi((c.g.vh + kSetupBlock - 1) / kSetupBlock, 2);
            hipLaunchKernelGGL(clover_invert_kernel, gi, dim3(kSetupBlock), 0, c.stream, c.g.vh,
                               (const char *)c.clover_term(p), 4.0 + m0[m], const_cast<char *>(c.clover_inv64(m, p)),
                               const_cast<char *>(c.clover_inv32(m, p)), d_bad);
            LAPH_TRY(check_launch("clover_invert_kernel"));
        }
    }
    LAPH_HIP(hipMemcpyAsync(diag, hdiag.data(), n_mass * sizeof(double), hipMemcpyHostToDevice, c.stream));
    int hbad = 0;
    LAPH_HIP(hipMemcpyAsync(&hbad, d_bad, sizeof(int), hipMemcpyDeviceToHost, c.stream));
    LAPH_HIP(hipStreamSynchronize(c.stream));
    if (hbad) {
        c.n_mass = 0;
        return set_error(LAPH_ERR_INVALID, "clover block not positive definite (4 + m0 too small?)");
    }
    c.n_mass = n_mass;
    c.csw = csw;
    c.m0.assign(m0, m0 + n_mass);
    return LAPH_OK;
}

// ---------------------------------------------------------------------------
// spinor pack / unpack
// ---------------------------------------------------------------------------
template <class P>
__global__ void pack_kernel(Geom g, Operand out, const double2 *in, size_t in_rhs_stride, int parity, int nparity) {
    using R = typename P::real;
    const int h = blockIdx.x * kSetupBlock + threadIdx.x;
    const int r = blockIdx.y;
    const int pi = blockIdx.z;
    if (h >= g.vh) return;
    const int p = nparity == 2 ? pi : parity;
    int x, y, z, t;
    site_coords(g, p, h, x, y, z, t);
    const size_t i = (size_t)x + (size_t)g.lx * (y + (size_t)g.ly * (z + (size_t)g.lz * t));
    const double2 *src = in + r * in_rhs_stride + i * 12;
    cplx<R> s[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        double2 v = src[c];
        s[c] = {R(v.x), R(v.y)};
    }
    char *hv = out.at(r) + (nparity == 2 ? pi * (out.stride / 2) : 0);
    SpinorIO<P>::store(hv, g.vh, h, s);
}

template <class P>
__global__ void unpack_kernel(Geom g, double2 *out, size_t out_rhs_stride, Operand in, int parity, int nparity) {
    using R = typename P::real;
    const int h = blockIdx.x * kSetupBlock + threadIdx.x;
    const int r = blockIdx.y;
    const int pi = blockIdx.z;
    if (h >= g.vh) return;
    const int p = nparity == 2 ? pi : parity;
    int x, y, z, t;
    site_coords(g, p, h, x, y, z, t);
    const size_t i = (size_t)x + (size_t)g.lx * (y + (size_t)g.ly * (z + (size_t)g.lz * t));
    const char *hv = in.at(r) + (nparity == 2 ? pi * (in.stride / 2) : 0);
    cplx<R> s[12];
    SpinorIO<P>::load(hv, g.vh, h, s);
    double2 *dst = out + r * out_rhs_stride + i * 12;
#pragma unroll
    for (int c = 0; c < 12; ++c) dst[c] = make_double2((double)s[c].re, (double)s[c].im);
}

laph_status pack_spinor(const Ctx &c, Operand out, const double *in, int prec, int nrhs, int parity,
                        size_t in_rhs_stride_elems) {
    if (nrhs <= 0) return LAPH_OK;
    const int np = parity < 0 ? 2 : 1;
    const size_t stride = in_rhs_stride_elems ? in_rhs_stride_elems : (size_t)2 * c.g.vh * 12;
    dim3 grid((c.g.vh + kSetupBlock - 1) / kSetupBlock, nrhs, np);
    const double2 *src = reinterpret_cast<const double2 *>(in);
    if (prec == LAPH_F64)
        hipLaunchKernelGGL(pack_kernel<F64>, grid, dim3(kSetupBlock), 0, c.stream, c.g, out, src, stride, parity, np);
    else if (prec == LAPH_F32)
        hipLaunchKernelGGL(pack_kernel<F32>, grid, dim3(kSetupBlock), 0, c.stream, c.g, out, src, stride, parity, np);
    else
        hipLaunchKernelGGL(pack_kernel<F16N>, grid, dim3(kSetupBlock), 0, c.stream, c.g, out, src, stride, parity, np);
    return check_launch("pack_kernel");
}

laph_status unpack_spinor(const Ctx &c, double *out, Operand in, int prec, int nrhs, int parity,
                          size_t out_rhs_stride_elems) {
    if (nrhs <= 0) return LAPH_OK;
    const int np = parity < 0 ? 2 : 1;
    const size_t stride = out_rhs_stride_elems ? out_rhs_stride_elems : (size_t)2 * c.g.vh * 12;
    dim3 grid((c.g.vh + kSetupBlock - 1) / kSetupBlock, nrhs, np);
    double2 *dst = reinterpret_cast<double2 *>(out);
    if (prec == LAPH_F64)
        hipLaunchKernelGGL(unpack_kernel<F64>, grid, dim3(kSetupBlock), 0, c.stream, c.g, dst, stride, in, parity, np);
    else if (prec == LAPH_F32)
        hipLaunchKernelGGL(unpack_kernel<F32>, grid, dim3(kSetupBlock), 0, c.stream, c.g, dst, stride, in, parity, np);
    else
        hipLaunchKernelGGL(unpack_kernel<F16N>, grid, dim3(kSetupBlock), 0, c.stream, c.g, dst, stride, in, parity,
                           np);
    return check_launch("unpack_kernel");
}

}  // namespace laph

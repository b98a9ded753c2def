// ugks_kernels.hip -- gfx950 kernels of the memory-saving UGKS time step.
//
// Reference: Zhang, Wei, Long, Xu, "An efficiency and memory-saving
// programming paradigm for the unified gas-kinetic scheme", arXiv:2412.06546.
//
// One step (Algorithm 1 of Section 3.2) on one stream:
//   k_cell_grad  per cell:  limited least-squares gradient of W (the
//                           macroscopic reconstruction)
//   k_face_eq    per face:  interface equilibrium g0, its space and time
//                           slopes, heat flux and time integrals
//   then the velocity loop and the updates after it, by one of two sweeps:
//   push sweep   (default)  each cell computes its own limited slope of f
//                once per velocity and, for every face the velocity leaves
//                through, the interface flux of Eq. fullSolution integrated
//                over the step, added with atomic adds into the stage-1 sums
//                (Eq. microS1) of both of the face's cells: k_push_wall (wall
//                densities), k_push_brick / k_push_pf / k_push (per colour class
//                of cells, or one launch of all cells), then k_push_final
//                (W^{n+1}, q^{n+1}, stage 2 of Eq. microS2);
//   gather sweep k_sweep    per cell, one workgroup owning the cell's whole
//                velocity slab: for every velocity the limited slope of f is
//                rebuilt in registers (own cell, and upwind neighbours when
//                the neighbour is upwind), the stage-1 value is kept in
//                registers, the wall density is reduced over velocities,
//                W^{n+1} and q^{n+1} come from workgroup reductions of the
//                same registers, and stage 2 is applied before the single
//                store.
// f is stored [cell][component][velocity]; lanes run over velocities, so a
// wavefront reads 64 consecutive velocities of one cell (coalesced) and all
// geometry and face data are wave-uniform (scalar loads).  f^n and the
// stage-1 sums (push) or f^{n+1} (gather) are in two buffers, or one buffer
// and a ring of one velocity chunk in place: no slope or residual of f ever
// reaches memory.
#include "ugks_internal.h"

#include <algorithm>
#include <mutex>

#include <cfloat>
#include <cmath>

namespace ugx {

constexpr double kPi = 3.14159265358979323846;
constexpr int N_DOF = 3;  // translational + internal degrees of freedom (monatomic)

// ------------------------------------------------------------------------
// storage types of f: FP64, FP32 or bfloat16 (all arithmetic is FP64)
// ------------------------------------------------------------------------
struct bf16s {
    unsigned short bits;
};
__device__ __forceinline__ double to_f64(double x) { return x; }
__device__ __forceinline__ double to_f64(float x) { return (double)x; }
__device__ __forceinline__ double to_f64(bf16s x) { return (double)__uint_as_float((unsigned)x.bits << 16); }

// The value itself, opaque to the compiler: a multiply that produced it can
// no longer be fused into a later add or subtract, so arithmetic on it sees
// the rounded value -- as it does when the value is read back from memory.
__device__ __forceinline__ double opaque(double x)
{
    asm volatile("" : "+v"(x));
    return x;
}

template <typename FT> __device__ __forceinline__ FT from_f64(double x);
template <> __device__ __forceinline__ double from_f64<double>(double x) { return x; }
template <> __device__ __forceinline__ float from_f64<float>(double x) { return (float)x; }
// Round to nearest, ties to even, directly from FP64 to the 8 significant
// bits of bfloat16: round the FP64 significand at its bit 45, then the
// result is exact in FP32 and its upper half is the bfloat16 pattern
// (values below the FP32 normal range are flushed to signed zero).
template <> __device__ __forceinline__ bf16s from_f64<bf16s>(double x)
{
    if (x != x) return bf16s{0x7fc0};
    unsigned long long u = (unsigned long long)__double_as_longlong(x);
    u += 0x00000fffffffffffull + ((u >> 45) & 1ull);
    u &= ~0x00001fffffffffffull;
    const double r = __longlong_as_double((long long)u);
    const float f = fabs(r) < 1.1754943508222875e-38 ? copysignf(0.0f, (float)r) : (float)r;
    return bf16s{(unsigned short)(__float_as_uint(f) >> 16)};
}

// ------------------------------------------------------------------------
// small helpers
// ------------------------------------------------------------------------
template <int D> __device__ __forceinline__ double pow_lam_pi(double lam)
{
    double r = lam / kPi;
    if constexpr (D == 2) return r;
    else return r * sqrt(r);
}

template <int BS, int N, typename Op>
__device__ __forceinline__ void block_reduce(double (&v)[N], double *lds, Op op)
{
    // butterfly inside the wavefront, then the wavefront results in fixed order
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[n] = op(v[n], __shfl_xor(v[n], off, 64));
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int n = 0; n < N; ++n) lds[wid * N + n] = v[n];
    __syncthreads();
#pragma unroll
    for (int n = 0; n < N; ++n) {
        double s = lds[n];
#pragma unroll
        for (int w = 1; w < BS / 64; ++w) s = op(s, lds[w * N + n]);
        v[n] = s;
    }
    __syncthreads();
}

struct OpAdd {
    __device__ double operator()(double a, double b) const { return a + b; }
};
struct OpMax {
    __device__ double operator()(double a, double b) const { return fmax(a, b); }
};

template <int D> struct Prim {
    double rho, U[D], lam;
};

template <int D> __device__ __forceinline__ Prim<D> to_prim(const double *W)
{
    Prim<D> p;
    p.rho = W[0];
    double ke = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        p.U[d] = W[1 + d] / p.rho;
        ke = fma(p.U[d], p.U[d], ke);  // (which product of a sum is fused may not be left to each kernel)
    }
    p.lam = N_DOF * p.rho / (4.0 * fma(-0.5 * p.rho, ke, W[D + 1]));
    return p;
}

__device__ __forceinline__ double collision_time(double rho, double lam, double mu_ref, double omega)
{
    double T = 1.0 / lam;
    return mu_ref * pow(T, omega) / (0.5 * rho * T);
}

// Reduced Maxwellian and Shakhov correction at u (Section 2.2):
// H = pref e^{-lam c^2}, B = M/(2 lam) H,
// H+ = shk (c.q)(2 lam c^2 - 2 - D) H, B+ = shk (c.q)(2 lam c^2 - D) M H / (2 lam)
template <int D>
__device__ __forceinline__ void equilibrium(const double (&u)[D], const double (&U)[D], double lam, double pref,
                                            double shk, const double (&q)[D], double &Hp, double &Bp)
{
    constexpr int M = Dim<D>::M;
    double c2 = 0.0, cq = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        double c = u[d] - U[d];
        c2 += c * c;
        cq += c * q[d];
    }
    double H = pref * exp(-lam * c2);
    double s = shk * cq;
    Hp = H + s * (2.0 * lam * c2 - 2.0 - D) * H;
    if constexpr (M > 0) {
        double B = (M / (2.0 * lam)) * H;
        Bp = B + s * (2.0 * lam * c2 - D) * B;
    } else {
        Bp = 0.0;
    }
}

// ------------------------------------------------------------------------
// limited least-squares slope of f_k in cell c (Section 3.1, step 2)
// ------------------------------------------------------------------------
// Reciprocal to full double precision: hardware estimate and two Newton steps.
__device__ __forceinline__ double rcp_nr(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    r = fma(r, fma(-x, r, 1.0), r);
    return r;
}

// The stencil of cell c at velocity k: its own value, then one value per face
// slot.  A slot without a neighbour (boundary face, or no face: nb = -1) reads
// the cell's own value, whose difference from it is exactly zero and whose
// least-squares weight is zero, so every load is issued and none sits behind a
// branch.  Loads take a uniform base and a 32-bit byte offset (a cell's slab
// is far below 4 GiB).  The sweep loads the next velocity's stencil while it
// works on the current one; limited_slope = load_stencil + slope_from.
template <typename FT> __device__ __forceinline__ FT load_at(const FT *__restrict__ base, unsigned idx)
{
    return *reinterpret_cast<const FT *>(reinterpret_cast<const char *>(base) + idx * (unsigned)sizeof(FT));
}

// The values stay in their storage type until the slope uses them: widened on
// arrival, a prefetched FP32 stencil takes twice the registers, and where that
// made the gather sweep spill, the reload inside its velocity loop waited for
// the prefetch behind it as well (20,000 cells x 3,600 in 2D with FP32 f: 3.20
// ms a step, 2.12 without).
template <int D, typename FT> struct Stencil {
    FT v0[Dim<D>::NC], vn[Dim<D>::MF][Dim<D>::NC];
};

template <int D, typename FT>
__device__ __forceinline__ void load_stencil(const CellGeo<D> &g, int c, const FT *__restrict__ f, int nv, int k,
                                             Stencil<D, FT> &s)
{
    constexpr int NC = Dim<D>::NC, MF = Dim<D>::MF;
    const FT *fcell = f + (size_t)c * NC * nv;
#pragma unroll
    for (int m = 0; m < NC; ++m) s.v0[m] = load_at(fcell, (unsigned)(m * nv + k));
#pragma unroll
    for (int j = 0; j < MF; ++j) {
        const int n = g.nb[j];
        const FT *fnb = f + (size_t)(n < 0 ? c : n) * NC * nv;
#pragma unroll
        for (int m = 0; m < NC; ++m) s.vn[j][m] = load_at(fnb, (unsigned)(m * nv + k));
    }
}

template <int D, typename FT>
__device__ __forceinline__ void slope_from(const CellGeo<D> &g, int limiter, const Stencil<D, FT> &st,
                                           double (&fc)[Dim<D>::NC], double (&gr)[Dim<D>::NC][D])
{
    constexpr int NC = Dim<D>::NC, MF = Dim<D>::MF;
    // extremes of the differences f_j - f_i (0 for the cell itself): equal to
    // max_j f_j - f_i and min_j f_j - f_i, as rounding is monotone
    double up[NC], dn[NC];
#pragma unroll
    for (int m = 0; m < NC; ++m) {
        fc[m] = to_f64(st.v0[m]);
        up[m] = dn[m] = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) gr[m][d] = 0.0;
    }
    const int nf = g.nf;
    // a cell has at least D + 1 faces; the slots beyond are skipped
#pragma unroll
    for (int j = 0; j < MF; ++j) {
        if (j > D && j >= nf) break;
#pragma unroll
        for (int m = 0; m < NC; ++m) {
            const double df = to_f64(st.vn[j][m]) - fc[m];
#pragma unroll
            for (int d = 0; d < D; ++d) gr[m][d] = fma(g.lsq[j][d], df, gr[m][d]);
            up[m] = fmax(up[m], df);
            dn[m] = fmin(dn[m], df);
        }
    }
    if (!limiter) return;
    // phi = min(1, min over faces of the Venkatakrishnan factor
    //   (dp^2 + e + 2 dm dp) / (dp^2 + e + 2 dm^2 + dm dp)),
    // dp = up or dn by the sign of the face increment dm.  For a given sign
    // min(1, factor) never grows with |dm|: the factor is at least 1 up to
    // |dm| = |dp| / 2, and beyond that its derivative has the sign of
    // a^3 + a e - 4 a x^2 - 4 a^2 x - 4 x e < 0 (a = |dp|, x = |dm|).  So the
    // two extreme increments decide, and the factor is evaluated twice
    // instead of once per face (60 VALU instructions fewer per hexahedron
    // and velocity).  The fractions are compared by cross-multiplication
    // (denominators are positive); a sign without an increment gives
    // num = den and never wins.
#pragma unroll
    for (int m = 0; m < NC; ++m) {
        double hi = 0.0, lo = 0.0;
#pragma unroll
        for (int j = 0; j < MF; ++j) {
            if (j > D && j >= nf) break;
            double dm = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) dm = fma(gr[m][d], g.dvec[j][d], dm);
            hi = fmax(hi, dm);
            lo = fmin(lo, dm);
        }
        double bn = 1.0, bd = 1.0;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const double dm = s == 0 ? hi : lo, dp = s == 0 ? up[m] : dn[m];
            const double dp2e = fma(dp, dp, g.eps2);
            const double num = fma(2.0 * dm, dp, dp2e);
            const double den = fma(dm, fma(2.0, dm, dp), dp2e);
            const bool take = num * bd < bn * den;
            bn = take ? num : bn;
            bd = take ? den : bd;
        }
        const double phi = bn * rcp_nr(bd);
#pragma unroll
        for (int d = 0; d < D; ++d) gr[m][d] *= phi;
    }
}

template <int D, typename FT>
__device__ __forceinline__ void limited_slope(const CellGeo<D> &g, int c, const FT *__restrict__ f, int nv, int k,
                                              int limiter, double (&fc)[Dim<D>::NC], double (&gr)[Dim<D>::NC][D])
{
    Stencil<D, FT> st;
    load_stencil<D, FT>(g, c, f, nv, k, st);
    slope_from<D, FT>(g, limiter, st, fc, gr);
}

// Shakhov equilibrium f+ = H + H+ (and B + B+) at u, given the reduced
// Maxwellian value H there (Section 2.2):
// H+ = shk (c.q)(2 lam c^2 - 2 - D) H, B = M/(2 lam) H,
// B+ = shk (c.q)(2 lam c^2 - D) B, with shk = 4 (1 - Pr) lam^2 / (5 rho).
// Every multiply-add is written out: the push sweep's base and final kernels
// have to form the same bits, which may not hang on what the compiler fuses.
template <int D>
__device__ __forceinline__ void shakhov_at(const double (&c)[D], double c2, double lam, double shk, const double (&q)[D],
                                           double bh, double H, double &fh, double &fb)
{
    constexpr int M = Dim<D>::M;
    double cq = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) cq = fma(c[d], q[d], cq);
    const double s = shk * cq, l = 2.0 * lam;
    fh = fma(s * fma(l, c2, -(2.0 + D)), H, H);
    if constexpr (M > 0) {
        const double B = bh * H;  // bh = M / (2 lam)
        fb = fma(s * fma(l, c2, -(double)D), B, B);
    } else {
        fb = 0.0;
    }
}

// the peculiar velocity about U and its square
template <int D>
__device__ __forceinline__ void peculiar(const double (&u)[D], const double *U, double (&c)[D], double &c2)
{
    c2 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        c[d] = u[d] - U[d];
        c2 = fma(c[d], c[d], c2);
    }
}

template <int D>
__device__ __forceinline__ void shakhov(const double (&u)[D], const double (&U)[D], double lam, double shk,
                                        const double (&q)[D], double bh, double H, double &fh, double &fb)
{
    double c[D], c2;
    peculiar<D>(u, U, c, c2);
    shakhov_at<D>(c, c2, lam, shk, q, bh, H, fh, fb);
}

// The equilibrium part of the time-integrated interface value (Eq.
// fullSolution integrated over [0, dt]) at the peculiar velocity c of the
// face's Maxwellian: G times a cubic in c (FaceEq).  18 FP64 instructions in
// 3D where g0+, u . grad g0 and d_t g0 evaluated one by one took about 50.
template <int D>
__device__ __forceinline__ void face_equilibrium(const FaceEq<D> &e, const double (&c)[D], double c2, double G,
                                                 double (&I)[Dim<D>::NC])
{
    double P = e.k0;
    int t = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        double r = fma(e.k3[a], c2, e.k1[a]);
#pragma unroll
        for (int b = a; b < D; ++b) r = fma(e.k2[t++], c[b], r);
        P = fma(c[a], r, P);
    }
    I[0] = G * P;
    if constexpr (Dim<D>::NC > 1) {
        double B = fma(e.bh, P, e.d0);
#pragma unroll
        for (int a = 0; a < D; ++a) B = fma(e.d1[a], c[a], B);
        I[Dim<D>::NC - 1] = G * B;
    }
}

// The time-integrated interface value of h (and b) at velocity u through an
// interior face: the upwind cell's values f and limited slopes gr, its
// centroid-to-face vector, ug = u . gr; G the face's Gaussian at u.
template <int D>
__device__ __forceinline__ void interface_integral(const FaceEq<D> &e, const double (&u)[D], double G,
                                                   const double (&f)[Dim<D>::NC], const double (&gr)[Dim<D>::NC][D],
                                                   const double *dvec, const double (&ug)[Dim<D>::NC],
                                                   double (&I)[Dim<D>::NC])
{
    double c[D], c2;
    peculiar<D>(u, e.U, c, c2);
    face_equilibrium<D>(e, c, c2, G, I);
#pragma unroll
    for (int m = 0; m < Dim<D>::NC; ++m) {
        double v = f[m];
#pragma unroll
        for (int d = 0; d < D; ++d) v = fma(gr[m][d], dvec[d], v);
        I[m] = fma(e.c0, v, fma(e.c1, ug[m], I[m]));
    }
}

// Free transport of the reconstruction over the step, out through a boundary face.
template <int D>
__device__ __forceinline__ void boundary_outgoing(const FaceEq<D> &e, const double (&f)[Dim<D>::NC],
                                                  const double (&gr)[Dim<D>::NC][D], const double *dvec,
                                                  const double (&ug)[Dim<D>::NC], double (&I)[Dim<D>::NC])
{
#pragma unroll
    for (int m = 0; m < Dim<D>::NC; ++m) {
        double v = f[m];
#pragma unroll
        for (int d = 0; d < D; ++d) v = fma(gr[m][d], dvec[d], v);
        I[m] = fma(e.c1, ug[m], e.c0 * v);
    }
}

// u . gr of every component
template <int D>
__device__ __forceinline__ void along(const double (&u)[D], const double (&gr)[Dim<D>::NC][D], double (&ug)[Dim<D>::NC])
{
#pragma unroll
    for (int m = 0; m < Dim<D>::NC; ++m) {
        ug[m] = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) ug[m] = fma(u[d], gr[m][d], ug[m]);
    }
}

// ------------------------------------------------------------------------
// time step: per cell, the largest upwind outflow over the velocities
// ------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void k_cfl(Params p, double *cell_dt)
{
    const int i = blockIdx.x;
    const CellGeo<D> &g = static_cast<const CellGeo<D> *>(p.cgeo)[i];
    const FaceGeo<D> *fg = static_cast<const FaceGeo<D> *>(p.fgeo);
    double mx[1] = {0.0};
    for (int k = threadIdx.x; k < p.nv; k += 256) {
        double out = 0.0;
        for (int j = 0; j < g.nf; ++j) {
            const FaceGeo<D> &F = fg[g.face[j]];
            double un = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) un += p.u[d * p.nv + k] * F.n[d];
            if (g.side[j]) un = -un;
            if (un > 0.0) out += F.area * un;
        }
        mx[0] = fmax(mx[0], out);
    }
    __shared__ double lds[4];
    block_reduce<256>(mx, lds, OpMax{});
    if (threadIdx.x == 0) cell_dt[i] = mx[0] > 0.0 ? (1.0 / g.inv_vol) / mx[0] : DBL_MAX;
}

// ------------------------------------------------------------------------
// initial state: discrete Maxwellian of (rho, U, T)
// ------------------------------------------------------------------------
// One workgroup per cell, threads over its velocities (a thread per
// (cell, velocity) would exceed the 2^32 work-items of one grid dimension on
// the largest meshes).
template <int D, typename FT>
__global__ __launch_bounds__(256) void k_init(Params p, const double *__restrict__ prim0, FT *__restrict__ f)
{
    constexpr int NC = Dim<D>::NC;
    const int i = blockIdx.x;
    const double *pr = prim0 + (size_t)i * (D + 2);
    double U[D], zq[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        U[d] = pr[1 + d];
        zq[d] = 0.0;
    }
    const double lam = 1.0 / pr[D + 1];
    const double pref = pr[0] * pow_lam_pi<D>(lam);
    for (int k = threadIdx.x; k < p.nv; k += 256) {
        double u[D];
#pragma unroll
        for (int d = 0; d < D; ++d) u[d] = p.u[d * p.nv + k];
        double H, B;
        equilibrium<D>(u, U, lam, pref, 0.0, zq, H, B);
        f[((size_t)i * NC + 0) * p.nv + k] = from_f64<FT>(H);
        if constexpr (NC > 1) f[((size_t)i * NC + 1) * p.nv + k] = from_f64<FT>(B);
    }
}

// ------------------------------------------------------------------------
// W and q as direct discrete moments of f (start, or after a set_f)
// ------------------------------------------------------------------------
template <int D, typename FT>
__global__ __launch_bounds__(256) void k_moments(Params p, const FT *__restrict__ f)
{
    constexpr int NC = Dim<D>::NC, NW = D + 2;
    const int i = blockIdx.x;
    __shared__ double lds[4 * NW];
    double m[NW];
#pragma unroll
    for (int n = 0; n < NW; ++n) m[n] = 0.0;
    for (int k = threadIdx.x; k < p.nv; k += 256) {
        double h = to_f64(f[((size_t)i * NC) * p.nv + k]);
        double b = NC > 1 ? to_f64(f[((size_t)i * NC + NC - 1) * p.nv + k]) : 0.0;
        double w = p.w[k], u2 = 0.0;
        m[0] += w * h;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            double ud = p.u[d * p.nv + k];
            m[1 + d] += w * ud * h;
            u2 += ud * ud;
        }
        m[NW - 1] += w * 0.5 * (u2 * h + b);
    }
    block_reduce<256>(m, lds, OpAdd{});
    Prim<D> pr = to_prim<D>(m);
    double qq[D];
#pragma unroll
    for (int d = 0; d < D; ++d) qq[d] = 0.0;
    for (int k = threadIdx.x; k < p.nv; k += 256) {
        double h = to_f64(f[((size_t)i * NC) * p.nv + k]);
        double b = NC > 1 ? to_f64(f[((size_t)i * NC + NC - 1) * p.nv + k]) : 0.0;
        double c[D], c2 = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            c[d] = p.u[d * p.nv + k] - pr.U[d];
            c2 += c[d] * c[d];
        }
        double wt = 0.5 * p.w[k] * (c2 * h + b);
#pragma unroll
        for (int d = 0; d < D; ++d) qq[d] += wt * c[d];
    }
    block_reduce<256>(qq, lds, OpAdd{});
    if (threadIdx.x == 0) {
#pragma unroll
        for (int n = 0; n < NW; ++n) p.W[(size_t)i * NW + n] = m[n];
#pragma unroll
        for (int d = 0; d < D; ++d) p.q[(size_t)i * D + d] = qq[d];
    }
}

// ------------------------------------------------------------------------
// Algorithm 1, macroscopic reconstruction: limited gradients of the conservative variables
// ------------------------------------------------------------------------
// The constants of f+^n and of the source in cell i.
template <int D> __device__ __forceinline__ CellConst<D> cell_const(const Params &p, int i)
{
    const Prim<D> pn = to_prim<D>(p.W + (size_t)i * (D + 2));
    CellConst<D> c;
#pragma unroll
    for (int d = 0; d < D; ++d) c.U[d] = pn.U[d];
    c.lam = pn.lam;
    c.pref = pn.rho * pow_lam_pi<D>(pn.lam);
    c.shk = 4.0 * (1.0 - p.Pr) * pn.lam * pn.lam / (5.0 * pn.rho);
    c.hdt_tau = 0.5 * p.dt / collision_time(pn.rho, pn.lam, p.mu_ref, p.omega);
    return c;
}

template <int D>
__device__ __forceinline__ void cell_grad(const Params p, int i)
{
    constexpr int NW = D + 2, MF = Dim<D>::MF;
    if (i >= p.nc) return;
    if (p.cconst) static_cast<CellConst<D> *>(p.cconst)[i] = cell_const<D>(p, i);
    const CellGeo<D> &g = static_cast<const CellGeo<D> *>(p.cgeo)[i];
    const int nf = g.nf;
    // the cell's W and its neighbours' (the cell's own where a slot has no
    // neighbour: its difference is exactly zero), all loads issued at once
    double Wi[NW], Wn[MF][NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) Wi[m] = p.W[(size_t)i * NW + m];
#pragma unroll
    for (int j = 0; j < MF; ++j) {
        const int n = j < nf ? g.nb[j] : -1;
        const size_t src = (size_t)(n < 0 ? i : n) * NW;
#pragma unroll
        for (int m = 0; m < NW; ++m) Wn[j][m] = p.W[src + m];
    }
    double gr[NW][D];
#pragma unroll
    for (int m = 0; m < NW; ++m) {
        double up = 0.0, dn = 0.0;  // extremes of W_j - W_i (0 for the cell itself)
#pragma unroll
        for (int d = 0; d < D; ++d) gr[m][d] = 0.0;
#pragma unroll
        for (int j = 0; j < MF; ++j) {
            if (j >= nf) break;
            const double df = Wn[j][m] - Wi[m];
#pragma unroll
            for (int d = 0; d < D; ++d) gr[m][d] += g.lsq[j][d] * df;
            up = fmax(up, df);
            dn = fmin(dn, df);
        }
        if (p.limiter) {
            // the two extreme face increments decide (as for f, slope_from);
            // one division a component where every face took one
            double hi = 0.0, lo = 0.0;
#pragma unroll
            for (int j = 0; j < MF; ++j) {
                if (j >= nf) break;
                double dm = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) dm += gr[m][d] * g.dvec[j][d];
                hi = fmax(hi, dm);
                lo = fmin(lo, dm);
            }
            const double nu = up * up + g.eps2 + 2.0 * hi * up, du = up * up + 2.0 * hi * hi + hi * up + g.eps2;
            const double nd = dn * dn + g.eps2 + 2.0 * lo * dn, dd = dn * dn + 2.0 * lo * lo + lo * dn + g.eps2;
            double bn = 1.0, bd = 1.0;
            if (hi > 0.0 && nu < du) {
                bn = nu;
                bd = du;
            }
            if (lo < 0.0 && nd * bd < bn * dd) {
                bn = nd;
                bd = dd;
            }
            const double phi = bn / bd;
#pragma unroll
            for (int d = 0; d < D; ++d) gr[m][d] *= phi;
        }
    }
    // first order where a reconstructed face state is not physical
    bool bad = false;
#pragma unroll
    for (int j = 0; j < MF; ++j) {
        if (j >= nf) break;
        double Wf[NW], ke = 0.0;
#pragma unroll
        for (int m = 0; m < NW; ++m) {
            Wf[m] = Wi[m];
#pragma unroll
            for (int d = 0; d < D; ++d) Wf[m] += gr[m][d] * g.dvec[j][d];
        }
#pragma unroll
        for (int d = 0; d < D; ++d) ke += Wf[1 + d] * Wf[1 + d];
        // rho E > |rho U|^2 / 2, both sides of E > rho U^2 / 2 times rho > 0
        if (!(Wf[0] > 0.0) || !(Wf[NW - 1] * Wf[0] - 0.5 * ke > 0.0)) bad = true;
    }
#pragma unroll
    for (int m = 0; m < NW; ++m)
#pragma unroll
        for (int d = 0; d < D; ++d) p.gW[((size_t)i * NW + m) * D + d] = bad ? 0.0 : gr[m][d];
}

template <int D>
__global__ __launch_bounds__(kGradBlock) void k_cell_grad(Params p)
{
    cell_grad<D>(p, blockIdx.x * kGradBlock + threadIdx.x);
}

// ------------------------------------------------------------------------
// Algorithm 1, interface equilibrium state and time coefficients
// ------------------------------------------------------------------------
// Slopes of a Maxwellian in its own frame: with c = u - U, a quantity
// a . (1, c, (|c|^2 + |xi|^2) / 2) with <(1, c, ..) (a . (1, c, ..))>_g = Delta
// for the rho-normalised moments of g (N = 3 degrees of freedom), s = 1 / (2 lam), is = 1 / s;
// Dl holds Delta for (1, u, |u|^2 / 2 + |xi|^2 / 2), as a gradient of W / rho is given.
template <int D>
__device__ __forceinline__ void slope_solve(const double (&U)[D], double s, double is, const double *Dl, double (&a)[D + 2])
{
    constexpr int NW = D + 2;
    double U2 = 0.0, Um = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        U2 = fma(U[d], U[d], U2);
        Um = fma(U[d], Dl[1 + d], Um);
        a[1 + d] = (Dl[1 + d] - U[d] * Dl[0]) * is;
    }
    const double De = Dl[NW - 1] - Um + 0.5 * U2 * Dl[0];
    a[NW - 1] = (De - 0.5 * N_DOF * s * Dl[0]) * (2.0 / N_DOF * is * is);
    a[0] = Dl[0] - 0.5 * N_DOF * s * a[NW - 1];
}

// Time slope from the compatibility condition <psi (u . grad g0 + d_t g0)> = 0
// (Section 2.4), in the same frame: the right side
// -sum_d <(1, c, ..) (U_d + c_d) (a^d . (1, c, ..))> by the Maxwellian's even
// moments <c_i c_j> = s, <e> = N s / 2, <c_i c_j e> = (N + 2) s^2 / 2,
// <e^2> = N (N + 2) s^2 / 4, then the same solve.
template <int D>
__device__ __forceinline__ void time_slope(const double (&U)[D], double s, double is, const double (&a)[D][D + 2],
                                           double (&A)[D + 2])
{
    constexpr int NW = D + 2, N = N_DOF;
    double r0 = 0.0, re = 0.0, rb[D];
#pragma unroll
    for (int b = 0; b < D; ++b) rb[b] = -(s * a[b][0] + 0.5 * (N + 2) * s * s * a[b][NW - 1]);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        r0 -= U[d] * (a[d][0] + 0.5 * N * s * a[d][NW - 1]) + s * a[d][1 + d];
        re -= U[d] * (0.5 * N * s * a[d][0] + 0.25 * N * (N + 2) * s * s * a[d][NW - 1]) +
              0.5 * (N + 2) * s * s * a[d][1 + d];
#pragma unroll
        for (int b = 0; b < D; ++b) rb[b] -= s * U[d] * a[d][1 + b];
    }
#pragma unroll
    for (int b = 0; b < D; ++b) A[1 + b] = rb[b] * is;
    A[NW - 1] = (re - 0.5 * N * s * r0) * (2.0 / N * is * is);
    A[0] = r0 - 0.5 * N * s * A[NW - 1];
}

__device__ __forceinline__ void time_integrals(double dt, double tau, double *c)
{
    const double x = dt / tau;
    if (x < 1.0) {
        // Taylor series (the closed forms cancel catastrophically for small
        // x): with e_m = (-1)^(m+1) / m!,
        //   sum_{m>=1} e_m x^m, sum_{m>=2} (m-1) e_m x^m, -sum_{m>=2} e_m x^m,
        //   -sum_{m>=3} (m-2) e_m x^m, sum_{m>=3} e_m x^m
        // by Horner's rule, without their leading powers of x.  The terms left
        // out after m = 22 are below 1e-19 of the first.
        constexpr int M = 22;
        double inv = 1.0;
#pragma unroll
        for (int m = 2; m <= M; ++m) inv /= m;  // 1 / M!, folded at compile time
        double s1 = 0, s2 = 0, s3 = 0, s4 = 0, s5 = 0;
#pragma unroll
        for (int m = M; m >= 1; --m) {
            const double e = (m & 1) ? inv : -inv;
            s1 = fma(s1, x, e);
            if (m >= 2) {
                s2 = fma(s2, x, (m - 1) * e);
                s3 = fma(s3, x, -e);
            }
            if (m >= 3) {
                s4 = fma(s4, x, -(m - 2) * e);
                s5 = fma(s5, x, e);
            }
            inv *= m;
        }
        c[0] = dt * s1;              // tau x = dt
        c[1] = dt * dt * s2;
        c[2] = dt * x * s3;
        c[3] = dt * dt * x * s4;
        c[4] = dt * dt * x * s5;
    } else {
        const double e = exp(-x), ome = -expm1(-x);
        c[0] = tau * ome;
        c[1] = tau * dt * e - tau * tau * ome;
        c[2] = dt - tau * ome;
        c[3] = 2.0 * tau * tau * ome - tau * dt * (1.0 + e);
        c[4] = 0.5 * dt * dt - tau * dt + tau * tau * ome;
    }
}

template <int D>
__device__ __forceinline__ void face_eq(const Params p, int f)
{
    constexpr int NW = D + 2;
    if (f >= p.nf) return;
    const FaceGeo<D> &F = static_cast<const FaceGeo<D> *>(p.fgeo)[f];
    FaceEq<D> &e = static_cast<FaceEq<D> *>(p.feq)[f];
    if (F.bc != 0) {
        // boundary: store the Maxwellian the incoming particles come from
        double rho, U[D], lam;
        if (F.bc == 2) {
            Prim<D> pr = to_prim<D>(p.W + (size_t)F.l * NW);
            rho = pr.rho;
            lam = pr.lam;
            for (int d = 0; d < D; ++d) U[d] = pr.U[d];
        } else {
            const double *bp = p.bc_prim + (size_t)F.bcid * NW;
            rho = F.bc == 3 ? 1.0 : bp[0];
            for (int d = 0; d < D; ++d) U[d] = bp[1 + d];
            lam = 1.0 / bp[NW - 1];
        }
        // (the coefficients not written here are zero since creation)
        e.lam = lam;
        for (int d = 0; d < D; ++d) e.U[d] = U[d];
        e.c0 = p.dt;
        e.c1 = -0.5 * p.dt * p.dt;
        e.k0 = p.dt * rho * pow_lam_pi<D>(lam);
        if constexpr (Dim<D>::M > 0) e.bh = Dim<D>::M / (2.0 * lam);
        return;
    }
    // reconstructed states on both sides
    double Wl[NW], Wr[NW], gl[NW][D], gr[NW][D];
#pragma unroll
    for (int m = 0; m < NW; ++m) {
        Wl[m] = p.W[(size_t)F.l * NW + m];
        Wr[m] = p.W[(size_t)F.r * NW + m];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            gl[m][d] = p.gW[((size_t)F.l * NW + m) * D + d];
            gr[m][d] = p.gW[((size_t)F.r * NW + m) * D + d];
        }
    }
#pragma unroll
    for (int m = 0; m < NW; ++m)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            Wl[m] += gl[m][d] * F.dl[d];
            Wr[m] += gr[m][d] * F.dr[d];
        }
    // W0 from the two half-Maxwellians in the face-normal frame
    double W0[NW];
    for (int m = 0; m < NW; ++m) W0[m] = 0.0;
    for (int side = 0; side < 2; ++side) {
        Prim<D> pr = to_prim<D>(side == 0 ? Wl : Wr);
        double Un = 0.0;
        for (int d = 0; d < D; ++d) Un += pr.U[d] * F.n[d];
        double Ut[D], ut2 = 0.0;
        for (int d = 0; d < D; ++d) {
            Ut[d] = pr.U[d] - Un * F.n[d];
            ut2 += Ut[d] * Ut[d];
        }
        const double t = sqrt(pr.lam) * Un;
        const double g = exp(-pr.lam * Un * Un) / (2.0 * sqrt(kPi * pr.lam));
        double m0, m1;
        if (side == 0) {
            m0 = 0.5 * erfc(-t);
            m1 = Un * m0 + g;
        } else {
            m0 = 0.5 * erfc(t);
            m1 = Un * m0 - g;
        }
        const double m2 = Un * m1 + m0 / (2.0 * pr.lam);
        W0[0] += pr.rho * m0;
        for (int d = 0; d < D; ++d) W0[1 + d] += pr.rho * (m1 * F.n[d] + Ut[d] * m0);
        W0[NW - 1] += 0.5 * pr.rho * (m2 + (ut2 + (N_DOF - 1) / (2.0 * pr.lam)) * m0);
    }
    const Prim<D> p0 = to_prim<D>(W0);
    const double is = 2.0 * p0.lam, s = 1.0 / is, half_rho = 0.5 / p0.rho;
    // spatial slopes from the averaged limited gradients, the time slope
    double a[D][NW], A[NW], q[D], c[5];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        double Dl[NW];
#pragma unroll
        for (int m = 0; m < NW; ++m)
            Dl[m] = half_rho * (gl[m][d] + gr[m][d]);
        slope_solve<D>(p0.U, s, is, Dl, a[d]);
        q[d] = 0.5 * (p.q[(size_t)F.l * D + d] + p.q[(size_t)F.r * D + d]);
    }
    time_slope<D>(p0.U, s, is, a, A);
    time_integrals(p.dt, collision_time(p0.rho, p0.lam, p.mu_ref, p.omega), c);
    // the cubic in c: c[2] (1 + Shakhov) + c[3] u . a + c[4] A.  Integrated
    // over xi the energy moment (|c|^2 + |xi|^2) / 2 becomes
    // (|c|^2 + M s) / 2 for h and (|c|^2 + (M + 2) s) / 2 for b = M s h.
    constexpr int M = Dim<D>::M;
    const double pref = p0.rho * pow_lam_pi<D>(p0.lam);
    const double sh = c[2] * 4.0 * (1.0 - p.Pr) * p0.lam * p0.lam / (5.0 * p0.rho);  // Shakhov's factor
    const double th = 0.5 * M * s;
    double Ua0 = 0.0, UaE = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        Ua0 += p0.U[d] * a[d][0];
        UaE += p0.U[d] * a[d][NW - 1];
    }
    const double e2 = c[3] * UaE + c[4] * A[NW - 1];  // factor of the energy moment
    e.lam = p0.lam;
    e.c0 = c[0];
    e.c1 = c[1];
    e.k0 = pref * (c[2] + c[3] * Ua0 + c[4] * A[0] + th * e2);
    int t = 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        e.U[d] = p0.U[d];
        double lin = a[d][0] + th * a[d][NW - 1];
#pragma unroll
        for (int b = 0; b < D; ++b) lin += p0.U[b] * a[b][1 + d];
        e.k1[d] = pref * (c[3] * lin + c[4] * A[1 + d] - sh * (2.0 + D) * q[d]);
        e.k3[d] = pref * (0.5 * c[3] * a[d][NW - 1] + 2.0 * sh * p0.lam * q[d]);
#pragma unroll
        for (int b = d; b < D; ++b)
            e.k2[t++] = pref * (b == d ? c[3] * a[d][1 + d] + 0.5 * e2 : c[3] * (a[d][1 + b] + a[b][1 + d]));
    }
    if constexpr (M > 0) {
        e.bh = M * s;
        e.d0 = e.bh * pref * s * e2;
#pragma unroll
        for (int d = 0; d < D; ++d) e.d1[d] = e.bh * pref * (c[3] * s * a[d][NW - 1] + 2.0 * sh * q[d]);
    }
}

template <int D>
__global__ __launch_bounds__(kFaceBlock) void k_face_eq(Params p)
{
    face_eq<D>(p, blockIdx.x * kFaceBlock + threadIdx.x);
}

// ------------------------------------------------------------------------
// Algorithm 1 from the velocity loop on, fused: the sweep over one cell's velocity slab
// ------------------------------------------------------------------------
// Unit-density Gaussian exp(-lam |u_k - U|^2).  On a Cartesian velocity grid
// it is the product of one-dimensional factors, tabulated in LDS once per
// workgroup (nx + ny [+ nz] exponentials instead of nx * ny [* nz]).
template <int D, bool TENSOR> struct Gauss {
    const double *tab;  // LDS tables, ntab doubles each
    int ntab;
    __device__ __forceinline__ double operator()(int t, unsigned kx, const double (&u)[D], double lam,
                                                 const double *U) const
    {
        if constexpr (TENSOR) {
            const double *tb = tab + t * ntab;
            double g = tb[kx & 1023u] * tb[kx >> 10 & 1023u];
            if constexpr (D == 3) g *= tb[kx >> 20];
            return g;
        } else {
            double c2 = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const double c = u[d] - U[d];
                c2 += c * c;
            }
            return exp(-lam * c2);
        }
    }
};

// One workgroup per cell; threads stride over the cell's velocities.
//   wall:   (wall cells only) incident and unit-density reflected mass fluxes
//           summed over velocities -> wall density;
//   pass 1: for each velocity, limited slopes (own cell, and the upwind
//           neighbour where it is upwind), the time-integrated flux through
//           every face, the stage-1 value -> written to f_out; moments of the
//           net outflow accumulated on the fly;
//   macro:  workgroup reduction -> W^{n+1}, tau^{n+1};
//   heat:   each thread re-reads its stage-1 values -> q^{n+1};
//   pass 2: each thread re-reads its stage-1 values, applies stage 2 and
//           writes f^{n+1}.
// Pass 1 parks the stage-1 values in LDS when the cell's slab fits there
// beside the tables with four workgroups per CU (then f_out is written once),
// otherwise in f_out itself.
#ifndef UGKS_XCDS
#define UGKS_XCDS 8  // accelerator complex dies of an MI355X
#endif
#ifndef UGKS_XCD_RUN
#define UGKS_XCD_RUN 32
#endif
// S1L: the stage-1 values of the cell are kept in LDS (when the slab fits
// beside the tables without costing occupancy), else in f_out until stage 2.
// Workgroups are dealt to the XCDs round-robin; hand each XCD runs of
// UGKS_XCD_RUN consecutive cells, so that mesh neighbours (whose slabs every
// workgroup re-reads) mostly meet in the same L2 while the runs, interleaved
// over the XCDs, keep the load balanced.  b is the workgroup's index within
// its case's grid, which starts at a multiple of UGKS_XCDS * UGKS_XCD_RUN.
__device__ __forceinline__ int xcd_cell(int b)
{
    const int t = b / UGKS_XCDS;
    return ((t / UGKS_XCD_RUN) * UGKS_XCDS + b % UGKS_XCDS) * UGKS_XCD_RUN + t % UGKS_XCD_RUN;
}

// The workgroup's index where the workgroups of a launch go in rows (cell_grid)
__device__ __forceinline__ int row_block() { return (int)(blockIdx.y * gridDim.x + blockIdx.x); }

// Per-cell constants of a step (uniform in the workgroup): W^n, the
// primitive state, tau^n, q^n and the coefficients of f+^n and of the source.
template <int D> struct CellStep {
    static constexpr int NW = D + 2;
    double Wn[NW];
    Prim<D> pn;
    double qn[D];
    double pref_n, shk_n, hdt_tau, bh_n;
};

template <int D> __device__ __forceinline__ CellStep<D> cell_step(const Params &p, int i)
{
    constexpr int NW = D + 2;
    CellStep<D> s;
#pragma unroll
    for (int m = 0; m < NW; ++m) s.Wn[m] = p.W[(size_t)i * NW + m];
    s.pn = to_prim<D>(s.Wn);
    const double tau_n = collision_time(s.pn.rho, s.pn.lam, p.mu_ref, p.omega);
#pragma unroll
    for (int d = 0; d < D; ++d) s.qn[d] = p.q[(size_t)i * D + d];
    s.pref_n = s.pn.rho * pow_lam_pi<D>(s.pn.lam);
    s.shk_n = 4.0 * (1.0 - p.Pr) * s.pn.lam * s.pn.lam / (5.0 * s.pn.rho);
    s.hdt_tau = 0.5 * p.dt / tau_n;
    s.bh_n = Dim<D>::M / (2.0 * s.pn.lam);
    return s;
}

// One-dimensional Gaussian factors of every face's Maxwellian and of f+^n
// (tables 0..MF-1: the face slots, table MF: the cell); no barrier inside.
template <int D, int BS>
__device__ __forceinline__ void fill_tables(const Params &p, const CellGeo<D> &gi, double lam_c, double U0, double U1,
                                            double U2, double *tab)
{
    constexpr int NT = Dim<D>::MF + 1;
    const FaceEq<D> *fe = static_cast<const FaceEq<D> *>(p.feq);
    const int ntab = p.ntab, nf = gi.nf;
    for (int t = threadIdx.x; t < NT * ntab; t += BS) {
        const int which = t / ntab, idx = t - which * ntab;
        const int ax = idx < p.n1d[0] ? 0 : (idx < p.n1d[0] + p.n1d[1] ? 1 : 2);
        double lam, Ud;
        if (which < nf) {
            const FaceEq<D> &e = fe[gi.face[which]];
            lam = e.lam;
            Ud = e.U[0];
            if (ax == 1) Ud = e.U[1];
            if (D == 3 && ax == 2) Ud = e.U[D - 1];
        } else {
            lam = lam_c;
            Ud = ax == 0 ? U0 : (ax == 1 ? U1 : U2);
        }
        const double c = p.u1d[idx] - Ud;
        tab[t] = exp(-lam * c * c);
    }
}

// (the cell's state passed as scalars: a choice between fields of a
// structure would become a load at a chosen address, which keeps the
// structure in scratch memory)
template <int D, int BS>
__device__ __forceinline__ void fill_tables(const Params &p, const CellGeo<D> &gi, const Prim<D> &pn, double *tab)
{
    fill_tables<D, BS>(p, gi, pn.lam, pn.U[0], pn.U[1], pn.U[D - 1], tab);
}

template <int D> __device__ __forceinline__ int has_wall_face(const Params &p, const CellGeo<D> &gi)
{
    const FaceGeo<D> *fg = static_cast<const FaceGeo<D> *>(p.fgeo);
    int w = 0;
    for (int j = 0; j < gi.nf; ++j) w |= (fg[gi.face[j]].bc == 3);
    return w;
}

// Algorithm 1's boundary flux (wall density), for a cell with a wall face: the incident
// particles' mass flux and the unit-density reflected flux, summed over
// velocities; rho_w makes the net mass flux through the wall vanish
// (Eq. maxWalldes).  Knowing rho_w up front, the sweep adds the reflected
// particles directly.  Workgroup-wide (contains barriers).
template <int D, typename FT, int BS, bool TENSOR>
__device__ __forceinline__ void wall_density(const Params &p, const CellGeo<D> &gi, int i, const FT *__restrict__ fin,
                                             const Gauss<D, TENSOR> &gauss, double *red, double (&rho_w)[Dim<D>::MF])
{
    constexpr int NC = Dim<D>::NC, MF = Dim<D>::MF;
    const FaceGeo<D> *fg = static_cast<const FaceGeo<D> *>(p.fgeo);
    const FaceEq<D> *fe = static_cast<const FaceEq<D> *>(p.feq);
    const int nv = p.nv, nf = gi.nf;
    const double dt = p.dt;
    double wsum[2 * MF];
#pragma unroll
    for (int j = 0; j < 2 * MF; ++j) wsum[j] = 0.0;
    for (int k = threadIdx.x; k < nv; k += BS) {
        double u[D];
#pragma unroll
        for (int d = 0; d < D; ++d) u[d] = p.u[d * nv + k];
        const unsigned kx = TENSOR ? (unsigned)p.kidx[k] : 0u;
        const double wk = p.w[k];
        double fi[NC], gri[NC][D];
        limited_slope<D, FT>(gi, i, fin, nv, k, p.limiter, fi, gri);
#pragma unroll
        for (int j = 0; j < MF; ++j) {
            if (j >= nf) break;
            const FaceGeo<D> &F = fg[gi.face[j]];
            if (F.bc != 3) continue;
            double un = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) un += u[d] * F.n[d];
            if (un > 0.0) {
                double v = fi[0], ug = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    v += gri[0][d] * gi.dvec[j][d];
                    ug += u[d] * gri[0][d];
                }
                wsum[2 * j] += wk * un * (dt * v - 0.5 * dt * dt * ug);
            } else {
                const FaceEq<D> &e = fe[gi.face[j]];
                wsum[2 * j + 1] += wk * un * e.k0 * gauss(j, kx, u, e.lam, e.U);
            }
        }
    }
    block_reduce<BS>(wsum, red, OpAdd{});
#pragma unroll
    for (int j = 0; j < MF; ++j) rho_w[j] = (j < nf && wsum[2 * j + 1] != 0.0) ? -wsum[2 * j] / wsum[2 * j + 1] : 0.0;
}

// After pass 1 of cell i: W^{n+1} (Eq. macroscopicUpdata) from the reduced
// moments, tau^{n+1}, q^{n+1} from the stage-1 values re-read, then stage 2
// (Eq. microS2) and the single store of f^{n+1}; tab holds the cell's tables
// (its own f+ table is refreshed for t^{n+1}).  Workgroup-wide.
template <int D, typename FT, int BS, bool TENSOR>
__device__ __forceinline__ void finish_cell(const Params &p, int i, const CellStep<D> &cs, double (&mom)[D + 2],
                                            const FT *s1, double *red, double *tab, const Gauss<D, TENSOR> &gauss,
                                            FT *__restrict__ fout)
{
    constexpr int NC = Dim<D>::NC, MF = Dim<D>::MF, NW = D + 2;
    const CellGeo<D> &gi = static_cast<const CellGeo<D> *>(p.cgeo)[i];
    const int tid = threadIdx.x, nv = p.nv;
    const double dt = p.dt, Pr = p.Pr;
    const size_t base = (size_t)i * NC * nv;

    // Algorithm 1's macroscopic update: Eq. macroscopicUpdata, then tau at t^{n+1}
    block_reduce<BS>(mom, red, OpAdd{});
    double W1[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) W1[m] = cs.Wn[m] - mom[m] * gi.inv_vol;
    const Prim<D> p1 = to_prim<D>(W1);
    const double tau1 = collision_time(p1.rho, p1.lam, p.mu_ref, p.omega);

    // heat flux of the stage-1 distribution about U^{n+1} (each thread
    // re-reads the values it wrote)
    double qt[D];
#pragma unroll
    for (int d = 0; d < D; ++d) qt[d] = 0.0;
    for (int k = tid; k < nv; k += BS) {
        double c[D], c2 = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            c[d] = p.u[d * nv + k] - p1.U[d];
            c2 += c[d] * c[d];
        }
        const double h = to_f64(s1[k]);
        const double b = NC > 1 ? to_f64(s1[(size_t)(NC - 1) * nv + k]) : 0.0;
        const double wt = 0.5 * p.w[k] * (c2 * h + b);
#pragma unroll
        for (int d = 0; d < D; ++d) qt[d] += wt * c[d];
    }
    block_reduce<BS>(qt, red, OpAdd{});
    double q1[D];
#pragma unroll
    for (int d = 0; d < D; ++d) q1[d] = qt[d] / (1.0 + Pr * dt / (2.0 * tau1));

    if constexpr (TENSOR) {
        // the cell's table now holds the factors of f+^{n+1}
        const int ntab = p.ntab;
        for (int idx = tid; idx < ntab; idx += BS) {
            const int ax = idx < p.n1d[0] ? 0 : (idx < p.n1d[0] + p.n1d[1] ? 1 : 2);
            double Ud = p1.U[0];
            if (ax == 1) Ud = p1.U[1];
            if (D == 3 && ax == 2) Ud = p1.U[D - 1];
            const double c = p.u1d[idx] - Ud;
            tab[MF * ntab + idx] = exp(-p1.lam * c * c);
        }
        __syncthreads();
    }

    // Algorithm 1's last step: Eq. microS2
    const double pref_1 = p1.rho * pow_lam_pi<D>(p1.lam);
    const double shk_1 = 4.0 * (1.0 - Pr) * p1.lam * p1.lam / (5.0 * p1.rho);
    const double a1 = 0.5 * dt / tau1, inv1 = 1.0 / (1.0 + a1);
    const double bh_1 = Dim<D>::M / (2.0 * p1.lam);
    for (int k = tid; k < nv; k += BS) {
        double u[D];
#pragma unroll
        for (int d = 0; d < D; ++d) u[d] = p.u[d * nv + k];
        const unsigned kx = TENSOR ? (unsigned)p.kidx[k] : 0u;
        double fp[2];
        const double H = pref_1 * gauss(MF, kx, u, p1.lam, p1.U);
        shakhov<D>(u, p1.U, p1.lam, shk_1, q1, bh_1, H, fp[0], fp[1]);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            fout[base + (size_t)c * nv + k] = from_f64<FT>((to_f64(s1[(size_t)c * nv + k]) + a1 * fp[c]) * inv1);
        }
    }
    if (tid == 0) {
        bool ok = p1.rho > 0.0 && p1.lam > 0.0 && isfinite(p1.rho) && isfinite(p1.lam);
#pragma unroll
        for (int m = 0; m < NW; ++m) {
            ok = ok && isfinite(W1[m]);
            p.W[(size_t)i * NW + m] = W1[m];
            const double dw = W1[m] - cs.Wn[m];
            p.dW2[(size_t)i * NW + m] = dw * dw;
        }
#pragma unroll
        for (int d = 0; d < D; ++d) p.q[(size_t)i * D + d] = q1[d];
        if (!ok) {
            atomicOr(p.err, 1);
            atomicMin(p.err + 1, i);
        }
    }
}


// PF: the own cell's stencil of the next velocity is loaded one iteration
// ahead (20 more registers: used where they fit in the four-wave budget).
// CHUNK: the in-place mode's chunk kernel -- pass 1 over velocities
// [c0, c0 + cn) only, reading f^n and writing the stage-1 values to the ring
// (after writing the previous chunk's ring back into f), adding the chunk's
// moments to the cell's running sum (mom_part, started from zero by chunk 0),
// and the wall densities read from the wall kernel's array.
template <int D, typename FT, int BS, bool TENSOR, bool S1L, bool PF, bool CHUNK = false>
__device__ __forceinline__ void sweep_cell(const Params p, int i, const FT *__restrict__ fin, FT *__restrict__ fout,
                                           int c0 = 0, int cn = 0, int prev0 = 0, int prevn = 0, int ichunk = 0)
{
    constexpr int NC = Dim<D>::NC, MF = Dim<D>::MF, NW = D + 2;
    constexpr int NT = MF + 1;  // Gaussian tables: one per face slot, one for the cell
    extern __shared__ double smem[];
    if (i >= p.nc) return;
    const int tid = threadIdx.x;
    const CellGeo<D> *cg = static_cast<const CellGeo<D> *>(p.cgeo);
    const FaceGeo<D> *fg = static_cast<const FaceGeo<D> *>(p.fgeo);
    const FaceEq<D> *fe = static_cast<const FaceEq<D> *>(p.feq);
    const CellGeo<D> &gi = cg[i];
    const int nv = p.nv, nf = gi.nf;
    const double dt = p.dt, Pr = p.Pr;
    const int ntab = TENSOR ? p.ntab : 0;
    double *red = smem + NT * ntab;
    const Gauss<D, TENSOR> gauss{smem, ntab};
    const size_t base = (size_t)i * NC * nv;
    constexpr int NRED = (NW > 2 * MF) ? NW : 2 * MF;
    // stage-1 values: LDS, f_out, or (chunk mode) the cell's ring, as
    // s1[c s1_stride + k - s1_off] for component c at velocity k
    FT *s1 = CHUNK ? static_cast<FT *>(p.ring) + (size_t)i * NC * p.chunk
                   : (S1L ? reinterpret_cast<FT *>(red + (BS / 64) * NRED) : fout + base);
    const size_t s1_stride = CHUNK ? (size_t)p.chunk : (size_t)nv;
    const int s1_off = CHUNK ? c0 : 0;
    const int k_end = CHUNK ? c0 + cn : nv;
    if constexpr (CHUNK) {
        // the previous chunk's stage-1 values go back into f (no workgroup
        // reads those velocities any more)
        for (int t = tid; t < prevn; t += BS)
#pragma unroll
            for (int c = 0; c < NC; ++c) fout[base + (size_t)c * nv + prev0 + t] = s1[(size_t)c * s1_stride + t];
    }

    // state at t^n
    double Wn[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) Wn[m] = p.W[(size_t)i * NW + m];
    const Prim<D> pn = to_prim<D>(Wn);
    const double tau_n = collision_time(pn.rho, pn.lam, p.mu_ref, p.omega);
    double qn[D];
#pragma unroll
    for (int d = 0; d < D; ++d) qn[d] = p.q[(size_t)i * D + d];
    const double pref_n = pn.rho * pow_lam_pi<D>(pn.lam);
    const double shk_n = 4.0 * (1.0 - Pr) * pn.lam * pn.lam / (5.0 * pn.rho);
    const double hdt_tau = 0.5 * dt / tau_n;
    const double bh_n = Dim<D>::M / (2.0 * pn.lam);

    int has_wall = 0;
    if constexpr (!CHUNK)
        for (int j = 0; j < nf; ++j) has_wall |= (fg[gi.face[j]].bc == 3);

    if constexpr (TENSOR) {
        // one-dimensional Gaussian factors of every face's Maxwellian and of f+^n
        for (int t = tid; t < NT * ntab; t += BS) {
            const int which = t / ntab, idx = t - which * ntab;
            const int ax = idx < p.n1d[0] ? 0 : (idx < p.n1d[0] + p.n1d[1] ? 1 : 2);
            double lam, Ud;
            if (which < nf) {
                const FaceEq<D> &e = fe[gi.face[which]];
                lam = e.lam;
                Ud = e.U[0];
                if (ax == 1) Ud = e.U[1];
                if (D == 3 && ax == 2) Ud = e.U[D - 1];
            } else {
                lam = pn.lam;
                Ud = pn.U[0];
                if (ax == 1) Ud = pn.U[1];
                if (D == 3 && ax == 2) Ud = pn.U[D - 1];
            }
            const double c = p.u1d[idx] - Ud;
            smem[t] = exp(-lam * c * c);
        }
    }
    __syncthreads();

    // Algorithm 1's boundary flux (wall density) first, for wall cells only: the incident
    // particles' mass flux and the unit-density reflected flux, summed over
    // velocities; rho_w makes the net mass flux through the wall vanish
    // (Eq. maxWalldes).  Knowing rho_w up front, the sweep below adds the
    // reflected particles directly.
    double rho_w[MF];
#pragma unroll
    for (int j = 0; j < MF; ++j) rho_w[j] = CHUNK ? p.rho_w[(size_t)i * MF + j] : 0.0;
    if (has_wall) {
        double wsum[2 * MF];
#pragma unroll
        for (int j = 0; j < 2 * MF; ++j) wsum[j] = 0.0;
        for (int k = tid; k < nv; k += BS) {
            double u[D];
#pragma unroll
            for (int d = 0; d < D; ++d) u[d] = p.u[d * nv + k];
            const unsigned kx = TENSOR ? (unsigned)p.kidx[k] : 0u;
            const double wk = p.w[k];
            double fi[NC], gri[NC][D];
            limited_slope<D, FT>(gi, i, fin, nv, k, p.limiter, fi, gri);
#pragma unroll
            for (int j = 0; j < MF; ++j) {
                if (j >= nf) break;
                const FaceGeo<D> &F = fg[gi.face[j]];
                if (F.bc != 3) continue;
                double un = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) un += u[d] * F.n[d];
                if (un > 0.0) {
                    double v = fi[0], ug = 0.0;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        v += gri[0][d] * gi.dvec[j][d];
                        ug += u[d] * gri[0][d];
                    }
                    wsum[2 * j] += wk * un * (dt * v - 0.5 * dt * dt * ug);
                } else {
                    const FaceEq<D> &e = fe[gi.face[j]];
                    wsum[2 * j + 1] += wk * un * e.k0 * gauss(j, kx, u, e.lam, e.U);
                }
            }
        }
        block_reduce<BS>(wsum, red, OpAdd{});
#pragma unroll
        for (int j = 0; j < MF; ++j) rho_w[j] = (j < nf && wsum[2 * j + 1] != 0.0) ? -wsum[2 * j] / wsum[2 * j + 1] : 0.0;
    }

    // Algorithm 1's velocity loop: per velocity, limited slopes, interface fluxes,
    // stage 1; the moments of the net outflow give W^{n+1}
    double mom[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) mom[m] = 0.0;
    Stencil<D, FT> next;
    if (PF && s1_off + tid < k_end) load_stencil<D, FT>(gi, i, fin, nv, s1_off + tid, next);
    for (int k = s1_off + tid; k < k_end; k += BS) {
        Stencil<D, FT> own;
        if constexpr (PF) {
            own = next;
            if (k + BS < k_end) load_stencil<D, FT>(gi, i, fin, nv, k + BS, next);
        }
        double u[D], u2 = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            u[d] = p.u[d * nv + k];
            u2 += u[d] * u[d];
        }
        const unsigned kx = TENSOR ? (unsigned)p.kidx[k] : 0u;
        double fi[NC], gri[NC][D];
        if constexpr (PF) slope_from<D, FT>(gi, p.limiter, own, fi, gri);
        else limited_slope<D, FT>(gi, i, fin, nv, k, p.limiter, fi, gri);
        double out[NC], ugi[NC];
        along<D>(u, gri, ugi);
#pragma unroll
        for (int c = 0; c < NC; ++c) out[c] = 0.0;
#pragma unroll
        for (int j = 0; j < MF; ++j) {
            if (j >= nf) break;
            const int f = gi.face[j];
            const FaceGeo<D> &F = fg[f];
            const FaceEq<D> &e = fe[f];
            double un = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) un += u[d] * F.n[d];
            double I[NC];
            if (F.bc == 0) {
                const bool self_up = (un > 0.0) == (gi.side[j] == 0);
                const double G = gauss(j, kx, u, e.lam, e.U);
                if (self_up) {
                    interface_integral<D>(e, u, G, fi, gri, gi.dvec[j], ugi, I);
                } else {
                    const int n = gi.nb[j];
                    const CellGeo<D> &gn = cg[n];
                    double fn[NC], grn[NC][D], ug[NC];
                    limited_slope<D, FT>(gn, n, fin, nv, k, p.limiter, fn, grn);
                    along<D>(u, grn, ug);
                    interface_integral<D>(e, u, G, fn, grn, gn.dvec[gi.back[j]], ug, I);
                }
            } else if (un > 0.0) {
                boundary_outgoing<D>(e, fi, gri, gi.dvec[j], ugi, I);
            } else {
                // incoming from the wall (density rho_w) or the ghost Maxwellian
                I[0] = (F.bc == 3 ? rho_w[j] : 1.0) * e.k0 * gauss(j, kx, u, e.lam, e.U);
                if constexpr (NC > 1) I[1] = e.bh * I[0];
            }
            const double sa = (gi.side[j] ? -F.area : F.area) * un;
#pragma unroll
            for (int c = 0; c < NC; ++c) out[c] += sa * I[c];
        }
        // Eq. microS1 with the source at t^n
        double fpn[2];
        {
            const double H = pref_n * gauss(MF, kx, u, pn.lam, pn.U);
            shakhov<D>(u, pn.U, pn.lam, shk_n, qn, bh_n, H, fpn[0], fpn[1]);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
            s1[(size_t)c * s1_stride + (k - s1_off)] =
                from_f64<FT>(fi[c] - out[c] * gi.inv_vol + hdt_tau * (fpn[c] - fi[c]));
        // moments of the net outflow (Eq. macroscopicFlux summed over faces)
        const double wk = p.w[k];
        mom[0] += wk * out[0];
#pragma unroll
        for (int d = 0; d < D; ++d) mom[1 + d] += wk * u[d] * out[0];
        mom[NW - 1] += wk * 0.5 * (u2 * out[0] + (NC > 1 ? out[NC - 1] : 0.0));
    }

    // Algorithm 1's macroscopic update: Eq. macroscopicUpdata, then tau at t^{n+1}
    block_reduce<BS>(mom, red, OpAdd{});
    if constexpr (CHUNK) {
        // add this chunk's moments to the cell's sum; the chunks run one
        // launch after another, so the sum is taken in chunk order
        if (tid == 0) {
            double *acc = p.mom_part + (size_t)i * NW;
#pragma unroll
            for (int m = 0; m < NW; ++m) acc[m] = (ichunk == 0 ? 0.0 : acc[m]) + mom[m];
        }
        return;
    }
    double W1[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) W1[m] = Wn[m] - mom[m] * gi.inv_vol;
    const Prim<D> p1 = to_prim<D>(W1);
    const double tau1 = collision_time(p1.rho, p1.lam, p.mu_ref, p.omega);

    // heat flux of the stage-1 distribution about U^{n+1} (each thread
    // re-reads the values it wrote)
    double qt[D];
#pragma unroll
    for (int d = 0; d < D; ++d) qt[d] = 0.0;
    for (int k = tid; k < nv; k += BS) {
        double c[D], c2 = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            c[d] = p.u[d * nv + k] - p1.U[d];
            c2 += c[d] * c[d];
        }
        const double h = to_f64(s1[k]);
        const double b = NC > 1 ? to_f64(s1[(size_t)(NC - 1) * nv + k]) : 0.0;
        const double wt = 0.5 * p.w[k] * (c2 * h + b);
#pragma unroll
        for (int d = 0; d < D; ++d) qt[d] += wt * c[d];
    }
    block_reduce<BS>(qt, red, OpAdd{});
    double q1[D];
#pragma unroll
    for (int d = 0; d < D; ++d) q1[d] = qt[d] / (1.0 + Pr * dt / (2.0 * tau1));

    if constexpr (TENSOR) {
        // the cell's table now holds the factors of f+^{n+1}
        for (int idx = tid; idx < ntab; idx += BS) {
            const int ax = idx < p.n1d[0] ? 0 : (idx < p.n1d[0] + p.n1d[1] ? 1 : 2);
            double Ud = p1.U[0];
            if (ax == 1) Ud = p1.U[1];
            if (D == 3 && ax == 2) Ud = p1.U[D - 1];
            const double c = p.u1d[idx] - Ud;
            smem[MF * ntab + idx] = exp(-p1.lam * c * c);
        }
        __syncthreads();
    }

    // Algorithm 1's last step: Eq. microS2
    const double pref_1 = p1.rho * pow_lam_pi<D>(p1.lam);
    const double shk_1 = 4.0 * (1.0 - Pr) * p1.lam * p1.lam / (5.0 * p1.rho);
    const double a1 = 0.5 * dt / tau1, inv1 = 1.0 / (1.0 + a1);
    const double bh_1 = Dim<D>::M / (2.0 * p1.lam);
    for (int k = tid; k < nv; k += BS) {
        double u[D];
#pragma unroll
        for (int d = 0; d < D; ++d) u[d] = p.u[d * nv + k];
        const unsigned kx = TENSOR ? (unsigned)p.kidx[k] : 0u;
        double fp[2];
        const double H = pref_1 * gauss(MF, kx, u, p1.lam, p1.U);
        shakhov<D>(u, p1.U, p1.lam, shk_1, q1, bh_1, H, fp[0], fp[1]);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            fout[base + (size_t)c * nv + k] = from_f64<FT>((to_f64(s1[(size_t)c * nv + k]) + a1 * fp[c]) * inv1);
        }
    }
    if (tid == 0) {
        bool ok = p1.rho > 0.0 && p1.lam > 0.0 && isfinite(p1.rho) && isfinite(p1.lam);
#pragma unroll
        for (int m = 0; m < NW; ++m) {
            ok = ok && isfinite(W1[m]);
            p.W[(size_t)i * NW + m] = W1[m];
            const double dw = W1[m] - Wn[m];
            p.dW2[(size_t)i * NW + m] = dw * dw;
        }
#pragma unroll
        for (int d = 0; d < D; ++d) p.q[(size_t)i * D + d] = q1[d];
        if (!ok) {
            atomicOr(p.err, 1);
            atomicMin(p.err + 1, i);
        }
    }
}

// ------------------------------------------------------------------------
// In-place mode (one f buffer): the velocities are swept in chunks.  A chunk
// kernel reads f^n of its velocities only (the cell's two-ring stencil),
// parks the stage-1 values in a ring buffer of one chunk per cell and adds
// the chunk's moments of the net outflow to the cell's running sum
// (mom_part: chunk 0 starts it from zero, the chunks run one launch after
// another); the next chunk kernel first writes its cell's ring back into f
// (no workgroup reads those velocities any more), and a final kernel writes
// the last chunk, reads that sum (W^{n+1}), forms q^{n+1} from the stage-1
// values now in f, and applies stage 2 in place.  This is the paper's in-place
// update of f (Section 3.2) with the ring as the only extra storage.  The
// wall density of every wall cell is reduced over all velocities first.
// ------------------------------------------------------------------------
template <int D, typename FT, int BS, bool TENSOR>
__global__ __launch_bounds__(BS) void k_wall_density(Params p, const FT *__restrict__ f)
{
    constexpr int MF = Dim<D>::MF, NT = MF + 1;
    extern __shared__ double smem[];
    const int i = xcd_cell(blockIdx.x);
    if (i >= p.nc) return;
    const CellGeo<D> &gi = static_cast<const CellGeo<D> *>(p.cgeo)[i];
    if (!has_wall_face<D>(p, gi)) return;  // uniform: the whole workgroup leaves
    const int ntab = TENSOR ? p.ntab : 0;
    const CellStep<D> cs = cell_step<D>(p, i);
    if constexpr (TENSOR) fill_tables<D, BS>(p, gi, cs.pn, smem);
    __syncthreads();
    const Gauss<D, TENSOR> gauss{smem, ntab};
    double rho_w[MF];
    wall_density<D, FT, BS, TENSOR>(p, gi, i, f, gauss, smem + NT * ntab, rho_w);
    if (threadIdx.x == 0)
#pragma unroll
        for (int j = 0; j < MF; ++j) p.rho_w[(size_t)i * MF + j] = rho_w[j];
}

// The chunk sweep under the four-wave budget; the next velocity's stencil is
// prefetched for FP32 and BF16 f (with FP64 f the prefetch registers would
// spill: measured 8.9 against 7.7 ms per step on the cylinder).
template <int D, typename FT, int BS, bool TENSOR>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_sweep_chunk(
    Params p, FT *__restrict__ f, int c0, int cn, int prev0, int prevn, int ichunk)
{
    constexpr bool PF = TENSOR && sizeof(FT) < sizeof(double);
    sweep_cell<D, FT, BS, TENSOR, false, PF, true>(p, xcd_cell(blockIdx.x), f, f, c0, cn, prev0, prevn, ichunk);
}

template <int D, typename FT, int BS, bool TENSOR>
__global__ __launch_bounds__(BS) void k_sweep_finish(Params p, FT *__restrict__ f, int last0, int lastn)
{
    constexpr int NC = Dim<D>::NC, NW = D + 2;
    extern __shared__ double smem[];
    const int i = xcd_cell(blockIdx.x);
    if (i >= p.nc) return;
    const int tid = threadIdx.x, nv = p.nv, ch = p.chunk;
    const CellGeo<D> &gi = static_cast<const CellGeo<D> *>(p.cgeo)[i];
    const FT *ring = static_cast<const FT *>(p.ring) + (size_t)i * NC * ch;
    FT *fc = f + (size_t)i * NC * nv;
    for (int t = tid; t < lastn; t += BS)
#pragma unroll
        for (int c = 0; c < NC; ++c) fc[(size_t)c * nv + last0 + t] = ring[(size_t)c * ch + t];
    const int ntab = TENSOR ? p.ntab : 0;
    const CellStep<D> cs = cell_step<D>(p, i);
    if constexpr (TENSOR) fill_tables<D, BS>(p, gi, cs.pn, smem);
    // the chunks' moments, summed in chunk order by the chunk kernels
    double mom[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) mom[m] = p.mom_part[(size_t)i * NW + m];
    // block_reduce in finish_cell sums over the workgroup: only thread 0
    // carries the moments
    if (tid != 0)
#pragma unroll
        for (int m = 0; m < NW; ++m) mom[m] = 0.0;
    __syncthreads();
    constexpr int NT = Dim<D>::MF + 1;
    const Gauss<D, TENSOR> gauss{smem, ntab};
    finish_cell<D, FT, BS, TENSOR>(p, i, cs, mom, fc, smem + NT * ntab, smem, gauss, f);
}

template <int D, typename FT, int BS, bool TENSOR, bool S1L>
__global__ __launch_bounds__(BS) void k_sweep(Params p, const FT *__restrict__ fin, FT *__restrict__ fout)
{
    sweep_cell<D, FT, BS, TENSOR, S1L, false>(p, xcd_cell(blockIdx.x), fin, fout);
}

// Cartesian (tabulated) velocity sets: the same with the stencil prefetch,
// held to four waves per SIMD.
template <int D, typename FT, int BS, bool S1L>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_sweep_pf(Params p, const FT *__restrict__ fin, FT *__restrict__ fout)
{
    sweep_cell<D, FT, BS, true, S1L, true>(p, xcd_cell(blockIdx.x), fin, fout);
}

// ------------------------------------------------------------------------
// Push sweep (FP64 or FP32 f; two f buffers, or in place one f and a ring of
// one velocity chunk): each face flux once.
//
// Per velocity, the flux through an interior face needs the limited slope
// of the upwind cell only (Eq. fullSolution).  The cells are split into
// colours such that no two cells of a colour are neighbours or share a
// neighbour (distance-2 colouring), and one launch per colour advances its
// cells: a workgroup owns one cell's velocity slab (or a share of it, when
// a class is too small to fill the chip), rebuilds that cell's own limited
// slope, and for every face through which the cell is upwind
// at a velocity it evaluates the time-integrated flux once and adds it to
// the stage-1 accumulator of both cells (- F / |Omega_i| here, + F /
// |Omega_n| there) with hardware atomic adds that return nothing, so that
// the velocity loop never waits on an accumulator load.  Faces through which the cell is downwind are added by
// the neighbour in its own colour's launch.  No two workgroups of a launch
// touch the same accumulator, and the colours run in a fixed order, so the
// sums are deterministic; the accumulator holds, before the first colour,
// the stage-1 base f^n + (dt / 2 tau^n)(f+^n - f^n) of Eq. microS1 and,
// after the last, the stage-1 value itself.  A final kernel per cell then
// forms W^{n+1} = W^n + M(f~) - M(base) (M the moments (1, u, (|u|^2 h + b)
// / 2) summed over velocities: their difference is the sum over faces of
// the moments of the micro flux, Eqs. macroscopicFlux and
// macroscopicUpdata), tau^{n+1}, q^{n+1}, stage 2 (Eq. microS2) into the f
// buffer, and the next step's base (with its moments) into the
// accumulator.  Wall cells reduce the wall density over their velocities
// first (Eq. maxWalldes) and record the step's wall flux.
// ------------------------------------------------------------------------

// moments (1, u, (|u|^2 h + b) / 2) of one velocity's values, weighted
template <int D>
__device__ __forceinline__ void add_moments(double (&m)[D + 2], double w, const double (&u)[D], double u2, double h,
                                            double b)
{
    m[0] = fma(w, h, m[0]);
#pragma unroll
    for (int d = 0; d < D; ++d) m[1 + d] = fma(w * u[d], h, m[1 + d]);
    m[D + 1] = fma(0.5 * w, fma(u2, h, b), m[D + 1]);
}

// Two consecutive values of an f slab in one 2-wide access (the element
// offset even, so the access is aligned): the per-cell streaming kernels
// take velocities in pairs when the velocity count is even, which doubles
// the bytes each load keeps in flight.
template <typename FT> struct Vec2;
template <> struct Vec2<double> { using T = double2; };
template <> struct Vec2<float> { using T = float2; };
template <typename FT> __device__ __forceinline__ void load2(const FT *__restrict__ q, double &a, double &b)
{
    const typename Vec2<FT>::T v = *reinterpret_cast<const typename Vec2<FT>::T *>(q);
    a = to_f64(v.x);
    b = to_f64(v.y);
}
template <typename FT> __device__ __forceinline__ void store2(FT *__restrict__ q, FT a, FT b)
{
    typename Vec2<FT>::T v;
    v.x = a;
    v.y = b;
    *reinterpret_cast<typename Vec2<FT>::T *>(q) = v;
}
// bfloat16 pairs: one 32-bit word, the first value in its lower half
template <> __device__ __forceinline__ void load2<bf16s>(const bf16s *__restrict__ q, double &a, double &b)
{
    const unsigned v = *reinterpret_cast<const unsigned *>(q);
    a = to_f64(bf16s{(unsigned short)(v & 0xffffu)});
    b = to_f64(bf16s{(unsigned short)(v >> 16)});
}
template <> __device__ __forceinline__ void store2<bf16s>(bf16s *__restrict__ q, bf16s a, bf16s b)
{
    *reinterpret_cast<unsigned *>(q) = (unsigned)a.bits | ((unsigned)b.bits << 16);
}

// The push sweep's accumulator (the stage-1 sums) is kept in f's storage
// type, except with bfloat16 f: there it holds FP32, since a bfloat16 sum
// would round away most of every flux added to it.
template <typename FT> struct AccOf {
    using T = FT;
};
template <> struct AccOf<bf16s> {
    using T = float;
};

// Wall faces of cell i (Section 2.5): per wall face, the incident particles'
// mass flux (free transport of the interior reconstruction) and the
// unit-density reflected one, summed over velocities, give rho_w
// (Eq. maxWalldes); the face's macroscopic flux over the step (incident +
// rho_w reflected) per unit area and time is recorded.  Workgroup-wide.
template <int D, typename FT, int BS, bool TENSOR>
__device__ __forceinline__ void push_wall(const Params &p, const CellGeo<D> &gi, int i, const FT *__restrict__ fin,
                                          const Gauss<D, TENSOR> &gauss, double *red, double (&rho_w)[Dim<D>::MF])
{
    constexpr int NC = Dim<D>::NC, MF = Dim<D>::MF, NW = D + 2;
    const FaceGeo<D> *fg = static_cast<const FaceGeo<D> *>(p.fgeo);
    const FaceEq<D> *fe = static_cast<const FaceEq<D> *>(p.feq);
    const int nv = p.nv, nf = gi.nf;
    const double dt = p.dt;
#pragma unroll
    for (int j = 0; j < MF; ++j) rho_w[j] = 0.0;
    for (int j = 0; j < nf; ++j) {
        const int f = gi.face[j];
        const FaceGeo<D> &F = fg[f];
        if (F.bc != 3) continue;  // uniform
        const FaceEq<D> &e = fe[f];
        double s[2 * NW + 2];
#pragma unroll
        for (int m = 0; m < 2 * NW + 2; ++m) s[m] = 0.0;
        for (int k = threadIdx.x; k < nv; k += BS) {
            double u[D], u2 = 0.0, un = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                u[d] = p.u[d * nv + k];
                u2 = fma(u[d], u[d], u2);
                un = fma(u[d], F.n[d], un);
            }
            const double wk = p.w[k];
            double I[2] = {0.0, 0.0};
            if (un > 0.0) {
                double fi[NC], gri[NC][D];
                limited_slope<D, FT>(gi, i, fin, nv, k, p.limiter, fi, gri);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    double v = fi[c], ug = 0.0;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        v = fma(gri[c][d], gi.dvec[j][d], v);
                        ug = fma(u[d], gri[c][d], ug);
                    }
                    I[c] = dt * v - 0.5 * dt * dt * ug;
                }
                s[2 * NW] = fma(wk * un, I[0], s[2 * NW]);
                double mm[NW];
#pragma unroll
                for (int m = 0; m < NW; ++m) mm[m] = 0.0;
                add_moments<D>(mm, wk * un, u, u2, I[0], NC > 1 ? I[NC - 1] : 0.0);
#pragma unroll
                for (int m = 0; m < NW; ++m) s[m] += mm[m];
            } else {
                const double H = e.k0 * gauss(j, (TENSOR ? (unsigned)p.kidx[k] : 0u), u, e.lam, e.U);
                I[0] = H;
                if constexpr (NC > 1) I[1] = e.bh * H;
                s[2 * NW + 1] = fma(wk * un, I[0], s[2 * NW + 1]);
                double mm[NW];
#pragma unroll
                for (int m = 0; m < NW; ++m) mm[m] = 0.0;
                add_moments<D>(mm, wk * un, u, u2, I[0], NC > 1 ? I[NC - 1] : 0.0);
#pragma unroll
                for (int m = 0; m < NW; ++m) s[NW + m] += mm[m];
            }
        }
        block_reduce<BS>(s, red, OpAdd{});
        const double rw = s[2 * NW + 1] != 0.0 ? -s[2 * NW] / s[2 * NW + 1] : 0.0;
#pragma unroll
        for (int jj = 0; jj < MF; ++jj)
            if (jj == j) rho_w[jj] = rw;
        if (threadIdx.x == 0 && p.wall_index) {
            const int widx = p.wall_index[f];
            if (widx >= 0)
#pragma unroll
                for (int m = 0; m < NW; ++m) p.wflux[(size_t)widx * NW + m] = (s[m] + rw * s[NW + m]) / dt;
        }
    }
}

// One colour's cells: cells[0..ncell) (stored indices), workgroups dealt to
// the XCDs in runs as for the gather sweep.  PF: the own stencil of the
// next velocity is loaded one iteration ahead.
template <int D, typename FT, int BS, bool TENSOR, bool PF>
__device__ __forceinline__ void push_cell(const Params p, int i, const FT *__restrict__ fin,
                                          typename AccOf<FT>::T *__restrict__ acc, int k0, int kn, int accv)
{
    using AT = typename AccOf<FT>::T;
    constexpr int NC = Dim<D>::NC, MF = Dim<D>::MF;
    extern __shared__ double smem[];
    const int tid = threadIdx.x;
    const CellGeo<D> &gi = static_cast<const CellGeo<D> *>(p.cgeo)[i];
    const FaceGeo<D> *fg = static_cast<const FaceGeo<D> *>(p.fgeo);
    const FaceEq<D> *fe = static_cast<const FaceEq<D> *>(p.feq);
    const int nv = p.nv, nf = gi.nf, ntab = TENSOR ? p.ntab : 0;
    if constexpr (TENSOR) fill_tables<D, BS>(p, gi, to_prim<D>(p.W + (size_t)i * (D + 2)), smem);
    __syncthreads();
    const Gauss<D, TENSOR> gauss{smem, ntab};
    // wall densities of this cell's wall faces, from the step's wall kernel
    const double *rho_w = p.rho_w + (size_t)i * MF;

    // velocities [k0, k0 + kn); the accumulator holds accv velocities per
    // cell and component, starting at k0 (the whole set, or one chunk)
    const int kend = k0 + kn;
    const size_t base = (size_t)i * NC * accv;
    Stencil<D, FT> next;
    if (PF && k0 + tid < kend) load_stencil<D, FT>(gi, i, fin, nv, k0 + tid, next);
    for (int k = k0 + tid; k < kend; k += BS) {
        Stencil<D, FT> own;
        if constexpr (PF) {
            own = next;
            if (k + BS < kend) load_stencil<D, FT>(gi, i, fin, nv, k + BS, next);
        } else {
            load_stencil<D, FT>(gi, i, fin, nv, k, own);
        }
        double u[D], u2 = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            u[d] = p.u[d * nv + k];
            u2 = fma(u[d], u[d], u2);
        }
        const unsigned kx = TENSOR ? (unsigned)p.kidx[k] : 0u;
        double fi[NC], gri[NC][D];
        slope_from<D, FT>(gi, p.limiter, own, fi, gri);
        double out[NC], ug[NC];
        along<D>(u, gri, ug);
#pragma unroll
        for (int c = 0; c < NC; ++c) out[c] = 0.0;
        // faces one at a time (not unrolled: their records are read with
        // scalar loads per face, which keeps the vector registers for the
        // velocities' values)
#pragma unroll 1
        for (int j = 0; j < nf; ++j) {
            const int f = gi.face[j];
            const FaceGeo<D> &F = fg[f];
            const FaceEq<D> &e = fe[f];
            double un = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) un = fma(u[d], F.n[d], un);
            const double uo = gi.side[j] ? -un : un;  // along this cell's outward normal
            if (F.bc == 0) {
                if (!(uo > 0.0)) continue;  // the neighbour is upwind: it adds this flux
                AT *an = acc + (size_t)gi.nb[j] * NC * accv;
                double I[NC];
                interface_integral<D>(e, u, gauss(j, kx, u, e.lam, e.U), fi, gri, gi.dvec[j], ug, I);
                const double sa = F.area * uo;
                const double vn_inv = gi.nb_inv_vol[j];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const double fl = sa * I[c];
                    out[c] += fl;
                    // an atomic add without return: no load waits in the
                    // velocity loop (in a colour launch no other workgroup
                    // adds to this element, so the order of the sums stays
                    // fixed; the one-class unordered sweep gives that up)
                    unsafeAtomicAdd(an + (size_t)c * accv + (k - k0), from_f64<AT>(fl * vn_inv));
                }
            } else {
                double I[NC];
                if (un > 0.0) {
                    boundary_outgoing<D>(e, fi, gri, gi.dvec[j], ug, I);
                } else {
                    // incoming from the wall (density rho_w) or the ghost Maxwellian
                    I[0] = (F.bc == 3 ? rho_w[j] : 1.0) * e.k0 * gauss(j, kx, u, e.lam, e.U);
                    if constexpr (NC > 1) I[1] = e.bh * I[0];
                }
                const double sa = F.area * un;  // a boundary cell is the face's left cell
#pragma unroll
                for (int c = 0; c < NC; ++c) out[c] += sa * I[c];
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            AT *a = acc + base + (size_t)c * accv + (k - k0);
            unsafeAtomicAdd(a, from_f64<AT>(-out[c] * gi.inv_vol));
        }
    }
}

// The push sweep over bricks of kBrickCells cells (FP64 f): a workgroup
// carries its velocities through one cell of its brick after the other, keeps
// the stage-1 sums of the brick in LDS (a column per thread) and adds a flux
// to them where the neighbour belongs to the brick.  The push is bound by its
// atomic adds, which are performed beyond the L2 (without them k_push_pf takes
// 6.5 ms of 12): a compact brick of 4 cells leaves 3 a cell and velocity
// instead of 4.  107,118 cells x 4,548: all cells in one launch 11.97 -> 9.6
// ms, 15 colours 14.2 -> 12.05.  Bricks of 2, 3 and 8 measured 11.1, 10.6 and
// 18.0 against 10.2 (before whole bricks were put first in the list), and
// workgroups of 256, 512 and 1,024 threads 13.4, 10.3 and 10.3: 768 threads at
// two workgroups a CU keep 24 wavefronts on few enough records for the scalar
// cache.  Scattered sets, whose exponentials take more registers, have two
// workgroups of 512 threads a CU, which spill nothing (107,118 x 4,548 in one
// launch: a step 13.98 ms, 14.86 with 768 threads and 8 spilled registers).
// A workgroup takes the ksplit velocities of its blockIdx.y.
template <int D, bool TENSOR, int BS>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(TENSOR ? 6 : 4))) void k_push_brick(
    Params p, const double *__restrict__ fin, double *__restrict__ acc, const int *__restrict__ cells, int ncell,
    int ksplit)
{
    constexpr int NC = Dim<D>::NC, MF = Dim<D>::MF, NT = MF + 1, B = kBrickCells;
    extern __shared__ double smem[];
    __shared__ double sums[B][NC][BS];
    const int b = xcd_cell(blockIdx.x) * B;
    if (b >= ncell) return;
    const int nb = min(B, ncell - b), tid = threadIdx.x;
    const CellGeo<D> *cg = static_cast<const CellGeo<D> *>(p.cgeo);
    const FaceGeo<D> *fg = static_cast<const FaceGeo<D> *>(p.fgeo);
    const FaceEq<D> *fe = static_cast<const FaceEq<D> *>(p.feq);
    const int nv = p.nv, ntab = TENSOR ? p.ntab : 0, nt = NT * ntab;
    const int k0 = (int)blockIdx.y * ksplit + tid, kend = min(nv, ((int)blockIdx.y + 1) * ksplit);
    int cell[B];
#pragma unroll
    for (int c = 0; c < B; ++c) cell[c] = c < nb ? cells[b + c] : -2;
    if constexpr (TENSOR)
        for (int c = 0; c < nb; ++c)
            fill_tables<D, BS>(p, cg[cells[b + c]], to_prim<D>(p.W + (size_t)cells[b + c] * (D + 2)), smem + c * nt);
    __syncthreads();
    Stencil<D, double> next;
    if (k0 < kend) load_stencil<D, double>(cg[cell[0]], cell[0], fin, nv, k0, next);
    for (int k = k0; k < kend; k += BS) {
#pragma unroll
        for (int c = 0; c < B; ++c)
#pragma unroll
            for (int m = 0; m < NC; ++m) sums[c][m][tid] = 0.0;
        double u[D];
#pragma unroll
        for (int d = 0; d < D; ++d) u[d] = p.u[d * nv + k];
        const unsigned kx = TENSOR ? (unsigned)p.kidx[k] : 0u;
#pragma unroll 1
        for (int c = 0; c < nb; ++c) {
            const int i = cells[b + c];
            const CellGeo<D> &gi = cg[i];
            const Gauss<D, TENSOR> gauss{smem + c * nt, ntab};
            const int nf = gi.nf;
            const Stencil<D, double> own = next;
            {
                const int cn = c + 1 < nb ? cells[b + c + 1] : cell[0], kk = c + 1 < nb ? k : k + BS;
                if (kk < kend) load_stencil<D, double>(cg[cn], cn, fin, nv, kk, next);
            }
            double fi[NC], gri[NC][D], out[NC], ug[NC];
            slope_from<D, double>(gi, p.limiter, own, fi, gri);
            along<D>(u, gri, ug);
#pragma unroll
            for (int m = 0; m < NC; ++m) out[m] = 0.0;
#pragma unroll 1
            for (int j = 0; j < nf; ++j) {
                const int f = gi.face[j];
                const FaceGeo<D> &F = fg[f];
                const FaceEq<D> &e = fe[f];
                double un = 0.0, I[NC];
#pragma unroll
                for (int d = 0; d < D; ++d) un = fma(u[d], F.n[d], un);
                const double uo = gi.side[j] ? -un : un;  // along this cell's outward normal
                if (F.bc == 0) {
                    if (!(uo > 0.0)) continue;  // the neighbour is upwind: it adds this flux
                    const int n = gi.nb[j];
                    int to = -1;
#pragma unroll
                    for (int q = 0; q < B; ++q) to = n == cell[q] ? q : to;
                    interface_integral<D>(e, u, gauss(j, kx, u, e.lam, e.U), fi, gri, gi.dvec[j], ug, I);
                    const double sa = F.area * uo, vn_inv = gi.nb_inv_vol[j];
#pragma unroll
                    for (int m = 0; m < NC; ++m) {
                        const double fl = sa * I[m];
                        out[m] += fl;
                        if (to >= 0) unsafeAtomicAdd(&sums[to][m][tid], fl * vn_inv);
                        else unsafeAtomicAdd(acc + (size_t)n * NC * nv + (size_t)m * nv + k, fl * vn_inv);
                    }
                } else {
                    if (un > 0.0) {
                        boundary_outgoing<D>(e, fi, gri, gi.dvec[j], ug, I);
                    } else {
                        // incoming from the wall (density rho_w) or the ghost Maxwellian
                        I[0] = (F.bc == 3 ? p.rho_w[(size_t)i * MF + j] : 1.0) * e.k0 * gauss(j, kx, u, e.lam, e.U);
                        if constexpr (NC > 1) I[NC - 1] = e.bh * I[0];
                    }
                    const double sa = F.area * un;  // a boundary cell is the face's left cell
#pragma unroll
                    for (int m = 0; m < NC; ++m) out[m] += sa * I[m];
                }
            }
#pragma unroll
            for (int m = 0; m < NC; ++m) unsafeAtomicAdd(&sums[c][m][tid], -out[m] * gi.inv_vol);
        }
#pragma unroll
        for (int c = 0; c < B; ++c)
            if (c < nb)
#pragma unroll
                for (int m = 0; m < NC; ++m)
                    unsafeAtomicAdd(acc + ((size_t)cell[c] * NC + m) * nv + k, sums[c][m][tid]);
    }
}

// The wall cells of a step (before the colours): wall densities per face slot
// into rho_w [cell][MF] and the wall flux of the step per wall face.
template <int D, typename FT, int BS, bool TENSOR>
__global__ __launch_bounds__(BS) void k_push_wall(Params p, const FT *__restrict__ fin, const int *__restrict__ cells,
                                                  int ncell)
{
    constexpr int MF = Dim<D>::MF, NT = MF + 1;
    extern __shared__ double smem[];
    if ((int)blockIdx.x >= ncell) return;
    const int i = cells[blockIdx.x];
    const CellGeo<D> &gi = static_cast<const CellGeo<D> *>(p.cgeo)[i];
    const int ntab = TENSOR ? p.ntab : 0;
    const CellStep<D> cs = cell_step<D>(p, i);
    if constexpr (TENSOR) fill_tables<D, BS>(p, gi, cs.pn, smem);
    __syncthreads();
    const Gauss<D, TENSOR> gauss{smem, ntab};
    double rho_w[MF];
    push_wall<D, FT, BS, TENSOR>(p, gi, i, fin, gauss, smem + NT * ntab, rho_w);
    if (threadIdx.x == 0)
#pragma unroll
        for (int j = 0; j < MF; ++j) p.rho_w[(size_t)i * MF + j] = rho_w[j];
}

template <int D, typename FT, int BS, bool TENSOR>
__global__ __launch_bounds__(BS) void k_push(Params p, const FT *__restrict__ fin, typename AccOf<FT>::T *__restrict__ acc,
                                             const int *__restrict__ cells, int ncell, int k0, int kn, int accv,
                                             int ksplit)
{
    const int b = xcd_cell(blockIdx.x);
    if (b >= ncell) return;
    // this workgroup's share of [k0, k0 + kn): ksplit velocities from
    // k0 + blockIdx.y ksplit (the accumulator's velocity k0 is its column 0)
    const int ka = k0 + (int)blockIdx.y * ksplit, kb = min(k0 + kn, ka + ksplit);
    if (ka >= kb) return;
    push_cell<D, FT, BS, TENSOR, false>(p, cells[b], fin, acc + (ka - k0), ka, kb - ka, accv);
}

// (3D: held to 6 waves per SIMD, which fits without spills and measured 2 %
// faster than the 5 the compiler chooses; 2D would spill)
template <int D, typename FT, int BS>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(D == 3 ? 6 : 1))) void k_push_pf(Params p, const FT *__restrict__ fin, typename AccOf<FT>::T *__restrict__ acc,
                                                const int *__restrict__ cells, int ncell, int k0, int kn, int accv,
                                                int ksplit)
{
    const int b = xcd_cell(blockIdx.x);
    if (b >= ncell) return;
    const int ka = k0 + (int)blockIdx.y * ksplit, kb = min(k0 + kn, ka + ksplit);
    if (ka >= kb) return;
    push_cell<D, FT, BS, true, true>(p, cells[b], fin, acc + (ka - k0), ka, kb - ka, accv);
}

// Velocity splits of a colour launch: a class of n cells gets up to enough
// workgroups to fill the chip (kPushFill), each with a share of the kn
// velocities that is a multiple of the workgroup size.  A class too small to
// fill the chip is bound by the length of one workgroup, not by the cell
// set-up that every workgroup repeats, so a share may be a single iteration:
// with at least four iterations a share, a colour launch of a 2,197-cell
// channel (1,331 velocities) took 24.2 us and now takes 13.0, one of a
// 4,096-cell box with 2,145 scattered velocities 32.8 and now 23.3 (with a fill
// of 8,192).  Where the tables that every share fills are long (`tables`
// entries in all), a share is at least as long as they are worth: 16,200 cells
// in 2D x 400 velocities with 800 coordinate values, in colours, 0.61 ms a step
// in shares of one iteration, 0.45 unsplit; 1,800 cells 0.138 and 0.124; 512
// in 3D x 285, classes of about 40, 0.242 and 0.262: those stay split.
constexpr int kPushFill = 4096;
inline int push_ksplit(int n, int kn, int bs, int tables)
{
    const int iters = (kn + bs - 1) / bs;  // velocity iterations of one workgroup
    const int split = std::max(1, std::min(iters, (kPushFill + n - 1) / n));
    const int least = n >= 128 ? std::min(iters, (tables + 8 * bs - 1) / (8 * bs)) : 1;
    const int per = std::max((iters + split - 1) / split, least);
    return per * bs;
}

template <int D> constexpr int sym_index(int a, int b)
{
    return a <= b ? a * D - a * (a - 1) / 2 + (b - a) : b * D - b * (b - 1) / 2 + (a - b);
}

// ------------------------------------------------------------------------
// Surface quantities (Section 2.5): the macroscopic flux through each wall
// face in a step, from the f that started the step.  One workgroup per wall
// face: particles leaving the gas carry the limited reconstruction of f
// (free transport over the step), particles leaving the wall the wall
// Maxwellian of density rho_w; both sums are kept apart, rho_w follows from
// zero net mass flux, and F = (out + rho_w * in) / dt per unit area.
// ------------------------------------------------------------------------
template <int D, typename FT, int BS>
__global__ __launch_bounds__(BS) void k_wall_flux(Params p, const FT *__restrict__ fin,
                                                  const int *__restrict__ wall_faces, double *__restrict__ out)
{
    constexpr int NC = Dim<D>::NC, NW = D + 2;
    __shared__ double red[(BS / 64) * 2 * NW];
    const int f = wall_faces[blockIdx.x];
    const FaceGeo<D> &F = static_cast<const FaceGeo<D> *>(p.fgeo)[f];
    const FaceEq<D> &e = static_cast<const FaceEq<D> *>(p.feq)[f];
    const int i = F.l;
    const CellGeo<D> &gi = static_cast<const CellGeo<D> *>(p.cgeo)[i];
    int j = 0;
    for (int t = 0; t < gi.nf; ++t)
        if (gi.face[t] == f) j = t;
    const int nv = p.nv;
    const double dt = p.dt;
    double acc[2 * NW];
#pragma unroll
    for (int m = 0; m < 2 * NW; ++m) acc[m] = 0.0;
    for (int k = threadIdx.x; k < nv; k += BS) {
        double u[D], u2 = 0.0, un = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            u[d] = p.u[d * nv + k];
            u2 += u[d] * u[d];
            un += u[d] * F.n[d];
        }
        const double wk = p.w[k];
        double I[2] = {0.0, 0.0};
        int off = 0;
        if (un > 0.0) {
            double fi[NC], gri[NC][D];
            limited_slope<D, FT>(gi, i, fin, nv, k, p.limiter, fi, gri);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double v = fi[c], ug = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    v += gri[c][d] * gi.dvec[j][d];
                    ug += u[d] * gri[c][d];
                }
                I[c] = dt * v - 0.5 * dt * dt * ug;
            }
        } else {
            double c2 = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const double cd = u[d] - e.U[d];
                c2 += cd * cd;
            }
            I[0] = e.k0 * exp(-e.lam * c2);
            if constexpr (NC > 1) I[1] = e.bh * I[0];
            off = NW;
        }
        const double a = wk * un;
        double mom[NW];
        mom[0] = a * I[0];
#pragma unroll
        for (int d = 0; d < D; ++d) mom[1 + d] = a * u[d] * I[0];
        mom[NW - 1] = a * 0.5 * (u2 * I[0] + I[1]);
#pragma unroll
        for (int m = 0; m < NW; ++m) {
            acc[m] += off ? 0.0 : mom[m];
            acc[NW + m] += off ? mom[m] : 0.0;
        }
    }
    block_reduce<BS>(acc, red, OpAdd{});
    if (threadIdx.x == 0) {
        const double rho_w = acc[NW] != 0.0 ? -acc[0] / acc[NW] : 0.0;
#pragma unroll
        for (int m = 0; m < NW; ++m) out[(size_t)blockIdx.x * NW + m] = (acc[m] + rho_w * acc[NW + m]) / dt;
    }
}

// ------------------------------------------------------------------------
// L2 norm over cells of the last step's change of W (fixed order)
// ------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void residual(const Params p, double *out)
{
    constexpr int NW = D + 2;
    __shared__ double lds[4 * NW];
    double s[NW];
    for (int m = 0; m < NW; ++m) s[m] = 0.0;
    for (int i = threadIdx.x; i < p.nc; i += 256)
        for (int m = 0; m < NW; ++m) s[m] += p.dW2[(size_t)i * NW + m];
    block_reduce<256>(s, lds, OpAdd{});
    if (threadIdx.x == 0)
        for (int m = 0; m < NW; ++m) out[m] = sqrt(s[m]);
}

// One case: workgroup g sums the squared changes of a contiguous range of
// cells into part[g] (fixed order), then one workgroup sums the partial sums
// in order and takes the square roots.  Deterministic, and spread over the
// chip instead of one compute unit.
template <int D>
__global__ __launch_bounds__(256) void k_residual_part(Params p, double *part, int per, double *out)
{
    constexpr int NW = D + 2;
    __shared__ double lds[4 * NW];
    double s[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) s[m] = 0.0;
    const int i0 = blockIdx.x * per, i1 = min(p.nc, i0 + per);
    for (int i = i0 + threadIdx.x; i < i1; i += 256)
#pragma unroll
        for (int m = 0; m < NW; ++m) s[m] += p.dW2[(size_t)i * NW + m];
    block_reduce<256>(s, lds, OpAdd{});
    if (threadIdx.x == 0)
#pragma unroll
        for (int m = 0; m < NW; ++m) {
            part[(size_t)blockIdx.x * NW + m] = s[m];
            if (gridDim.x == 1) out[m] = sqrt(s[m]);  // the only group: no second launch
        }
}

template <int D>
__global__ __launch_bounds__(256) void k_residual_final(const double *__restrict__ part, int ng, double *out)
{
    constexpr int NW = D + 2;
    __shared__ double lds[4 * NW];
    double s[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) s[m] = 0.0;
    for (int g = threadIdx.x; g < ng; g += 256)
#pragma unroll
        for (int m = 0; m < NW; ++m) s[m] += part[(size_t)g * NW + m];
    block_reduce<256>(s, lds, OpAdd{});
    if (threadIdx.x == 0)
#pragma unroll
        for (int m = 0; m < NW; ++m) out[m] = sqrt(s[m]);
}

// ------------------------------------------------------------------------
// Batched launches: the cases of a batch are laid end to end in one grid;
// off[c] is the first workgroup of case c.  Every workgroup finds its case
// by a binary search over off (wave-uniform, scalar) and runs the same
// per-cell or per-face code as the single-case kernels, on that case's
// parameters and buffers, so a case's result does not depend on the batch.
// ------------------------------------------------------------------------
// The descriptors are read-only for a launch: they are read through the
// constant address space, as kernel arguments are, so that the compiler may
// reload a case's parameters instead of holding them all in registers.
#if defined(__HIP_DEVICE_COMPILE__)
typedef const __attribute__((address_space(4))) BatchItem *ConstItems;
#else
typedef const BatchItem *ConstItems;  // the host pass only parses the kernels
#endif

__device__ __forceinline__ int batch_case(const int *__restrict__ off, int n, int b)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <int D>
__global__ __launch_bounds__(kGradBlock) void k_cell_grad_batch(const BatchItem *__restrict__ items, const int *__restrict__ off,
                                                         int n)
{
    const int c = batch_case(off, n, blockIdx.x);
    cell_grad<D>(((ConstItems)items)[c].p, (blockIdx.x - off[c]) * kGradBlock + threadIdx.x);
}

template <int D>
__global__ __launch_bounds__(kFaceBlock) void k_face_eq_batch(const BatchItem *__restrict__ items, const int *__restrict__ off,
                                                       int n)
{
    const int c = batch_case(off, n, blockIdx.x);
    face_eq<D>(((ConstItems)items)[c].p, (blockIdx.x - off[c]) * kFaceBlock + threadIdx.x);
}

template <int D, typename FT, int BS, bool TENSOR, bool S1L>
__device__ __forceinline__ void sweep_batch(const BatchItem *__restrict__ items, const int *__restrict__ off, int n,
                                            int step)
{
    const int c = batch_case(off, n, blockIdx.x);
    ConstItems ci = (ConstItems)(items);
    const int cur = (ci[c].cur + step) & 1;
    sweep_cell<D, FT, BS, TENSOR, S1L, TENSOR>(ci[c].p, xcd_cell(blockIdx.x - off[c]),
                                               static_cast<const FT *>(ci[c].f[cur]),
                                               static_cast<FT *>(const_cast<void *>(ci[c].f[1 - cur])));
}
template <int D, typename FT, int BS, bool S1L>
__global__ __launch_bounds__(BS) void k_sweep_batch(const BatchItem *__restrict__ items, const int *__restrict__ off,
                                                    int n, int step)
{
    sweep_batch<D, FT, BS, false, S1L>(items, off, n, step);
}
template <int D, typename FT, int BS, bool S1L>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_sweep_batch_pf(
    const BatchItem *__restrict__ items, const int *__restrict__ off, int n, int step)
{
    sweep_batch<D, FT, BS, true, S1L>(items, off, n, step);
}

template <int D>
__global__ __launch_bounds__(256) void k_residual_batch(const BatchItem *__restrict__ items)
{
    ConstItems ci = (ConstItems)(items);
    residual<D>(ci[blockIdx.x].p, ci[blockIdx.x].res);
}

// ------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------
template <int D> hipError_t cfl_d(const Params &p, double *cell_dt, hipStream_t s)
{
    hipLaunchKernelGGL(k_cfl<D>, dim3(p.nc), dim3(256), 0, s, p, cell_dt);
    return hipGetLastError();
}
hipError_t launch_cfl(const Params &p, double *cell_dt, hipStream_t s)
{
    return p.dim == 2 ? cfl_d<2>(p, cell_dt, s) : cfl_d<3>(p, cell_dt, s);
}

template <int D, typename FT> hipError_t init_d(const Params &p, const double *prim0, void *f, hipStream_t s)
{
    hipLaunchKernelGGL((k_init<D, FT>), dim3(p.nc), dim3(256), 0, s, p, prim0, static_cast<FT *>(f));
    return hipGetLastError();
}
hipError_t launch_init(const Params &p, const double *prim0, void *f, hipStream_t s)
{
    if (p.dim == 2)
        return p.fstore == 2 ? init_d<2, bf16s>(p, prim0, f, s)
                             : (p.fstore ? init_d<2, float>(p, prim0, f, s) : init_d<2, double>(p, prim0, f, s));
    return p.fstore == 2 ? init_d<3, bf16s>(p, prim0, f, s)
                         : (p.fstore ? init_d<3, float>(p, prim0, f, s) : init_d<3, double>(p, prim0, f, s));
}

template <int D, typename FT> hipError_t moments_d(const Params &p, const void *f, hipStream_t s)
{
    hipLaunchKernelGGL((k_moments<D, FT>), dim3(p.nc), dim3(256), 0, s, p, static_cast<const FT *>(f));
    return hipGetLastError();
}
hipError_t launch_moments(const Params &p, const void *f, hipStream_t s)
{
    if (p.dim == 2)
        return p.fstore == 2 ? moments_d<2, bf16s>(p, f, s)
                             : (p.fstore ? moments_d<2, float>(p, f, s) : moments_d<2, double>(p, f, s));
    return p.fstore == 2 ? moments_d<3, bf16s>(p, f, s)
                         : (p.fstore ? moments_d<3, float>(p, f, s) : moments_d<3, double>(p, f, s));
}

template <int D> hipError_t prologue_d(const Params &p, hipStream_t s)
{
    hipLaunchKernelGGL(k_cell_grad<D>, dim3((p.nc + kGradBlock - 1) / kGradBlock), dim3(kGradBlock), 0, s, p);
    hipLaunchKernelGGL(k_face_eq<D>, dim3((p.nf + kFaceBlock - 1) / kFaceBlock), dim3(kFaceBlock), 0, s, p);
    return hipGetLastError();
}
hipError_t launch_prologue(const Params &p, hipStream_t s)
{
    return p.dim == 2 ? prologue_d<2>(p, s) : prologue_d<3>(p, s);
}

// LDS a workgroup may take while four of them still fit on a CU (160 KB)
constexpr size_t kLdsPerWorkgroup = 40 * 1024;

size_t sweep_lds_bytes(const Params &p, bool *s1l)
{
    const int MF = p.dim == 2 ? Dim<2>::MF : Dim<3>::MF, NW = p.dim + 2, NC = p.dim == 2 ? Dim<2>::NC : Dim<3>::NC;
    const int NRED = NW > 2 * MF ? NW : 2 * MF;
    const size_t lds = sizeof(double) * ((size_t)(MF + 1) * (size_t)p.ntab + (256 / 64) * (size_t)NRED);
    const size_t fv = p.fstore == 2 ? 2 : (p.fstore == 1 ? 4 : 8);
    const size_t slab = fv * NC * (size_t)p.nv;
    *s1l = lds + slab <= kLdsPerWorkgroup;
    return *s1l ? lds + slab : lds;
}

int sweep_grid(int nc)
{
    constexpr int span = UGKS_XCDS * UGKS_XCD_RUN;
    return ((nc + span - 1) / span) * span;
}

// The same as a grid of workgroups of bs threads.  A dimension of a launch
// takes fewer than 2^32 work-items, which 16,000,000 workgroups of 256 threads
// keep and wider ones do not: those go in rows (row_block).
inline dim3 cell_grid(int nc, int bs)
{
    constexpr unsigned span = UGKS_XCDS * UGKS_XCD_RUN;
    const unsigned n = (unsigned)sweep_grid(nc), row = 0xffffffffu / (unsigned)bs / span * span;
    return n <= row ? dim3(n) : dim3(row, (n + row - 1) / row);
}

template <int D, typename FT, int BS, bool TENSOR>
void sweep_launch(const Params &p, const void *fi, void *fo, hipStream_t s)
{
    bool s1l = false;
    const size_t lds = sweep_lds_bytes(p, &s1l);
    const unsigned grid = (unsigned)sweep_grid(p.nc);
    const FT *in = static_cast<const FT *>(fi);
    FT *out = static_cast<FT *>(fo);
    if constexpr (TENSOR) {
        if (s1l) hipLaunchKernelGGL((k_sweep_pf<D, FT, BS, true>), dim3(grid), dim3(BS), lds, s, p, in, out);
        else hipLaunchKernelGGL((k_sweep_pf<D, FT, BS, false>), dim3(grid), dim3(BS), lds, s, p, in, out);
    } else {
        if (s1l) hipLaunchKernelGGL((k_sweep<D, FT, BS, false, true>), dim3(grid), dim3(BS), lds, s, p, in, out);
        else hipLaunchKernelGGL((k_sweep<D, FT, BS, false, false>), dim3(grid), dim3(BS), lds, s, p, in, out);
    }
}

template <int D, typename FT> hipError_t sweep_d(const Params &p, const void *fi, void *fo, hipStream_t s)
{
    if (p.ntab > 0) sweep_launch<D, FT, 256, true>(p, fi, fo, s);
    else sweep_launch<D, FT, 256, false>(p, fi, fo, s);
    return hipGetLastError();
}
template <int D, typename FT, bool TENSOR> hipError_t inplace_d(const Params &p, void *fv, bool walls, hipStream_t s)
{
    constexpr int MF = Dim<D>::MF, NW = D + 2, NRED = (NW > 2 * MF) ? NW : 2 * MF;
    const size_t lds = sizeof(double) * ((size_t)(MF + 1) * (TENSOR ? p.ntab : 0) + (256 / 64) * NRED);
    const unsigned grid = (unsigned)sweep_grid(p.nc);
    FT *f = static_cast<FT *>(fv);
    if (walls) hipLaunchKernelGGL((k_wall_density<D, FT, 256, TENSOR>), dim3(grid), dim3(256), lds, s, p, f);
    for (int q = 0; q < p.nchunk; ++q) {
        const int c0 = q * p.chunk, cn = std::min(p.chunk, p.nv - c0);
        const int prev0 = (q - 1) * p.chunk, prevn = q > 0 ? p.chunk : 0;
        hipLaunchKernelGGL((k_sweep_chunk<D, FT, 256, TENSOR>), dim3(grid), dim3(256), lds, s, p, f, c0, cn, prev0,
                           prevn, q);
    }
    const int last0 = (p.nchunk - 1) * p.chunk;
    hipLaunchKernelGGL((k_sweep_finish<D, FT, 256, TENSOR>), dim3(grid), dim3(256), lds, s, p, f, last0,
                       p.nv - last0);
    return hipGetLastError();
}
template <int D, typename FT> hipError_t inplace_t(const Params &p, void *f, bool walls, hipStream_t s)
{
    return p.ntab > 0 ? inplace_d<D, FT, true>(p, f, walls, s) : inplace_d<D, FT, false>(p, f, walls, s);
}
hipError_t launch_sweep_inplace(const Params &p, void *f, bool walls, hipStream_t s)
{
    if (p.dim == 2)
        return p.fstore == 2 ? inplace_t<2, bf16s>(p, f, walls, s)
                             : (p.fstore ? inplace_t<2, float>(p, f, walls, s) : inplace_t<2, double>(p, f, walls, s));
    return p.fstore == 2 ? inplace_t<3, bf16s>(p, f, walls, s)
                         : (p.fstore ? inplace_t<3, float>(p, f, walls, s) : inplace_t<3, double>(p, f, walls, s));
}

hipError_t launch_sweep(const Params &p, const void *fi, void *fo, hipStream_t s)
{
    if (p.dim == 2)
        return p.fstore == 2 ? sweep_d<2, bf16s>(p, fi, fo, s)
                             : (p.fstore ? sweep_d<2, float>(p, fi, fo, s) : sweep_d<2, double>(p, fi, fo, s));
    return p.fstore == 2 ? sweep_d<3, bf16s>(p, fi, fo, s)
                         : (p.fstore ? sweep_d<3, float>(p, fi, fo, s) : sweep_d<3, double>(p, fi, fo, s));
}

// ------------------------------------------------------------------------
// Sums over a wavefront of N values at once, the totals uniform.  Two values
// share each of the first two steps: a half-wave swap turns (a, b) into one
// register that holds a's pair sums in the lower 32 lanes and b's in the
// upper 32, a row swap does the same for the two 16-lane rows, and four row
// rotations finish four values together.  21 vector instructions for four
// values and no LDS, where a butterfly of every value takes 72 and 48 LDS
// permutes.
// ------------------------------------------------------------------------
template <bool ROW> __device__ __forceinline__ double swap_add(double a, double b)
{
    typedef unsigned uint2v __attribute__((ext_vector_type(2)));
    auto swap = [](unsigned x, unsigned y) -> uint2v {
        if constexpr (ROW) return __builtin_bit_cast(uint2v, __builtin_amdgcn_permlane16_swap(x, y, false, false));
        else return __builtin_bit_cast(uint2v, __builtin_amdgcn_permlane32_swap(x, y, false, false));
    };
    const uint2v lo = swap((unsigned)__double2loint(a), (unsigned)__double2loint(b));
    const uint2v hi = swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b));
    return __hiloint2double((int)hi.x, (int)lo.x) + __hiloint2double((int)hi.y, (int)lo.y);
}
template <int CTRL> __device__ __forceinline__ double row_rotate(double x)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ double read_lane(double x, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}
template <int N> __device__ __forceinline__ void wave_sums(double (&v)[N])
{
#pragma unroll
    for (int g = 0; g < N; g += 4) {
        const double b = g + 1 < N ? v[g + 1 < N ? g + 1 : 0] : 0.0, c = g + 2 < N ? v[g + 2 < N ? g + 2 : 0] : 0.0,
                     d = g + 3 < N ? v[g + 3 < N ? g + 3 : 0] : 0.0;
        // rows of 16 lanes: v[g], v[g + 2], v[g + 1], v[g + 3]
        double x = swap_add<true>(swap_add<false>(v[g], b), swap_add<false>(c, d));
        x += row_rotate<0x128>(x);
        x += row_rotate<0x124>(x);
        x += row_rotate<0x122>(x);
        x += row_rotate<0x121>(x);
        v[g] = read_lane(x, 0);
        if (g + 1 < N) v[g + 1 < N ? g + 1 : 0] = read_lane(x, 32);
        if (g + 2 < N) v[g + 2 < N ? g + 2 : 0] = read_lane(x, 16);
        if (g + 3 < N) v[g + 3 < N ? g + 3 : 0] = read_lane(x, 48);
    }
}

template <int D> struct Shift {
    static constexpr int NC = Dim<D>::NC, NM = D * (D + 1) / 2;
    static constexpr int N = 1 + D + NM + D + (NC > 1 ? 1 + D : 0);
};

// one velocity's contribution to the moments about U^n (c = u - U^n)
template <int D>
__device__ __forceinline__ void add_shift_moments(double (&mm)[Shift<D>::N], double w, const double (&c)[D], double c2,
                                                  double h, double b)
{
    constexpr int NM = Shift<D>::NM;
    const double wh = w * h;
    mm[0] += wh;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const double whc = wh * c[a];
        mm[1 + a] += whc;
        mm[1 + D + NM + a] = fma(whc, c2, mm[1 + D + NM + a]);
#pragma unroll
        for (int bb = a; bb < D; ++bb) mm[1 + D + sym_index<D>(a, bb)] = fma(whc, c[bb], mm[1 + D + sym_index<D>(a, bb)]);
    }
    if constexpr (Dim<D>::NC > 1) {
        const double wb = w * b;
        mm[1 + 2 * D + NM] += wb;
#pragma unroll
        for (int a = 0; a < D; ++a) mm[2 + 2 * D + NM + a] = fma(wb, c[a], mm[2 + 2 * D + NM + a]);
    }
}

// W^{n+1} (W^n + the stage-1 moments - the base's moments), its primitive
// state, tau^{n+1} and q^{n+1} (the re-centred heat flux of the stage-1
// values) from the moments about U^n
template <int D>
__device__ __forceinline__ void macro_from_shift(const Params &p, const double (&mm)[Shift<D>::N],
                                                 const double (&Wn)[D + 2], const Prim<D> &pn, const double *mom_base,
                                                 double (&W1)[D + 2], Prim<D> &p1, double &tau1, double (&q1)[D])
{
    constexpr int NW = D + 2, NM = Shift<D>::NM, NC = Dim<D>::NC;
    const double m0 = mm[0];
    const double b0 = NC > 1 ? mm[1 + 2 * D + NM] : 0.0;
    double m1[D], m3[D], b1[D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        m1[a] = mm[1 + a];
        m3[a] = mm[1 + D + NM + a];
        b1[a] = NC > 1 ? mm[2 + 2 * D + NM + a] : 0.0;
    }
    double mom[NW], trm2 = 0.0, um1 = 0.0, uu = 0.0;
    mom[0] = m0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        mom[1 + a] = fma(pn.U[a], m0, m1[a]);
        trm2 += mm[1 + D + sym_index<D>(a, a)];
        um1 = fma(pn.U[a], m1[a], um1);
        uu = fma(pn.U[a], pn.U[a], uu);
    }
    mom[D + 1] = 0.5 * (trm2 + 2.0 * um1 + uu * m0 + b0);
#pragma unroll
    for (int m = 0; m < NW; ++m) W1[m] = Wn[m] + (mom[m] - mom_base[m]);
    p1 = to_prim<D>(W1);
    tau1 = collision_time(p1.rho, p1.lam, p.mu_ref, p.omega);
    double dl[D], d2 = 0.0, m1d = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        dl[a] = p1.U[a] - pn.U[a];
        d2 = fma(dl[a], dl[a], d2);
        m1d = fma(m1[a], dl[a], m1d);
    }
    const double qden = 1.0 + p.Pr * p.dt / (2.0 * tau1);
#pragma unroll
    for (int a = 0; a < D; ++a) {
        double m2d = 0.0;
#pragma unroll
        for (int bb = 0; bb < D; ++bb) m2d = fma(mm[1 + D + sym_index<D>(a, bb)], dl[bb], m2d);
        const double qa = m3[a] - 2.0 * m2d + d2 * m1[a] - dl[a] * trm2 + 2.0 * dl[a] * m1d - dl[a] * d2 * m0 + b1[a] -
                          dl[a] * b0;
        q1[a] = 0.5 * qa / qden;
    }
}

// ------------------------------------------------------------------------
// The push sweep's per-cell kernels: one workgroup per cell, thread t taking
// the velocity pairs t, t + BS, ... of its slab.  The final kernel takes the
// moments of the stage-1 slab about U^n (orders 0-3 of h, 0-1 of b), from
// which one wavefront forms W^{n+1}, tau^{n+1} and the heat flux about U^{n+1}
// (macro_from_shift), and applies stage 2 into f and the next step's base into
// acc.  The base kernel takes the velocities in the same order and reduces the
// same way, so both give the same bits.
//
// FP64 stage-1 sums are loaded in one go into registers -- every load of a
// thread in flight together -- and the slab is read once: NP pairs a thread at
// most, every velocity count a handle takes fits one of the forms of
// launch_final (of the eight pairs of the widest, up to 18 registers are
// spilled in 2D in the 128 that its 1,024 threads leave).  Bound by the latency of a
// cell's phases at two workgroups a CU (VALUs half busy); 107,118 cells x
// 4,548: 3.78 -> 2.90 ms (11.7 GB, 4.0 TB/s); 50,688 x 13,824 7.36 -> 4.95 ms;
// against one wavefront per cell (and slabs of at most 24 values in 256
// threads), butterfly sums and the points read from memory in both passes.
//
// FP32 stage-1 sums (FP32 and BF16 f) are read again in the second pass (NP =
// 0): half the bytes, found in L2, and workgroups of few wavefronts and registers
// (held to six waves a SIMD, five for scattered BF16, which spills at six)
// overlap the phases of more cells on a CU.  The final kernel with the slab in
// registers / read again, FP32 f: 16,200 cells in 2D x 2,145 396 / 328 us, x
// 3,600 553 / 491; 64,000 in 3D x 100 297 / 126; a step of 19,683 in 3D x 6,000
// 2,751 / 2,394 us, BF16 2,755 / 2,328.
// ------------------------------------------------------------------------
// Elements k, k + 1 of an array of n (k < n): one access where the pair is
// aligned (pairs from even elements of slabs that start at even elements),
// else two, of k and k + step; zero past the end.
template <typename T>
__device__ __forceinline__ void load_pair(const T *__restrict__ q, int k, int n, bool aligned, double &a, double &b,
                                          int step = 1)
{
    if (aligned) {
        load2<T>(q + k, a, b);
    } else {
        a = to_f64(q[k]);
        b = k + step < n ? to_f64(q[k + step]) : 0.0;
    }
}
template <typename T>
__device__ __forceinline__ void store_pair(T *__restrict__ q, int k, int n, bool aligned, T a, T b, int step = 1)
{
    if (aligned) {
        store2<T>(q + k, a, b);
    } else {
        q[k] = a;
        if (k + step < n) q[k + step] = b;
    }
}

// The first velocity of a thread's j-th pair in a slab: neighbours where pairs
// are aligned, else two a workgroup's width apart, so that the single accesses
// of a wavefront still lie side by side.
template <int BS> __device__ __forceinline__ int pair_first(int j, bool aligned)
{
    return aligned ? 2 * ((int)threadIdx.x + BS * j) : (int)threadIdx.x + 2 * BS * j;
}

// A velocity pair's weights (zero past the last velocity) and, where the set
// is tabulated, its table positions, else its points.  The streaming kernels
// take the points of a tabulated set from LDS: the 24 bytes a velocity that a
// point takes, twice a cell, were two thirds of what these kernels drew from
// L2, which they ran at the rate of (12 TB/s).
template <int D, bool TENSOR> struct VelPair {
    double w[2], u[TENSOR ? 1 : 2][D];
    unsigned kx[2];
    // velocities k0, k0 + 1 (not aligned: k0 + step) of those below n
    __device__ __forceinline__ void load(const Params &p, int k0, int n, bool aligned, int step = 1)
    {
        load_pair<double>(p.w, k0, n, aligned, w[0], w[1], step);
        kx[0] = kx[1] = 0u;
        if constexpr (TENSOR) {
            if (!aligned) {
                kx[0] = (unsigned)p.kidx[k0];
                if (k0 + step < n) kx[1] = (unsigned)p.kidx[k0 + step];
            } else {
                const int2 x = *reinterpret_cast<const int2 *>(p.kidx + k0);
                kx[0] = (unsigned)x.x;
                kx[1] = (unsigned)x.y;
            }
        } else {
#pragma unroll
            for (int d = 0; d < D; ++d) load_pair<double>(p.u + (size_t)d * p.nv, k0, n, aligned, u[0][d], u[1][d], step);
        }
    }
    // peculiar velocity of element e: from the table of u_d - U_d, or the points
    __device__ __forceinline__ void peculiar_of(int e, const double *tc, const double (&U)[D], double (&c)[D],
                                                double &c2) const
    {
        if constexpr (TENSOR) {
            c2 = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                c[d] = tc[kx[e] >> (10 * d) & 1023u];
                c2 = fma(c[d], c[d], c2);
            }
        } else {
            peculiar<D>(u[e], U, c, c2);
        }
    }
    // the same and the Gaussian, from the table of (u_d - U_d, exp(-lam (u_d - U_d)^2))
    __device__ __forceinline__ double gauss_of(int e, const double2 *tg, const double (&U)[D], double lam,
                                               double (&c)[D], double &c2) const
    {
        if constexpr (TENSOR) {
            double g = 1.0;
            c2 = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const double2 x = tg[kx[e] >> (10 * d) & 1023u];
                c[d] = x.x;
                c2 = fma(c[d], c[d], c2);
                g = d == 0 ? x.y : g * x.y;
            }
            return g;
        } else {
            peculiar<D>(u[e], U, c, c2);
            return exp(-lam * c2);
        }
    }
};

__device__ __forceinline__ double axis_point(const Params &p, int idx, double U0, double U1, double U2)
{
    return p.u1d[idx] - (idx < p.n1d[0] ? U0 : (idx < p.n1d[0] + p.n1d[1] ? U1 : U2));
}
template <int BS>
__device__ __forceinline__ void fill_points(const Params &p, double U0, double U1, double U2, double *tc)
{
    for (int idx = threadIdx.x; idx < p.ntab; idx += BS) tc[idx] = axis_point(p, idx, U0, U1, U2);
}
template <int BS>
__device__ __forceinline__ void fill_gauss(const Params &p, double lam, double U0, double U1, double U2, double2 *tg)
{
    for (int idx = threadIdx.x; idx < p.ntab; idx += BS) {
        const double c = axis_point(p, idx, U0, U1, U2);
        tg[idx] = make_double2(c, exp(-lam * c * c));
    }
}

// conservative moments (1, u, (|u|^2 h + b) / 2) from those of c = u - U
template <int D> __device__ __forceinline__ double recentred(const double *m, const double (&U)[D], int n)
{
    if (n == 0) return m[0];
    double um = 0.0, uu = 0.0, r = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        um = fma(U[d], m[1 + d], um);
        uu = fma(U[d], U[d], uu);
        if (n == 1 + d) r = fma(U[d], m[0], m[1 + d]);
    }
    return n == D + 1 ? fma(0.5 * uu, m[0], um) + m[D + 1] : r;
}

// moments of the workgroup's wavefronts summed in their order by threads 0..N
template <int BS, int N> __device__ __forceinline__ double group_total(const double *red, int n)
{
    double s = red[n];
    for (int w = 1; w < BS / 64; ++w) s += red[w * N + n];
    return s;
}

// the base's moments, from the wavefronts' sums about U (first wavefront)
template <int D, int BS>
__device__ __forceinline__ void store_base_moments(const Params &p, int i, const double *red, const double (&U)[D])
{
    constexpr int NW = D + 2;
    if (threadIdx.x >= 64) return;
    const int n = threadIdx.x;
    const double s = n < NW ? group_total<BS, NW>(red, n) : 0.0;
    double m[NW];
#pragma unroll
    for (int t = 0; t < NW; ++t) m[t] = read_lane(s, t);
    const double r = recentred<D>(m, U, n);
    if (n < NW) p.mom_part[(size_t)i * NW + n] = r;
}

template <int D, typename FT, bool TENSOR, int BS>
__global__ __launch_bounds__(BS) void k_push_base(Params p, const FT *__restrict__ fin,
                                                  typename AccOf<FT>::T *__restrict__ acc)
{
    using AT = typename AccOf<FT>::T;
    constexpr int NC = Dim<D>::NC, NW = D + 2;
    extern __shared__ double smem[];
    const int i = xcd_cell(row_block());
    if (i >= p.nc) return;
    const int nv = p.nv, tid = threadIdx.x;
    const bool aligned = nv % 2 == 0;
    const CellStep<D> cs = cell_step<D>(p, i);
    double2 *tg = reinterpret_cast<double2 *>(smem);
    double *red = smem + (TENSOR ? 2 * p.ntab : 0);
    if constexpr (TENSOR) {
        fill_gauss<BS>(p, cs.pn.lam, cs.pn.U[0], cs.pn.U[1], cs.pn.U[D - 1], tg);
        __syncthreads();
    }
    const size_t base = (size_t)i * NC * nv;
    double mom[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) mom[m] = 0.0;
#pragma unroll 2
    for (int k0 = pair_first<BS>(0, aligned); k0 < nv; k0 += 2 * BS) {
        double f[NC][2];
        VelPair<D, TENSOR> vp;
        vp.load(p, k0, nv, aligned, BS);
#pragma unroll
        for (int c = 0; c < NC; ++c) load_pair<FT>(fin + base + (size_t)c * nv, k0, nv, aligned, f[c][0], f[c][1], BS);
        AT sv[NC][2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            double c3[D], c2, fp[2], bv[2] = {0.0, 0.0};
            const double H = cs.pref_n * vp.gauss_of(e, tg, cs.pn.U, cs.pn.lam, c3, c2);
            shakhov_at<D>(c3, c2, cs.pn.lam, cs.shk_n, cs.qn, cs.bh_n, H, fp[0], fp[1]);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                sv[c][e] = from_f64<AT>(fma(cs.hdt_tau, fp[c] - f[c][e], f[c][e]));
                bv[c] = to_f64(sv[c][e]);
            }
            add_moments<D>(mom, vp.w[e], c3, c2, bv[0], NC > 1 ? bv[NC - 1] : 0.0);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) store_pair<AT>(acc + base + (size_t)c * nv, k0, nv, aligned, sv[c][0], sv[c][1], BS);
    }
    wave_sums<NW>(mom);
    if ((tid & 63) == 0)
#pragma unroll
        for (int m = 0; m < NW; ++m) red[(tid >> 6) * NW + m] = mom[m];
    __syncthreads();
    store_base_moments<D, BS>(p, i, red, cs.pn.U);
}

// The macroscopic update of cell i from the stage-1 moments about U^n, by one
// wavefront: W^{n+1}, q^{n+1} and the squared change of W to memory, and for
// the workgroup's pass over f^{n+1} to LDS lam, the prefactors of f+, dt / 2
// tau (res[0..4)), U and q (then).
template <int D>
__device__ __forceinline__ void group_macro(const Params &p, int i, const double (&mm)[Shift<D>::N],
                                            const double (&Wn)[D + 2], const Prim<D> &pn, double *res)
{
    constexpr int NW = D + 2;
    const int tid = threadIdx.x;
    double W1[NW], tau1, q1[D];
    Prim<D> p1;
    macro_from_shift<D>(p, mm, Wn, pn, p.mom_part + (size_t)i * NW, W1, p1, tau1, q1);
    if (tid == 0) {
        res[0] = p1.lam;
        res[1] = p1.rho * pow_lam_pi<D>(p1.lam);
        res[2] = 4.0 * (1.0 - p.Pr) * p1.lam * p1.lam / (5.0 * p1.rho);
        res[3] = 0.5 * p.dt / tau1;
        bool ok = p1.rho > 0.0 && p1.lam > 0.0 && isfinite(p1.rho) && isfinite(p1.lam);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            res[4 + d] = p1.U[d];
            res[4 + D + d] = q1[d];
            p.q[(size_t)i * D + d] = q1[d];
        }
#pragma unroll
        for (int m = 0; m < NW; ++m) {
            ok = ok && isfinite(W1[m]);
            p.W[(size_t)i * NW + m] = W1[m];
            const double dw = W1[m] - Wn[m];
            p.dW2[(size_t)i * NW + m] = dw * dw;
        }
        if (!ok) {
            atomicOr(p.err, 1);
            atomicMin(p.err + 1, i);
        }
    }
}

template <int D, typename FT, bool TENSOR, int BS, int NP>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(NP > 0 ? 1 : (TENSOR || sizeof(FT) == 4 ? 6 : 5)))) void k_push_final(Params p, FT *__restrict__ fout, typename AccOf<FT>::T *__restrict__ acc)
{
    using AT = typename AccOf<FT>::T;
    constexpr int NC = Dim<D>::NC, NW = D + 2, N = Shift<D>::N;
    extern __shared__ double smem[];
    const int i = xcd_cell(row_block());
    if (i >= p.nc) return;
    const int tid = threadIdx.x, nv = p.nv;
    const bool aligned = nv % 2 == 0;
    const size_t base = (size_t)i * NC * nv;
    double2 *tg = reinterpret_cast<double2 *>(smem);  // about U^{n+1}
    double *tc = smem + (TENSOR ? 2 * p.ntab : 0);    // about U^n
    double *red = tc + (TENSOR ? p.ntab : 0), *res = red + (BS / 64) * N;
    double Wn[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) Wn[m] = p.W[(size_t)i * NW + m];
    const Prim<D> pn = to_prim<D>(Wn);

    // pass 1: the slab into registers, in its storage precision (all loads
    // issued before any use), its moments about U^n; without register pairs
    // each pass loads a pair as it comes to it
    constexpr bool REG = NP > 0;
    AT v[REG ? NP : 1][NC][2];
    auto load_slab = [&](int k0, AT (&x)[NC][2]) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            x[c][0] = x[c][1] = from_f64<AT>(0.0);
            if (k0 < nv) {
                const AT *q = acc + base + (size_t)c * nv + k0;
                if (!aligned) {
                    x[c][0] = q[0];
                    if (k0 + BS < nv) x[c][1] = q[BS];
                } else {
                    const typename Vec2<AT>::T y = *reinterpret_cast<const typename Vec2<AT>::T *>(q);
                    x[c][0] = y.x;
                    x[c][1] = y.y;
                }
            }
        }
    };
    if constexpr (REG)
#pragma unroll
        for (int j = 0; j < NP; ++j) load_slab(pair_first<BS>(j, aligned), v[j]);
    if constexpr (TENSOR) {
        fill_points<BS>(p, pn.U[0], pn.U[1], pn.U[D - 1], tc);
        __syncthreads();
    }
    double mm[N];
#pragma unroll
    for (int t = 0; t < N; ++t) mm[t] = 0.0;
#pragma unroll REG ? NP : 1
    for (int j = 0; REG ? j < NP : pair_first<BS>(j, aligned) < nv; ++j) {
        const int k0 = pair_first<BS>(j, aligned);
        AT (&x)[NC][2] = v[REG ? j : 0];
        if constexpr (!REG) load_slab(k0, x);
        if (k0 < nv) {
            VelPair<D, TENSOR> vp;
            vp.load(p, k0, nv, aligned, BS);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                double c[D], c2;
                vp.peculiar_of(e, tc, pn.U, c, c2);
                add_shift_moments<D>(mm, vp.w[e], c, c2, to_f64(x[0][e]), NC > 1 ? to_f64(x[NC - 1][e]) : 0.0);
            }
        }
    }
    wave_sums<N>(mm);
    if ((tid & 63) == 0)
#pragma unroll
        for (int t = 0; t < N; ++t) red[(tid >> 6) * N + t] = mm[t];
    __syncthreads();
    // macro, by the first wavefront for the others
    if (tid < 64) {
        const double s = tid < N ? group_total<BS, N>(red, tid) : 0.0;
#pragma unroll
        for (int t = 0; t < N; ++t) mm[t] = read_lane(s, t);
        group_macro<D>(p, i, mm, Wn, pn, res);
    }
    __syncthreads();
    const double lam = res[0], pref = res[1], shk = res[2], a1 = res[3], inv1 = 1.0 / (1.0 + a1);
    const double bh = Dim<D>::M / (2.0 * lam);
    double U[D], q1[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        U[d] = res[4 + d];
        q1[d] = res[4 + D + d];
    }
    if constexpr (TENSOR) {
        fill_gauss<BS>(p, lam, U[0], U[1], U[D - 1], tg);
        __syncthreads();
    }

    // pass 2: stage 2 into f, the next base into acc
    double mb[NW];
#pragma unroll
    for (int m = 0; m < NW; ++m) mb[m] = 0.0;
#pragma unroll REG ? NP : 1
    for (int j = 0; REG ? j < NP : pair_first<BS>(j, aligned) < nv; ++j) {
        const int k0 = pair_first<BS>(j, aligned);
        AT (&x)[NC][2] = v[REG ? j : 0];
        if constexpr (!REG) load_slab(k0, x);
        if (k0 < nv) {
            VelPair<D, TENSOR> vp;
            vp.load(p, k0, nv, aligned, BS);
            FT fo[NC][2];
            AT bo[NC][2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                double c3[D], c2, fp[2], bv[2] = {0.0, 0.0};
                const double H = pref * vp.gauss_of(e, tg, U, lam, c3, c2);
                shakhov_at<D>(c3, c2, lam, shk, q1, bh, H, fp[0], fp[1]);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    fo[c][e] = from_f64<FT>((to_f64(x[c][e]) + a1 * fp[c]) * inv1);
                    // the base from f^{n+1} as stored (bitwise what the base
                    // kernel computes from it after a restart)
                    const double fd = opaque(to_f64(fo[c][e]));
                    bo[c][e] = from_f64<AT>(fma(a1, fp[c] - fd, fd));
                    bv[c] = to_f64(bo[c][e]);
                }
                add_moments<D>(mb, vp.w[e], c3, c2, bv[0], NC > 1 ? bv[NC - 1] : 0.0);
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                store_pair<FT>(fout + base + (size_t)c * nv, k0, nv, aligned, fo[c][0], fo[c][1], BS);
                store_pair<AT>(acc + base + (size_t)c * nv, k0, nv, aligned, bo[c][0], bo[c][1], BS);
            }
        }
    }
    wave_sums<NW>(mb);
    if ((tid & 63) == 0)
#pragma unroll
        for (int m = 0; m < NW; ++m) red[(tid >> 6) * NW + m] = mb[m];
    __syncthreads();
    store_base_moments<D, BS>(p, i, red, U);
}

// ------------------------------------------------------------------------
// Push sweep with one f buffer (the in-place mode).  The velocities are taken
// in chunks; per chunk, the base of the chunk's velocities goes into a ring of
// one chunk per cell (its moments added to the cell's running sum), the
// colour launches push the chunk's face fluxes into the ring, and the next
// turn kernel writes the stage-1 values back into f -- no later launch reads
// f^n at those velocities -- adding their moments about U^n (orders 0-3 of h,
// 0-1 of b) to a second running sum, before it fills the ring with the next
// chunk's base.  After the last chunk a final kernel forms
// W^{n+1}, tau^{n+1}, q^{n+1} from the two sums and applies stage 2 in place.
// The wall kernel runs first, while f still holds f^n at every velocity.
// ------------------------------------------------------------------------
// The turn between two chunks, per cell: the previous chunk's stage-1
// values from the ring back into f, their moments about U^n added to mom_s;
// then the base of the next chunk's velocities into the ring, its moments
// added to mom_part (a chunk index of -1 skips that half; chunk 0 starts
// each sum).  Each cell's ring slice is touched only by its own workgroup.
// Bound by a cell's fixed work rather than its bytes at the default chunk (two
// velocity pairs a thread): the constants come from the prologue, the sums go
// by lane swaps, the points from the Gaussian table in LDS.  107,118 cells x
// 4,548 in FP64, a turn of both halves 1.35 -> 0.86 ms, the final kernel
// below 2.38 -> 1.60 (7.8 GB, 4.9 TB/s), against constants formed by every
// wavefront of every turn, butterfly sums and points from memory.
template <int D, typename FT, bool TENSOR>
__global__ __launch_bounds__(256) void k_push_chunk_turn(Params p, FT *__restrict__ f,
                                                         typename AccOf<FT>::T *__restrict__ ring, int pc0, int pcn,
                                                         int pq, int nc0, int ncn, int nq)
{
    using AT = typename AccOf<FT>::T;
    constexpr int NC = Dim<D>::NC, NW = D + 2, BS = 256, N = Shift<D>::N;
    extern __shared__ double smem[];
    const int i = xcd_cell(blockIdx.x);
    if (i >= p.nc) return;
    const int nv = p.nv, ch = p.chunk, tid = threadIdx.x;
    // (chunks start at multiples of ch)
    const bool aligned = (nv | ch) % 2 == 0;
    const size_t fb = (size_t)i * NC * nv, rb = (size_t)i * NC * ch;
    double2 *tg = reinterpret_cast<double2 *>(smem);
    double *red = smem + (TENSOR ? 2 * p.ntab : 0), *red2 = red + (BS / 64) * N;
    const CellConst<D> &cs = static_cast<const CellConst<D> *>(p.cconst)[i];
    double U[D], q[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        U[d] = cs.U[d];
        q[d] = p.q[(size_t)i * D + d];
    }
    const double lam = cs.lam, pref = cs.pref, shk = cs.shk, hdt_tau = cs.hdt_tau, bh = Dim<D>::M / (2.0 * lam);
    if constexpr (TENSOR) {
        fill_gauss<BS>(p, lam, U[0], U[1], U[D - 1], tg);
        __syncthreads();
    }
    if (pq >= 0) {
        double mm[N];
#pragma unroll
        for (int t = 0; t < N; ++t) mm[t] = 0.0;
#pragma unroll 2
        for (int kk = 2 * tid; kk < pcn; kk += 2 * BS) {
            VelPair<D, TENSOR> vp;
            vp.load(p, pc0 + kk, pc0 + pcn, aligned);
            double v[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                // the moments are taken of the stage-1 value as summed (FP32
                // for bfloat16 f), as in the two-buffer final kernel
                load_pair<AT>(ring + rb + (size_t)c * ch, kk, pcn, aligned, v[0][c], v[1][c]);
                store_pair<FT>(f + fb + (size_t)c * nv + pc0, kk, pcn, aligned, from_f64<FT>(v[0][c]),
                               from_f64<FT>(v[1][c]));
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                double c3[D], c2;
                if constexpr (TENSOR) {
                    (void)vp.gauss_of(e, tg, U, lam, c3, c2);
                } else {
                    vp.peculiar_of(e, nullptr, U, c3, c2);
                }
                add_shift_moments<D>(mm, vp.w[e], c3, c2, v[e][0], NC > 1 ? v[e][NC - 1] : 0.0);
            }
        }
        wave_sums<N>(mm);
        if ((tid & 63) == 0)
#pragma unroll
            for (int t = 0; t < N; ++t) red[(tid >> 6) * N + t] = mm[t];
    }
    if (nq >= 0) {
        double mom[NW];
#pragma unroll
        for (int m = 0; m < NW; ++m) mom[m] = 0.0;
#pragma unroll 2
        for (int kk = 2 * tid; kk < ncn; kk += 2 * BS) {
            VelPair<D, TENSOR> vp;
            vp.load(p, nc0 + kk, nc0 + ncn, aligned);
            double fv[NC][2];
#pragma unroll
            for (int c = 0; c < NC; ++c)
                load_pair<FT>(f + fb + (size_t)c * nv + nc0, kk, ncn, aligned, fv[c][0], fv[c][1]);
            AT sv[NC][2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                double c3[D], c2, fp[2], bv[2] = {0.0, 0.0};
                const double H = pref * vp.gauss_of(e, tg, U, lam, c3, c2);
                shakhov_at<D>(c3, c2, lam, shk, q, bh, H, fp[0], fp[1]);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    sv[c][e] = from_f64<AT>(fma(hdt_tau, fp[c] - fv[c][e], fv[c][e]));
                    bv[c] = to_f64(sv[c][e]);
                }
                add_moments<D>(mom, vp.w[e], c3, c2, bv[0], NC > 1 ? bv[NC - 1] : 0.0);
            }
#pragma unroll
            for (int c = 0; c < NC; ++c)
                store_pair<AT>(ring + rb + (size_t)c * ch, kk, ncn, aligned, sv[c][0], sv[c][1]);
        }
        wave_sums<NW>(mom);
        if ((tid & 63) == 0)
#pragma unroll
            for (int m = 0; m < NW; ++m) red2[(tid >> 6) * NW + m] = mom[m];
    }
    __syncthreads();
    // the chunks' sums, in chunk order
    if (pq >= 0 && tid < N) {
        double *m = p.mom_s + (size_t)i * N + tid;
        *m = (pq == 0 ? 0.0 : *m) + group_total<BS, N>(red, tid);
    }
    if (nq >= 0 && tid >= 64 && tid < 128) {
        const int n = tid - 64;
        const double s = n < NW ? group_total<BS, NW>(red2, n) : 0.0;
        double m[NW];
#pragma unroll
        for (int t = 0; t < NW; ++t) m[t] = read_lane(s, t);
        const double r = recentred<D>(m, U, n);
        if (n < NW) {
            double *mp = p.mom_part + (size_t)i * NW + n;
            *mp = (nq == 0 ? 0.0 : *mp) + r;
        }
    }
}

// after the last chunk: W^{n+1}, tau^{n+1}, q^{n+1}, stage 2 in place
template <int D, typename FT, bool TENSOR>
__global__ __launch_bounds__(256) void k_push_final_inplace(Params p, FT *__restrict__ f)
{
    constexpr int NC = Dim<D>::NC, NW = D + 2, BS = 256, N = Shift<D>::N;
    extern __shared__ double smem[];
    const int i = xcd_cell(blockIdx.x);
    if (i >= p.nc) return;
    const int nv = p.nv, tid = threadIdx.x;
    const bool aligned = nv % 2 == 0;
    double2 *tg = reinterpret_cast<double2 *>(smem);
    double *res = smem + (TENSOR ? 2 * p.ntab : 0);
    if (tid < 64) {
        double Wn[NW], mm[N];
#pragma unroll
        for (int m = 0; m < NW; ++m) Wn[m] = p.W[(size_t)i * NW + m];
        const Prim<D> pn = to_prim<D>(Wn);
#pragma unroll
        for (int t = 0; t < N; ++t) mm[t] = p.mom_s[(size_t)i * N + t];
        group_macro<D>(p, i, mm, Wn, pn, res);
    }
    __syncthreads();
    const double lam = res[0], pref = res[1], shk = res[2], a1 = res[3], inv1 = 1.0 / (1.0 + a1);
    const double bh = Dim<D>::M / (2.0 * lam);
    double U[D], q1[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        U[d] = res[4 + d];
        q1[d] = res[4 + D + d];
    }
    if constexpr (TENSOR) {
        fill_gauss<BS>(p, lam, U[0], U[1], U[D - 1], tg);
        __syncthreads();
    }
    const size_t fb = (size_t)i * NC * nv;
#pragma unroll 4
    for (int k0 = 2 * tid; k0 < nv; k0 += 2 * BS) {
        VelPair<D, TENSOR> vp;
        vp.load(p, k0, nv, aligned);
        double v[NC][2];
#pragma unroll
        for (int c = 0; c < NC; ++c) load_pair<FT>(f + fb + (size_t)c * nv, k0, nv, aligned, v[c][0], v[c][1]);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            double c3[D], c2, fp[2];
            const double H = pref * vp.gauss_of(e, tg, U, lam, c3, c2);
            shakhov_at<D>(c3, c2, lam, shk, q1, bh, H, fp[0], fp[1]);
#pragma unroll
            for (int c = 0; c < NC; ++c) v[c][e] = (v[c][e] + a1 * fp[c]) * inv1;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
            store_pair<FT>(f + fb + (size_t)c * nv, k0, nv, aligned, from_f64<FT>(v[c][0]), from_f64<FT>(v[c][1]));
    }
}

// ------------------------------------------------------------------------
// push sweep launches: the stage-1 base (when stale), the wall cells, one
// launch per colour (split over velocities when small), the final kernel
// ------------------------------------------------------------------------
// The form of the per-cell kernels for a velocity count: workgroup size and
// pairs per thread of FP64 sums.  Larger slabs take more threads rather than more pairs a
// thread: at 4,548 velocities 5 pairs in 512 threads 3.27 ms, 10 in 256 3.32,
// 20 in 128 3.72 (107,118 cells, FP64, before the points came from LDS), and
// held to more waves a SIMD than its 117 registers allow it spills (4.8-6.7).
// Above 5,120 velocities 1,024 threads take three, five or eight pairs: with
// eight alone, 5,200 velocities in 2D left five of them empty and spilled (a
// step of 12,800 cells 2.31 -> 2.05 ms; 2,744 cells x 9,000 in 3D 0.90 -> 0.87).
template <int D, typename FT, bool TENSOR, int BS>
void launch_base_form(const Params &p, const FT *f, typename AccOf<FT>::T *acc, hipStream_t s)
{
    const size_t lds = sizeof(double) * ((TENSOR ? 2 * (size_t)p.ntab : 0) + (BS / 64) * (D + 2));
    hipLaunchKernelGGL((k_push_base<D, FT, TENSOR, BS>), cell_grid(p.nc, BS), dim3(BS), lds, s, p, f, acc);
}
// Threads of a workgroup with FP32 stage-1 sums: one, two or four wavefronts by
// the velocities, and up to eight on meshes with too few cells to fill the chip
// so (steps with 64, 128, 256 and 512 threads, in us: 19,683 cells in 3D x 1,331
// 674, 686, 718, -; 7,200 in 2D x 400 98, 101, 109, 132; x 1,331 284, 279, 282,
// 302; x 3,501 783, 736, 742, 759; x 6,000 1,119, 1,093, 1,043, 1,059; 512 in 3D
// x 2,145 91, 84, 80, 79; 1,331 x 400 61, 60, 60, 66).  Long tables: at least
// four, so that the LDS leaves room for sixteen wavefronts a CU.
inline int stream_threads(const Params &p)
{
    int t = p.nv <= 1024 || (p.nv <= 2560 && p.nc >= 10240) ? 64 : (p.nv <= 5120 ? 128 : 256);
    while (t < 512 && (long)p.nc * t < 160 * 1024 && 2 * t < p.nv) t *= 2;
    return p.ntab > 256 ? std::max(t, 256) : t;
}

template <int D, typename FT, bool TENSOR>
void launch_base(const Params &p, const FT *f, typename AccOf<FT>::T *acc, hipStream_t s)
{
    if constexpr (sizeof(typename AccOf<FT>::T) == 4) {
        const int t = stream_threads(p);
        if (t == 64) launch_base_form<D, FT, TENSOR, 64>(p, f, acc, s);
        else if (t == 128) launch_base_form<D, FT, TENSOR, 128>(p, f, acc, s);
        else if (t == 256) launch_base_form<D, FT, TENSOR, 256>(p, f, acc, s);
        else launch_base_form<D, FT, TENSOR, 512>(p, f, acc, s);
    } else if (p.nv <= 1536) launch_base_form<D, FT, TENSOR, 256>(p, f, acc, s);
    else if (p.nv <= 5120) launch_base_form<D, FT, TENSOR, 512>(p, f, acc, s);
    else launch_base_form<D, FT, TENSOR, 1024>(p, f, acc, s);
}
template <int D, typename FT, bool TENSOR, int BS, int NP>
void launch_final_form(const Params &p, FT *f, typename AccOf<FT>::T *acc, hipStream_t s)
{
    const size_t lds = sizeof(double) * ((TENSOR ? 3 * (size_t)p.ntab : 0) + (BS / 64) * Shift<D>::N + 4 + 2 * D);
    hipLaunchKernelGGL((k_push_final<D, FT, TENSOR, BS, NP>), cell_grid(p.nc, BS), dim3(BS), lds, s, p, f, acc);
}
template <int D, typename FT, bool TENSOR>
void launch_final(const Params &p, FT *f, typename AccOf<FT>::T *acc, hipStream_t s)
{
    if constexpr (sizeof(typename AccOf<FT>::T) == 4) {
        const int t = stream_threads(p);
        if (t == 64) launch_final_form<D, FT, TENSOR, 64, 0>(p, f, acc, s);
        else if (t == 128) launch_final_form<D, FT, TENSOR, 128, 0>(p, f, acc, s);
        else if (t == 256) launch_final_form<D, FT, TENSOR, 256, 0>(p, f, acc, s);
        else launch_final_form<D, FT, TENSOR, 512, 0>(p, f, acc, s);
    } else if (p.nv <= 1536) launch_final_form<D, FT, TENSOR, 256, 3>(p, f, acc, s);
    else if (p.nv <= 3072) launch_final_form<D, FT, TENSOR, 512, 3>(p, f, acc, s);
    else if (p.nv <= 5120) launch_final_form<D, FT, TENSOR, 512, 5>(p, f, acc, s);
    else if (p.nv <= 6144) launch_final_form<D, FT, TENSOR, 1024, 3>(p, f, acc, s);
    else if (p.nv <= 10240) launch_final_form<D, FT, TENSOR, 1024, 5>(p, f, acc, s);
    else launch_final_form<D, FT, TENSOR, 1024, 8>(p, f, acc, s);  // up to 16,384 velocities
}

// Workgroups of a brick launch that the chip holds at once.
constexpr int brick_slots(bool tab, int threads) { return 256 * (4 * (tab ? 6 : 4) / (threads / 64)); }

// The rule of brick_threads.  Bricks save adds but put the work of four cells
// into one workgroup, so they gain where a launch has workgroups enough (from
// 8,192 cells in one class, 32,768 in the coloured sweep's dozen or so) and the
// velocities fill the lanes of the width that they fill best.  The line is put
// by that share of lanes.  Steps by cells against bricks, in ms:
//   3D, one class, 35,937 cells: 0.71 / 0.75 at 400 velocities (0.78 of 512
//   lanes), 0.81 / 0.75 at 450 (0.88), 0.96 / 1.06 at 640 (0.83 of 768, one
//   iteration), 1.04 / 1.09 at 784 (0.77 of 512), 1.24 / 1.17 at 1,000,
//   1.37 / 1.40 at 1,152 (0.75 of 768), 1.43 / 1.40 at 1,200 (0.78), 1.81 /
//   1.59 at 1,331, 5.1 / 4.2 at 4,548;
//   3D in colours: 0.58 / 0.83 at 100, 1.72 / 1.77 at 1,000, 2.03 / 2.10 at
//   1,280, 2.31 / 2.22 at 1,331 (0.87), 6.1 / 5.8 at 4,548, and 107,118 cells
//   17.5 / 15.2 there;
//   2D, 33,800 cells, one class: 0.27 / 0.36 at 37, 0.59 / 0.55 at 350 (0.68),
//   0.73 / 0.61 at 512, 1.04 / 0.87 at 784, 1.90 / 1.50 at 1,331; in colours
//   0.61 / 0.63 at 300 (0.59), 0.90 / 0.80 at 512, 2.18 / 1.78 at 1,331;
//   scattered, 3D, one class: 1.09 / 1.18 at 784, 1.96 / 1.78 at 1,331; in
//   colours by cells up to 9,000 velocities (6.2 / 6.4 at 4,548); 2D 1.05 /
//   0.90 and in colours 1.26 / 1.12 at 784.
// A workgroup's tables and sums must leave room for as many workgroups a CU
// as its width allows.
int brick_threads(int dim, bool unordered, int nc, int nv, int ntab)
{
    const bool tab = ntab > 0, colours3 = dim == 3 && !unordered;
    if (nc < (unordered ? 8192 : 32768) || (colours3 && !tab)) return 0;
    const size_t mf = dim == 2 ? Dim<2>::MF : Dim<3>::MF, comp = dim == 2 ? Dim<2>::NC : Dim<3>::NC;
    auto share = [&](int w) {  // of the lanes, 0 where the LDS does not do
        const size_t lds = sizeof(double) * kBrickCells * ((mf + 1) * (size_t)ntab + comp * w);
        if (lds * (brick_slots(tab, w) / 256) > 160 * 1024) return 0.0;
        return (double)nv / ((double)w * ((nv + w - 1) / w));
    };
    const double s512 = colours3 ? 0.0 : share(512), s768 = tab ? share(768) : 0.0;
    const int w = 1.05 * s768 >= s512 ? 768 : 512;
    const bool once = nv <= w;  // one iteration
    if (once && (!tab || colours3)) return 0;
    const double least = dim == 2 ? 0.65 : !unordered ? 0.85 : once ? 0.87 : 0.775;
    return (w == 768 ? s768 : s512) >= least ? w : 0;
}

// One launch over n cells in brick order.  A class with fewer bricks than the
// chip has slots is split over velocities, down to one iteration a workgroup:
// greedy colouring leaves few bricks to the last classes (35,937 cells of a
// channel: 1,436 bricks in the largest class, 137, 70, 44, 41, 3 and 2 in the
// last six; 2,145 velocities 3.31 -> 3.27 ms a step; 107,118 x 4,548 15.26 ->
// 15.21).
template <int D, bool TENSOR, int BS>
void launch_bricks(const Params &p, const double *fin, double *acc, const int *cells, int n, hipStream_t s)
{
    const int nb = (n + kBrickCells - 1) / kBrickCells, iters = (p.nv + BS - 1) / BS;
    const int split = std::max(1, std::min(iters, (brick_slots(TENSOR, BS) + nb - 1) / nb));
    const int ks = (iters + split - 1) / split * BS;
    const size_t tables = sizeof(double) * kBrickCells * (Dim<D>::MF + 1) * (TENSOR ? p.ntab : 0);
    hipLaunchKernelGGL((k_push_brick<D, TENSOR, BS>), dim3((unsigned)sweep_grid(nb), (unsigned)((p.nv + ks - 1) / ks)),
                       dim3(BS), tables, s, p, fin, acc, cells, n, ks);
}

template <int D, typename FT, bool TENSOR>
hipError_t push_t(const Params &p, void *fv, void *av, bool need_base, const int *cells, const int *coff, int ncol,
                  int bricks, const int *wall_cells, int n_wall_cells, hipStream_t s)
{
    constexpr int MF = Dim<D>::MF, NW = D + 2, BS = 256;
    using AT = typename AccOf<FT>::T;
    const FT *fin = static_cast<const FT *>(fv);
    FT *f = static_cast<FT *>(fv);
    AT *acc = static_cast<AT *>(av);
    const size_t tab = sizeof(double) * (size_t)(MF + 1) * (TENSOR ? p.ntab : 0);
    const size_t red = sizeof(double) * ((BS / 64) * (2 * NW + 2) + MF);
    if (need_base) launch_base<D, FT, TENSOR>(p, fin, acc, s);
    if (n_wall_cells > 0)
        hipLaunchKernelGGL((k_push_wall<D, FT, BS, TENSOR>), dim3(n_wall_cells), dim3(BS), tab + red, s, p, fin,
                           wall_cells, n_wall_cells);
    for (int c = 0; c < ncol; ++c) {
        const int n = coff[c + 1] - coff[c];
        if (n <= 0) continue;
        if constexpr (sizeof(FT) == 8) {
            if (bricks) {
                if (TENSOR && bricks == 768) launch_bricks<D, TENSOR, TENSOR ? 768 : 512>(p, fin, acc, cells + coff[c], n, s);
                else launch_bricks<D, TENSOR, 512>(p, fin, acc, cells + coff[c], n, s);
                continue;
            }
        }
        const unsigned g = (unsigned)sweep_grid(n);
        const int ks = push_ksplit(n, p.nv, BS, TENSOR ? (MF + 1) * p.ntab : 0);
        const dim3 grid(g, (unsigned)((p.nv + ks - 1) / ks));
        if constexpr (TENSOR)
            hipLaunchKernelGGL((k_push_pf<D, FT, BS>), grid, dim3(BS), tab + red, s, p, fin, acc, cells + coff[c], n, 0,
                               p.nv, p.nv, ks);
        else
            hipLaunchKernelGGL((k_push<D, FT, BS, false>), grid, dim3(BS), tab + red, s, p, fin, acc, cells + coff[c],
                               n, 0, p.nv, p.nv, ks);
    }
    launch_final<D, FT, TENSOR>(p, f, acc, s);
    return hipGetLastError();
}

template <int D, typename FT>
hipError_t push_d(const Params &p, void *f, void *acc, bool need_base, const int *cells, const int *coff, int ncol,
                  int bricks, const int *wc, int nwc, hipStream_t s)
{
    return p.ntab > 0 ? push_t<D, FT, true>(p, f, acc, need_base, cells, coff, ncol, bricks, wc, nwc, s)
                      : push_t<D, FT, false>(p, f, acc, need_base, cells, coff, ncol, bricks, wc, nwc, s);
}

template <int D, typename FT, bool TENSOR>
hipError_t push_inplace_t(const Params &p, void *fv, const int *cells, const int *coff, int ncol,
                          const int *wall_cells, int n_wall_cells, hipStream_t s)
{
    constexpr int MF = Dim<D>::MF, NW = D + 2, BS = 256;
    using AT = typename AccOf<FT>::T;
    FT *f = static_cast<FT *>(fv);
    AT *ring = static_cast<AT *>(p.ring);
    const size_t tab = sizeof(double) * (size_t)(MF + 1) * (TENSOR ? p.ntab : 0);
    const size_t red = sizeof(double) * ((BS / 64) * (2 * NW + 2) + MF);
    const unsigned gc = (unsigned)sweep_grid(p.nc);
    const size_t tg = sizeof(double) * (TENSOR ? 2 * (size_t)p.ntab : 0);
    const size_t lturn = tg + sizeof(double) * (BS / 64) * (Shift<D>::N + NW), lfin = tg + sizeof(double) * (4 + 2 * D);
    if (n_wall_cells > 0)
        hipLaunchKernelGGL((k_push_wall<D, FT, BS, TENSOR>), dim3(n_wall_cells), dim3(BS), tab + red, s, p, f,
                           wall_cells, n_wall_cells);
    for (int q = 0; q < p.nchunk; ++q) {
        const int c0 = q * p.chunk, cn = std::min(p.chunk, p.nv - c0);
        // the previous chunk back into f, this chunk's base into the ring
        const int pc0 = (q - 1) * p.chunk;
        hipLaunchKernelGGL((k_push_chunk_turn<D, FT, TENSOR>), dim3(gc), dim3(BS), lturn, s, p, f, ring, pc0,
                           q > 0 ? p.chunk : 0, q - 1, c0, cn, q);
        for (int c = 0; c < ncol; ++c) {
            const int n = coff[c + 1] - coff[c];
            if (n <= 0) continue;
            const unsigned g = (unsigned)sweep_grid(n);
            const int ks = push_ksplit(n, cn, BS, TENSOR ? (MF + 1) * p.ntab : 0);
            const dim3 grid(g, (unsigned)((cn + ks - 1) / ks));
            if constexpr (TENSOR)
                hipLaunchKernelGGL((k_push_pf<D, FT, BS>), grid, dim3(BS), tab + red, s, p, f, ring, cells + coff[c], n,
                                   c0, cn, p.chunk, ks);
            else
                hipLaunchKernelGGL((k_push<D, FT, BS, false>), grid, dim3(BS), tab + red, s, p, f, ring,
                                   cells + coff[c], n, c0, cn, p.chunk, ks);
        }
    }
    {
        const int q = p.nchunk - 1, c0 = q * p.chunk;
        hipLaunchKernelGGL((k_push_chunk_turn<D, FT, TENSOR>), dim3(gc), dim3(BS), lturn, s, p, f, ring, c0,
                           p.nv - c0, q, 0, 0, -1);
    }
    hipLaunchKernelGGL((k_push_final_inplace<D, FT, TENSOR>), dim3(gc), dim3(BS), lfin, s, p, f);
    return hipGetLastError();
}

template <int D, typename FT>
hipError_t push_inplace_d(const Params &p, void *f, const int *cells, const int *coff, int ncol, const int *wc,
                          int nwc, hipStream_t s)
{
    return p.ntab > 0 ? push_inplace_t<D, FT, true>(p, f, cells, coff, ncol, wc, nwc, s)
                      : push_inplace_t<D, FT, false>(p, f, cells, coff, ncol, wc, nwc, s);
}

hipError_t launch_push_inplace(const Params &p, void *f, const int *cells, const int *coff, int ncol,
                               const int *wall_cells, int n_wall_cells, hipStream_t s)
{
    // bfloat16 f: the ring holds FP32 stage-1 sums
    if (p.dim == 2)
        return p.fstore == 2 ? push_inplace_d<2, bf16s>(p, f, cells, coff, ncol, wall_cells, n_wall_cells, s)
               : p.fstore    ? push_inplace_d<2, float>(p, f, cells, coff, ncol, wall_cells, n_wall_cells, s)
                             : push_inplace_d<2, double>(p, f, cells, coff, ncol, wall_cells, n_wall_cells, s);
    return p.fstore == 2 ? push_inplace_d<3, bf16s>(p, f, cells, coff, ncol, wall_cells, n_wall_cells, s)
           : p.fstore    ? push_inplace_d<3, float>(p, f, cells, coff, ncol, wall_cells, n_wall_cells, s)
                         : push_inplace_d<3, double>(p, f, cells, coff, ncol, wall_cells, n_wall_cells, s);
}

hipError_t launch_push_step(const Params &p, void *f, void *acc, bool need_base, const int *cells, const int *coff,
                            int ncol, int bricks, const int *wall_cells, int n_wall_cells, hipStream_t s)
{
    // bfloat16 f: acc holds FP32 stage-1 sums
    if (p.dim == 2)
        return p.fstore == 2 ? push_d<2, bf16s>(p, f, acc, need_base, cells, coff, ncol, bricks, wall_cells, n_wall_cells, s)
               : p.fstore    ? push_d<2, float>(p, f, acc, need_base, cells, coff, ncol, bricks, wall_cells, n_wall_cells, s)
                             : push_d<2, double>(p, f, acc, need_base, cells, coff, ncol, bricks, wall_cells, n_wall_cells, s);
    return p.fstore == 2 ? push_d<3, bf16s>(p, f, acc, need_base, cells, coff, ncol, bricks, wall_cells, n_wall_cells, s)
           : p.fstore    ? push_d<3, float>(p, f, acc, need_base, cells, coff, ncol, bricks, wall_cells, n_wall_cells, s)
                         : push_d<3, double>(p, f, acc, need_base, cells, coff, ncol, bricks, wall_cells, n_wall_cells, s);
}

// Surface quantities of Section 2.5 from the wall flux of the last step (per
// unit area and time), one thread per wall face: surface pressure
// p_w = F_m . n (n out of the gas), shear stress sigma_w = |F_m - p_w n|,
// heat flux q_w = the energy component, and the coefficients of
// Section 4.1: Cp = p_w / d, Ct = sigma_w / d, Ch = q_w / (d u_inf) with
// d = rho_inf u_inf^2 / 2.  out [n][6].
template <int D>
__global__ __launch_bounds__(256) void k_surface(Params p, const int *__restrict__ wall_faces,
                                                 const double *__restrict__ flux, int n, double rho_inf, double u_inf,
                                                 double *__restrict__ out)
{
    constexpr int NW = D + 2;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    const FaceGeo<D> &F = static_cast<const FaceGeo<D> *>(p.fgeo)[wall_faces[t]];
    const double *w = flux + (size_t)t * NW;
    double pw = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) pw += w[1 + d] * F.n[d];
    double s2 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const double tang = w[1 + d] - pw * F.n[d];
        s2 += tang * tang;
    }
    const double sig = sqrt(s2), qw = w[NW - 1];
    const double dyn = 0.5 * rho_inf * u_inf * u_inf;
    double *o = out + (size_t)t * 6;
    o[0] = pw;
    o[1] = sig;
    o[2] = qw;
    o[3] = pw / dyn;
    o[4] = sig / dyn;
    o[5] = qw / (dyn * u_inf);
}

hipError_t launch_surface(const Params &p, const int *faces, const double *flux, int n, double rho_inf, double u_inf,
                          double *out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const dim3 grid((n + 255) / 256);
    if (p.dim == 2) hipLaunchKernelGGL(k_surface<2>, grid, dim3(256), 0, s, p, faces, flux, n, rho_inf, u_inf, out);
    else hipLaunchKernelGGL(k_surface<3>, grid, dim3(256), 0, s, p, faces, flux, n, rho_inf, u_inf, out);
    return hipGetLastError();
}

template <int D, typename FT>
hipError_t wall_flux_d(const Params &p, const void *f, const int *faces, int n, double *out, hipStream_t s)
{
    hipLaunchKernelGGL((k_wall_flux<D, FT, 256>), dim3(n), dim3(256), 0, s, p, static_cast<const FT *>(f), faces, out);
    return hipGetLastError();
}
hipError_t launch_wall_flux(const Params &p, const void *f, const int *faces, int n, double *out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (p.dim == 2)
        return p.fstore == 2 ? wall_flux_d<2, bf16s>(p, f, faces, n, out, s)
                             : (p.fstore ? wall_flux_d<2, float>(p, f, faces, n, out, s)
                                         : wall_flux_d<2, double>(p, f, faces, n, out, s));
    return p.fstore == 2 ? wall_flux_d<3, bf16s>(p, f, faces, n, out, s)
                         : (p.fstore ? wall_flux_d<3, float>(p, f, faces, n, out, s)
                                     : wall_flux_d<3, double>(p, f, faces, n, out, s));
}

hipError_t launch_batch_prologue(const BatchItem *items, int n, const int *off_grad, int grid_grad,
                                 const int *off_face, int grid_face, int dim, hipStream_t s)
{
    if (dim == 2) {
        hipLaunchKernelGGL(k_cell_grad_batch<2>, dim3(grid_grad), dim3(kGradBlock), 0, s, items, off_grad, n);
        hipLaunchKernelGGL(k_face_eq_batch<2>, dim3(grid_face), dim3(kFaceBlock), 0, s, items, off_face, n);
    } else {
        hipLaunchKernelGGL(k_cell_grad_batch<3>, dim3(grid_grad), dim3(kGradBlock), 0, s, items, off_grad, n);
        hipLaunchKernelGGL(k_face_eq_batch<3>, dim3(grid_face), dim3(kFaceBlock), 0, s, items, off_face, n);
    }
    return hipGetLastError();
}

template <int D, typename FT, bool TENSOR>
void batch_sweep_t(const BatchItem *items, int n, const int *off, int grid, int step, bool s1l, size_t lds, hipStream_t s)
{
    if constexpr (TENSOR) {
        if (s1l) hipLaunchKernelGGL((k_sweep_batch_pf<D, FT, 256, true>), dim3(grid), dim3(256), lds, s, items, off, n, step);
        else hipLaunchKernelGGL((k_sweep_batch_pf<D, FT, 256, false>), dim3(grid), dim3(256), lds, s, items, off, n, step);
    } else {
        if (s1l) hipLaunchKernelGGL((k_sweep_batch<D, FT, 256, true>), dim3(grid), dim3(256), lds, s, items, off, n, step);
        else hipLaunchKernelGGL((k_sweep_batch<D, FT, 256, false>), dim3(grid), dim3(256), lds, s, items, off, n, step);
    }
}
template <int D, typename FT>
void batch_sweep_f(const BatchItem *items, int n, const int *off, int grid, int step, bool tensor, bool s1l, size_t lds,
                   hipStream_t s)
{
    if (tensor) batch_sweep_t<D, FT, true>(items, n, off, grid, step, s1l, lds, s);
    else batch_sweep_t<D, FT, false>(items, n, off, grid, step, s1l, lds, s);
}
template <int D>
void batch_sweep_d(const BatchItem *items, int n, const int *off, int grid, int step, int fstore, bool tensor, bool s1l,
                   size_t lds, hipStream_t s)
{
    if (fstore == 2) batch_sweep_f<D, bf16s>(items, n, off, grid, step, tensor, s1l, lds, s);
    else if (fstore == 1) batch_sweep_f<D, float>(items, n, off, grid, step, tensor, s1l, lds, s);
    else batch_sweep_f<D, double>(items, n, off, grid, step, tensor, s1l, lds, s);
}
hipError_t launch_batch_sweep(const BatchItem *items, int n, const int *off, int grid, int step, int dim, int fstore,
                              bool tensor, bool s1l, size_t lds, hipStream_t s)
{
    if (dim == 2) batch_sweep_d<2>(items, n, off, grid, step, fstore, tensor, s1l, lds, s);
    else batch_sweep_d<3>(items, n, off, grid, step, fstore, tensor, s1l, lds, s);
    return hipGetLastError();
}

hipError_t launch_batch_residual(const BatchItem *items, int n, int dim, hipStream_t s)
{
    if (dim == 2) hipLaunchKernelGGL(k_residual_batch<2>, dim3(n), dim3(256), 0, s, items);
    else hipLaunchKernelGGL(k_residual_batch<3>, dim3(n), dim3(256), 0, s, items);
    return hipGetLastError();
}

int residual_groups(int nc) { return std::max(1, std::min(kResidualGroups, (nc + 2047) / 2048)); }

// ------------------------------------------------------------------------
// Fixed device scratch of the allocation-free batched step: the batch
// descriptors and offset tables.  Each GPU holds its own copy until the
// process ends.  In host code `scratch` names a host-side stand-in, not a
// device address: the device address is looked up once per device, with that
// device current, and only that address is ever handed to copies or kernels.
// ------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t launch_residual(const Params &p, double *out, hipStream_t s)
{
    const int ng = residual_groups(p.nc), per = (p.nc + ng - 1) / ng;
    double *part = out + (p.dim + 2);
    if (p.dim == 2) {
        hipLaunchKernelGGL(k_residual_part<2>, dim3(ng), dim3(256), 0, s, p, part, per, out);
        if (ng > 1) hipLaunchKernelGGL(k_residual_final<2>, dim3(1), dim3(256), 0, s, part, ng, out);
    } else {
        hipLaunchKernelGGL(k_residual_part<3>, dim3(ng), dim3(256), 0, s, p, part, per, out);
        if (ng > 1) hipLaunchKernelGGL(k_residual_final<3>, dim3(1), dim3(256), 0, s, part, ng, out);
    }
    return hipGetLastError();
}

}  // namespace ugx

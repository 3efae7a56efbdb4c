// Three-dimensional path: the modified lattice-BGK model (Secs. 2-3) on the D3Q19 lattice
// for the flow and the temperature populations, with x, y and z each periodic or bounded by
// walls under the non-equilibrium extrapolation (Sec. 3.4).  One thread per
// node: pull streaming from the previous step's post-collision buffer, the node's
// macroscopic state, BGK collision with forcing and sources, store.  Populations are kept
// as 38 planes [q][z][y][x] (flow 0-18, temperature 19-37) in deviation form (f_0 - rho0,
// g_i - omega_i sigma T0), FP64, FP32 or FP16 (scaled by 256), with arithmetic in the storage
// precision, FP32 for FP16 (the drag solve in FP64).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <new>

#include "../../include/lbm3d.h"
#include "lbm_error.h"
#include "lbm_hostslot.h"
#include "lbm_xcd.h"

namespace lbm3 {

constexpr int NQ = 19;
// rest, the six axis directions, the twelve edge directions; opposite velocities adjacent
__device__ constexpr int CX[NQ] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
__device__ constexpr int CY[NQ] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
__device__ constexpr int CZ[NQ] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
__host__ __device__ constexpr double W(int i) { return i == 0 ? 1.0 / 3.0 : (i < 7 ? 1.0 / 18.0 : 1.0 / 36.0); }

// Per-launch constants in the arithmetic type R, computed once on the host (no division or
// conversion of launch constants is left to the node code).
template <typename R> struct C3 {
    R itf, itT, of, og;            // 1 / tau, 1 - 1 / tau
    R fF, fT;                      // 1 - 1 / (2 tau)
    R tfh;                         // tau_f - 1/2
    R sig, isig, Q, halfQ, T0, gb;
    R a[3];
    R Sden;                        // 1 / (cs^2 (A - tau_f))
    R aM0;                         // cs^2 sigma (B - tau_T)
    R sigB3;                       // sigma B / 3 (the gradient term of g^eq per 3 omega)
    R A, A15;                      // A, 1.5 A
    R eps, ieps, dlin, dquad, bM;  // the uniform porosity's coefficients
};

// 1 / tau and 1 - 1 / tau in R with it + o == 1 exactly (o = fl(1 - fl(1 / tau)),
// it = fl(1 - o); for tau > 1/2 one of the two subtractions is exact by Sterbenz's lemma,
// and then so is the other): the collision's o f + it (...) then carries the state's zeroth
// moment with the factor 1, where a rounded pair would scale the temperature deviation by
// up to 1 + 6e-8 per FP32 step.
template <typename R> inline void relax_pair(double tau, R &it, R &o)
{
    const R i0 = R(1.0 / tau);
    o = R(1) - i0;
    it = R(1) - o;
}

// Launch constants (host-computed, passed by value).
struct K3 {
    int nx, ny, nz, px, py, pz;
    long long n;
    double tau_f, tau_T, A, B, sigma, Q, eps, T0, gbeta;
    double a[3];
    double c0, c1, dlin, dquad;      // drag solve: c0, c1; force: eps nu / K, eps F_eps / sqrt(K)
    const double *eps_field;         // porosity per node, or NULL for the uniform eps
    double nuK, isqK, Feps;          // nu / K, 1 / sqrt(K), F_eps (if not from the Ergun relation)
    int ergun;
    double L, dT;                    // characteristic length and temperature difference
    // walls: 0 z = 0, 1 z = nz - 1, 2 x = 0, 3 x = nx - 1, 4 y = 0, 5 y = ny - 1
    int wkind[6];
    double wu[6][3], wT[6], wdTdn[6];
    C3<double> cd;
    C3<float> cf;
};

template <typename R> __device__ __forceinline__ const C3<R> &cst3(const K3 &K);
template <> __device__ __forceinline__ const C3<double> &cst3<double>(const K3 &K) { return K.cd; }
template <> __device__ __forceinline__ const C3<float> &cst3<float>(const K3 &K) { return K.cf; }

// FP64 reciprocal and square root for the drag solve of the FP32 and FP16 paths, whose
// results are rounded to FP32: the hardware estimates refined by Newton steps (relative
// error below 1e-13).  The FP64 path keeps IEEE division and square root.
__device__ __forceinline__ double rcp_nr(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ double sqrt_nr(double x)
{
    const double r = __builtin_amdgcn_rsq(x);
    const double s = x * r;
    return x > 0.0 ? fma(fma(-s, s, x), 0.5 * r, s) : 0.0;
}
template <typename R> __device__ __forceinline__ double drag_rcp(double x) { return rcp_nr(x); }
template <> __device__ __forceinline__ double drag_rcp<double>(double x) { return 1.0 / x; }
template <typename R> __device__ __forceinline__ double drag_sqrt(double x) { return sqrt_nr(x); }
template <> __device__ __forceinline__ double drag_sqrt<double>(double x) { return sqrt(x); }

// The walls node (x, y, z) lies on: zw in {-1, 0, 1}, xw in {-1, 2, 3}, yw in {-1, 4, 5}.
__device__ __forceinline__ void wall_of(const K3 &K, int x, int y, int z, int &xw, int &yw, int &zw)
{
    xw = K.px ? -1 : (x == 0 ? 2 : (x == K.nx - 1 ? 3 : -1));
    yw = K.py ? -1 : (y == 0 ? 4 : (y == K.ny - 1 ? 5 : -1));
    zw = K.pz ? -1 : (z == 0 ? 0 : (z == K.nz - 1 ? 1 : -1));
}

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// Porosity-dependent coefficients of one node (Sec. 2, Eq. ForceEq; Sec. 3.1 drag solve; b of
// Eq. MatrM), in R; c0 and c1 of the drag solve in FP64.
template <typename R> struct Por {
    R eps, ieps, dlin, dquad, bM;
    double c0, c1;
};

template <typename R> __device__ __forceinline__ Por<R> por_of(const K3 &K, size_t k)
{
    Por<R> e;
    if (!K.eps_field) {
        const C3<R> &c = cst3<R>(K);
        e.eps = c.eps; e.ieps = c.ieps; e.dlin = c.dlin; e.dquad = c.dquad; e.bM = c.bM;
        e.c0 = K.c0; e.c1 = K.c1;
    } else {
        const double eps = K.eps_field[k];
        const double Feps = K.ergun ? 1.75 / sqrt(150.0 * eps * eps * eps) : K.Feps;
        const double ie = 1.0 / eps;
        e.eps = R(eps);
        e.ieps = R(ie);
        e.c0 = 0.5 * (1.0 + eps * 0.5 * K.nuK);
        e.c1 = eps * 0.5 * Feps * K.isqK;
        e.dlin = R(eps * K.nuK);
        e.dquad = R(eps * Feps * K.isqK);
        e.bM = R(0.5 * (ie - K.cd.isig));   // isig = 1 / sigma, rounded once on the host
    }
    return e;
}

// Arithmetic type of a storage type: FP64 storage computes in FP64, FP32 storage in FP32
// (the drag solve in FP64 for both).  The flow populations are handled as deviations
// throughout: the rest state is f_0 = rho0 and f_i = 0 otherwise, so the moments the node
// needs (sum over i > 0, first and second moments) involve only small values, and f_0
// enters as f_0 - rho0.
template <typename S> struct Arith;
template <> struct Arith<double> { using R = double; };
template <> struct Arith<float> { using R = float; };
template <> struct Arith<__half> { using R = float; };

// Load and store of one stored deviation.  FP16 holds 256 times the deviation: the
// deviations are small, and the scale keeps them clear of FP16's subnormal range.  NT: a
// non-temporal store, for launches whose wavefronts write whole cache lines (lines_whole).
template <typename S> struct St3 {
    template <typename R> static __device__ __forceinline__ R ld(const S *p) { return R(*p); }
    template <bool NT, typename R> static __device__ __forceinline__ void st(S *p, R v)
    {
        if (NT) __builtin_nontemporal_store(S(v), p);
        else *p = S(v);
    }
};
template <> struct St3<__half> {
    template <typename R> static __device__ __forceinline__ R ld(const __half *p)
    {
        return R(__half2float(*p) * (1.0f / 256.0f));
    }
    template <bool NT, typename R> static __device__ __forceinline__ void st(__half *p, R v)
    {
        const unsigned short h = __half_as_ushort(__float2half(float(v) * 256.0f));
        unsigned short *o = reinterpret_cast<unsigned short *>(p);
        if (NT) __builtin_nontemporal_store(h, o);
        else *o = h;
    }
};

// Pre-collision populations of node (x, y, z) pulled from the post-collision buffer, in the
// deviation form they are stored in (f_0 - rho0, g_q - omega_q sigma T0).  The source node of
// direction q is (x - c_q) with periodic wrap (a walled direction never leaves the grid:
// only nodes off its walls are pulled).  Offsets within a plane of populations are 32-bit
// (the host keeps a plane below 2^31 nodes), so each load adds one offset to the plane's
// base address.
template <typename S, typename R>
__device__ __forceinline__ void pull(const S *__restrict__ src, const K3 &K, int x, int y, int z, R *f, R *g)
{
    // source column, row and plane offsets for c = 0, +1 (from x - 1) and -1 (from x + 1)
    const unsigned nx = (unsigned)K.nx, pl = (unsigned)K.nx * (unsigned)K.ny;
    const unsigned xo[3] = {(unsigned)x, (unsigned)wrap(x - 1, K.nx), (unsigned)wrap(x + 1, K.nx)};
    const unsigned yo[3] = {(unsigned)y * nx, (unsigned)wrap(y - 1, K.ny) * nx, (unsigned)wrap(y + 1, K.ny) * nx};
    const unsigned zo[3] = {(unsigned)z * pl, (unsigned)wrap(z - 1, K.nz) * pl, (unsigned)wrap(z + 1, K.nz) * pl};
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int ix = CX[q] == 0 ? 0 : (CX[q] > 0 ? 1 : 2);
        const int iy = CY[q] == 0 ? 0 : (CY[q] > 0 ? 1 : 2);
        const int iz = CZ[q] == 0 ? 0 : (CZ[q] > 0 ? 1 : 2);
        const unsigned k = zo[iz] + yo[iy] + xo[ix];
        f[q] = St3<S>::template ld<R>(src + (size_t)q * K.n + k);
        g[q] = St3<S>::template ld<R>(src + (size_t)(NQ + q) * K.n + k);
    }
}

// G and F (Eq. ForceEq) at velocity u and temperature T = T0 + Td.
template <typename R>
__device__ __forceinline__ void force(const K3 &K, const Por<R> &e, const R *u, R Td, R *F)
{
    const C3<R> &c = cst3<R>(K);
    const R um = sqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    const R dl = e.dlin + e.dquad * um;
    F[0] = e.eps * c.a[0] - dl * u[0];
    F[1] = e.eps * c.a[1] - dl * u[1];
    F[2] = e.eps * (c.a[2] + c.gb * Td) - dl * u[2];
}

// Macroscopic state; Td = T - T0; S as xx, xy, xz, yy, yz, zz.
template <typename R> struct Mac {
    R Td, T, u[3], F[3], p, S[6], gT[3];
};

// Contractions with the lattice velocities over their nonzero components only.  D3Q19 has
// no velocity component other than 0 and +-1, and q is a compile-time constant once the
// loops over directions are unrolled, so the selections fold away and no multiplication by
// 0 or 1 is left (which IEEE arithmetic would otherwise have to carry out).
// c_q . v
template <typename R> __device__ __forceinline__ R cdot(int q, const R *v)
{
    const int c[3] = {CX[q], CY[q], CZ[q]};
    R r = R(0);
    bool any = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (c[a] == 0) continue;
        const R t = c[a] > 0 ? v[a] : -v[a];
        r = any ? r + t : t;
        any = true;
    }
    return r;
}
// c_q . S . c_q for the symmetric S stored as xx, xy, xz, yy, yz, zz
template <typename R> __device__ __forceinline__ R cScq(int q, const R *S)
{
    const int c[3] = {CX[q], CY[q], CZ[q]};
    constexpr int ix[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
    R r = R(0);
    bool any = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (c[a] == 0) continue;
        r = any ? r + S[ix[a][a]] : S[ix[a][a]];
        any = true;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = a + 1; b < 3; ++b) {
            if (c[a] == 0 || c[b] == 0) continue;
            const R t = R(2) * S[ix[a][b]];
            r = c[a] * c[b] > 0 ? r + t : r - t;
        }
    return r;
}
// acc += c_q,a v (the a-th component of c_q v), only where c_q,a is not zero
template <typename R> __device__ __forceinline__ void cacc(int cq, R &acc, R v)
{
    if (cq > 0) acc += v;
    else if (cq < 0) acc -= v;
}

// State of an interior node from its populations: T (Sec. 3.2), v and u (drag solve in
// FP64, Sec. 3.1), F, p (Sec. 3.1 with omega_0 = 1/3 in the closed forms of App. A), S from
// the non-equilibrium second moment (Eq. ShearEqCom; the D3Q19 equilibrium's second moment
// is eps p I + u u / eps), grad T = <M>^-1 <N> by the Sherman-Morrison form of
// <M> = a I - b u u.  Directions come in opposite pairs (q, q + 1), q odd: the first
// moments take the pair's difference, the second moments its sum.
template <typename R>
__device__ __forceinline__ void macro3(const R *f, const R *g, const K3 &K, const Por<R> &e, Mac<R> &m)
{
    R sg = g[0], s18 = R(0), j[3] = {R(0), R(0), R(0)}, P[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
    R h[3] = {R(0), R(0), R(0)};
#pragma unroll
    for (int q = 1; q < NQ; q += 2) {
        const R sf = f[q] + f[q + 1], df = f[q] - f[q + 1];
        const R dg = g[q] - g[q + 1];
        sg += g[q] + g[q + 1];
        s18 += sf;
        cacc(CX[q], j[0], df); cacc(CY[q], j[1], df); cacc(CZ[q], j[2], df);
        cacc(CX[q], h[0], dg); cacc(CY[q], h[1], dg); cacc(CZ[q], h[2], dg);
        cacc(CX[q] * CX[q], P[0], sf); cacc(CX[q] * CY[q], P[1], sf); cacc(CX[q] * CZ[q], P[2], sf);
        cacc(CY[q] * CY[q], P[3], sf); cacc(CY[q] * CZ[q], P[4], sf); cacc(CZ[q] * CZ[q], P[5], sf);
    }
    const C3<R> &c = cst3<R>(K);
    const R eps = e.eps, ieps = e.ieps, isig = c.isig, Q = c.Q;
    m.Td = (sg + c.halfQ) * isig;      // sigma T = sum g + Q/2, the rest state sigma T0 taken out
    m.T = c.T0 + m.Td;
    const R G[3] = {c.a[0], c.a[1], c.a[2] + c.gb * m.Td};
    double v[3];
    for (int a = 0; a < 3; ++a) v[a] = double(j[a] + R(0.5) * eps * G[a]);
    const double vm = drag_sqrt<R>(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const double iden = drag_rcp<R>(e.c0 + drag_sqrt<R>(e.c0 * e.c0 + e.c1 * vm));
    for (int a = 0; a < 3; ++a) m.u[a] = R(v[a] * iden);
    force<R>(K, e, m.u, m.Td, m.F);
    const R uu = m.u[0] * m.u[0] + m.u[1] * m.u[1] + m.u[2] * m.u[2];
    const R uF = m.u[0] * m.F[0] + m.u[1] * m.F[1] + m.u[2] * m.F[2];
    // rho0 s_0 = -omega_0 |u|^2 / (2 eps cs^2) = -|u|^2 / (2 eps); tau_f F_0 = -tau_f (1 - 1/(2 tau_f)) u.F / eps
    const R s0 = R(-0.5) * uu * ieps, tF0 = -c.tfh * uF * ieps;
    m.p = R(0.5) * ieps * (s18 + tF0 + s0);            // cs^2 / (eps (1 - omega_0)) = 1 / (2 eps)
    const R ep = eps * m.p;
    const int ia[6] = {0, 0, 0, 1, 1, 2}, ib[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        const R neq = P[t] - (ia[t] == ib[t] ? ep : R(0)) - m.u[ia[t]] * m.u[ib[t]] * ieps;
        m.S[t] = (neq + R(0.5) * (m.u[ia[t]] * m.F[ib[t]] + m.F[ia[t]] * m.u[ib[t]]) * ieps) * c.Sden;
    }
    R N[3];
    for (int a = 0; a < 3; ++a) N[a] = h[a] - m.T * m.u[a] + R(0.5) * (m.T * m.F[a] + m.u[a] * Q * isig);
    const R am = c.aM0 - R(0.5) * ep;
    const R bm = e.bM;
    const R uN = m.u[0] * N[0] + m.u[1] * N[1] + m.u[2] * N[2];
    const R sm = bm * uN / (am - bm * uu);
    const R iam = R(1) / am;
    for (int a = 0; a < 3; ++a) m.gT[a] = (N[a] + sm * m.u[a]) * iam;
}

// 3 omega_q for an axis and an edge direction with 2 w3a + 8 w3e = 1 exactly in R: the
// first moment of every term 3 omega_q (c_q . v) is then exactly v in the arithmetic
// itself (sum over the lattice of omega c c = cs^2 I), not only up to the rounding of the
// weights, which would scale the momentum and the heat flux by a fixed factor every step.
template <typename R> __device__ __forceinline__ R w3e() { return R(1.0 / 12.0); }
template <typename R> __device__ __forceinline__ R w3a() { return (R(1) - R(8) * w3e<R>()) * R(0.5); }
template <typename R> __device__ __forceinline__ R w3(int q) { return q < 7 ? w3a<R>() : w3e<R>(); }

// Equilibria (Eqs. EQFIN, EQTSHIN, TeEDFEQ) of direction q for pressure term ep = eps p;
// the flow equilibrium as a deviation (f_0^eq - rho0 for q = 0).  Used by the boundary
// scheme and the initialisation; the collision below evaluates the same terms pairwise.
// The contractions of one direction: its weight, 3 omega_q, c.u and c.S.c (0 at rest).
template <typename R>
__device__ __forceinline__ R feq_of(bool rest, R w, R w3q, R cu, R cSc, const K3 &K, const Por<R> &e, R ep, const R *u,
                                    const R *S)
{
    const R uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const R trS = S[0] + S[3] + S[5];
    const R base = rest ? R(-2) * ep : R(3) * w * ep;      // -(1 - omega_0) eps p / cs^2; omega_q eps p / cs^2
    return base + (rest ? R(0) : w3q * cu) + w * R(4.5) * (cu * cu - uu * R(1.0 / 3.0)) * e.ieps
         + w * cst3<R>(K).A15 * (cSc - trS * R(1.0 / 3.0));
}
template <typename R>
__device__ __forceinline__ R feq(int q, const K3 &K, const Por<R> &e, R ep, const R *u, const R *S)
{
    return feq_of<R>(q == 0, R(W(q)), w3<R>(q), cdot<R>(q, u), cScq<R>(q, S), K, e, ep, u, S);
}

// The temperature equilibrium as a deviation, g^eq_q - omega_q sigma T0, for T = T0 + Td.
template <typename R>
__device__ __forceinline__ R geq_of(bool rest, R w, R w3q, R cu, R cg, const K3 &K, const Por<R> &e, R Td, R T, R ep,
                                    const R *u)
{
    const R uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const R pres = rest ? R(-2) * T * ep : R(3) * w * T * ep;   // varpi_q T eps p / (cs^2 rho0)
    return w * (cst3<R>(K).sig * Td + T * R(4.5) * (cu * cu - uu * R(1.0 / 3.0)) * e.ieps) + pres
         + (rest ? R(0) : w3q * (T * cu + cst3<R>(K).sigB3 * cg));
}
template <typename R>
__device__ __forceinline__ R geq(int q, const K3 &K, const Por<R> &e, R Td, R T, R ep, const R *u, const R *gT)
{
    return geq_of<R>(q == 0, R(W(q)), w3<R>(q), cdot<R>(q, u), cdot<R>(q, gT), K, e, Td, T, ep, u);
}

// BGK collision with forcing and sources (Eqs. LBEeq, FtermF, TEqColli, Eq:Tforce),
//   f* = f - (f - f^eq) / tau_f + F_q,   g* = g - (g - g^eq) / tau_T + P_q + Q_q.
// Opposite directions (q, q + 1) are updated together from the parts of every term that are
// even and odd in c (as in two dimensions):
//   f*_q = (1 - 1/tau_f) f_q + Ae + Ao,   f*_q+1 = (1 - 1/tau_f) f_q+1 + Ae - Ao,
// Ae = omega [(b0 + 4.5 (c.u)^2 / eps + 1.5 A c.S.c) / tau_f + fF (9 (c.u)(c.F) - 3 u.F) / eps],
// Ao = 3 omega [(c.u) / tau_f + fF c.F], and for the temperature
// Ge = omega [(b1 + 4.5 T (c.u)^2 / eps) / tau_T + fT Q] (b1 with sigma (T - T0): the
// populations are deviations from omega sigma T0),
// Go = 3 omega [s (c.u) + sigma B c.grad T / (3 tau_T) + fT c.(T F + eps p grad T / rho0)].
// The rest direction takes what the other 18 leave of the zeroth moments the moment lists
// fix (App. A; Sec. 3.2): sum_q (f^eq_q / tau_f + F_q) = rho0 / tau_f and
// sum_q (g^eq_q / tau_T + P_q + Q_q) = sigma T / tau_T + (1 - 1/(2 tau_T)) Q, i.e. 0 and
// sigma (T - T0) / tau_T + (1 - 1/(2 tau_T)) Q for the deviations, so that mass and thermal
// energy are conserved by the arithmetic, not only up to the rounding of the lattice
// weights (in FP32 that rounding biases the heat balance by about 1e-8 sigma T / tau_T per
// step).
template <typename R> struct Coll {
    R b0, k45, c9, m3b5, b1, T45, sc, bsg, V[3], Ef, Eg;
};

// The per-node coefficients.
template <typename R>
__device__ __forceinline__ Coll<R> coll_of(const Mac<R> &m, const K3 &K, const Por<R> &e)
{
    const C3<R> &c = cst3<R>(K);
    const R ep = e.eps * m.p, ieps = e.ieps;
    const R uu = m.u[0] * m.u[0] + m.u[1] * m.u[1] + m.u[2] * m.u[2];
    const R uF = m.u[0] * m.F[0] + m.u[1] * m.F[1] + m.u[2] * m.F[2];
    const R ugT = m.u[0] * m.gT[0] + m.u[1] * m.gT[1] + m.u[2] * m.gT[2];
    const R trS = m.S[0] + m.S[3] + m.S[5];
    Coll<R> t;
    t.V[0] = m.T * m.F[0] + ep * m.gT[0];
    t.V[1] = m.T * m.F[1] + ep * m.gT[1];
    t.V[2] = m.T * m.F[2] + ep * m.gT[2];
    t.b0 = R(3) * ep - R(1.5) * uu * ieps - R(0.5) * c.A * trS;
    t.k45 = R(4.5) * ieps;
    t.c9 = R(9) * c.fF * ieps;
    t.m3b5 = R(-3) * (c.fF * uF * ieps);
    t.b1 = c.sig * m.Td - R(1.5) * m.T * uu * ieps + R(3) * m.T * ep;
    t.T45 = t.k45 * m.T;
    t.sc = c.itT * m.T + c.fT * ((ieps - c.isig) * ugT + c.Q * c.isig);
    t.bsg = c.itT * c.sigB3;
    t.Ef = t.Eg = R(0);
    return t;
}

// One pair of opposite directions, from the first one's contractions c.u, c.F, c.V, c.grad T
// and c.S.c; Ae and Ge are the even parts.
template <typename R>
__device__ __forceinline__ void collide_of(R w, R w3q, R cu, R cF, R cV, R cg, R cSc, const K3 &K, const Coll<R> &t,
                                           R *f, R *g, R &Ae, R &Ge)
{
    const C3<R> &c = cst3<R>(K);
    const R cu2 = cu * cu;
    Ae = w * (c.itf * (c.A15 * cSc + (t.k45 * cu2 + t.b0)) + (t.c9 * (cu * cF) + t.m3b5));
    const R Ao = w3q * (c.itf * cu + c.fF * cF);
    Ge = w * (c.itT * (t.T45 * cu2 + t.b1) + c.fT * c.Q);
    const R Go = w3q * (t.sc * cu + (t.bsg * cg + c.fT * cV));
    f[0] = c.of * f[0] + (Ae + Ao);
    f[1] = c.of * f[1] + (Ae - Ao);
    g[0] = c.og * g[0] + (Ge + Go);
    g[1] = c.og * g[1] + (Ge - Go);
}

// Directions q and q + 1 (q odd).
template <typename R>
__device__ __forceinline__ void collide_pair(int q, R *f, R *g, const Mac<R> &m, const K3 &K, Coll<R> &t)
{
    R Ae, Ge;
    collide_of<R>(R(W(q)), w3<R>(q), cdot<R>(q, m.u), cdot<R>(q, m.F), cdot<R>(q, t.V), cdot<R>(q, m.gT),
                  cScq<R>(q, m.S), K, t, f + q, g + q, Ae, Ge);
    t.Ef += Ae;
    t.Eg += Ge;
}

template <typename R>
__device__ __forceinline__ void collide_rest(R *f, R *g, const Mac<R> &m, const K3 &K, const Coll<R> &t)
{
    const C3<R> &c = cst3<R>(K);
    f[0] = c.of * f[0] - R(2) * t.Ef;
    g[0] = c.og * g[0] + (c.sig * m.Td * c.itT + c.fT * c.Q - R(2) * t.Eg);
}

// The boundary scheme, the non-equilibrium extrapolation from the next node inward x_f (and T
// of x_ff on prescribed-gradient walls), whose state is the one the scheme assigns (T_b, u_b, p
// and S of x_f, the boundary grad T).  On an edge or a vertex where two or three walls meet,
// x_f is the inward diagonal neighbour, the wall is at rest, an isothermal wall's temperature
// wins over a prescribed gradient (among isothermal walls x first, then y, then z), and each
// prescribed gradient sets its own normal component of grad T, as at the corners in two
// dimensions.
// The walls of a node, the step towards x_f, and the isothermal wall that gives T (or -1).
struct Wall3 { int xw, yw, zw, dx, dy, dz, iso; };

__device__ __forceinline__ Wall3 wall3(const K3 &K, int x, int y, int z)
{
    Wall3 w;
    wall_of(K, x, y, z, w.xw, w.yw, w.zw);
    w.dx = w.xw == 2 ? 1 : (w.xw == 3 ? -1 : 0);
    w.dy = w.yw == 4 ? 1 : (w.yw == 5 ? -1 : 0);
    w.dz = w.zw == 0 ? 1 : (w.zw == 1 ? -1 : 0);
    w.iso = (w.xw >= 0 && K.wkind[w.xw] == 0) ? w.xw
          : ((w.yw >= 0 && K.wkind[w.yw] == 0) ? w.yw : ((w.zw >= 0 && K.wkind[w.zw] == 0) ? w.zw : -1));
    return w;
}

// T - T0 of a node from its temperature populations.
template <typename S, typename R>
__device__ __forceinline__ R pull_Td(const S *__restrict__ src, const K3 &K, int x, int y, int z)
{
    R f[NQ], g[NQ];
    pull<S, R>(src, K, x, y, z, f, g);
    R sg = R(0);
#pragma unroll
    for (int q = 0; q < NQ; ++q) sg += g[q];
    return (sg + cst3<R>(K).halfQ) * cst3<R>(K).isig;
}

// State of a wall node from x_f's and, off the isothermal walls, T - T0 of x_ff.
template <typename R>
__device__ __forceinline__ void wall_mac(const K3 &K, const Wall3 &w, const Por<R> &e, const Mac<R> &mf, R Tdff, Mac<R> &m)
{
    R Tdb, gb[3] = {mf.gT[0], mf.gT[1], mf.gT[2]};
    if (w.iso >= 0) {
        Tdb = R(K.wT[w.iso] - K.T0);
    } else {
        if (w.xw >= 0) gb[0] = R(w.dx * K.wdTdn[w.xw]);
        if (w.yw >= 0) gb[1] = R(w.dy * K.wdTdn[w.yw]);
        if (w.zw >= 0) gb[2] = R(w.dz * K.wdTdn[w.zw]);
        Tdb = (R(4) * mf.Td - Tdff - R(2) * (R(w.dx) * gb[0] + R(w.dy) * gb[1] + R(w.dz) * gb[2])) * R(1.0 / 3.0);
    }
    m.Td = Tdb;
    m.T = cst3<R>(K).T0 + Tdb;
    const int nwall = (w.xw >= 0) + (w.yw >= 0) + (w.zw >= 0);
    const int wu = nwall > 1 ? -1 : (w.xw >= 0 ? w.xw : (w.yw >= 0 ? w.yw : w.zw));   // an edge or a vertex is at rest
    for (int a = 0; a < 3; ++a) { m.u[a] = wu < 0 ? R(0) : R(K.wu[wu][a]); m.gT[a] = gb[a]; }
    force<R>(K, e, m.u, m.Td, m.F);
    m.p = mf.p;
    for (int c = 0; c < 6; ++c) m.S[c] = mf.S[c];
}

// Populations q of a wall node in place of x_f's.
template <typename R>
__device__ __forceinline__ void wall_pop(int q, const K3 &K, const Por<R> &e, const Mac<R> &m, const Por<R> &ef,
                                         const Mac<R> &mf, R *f, R *g)
{
    const R epb = e.eps * mf.p, epf = ef.eps * mf.p;   // the wall node's porosity, x_f's pressure
    f[q] = feq<R>(q, K, e, epb, m.u, mf.S) + (f[q] - feq<R>(q, K, ef, epf, mf.u, mf.S));
    g[q] = geq<R>(q, K, e, m.Td, m.T, epb, m.u, m.gT) + (g[q] - geq<R>(q, K, ef, mf.Td, mf.T, epf, mf.u, mf.gT));
}

// Pre-collision populations and state of node (x, y, z).  Interior: pulled populations
// and their moments.  Wall node: the boundary scheme.
template <typename S, typename R>
__device__ __forceinline__ void node_state(const S *__restrict__ src, const K3 &K, int x, int y, int z,
                                           R *f, R *g, Mac<R> &m, Por<R> &e)
{
    const long long plane = (long long)K.nx * K.ny, k = z * plane + (long long)y * K.nx + x;
    e = por_of<R>(K, (size_t)k);
    const Wall3 w = wall3(K, x, y, z);
    pull<S, R>(src, K, x + w.dx, y + w.dy, z + w.dz, f, g);
    if (w.xw < 0 && w.yw < 0 && w.zw < 0) {
        macro3<R>(f, g, K, e, m);
        return;
    }
    R Tdff = R(0);
    if (w.iso < 0) Tdff = pull_Td<S, R>(src, K, x + 2 * w.dx, y + 2 * w.dy, z + 2 * w.dz);
    const Por<R> ef = por_of<R>(K, (size_t)(k + w.dz * plane + w.dy * (long long)K.nx + w.dx));
    Mac<R> mf;
    macro3<R>(f, g, K, ef, mf);
    wall_mac<R>(K, w, e, mf, Tdff, m);
#pragma unroll
    for (int q = 0; q < NQ; ++q) wall_pop<R>(q, K, e, m, ef, mf, f, g);
}

__device__ __forceinline__ bool node_xyz(const K3 &K, int &x, int &y, int &z)
{
    const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K.n) return false;
    x = (int)(k % K.nx);
    y = (int)((k / K.nx) % K.ny);
    z = (int)(k / ((long long)K.nx * K.ny));
    return true;
}

// Post-collision populations (deviations) into the buffer.
template <typename S, bool NT, typename R>
__device__ __forceinline__ void store(S *__restrict__ dst, const K3 &K, unsigned k, const R *f, const R *g)
{
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        St3<S>::template st<NT, R>(dst + (size_t)q * K.n + k, f[q]);
        St3<S>::template st<NT, R>(dst + (size_t)(NQ + q) * K.n + k, g[q]);
    }
}

constexpr int B3 = 256;
constexpr unsigned SLAB_NODES = 2048;      // interior nodes of a slab, at least (whole planes)

// Extent of the interior along x, y and z: all nodes of a periodic direction, all but the two
// wall nodes of a walled one.
__host__ __device__ __forceinline__ int inner_x(const K3 &K) { return K.px ? K.nx : K.nx - 2; }
__host__ __device__ __forceinline__ int inner_y(const K3 &K) { return K.py ? K.ny : K.ny - 2; }
__host__ __device__ __forceinline__ int inner_z(const K3 &K) { return K.pz ? K.nz : K.nz - 2; }

// How one launch shares out a step: slabs of `planes` interior planes; a slab's first nbw
// blocks take the wall nodes of its planes (`walls` each) and its share (zw nodes) of the two z
// walls, the next nbi its interior nodes.
// The wall nodes x = 0 and x = nx - 1 off the edges are left to the interior blocks that hold
// their x_f (XW) where a row has XW_ROW interior nodes or more.  In wall blocks their lanes lie
// a row apart, so that each load instruction touches 64 lines for one value each.  Time of a
// step with the x walls in wall blocks and inside: 120 x 4 x 120 FP64 16.3 and 11.8 us,
// 121 x 95 x 83 with porosity per node 186 and 162 (FP64), 95 and 73 (FP32), 54 and 48 (FP16);
// 10 x 180 x 60, the shortest such row, 29.0 and 22.6 (FP64), 17.6 and 14.3 (FP32).  In FP16 rows of
// 8 to 10 are faster with them in wall blocks, 10 x 40 x 40 9.3 and 10.8, 12 x 40 x 200 11.9 and 14.2, rows of 14
// are not: 14 x 180 x 60 14.2 and 14.1, 16 x 40 x 40 12.2 and 9.4.  Below XW_ROW a block would hold more than
// 68 such nodes.
constexpr int XW_ROW = 8, XW_ROW_F16 = 14;
// FP16 grids of whole cache lines have all wall blocks ahead of the first slab instead (`lead`): layers
// 192 x 192 x 96 107.5 us a step, spread over the slabs 108.7, 64 x 64 x 96 with porosity per node 16.8 and 17.3,
// with y walls 128 x 100 x 30 16.4 and 18.9, with y walls alone 128 x 128 x 64 36.9 and 41.9; FP32 grids where
// the y walls are the only ones: 128 x 128 x 64 62.4 and 66.6, 128 x 12 x 200 20.4 and 21.6.  FP32 layers and FP64
// grids are not (192 x 100 x 50 57.3 and 56.7; FP64 with y walls 110 and 108).
struct Slabs {
    unsigned planes, count;
    unsigned inner, walls, zw;     // interior and wall nodes per plane, z wall nodes per slab
    unsigned nbw, nbi;
    unsigned lead;
};

// What an interior node hands over to the wall node next to it: x_f's pre-collision
// populations, its state, T - T0 of x_ff, its porosity; [value][slot], two slots per row.
constexpr int XW_SLOTS = 2 * (B3 / XW_ROW + 2), XW_VALS = 2 * NQ + 18;
template <typename R> struct XWall {
    R v[XW_VALS][XW_SLOTS];
    R Ae[NQ / 2][XW_SLOTS], Ge[NQ / 2][XW_SLOTS];
};

// Components of the first direction of pair j (q = 2 j + 1) plus 1, two bits per pair.
constexpr unsigned pair_code(int axis)
{
    unsigned r = 0;
    for (int j = 0; j < NQ / 2; ++j) {
        const int q = 2 * j + 1, c = axis == 0 ? CX[q] : (axis == 1 ? CY[q] : CZ[q]);
        r |= (unsigned)(c + 1) << (2 * j);
    }
    return r | 1u << (2 * (NQ / 2));     // the rest direction, j = 9
}

// Wall node in slot s, its directions shared out over ten lanes: lane j < 9 extrapolates and
// collides pair j, lane 9 the rest direction, after all even parts are there.  The
// contractions are sums of the same terms in the same order as for compile-time directions
// (products by 0 and +-1 are exact).
template <typename S, typename R>
__device__ __forceinline__ void x_wall_pair(S *__restrict__ dst, const K3 &K, XWall<R> &sh, bool on, int s, int j,
                                            int x, int y, int z)
{
    const unsigned k = ((unsigned)z * (unsigned)K.ny + (unsigned)y) * (unsigned)K.nx + (unsigned)x;
    Mac<R> mf, m;
    Por<R> e, ef;
    Coll<R> t;
    R f[2], g[2];
    const bool rest = j == NQ / 2;
    const int q = rest ? 0 : 2 * j + 1;
    if (on) {
        mf.Td = sh.v[2 * NQ][s];
        mf.T = sh.v[2 * NQ + 1][s];
        for (int a = 0; a < 3; ++a) { mf.u[a] = sh.v[2 * NQ + 2 + a][s]; mf.gT[a] = sh.v[2 * NQ + 5 + a][s]; }
        for (int a = 0; a < 6; ++a) mf.S[a] = sh.v[2 * NQ + 8 + a][s];
        mf.p = sh.v[2 * NQ + 14][s];
        ef.eps = sh.v[2 * NQ + 16][s];
        ef.ieps = sh.v[2 * NQ + 17][s];
        e = por_of<R>(K, k);
        wall_mac<R>(K, wall3(K, x, y, z), e, mf, sh.v[2 * NQ + 15][s], m);
        t = coll_of<R>(m, K, e);
        const R c[3] = {R((int)(pair_code(0) >> (2 * j) & 3) - 1), R((int)(pair_code(1) >> (2 * j) & 3) - 1),
                        R((int)(pair_code(2) >> (2 * j) & 3) - 1)};
        auto dot = [&](const R *v) { return c[0] * v[0] + c[1] * v[1] + c[2] * v[2]; };
        const R *A = mf.S;
        const R cSc = c[0] * c[0] * A[0] + c[1] * c[1] * A[3] + c[2] * c[2] * A[5] + c[0] * c[1] * (R(2) * A[1])
                    + c[0] * c[2] * (R(2) * A[2]) + c[1] * c[2] * (R(2) * A[4]);
        const R w = rest ? R(W(0)) : (q < 7 ? R(W(1)) : R(W(7))), w3q = q < 7 ? w3a<R>() : w3e<R>();
        const R epb = e.eps * mf.p, epf = ef.eps * mf.p;
        const R ub = dot(m.u), uf = dot(mf.u), gb = dot(m.gT), gf = dot(mf.gT);
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const R sg = o ? R(-1) : R(1);
            const int qo = rest ? 0 : q + o;
            f[o] = feq_of<R>(rest, w, w3q, sg * ub, cSc, K, e, epb, m.u, mf.S)
                 + (sh.v[qo][s] - feq_of<R>(rest, w, w3q, sg * uf, cSc, K, ef, epf, mf.u, mf.S));
            g[o] = geq_of<R>(rest, w, w3q, sg * ub, sg * gb, K, e, m.Td, m.T, epb, m.u)
                 + (sh.v[NQ + qo][s] - geq_of<R>(rest, w, w3q, sg * uf, sg * gf, K, ef, mf.Td, mf.T, epf, mf.u));
        }
        if (!rest) {
            collide_of<R>(w, w3q, ub, dot(m.F), dot(t.V), gb, cSc, K, t, f, g, sh.Ae[j][s], sh.Ge[j][s]);
            for (int o = 0; o < 2; ++o) {
                St3<S>::template st<false, R>(dst + (size_t)(q + o) * K.n + k, f[o]);
                St3<S>::template st<false, R>(dst + (size_t)(NQ + q + o) * K.n + k, g[o]);
            }
        }
    }
    __syncthreads();
    if (on && rest) {
        for (int i = 0; i < NQ / 2; ++i) { t.Ef += sh.Ae[i][s]; t.Eg += sh.Ge[i][s]; }
        collide_rest<R>(f, g, m, K, t);
        St3<S>::template st<false, R>(dst + k, f[0]);
        St3<S>::template st<false, R>(dst + (size_t)NQ * K.n + k, g[0]);
    }
}

// An interior block: nodes i0 + threadIdx.x of np planes from z0, numbered over the interior
// (no boundary-scheme code but for XW): pull, state, collide, store.
template <typename S, bool XW, bool NT>
__device__ __forceinline__ void k3_interior(const S *__restrict__ src, S *__restrict__ dst, const K3 &K, unsigned i0,
                                            unsigned count, int z0)
{
    using R = typename Arith<S>::R;
    const unsigned nxi = (unsigned)inner_x(K), nyi = (unsigned)inner_y(K);
    const unsigned ox = K.px ? 0 : 1, oy = K.py ? 0 : 1;
    const unsigned i = i0 + threadIdx.x, row = i / nxi;
    unsigned zi = count == nxi * nyi ? 0 : row / nyi;      // one plane: a division less, FP16 layer 116 -> 113 us
    __shared__ XWall<R> sh[1];
    if (i < count) {
        const int x = (int)(i - row * nxi + ox), y = (int)(row - zi * nyi + oy), z = z0 + (int)zi;
        const unsigned k = ((unsigned)z * (unsigned)K.ny + (unsigned)y) * (unsigned)K.nx + (unsigned)x;
        R f[NQ], g[NQ];
        Mac<R> m;
        const Por<R> e = por_of<R>(K, k);
        pull<S, R>(src, K, x, y, z, f, g);
        // FP16: all loads ahead of the first wait, the state ahead of the collision (192 x 192 x 96: 108 us a
        // step instead of 109.3, 192 x 100 x 50 35.5 instead of 36.7; FP32 195 instead of 193)
        if (sizeof(S) == 2) __builtin_amdgcn_sched_barrier(0);
        macro3<R>(f, g, K, e, m);
        if (sizeof(S) == 2) __builtin_amdgcn_sched_barrier(0);
        if (XW && (x == 1 || x == K.nx - 2)) {
            const int hi = x == 1 ? 0 : 1, s = (int)(2 * (row - i0 / nxi)) + hi;
            R(*v)[XW_SLOTS] = sh[0].v;
            for (int q = 0; q < NQ; ++q) { v[q][s] = f[q]; v[NQ + q][s] = g[q]; }
            v[2 * NQ][s] = m.Td;
            v[2 * NQ + 1][s] = m.T;
            for (int a = 0; a < 3; ++a) { v[2 * NQ + 2 + a][s] = m.u[a]; v[2 * NQ + 5 + a][s] = m.gT[a]; }
            for (int a = 0; a < 6; ++a) v[2 * NQ + 8 + a][s] = m.S[a];
            v[2 * NQ + 14][s] = m.p;
            const S *p = src;
            asm volatile("" : "+s"(p));     // its own plane addresses: kept from pull() they spill
            v[2 * NQ + 15][s] = (hi ? K.wkind[3] : K.wkind[2]) == 0 ? R(0) : pull_Td<S, R>(p, K, x + (hi ? -1 : 1), y, z);
            v[2 * NQ + 16][s] = e.eps;
            v[2 * NQ + 17][s] = e.ieps;
        }
        Coll<R> t = coll_of<R>(m, K, e);
#pragma unroll
        for (int q = 1; q < NQ; q += 2) collide_pair<R>(q, f, g, m, K, t);
        collide_rest<R>(f, g, m, K, t);
        store<S, NT, R>(dst, K, k, f, g);
    }
    if (!XW) return;
    __syncthreads();
    const unsigned row0 = i0 / nxi, end = min(i0 + B3, count);
    const unsigned slots = 2 * ((end - 1) / nxi - row0 + 1);
    for (unsigned s0 = 0; s0 < slots; s0 += B3 / 10) {
        const unsigned s = s0 + threadIdx.x / 10, r = row0 + s / 2, at = r * nxi + (s & 1 ? nxi - 1 : 0);   // its x_f
        const bool on = threadIdx.x < B3 / 10 * 10 && s < slots && at >= i0 && at < end;
        zi = count == nxi * nyi ? 0 : r / nyi;
        x_wall_pair<S, R>(dst, K, sh[0], on, (int)s, (int)(threadIdx.x % 10), s & 1 ? K.nx - 1 : 0,
                          (int)(r - zi * nyi + oy), z0 + (int)zi);
    }
}

// A wall node: as node_state, but a pair of directions is extrapolated, collided and stored
// before the next, so that nothing but x_f's populations and the two states stays in
// registers.
template <typename S, bool NT>
__device__ __forceinline__ void k3_wall_node(const S *__restrict__ src, S *__restrict__ dst, const K3 &K,
                                             int x, int y, int z)
{
    using R = typename Arith<S>::R;
    const unsigned k = ((unsigned)z * (unsigned)K.ny + (unsigned)y) * (unsigned)K.nx + (unsigned)x;
    const Wall3 w = wall3(K, x, y, z);
    const int xf = x + w.dx, yf = y + w.dy, zf = z + w.dz;
    R f[NQ], g[NQ];
    pull<S, R>(src, K, xf, yf, zf, f, g);
    R Tdff = R(0);
    if (w.iso < 0) Tdff = pull_Td<S, R>(src, K, xf + w.dx, yf + w.dy, zf + w.dz);
    const Por<R> e = por_of<R>(K, k);
    const Por<R> ef = por_of<R>(K, ((size_t)zf * K.ny + yf) * K.nx + xf);
    Mac<R> mf, m;
    macro3<R>(f, g, K, ef, mf);
    wall_mac<R>(K, w, e, mf, Tdff, m);
    Coll<R> t = coll_of<R>(m, K, e);
    auto put = [&](int q) {
        St3<S>::template st<NT, R>(dst + (size_t)q * K.n + k, f[q]);
        St3<S>::template st<NT, R>(dst + (size_t)(NQ + q) * K.n + k, g[q]);
    };
#pragma unroll
    for (int q = 1; q < NQ; q += 2) {
        wall_pop<R>(q, K, e, m, ef, mf, f, g);
        wall_pop<R>(q + 1, K, e, m, ef, mf, f, g);
        collide_pair<R>(q, f, g, m, K, t);
        put(q);
        put(q + 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    wall_pop<R>(0, K, e, m, ef, mf, f, g);
    collide_rest<R>(f, g, m, K, t);
    put(0);
}

// One time step in one launch.  Where every wavefront writes whole cache lines (NT), stores
// are non-temporal and blocks run in the dispatched order: 192 x 192 x 96 FP32 192 us a step
// (5.6 TB/s; 6 % more with plain stores, 8 % more in the order of the XCDs).  Elsewhere rows begin and
// end inside cache lines whose other part another block writes: a plain store lets the L2 join
// the two and the order of the XCDs puts neighbouring blocks on one L2, 121 x 95 x 83 with
// porosity per node 68 -> 43 us (FP16), 97 -> 73 (FP32), 178 -> 162 (FP64), 185 x 171 x 90
// periodic in x and y 268 -> 201 (FP32).
// Wavefronts per SIMD: as many as leave nothing to spill (FP64 204 registers, FP32 105); one
// more, with the wall blocks' spills, takes longer also where the step is bound by memory:
// 192 x 192 x 96 FP64 416 against 401 us, FP32 199 against 195, the FP64 box 162 against 146,
// 120 x 4 x 120 FP64 11.8 against 10.7.  FP16 runs five with 10 spilled registers: 42 us against
// 44 with four, 75 with six (21 spilled registers where the wall path is there twice, for the leading blocks).
template <typename S> struct StepWaves { static constexpr int v = sizeof(S) == 8 ? 2 : (sizeof(S) == 4 ? 4 : 5); };

template <typename S, bool XW, bool NT>
__global__ void __launch_bounds__(B3, (StepWaves<S>::v))
k3_step(const S *__restrict__ src, S *__restrict__ dst, K3 K, Slabs L)
{
    unsigned b = NT ? blockIdx.x : (unsigned)lbm::xcd_block((int)blockIdx.x, (int)gridDim.x);
    // one call of k3_wall_node for both kinds of wall blocks spills less but takes longer: 192 x 192 x 96 FP16
    // 108.0 us a step against 107.3
    if (NT && sizeof(S) <= 4) {
        if (b < L.lead) {
            // the y walls of all interior planes (2 nx nodes each), then the two z walls
            const unsigned nx = (unsigned)K.nx, ny = (unsigned)K.ny, pl = nx * ny, ys = (unsigned)inner_z(K) * L.walls;
            unsigned i = b * B3 + threadIdx.x, x, y, z;
            if (i < ys) {
                z = i / L.walls;
                i -= z * L.walls;
                z += K.pz ? 0 : 1;
                y = i < nx ? 0 : ny - 1;
                x = i < nx ? i : i - nx;
            } else {
                i -= ys;
                if (K.pz || i >= 2 * pl) return;
                z = i < pl ? 0 : (unsigned)K.nz - 1;
                i = i < pl ? i : i - pl;
                y = i / nx;
                x = i - y * nx;
            }
            k3_wall_node<S, NT>(src, dst, K, (int)x, (int)y, (int)z);
            return;
        }
        b -= L.lead;
    }
    const unsigned nb = L.nbw + L.nbi, slab = b / nb, r = b - slab * nb;
    const unsigned p0 = slab * L.planes, np = min(L.planes, (unsigned)inner_z(K) - p0);   // interior planes p0, ...
    const unsigned z0 = p0 + (K.pz ? 0 : 1);
    if (r >= L.nbw) {
        const unsigned i0 = (r - L.nbw) * B3;
        if (i0 < np * L.inner) k3_interior<S, XW, NT>(src, dst, K, i0, np * L.inner, (int)z0);
        return;
    }
    unsigned i = r * B3 + threadIdx.x;
    const unsigned nx = (unsigned)K.nx, ny = (unsigned)K.ny;
    unsigned x, y, z;
    if (i < np * L.walls) {
        // the x walls (all their rows), then the y walls' other nodes; XW: the y walls alone
        const unsigned zi = i / L.walls, xs = XW || K.px ? 0 : 2 * ny, yw = XW ? nx : (unsigned)inner_x(K);
        i -= zi * L.walls;
        z = z0 + zi;
        if (i < xs) {
            x = i < ny ? 0 : nx - 1;
            y = i < ny ? i : i - ny;
        } else {
            i -= xs;
            y = i < yw ? 0 : ny - 1;
            x = (i < yw ? i : i - yw) + (XW || K.px ? 0 : 1);
        }
    } else {
        const unsigned pl = nx * ny, zn = K.pz ? 0 : 2 * pl;
        i -= np * L.walls;
        if (i >= L.zw) return;
        i += slab * L.zw;
        if (i >= zn) return;
        z = i < pl ? 0 : (unsigned)K.nz - 1;
        i = i < pl ? i : i - pl;
        y = i / nx;
        x = i - y * nx;
    }
    k3_wall_node<S, NT>(src, dst, K, (int)x, (int)y, (int)z);
}

// Result area after the two buffers: the reduction's value and the number of its blocks that
// are done (zero between launches).
struct Result3 {
    double value;
    unsigned done;
};

// Initial post-collision populations: the equilibria of the initial fields (S = 0,
// grad T = 0, p = 0), computed in FP64.
template <typename S>
__global__ void __launch_bounds__(B3) k3_init(S *__restrict__ dst, K3 K, const double *T_init, const double *u_init, Result3 *res)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) res->done = 0;
    int x, y, z;
    if (!node_xyz(K, x, y, z)) return;
    const size_t k = ((size_t)z * K.ny + y) * K.nx + x;
    double T = K.T0;
    int xw, yw, zw;
    wall_of(K, x, y, z, xw, yw, zw);
    if (T_init) T = T_init[k];
    else if (xw >= 0 && K.wkind[xw] == 0) T = K.wT[xw];
    else if (yw >= 0 && K.wkind[yw] == 0) T = K.wT[yw];
    else if (zw >= 0 && K.wkind[zw] == 0) T = K.wT[zw];
    double u[3] = {0.0, 0.0, 0.0};
    if (u_init)
        for (int a = 0; a < 3; ++a) u[a] = u_init[(size_t)a * K.n + k];
    const double S0[6] = {0, 0, 0, 0, 0, 0}, g0[3] = {0, 0, 0};
    const Por<double> e = por_of<double>(K, k);
    double f[NQ], g[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        f[q] = feq<double>(q, K, e, 0.0, u, S0);
        g[q] = geq<double>(q, K, e, T - K.T0, T, 0.0, u, g0);
    }
    store<S, true, double>(dst, K, (unsigned)k, f, g);
}

// Fixed-order sum of one value per thread over the block, returned to thread 0.
__device__ __forceinline__ double block_sum(double v, double *part)
{
    part[threadIdx.x] = v;
    __syncthreads();
    for (int h = B3 / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
        __syncthreads();
    }
    return part[0];
}

// Average Nusselt number of wall w (0: z = 0, 1: z = nz - 1, 2: x = 0, 3: x = nx - 1,
// 4: y = 0, 5: y = ny - 1): -L dT/dn / dT (n = +z, +x or +y along the wall's axis) by the
// one-sided second-order difference at each wall node, averaged over the wall plane, as in
// two dimensions (Eq. AvNuss): a plain mean along each periodic in-plane direction, the
// trapezoid rule along each walled one.
// The work is one latency: a cell loads the 19 temperature populations of three nodes.  One
// cell per thread over as many blocks as that takes keeps every cell's loads in flight
// together: a call on the 192 x 192 wall of an FP32 layer took 391 us with one block walking
// the wall and takes 21 us, on the 95 x 83 adiabatic-edged wall of an FP16 box with porosity
// per node 670 us and 42 us.
// Each block leaves its sum in part[], the block that finishes last adds those in
// a fixed order: the FP64 result does not depend on which one that is.
template <typename S>
__global__ void __launch_bounds__(B3) k3_nusselt(const S *__restrict__ src, K3 K, int w, double *part, Result3 *res, double *out)
{
    using R = typename Arith<S>::R;
    __shared__ double sh[B3];
    __shared__ bool last;
    const int ax = w < 2 ? 2 : (w < 4 ? 0 : 1), hi = w & 1;          // normal axis, far wall
    // the in-plane axes: the first is y for x walls and x otherwise, the second y for z walls
    // and z otherwise (selected explicitly, so nothing is indexed at run time)
    const int na = ax == 0 ? K.nx : (ax == 1 ? K.ny : K.nz);
    const int n0 = ax == 0 ? K.ny : K.nx, p0 = ax == 0 ? K.py : K.px;
    const int n1 = ax == 2 ? K.ny : K.nz, p1 = ax == 2 ? K.py : K.pz;
    const unsigned c = blockIdx.x * B3 + threadIdx.x;                 // below 2^31, as the grid
    double v = 0.0;
    if (c < (unsigned)n0 * (unsigned)n1) {
        const int i1 = (int)(c / (unsigned)n0), i0 = (int)(c - (unsigned)i1 * (unsigned)n0);
        double T[3];
        for (int d = 0; d < 3; ++d) {
            const int ia = hi ? na - 1 - d : d;
            const int x = ax == 0 ? ia : i0;
            const int y = ax == 1 ? ia : (ax == 0 ? i0 : i1);
            const int z = ax == 2 ? ia : i1;
            R f[NQ], g[NQ];
            Mac<R> m;
            Por<R> p;
            node_state<S, R>(src, K, x, y, z, f, g, m, p);
            T[d] = double(m.T);
        }
        const double d1 = (-3.0 * T[0] + 4.0 * T[1] - T[2]) / 2.0;   // along the inward normal
        double wt = 1.0;
        if (!p0 && (i0 == 0 || i0 == n0 - 1)) wt *= 0.5;
        if (!p1 && (i1 == 0 || i1 == n1 - 1)) wt *= 0.5;
        v = wt * (-K.L * (hi ? -d1 : d1) / K.dT);
    }
    v = block_sum(v, sh);
    if (threadIdx.x == 0) {
        __hip_atomic_store(part + blockIdx.x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = __hip_atomic_fetch_add(&res->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    v = 0.0;
    for (unsigned b = threadIdx.x; b < gridDim.x; b += B3)
        v += __hip_atomic_load(part + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v = block_sum(v, sh);
    if (threadIdx.x == 0) {
        *out = v / (double(p0 ? n0 : n0 - 1) * double(p1 ? n1 : n1 - 1));
        res->done = 0;
    }
}

struct FieldOut3 { double *p, *u, *T, *S, *gT; };

template <typename S>
__global__ void __launch_bounds__(B3) k3_fields(const S *__restrict__ src, K3 K, FieldOut3 o)
{
    using R = typename Arith<S>::R;
    int x, y, z;
    if (!node_xyz(K, x, y, z)) return;
    R f[NQ], g[NQ];
    Mac<R> m;
    Por<R> e;
    node_state<S, R>(src, K, x, y, z, f, g, m, e);
    const size_t k = ((size_t)z * K.ny + y) * K.nx + x, n = (size_t)K.n;
    if (o.p) o.p[k] = double(m.p);
    if (o.T) o.T[k] = double(m.T);
    for (int a = 0; a < 3; ++a) {
        if (o.u) o.u[a * n + k] = double(m.u[a]);
        if (o.gT) o.gT[a * n + k] = double(m.gT[a]);
    }
    if (o.S)
        for (int c = 0; c < 6; ++c) o.S[c * n + k] = double(m.S[c]);
}

// Pre-collision populations with the rest state added back (f_0 + rho0).
template <typename S>
__global__ void __launch_bounds__(B3) k3_populations(const S *__restrict__ src, K3 K, double *fo, double *go)
{
    using R = typename Arith<S>::R;
    int x, y, z;
    if (!node_xyz(K, x, y, z)) return;
    R f[NQ], g[NQ];
    Mac<R> m;
    Por<R> e;
    node_state<S, R>(src, K, x, y, z, f, g, m, e);
    const size_t k = ((size_t)z * K.ny + y) * K.nx + x;
    for (int q = 0; q < NQ; ++q) {
        if (fo) fo[(size_t)q * K.n + k] = double(f[q]) + (q == 0 ? 1.0 : 0.0);
        if (go) go[(size_t)q * K.n + k] = double(g[q]) + W(q) * K.sigma * K.T0;
    }
}

}  // namespace lbm3

using namespace lbm3;

struct lbm3_ctx {
    K3 K;
    int storage;
    char *buf[2];
    Result3 *result;
    double *host;                  // pinned slot for the reduction's value, or NULL
    int cur;
    hipStream_t stream;
    int64_t t;
};

namespace {

lbm_status fail3(lbm_status st, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
lbm_status fail3(lbm_status st, const char *fmt, ...)
{
    char msg[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(msg, sizeof(msg), fmt, ap);
    va_end(ap);
    return lbm::set_error(st, msg);
}

size_t elem3(int storage) { return storage == LBM_F64 ? 8 : (storage == LBM_F32 ? 4 : 2); }

// Calls f with a tag naming the storage type of a context.
template <typename S> struct Tag { using type = S; };
template <typename F> void by_storage(int storage, F &&f)
{
    if (storage == LBM_F64) f(Tag<double>{});
    else if (storage == LBM_F32) f(Tag<float>{});
    else f(Tag<__half>{});
}

size_t buffer_bytes(const lbm3_params *p)
{
    const size_t n = (size_t)p->nx * p->ny * p->nz;
    return (2 * NQ * n * elem3(p->storage) + 255) / 256 * 256;
}

constexpr size_t RESULT_BYTES = 256;   // after the two buffers: the reduction's result

// Derived lattice constants, as for two dimensions (Sec. 2, Sec. 3.1, Eq. Therdiff,
// Eq. EQA&B, Eq. ForceEq with the Ergun relation).
lbm_status make_constants(const lbm3_params *p, K3 &K)
{
    if (!p) return fail3(LBM_ERR_INVALID, "params is NULL");
    if (p->nx < 1 || p->ny < 1 || p->nz < 1) return fail3(LBM_ERR_INVALID, "grid must be at least 1 x 1 x 1");
    if (!p->periodic_z && p->nz < 4) return fail3(LBM_ERR_INVALID, "walled z needs nz >= 4 (got %d)", p->nz);
    if (!p->periodic_x && p->nx < 4) return fail3(LBM_ERR_INVALID, "walled x needs nx >= 4 (got %d)", p->nx);
    if (!p->periodic_y && p->ny < 4) return fail3(LBM_ERR_INVALID, "walled y needs ny >= 4 (got %d)", p->ny);
    if (p->storage != LBM_F64 && p->storage != LBM_F32 && p->storage != LBM_F16)
        return fail3(LBM_ERR_INVALID, "storage must be LBM_F64, LBM_F32 or LBM_F16");
    if ((double)p->nx * p->ny * p->nz >= 2147483648.0 || (p->periodic_z ? p->nz : p->nz - 2) > 65535)
        return fail3(LBM_ERR_INVALID, "grid too large (at most 2^31 - 1 nodes and 65535 interior z planes)");
    if (!(p->tau_f > 0.5) || !(p->tau_T > 0.5)) return fail3(LBM_ERR_INVALID, "tau_f and tau_T must exceed 1/2");
    if (!(p->eps > 0.0) || !(p->eps <= 1.0) || !(p->sigma > 0.0) || !(p->J > 0.0))
        return fail3(LBM_ERR_INVALID, "eps must lie in (0, 1]; sigma and J must be positive");
    if (p->eps_field && ((uintptr_t)p->eps_field) % 8)
        return fail3(LBM_ERR_INVALID, "eps_field must be 8-byte aligned");
    const double L = p->L > 0 ? p->L : (!p->periodic_x ? p->nx - 1 : (p->periodic_z ? p->nz : p->nz - 1));
    double A = p->A, B = p->B;
    if (std::isnan(A) || std::isnan(B)) {
        if (!(p->Ra > 0) || !(p->Pr > 0)) return fail3(LBM_ERR_INVALID, "A, B from Ma need Ra > 0 and Pr > 0");
        A = p->tau_f - 0.5 - p->J * p->Ma * L * sqrt(3.0 * p->Pr / p->Ra);
        B = p->tau_T - 0.5 - (p->Ma / p->sigma) * L * sqrt(3.0 / (p->Pr * p->Ra));
    }
    const double nu_e = (p->tau_f - A - 0.5) / 3.0, nu = nu_e / p->J;
    const double alpha = p->sigma * (p->tau_T - B - 0.5) / 3.0;
    const double Kp = p->Da * L * L;
    if (!(nu_e > 0)) return fail3(LBM_ERR_INVALID, "nu_e <= 0 (A = %g >= tau_f - 1/2)", A);
    if (!(alpha > 0)) return fail3(LBM_ERR_INVALID, "alpha_e <= 0 (B = %g >= tau_T - 1/2)", B);
    if (!(Kp > 0)) return fail3(LBM_ERR_INVALID, "K = Da L^2 must be positive");
    const double dT = p->T_hot - p->T_cold;
    const double Feps = std::isnan(p->F_eps) ? 1.75 / sqrt(150.0 * p->eps * p->eps * p->eps) : p->F_eps;
    K.nx = p->nx; K.ny = p->ny; K.nz = p->nz; K.px = p->periodic_x ? 1 : 0; K.py = p->periodic_y ? 1 : 0; K.pz = p->periodic_z ? 1 : 0;
    K.n = (long long)p->nx * p->ny * p->nz;
    K.tau_f = p->tau_f; K.tau_T = p->tau_T; K.A = A; K.B = B; K.sigma = p->sigma; K.Q = p->Q; K.eps = p->eps;
    K.T0 = 0.5 * (p->T_hot + p->T_cold);
    K.gbeta = (p->Ra > 0 && dT != 0.0) ? p->Ra * nu * alpha / (dT * L * L * L) : 0.0;
    for (int a = 0; a < 3; ++a) K.a[a] = p->a[a];
    K.c0 = 0.5 * (1.0 + p->eps * 0.5 * nu / Kp);
    K.c1 = p->eps * 0.5 * Feps / sqrt(Kp);
    K.dlin = p->eps * nu / Kp;
    K.dquad = p->eps * Feps / sqrt(Kp);
    K.eps_field = p->eps_field;
    K.L = L;
    K.dT = dT;
    K.nuK = nu / Kp;
    K.isqK = 1.0 / sqrt(Kp);
    K.ergun = std::isnan(p->F_eps) ? 1 : 0;
    K.Feps = K.ergun ? 0.0 : p->F_eps;
    C3<double> &c = K.cd;
    relax_pair(p->tau_f, c.itf, c.of);
    relax_pair(p->tau_T, c.itT, c.og);
    c.fF = 1.0 - 0.5 / p->tau_f;
    c.fT = 1.0 - 0.5 / p->tau_T;
    c.tfh = p->tau_f - 0.5;
    c.sig = p->sigma;
    c.isig = 1.0 / p->sigma;
    c.Q = p->Q;
    c.halfQ = 0.5 * p->Q;
    c.T0 = K.T0;
    c.gb = K.gbeta;
    for (int a = 0; a < 3; ++a) c.a[a] = p->a[a];
    c.Sden = 3.0 / (A - p->tau_f);
    c.aM0 = p->sigma * (B - p->tau_T) / 3.0;
    c.sigB3 = p->sigma * B / 3.0;
    c.A = A;
    c.A15 = 1.5 * A;
    c.eps = p->eps;
    c.ieps = 1.0 / p->eps;
    c.dlin = K.dlin;
    c.dquad = K.dquad;
    c.bM = 0.5 * (1.0 / p->eps - 1.0 / p->sigma);
    C3<float> &cf = K.cf;
    relax_pair(p->tau_f, cf.itf, cf.of);
    relax_pair(p->tau_T, cf.itT, cf.og);
    cf.fF = (float)c.fF; cf.fT = (float)c.fT; cf.tfh = (float)c.tfh; cf.sig = (float)c.sig;
    cf.isig = (float)c.isig; cf.Q = (float)c.Q; cf.halfQ = (float)c.halfQ; cf.T0 = (float)c.T0;
    cf.gb = (float)c.gb;
    for (int a = 0; a < 3; ++a) cf.a[a] = (float)c.a[a];
    cf.Sden = (float)c.Sden; cf.aM0 = (float)c.aM0; cf.sigB3 = (float)c.sigB3; cf.A = (float)c.A; cf.A15 = (float)c.A15;
    cf.eps = (float)c.eps; cf.ieps = (float)c.ieps; cf.dlin = (float)c.dlin; cf.dquad = (float)c.dquad;
    cf.bM = (float)c.bM;
    for (int w = 0; w < 6; ++w) {
        K.wkind[w] = p->wall[w].t_kind == LBM_T_NEUMANN ? 1 : 0;
        for (int a = 0; a < 3; ++a) K.wu[w][a] = p->wall[w].u[a];
        K.wT[w] = p->wall[w].T;
        K.wdTdn[w] = p->wall[w].dTdn;
    }
    return LBM_OK;
}

unsigned blocks_for(long long n) { return (unsigned)((n + B3 - 1) / B3); }

// Whether the runs of consecutive interior nodes (whole planes, or whole rows between y walls)
// start and end on 128-byte lines.
template <typename S> bool lines_whole(const K3 &K)
{
    return K.px && (long long)K.nx * (K.py ? K.ny : 1) * (long long)sizeof(S) % 128 == 0;
}

template <typename S> bool x_walls_inside(const K3 &K) { return !K.px && inner_x(K) >= (sizeof(S) == 2 ? XW_ROW_F16 : XW_ROW); }

Slabs slabs_of(const K3 &K, int storage, bool whole, bool inside)
{
    Slabs L;
    const unsigned pl = (unsigned)K.nx * (unsigned)K.ny, nz = (unsigned)inner_z(K);
    L.inner = (unsigned)inner_x(K) * (unsigned)inner_y(K);
    L.walls = inside ? (K.py ? 0 : 2 * (unsigned)K.nx) : pl - L.inner;
    L.planes = std::min(nz, std::max(1u, (SLAB_NODES + L.inner - 1) / L.inner));
    L.count = (nz + L.planes - 1) / L.planes;
    const bool lead = whole && (storage == LBM_F16 || (storage == LBM_F32 && K.pz));
    L.lead = lead ? blocks_for((long long)L.walls * nz + (K.pz ? 0 : 2LL * pl)) : 0;
    L.zw = K.pz || lead ? 0 : (unsigned)((2LL * pl + L.count - 1) / L.count);
    L.nbw = lead ? 0 : blocks_for((long long)L.walls * L.planes + L.zw);
    // large layers are bound by memory: wall blocks are filled (the last slabs have no z wall nodes
    // left), 192 x 192 x 96 FP32 192 us a step instead of 193.5; on rows with x walls the grids are often
    // too small for that, 120 x 4 x 120 12.1 instead of 10.5
    if (whole && !K.pz && !lead) L.zw = L.nbw * B3 - L.walls * L.planes;
    L.nbi = blocks_for((long long)L.inner * L.planes);
    return L;
}

lbm_status launched(const char *what)
{
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? LBM_OK : fail3(LBM_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace

extern "C" {

size_t lbm3_workspace_bytes(const lbm3_params *params)
{
    K3 K;
    if (make_constants(params, K) != LBM_OK) return 0;
    return 2 * buffer_bytes(params) + RESULT_BYTES;
}

lbm_status lbm3_init(const lbm3_params *params, void *workspace, size_t workspace_bytes, void *hip_stream,
                     lbm3_ctx **out)
{
    if (!out) return fail3(LBM_ERR_INVALID, "out is NULL");
    *out = nullptr;
    K3 K;
    lbm_status st = make_constants(params, K);
    if (st != LBM_OK) return st;
    if (!workspace || ((uintptr_t)workspace) % 256) return fail3(LBM_ERR_INVALID, "workspace must be non-NULL and 256-byte aligned");
    const size_t need = 2 * buffer_bytes(params) + RESULT_BYTES;
    if (workspace_bytes < need) return fail3(LBM_ERR_INVALID, "workspace too small: %zu < %zu bytes", workspace_bytes, need);
    lbm3_ctx *c = new (std::nothrow) lbm3_ctx;
    if (!c) return fail3(LBM_ERR_DEVICE, "out of host memory");
    c->K = K;
    c->storage = params->storage;
    c->buf[0] = static_cast<char *>(workspace);
    c->buf[1] = c->buf[0] + buffer_bytes(params);
    c->result = reinterpret_cast<Result3 *>(c->buf[1] + buffer_bytes(params));
    c->cur = 0;
    c->stream = static_cast<hipStream_t>(hip_stream);
    c->t = 0;
    by_storage(c->storage, [&](auto t) {
        using S = typename decltype(t)::type;
        hipLaunchKernelGGL((k3_init<S>), dim3(blocks_for(K.n)), dim3(B3), 0, c->stream,
                           reinterpret_cast<S *>(c->buf[0]), K, params->T_init, params->u_init, c->result);
    });
    st = launched("initial populations");
    if (st == LBM_OK) {
        const hipError_t e = hipStreamSynchronize(c->stream);
        if (e != hipSuccess) st = fail3(LBM_ERR_DEVICE, "initial populations: %s", hipGetErrorString(e));
    }
    if (st != LBM_OK) { delete c; return st; }
    c->host = lbm::host_slot_take();
    *out = c;
    return LBM_OK;
}

lbm_status lbm3_step(lbm3_ctx *c, int64_t nsteps)
{
    if (!c) return fail3(LBM_ERR_INVALID, "ctx is NULL");
    if (nsteps < 0) return fail3(LBM_ERR_INVALID, "nsteps must be >= 0");
    bool whole = false, inside = false;
    by_storage(c->storage, [&](auto t) {
        whole = lines_whole<typename decltype(t)::type>(c->K);
        inside = x_walls_inside<typename decltype(t)::type>(c->K);
    });
    const Slabs L = slabs_of(c->K, c->storage, whole, inside);
    const unsigned nb = L.lead + L.count * (L.nbw + L.nbi);
    for (int64_t s = 0; s < nsteps; ++s) {
        by_storage(c->storage, [&](auto t) {
            using S = typename decltype(t)::type;
            const S *src = reinterpret_cast<const S *>(c->buf[c->cur]);
            S *dst = reinterpret_cast<S *>(c->buf[c->cur ^ 1]);
            const auto k = inside ? &k3_step<S, true, false>
                         : (whole ? &k3_step<S, false, true> : &k3_step<S, false, false>);
            hipLaunchKernelGGL(k, dim3(nb), dim3(B3), 0, c->stream, src, dst, c->K, L);
        });
        c->cur ^= 1;
        c->t += 1;
    }
    return launched("3-D step");
}

lbm_status lbm3_fields(lbm3_ctx *c, double *p, double *u, double *T, double *S, double *gradT)
{
    if (!c) return fail3(LBM_ERR_INVALID, "ctx is NULL");
    const FieldOut3 o{p, u, T, S, gradT};
    by_storage(c->storage, [&](auto t) {
        using S = typename decltype(t)::type;
        hipLaunchKernelGGL((k3_fields<S>), dim3(blocks_for(c->K.n)), dim3(B3), 0, c->stream,
                           reinterpret_cast<const S *>(c->buf[c->cur]), c->K, o);
    });
    return launched("3-D fields");
}

lbm_status lbm3_populations(lbm3_ctx *c, double *f, double *g)
{
    if (!c) return fail3(LBM_ERR_INVALID, "ctx is NULL");
    by_storage(c->storage, [&](auto t) {
        using S = typename decltype(t)::type;
        hipLaunchKernelGGL((k3_populations<S>), dim3(blocks_for(c->K.n)), dim3(B3), 0, c->stream,
                           reinterpret_cast<const S *>(c->buf[c->cur]), c->K, f, g);
    });
    return launched("3-D populations");
}

lbm_status lbm3_nusselt(lbm3_ctx *c, int32_t wall, double *nu_host)
{
    if (!c || !nu_host) return fail3(LBM_ERR_INVALID, "ctx and nu_host must be non-NULL");
    if (wall < 0 || wall > 5)
        return fail3(LBM_ERR_INVALID, "wall must be 0 (z = 0), 1 (z = nz - 1), 2 (x = 0), 3 (x = nx - 1), 4 (y = 0) or 5 (y = ny - 1)");
    if (wall < 2 ? c->K.pz : (wall < 4 ? c->K.px : c->K.py))
        return fail3(LBM_ERR_INVALID, "wall %d does not exist (periodic direction)", (int)wall);
    if (!(c->K.dT != 0.0)) return fail3(LBM_ERR_INVALID, "T_hot - T_cold is zero");
    // the block sums go to the buffer that the next step overwrites
    const K3 &K = c->K;
    const long long cells = K.n / (wall < 2 ? K.nz : (wall < 4 ? K.nx : K.ny));
    double *part = reinterpret_cast<double *>(c->buf[c->cur ^ 1]);
    double *out = c->host ? c->host : &c->result->value;
    by_storage(c->storage, [&](auto t) {
        using S = typename decltype(t)::type;
        hipLaunchKernelGGL((k3_nusselt<S>), dim3(blocks_for(cells)), dim3(B3), 0, c->stream,
                           reinterpret_cast<const S *>(c->buf[c->cur]), K, (int)wall, part, c->result, out);
    });
    lbm_status st = launched("3-D Nusselt number");
    if (st != LBM_OK) return st;
    hipError_t e = hipSuccess;
    if (!c->host) e = hipMemcpyAsync(nu_host, out, sizeof(double), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e == hipSuccess && c->host) *nu_host = *out;
    if (e != hipSuccess) return fail3(LBM_ERR_DEVICE, "3-D Nusselt number: %s", hipGetErrorString(e));
    return LBM_OK;
}

int32_t lbm3_lattice(int32_t *c)
{
    static const int32_t v[NQ][3] = {{0, 0, 0}, {1, 0, 0}, {-1, 0, 0}, {0, 1, 0}, {0, -1, 0}, {0, 0, 1}, {0, 0, -1},
                                     {1, 1, 0}, {-1, -1, 0}, {1, -1, 0}, {-1, 1, 0}, {1, 0, 1}, {-1, 0, -1},
                                     {1, 0, -1}, {-1, 0, 1}, {0, 1, 1}, {0, -1, -1}, {0, 1, -1}, {0, -1, 1}};
    if (c) memcpy(c, v, sizeof(v));
    return NQ;
}

int64_t lbm3_time(const lbm3_ctx *c) { return c ? c->t : -1; }

void lbm3_destroy(lbm3_ctx *c)
{
    if (!c) return;
    (void)hipStreamSynchronize(c->stream);
    lbm::host_slot_give(c->host);
    delete c;
}

}  // extern "C"

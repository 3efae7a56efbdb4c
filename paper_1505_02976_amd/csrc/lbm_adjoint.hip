// Discrete adjoint of the fused step: vector-Jacobian products of one time step for the
// gradient of an average Nusselt number with respect to the porosity of every node.
//
// One step maps the post-collision state s_t to s_{t+1}: node x gathers its pre-collision
// populations pre(x) (streaming; at wall nodes the boundary scheme builds them from the
// reference node x_f and, on prescribed-gradient walls, T at x_ff) and collides them,
// s_{t+1}(x) = C_x(pre(x), eps(x)).  Given lambda_{t+1} = dJ/ds_{t+1} the adjoint step forms,
// at every node z off the walls, the adjoint mu_t(z, q) of its pre-collision population q:
//   (dC_z/dpre)^T lambda_{t+1}(z), plus, from every wall node b whose reference node x_f is z,
//   the adjoint of b's update with respect to the populations of x_f, plus, from every
//   prescribed-gradient wall node whose x_ff is z, its adjoint with respect to T(x_ff).
// Streaming is transposed by the next step's pull, lambda_t(y, q) = mu_t(y + c_q, q), with
// mu = 0 at wall nodes (whose own pulled populations the boundary scheme replaces) and off
// the grid.  The porosity's adjoint of a node's update adds to its gradient; wall nodes also
// add one with respect to the porosity of x_f.
//
// Off the walls the products are reversed by hand in the storage's arithmetic type (node_vjp),
// at the wall nodes in FP64 (wall_vjp).
//
// A launch takes several adjoint steps on tiles, as the forward kernel of lbm_tile.hip does
// and for the same reason: at 256 x 256 a step's work is a few microseconds, its launches cost
// more.  mu is kept in LDS between the steps (FP64); the forward states come from memory.  The
// wall nodes of a tile's region have wavefronts of their own, so that their products run
// beside those of the other nodes instead of after them; they leave their results in LDS, and
// the threads of x_f and x_ff add them.  Region sides that come within two nodes of a wall
// are moved to the wall, because a node at x_ff needs the wall node's product at its own last
// step.
#include <cmath>

#include "lbm_tile.h"

namespace lbm {

constexpr int ADJ_NT = 512;      // threads of a block: the nodes of its region, then its wall nodes
constexpr int ADJ_WALLS = 128;   // wall nodes of a region at most

// Constants of the reverse pass that Cst does not hold.
template <typename R> struct AdjK {
    Cst<R> k;
    R T0;
    double nuK, isqK;            // nu / K, 1 / sqrt(K)
};

// Porosity of a node: coefficients, F_eps and d(eps F_eps) / d eps (Sec. 2: F_eps from the Ergun
// relation or fixed).
template <typename R> struct AdjEps {
    EpsC<R> e;
    double dEF;
};
template <typename R> __device__ __forceinline__ AdjEps<R> adj_eps(const KParams &P, double eps)
{
    AdjEps<R> a;
    a.e = eps_coeffs<R>(P, eps);
    const double Fe = P.ergun ? 1.75 / sqrt(150.0 * eps * eps * eps) : P.Feps;
    a.dEF = P.ergun ? -0.5 * Fe : Fe;
    return a;
}

// Forward state of a node from its pre-collision populations (node_macro and node_gradT), with
// the intermediate values the reverse pass uses.
template <typename R> struct FwdState {
    R Td, T, Gx, Gy, ux, uy, um, dl, Fx, Fy, uu, uF, X, p, ep, cuu, cuF;
    R qxx, qyy, qxy, Nx, Ny, uN, d, cc, ia, gx, gy;
    double vx, vy, vm, Rt, iden;
};

template <typename R>
__device__ __forceinline__ void fwd_state(const R *f, const R *g, const AdjK<R> &c, const AdjEps<R> &ae, FwdState<R> &m)
{
    const Cst<R> &k = c.k;
    const EpsC<R> &e = ae.e;
    const R sg = ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7])) + g[8];
    m.Td = (sg + k.halfQ) * k.isig;
    m.Gx = k.ax;
    m.Gy = k.ay + k.gb * m.Td;
    const R jx = (f[1] - f[3]) + (f[5] - f[6]) + (f[8] - f[7]);
    const R jy = (f[2] - f[4]) + (f[5] + f[6]) - (f[7] + f[8]);
    m.vx = double(jx) + 0.5 * e.epsd * double(m.Gx);
    m.vy = double(jy) + 0.5 * e.epsd * double(m.Gy);
    m.vm = sqrt(m.vx * m.vx + m.vy * m.vy);
    m.Rt = sqrt(e.c0 * e.c0 + e.c1 * m.vm);
    m.iden = 1.0 / (e.c0 + m.Rt);
    m.ux = R(m.vx * m.iden);
    m.uy = R(m.vy * m.iden);
    m.um = R(m.vm * m.iden);
    const R eps = e.eps, ieps = e.ieps;
    m.dl = e.dlin + e.dquad * m.um;
    m.Fx = eps * m.Gx - m.dl * m.ux;
    m.Fy = eps * m.Gy - m.dl * m.uy;
    m.uu = m.ux * m.ux + m.uy * m.uy;
    m.uF = m.ux * m.Fx + m.uy * m.Fy;
    const R s18 = ((f[1] + f[2]) + (f[3] + f[4])) + ((f[5] + f[6]) + (f[7] + f[8]));
    m.cuu = R(-2.0 / 3.0) * ieps;
    m.cuF = R(-4.0 / 3.0) * k.fF * k.tau_f * ieps;
    m.X = s18 + m.cuu * m.uu + m.cuF * m.uF;
    m.p = (R(0.6) * ieps) * m.X;
    m.ep = eps * m.p;
    m.qxx = m.ux * m.ux - m.ux * m.Fx;
    m.qyy = m.uy * m.uy - m.uy * m.Fy;
    m.qxy = m.ux * m.uy - R(0.5) * (m.ux * m.Fy + m.Fx * m.uy);
    const R hx = (g[1] - g[3]) + (g[5] - g[6]) + (g[8] - g[7]);
    const R hy = (g[2] - g[4]) + (g[5] + g[6]) - (g[7] + g[8]);
    m.T = c.T0 + m.Td;
    m.Nx = hx - m.T * m.ux + R(0.5) * (m.T * m.Fx + m.ux * k.Q * k.isig);
    m.Ny = hy - m.T * m.uy + R(0.5) * (m.T * m.Fy + m.uy * k.Q * k.isig);
    const R a = k.aM0 - R(0.5) * m.ep;
    m.uN = m.ux * m.Nx + m.uy * m.Ny;
    m.d = a - e.bM * m.uu;
    m.cc = e.bM * m.uN / m.d;
    m.ia = R(1) / a;
    m.gx = (m.Nx + m.cc * m.ux) * m.ia;
    m.gy = (m.Ny + m.cc * m.uy) * m.ia;
}

// The state a node collides with (FwdState's own off the walls, the boundary scheme's at a
// wall node; the collision is linear in S, whose value the reverse pass does not need).
template <typename R> struct ColState {
    R ux, uy, Fx, Fy, uu, uF, T, ep, gx, gy, ieps;
};

// Adjoints of a node's state: T - T0, T, u, F, p, S, grad T, eps p, |u|^2, u.F and 1 / eps, each
// counted as an argument of its own.
template <typename R> struct StateAdj {
    R Td, T, ux, uy, Fx, Fy, p, Sxx, Syy, Sxy, gx, gy, ep, uu, uF, ieps;
};

// Reverse of the collision (node_collide): adjoints lam of the post-collision populations
// (lam[q ST]: f 0-8, g 9-17) to those of the state.  The adjoints of the pre-collision
// populations at fixed state are (1 - 1/tau) lam.  Opposite directions are reversed together,
// as the collision pairs them.
template <typename R, int ST>
__device__ __forceinline__ void collide_vjp(const R *lam, const ColState<R> &s, const AdjK<R> &c, StateAdj<R> &a)
{
    const R *const lf = lam, *const lg = lam + 9 * ST;
    const Cst<R> &k = c.k;
    const R ieps = s.ieps;
    const R ugT = s.ux * s.gx + s.uy * s.gy;
    const R k45 = R(4.5) * ieps, c9 = R(9) * k.fF * ieps;
    const R T45 = k45 * s.T;
    const R sco = k.itT * s.T + k.fT * ((ieps - k.isig) * ugT + k.Q * k.isig);
    a.Td = lg[0] * k.itT * k.sig;
    a.ux = R(0); a.uy = R(0); a.Fx = R(0); a.Fy = R(0); a.Sxx = R(0); a.Syy = R(0); a.Sxy = R(0);
    a.gx = R(0); a.gy = R(0); a.p = R(0);
    R a_vx = R(0), a_vy = R(0);
    R A_k45 = R(0), A_b0 = R(0), A_c9 = R(0), A_m3b5 = R(0), A_T45 = R(0), A_b1 = R(0), A_s = R(0);
    // the four pairs (a, b) with c_b = -c_a: (1,3) (1,0); (2,4) (0,1); (5,7) (1,1); (6,8) (-1,1)
    const int pa[4] = {1, 2, 5, 6}, pb[4] = {3, 4, 7, 8};
    const int pcx[4] = {1, 0, 1, -1}, pcy[4] = {0, 1, 1, 1};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const R cx = R(pcx[t]), cy = R(pcy[t]);
        const R w = t < 2 ? k.w1 : k.w5, w3 = t < 2 ? k.w3a : k.w3d;
        const R fa = lf[pa[t] * ST], fb = lf[pb[t] * ST], ga = lg[pa[t] * ST], gb = lg[pb[t] * ST];
        const R sf = fa + fb - R(2) * lf[0], df = fa - fb;
        const R sgm = ga + gb - R(2) * lg[0], dg = ga - gb;
        const R cu = cx * s.ux + cy * s.uy, cF = cx * s.Fx + cy * s.Fy;
        const R witf = w * k.itf, witT = w * k.itT;
        const R a_cSc = sf * witf * (R(1.5) * k.A);
        const R a_cu = sf * (witf * k45 * R(2) * cu + w * c9 * cF) + df * k.itf * w3
                     + sgm * witT * T45 * R(2) * cu + dg * w3 * sco;
        const R a_cF = sf * w * c9 * cu + df * w3 * k.fF;
        const R a_cg = dg * k.itT * w * k.sigB;
        const R a_cv = dg * w3 * k.fT;
        A_k45 += sf * witf * cu * cu;
        A_b0 += sf * witf;
        A_c9 += sf * w * cu * cF;
        A_m3b5 += sf * w;
        A_T45 += sgm * witT * cu * cu;
        A_b1 += sgm * witT;
        A_s += dg * w3 * cu;
        a.ux += cx * a_cu; a.uy += cy * a_cu;
        a.Fx += cx * a_cF; a.Fy += cy * a_cF;
        a.Sxx += cx * cx * a_cSc; a.Syy += cy * cy * a_cSc; a.Sxy += R(2) * cx * cy * a_cSc;
        a.gx += cx * a_cg; a.gy += cy * a_cg;
        a_vx += cx * a_cv; a_vy += cy * a_cv;
    }
    // per-node coefficients: b0 = 3 ep - 1.5 uu / eps - A trS / 2,
    // b1 = sigma Td - 1.5 T uu / eps + 3 T ep, k45, c9, m3b5 = -3 fF uF / eps, T45, s
    a.ep = R(3) * A_b0 + R(3) * s.T * A_b1;
    a.uu = R(-1.5) * ieps * A_b0 - R(1.5) * s.T * ieps * A_b1;
    a.ieps = R(-1.5) * s.uu * A_b0 - R(1.5) * s.T * s.uu * A_b1 + R(4.5) * A_k45 + R(9) * k.fF * A_c9
           - R(3) * k.fF * s.uF * A_m3b5 + R(4.5) * s.T * A_T45 + k.fT * ugT * A_s;
    a.Sxx += R(-0.5) * k.A * A_b0;
    a.Syy += R(-0.5) * k.A * A_b0;
    a.Td += k.sig * A_b1;
    a.T = (R(-1.5) * s.uu * ieps + R(3) * s.ep) * A_b1 + k45 * A_T45 + k.itT * A_s;
    a.uF = R(-3) * k.fF * ieps * A_m3b5;
    const R a_ugT = k.fT * (ieps - k.isig) * A_s;
    // v = T F + eps p grad T
    a.T += s.Fx * a_vx + s.Fy * a_vy;
    a.Fx += s.T * a_vx; a.Fy += s.T * a_vy;
    a.ep += s.gx * a_vx + s.gy * a_vy;
    a.gx += s.ep * a_vx; a.gy += s.ep * a_vy;
    // u . grad T
    a.ux += s.gx * a_ugT; a.uy += s.gy * a_ugT;
    a.gx += s.ux * a_ugT; a.gy += s.uy * a_ugT;
}

// Adjoints of the moments a node's state is built from: sum_{i>0} f, first and second moments
// of f; sum g, first moment of g.
template <typename R> struct MomentAdj { R s18, jx, jy, Pxx, Pyy, Pxy, sg, hx, hy; };

// Adjoint of population q (f 0-8, g 9-17) of a node: its direct part (1 - 1/tau) lam plus the
// moments' part.
template <typename R> __device__ __forceinline__ R population_adj(int q, R lam, const Cst<R> &k, const MomentAdj<R> &a)
{
    const int i = q < 9 ? q : q - 9;
    const R cx = R(CXd[i]), cy = R(CYd[i]);
    R v = (q < 9 ? k.of : k.og) * lam;
    if (q < 9) v += cx * a.jx + cy * a.jy + cx * cx * a.Pxx + cy * cy * a.Pyy + cx * cy * a.Pxy + (i ? a.s18 : R(0));
    else v += a.sg + cx * a.hx + cy * a.hy;
    return v;
}

// Reverse of fwd_state: the state's adjoints to those of the moments and of the porosity
// (returned).  WALL: a.p holds an adjoint of the pressure of its own.
template <typename R, bool WALL>
__device__ __forceinline__ double state_vjp(const FwdState<R> &m, StateAdj<R> a, const AdjK<R> &c, const AdjEps<R> &ae,
                                            MomentAdj<R> &o)
{
    const Cst<R> &k = c.k;
    const EpsC<R> &e = ae.e;
    const R eps = e.eps, ieps = e.ieps, bM = e.bM;
    // grad T = (N + c u) / a, c = b (u . N) / d, d = a - b |u|^2, a = aM0 - eps p / 2
    R a_Nx = a.gx * m.ia, a_Ny = a.gy * m.ia;
    const R a_c = (a.gx * m.ux + a.gy * m.uy) * m.ia;
    a.ux += m.cc * a.gx * m.ia; a.uy += m.cc * a.gy * m.ia;
    R a_a = -(m.gx * a.gx + m.gy * a.gy) * m.ia;
    R a_bM = a_c * m.uN / m.d;
    const R a_uN = a_c * bM / m.d;
    const R a_d = -a_c * m.cc / m.d;
    a_a += a_d;
    a_bM += -m.uu * a_d;
    a.uu += -bM * a_d;
    a.ux += m.Nx * a_uN; a.uy += m.Ny * a_uN;
    a_Nx += m.ux * a_uN; a_Ny += m.uy * a_uN;
    a.ep += R(-0.5) * a_a;
    // N = h - T u + (T F + u Q / sigma) / 2
    const R a_hx = a_Nx, a_hy = a_Ny;
    a.T += (R(0.5) * m.Fx - m.ux) * a_Nx + (R(0.5) * m.Fy - m.uy) * a_Ny;
    a.ux += (R(0.5) * k.Q * k.isig - m.T) * a_Nx;
    a.uy += (R(0.5) * k.Q * k.isig - m.T) * a_Ny;
    a.Fx += R(0.5) * m.T * a_Nx; a.Fy += R(0.5) * m.T * a_Ny;
    a.Td += a.T;
    a.ieps += R(0.5) * a_bM;                           // b = (1/eps - 1/sigma) / 2
    // S (Eq. ShearEqCom)
    const R a_Pxx = k.Sden * a.Sxx, a_Pyy = k.Sden * a.Syy, a_Pxy = k.Sden * a.Sxy;
    a.ep += -k.Sden * (a.Sxx + a.Syy);
    a.ieps += -k.Sden * (m.qxx * a.Sxx + m.qyy * a.Syy + m.qxy * a.Sxy);
    const R sx = -ieps * k.Sden;
    a.ux += sx * ((R(2) * m.ux - m.Fx) * a.Sxx + (m.uy - R(0.5) * m.Fy) * a.Sxy);
    a.uy += sx * ((R(2) * m.uy - m.Fy) * a.Syy + (m.ux - R(0.5) * m.Fx) * a.Sxy);
    a.Fx += -sx * (m.ux * a.Sxx + R(0.5) * m.uy * a.Sxy);
    a.Fy += -sx * (m.uy * a.Syy + R(0.5) * m.ux * a.Sxy);
    // ep = eps p
    R a_p = eps * a.ep;
    if (WALL) a_p += a.p;
    double a_eps = double(m.p * a.ep);
    // p = 0.6 X / eps, X = s18 - (2/3) uu / eps - (4/3) fF tau_f uF / eps
    const R a_X = R(0.6) * ieps * a_p;
    a.ieps += R(0.6) * m.X * a_p + a_X * (R(-2.0 / 3.0) * m.uu + R(-4.0 / 3.0) * k.fF * k.tau_f * m.uF);
    const R a_s18 = a_X;
    a.uu += m.cuu * a_X;
    a.uF += m.cuF * a_X;
    a.ux += R(2) * m.ux * a.uu + m.Fx * a.uF;
    a.uy += R(2) * m.uy * a.uu + m.Fy * a.uF;
    a.Fx += m.ux * a.uF;
    a.Fy += m.uy * a.uF;
    // F = eps G - (dlin + dquad |u|) u (Eq. ForceEq)
    a_eps += double(m.Gx * a.Fx + m.Gy * a.Fy);
    R a_Gy = eps * a.Fy;
    const R a_dl = -(m.ux * a.Fx + m.uy * a.Fy);
    a.ux += -m.dl * a.Fx; a.uy += -m.dl * a.Fy;
    const double a_um = double(e.dquad * a_dl);
    a_eps += double(a_dl) * (c.nuK + double(m.um) * ae.dEF * c.isqK);
    // u = v / (c0 + sqrt(c0^2 + c1 |v|)) in FP64 (Sec. 3.1)
    double a_vxd = m.iden * double(a.ux), a_vyd = m.iden * double(a.uy), a_vm = m.iden * a_um;
    const double a_iden = m.vx * double(a.ux) + m.vy * double(a.uy) + m.vm * a_um;
    const double a_den = -m.iden * m.iden * a_iden;
    const double a_c0 = a_den * (1.0 + e.c0 / m.Rt), a_c1 = a_den * m.vm / (2.0 * m.Rt);
    a_vm += a_den * e.c1 / (2.0 * m.Rt);
    if (m.vm > 0.0) { a_vxd += m.vx / m.vm * a_vm; a_vyd += m.vy / m.vm * a_vm; }   // |v| has derivative 0 at v = 0
    a_eps += 0.25 * c.nuK * a_c0 + 0.5 * c.isqK * ae.dEF * a_c1;
    // v = j + eps G / 2
    a_eps += 0.5 * (double(m.Gx) * a_vxd + double(m.Gy) * a_vyd);
    a_Gy += R(0.5 * e.epsd * a_vyd);
    const R a_jx = R(a_vxd), a_jy = R(a_vyd);
    a.Td += k.gb * a_Gy;
    a_eps += -double(ieps) * double(ieps) * double(a.ieps);
    o.s18 = a_s18; o.jx = a_jx; o.jy = a_jy; o.Pxx = a_Pxx; o.Pyy = a_Pyy; o.Pxy = a_Pxy;
    o.sg = k.isig * a.Td; o.hx = a_hx; o.hy = a_hy;
    return a_eps;
}

// Reverse mode (vector-Jacobian product) of the update of a node off the walls, in the
// arithmetic type R of the storage (FP64 for FP64 storage, FP32 for FP32 and FP16), the
// drag solve in FP64 as in the forward step.  The update is
//   f*_i = (1 - 1/tau_f) f_i + Phi_i(M(f, g), eps),   g*_i = (1 - 1/tau_T) g_i + Psi_i(M, eps),
// with M the moments the node state is built from (sum g, first moments of f and g, the
// sum over i > 0 of f, the second moments of f) and Phi, Psi the equilibrium, forcing and
// source parts of the collision (Eqs. LBEeq, FtermF, TEqColli, Eq:Tforce) of the state of
// Secs. 3.1-3.3 (drag solve, pressure, S, grad T).  Given the adjoints lam of the
// post-collision populations, this gives the adjoints of the moments (population_adj makes
// those of the populations of them) and returns the derivative with respect to the node's
// porosity.
template <typename R>
__device__ __forceinline__ double node_vjp(const R *f, const R *g, const AdjK<R> &c, const AdjEps<R> &ae, const R *lam,
                                           MomentAdj<R> &o)
{
    FwdState<R> m;
    fwd_state<R>(f, g, c, ae, m);
    const ColState<R> s = {m.ux, m.uy, m.Fx, m.Fy, m.uu, m.uF, m.T, m.ep, m.gx, m.gy, ae.e.ieps};
    StateAdj<R> a;
    collide_vjp<R, 1>(lam, s, c, a);
    return state_vjp<R, false>(m, a, c, ae, o);
}

// A wall node's constants, those of its x_f (kept from step to step) and the forward state of
// x_f (formed while the other wavefronts end the step before) in LDS [WALL_ROWS][ADJ_WALLS]: in
// registers they make the reverse pass spill.
constexpr int WALL_ROWS = 47;
struct WallLds {
    double *p;
    __device__ __forceinline__ void put(const FwdState<double> &m) const
    {
        const double v[21] = {m.Td, m.ux, m.uy, m.um, m.dl, m.Fx, m.Fy, m.X, m.p, m.Nx, m.Ny,
                              m.d, m.cc, m.ia, m.gx, m.gy, m.vx, m.vy, m.vm, m.Rt, m.iden};
#pragma unroll
        for (int i = 0; i < 21; ++i) p[(26 + i) * ADJ_WALLS] = v[i];
    }
    // the stored values and those formed of them (as in fwd_state)
    __device__ __forceinline__ FwdState<double> state(const AdjK<double> &c, const EpsC<double> &e) const
    {
        const double *const q = p + 26 * ADJ_WALLS;
        FwdState<double> m;
        m.Td = q[0]; m.ux = q[ADJ_WALLS]; m.uy = q[2 * ADJ_WALLS]; m.um = q[3 * ADJ_WALLS]; m.dl = q[4 * ADJ_WALLS];
        m.Fx = q[5 * ADJ_WALLS]; m.Fy = q[6 * ADJ_WALLS]; m.X = q[7 * ADJ_WALLS]; m.p = q[8 * ADJ_WALLS];
        m.Nx = q[9 * ADJ_WALLS]; m.Ny = q[10 * ADJ_WALLS]; m.d = q[11 * ADJ_WALLS]; m.cc = q[12 * ADJ_WALLS];
        m.ia = q[13 * ADJ_WALLS]; m.gx = q[14 * ADJ_WALLS]; m.gy = q[15 * ADJ_WALLS]; m.vx = q[16 * ADJ_WALLS];
        m.vy = q[17 * ADJ_WALLS]; m.vm = q[18 * ADJ_WALLS]; m.Rt = q[19 * ADJ_WALLS]; m.iden = q[20 * ADJ_WALLS];
        m.T = c.T0 + m.Td;
        m.Gx = c.k.ax;
        m.Gy = c.k.ay + c.k.gb * m.Td;
        m.uu = m.ux * m.ux + m.uy * m.uy;
        m.uF = m.ux * m.Fx + m.uy * m.Fy;
        m.cuu = (-2.0 / 3.0) * e.ieps;
        m.cuF = (-4.0 / 3.0) * c.k.fF * c.k.tau_f * e.ieps;
        m.ep = e.eps * m.p;
        m.qxx = m.ux * m.ux - m.ux * m.Fx;
        m.qyy = m.uy * m.uy - m.uy * m.Fy;
        m.qxy = m.ux * m.uy - 0.5 * (m.ux * m.Fy + m.Fx * m.uy);
        m.uN = m.ux * m.Nx + m.uy * m.Ny;
        return m;
    }
    __device__ __forceinline__ void put(const AdjEps<double> &a, int o) const
    {
        const double v[9] = {a.e.eps, a.e.ieps, a.e.dlin, a.e.dquad, a.e.bM, a.e.c0, a.e.c1, a.e.epsd, a.dEF};
#pragma unroll
        for (int i = 0; i < 9; ++i) p[(o + i) * ADJ_WALLS] = v[i];
    }
    __device__ __forceinline__ AdjEps<double> eps(int o) const
    {
        const double *const q = p + o * ADJ_WALLS;
        AdjEps<double> a;
        a.e.eps = q[0]; a.e.ieps = q[ADJ_WALLS]; a.e.dlin = q[2 * ADJ_WALLS]; a.e.dquad = q[3 * ADJ_WALLS];
        a.e.bM = q[4 * ADJ_WALLS]; a.e.c0 = q[5 * ADJ_WALLS]; a.e.c1 = q[6 * ADJ_WALLS]; a.e.epsd = q[7 * ADJ_WALLS];
        a.dEF = q[8 * ADJ_WALLS];
        return a;
    }
    __device__ __forceinline__ void put(const WallC<double> &w) const
    {
        const double v[8] = {w.ux, w.uy, w.um, w.Td, w.gx, w.gy, w.dx, w.dy};
#pragma unroll
        for (int i = 0; i < 8; ++i) p[(18 + i) * ADJ_WALLS] = v[i];
    }
    __device__ __forceinline__ WallC<double> wall(bool iso, bool px, bool py) const
    {
        const double *const q = p + 18 * ADJ_WALLS;
        WallC<double> w;
        w.ux = q[0]; w.uy = q[ADJ_WALLS]; w.um = q[2 * ADJ_WALLS]; w.Td = q[3 * ADJ_WALLS];
        w.gx = q[4 * ADJ_WALLS]; w.gy = q[5 * ADJ_WALLS]; w.dx = q[6 * ADJ_WALLS]; w.dy = q[7 * ADJ_WALLS];
        w.iso = iso; w.px = px; w.py = py;
        return w;
    }
};
constexpr int WALL_OWN = 0, WALL_REF = 9;     // rows of the node's own porosity and of x_f's

// The same for a wall node (wall_from_state, then the collision with the state it assigns),
// in FP64: adjoints of the moments of its reference node x_f, wt of T(x_ff), geb of its own
// porosity and gef of that of x_f.  lam[q ST].  The state of x_f is read from LDS twice, for the
// reverse of the collision and the scheme and then for its own (held across, it does not fit
// the registers).
template <int ST>
__device__ __forceinline__ void wall_vjp(double Tdff, const WallLds &wd, bool iso, bool px, bool py, const AdjK<double> &c,
                                         const double *lam, MomentAdj<double> &o, double &wt, double &geb, double &gef)
{
    const Cst<double> &k = c.k;
    const AdjEps<double> af = wd.eps(WALL_REF), ab = wd.eps(WALL_OWN);
    const EpsC<double> &eb = ab.e;
    const WallC<double> w = wd.wall(iso, px, py);
    const FwdState<double> m = wd.state(c, af.e);
    // the state of the wall node
    const double ief = af.e.ieps, ieb = eb.ieps;
    const double gbx = w.px ? w.gx : m.gx, gby = w.py ? w.gy : m.gy;
    const double Tdb = w.iso ? w.Td : (4.0 * m.Td - Tdff - 2.0 * (w.dx * gbx + w.dy * gby)) * (1.0 / 3.0);
    const double Tb = c.T0 + Tdb, epb = eb.eps * m.p;
    const double dl = eb.dlin + eb.dquad * w.um;
    const double Gx = k.ax, Gy = k.ay + k.gb * Tdb;
    const double Fx = eb.eps * Gx - dl * w.ux, Fy = eb.eps * Gy - dl * w.uy;
    const double ub2 = w.ux * w.ux + w.uy * w.uy, uf2 = m.uu;
    const ColState<double> s = {w.ux, w.uy, Fx, Fy, ub2, w.ux * Fx + w.uy * Fy, Tb, epb, gbx, gby, ieb};
    StateAdj<double> a;
    collide_vjp<double, ST>(lam, s, c, a);
    // (1 - 1/tau) lam: adjoints of f = ff + f^eq(x_b) - f^eq(x_f) and g likewise, so of ff, gf directly
    double a_Tdb = a.Td, a_Tb = a.T, a_ieb = a.ieps, a_epb = a.ep;
    const double aFx = a.Fx + w.ux * a.uF, aFy = a.Fy + w.uy * a.uF;
    geb = Gx * aFx + Gy * aFy - (w.ux * aFx + w.uy * aFy) * (c.nuK + w.um * ab.dEF * c.isqK);
    a_Tdb += eb.eps * k.gb * aFy;
    double a_gbx = a.gx, a_gby = a.gy;
    // sums over the directions i > 0 of omega_i times the adjoint of f_i or g_i
    double fs = 0.0, fcx = 0.0, fcy = 0.0, fuu = 0.0, fux = 0.0, fuy = 0.0, fbb = 0.0;
    double gs = 0.0, gcx = 0.0, gcy = 0.0, guu = 0.0, gux = 0.0, guy = 0.0, gbb = 0.0, gb1 = 0.0, gu1 = 0.0;
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        const double cx = CXd[i], cy = CYd[i];
        const double cub = cx * w.ux + cy * w.uy, cuf = cx * m.ux + cy * m.uy;
        const double wf = Wd(i) * (k.of * lam[i * ST]), wg = Wd(i) * (k.og * lam[(9 + i) * ST]);
        fs += wf; fcx += cx * wf; fcy += cy * wf; fuu += wf * cuf * cuf; fux += wf * cuf * cx; fuy += wf * cuf * cy;
        fbb += wf * cub * cub;
        gs += wg; gcx += cx * wg; gcy += cy * wg; guu += wg * cuf * cuf; gux += wg * cuf * cx; guy += wg * cuf * cy;
        gbb += wg * cub * cub; gb1 += wg * cub; gu1 += wg * cuf;
    }
    const double rf0 = k.of * lam[0], rg0 = k.og * lam[9 * ST];
    const double Tfi = m.T * ief;
    const double uub = ub2 * ieb, uuf = uf2 * ief;
    // f: omega_i (fe + 3 (c.u_b - c.u_f) + 4.5 ((c.u_b)^2 / eps_b - (c.u_f)^2 / eps_f)), fe = 3 dep - 1.5 duu
    const double a_dep = 3.0 * fs - (5.0 / 3.0) * rf0, a_duu = -1.5 * fs - (2.0 / 3.0) * rf0;
    // g: omega_i (ge + 3 (T_b c.u_b - T_f c.u_f) + 4.5 (...) + sigma B c.(grad T_b - grad T_f)),
    // ge = dsT - 1.5 dTuu + 3 dTep
    const double a_dsT = gs + (4.0 / 9.0) * rg0, a_dTuu = -1.5 * gs - (2.0 / 3.0) * rg0;
    const double a_dTep = 3.0 * gs - (5.0 / 3.0) * rg0;
    StateAdj<double> b = {};
    b.ux = -3.0 * fcx - 9.0 * ief * fux - 3.0 * m.T * gcx - 9.0 * Tfi * gux;
    b.uy = -3.0 * fcy - 9.0 * ief * fuy - 3.0 * m.T * gcy - 9.0 * Tfi * guy;
    const double a_Tfi = -4.5 * guu;
    b.ieps = -4.5 * fuu + m.T * a_Tfi;
    b.T = -3.0 * gu1 + ief * a_Tfi - uuf * a_dTuu - m.ep * a_dTep;
    b.uu = ief * (-a_duu - m.T * a_dTuu);
    b.ieps += uf2 * (-a_duu - m.T * a_dTuu);
    b.Td = -k.sig * a_dsT;
    b.ep = -a_dep - m.T * a_dTep;
    b.gx = -k.sigB * gcx;
    b.gy = -k.sigB * gcy;
    a_Tb += 3.0 * gb1 + 4.5 * ieb * gbb + uub * a_dTuu + epb * a_dTep;
    a_ieb += 4.5 * fbb + 4.5 * Tb * gbb + ub2 * (a_duu + Tb * a_dTuu);
    a_Tdb += k.sig * a_dsT + a_Tb;
    a_epb += a_dep + Tb * a_dTep;
    a_gbx += k.sigB * gcx;
    a_gby += k.sigB * gcy;
    b.p = eb.eps * a_epb;
    geb += m.p * a_epb - ieb * ieb * a_ieb;
    wt = 0.0;
    if (!w.iso) {
        const double t = a_Tdb * (1.0 / 3.0);
        b.Td += 4.0 * t;
        wt = -t;
        a_gbx -= 2.0 * w.dx * t;
        a_gby -= 2.0 * w.dy * t;
    }
    if (!w.px) b.gx += a_gbx;
    if (!w.py) b.gy += a_gby;
    b.Sxx = a.Sxx; b.Syy = a.Syy; b.Sxy = a.Sxy;
    asm volatile("" ::: "memory");
    const AdjEps<double> ar = wd.eps(WALL_REF);
    gef = state_vjp<double, true>(wd.state(c, ar.e), b, c, ar, o);
}

// Region of a tile: its nodes' mu is needed at the launch's first step.
struct AdjRegion {
    int X0, X1, Y0, Y1;              // the tile (written by this block)
    int xlo, xhi, ylo, yhi;
    bool oxl, oxh, oyl, oyh;         // sides that shrink by one node per step
    int nb, nt, nl, nr;              // wall nodes of the region: rows y = 0, ny - 1, columns x = 0, nx - 1
};

// One direction: tile [a, b) of n nodes, `one` = it spans the grid, per = periodic.  A side
// that comes within two nodes of a wall is moved to the wall.
__host__ __device__ __forceinline__ void adj_extent(int a, int b, int n, bool one, bool per, int ns, int &lo, int &hi,
                                                    bool &ol, bool &oh)
{
    lo = a - (ns - 1);
    hi = b + (ns - 1);
    ol = oh = true;
    if (one || (!per && lo <= 2)) { lo = 0; ol = false; }
    if (one || (!per && hi >= n - 2)) { hi = n; oh = false; }
}

__host__ __device__ __forceinline__ AdjRegion adj_region(const KParams &P, const TileGrid &g, int tx, int ty, int ns)
{
    AdjRegion t;
    t.X0 = tx * g.tw + (tx < g.rx ? tx : g.rx); t.X1 = t.X0 + g.tw + (tx < g.rx ? 1 : 0);
    t.Y0 = ty * g.th + (ty < g.ry ? ty : g.ry); t.Y1 = t.Y0 + g.th + (ty < g.ry ? 1 : 0);
    adj_extent(t.X0, t.X1, P.nx, g.nbx == 1, P.px, ns, t.xlo, t.xhi, t.oxl, t.oxh);
    adj_extent(t.Y0, t.Y1, P.ny, g.nby == 1, P.py, ns, t.ylo, t.yhi, t.oyl, t.oyh);
    t.nb = !P.py && !t.oyl ? t.xhi - t.xlo : 0;
    t.nt = !P.py && !t.oyh ? t.xhi - t.xlo : 0;
    t.nl = !P.px && !t.oxl ? t.yhi - t.ylo : 0;
    t.nr = !P.px && !t.oxh ? t.yhi - t.ylo : 0;
    return t;
}

__host__ __device__ __forceinline__ int adj_node_threads(const AdjRegion &t)
{
    return ((t.xhi - t.xlo) * (t.yhi - t.ylo) + 63) / 64 * 64;
}

// Forward state t of a segment: states t > 0 lie `stride` elements apart, t = 0 at ck.
template <typename S> struct AdjStates {
    const S *ck, *seg;
    long long stride;
    __device__ __forceinline__ const S *at(int i) const { return i == 0 ? ck : seg + i * stride; }
};

template <typename R> __device__ __forceinline__ void adj_consts(KConst p, AdjK<R> &c)
{
    load_consts(p, c.k);
    c.T0 = R(p->T0);
    c.nuK = p->nu_over_K;
    c.isqK = p->inv_sqrtK;
}

// What the two kinds of wavefronts of a block share.
template <typename S> struct AdjTile {
    AdjStates<S> st;
    KConst Pc;
    AdjRegion t;
    bool wx, wy;                 // the region spans the grid along a periodic direction: pulls wrap inside it
    int i1, ns;
    double *mu;                  // LDS [18][ADJ_NT]
    double *wr, *wt, *we;        // LDS: adjoints of wall nodes with respect to the populations of x_f
                                 // [18][ADJ_WALLS], T(x_ff) and the porosity of x_f
    double *wc;                  // LDS: WallLds [WALL_ROWS][ADJ_WALLS]
};

// mu_in(y + c_q, q) of node (x, y) from memory, 0 off the grid: lam[q ST].  The loads are
// unconditional (clamped to the grid) so that all are in flight together; one after the
// other, as conditional loads, they took 7 us.
template <int ST, typename R>
__device__ __forceinline__ void adj_pull(const KParams &P, const double *__restrict__ mu, int x, int y, R *lam)
{
    const long long N = (long long)P.nx * P.ny;
    const int xc[3] = {x > 0 ? x - 1 : (P.px ? P.nx - 1 : 0), x, x < P.nx - 1 ? x + 1 : (P.px ? 0 : x)};
    const int yc[3] = {y > 0 ? y - 1 : (P.py ? P.ny - 1 : 0), y, y < P.ny - 1 ? y + 1 : (P.py ? 0 : y)};
    const bool xin[3] = {P.px || x > 0, true, P.px || x < P.nx - 1}, yin[3] = {P.py || y > 0, true, P.py || y < P.ny - 1};
    double v[18];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const long long n = (long long)yc[1 + CYd[i]] * P.nx + xc[1 + CXd[i]];
        v[i] = mu[i * N + n];
        v[9 + i] = mu[(9 + i) * N + n];
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const bool in = xin[1 + CXd[i]] && yin[1 + CYd[i]];
        lam[i * ST] = in ? R(v[i]) : R(0);
        lam[(9 + i) * ST] = in ? R(v[9 + i]) : R(0);
    }
}

// The last step a node at (lx, ly) of the region takes: one less per node of distance from
// the tile towards a side that shrinks.
__device__ __forceinline__ int adj_last(const AdjRegion &t, int lx, int ly, int ns)
{
    int last = ns;
    if (t.oxl) last = min(last, lx + 1);
    if (t.oxh) last = min(last, t.xhi - t.xlo - lx);
    if (t.oyl) last = min(last, ly + 1);
    if (t.oyh) last = min(last, t.yhi - t.ylo - ly);
    return last;
}

// The wall nodes of the region, one per lane (a corner among the rows only).
template <typename S>
__device__ __forceinline__ void adj_walls(const AdjTile<S> &a, const KParams &P, const AdjBufs &A, int slot)
{
    const AdjRegion &t = a.t;
    const int rw = t.xhi - t.xlo, rh = t.yhi - t.ylo, rows = t.nb + t.nt, all = rows + t.nl + t.nr;
    int lx, ly;
    if (slot < t.nb) { lx = slot; ly = 0; }
    else if (slot < rows) { lx = slot - t.nb; ly = rh - 1; }
    else if (slot < rows + t.nl) { lx = 0; ly = slot - rows; }
    else { lx = rw - 1; ly = slot - rows - t.nl; }
    int x = t.xlo + lx, y = t.ylo + ly;
    const bool own = x >= t.X0 && x < t.X1 && y >= t.Y0 && y < t.Y1;
    if (P.px) x = ((x % P.nx) + P.nx) % P.nx;
    if (P.py) y = ((y % P.ny) + P.ny) % P.ny;
    const WallInfo w = wall_info(P, x, y);
    // a wall node takes part as long as its x_f does
    const int last = slot < all && (slot < rows || w.yw < 0) ? adj_last(t, lx + w.dx, ly + w.dy, a.ns) : 0;
    const bool hasl = P.px || x > 0, hasr = P.px || x < P.nx - 1, hasd = P.py || y > 0, hasu = P.py || y < P.ny - 1;
    const int cm = a.wx && lx == 0 ? rw - 1 : -1, cp = a.wx && lx == rw - 1 ? 1 - rw : 1;
    const int rm = a.wy && ly == 0 ? (rh - 1) * rw : -rw, rp = a.wy && ly == rh - 1 ? (1 - rh) * rw : rw;
    const double *const M = a.mu + (ly * rw + lx), *const Mm = M + rm, *const Mp = M + rp;
    // the longest chain of the step: issue ahead of the other wavefronts on the SIMD (256^2 FP32,
    // 300 steps back: 4.64 against 4.94 ms)
    __builtin_amdgcn_s_setprio(3);
    double *const lam = a.wr + slot;     // in LDS: replaced by the step's results, and those by the next lam
    double grad = 0.0;
    const WallLds wd = {a.wc + slot};
    bool iso = true, px = false, py = false;
    if (last > 0) {
        const double eb = eps_value(P, x, y), ef = eps_value(P, x + w.dx, y + w.dy);
        const WallC<double> wc = wall_consts<double>(P, w);
        adj_pull<ADJ_WALLS, double>(P, A.mu_in, x, y, lam);
        iso = wc.iso; px = wc.px; py = wc.py;
        wd.put(wc);
        wd.put(adj_eps<double>(P, eb), WALL_OWN);
        wd.put(adj_eps<double>(P, ef), WALL_REF);
    }
    double Tdff = 0.0;
    // the state of x_f (and T at x_ff) for step s
    auto forward = [&](int s) {
        const S *src = a.st.at(a.i1 + 1 - s);
        int xs = x, ys = y;
        asm volatile("" : "+v"(xs), "+v"(ys));     // the gather's addresses are formed in every step
        double f[9], g[9];
        gather<S, double>(src, P, xs + w.dx, ys + w.dy, f, g);
        if (!iso) Tdff = gather_Td<S, double>(src, P, P.cd, xs + 2 * w.dx, ys + 2 * w.dy);
        AdjK<double> c;
        adj_consts(fresh(a.Pc), c);
        FwdState<double> m;
        fwd_state<double>(f, g, c, wd.eps(WALL_REF), m);
        wd.put(m);
    };
    if (last > 0) forward(1);
#pragma clang loop unroll(disable)
    for (int s = 1;; ++s) {
        if (s <= last) {
            AdjK<double> c;
            adj_consts(fresh(a.Pc), c);
            MomentAdj<double> o;
            double wt, geb, gef;
            wall_vjp<ADJ_WALLS>(Tdff, wd, iso, px, py, c, lam, o, wt, geb, gef);
#pragma unroll
            for (int q = 0; q < 18; ++q) lam[q * ADJ_WALLS] = population_adj<double>(q, lam[q * ADJ_WALLS], c.k, o);
            a.wt[slot] = wt;
            a.we[slot] = gef;
            grad += geb;
        }
        __syncthreads();
        if (s == a.ns) break;
        if (s < last) forward(s + 1);
        __syncthreads();
        if (s < last) {
            const double *const b[9] = {M, M + cp, Mp, M + cm, Mm, Mp + cp, Mp + cm, Mm + cm, Mm + cp};
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const bool in = (CXd[i] > 0 ? hasr : (CXd[i] < 0 ? hasl : true)) && (CYd[i] > 0 ? hasu : (CYd[i] < 0 ? hasd : true));
                lam[i * ADJ_WALLS] = in ? b[i][i * ADJ_NT] : 0.0;
                lam[(9 + i) * ADJ_WALLS] = in ? b[i][(9 + i) * ADJ_NT] : 0.0;
            }
        }
    }
    if (own && last > 0) A.grad[(long long)y * P.nx + x] += grad;
}

// The nodes of the region, one per lane.
template <typename S>
__device__ __forceinline__ void adj_nodes(const AdjTile<S> &a, const KParams &P, const AdjBufs &A)
{
    using R = typename Prec<S>::R;
    const AdjRegion &t = a.t;
    const int rw = t.xhi - t.xlo, rh = t.yhi - t.ylo;
    const int ly = (int)(((float)threadIdx.x + 0.5f) * __builtin_amdgcn_rcpf((float)rw)), lx = (int)threadIdx.x - ly * rw;
    int x = t.xlo + lx, y = t.ylo + ly;
    const bool in = ly < rh, own = in && x >= t.X0 && x < t.X1 && y >= t.Y0 && y < t.Y1;
    if (P.px) x = ((x % P.nx) + P.nx) % P.nx;
    if (P.py) y = ((y % P.ny) + P.ny) % P.ny;
    const bool wall = on_wall(P, x, y);
    const int last = in && !wall ? adj_last(t, lx, ly, a.ns) : 0;     // mu is 0 at a wall node
    const int cm = a.wx && lx == 0 ? rw - 1 : -1, cp = a.wx && lx == rw - 1 ? 1 - rw : 1;
    const int rm = a.wy && ly == 0 ? (rh - 1) * rw : -rw, rp = a.wy && ly == rh - 1 ? (1 - rh) * rw : rw;
    double *const M = a.mu + (ly * rw + lx);
    const double *const Mm = M + rm, *const Mp = M + rp;
    // the wall nodes whose x_f (bit i - 1) or x_ff (bit 7 + i) this node is, by their inward
    // direction c_i
    unsigned refs = 0;
    if (t.nb + t.nt + t.nl + t.nr > 0 && last > 0) {
#pragma unroll
        for (int i = 1; i < 9; ++i)
            for (int dist = 1; dist <= 2; ++dist) {
                const int bx = lx - dist * CXd[i], by = ly - dist * CYd[i];
                if (bx < 0 || bx >= rw || by < 0 || by >= rh) continue;
                const WallInfo b = wall_info(P, x - dist * CXd[i], y - dist * CYd[i]);
                if (b.dx != CXd[i] || b.dy != CYd[i]) continue;
                if (dist == 1) refs |= 1u << (i - 1);
                else if (thermal_dirichlet_wall(P, b) < 0) refs |= 1u << (7 + i);
            }
    }
    // slot of such a wall node at distance dist
    auto slot_of = [&](int i, int dist) {
        const int dx = ((0x122 >> i) & 1) - ((0xc8 >> i) & 1), dy = ((0x64 >> i) & 1) - ((0x190 >> i) & 1);   // c_i
        const int bx = lx - dist * dx, by = ly - dist * dy;
        return dy > 0 ? bx : (dy < 0 ? t.nb + bx : (dx > 0 ? t.nb + t.nt + by : t.nb + t.nt + t.nl + by));
    };
    R lam[18];
    AdjEps<R> ae;
    double m[18], grad = 0.0;
    R f[9], g[9];
    // the populations of step s, loaded while step s - 1 ends (FP64: at its start, or the step spills)
    constexpr bool AHEAD = sizeof(R) == 4;
    auto load = [&](int s) {
        int xs = x, ys = y;
        asm volatile("" : "+v"(xs), "+v"(ys));     // the gather's addresses are formed in every step
        gather<S, R>(a.st.at(a.i1 + 1 - s), P, xs, ys, f, g);
    };
    if (last > 0) {
        // all loads first: each wait for memory costs more than what follows it
        const double eps = eps_value(P, x, y);
        if (AHEAD) load(1);
        adj_pull<1, R>(P, A.mu_in, x, y, lam);
        ae = adj_eps<R>(P, eps);
    }
#pragma clang loop unroll(disable)
    for (int s = 1;; ++s) {
        const KConst pc = fresh(a.Pc);
        if (s <= last) {
            if (!AHEAD) load(s);
            AdjK<R> c;
            adj_consts(pc, c);
            MomentAdj<R> o;
            grad += node_vjp<R>(f, g, c, ae, lam, o);
#pragma unroll
            for (int q = 0; q < 18; ++q) m[q] = double(population_adj<R>(q, lam[q], c.k, o));
        } else {
#pragma unroll
            for (int q = 0; q < 18; ++q) m[q] = 0.0;
        }
        if (AHEAD && s < last) load(s + 1);
        __syncthreads();
        if (s <= last) {
            for (unsigned b = refs; b; b &= b - 1) {
                const int j = __builtin_ctz(b);
                if (j < 8) {
                    const int k = slot_of(j + 1, 1);
#pragma unroll
                    for (int q = 0; q < 18; ++q) m[q] += a.wr[q * ADJ_WALLS + k];
                    grad += a.we[k];
                } else {
                    const double v = a.wt[slot_of(j - 7, 2)] * pc->cd.isig;
#pragma unroll
                    for (int q = 9; q < 18; ++q) m[q] += v;
                }
            }
        }
        if (s == a.ns) break;
        if (in) {
#pragma unroll
            for (int q = 0; q < 18; ++q) M[q * ADJ_NT] = m[q];
        }
        __syncthreads();
        if (s < last) {
            const double *const b[9] = {M, M + cp, Mp, M + cm, Mm, Mp + cp, Mp + cm, Mm + cm, Mm + cp};
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                lam[i] = R(b[i][i * ADJ_NT]);
                lam[9 + i] = R(b[i][(9 + i) * ADJ_NT]);
            }
        }
    }
    if (own) {
        const long long N = (long long)P.nx * P.ny, n = (long long)y * P.nx + x;
#pragma unroll
        for (int q = 0; q < 18; ++q) A.mu_out[q * N + n] = m[q];
        if (!wall) A.grad[n] += grad;
    }
}

template <typename S>
__global__ void __launch_bounds__(ADJ_NT)
k_adj(AdjStates<S> st, KParams P, AdjBufs A, TileGrid g, int i1, int ns)
{
    __shared__ double mu[18 * ADJ_NT];
    __shared__ double wr[(20 + WALL_ROWS) * ADJ_WALLS];
    const int b = xcd_block(blockIdx.x, gridDim.x), ty = tile_row(g, b);
    const KConst Pc = (KConst)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr()
                               + sizeof(AdjStates<S>));
    const AdjTile<S> a = {st, Pc, adj_region(P, g, b - ty * g.nbx, ty, ns), P.px && g.nbx == 1, P.py && g.nby == 1, i1, ns,
                          mu, wr, wr + 18 * ADJ_WALLS, wr + 19 * ADJ_WALLS, wr + 20 * ADJ_WALLS};
    // wavefront-uniform: both kinds pass the same barriers, two per step but the last
    const int nodes = adj_node_threads(a.t);
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 64 < nodes) adj_nodes<S>(a, P, A);
    else adj_walls<S>(a, P, A, (int)threadIdx.x - nodes);
}

// Tiles and steps per launch: as tile_plan, over the regions and the wall nodes of this kernel,
// whose registers allow one block of eight wavefronts on a CU.
int adjoint_plan(const KParams &P, TileGrid &grid, int &threads)
{
    static const int shapes[][2] = {{8, 8}, {12, 8}, {16, 8}, {12, 12}, {16, 12}, {16, 16}, {20, 16}, {24, 14}};
    const double cus = 256.0;
    int best = 0;
    double cost = 0.0;
    for (const auto &sh : shapes) {
        const TileGrid g = tile_grid(P, sh[0], sh[1]);
        if ((g.nbx > 1 && g.tw < 4) || (g.nby > 1 && g.th < 4)) continue;
        for (int ns = 1; ns <= 6; ++ns) {
            int most = 0, walls = 0;
            // the tiles' regions differ near the walls and by one node in width and height
            const int cx[8] = {0, 1, 2, g.rx - 1, g.rx, g.nbx - 3, g.nbx - 2, g.nbx - 1};
            const int cy[8] = {0, 1, 2, g.ry - 1, g.ry, g.nby - 3, g.nby - 2, g.nby - 1};
            for (int ty : cy)
                for (int tx : cx) {
                    if (tx < 0 || tx >= g.nbx || ty < 0 || ty >= g.nby) continue;
                    const AdjRegion t = adj_region(P, g, tx, ty, ns);
                    const int nw = t.nb + t.nt + t.nl + t.nr;
                    walls = std::max(walls, nw);
                    most = std::max(most, adj_node_threads(t) + (nw + 63) / 64 * 64);
                }
            if (most > ADJ_NT || walls > ADJ_WALLS) break;
            const double nb = (double)g.nbx * g.nby, rounds = std::ceil(nb / cus);
            const double c = rounds * (1.0 + 0.4 * ns) / ns;
            if (best == 0 || c < cost) {
                cost = c;
                best = ns;
                grid = g;
                threads = most;
            }
        }
    }
    return best;
}

// Seed: mu(z, q) of the state J is evaluated at, J depending on T at interior nodes with
// weights wtj (T = T0 + (sum_i g_i + Q/2) / sigma, g_i(z) = s(z - c_i, 9 + i)).
__global__ void __launch_bounds__(256) k_adj_seed(KParams P, const double *__restrict__ wtj, double *__restrict__ mu)
{
    const long long N = (long long)P.nx * P.ny;
    const long long n = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    const double v = on_wall(P, int(n % P.nx), int(n / P.nx)) ? 0.0 : wtj[n] * (1.0 / P.sigma);
    for (int q = 0; q < 18; ++q) mu[q * N + n] = q < 9 ? 0.0 : v;
}

hipError_t launch_adjoint_seed(const KParams &P, const double *wtj, double *mu, hipStream_t st)
{
    const long long N = (long long)P.nx * P.ny;
    hipLaunchKernelGGL(k_adj_seed, dim3(unsigned((N + 255) / 256)), dim3(256), 0, st, P, wtj, mu);
    return hipGetLastError();
}

template <typename S>
static hipError_t adj_steps_t(const void *ck, const void *seg, long long stride, const KParams &P, const AdjBufs &A,
                              const TileGrid &g, int threads, int i1, int ns, hipStream_t st)
{
    const AdjStates<S> s = {(const S *)ck, (const S *)seg, stride};
    hipLaunchKernelGGL((k_adj<S>), dim3(g.nbx * g.nby), dim3(threads), 0, st, s, P, A, g, i1, ns);
    return hipGetLastError();
}

hipError_t launch_adjoint_steps(int storage, const void *ck, const void *seg, long long stride, const KParams &P,
                                const AdjBufs &A, const TileGrid &g, int threads, int i1, int ns, hipStream_t st)
{
    switch (storage) {
    case 0: return adj_steps_t<double>(ck, seg, stride, P, A, g, threads, i1, ns, st);
    case 1: return adj_steps_t<float>(ck, seg, stride, P, A, g, threads, i1, ns, st);
    case 2: return adj_steps_t<__half>(ck, seg, stride, P, A, g, threads, i1, ns, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm

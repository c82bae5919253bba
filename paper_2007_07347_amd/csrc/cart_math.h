// Per-cell and per-face arithmetic of the structured step (tensor-product quad
// meshes), shared by every kernel that advances such meshes.  All of it is
// written with explicit fused multiply-adds in a fixed order, so a cell's new
// state has the same bits whichever kernel, strip or tile computes it.
//
// The faces are normal to x or to y.  A side of a cell, seen along the axis of
// its face, is five values of the reconstruction at the foot points
// x_f - e_i dt: the three velocities that leave the cell through the side
// (along the axis; with the positive tangential component; with the negative
// one), and of the three velocities along the face their sum and the
// difference of the two moving ones, which is all the face macros need.
#pragma once

#include "mesh.h"
#include "step_common.h"

namespace sdg {
namespace {

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Arithmetic type of fbar+, gradients and face states; type of stored f.
template <int PM>
using Arith = typename std::conditional<PM == SDUGKS_FP32DEV, float, double>::type;
template <int PM>
using Stored = typename std::conditional<PM == SDUGKS_FP64, double, float>::type;

// Velocities with a positive (P) and a negative (N) component along an axis, in
// the order: along the axis, positive tangential, negative tangential; and the
// velocities without one: rest, positive tangential, negative tangential.
constexpr int cP[2][3] = {{1, 5, 8}, {2, 5, 6}};
constexpr int cN[2][3] = {{3, 6, 7}, {4, 8, 7}};
constexpr int cT[2][3] = {{0, 2, 4}, {0, 1, 3}};
constexpr bool axis_tables_match()
{
    for (int a = 0; a < 2; a++)
        for (int k = 0; k < 3; k++) {
            const int t = k == 0 ? 0 : (k == 1 ? 1 : -1);
            const int pn = a == 0 ? cEx[cP[a][k]] : cEy[cP[a][k]], pt = a == 0 ? cEy[cP[a][k]] : cEx[cP[a][k]];
            const int nn = a == 0 ? cEx[cN[a][k]] : cEy[cN[a][k]], nt = a == 0 ? cEy[cN[a][k]] : cEx[cN[a][k]];
            const int zn = a == 0 ? cEx[cT[a][k]] : cEy[cT[a][k]], zt = a == 0 ? cEy[cT[a][k]] : cEx[cT[a][k]];
            if (pn != 1 || pt != t || nn != -1 || nt != t || zn != 0 || zt != t) return false;
        }
    return true;
}
static_assert(axis_tables_match(), "velocity tables along the axes");

// One side of a cell (see the file comment).
template <typename R>
struct Side {
    R c[3], s, d;
};

constexpr double cWt[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};

// The nine equilibria of Eq. Feq (its second-order discrete form) minus w_i
// off, each divided by its weight w_i, grouped by opposite velocities: for a
// lattice direction d, f(+d) = w_d (S_d + 3 d.m) and f(-d) = w_d (S_d - 3 d.m),
// where S_d = B + 4.5 (d.m)(d.u), B = (rho - off) - 1.5 m.u and m = rho u.  The
// weights go into the factors the results are used with.
__device__ __forceinline__ void feq9(double rho, double mx, double my, double ux, double uy, double off, double fe[9])
{
    const double B = fma_(-1.5, fma_(mx, ux, my * uy), rho - off);
    fe[0] = B;
    auto pair = [&](int ip, int im, double dm, double du) {
        const double S = fma_(4.5 * dm, du, B);
        fe[ip] = fma_(3.0, dm, S);
        fe[im] = fma_(-3.0, dm, S);
    };
    pair(1, 3, mx, ux);
    pair(2, 4, my, uy);
    pair(5, 7, mx + my, ux + uy);
    pair(6, 8, my - mx, uy - ux);
}

// 1 / x for a density (a positive normal number): the hardware's approximation,
// off by some 2^-24 = e; one step to e^3, and a last one by its residual, which is
// exact.  The result is that of a division at every density tried, at half its
// cost; without the last step it misses the nearest number just below a power of
// two (1 - 3 2^-53).
__device__ __forceinline__ double recip(double x)
{
    const double y0 = __builtin_amdgcn_rcp(x), e = fma_(-x, y0, 1.0);
    const double y = fma_(y0, fma_(e, e, e), y0);
    return fma_(fma_(-x, y, 1.0), y, y);
}

// A value that is alike in all lanes, moved to scalar registers.
// (The empty asm keeps the compiler from holding it in vector registers all the
// same, where it is computed.)
__device__ __forceinline__ int uniform(int v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+v"(v));
#endif
    return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ float uniform(float v) { return __int_as_float(uniform(__float_as_int(v))); }
__device__ __forceinline__ double uniform(double v)
{
    return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}

// The step's constants in its arithmetic: fbar+ = a f + rb[] S with rb[] = b
// times the weights (rest, along the axes, diagonal; in NEQ a + b = 1 and f^n =
// feq + stored part, so b is 1 there), the time to the foot point, the factors
// of the face distribution.  rb[] stays in FP64, as the S do: rounded to FP32 it is
// off by the same factor in every cell and step, which adds up (256 x 256 cells in
// FP32 deviations after 2000 steps: 4.9e-8 to 6e-8 off FP64 arithmetic, 3.1e-8 to
// 3.6e-8 this way; a step of 1024 x 1024 cells takes 2 % longer).
template <int PM>
struct Factors {
    Arith<PM> ra, dt, c1, k1, k5;
    double rb[3];
    __device__ __forceinline__ explicit Factors(const DevMesh &m)
    {
        using R = Arith<PM>;
        const double b = PM == SDUGKS_FP32NEQ ? 1.0 : m.b;
        ra = uniform((R)m.a);
        rb[0] = uniform(b * (4.0 / 9));
        rb[1] = uniform(b * (1.0 / 9));
        rb[2] = uniform(b * (1.0 / 36));
        dt = uniform((R)m.dtr);
        c1 = uniform((R)m.fc1);
        k1 = uniform((R)(m.fb / 9.0));
        k5 = uniform((R)(m.fb / 36.0));
    }
};

// fbar+ of a cell (Eq. fbarplus) from its macros and stored f (in DEV the
// deviation from w_i rho0 in FP32; in NEQ f - feq).
template <int PM>
__device__ __forceinline__ void cell_plus(const DevMesh &m, const Factors<PM> &c, double r, double mu, double mv,
                                          const Stored<PM> fv[9], Arith<PM> fb[9])
{
    using R = Arith<PM>;
    const double ir = recip(r);
    double fe[9];
    feq9(r, mu, mv, mu * ir, mv * ir, PM == SDUGKS_FP32DEV ? m.rho0 : 0.0, fe);
#pragma unroll
    for (int i = 0; i < 9; i++) fb[i] = fma_(c.ra, (R)fv[i], (R)(c.rb[i == 0 ? 0 : (i < 5 ? 1 : 2)] * fe[i]));
}

// A boundary-condition entry; type as a number.
struct WallBC {
    double type, rho, u, v;
};
// The boundary state of Section III behind a wall of a cell differs from the
// cell's own by fbar+_b - fbar+_c = feq(rho_b, u_b) - feq(W_c), here pair by
// pair: few cells have walls, and the registers that all 18 equilibria take
// would be every wave's.
template <int PM>
__device__ __forceinline__ void wall_diff(const DevMesh &m, const WallBC &e, double r, double mu, double mv,
                                          Arith<PM> df[9])
{
    using R = Arith<PM>;
    const double off = PM == SDUGKS_FP32DEV ? m.rho0 : 0.0;
    const double ir = recip(r), ux = mu * ir, uy = mv * ir;
    const bool inlet = e.type == SDUGKS_BC_INLET, outlet = e.type == SDUGKS_BC_OUTLET;
    const bool sym = e.type == SDUGKS_BC_SYMMETRY;
    const double un = fma_(ux, e.u, uy * e.v);           // symmetry: (u, v) = unit normal
    const double rw = inlet ? e.rho : r;                 // inlet / far field
    const double uw = outlet ? ux : (sym ? fma_(-un, e.u, ux) : e.u);
    const double vw = outlet ? uy : (sym ? fma_(-un, e.v, uy) : e.v);
    const double mw = rw * uw, nw = rw * vw;
    const double Bc = fma_(-1.5, fma_(mu, ux, mv * uy), r - off), Bw = fma_(-1.5, fma_(mw, uw, nw * vw), rw - off);
    df[0] = (R)(cWt[0] * (Bw - Bc));
    auto pair = [&](int ip, int iq, double dmc, double duc, double dmw, double duw) {
        const double Sc = fma_(4.5 * dmc, duc, Bc), Sw = fma_(4.5 * dmw, duw, Bw);
        df[ip] = (R)(cWt[ip] * (fma_(3.0, dmw, Sw) - fma_(3.0, dmc, Sc)));
        df[iq] = (R)(cWt[iq] * (fma_(-3.0, dmw, Sw) - fma_(-3.0, dmc, Sc)));
    };
    pair(1, 3, mu, ux, mw, uw);
    pair(2, 4, mv, uy, nw, vw);
    pair(5, 7, mu + mv, ux + uy, mw + nw, uw + vw);
    pair(6, 8, mv - mu, uy - ux, nw - mw, vw - uw);
}

// Least-squares slope along an axis: the normal equations are diagonal on the
// four-point stencil, so it is the weighted sum of the differences to the two
// points on the axis (dm = own - lower, dp = upper - own; wm, wp the weights).
template <typename R>
__device__ __forceinline__ R slope(R wm, R wp, R dm, R dp)
{
    return fma_(wp, dp, (-wm) * dm);
}

// Reconstruction at the foot points x_f - e dt, as two steps: carried() serves
// the faces along axis AX, sides() adds what differs from face to face.  In FP32
// carried() holds fbar+_i - dt e_t g_t, the part across the axis, and along it a
// velocity's offset h - e dt from the centre is taken in one piece: dt e g first
// and h g after is rounded once more in between, up to an ulp of the slopes' part.
// In FP64 that is no part of any error that shows, and carried() holds both
// parts, alike for the two axes (half the registers: the FP64 march has none left,
// and took 2 to 3 % more with the other order).
template <typename R>
constexpr bool kOneOffset = std::is_same<R, float>::value;
template <int AX, typename R>
__device__ __forceinline__ void carried(R rdt, const R fb[9], const R gx[9], const R gy[9], R b[9])
{
    static_for<9>([&](auto I) {
        constexpr int i = I;
        R v = fb[i];
        if constexpr (cEx[i] != 0 && (AX == 1 || !kOneOffset<R>)) v = fma_(cEx[i] > 0 ? -rdt : rdt, gx[i], v);
        if constexpr (cEy[i] != 0 && (AX == 0 || !kOneOffset<R>)) v = fma_(cEy[i] > 0 ? -rdt : rdt, gy[i], v);
        b[i] = v;
    });
}

// fbar+ carried back along the whole of the k-th velocity that enters a cell on
// its lower (LOWER) or upper side along axis AX: b as carried(), g the slopes
// along the axis.
template <int AX, bool LOWER, typename R>
__device__ __forceinline__ R entering(R rdt, const R b[9], const R g[9], int k)
{
    const int i = LOWER ? cP[AX][k] : cN[AX][k];
    if constexpr (kOneOffset<R>) return fma_(LOWER ? -rdt : rdt, g[i], b[i]);
    else return b[i];
}

// The two sides of a cell along axis AX: offsets hm, hp of its lower and upper
// face from the centre, b as carried(), g the slopes along the axis.
template <int AX, typename R>
__device__ __forceinline__ void sides(R rdt, R hm, R hp, const R b[9], const R g[9], Side<R> &lower, Side<R> &upper)
{
    const R lo = kOneOffset<R> ? hm + rdt : hm, up = kOneOffset<R> ? hp - rdt : hp;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        upper.c[k] = fma_(up, g[cP[AX][k]], b[cP[AX][k]]);
        lower.c[k] = fma_(lo, g[cN[AX][k]], b[cN[AX][k]]);
    }
    const R sb = b[cT[AX][0]] + (b[cT[AX][1]] + b[cT[AX][2]]), sg = g[cT[AX][0]] + (g[cT[AX][1]] + g[cT[AX][2]]);
    const R db = b[cT[AX][1]] - b[cT[AX][2]], dg = g[cT[AX][1]] - g[cT[AX][2]];
    upper.s = fma_(hp, sg, sb);
    lower.s = fma_(hm, sg, sb);
    upper.d = fma_(hp, dg, db);
    lower.d = fma_(hm, dg, db);
}

// Fluxes through a face between the upper side of its lower cell and the lower
// side of its upper cell (Eqs. fbar, Macro, f_t_n+1, MesoFlux): p[k] carries
// velocity cP[AX][k] and n[k] velocity cN[AX][k], both counted along +axis for
// p and along -axis for n (so the flux of n[k] is -n[k]).  C = l fc1, K1 and
// K5 = C fb / 9 and C fb / 36.
template <int PM>
__device__ __forceinline__ void face_flux(const DevMesh &m, const Side<Arith<PM>> &lo, const Side<Arith<PM>> &hi,
                                          Arith<PM> C, Arith<PM> K1, Arith<PM> K5, Arith<PM> p[3], Arith<PM> n[3])
{
    using R = Arith<PM>;
    constexpr bool DEV = PM == SDUGKS_FP32DEV;
    const R P = lo.c[0] + (lo.c[1] + lo.c[2]), N = hi.c[0] + (hi.c[1] + hi.c[2]);
    const R rsum = fma_((R)0.5, lo.s + hi.s, P + N);
    const R mn = P - N;                                                              // momentum along the axis
    const R mt = fma_((R)0.5, lo.d + hi.d, (lo.c[1] - lo.c[2]) + (hi.c[1] - hi.c[2]));   // and along the face
    // in DEV sums of deviations: rho_f = rho0 + sum, the momentum unchanged
    const R rf = DEV ? (R)m.rho0 + rsum : rsum;
    R irf;
    if constexpr (DEV) irf = __builtin_amdgcn_rcpf(rf);
    else irf = recip(rf);
    const R un = mn * irf, ut = mt * irf;
    const R B = fma_((R)-1.5, fma_(mn, un, mt * ut), rsum);
    // the equilibria by opposite pairs (as feq9)
    auto pair = [&](R fp, R fn, R K, R dm, R du, R &op, R &on) {
        const R S = fma_((R)4.5 * dm, du, B);
        op = fma_(K, fma_((R)3, dm, S), C * fp);
        on = fma_(K, fma_((R)-3, dm, S), C * fn);
    };
    pair(lo.c[0], hi.c[0], K1, mn, un, p[0], n[0]);
    pair(lo.c[1], hi.c[2], K5, mn + mt, un + ut, p[1], n[2]);
    pair(lo.c[2], hi.c[1], K5, mn - mt, un - ut, p[2], n[1]);
}

// Net outflow of a cell by velocity, accumulated in FP64 side by side in the
// order x (upper minus lower), lower y, upper y.
struct Outflow {
    double F[9];                        // F[0] unused: the rest velocity crosses no face
};
template <int AX, typename R>
__device__ __forceinline__ void outflow_x(Outflow &o, const R pu[3], const R nu[3], const R pl[3], const R nl[3])
{
    static_assert(AX == 0, "x first");
    o.F[2] = 0.0;
    o.F[4] = 0.0;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        o.F[cP[0][k]] = (double)pu[k] - (double)pl[k];
        o.F[cN[0][k]] = (double)nl[k] - (double)nu[k];
    }
}
// the lower y face: inflow of p, outflow of n
template <typename R>
__device__ __forceinline__ void outflow_below(Outflow &o, const R p[3], const R n[3])
{
#pragma unroll
    for (int k = 0; k < 3; k++) {
        o.F[cP[1][k]] = k == 0 ? -(double)p[k] : o.F[cP[1][k]] - (double)p[k];
        o.F[cN[1][k]] = k == 0 ? (double)n[k] : o.F[cN[1][k]] + (double)n[k];
    }
}
template <typename R>
__device__ __forceinline__ void outflow_above(Outflow &o, const R p[3], const R n[3])
{
#pragma unroll
    for (int k = 0; k < 3; k++) {
        o.F[cP[1][k]] += (double)p[k];
        o.F[cN[1][k]] -= (double)n[k];
    }
}

// Cell update (Eqs. MacroUpdate, fn+1): W^n = (ro, mxo, myo), the outflow, the
// stored f^n; in lagged mode g holds the previous step's macroscopic flux and
// returns this step's.  Writes W^{n+1} into (rn, mxn, myn) and what f^{n+1} is
// stored as into v.
template <int PM>
__device__ __forceinline__ void cell_update(const DevMesh &m, int lagged, double dtv, double ro, double mxo,
                                            double myo, const Outflow &o, const Stored<PM> fo[9], double g[3],
                                            double &rn, double &mxn, double &myn, Stored<PM> v[9])
{
    constexpr bool DEV = PM == SDUGKS_FP32DEV, NEQ = PM == SDUGKS_FP32NEQ;
    const double *F = o.F;
    // the macroscopic flux: the moments of the mesoscopic one (Eq. MacroFlux)
    const double s57 = F[5] + F[7], s68 = F[6] + F[8], d57 = F[5] - F[7], d68 = F[6] - F[8];
    const double g0 = ((F[1] + F[3]) + (F[2] + F[4])) + (s57 + s68);
    const double g1 = (F[1] - F[3]) + (d57 - d68);
    const double g2 = (F[2] - F[4]) + (d57 + d68);
    const double G0 = lagged ? g[0] : g0, G1 = lagged ? g[1] : g1, G2 = lagged ? g[2] : g2;
    g[0] = g0;
    g[1] = g1;
    g[2] = g2;
    rn = fma_(-dtv, G0, ro);
    mxn = fma_(-dtv, G1, mxo);
    myn = fma_(-dtv, G2, myo);
    const double irn = recip(rn), un = mxn * irn, vn = myn * irn, off = DEV ? m.rho0 : 0.0;
    const double inv = m.inv1l, lw[3] = {m.lam * (4.0 / 9), m.lam * (1.0 / 9), m.lam * (1.0 / 36)};
    double fe[9], feo[9], x[9];
    // feq(W^n), that the storage form or the original scheme needs
    auto before = [&]() {
        const double iro = recip(ro);
        feq9(ro, mxo, myo, mxo * iro, myo * iro, off, feo);
    };
    // the original scheme: ft^{n+1} = (4/3) fbar+ - (1/3) ft - dt/V F
    auto original = [&](int i, double f0) {
        const double c = fma_(4.0 / 3.0, fma_(m.a, f0, m.b * (cWt[i] * feo[i])), (-1.0 / 3.0) * f0);
        return i == 0 ? c : fma_(-dtv, F[i], c);
    };
    if constexpr (NEQ) {
        feq9(rn, mxn, myn, un, vn, off, fe);
        before();
        static_for<9>([&](auto I) {
            constexpr int i = I;
            const double f0 = fma_(cWt[i], feo[i], (double)fo[i]);
            x[i] = m.scheme != 0 ? original(i, f0)
                                 : fma_(lw[i == 0 ? 0 : (i < 5 ? 1 : 2)], fe[i], i == 0 ? f0 : fma_(-dtv, F[i], f0)) * inv;
            v[i] = (Stored<PM>)fma_(-cWt[i], fe[i], x[i]);
        });
    } else if (m.scheme == 0) {
        // (the equilibria in either branch: held across them they cost the march
        // the registers of a third wave)
        static_for<9>([&](auto I) {
            constexpr int i = I;
            x[i] = (double)fo[i];
            if constexpr (i != 0) x[i] = fma_(-dtv, F[i], x[i]);
        });
        feq9(rn, mxn, myn, un, vn, off, fe);
        static_for<9>([&](auto I) {
            constexpr int i = I;
            v[i] = (Stored<PM>)(fma_(lw[i == 0 ? 0 : (i < 5 ? 1 : 2)], fe[i], x[i]) * inv);
        });
    } else {
        before();
        static_for<9>([&](auto I) {
            constexpr int i = I;
            v[i] = (Stored<PM>)original(i, (double)fo[i]);
        });
    }
}

}  // namespace
}  // namespace sdg

// fv_adjoint.hip -- discrete adjoint of the single-phase Euler right-hand side
// (vector-Jacobian product of Eq. (FVD) with WENO5-Z and HLLC, Sec. 3.2) and
// of the TVD-RK3 step at a fixed time step (Sec. 3.4), the reverse sweep that
// the paper obtains by automatic differentiation (Sec. 6).
//
// The face cotangents Fbar_f = (Rbar_f - Rbar_{f-1}) / h (R_i = -(F_{i+1/2} - F_{i-1/2}) / h)
// are pulled back through HLLC, WENO5-Z and the U -> W map (reverse sweeps written out
// below) along each direction by workgroups that own pieces of lines (rhs_adjoint_all).
// Non-differentiable points take the conventions of the adjoint's reference:
// |x|' = sgn(x) with sgn(0) = 0; min / max at a tie split the cotangent evenly; the
// upwind switch of the HLLC flux (the sign of s*) is piecewise constant; the
// hardware-estimate helpers rcp, rsqrt and sqrt_fast are differentiated exactly
// (d(1/x) = -dx/x^2, ...), not through their refinement steps.  The three directions'
// shares meet in atomic additions whose order is not fixed, so the result is
// reproducible to round-off, not bitwise.
#include <hip/hip_runtime.h>

#include "fv_kernels.h"
#include "fv_launch_plan.h"

namespace fv {

namespace {

// Reverse sweep of weno5z_pair (fv_physics.h): adds vbm dvm/dv + vbp dvp/dv to g[0..4], the
// cotangents of v = a, b, c, d, e.  The forward steps are those of weno5z_pair with the
// weights written as G_k = 1 + tau / e_k.
__device__ __forceinline__ void weno5z_pair_vjp(double a, double b, double c, double d, double e, double eps,
                                                double vbm, double vbp, double* g)
{
    const double k13 = 13.0 / 12.0;
    const double d1 = b - a, d2 = c - b, d3 = d - c, d4 = e - d;
    const double t0 = d2 - d1, t1 = d3 - d2, t2 = d4 - d3;
    const double h0 = fma(0.5, t0, d2), h2 = fma(-0.5, t2, d3), x = d2 + d3;
    const double e0 = fma(h0, h0, weno5z_curvature(t0, eps)), e1 = fma(0.25 * x, x, weno5z_curvature(t1, eps));
    const double e2 = fma(h2, h2, weno5z_curvature(t2, eps));
    const double diff = e0 - e2, tau = ::fabs(diff);
    const double p01 = e0 * e1, R = rcp(p01 * e2), t = e2 * R;
    const double r0 = e1 * t, r1 = e0 * t, r2 = p01 * R;
    const double G0 = fma(tau, r0, 1.0), G1 = fma(tau, r1, 1.0), G2 = fma(tau, r2, 1.0);
    // + face: v_i + N / D with candidates q0, q1, q2; - face: the mirror image (u0, u1, u2)
    const double third = 1.0 / 3.0;
    const double q0 = fma(2.5, d2, -d1), q1 = fma(2.0, d3, d2), q2 = fma(-0.5, d4, 2.0 * d3);
    const double u0 = fma(-2.5, d3, d4), u1 = -fma(2.0, d2, d3), u2 = fma(0.5, d1, -2.0 * d2);
    const double im = rcp(fma(3.0, G2, fma(6.0, G1, G0))), ip = rcp(fma(3.0, G0, fma(6.0, G1, G2)));
    const double nm = vbm * im, np = vbp * ip;  // cotangents of the numerators
    const double dm = -nm * im * fma(third * G0, q0, fma(G1, q1, G2 * q2));  // and of the denominators
    const double dp = -np * ip * fma(third * G2, u0, fma(G1, u1, G0 * u2));
    const double b0 = fma(third * nm, q0, dm) + fma(np, u2, 3.0 * dp);
    const double b1 = fma(nm, q1, 6.0 * dm) + fma(np, u1, 6.0 * dp);
    const double b2 = fma(nm, q2, 3.0 * dm) + fma(third * np, u0, dp);
    const double qb0 = third * nm * G0, qb1 = nm * G1, qb2 = nm * G2;
    const double ub0 = third * np * G2, ub1 = np * G1, ub2 = np * G0;
    double db1 = fma(0.5, ub2, -qb0), db4 = fma(-0.5, qb2, ub0);
    double db2 = fma(2.5, qb0, qb1) - 2.0 * (ub1 + ub2);
    double db3 = 2.0 * (qb1 + qb2) - fma(2.5, ub0, ub1);
    // G_k = 1 + tau / e_k, tau = |e0 - e2|
    const double taub = fma(b0, r0, fma(b1, r1, b2 * r2));
    const double sg = diff > 0.0 ? taub : (diff < 0.0 ? -taub : 0.0);
    const double eb0 = fma(-b0 * tau * r0, r0, sg), eb1 = -b1 * tau * r1 * r1, eb2 = fma(-b2 * tau * r2, r2, -sg);
    // e_k = 13/12 t_k^2 + (its first-difference term)^2 + eps
    const double hb0 = 2.0 * h0 * eb0, hb2 = 2.0 * h2 * eb2, xb = 0.5 * x * eb1;
    const double tb0 = fma(2.0 * k13 * t0, eb0, 0.5 * hb0), tb1 = 2.0 * k13 * t1 * eb1;
    const double tb2 = fma(2.0 * k13 * t2, eb2, -0.5 * hb2);
    db1 -= tb0;
    db2 += hb0 + xb + tb0 - tb1;
    db3 += hb2 + xb + tb1 - tb2;
    db4 += tb2;
    g[0] -= db1;
    g[1] += db1 - db2;
    g[2] += db2 - db3 + (vbm + vbp);
    g[3] += db3 - db4;
    g[4] += db4;
}

// Reverse sweep of the single-phase U -> W map: Ub = (dW/dU)^T Wb.
__device__ __forceinline__ void cons_to_prim_vjp(const Material<double>& mat, const double* w, const double* wb,
                                                 double* ub)
{
    const double ir = rcp(w[0]);
    const double gm1 = mat.gm1;
    const double ke = 0.5 * (w[1] * w[1] + w[2] * w[2] + w[3] * w[3]);
    ub[0] = wb[0] - (wb[1] * w[1] + wb[2] * w[2] + wb[3] * w[3]) * ir + wb[4] * gm1 * ke;
#pragma unroll
    for (int i = 0; i < 3; i++) ub[1 + i] = wb[1 + i] * ir - wb[4] * gm1 * w[1 + i];
    ub[4] = wb[4] * gm1;
}

// Reverse sweep of one star-side flux of hllc (hllc_side in fv_physics.h, single-phase
// layout): G is the cotangent of that side's flux; adds G . dF/dw to wb and returns the
// cotangents of the side's wave speed sK, its upwind factor sw and s*.
template <int DIR>
__device__ __forceinline__ void hllc_side_vjp(const Material<double>& mat, const double* w, double sK, double sw,
                                              double sstar, const double* G, double* wb, double& sKb, double& swb,
                                              double& sstarb)
{
    constexpr int V = 1, P = 4;
    const double rho = w[0], un = w[V + DIR], p = w[P];
    const double r = rcp(sK - sstar);
    const double fac = (sK - un) * r;
    const double q = un + sw * (fac - 1.0);
    const double v2 = w[V] * w[V] + w[V + 1] * w[V + 1] + w[V + 2] * w[V + 2];
    const double E = (p + mat.gpinf) * mat.iG1 + 0.5 * rho * v2;
    const double ds = sstar - un;
    const double Estar = fac * (E + ds * rho * sstar) + ds * p * r;
    const double Gn = G[V + DIR], Ge = G[P];
    // F[0] = rho q; tangential momenta rho u_t q
    double qb = G[0] * rho, rhob = G[0] * q;
#pragma unroll
    for (int m = 0; m < 3; m++) {
        if (m == DIR) continue;
        rhob += G[V + m] * w[V + m] * q;
        wb[V + m] += G[V + m] * rho * q;
        qb += G[V + m] * rho * w[V + m];
    }
    // normal momentum rho un^2 + p + sw (fac rho s* - rho un)
    rhob += Gn * (un * un + sw * (fac * sstar - un));
    double unb = Gn * (2.0 * rho * un - sw * rho);
    double pb = Gn;
    swb = Gn * (fac * rho * sstar - rho * un);
    double facb = Gn * sw * rho * sstar;
    sstarb = Gn * sw * fac * rho;
    // energy un (E + p) + sw (E* - E), E* = fac (E + ds rho s*) + ds p r
    unb += Ge * (E + p);
    double Eb = Ge * (un - sw);
    pb += Ge * un;
    swb += Ge * (Estar - E);
    const double Esb = Ge * sw;
    facb += Esb * (E + ds * rho * sstar);
    Eb += Esb * fac;
    const double dsb = Esb * (fac * rho * sstar + p * r);
    rhob += Esb * fac * ds * sstar;
    sstarb += Esb * fac * ds * rho;
    pb += Esb * ds * r;
    double rb = Esb * ds * p;
    sstarb += dsb;
    unb -= dsb;
    // E = (p + gpinf) / (gamma - 1) + rho |u|^2 / 2
    pb += Eb * mat.iG1;
    rhob += Eb * 0.5 * v2;
#pragma unroll
    for (int m = 0; m < 3; m++) wb[V + m] += Eb * rho * w[V + m];
    // q = un + sw (fac - 1); fac = (sK - un) r; r = 1 / (sK - s*)
    unb += qb;
    swb += qb * (fac - 1.0);
    facb += qb * sw;
    sKb = facb * r;
    unb -= facb * r;
    rb += facb * (sK - un);
    const double dKb = -rb * r * r;
    sKb += dKb;
    sstarb -= dKb;
    wb[0] += rhob;
    wb[V + DIR] += unb;
    wb[P] += pb;
}

// Reverse sweep of hllc<double, EULER, DIR> (fv_physics.h): adds g . dF/d(wl, wr) to
// wlb, wrb, the flux recomputed once and pulled back step by step in reverse order
// (s* = 0 averages the two star-side fluxes, so both are pulled back with half the
// cotangent).  Replaces ten forward-mode tangent evaluations of the flux (one per
// face-state input): the RHS adjoint at 64^3 took 0.25 against 0.34 ms.
template <int DIR>
__device__ __forceinline__ void hllc_vjp(const Material<double>& mat, const double* wl, const double* wr,
                                         const double* g, double* wlb, double* wrb)
{
    constexpr int V = 1, P = 4, NC = 5;
    // forward
    const double rhoL = wl[0], rhoR = wr[0], uL = wl[V + DIR], uR = wr[V + DIR], pL = wl[P], pR = wr[P];
    const double yL = rsqrt(rhoL), yR = rsqrt(rhoR);
    const double sqL = rhoL * yL, sqR = rhoR * yR;
    const double rc2L = mat.gamma * (pL + mat.pinf), rc2R = mat.gamma * (pR + mat.pinf);
    const double c2L = rc2L * (yL * yL), c2R = rc2R * (yR * yR);
    const double srL = sqrt_fast(rc2L), srR = sqrt_fast(rc2R);
    const double cL = srL * yL, cR = srR * yR;
    const double isum = rcp(sqL + sqR);
    const double ubar = (sqL * uL + sqR * uR) * isum;
    const double du = uR - uL;
    const double A = sqL * c2L + sqR * c2R;
    const double cbar2 = A * isum + 0.5 * sqL * sqR * isum * isum * du * du;
    const double cbar = sqrt_fast(cbar2);
    const double aL = ubar - cbar, bL = uL - cL, aR = ubar + cbar, bR = uR + cR;
    const double sL = ::fmin(aL, bL), sR = ::fmax(aR, bR);
    const double mL = rhoL * (sL - uL), mR = rhoR * (sR - uR);
    const double num = (pR - pL) + (mL * uL - mR * uR);
    const double rd = rcp(mL - mR);
    const double sstar = num * rd;
    const double sminus = ::fmin(0.0, sL), splus = ::fmax(0.0, sR);
    // star-side flux of the upwind side, chosen by operand selection as in the forward; both
    // sides with half the cotangent where s* = 0
    const bool left = !(sstar < 0.0), both = sstar == 0.0;
    double ws[NC], gs[NC], wsb[NC];
#pragma unroll
    for (int m = 0; m < NC; m++) {
        ws[m] = left ? wl[m] : wr[m];
        gs[m] = both ? 0.5 * g[m] : g[m];
        wsb[m] = 0.0;
    }
    double sKb, swb, sstarb;
    hllc_side_vjp<DIR>(mat, ws, left ? sL : sR, left ? sminus : splus, sstar, gs, wsb, sKb, swb, sstarb);
    double sLb = left ? sKb : 0.0, sRb = left ? 0.0 : sKb, smb = left ? swb : 0.0, spb = left ? 0.0 : swb;
#pragma unroll
    for (int m = 0; m < NC; m++) {
        wlb[m] += left ? wsb[m] : 0.0;
        wrb[m] += left ? 0.0 : wsb[m];
    }
    if (both) {
        double sb;
        hllc_side_vjp<DIR>(mat, wr, sR, splus, sstar, gs, wrb, sRb, spb, sb);
        sstarb += sb;
    }
    // s^- = min(0, sL), s^+ = max(0, sR)
    sLb += smb * (sL < 0.0 ? 1.0 : (sL == 0.0 ? 0.5 : 0.0));
    sRb += spb * (sR > 0.0 ? 1.0 : (sR == 0.0 ? 0.5 : 0.0));
    // s* = ((pR - pL) + mL uL - mR uR) / (mL - mR)
    const double numb = sstarb * rd;
    const double denb = -sstarb * num * rd * rd;
    double pLb = -numb, pRb = numb;
    const double mLb = numb * uL + denb, mRb = -numb * uR - denb;
    double uLb = numb * mL, uRb = -numb * mR;
    // m_K = rho_K (s_K - u_K)
    double rhoLb = mLb * (sL - uL), rhoRb = mRb * (sR - uR);
    sLb += mLb * rhoL;
    uLb -= mLb * rhoL;
    sRb += mRb * rhoR;
    uRb -= mRb * rhoR;
    // sL = min(ubar - cbar, uL - cL), sR = max(ubar + cbar, uR + cR)
    const double kL = aL < bL ? 1.0 : (bL < aL ? 0.0 : 0.5);
    const double kR = aR > bR ? 1.0 : (bR > aR ? 0.0 : 0.5);
    const double aLb = sLb * kL, bLb = sLb * (1.0 - kL), aRb = sRb * kR, bRb = sRb * (1.0 - kR);
    const double ubarb = aLb + aRb, cbarb = aRb - aLb;
    uLb += bLb;
    uRb += bRb;
    const double cLb = -bLb, cRb = bRb;
    // cbar = sqrt(cbar2), cbar2 = A isum + sqL sqR isum^2 du^2 / 2
    const double c2b = cbarb * 0.5 * rsqrt(cbar2);
    const double t = 0.5 * isum * isum * du * du;
    double sqLb = c2b * (sqR * t + c2L * isum), sqRb = c2b * (sqL * t + c2R * isum);
    double isumb = c2b * (A + sqL * sqR * isum * du * du);
    const double dub = c2b * sqL * sqR * isum * isum * du;
    const double c2Lb = c2b * isum * sqL, c2Rb = c2b * isum * sqR;
    uRb += dub;
    uLb -= dub;
    // ubar = (sqL uL + sqR uR) isum
    sqLb += ubarb * uL * isum;
    sqRb += ubarb * uR * isum;
    uLb += ubarb * sqL * isum;
    uRb += ubarb * sqR * isum;
    isumb += ubarb * (sqL * uL + sqR * uR);
    // isum = 1 / (sqL + sqR)
    const double ssb = -isumb * isum * isum;
    sqLb += ssb;
    sqRb += ssb;
    // c_K = sqrt(rc2_K) y_K, c2_K = rc2_K y_K^2, sq_K = rho_K y_K, y_K = rho_K^-1/2
    const double rc2Lb = cLb * yL * 0.5 * rsqrt(rc2L) + c2Lb * yL * yL;
    const double rc2Rb = cRb * yR * 0.5 * rsqrt(rc2R) + c2Rb * yR * yR;
    const double yLb = cLb * srL + c2Lb * 2.0 * rc2L * yL + sqLb * rhoL;
    const double yRb = cRb * srR + c2Rb * 2.0 * rc2R * yR + sqRb * rhoR;
    rhoLb += sqLb * yL - 0.5 * yLb * yL * yL * yL;
    rhoRb += sqRb * yR - 0.5 * yRb * yR * yR * yR;
    pLb += rc2Lb * mat.gamma;
    pRb += rc2Rb * mat.gamma;
    wlb[0] += rhoLb;
    wlb[V + DIR] += uLb;
    wlb[P] += pLb;
    wrb[0] += rhoRb;
    wrb[V + DIR] += uRb;
    wrb[P] += pRb;
}

// ---- the right-hand side's adjoint.  A workgroup owns LN lines along one direction and,
// of each, the cells [i0, i1); thread (line, slot) holds the line position p = i0 - 3 + slot
// (a position may lie outside the domain: it is mapped by the boundary conditions) and
// works in turn on
//   cell p   conversion to primitive variables (staged in LDS, two more positions on
//            either side) and both WENO5-Z values of the cell;
//   face p   (between p - 1 and p) the reverse sweep of HLLC with the face's cotangent,
//            in place of the two face states;
//   cell p   the reverse sweep of its reconstruction: cotangents of positions p-2 .. p+2,
//            collected across the threads through LDS;
//   cell p   the cotangents of halo positions added to the cells they mirror, the reverse
//            sweep of U -> W, and the sum into Ubar.
// A periodic line that fits a workgroup, and any line of one cell, closes on itself
// (positions 0 .. n-1, no halo).
// What bounds it: the latency of that chain (~1700 vector instructions) at three waves per
// SIMD.  A thread per face, which rebuilt ten cell reconstructions and added 30 values with
// atomics at one wave per SIMD, took 214 us per right-hand side at 64^3; this takes 69
// (24^3: 12).  Measured for the 5-step gradient at 64^3 / 24^3: 256 threads at three
// waves per SIMD 2.29 / 1.44 ms, at four (spills) 2.54 / 1.47, 512 threads at four 2.45 /
// 1.51, 128 threads at three 2.75 / 1.47.  One launch for the three directions, meeting in
// five atomic additions per cell and direction, against three launches that add without
// atomics: 2.45 against 2.62 ms, at 24^3 1.51 against 1.98, at 128^3 equal within 1 %.
struct AdjointLds {
    // primitive states of the slots and, in pieces of a line, of two more positions on
    // either side (4 lines <= ADJ_NT / 2 entries: a piece has at least 8 slots)
    double W[5][ADJ_NT + ADJ_NT / 2];
    // face states, then their cotangents, then the exchanged cotangents of neighbouring cells
    double X[10][ADJ_NT];
};

template <int DIR>
__device__ __forceinline__ void rhs_adjoint_body(AdjointLds& lds, const AdjointArgs& a, const AdjointSplit& sp,
                                                 unsigned block,
                                                 const double* __restrict__ U, const double* __restrict__ Rbar,
                                                 double* __restrict__ Ubar, const double scale)
{
    constexpr int NC = 5, V = 1;
    const double ih = (DIR == 0 ? a.idx : (DIR == 1 ? a.idy : a.idz)) * scale;
    auto& W = lds.W;
    auto& X = lds.X;
    const int n = DIR == 0 ? a.nx : (DIR == 1 ? a.ny : a.nz);
    const int SL = sp.slots, LN = sp.lines;
    const bool periodic = sp.closed || a.bc[2 * DIR] == PERIODIC;
    const int tid = threadIdx.x;
    // (slot, line): along x the slots are consecutive in memory, else the lines are
    const int slot = DIR == 0 ? tid % SL : tid / LN, ln = DIR == 0 ? tid / SL : tid % LN;
    const bool active = DIR == 0 ? ln < LN : slot < SL;
    // lines < 2^32: a state of that many cells would not fit the memory
    const unsigned nx = (unsigned)a.nx;
    const unsigned nlines = DIR == 0 ? (unsigned)a.ny * (unsigned)a.nz : nx * (unsigned)(DIR == 1 ? a.nz : a.ny);
    unsigned piece = 0;
    if (sp.pieces > 1) {
        piece = block % (unsigned)sp.pieces;
        block /= (unsigned)sp.pieces;
    }
    const unsigned line = block * (unsigned)LN + (unsigned)ln;
    const bool on = active && line < nlines;
    // equal pieces: the first `longer` ones have a cell more
    const int len = n / sp.pieces, longer = n - len * sp.pieces;
    const int i0 = len * (int)piece + min((int)piece, longer), i1 = i0 + len + ((int)piece < longer ? 1 : 0);
    const int p0 = sp.closed ? 0 : i0 - 3;
    const int p = p0 + slot;
    // cell 0 of the line and the stride along it
    long long base, stride;
    if (DIR == 0) {
        base = (long long)line * n;
        stride = 1;
    } else if (DIR == 1) {
        const unsigned k = line / nx;
        base = (long long)k * a.ny * a.nx + (line - k * nx);
        stride = a.nx;
    } else {
        base = line;
        stride = (long long)a.nx * a.ny;
    }
    const Material<double> mat = a.mat;
    auto at = [&](int s) { return DIR == 0 ? ln * SL + s : s * LN + ln; };          // X entry of a slot
    const int SR = sp.closed ? SL : SL + 4;                                         // staged positions
    auto row = [&](int r) { return DIR == 0 ? ln * SR + r : r * LN + ln; };         // W entry of a staged position
    auto wrap = [&](int s) {  // slots -2 .. SL + 1 of a closed line (of one cell or more)
        s += s < 0 ? SL : 0;
        s += s < 0 ? SL : 0;
        s -= s >= SL ? SL : 0;
        return s >= SL ? s - SL : s;
    };

    // ---- loads, all issued before the first is used: the state at the position and, for the
    // first four slots of a piece, at one of the four positions beyond its slots; Rbar of the
    // two cells of the face below p (in bounds for every thread, set to zero where the face
    // or the cell does not exist)
    double u[NC], uh[NC], rl[NC], rr[NC], g[NC];
    bool fl = false, flh = false;
    const bool second = SL + slot < SR;
    if (on) {
        const long long q = base + map_index(sp.closed ? slot : i0 - 5 + slot, n, a.bc[2 * DIR], a.bc[2 * DIR + 1], fl) * stride;
        const long long qh =
            second ? base + map_index(i0 - 5 + SL + slot, n, a.bc[2 * DIR], a.bc[2 * DIR + 1], flh) * stride : q;
        int lo = p - 1, hi = p;
        if (periodic) {
            lo += lo < 0 ? n : 0;  // p - 1 >= -1, or n > ADJ_CELLS + 7
            hi += hi < 0 ? n : 0;
            lo -= lo >= n ? n : 0;
            hi -= hi >= n ? n : 0;
        }
        const long long ql = base + min(max(lo, 0), n - 1) * stride, qr = base + min(max(hi, 0), n - 1) * stride;
#pragma unroll
        for (int m = 0; m < NC; m++) u[m] = U[m * a.ncell + q];
        if (second)
#pragma unroll
            for (int m = 0; m < NC; m++) uh[m] = U[m * a.ncell + qh];
#pragma unroll
        for (int m = 0; m < NC; m++) {
            rl[m] = Rbar[m * a.ncell + ql];
            rr[m] = Rbar[m * a.ncell + qr];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // faces -1 and below, n + 1 and above of a line with boundaries have no cotangent
    const bool face = on && (sp.closed || slot > 0) && (periodic || (p >= 0 && p <= n));
    auto stage = [&](int r, double* v, bool flip) {
        if (flip) v[V + DIR] = -v[V + DIR];
        double w[NC];
        cons_to_prim<double, EULER>(mat, v, w);
#pragma unroll
        for (int m = 0; m < NC; m++) W[m][row(r)] = w[m];
    };
    if (on) {
        stage(slot, u, fl);
        if (second) stage(SL + slot, uh, flh);
#pragma unroll
        for (int m = 0; m < NC; m++) {
            const double v = (periodic || p < n ? rr[m] : 0.0) - (periodic || p >= 1 ? rl[m] : 0.0);
            g[m] = v * ih;
        }
    }
    __syncthreads();
    // the five staged positions around the thread's
    int r5[5];
#pragma unroll
    for (int k = 0; k < 5; k++) {
        r5[k] = row(sp.closed ? wrap(slot + k - 2) : slot + k);
    }
    // ---- both reconstructed values of the cell: X[m] the one at its + face, X[5 + m] at its - face
    if (on) {
#pragma unroll
        for (int m = 0; m < NC; m++) {
            double vm, vp;
            weno5z_pair(W[m][r5[0]], W[m][r5[1]], W[m][r5[2]], W[m][r5[3]], W[m][r5[4]], a.weps, vm, vp);
            X[m][at(slot)] = vm;
            X[NC + m][at(slot)] = vp;
        }
    }
    __syncthreads();
    // ---- the face's states replaced by their cotangents (each is read by this thread only)
    if (on && (sp.closed || slot > 0)) {
        const int el = at(sp.closed ? wrap(slot - 1) : slot - 1), er = at(slot);
        double wlb[NC], wrb[NC];
#pragma unroll
        for (int m = 0; m < NC; m++) wlb[m] = wrb[m] = 0.0;
        if (face) {
            double wl[NC], wr[NC];
#pragma unroll
            for (int m = 0; m < NC; m++) {
                wl[m] = X[m][el];
                wr[m] = X[NC + m][er];
            }
            hllc_vjp<DIR>(mat, wl, wr, g, wlb, wrb);
        }
#pragma unroll
        for (int m = 0; m < NC; m++) {
            X[m][el] = wlb[m];
            X[NC + m][er] = wrb[m];
        }
    }
    __syncthreads();
    // ---- reverse sweep of the cell's reconstruction, and the cotangent of the position
    const bool cell = on && (sp.closed || (slot > 0 && slot < SL - 1));
    double cm[NC], cp[NC], wb[NC];
#pragma unroll
    for (int m = 0; m < NC; m++) {
        cm[m] = cell ? X[m][at(slot)] : 0.0;
        cp[m] = cell ? X[NC + m][at(slot)] : 0.0;
        wb[m] = 0.0;
    }
    // the exchange needs four of the ten arrays per component: two components at a time
    // (the position's own share stays in a register)
    constexpr int K4[4] = {0, 1, 3, 4};
    auto nb = [&](int k) {  // entry of the cell whose k-th cotangent belongs to this position
        const int s = sp.closed ? wrap(slot + 2 - k) : slot + 2 - k;
        return s >= 0 && s < SL ? at(s) : -1;
    };
#pragma unroll
    for (int m0 = 0; m0 < NC; m0 += 2) {
        __syncthreads();  // the arrays' last readers are done
#pragma unroll
        for (int m = m0; m < m0 + 2 && m < NC; m++) {
            double gs[5] = {0, 0, 0, 0, 0};
            if (cell)
                weno5z_pair_vjp(W[m][r5[0]], W[m][r5[1]], W[m][r5[2]], W[m][r5[3]], W[m][r5[4]], a.weps, cm[m], cp[m], gs);
            wb[m] = gs[2];
            if (on)
#pragma unroll
                for (int k = 0; k < 4; k++) X[4 * (m - m0) + k][at(slot)] = gs[K4[k]];
        }
        __syncthreads();
        if (on)
#pragma unroll
            for (int m = m0; m < m0 + 2 && m < NC; m++)
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const int e = nb(K4[k]);
                    if (e >= 0) wb[m] += X[4 * (m - m0) + k][e];
                }
    }
    // ---- halo positions of a boundary (not periodic): added to the cell they mirror
    if (!periodic && (i0 == 0 || i1 == n)) {  // uniform
        __syncthreads();
        if (on)
#pragma unroll
            for (int m = 0; m < NC; m++) X[m][at(slot)] = wb[m];
        __syncthreads();
        if (on && p >= i0 && p < i1) {
#pragma unroll
            for (int side = 0; side < 2; side++) {
                if (side == 0 ? i0 != 0 : i1 != n) continue;
                for (int h = 0; h < 3; h++) {
                    const int q = side == 0 ? -1 - h : n + h;
                    bool fl = false;
                    if (map_index(q, n, a.bc[2 * DIR], a.bc[2 * DIR + 1], fl) != p) continue;
#pragma unroll
                    for (int m = 0; m < NC; m++) {
                        const double v = X[m][at(q - p0)];
                        wb[m] += fl && m == V + DIR ? -v : v;
                    }
                }
            }
        }
    }
    // ---- U -> W, summed over the directions
    if (on && p >= i0 && p < i1) {
        double w[NC], ub[NC];
        const int rc = r5[2];
#pragma unroll
        for (int m = 0; m < NC; m++) w[m] = W[m][rc];
        cons_to_prim_vjp(mat, w, wb, ub);
        const long long q = base + p * stride;
#pragma unroll
        for (int m = 0; m < NC; m++) {
            atomicAdd(&Ubar[m * a.ncell + q], ub[m]);
        }
    }
}

// the three directions in one launch: blocks [0, b1) take x, [b1, b2) y, the rest z; the
// launch covers the blocks from `base` on
__global__ void __launch_bounds__(ADJ_NT, 3) rhs_adjoint_all(const AdjointArgs a, const AdjointSplit sx,
                                                            const AdjointSplit sy, const AdjointSplit sz,
                                                            const unsigned b1, const unsigned b2, const unsigned base,
                                                            const double* __restrict__ U,
                                                            const double* __restrict__ Rbar,
                                                            double* __restrict__ Ubar, const double scale)
{
    __shared__ AdjointLds lds;
    const unsigned b = base + blockIdx.x;
    if (b < b1) rhs_adjoint_body<0>(lds, a, sx, b, U, Rbar, Ubar, scale);
    else if (b < b2) rhs_adjoint_body<1>(lds, a, sy, b - b1, U, Rbar, Ubar, scale);
    else rhs_adjoint_body<2>(lds, a, sz, b - b2, U, Rbar, Ubar, scale);
}

// out = c0 x0 + c1 x1 + c2 x2 (null terms are skipped); out may alias an input
__global__ void lincomb_kernel(double* out, long long n, double c0, const double* x0, double c1, const double* x1,
                               double c2, const double* x2)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        double v = x0 ? c0 * x0[i] : 0.0;
        if (x1) v += c1 * x1[i];
        if (x2) v += c2 * x2[i];
        out[i] = v;
    }
}

int grid_for(long long n, int threads)
{
    long long b = (n + threads - 1) / threads;
    return (int)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

}  // namespace

hipError_t launch_rhs_adjoint(const AdjointArgs& a, const double* U, const double* Rbar, double* Ubar, double scale,
                              hipStream_t st)
{
    const int n3[3] = {a.nx, a.ny, a.nz};
    AdjointSplit sp[3];
    long long end[3], total = 0;
    for (int d = 0; d < 3; d++) {
        sp[d] = adjoint_split(n3[d], a.bc[2 * d] == PERIODIC);
        end[d] = total += adjoint_blocks(sp[d], a.ncell / n3[d]);
    }
    // the kernel's 32-bit line and block numbers: more would not fit the memory
    if (total > 0xffffffffll || a.ncell / n3[0] > 0xffffffffll || a.ncell / n3[1] > 0xffffffffll ||
        a.ncell / n3[2] > 0xffffffffll)
        return hipErrorInvalidValue;
    // one launch, but for the largest grids (1024^3: 3 x 5592416 workgroups)
    for (long long base = 0; base < total; base += max_blocks(ADJ_NT)) {
        const long long nb = total - base < max_blocks(ADJ_NT) ? total - base : max_blocks(ADJ_NT);
        hipLaunchKernelGGL(rhs_adjoint_all, dim3((unsigned)nb), dim3(ADJ_NT), 0, st, a, sp[0], sp[1], sp[2],
                           (unsigned)end[0], (unsigned)end[1], (unsigned)base, U, Rbar, Ubar, scale);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_lincomb(double* out, long long n, double c0, const double* x0, double c1, const double* x1, double c2,
                          const double* x2, hipStream_t st)
{
    hipLaunchKernelGGL(lincomb_kernel, dim3(grid_for(n, 256)), dim3(256), 0, st, out, n, c0, x0, c1, x1, c2, x2);
    return hipGetLastError();
}

}  // namespace fv

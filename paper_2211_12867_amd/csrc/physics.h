// physics.h -- pointwise ideal-MHD physics for the kernels (fp64).
//
// Variables: conserved u = (rho, m0, m1, m2, E, B0, B1, B2), primitive
// w = (rho, v0, v1, v2, p, B0, B1, B2), mu0 = 1, E = p/(g-1) + rho v^2/2 + B^2/2.
// NV = 9 adds the CME density tracer: conserved rho s, primitive s (the CME
// mass fraction), advected with the flow by the same flux (no source).
// Direction 0/1/2 = r/theta/phi (x/y/z in the cartesian test geometry).
#pragma once
#include <hip/hip_runtime.h>

#define DEV __device__ __forceinline__

// The hardware's estimates of 1/a and 1/sqrt(x) are off by less than 2^-24
// (relative; measured over 4 million values).  An error of one ulp below is
// that of the result's own binade.

// Reciprocal of a > 0 (normal): the estimate x and one step of third order,
// x (1 + e + e^2) with e = 1 - a x (one operation less than two Newton steps);
// at most 0.51 ulp from 1/a.
DEV double rcp_pos(double a)
{
    const double x = __builtin_amdgcn_rcp(a);
    const double e = fma(-a, x, 1.0);
    return fma(x, fma(e, e, e), x);
}

// Square root of x > 0 (normal): g = x y from the estimate y of 1/sqrt(x) and
// two Newton steps g + (x - g^2) y / 2, whose residuals carry no rounding of g;
// at most 0.51 ulp from sqrt(x).
DEV double sqrt_pos(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * y;
    double g = x * y;
    g = fma(fma(-g, g, x), h, g);
    return fma(fma(-g, g, x), h, g);
}

// sqrt(x / a) for x, a > 0 (normal, their product too): g = x y with y the
// estimate of 1/sqrt(a x), e = 1 - a g y from g as rounded, and one step of
// third order g (1 + e/2 + 3 e^2/8); half the roundings of g and a g and the
// last one remain, at most 1.5 ulp (1.2 seen).
DEV double sqrt_ratio_pos(double x, double a)
{
    const double y = __builtin_amdgcn_rsq(a * x);
    const double g = x * y, e = fma(-(a * g), y, 1.0);
    return fma(g * e, fma(0.375, e, 0.5), g);
}

// Reciprocals and square roots of the finite-volume update use these;
// IC_EXACT_MATH selects the IEEE-rounded operations.
#ifdef IC_EXACT_MATH
#define IC_RCP(x) (1.0 / (x))
#define IC_SQRT(x) sqrt(x)
#define IC_SQRT_RATIO(x, a) sqrt((x) / (a))
#else
#define IC_RCP(x) rcp_pos(x)
#define IC_SQRT(x) sqrt_pos(x)
#define IC_SQRT_RATIO(x, a) sqrt_ratio_pos(x, a)
#endif

struct Gas {
    double g;       // adiabatic index
    double gm1;     // g - 1
    double igm1;    // 1 / (g - 1)
};

// EXACT: IEEE division (the refinement indicator and the network features,
// whose threshold decisions are kept on the correctly rounded quotient).  The
// tracer fraction s = (rho s) / rho is always the correctly rounded quotient,
// so that s = 1 where rho s = rho.
template <bool EXACT = false, int NV = 8>
DEV void cons_to_prim(const double *u, double *w, const Gas &gs)
{
    const double ir = EXACT ? 1.0 / u[0] : IC_RCP(u[0]);
    w[0] = u[0];
    w[1] = u[1] * ir;
    w[2] = u[2] * ir;
    w[3] = u[3] * ir;
    const double kin = 0.5 * (u[1] * w[1] + u[2] * w[2] + u[3] * w[3]);
    const double mag = 0.5 * (u[5] * u[5] + u[6] * u[6] + u[7] * u[7]);
    w[4] = gs.gm1 * (u[4] - kin - mag);
    w[5] = u[5];
    w[6] = u[6];
    w[7] = u[7];
    if constexpr (NV > 8) w[8] = u[8] / u[0];
}

template <int NV = 8>
DEV void prim_to_cons(const double *w, double *u, const Gas &gs)
{
    const double v2 = w[1] * w[1] + w[2] * w[2] + w[3] * w[3];
    const double b2 = w[5] * w[5] + w[6] * w[6] + w[7] * w[7];
    u[0] = w[0];
    u[1] = w[0] * w[1];
    u[2] = w[0] * w[2];
    u[3] = w[0] * w[3];
    u[4] = w[4] * gs.igm1 + 0.5 * w[0] * v2 + 0.5 * b2;
    u[5] = w[5];
    u[6] = w[6];
    u[7] = w[7];
    if constexpr (NV > 8) u[8] = w[0] * w[8];
}

// Fast magnetosonic speed from A = g p + B^2, gp4 = 4 g p, the normal field bn
// and twice the density: c_f^2 = (A + S) / (2 rho), S^2 = A^2 - 4 g p bn^2,
// no reciprocal of the density; S is kept off zero by a value that vanishes
// beside A (A > 0 in every physical state).  Mean error 0.39 ulp over plasma
// betas from 0.3 to 30 as from 0.01 to 100; 0.41 to 0.42 in the form with a =
// (g p + B^2) / rho and correctly rounded parts.
DEV double fast_speed_of(double A, double gp4, double bn, double rho2)
{
    const double d = fmax(fma(-gp4, bn * bn, A * A), 1e-300);
    return IC_SQRT_RATIO(A + IC_SQRT(d), rho2);
}

// CFL rate of a cell, sum over the directions of (|v_d| + c_f,d) id (id the
// reciprocal widths).
DEV double cell_rate_of(const double w[8], double ir, double it, double ip, const Gas &gs)
{
    const double b2 = w[5] * w[5] + w[6] * w[6] + w[7] * w[7];
    const double A = fma(gs.g, w[4], b2), gp4 = 4.0 * gs.g * w[4], rho2 = w[0] + w[0];
    return (fabs(w[1]) + fast_speed_of(A, gp4, w[5], rho2)) * ir
         + (fabs(w[2]) + fast_speed_of(A, gp4, w[6], rho2)) * it
         + (fabs(w[3]) + fast_speed_of(A, gp4, w[7], rho2)) * ip;
}

template <int NV = 8>
DEV bool unphysical(const double *w)
{
    // rho <= 0, p <= 0 or NaN (comparisons with NaN are false)
    bool ok = (w[0] > 0.0) && (w[4] > 0.0);
#pragma unroll
    for (int v = 0; v < NV; ++v) ok = ok && (fabs(w[v]) <= 1.7976931348623157e308);
    return !ok;
}

// Local Lax-Friedrichs (Rusanov) flux along D between left state wl and right
// state wr: (F_l + F_r) / 2 - c / 2 (U_r - U_l); with the tracer, its flux
// rho v_n s takes the same maximum speed.  The halves go into the normal
// velocities and fields once, so that each component is one chain of fused
// multiply-adds.
template <int D, int NV = 8>
DEV void rusanov(const double *wl, const double *wr, double *f, const Gas &gs)
{
    const double vl2 = wl[1] * wl[1] + wl[2] * wl[2] + wl[3] * wl[3];
    const double vr2 = wr[1] * wr[1] + wr[2] * wr[2] + wr[3] * wr[3];
    const double bl2 = wl[5] * wl[5] + wl[6] * wl[6] + wl[7] * wl[7];
    const double br2 = wr[5] * wr[5] + wr[6] * wr[6] + wr[7] * wr[7];
    const double ptl = fma(0.5, bl2, wl[4]);
    const double ptr = fma(0.5, br2, wr[4]);
    const double El = fma(wl[4], gs.igm1, fma(0.5 * wl[0], vl2, 0.5 * bl2));
    const double Er = fma(wr[4], gs.igm1, fma(0.5 * wr[0], vr2, 0.5 * br2));
    const double vbl = wl[1] * wl[5] + wl[2] * wl[6] + wl[3] * wl[7];
    const double vbr = wr[1] * wr[5] + wr[2] * wr[6] + wr[3] * wr[7];
    // the larger of the two sides' maximum speeds, halved
    const double g4 = 4.0 * gs.g;
    const double sl = fabs(wl[1 + D]) + fast_speed_of(fma(gs.g, wl[4], bl2), g4 * wl[4], wl[5 + D], wl[0] + wl[0]);
    const double sr = fabs(wr[1 + D]) + fast_speed_of(fma(gs.g, wr[4], br2), g4 * wr[4], wr[5 + D], wr[0] + wr[0]);
    const double c = fmax(sl, sr), hc = 0.5 * c;

    const double hvl = 0.5 * wl[1 + D], hvr = 0.5 * wr[1 + D];
    const double hbl = 0.5 * wl[5 + D], hbr = 0.5 * wr[5 + D];
    const double hml = wl[0] * hvl, hmr = wr[0] * hvr;
    f[0] = fma(-hc, wr[0] - wl[0], hml + hmr);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        double s = fma(-hbr, wr[5 + q], fma(-hbl, wl[5 + q], fma(hmr, wr[1 + q], hml * wl[1 + q])));
        if (q == D) s = fma(0.5, ptl + ptr, s);
        f[1 + q] = q == D ? fma(-c, hmr - hml, s) : fma(-hc, fma(wr[0], wr[1 + q], -(wl[0] * wl[1 + q])), s);
    }
    f[4] = fma(-hc, Er - El, fma(-hbr, vbr, fma(-hbl, vbl, fma(Er + ptr, hvr, (El + ptl) * hvl))));
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const double d = wr[5 + q] - wl[5 + q];
        if (q == D) f[5 + q] = -hc * d;
        else f[5 + q] = fma(-hc, d, fma(-hbr, wr[1 + q], fma(-hbl, wl[1 + q], fma(hvr, wr[5 + q], hvl * wl[5 + q]))));
    }
    if constexpr (NV > 8)
        f[8] = fma(-hc, fma(wr[0], wr[8], -(wl[0] * wl[8])), fma(hmr, wr[8], hml * wl[8]));
}

// Physical ideal-MHD flux of a primitive state along D: rho v_n, rho v_n v -
// B_n B + p_tot e_n, (E + p_tot) v_n - B_n (v.B), v_n B - B_n v (B_n part 0),
// and rho v_n s for the tracer.
template <int D, int NV = 8>
DEV void phys_flux(const double *w, double *f, const Gas &gs)
{
    const double v2 = w[1] * w[1] + w[2] * w[2] + w[3] * w[3];
    const double b2 = w[5] * w[5] + w[6] * w[6] + w[7] * w[7];
    const double pt = w[4] + 0.5 * b2;
    const double E = w[4] * gs.igm1 + 0.5 * w[0] * v2 + 0.5 * b2;
    const double vn = w[1 + D], bn = w[5 + D];
    const double vb = w[1] * w[5] + w[2] * w[6] + w[3] * w[7];
    const double m = w[0] * vn;
    f[0] = m;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        f[1 + q] = m * w[1 + q] - bn * w[5 + q] + (q == D ? pt : 0.0);
        f[5 + q] = q == D ? 0.0 : vn * w[5 + q] - bn * w[1 + q];
    }
    f[4] = (E + pt) * vn - bn * vb;
    if constexpr (NV > 8) f[8] = m * w[8];
}

// Limiters of the reconstruction (the paper's runs use the monotonised-central
// "Woodward" form; its code offers others): zero where the one-sided
// differences differ in sign or one vanishes, else LIM_MC the smallest of
// 2 |dm|, |dc|, 2 |dp| with their sign, LIM_MINMOD the one-sided difference of
// smaller magnitude, LIM_VANLEER their harmonic mean 2 dm dp / (dm + dp).
// dm = (w0 - wm) im, dp = (wp - w0) ip, dc = (wp - wm) ic; im and ip are the
// reciprocal spacings, twice them for LIM_MC (slope_scale).  MC and minmod are
// clamps between 0 and the two differences: minima and maxima alone, no
// comparison, sign copy or select.
enum { LIM_MC = 0, LIM_MINMOD = 1, LIM_VANLEER = 2 };

template <int LIM>
DEV double slope_scale(double id) { return LIM == LIM_MC ? 2.0 * id : id; }

template <int LIM>
DEV double limited_slope(double wm, double w0, double wp, double im, double ip, double ic)
{
    const double dm = (w0 - wm) * im;
    const double dp = (wp - w0) * ip;
    if (LIM == LIM_VANLEER) {
        const double sl = 2.0 * dm * dp * IC_RCP(dm + dp);
        return (dm * dp <= 0.0) ? 0.0 : sl;
    }
    const double up = fmax(fmin(dm, dp), 0.0), dn = fmin(fmax(dm, dp), 0.0);   // one of them is zero
    if (LIM == LIM_MINMOD) return up + dn;
    return fmax(fmin((wp - wm) * ic, up), dn);
}

// Face values of a cell from its neighbours along one direction; falls back to
// zero slope for all variables if a face density or pressure is not positive
// (rare: a branch that no lane takes is skipped).
template <int LIM = LIM_MC, int NV = 8>
DEV void reconstruct(const double *wm, const double *w0, const double *wp, double im,
                     double ip, double ic, double hm, double hp, double *lo, double *hi)
{
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const double s = limited_slope<LIM>(wm[v], w0[v], wp[v], im, ip, ic);
        lo[v] = fma(-s, hm, w0[v]);
        hi[v] = fma(s, hp, w0[v]);
    }
    const bool ok = lo[0] > 0.0 && hi[0] > 0.0 && lo[4] > 0.0 && hi[4] > 0.0;
    if (!ok)
#pragma unroll
        for (int v = 0; v < NV; ++v) lo[v] = hi[v] = w0[v];
}

// Geometric (hoop), frame (Coriolis, centrifugal) and gravity sources of a
// cell in spherical geometry, added to acc.  Per cell: rt = 1/r and ctil = cot
// theta in finite-volume form, s2 = 2 omega sin, c2 = 2 omega cos (theta), and
// the accelerations at rest gr = omega^2 r sin^2 - G M / r^2 and gt = omega^2 r
// sin cos.
DEV void add_sources(const double w[8], double rt, double ctil, double s2, double c2, double gr, double gt,
                     double acc[8])
{
    const double vr = w[1], vt = w[2], vp = w[3];
    const double br = w[5], bt = w[6], bp = w[7];
    const double mr = w[0] * vr, mt = w[0] * vt, mp = w[0] * vp;
    const double pp = fma(mp, vp, -(bp * bp));           // rho v_p^2 - B_p^2
    const double tt = fma(mt, vt, -(bt * bt));
    const double ptot = fma(0.5, br * br + bt * bt + bp * bp, w[4]);
    acc[1] += rt * (pp + tt + 2.0 * ptot) + fma(s2, mp, w[0] * gr);
    acc[2] += rt * (ctil * (pp + ptot) - fma(mr, vt, -(br * bt))) + fma(c2, mp, w[0] * gt);
    acc[3] -= rt * (fma(mp, vr, -(bp * br)) + ctil * fma(mp, vt, -(bp * bt))) + fma(s2, mr, c2 * mt);
    acc[4] += fma(mr, gr, mt * gt);
    const double rp = vp * br - bp * vr;
    acc[6] += rt * (vr * bt - vt * br);
    acc[7] -= rt * (rp + ctil * (vp * bt - bp * vt));
}

// Small-value floors on a conserved state: density first (a cell below the
// density floor takes it at zero velocity), then pressure (energy raised); the
// tracer's rho s is left as it is.  Returns which floors acted: bit 0
// density, bit 1 pressure.
DEV int apply_floors(double u[8], const Gas &gs, double rho_min, double p_min)
{
    int fired = 0;
    if (u[0] < rho_min) {
        u[0] = rho_min;
        u[1] = 0.0;
        u[2] = 0.0;
        u[3] = 0.0;
        fired = 1;
    }
    const double kin = 0.5 * (u[1] * u[1] + u[2] * u[2] + u[3] * u[3]) * IC_RCP(u[0]);
    const double mag = 0.5 * (u[5] * u[5] + u[6] * u[6] + u[7] * u[7]);
    const double p = gs.gm1 * (u[4] - kin - mag);
    if (p < p_min) {
        u[4] = p_min * gs.igm1 + kin + mag;
        fired |= 2;
    }
    return fired;
}

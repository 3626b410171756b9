// FMM matrix-vector product of the direct BIE (Eq. dbem4) on one GPU, FP64 path.
//
// The product y = 1/2 x + L[sigma] + M[mu] at the element centroids, with single-layer density
// sigma = -i k beta x and double-layer density mu = x, is split as in Section 3.3:
//   near  : pairs closer than r_c (and the self pair) use accurate integrals, stored once per
//           (mesh, k) in a CSR table; all other pairs in neighbouring leaves use the one-point
//           rule, evaluated on the fly (P2P);
//   far   : boxes that are well separated exchange multipole/local expansions of Eq. (shft0):
//           P2M at the leaves, M2M up, M2L across, L2L down, L2P at the leaves.  Every
//           translation is rotation - coaxial translation - back-rotation (Section 3.3); the
//           coaxial coefficients come from the stabilised recursion, the rotations from the
//           quarter-turn matrices Delta^n (tables.hip).
//
// Expansion conventions (what the tables and the kernels below share):
//   G(x,y) = i k sum_{n,m} R_n^{-m}(y - C) S_n^m(x - C),  |x - C| > |y - C|,
//   multipole of a box: psi(x) = sum C_n^m S_n^m(x - C); local: psi(x) = sum D_n^m R_n^m(x - C).
//   Y_n^m orthonormal with P_n^|m| without the Condon-Shortley phase (Y_n^{-m} = conj Y_n^m).
// Rotation to align t = |t|(sin b cos a, sin b sin a, cos b) with +z, on a coefficient column c:
//   c <- e^{i m a} (-i)^m c ;  c <- Delta^T c ;  c <- e^{i m b} c ;  c <- Delta c ;  [ * i^m ]
// and back after the coaxial step:
//   [ * (-i)^m ] ;  d <- Delta^T d ;  d <- e^{-i m b} d ;  d <- Delta d ;  d <- i^m e^{-i m a} d.
// The bracketed phases cancel across the coaxial step (which is diagonal in m) and are omitted.
#include "internal.h"

namespace fmm {

__constant__ double GL8X[8] = {-0.96028985649753618, -0.79666647741362673, -0.52553240991632899,
                               -0.18343464249564978, 0.18343464249564978,  0.52553240991632899,
                               0.79666647741362673,  0.96028985649753618};
__constant__ double GL8W[8] = {0.10122853629037669, 0.22238103445337434, 0.31370664587788705,
                               0.36268378337836177, 0.36268378337836177, 0.31370664587788705,
                               0.22238103445337434, 0.10122853629037669};

// sin and cos of x for |x| <= 1e5 (k r of element pairs): x = q pi/2 + y with pi/2 split in two
// parts (Cody-Waite), |y| <= pi/4, then the Taylor polynomials of sin y through y^17 and of cos y
// through y^16 (truncation below 1e-17); the absolute error is a few 1e-16.  Larger arguments use
// the library routine.
__device__ inline void sincos_red(double x, double &s, double &c) {
    if (!(fabs(x) <= 1e5)) {
        sincos(x, &s, &c);
        return;
    }
    const double q = rint(x * 0.63661977236758134308);
    double y = fma(-q, 1.5707963267948966, x);
    y = fma(-q, 6.123233995736766e-17, y);
    // sum_i w^i / (2i+1)!  and  sum_i w^i / (2i)!, w = -y^2, as sums of coefficient x power from the
    // smallest term up: the powers are shared by both sums, and every step adds into its own
    // accumulator (Horner's steps add a constant held in a register, which the generated code copied
    // into the destination first: one more instruction per step); same accuracy (1.5e-16 absolute
    // against extended precision for |x| <= 1e5)
    const double w = -y * y, w2 = w * w, w3 = w2 * w, w4 = w2 * w2, w5 = w4 * w, w6 = w3 * w3, w7 = w4 * w3,
                 w8 = w4 * w4;
    double ts = w8 * (1.0 / 355687428096000.0);
    ts = fma(1.0 / 1307674368000.0, w7, ts);
    ts = fma(1.0 / 6227020800.0, w6, ts);
    ts = fma(1.0 / 39916800.0, w5, ts);
    ts = fma(1.0 / 362880.0, w4, ts);
    ts = fma(1.0 / 5040.0, w3, ts);
    ts = fma(1.0 / 120.0, w2, ts);
    ts = fma(1.0 / 6.0, w, ts);
    ts += 1.0;
    double tc = w8 * (1.0 / 20922789888000.0);
    tc = fma(1.0 / 87178291200.0, w7, tc);
    tc = fma(1.0 / 479001600.0, w6, tc);
    tc = fma(1.0 / 3628800.0, w5, tc);
    tc = fma(1.0 / 40320.0, w4, tc);
    tc = fma(1.0 / 720.0, w3, tc);
    tc = fma(1.0 / 24.0, w2, tc);
    tc = fma(0.5, w, tc);
    tc += 1.0;
    const double sy = y * ts, cy = tc;
    const int iq = (int)q & 3;
    const double a = (iq & 1) ? cy : sy, b = (iq & 1) ? sy : cy;  // sin and cos before the signs
    s = (iq & 2) ? -a : a;
    c = ((iq + 1) & 2) ? -b : b;
}

// ------------------------------------------------------------------ accurate element integrals
// L = int_T G(x,y) dS_y, M = int_T dG/dn_y dS_y and (NRM, normal nx at x) L' = int_T dG/dn_x dS,
// M' = d/dn_x int_T dG/dn_y dS of a flat triangle, term by term of e^{ikr}/r = sum_n (ik)^n r^{n-1}/n!.
// The moments of r over the triangle and its edges have closed recursions.  With h the height of x
// over the plane, and for edge e the foot of the perpendicular from x at signed in-plane distance d_e
// (outward), the end points at s0, s1 along the edge from it and rho_e^2 = d_e^2 + h^2:
//   K_m(e) = int_e r^m dl:   (m+1) K_m = [s r^m] + m rho_e^2 K_{m-2},   K_{-1} = log((r1+s1)/(r0+s0))
//   I_m = int_T r^m dS:      (m+2) I_m = m h^2 I_{m-2} + sum_e d_e K_m,  I_{-1} = sum_e d_e K_{-1} - |h| Omega
// (the divergence of the in-plane position times r^m), Omega the solid angle of the triangle:
//   4 pi L = sum_n (ik)^n/n! I_{n-1},   4 pi M = sgn(h) Omega - h sum_{n>=2} (n-1) (ik)^n/n! I_{n-3},
// and by the surface divergence theorem (n the triangle's normal, nu_e the outward in-plane normals,
// c_e = (f_e - x).(tau_e x n_x) with f_e the foot and tau_e the edge's direction)
//   L' = -(n_x.n) M - sum_e (n_x.nu_e) int_e G dl,
//   M' = k^2 (n_x.n) L + sum_e c_e int_e G (ikr - 1)/r^2 dl,
// whose edge integrals are the same sums over K.  On the element itself (self: h = 0, M = L' = 0) M'
// is the Hadamard finite part.  About 30 instructions per term and 20-33 terms.  Against an extended-
// precision sum, for k r <= 4, as multiples of |L|, of |L| / edge (M, L') and of |L| / edge^2 (M'): L, M
// and L' within 1e-14 on neighbours in the plane and across it and on and next to the edges' lines beyond
// the ends, M' within 1e-13 there (next to an edge itself, where M and L' grow like the logarithm of the
// distance and M' like its inverse, 5e-13 and 3e-10 at 1e-3 edges); eight Gauss panels an edge, whatever the
// distance, were 1e-4 of L off for a point 1e-9 off the plane through an edge.  Beyond k r = 4 the terms
// cancel, and the quadrature below takes over.
// Bound by FP64 instructions.  Measured on the near table of the 228,412-element shoebox (4.8 million
// entries): 7.85 ms by quadrature (192 nodes an entry), 0.27 ms by the series.
constexpr double TRI_SERIES_KR = 4.0;
constexpr int TRI_SERIES_MAX = 64;
struct RcpTable {
    double v[TRI_SERIES_MAX + 8];
};
constexpr RcpTable rcp_table() {
    RcpTable t{};
    for (int i = 1; i < TRI_SERIES_MAX + 8; ++i) t.v[i] = 1.0 / i;
    return t;
}
__constant__ RcpTable RCP = rcp_table();

template <bool NRM>
__device__ inline void tri_series(const double *x, const double *nx, const double *v, double k, int self, double rmax,
                                  const double *r, double2 &Lout, double2 &Mout, double2 &Lpout, double2 &Mpout) {
    double a[3][3];
    for (int i = 0; i < 3; ++i)
        for (int q = 0; q < 3; ++q) a[i][q] = v[3 * i + q] - x[q];
    double nn[3];
    {
        double e1[3], e2[3];
        for (int q = 0; q < 3; ++q) e1[q] = v[3 + q] - v[q], e2[q] = v[6 + q] - v[q];
        nn[0] = e1[1] * e2[2] - e1[2] * e2[1];
        nn[1] = e1[2] * e2[0] - e1[0] * e2[2];
        nn[2] = e1[0] * e2[1] - e1[1] * e2[0];
        const double nl = 1.0 / sqrt(nn[0] * nn[0] + nn[1] * nn[1] + nn[2] * nn[2]);
        for (int q = 0; q < 3; ++q) nn[q] *= nl;
    }
    const double h = self ? 0.0 : -(a[0][0] * nn[0] + a[0][1] * nn[1] + a[0][2] * nn[2]), h2 = h * h;
    auto dot = [&](int i, int j) { return a[i][0] * a[j][0] + a[i][1] * a[j][1] + a[i][2] * a[j][2]; };
    double om = 0.0;
    if (h != 0.0) {
        const double det = a[0][0] * (a[1][1] * a[2][2] - a[1][2] * a[2][1]) - a[0][1] * (a[1][0] * a[2][2] - a[1][2] * a[2][0]) +
                           a[0][2] * (a[1][0] * a[2][1] - a[1][1] * a[2][0]);
        om = 2.0 * atan2(fabs(det), r[0] * r[1] * r[2] + dot(0, 1) * r[2] + dot(0, 2) * r[1] + dot(1, 2) * r[0]);
    }
    // K[e][1] and I1 hold the last odd moment (first K_{-1}, I_{-1}), K[e][0] and I0 the last even one
    double s0[3], s1[3], d[3], rho2[3], K[3][2], cn[3], ce[3], I0 = 0.0, I1 = -fabs(h) * om;
    double l0r = 0.0, l0i = 0.0, m2r = 0.0, m2i = 0.0;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int f = e == 2 ? 0 : e + 1;
        double t[3] = {a[f][0] - a[e][0], a[f][1] - a[e][1], a[f][2] - a[e][2]};
        const double le2 = t[0] * t[0] + t[1] * t[1] + t[2] * t[2], le = sqrt(le2), il = 1.0 / le;
        for (int q = 0; q < 3; ++q) t[q] *= il;
        const double nu[3] = {t[1] * nn[2] - t[2] * nn[1], t[2] * nn[0] - t[0] * nn[2], t[0] * nn[1] - t[1] * nn[0]};
        s0[e] = a[e][0] * t[0] + a[e][1] * t[1] + a[e][2] * t[2];
        s1[e] = s0[e] + le;
        d[e] = a[e][0] * nu[0] + a[e][1] * nu[1] + a[e][2] * nu[2];
        rho2[e] = fma(d[e], d[e], h2);
        // log((r1 + s1) / (r0 + s0)) without cancellation on either side of the foot.  On the edge's line
        // beyond its ends it is finite, and the leading term of L' (d and c_e vanish there, n_x.nu_e need
        // not); with x on the edge itself the line integrals diverge, and the edge is left out of them
        const bool line = rho2[e] <= 1e-26 * le2, right = s0[e] + s1[e] >= 0.0;
        const double sa = right ? s0[e] : -s1[e], sb = right ? s1[e] : -s0[e];  // |sa| <= sb
        const double ra = right ? r[e] : r[f], rb = right ? r[f] : r[e];
        const double num = sa >= 0.0 ? rb + sb : (rb + sb) * (ra - sa), den = sa >= 0.0 ? ra + sa : rho2[e];
        K[e][1] = line && sa <= 1e-13 * le ? 0.0 : log(num / den);
        K[e][0] = 0.0;
        I1 = fma(d[e], K[e][1], I1);
        if (NRM) {
            cn[e] = nx[0] * nu[0] + nx[1] * nu[1] + nx[2] * nu[2];
            const double tn[3] = {t[1] * nx[2] - t[2] * nx[1], t[2] * nx[0] - t[0] * nx[2], t[0] * nx[1] - t[1] * nx[0]};
            ce[e] = 0.0;
            for (int q = 0; q < 3; ++q) ce[e] += (a[e][q] - s0[e] * t[q]) * tn[q];
            l0r = fma(cn[e], K[e][1], l0r);
            // (s1 / r1 - s0 / r0) / rho^2: beyond the edge's ends both quotients tend to the same +-1 towards
            // its line, so there in the equal form without their difference
            if (sa > 1e-13 * le) m2r = fma(-ce[e], le * (s0[e] + s1[e]) / (r[e] * r[f] * fma(s1[e], r[e], s0[e] * r[f])), m2r);
            else if (!line) m2r = fma(-ce[e], (s1[e] / r[f] - s0[e] / r[e]) / rho2[e], m2r);
        }
    }
    double Lr = I1, Li = 0.0, Mr = 0.0, Mi = 0.0, t = 1.0, pm = 1.0, pw[3] = {1.0, 1.0, 1.0};
#pragma unroll 1
    for (int n0 = 1; n0 < TRI_SERIES_MAX; n0 += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // n = n0 + q, m = n - 1
            const int n = n0 + q, o = q & 1;
            const double m = n - 1, rm1 = RCP.v[n], rm2 = RCP.v[n + 1];
            t *= k * rm1;
            double s = 0.0, sl = 0.0, sm = 0.0;
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const int f = e == 2 ? 0 : e + 1;
                if (NRM) sm = fma(ce[e], K[e][o], sm);
                K[e][o] = fma(m * rho2[e], K[e][o], fma(s1[e], pw[f], -s0[e] * pw[e])) * rm1;
                s = fma(d[e], K[e][o], s);
                if (NRM) sl = fma(cn[e], K[e][o], sl);
            }
            const double io = o ? I1 : I0, iv = fma(m * h2, io, s) * rm2, tm = t * m;
            (o ? I1 : I0) = iv;
            if (q == 0) {  // (ik)^n = i k^n
                Li = fma(t, iv, Li);
                Mi = fma(tm, io, Mi);
                if (NRM) l0i = fma(t, sl, l0i), m2i = fma(tm, sm, m2i);
            } else if (q == 1) {
                Lr = fma(-t, iv, Lr);
                Mr = fma(-tm, io, Mr);
                if (NRM) l0r = fma(-t, sl, l0r), m2r = fma(-tm, sm, m2r);
            } else if (q == 2) {
                Li = fma(-t, iv, Li);
                Mi = fma(-tm, io, Mi);
                if (NRM) l0i = fma(-t, sl, l0i), m2i = fma(-tm, sm, m2i);
            } else {
                Lr = fma(t, iv, Lr);
                Mr = fma(tm, io, Mr);
                if (NRM) l0r = fma(t, sl, l0r), m2r = fma(tm, sm, m2r);
            }
            for (int i = 0; i < 3; ++i) pw[i] *= r[i];
            pm *= rmax;
        }
        if (!__any(t * pm * n0 > 1e-17)) break;  // the next terms: t k^j r^j / ..., times at most n
    }
    const double i4 = 1.0 / (4.0 * FMM_PI);
    Lout = cmk(Lr * i4, Li * i4);
    Mout = h == 0.0 ? cmk(0, 0) : cmk(((h > 0 ? om : -om) - h * Mr) * i4, -h * Mi * i4);
    if (NRM) {
        const double nxn = nx[0] * nn[0] + nx[1] * nn[1] + nx[2] * nn[2];
        Lpout = self ? cmk(0, 0) : cmk(-nxn * Mout.x - l0r * i4, -nxn * Mout.y - l0i * i4);
        Mpout = cmk(k * k * nxn * Lout.x + m2r * i4, k * k * nxn * Lout.y + m2i * i4);
    }
}

// Panels of 8 points for an edge of extent w in the variable of s = d sinh(w), kr = k times the farthest
// vertex's distance: short beside the distance of the integrand's poles (pi/2 off the axis; 0.75), and
// TRI_PHASE of the phase k r each at most (dr/dw <= r).  Errors against an adaptive quadrature, points
// around a triangle, as multiples of (|L| without its oscillation) (k + 1 / edge)^(0, 1, 1, 2) for L, M, L',
// M': below 2e-13 for k r to 69 (8 panels an edge: 2e-12 at k r = 15, 1e-9 at 25, 5e-7 at 44; panels 0.75
// long whatever k: 3e-10, 5e-8, 3e-5).  At most 2.5 of phase is at rounding with room (3: the same, 4e-13 next
// to k r = 4); an edge at k r = 8 takes 4 to 10 panels.  The count is bounded (kr w of 1,280).  In FP32, and
// with the one kr for every edge: the field kernel's near part has no registers to spare.
constexpr float TRI_PHASE = 2.5f;
__device__ inline int tri_panels(double w, float kr) {
    return max(1, (int)fminf(512.0f, ceilf((float)w * fmaxf(1.0f / 0.75f, kr * (1.0f / TRI_PHASE)))));
}

// The same L and M by quadrature, for k r beyond the series: polar coordinates
// about the projection x_p of x on the triangle's plane.  With h the signed height of x and
// r^2 = rho^2 + h^2 the radial integrals are exact:
//   int_0^{rho_e} G rho drho        = (e^{ikR} - e^{ik|h|}) / (4 pi i k)
//   int_0^{rho_e} dG/dn_y rho drho  = -h/(4 pi) (e^{ikR}/R - e^{ik|h|}/|h|),   R = r(rho_e)
// leaving an angular integral per edge (signed by the edge orientation seen from x_p), done by
// 8-point Gauss-Legendre panels (tri_panels) after the substitution tan(psi) = sinh(w).
// self != 0: x is the triangle's centroid (h = 0, M = 0 by the principal value).
__device__ void tri_gauss(const double *x, const double *v, double k, float kr, int self, double2 &Lout, double2 &Mout) {
    double e1[3] = {v[3] - v[0], v[4] - v[1], v[5] - v[2]};
    double e2[3] = {v[6] - v[0], v[7] - v[1], v[8] - v[2]};
    double nn[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2], e1[0] * e2[1] - e1[1] * e2[0]};
    double nl = sqrt(nn[0] * nn[0] + nn[1] * nn[1] + nn[2] * nn[2]);
    nn[0] /= nl;
    nn[1] /= nl;
    nn[2] /= nl;
    double h = self ? 0.0 : (x[0] - v[0]) * nn[0] + (x[1] - v[1]) * nn[1] + (x[2] - v[2]) * nn[2];
    double xp[3] = {x[0] - h * nn[0], x[1] - h * nn[1], x[2] - h * nn[2]};
    double ah = fabs(h);
    double2 Lacc = cmk(0, 0), Macc = cmk(0, 0);
    double span = 0.0;
    for (int e = 0; e < 3; ++e) {
        int e2i = (e + 1) % 3;
        double a[3] = {v[3 * e] - xp[0], v[3 * e + 1] - xp[1], v[3 * e + 2] - xp[2]};
        double b[3] = {v[3 * e2i] - xp[0], v[3 * e2i + 1] - xp[1], v[3 * e2i + 2] - xp[2]};
        double ed[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
        double le = sqrt(ed[0] * ed[0] + ed[1] * ed[1] + ed[2] * ed[2]);
        double eh[3] = {ed[0] / le, ed[1] / le, ed[2] / le};
        double s0 = a[0] * eh[0] + a[1] * eh[1] + a[2] * eh[2];
        double s1 = b[0] * eh[0] + b[1] * eh[1] + b[2] * eh[2];
        double f[3] = {a[0] - s0 * eh[0], a[1] - s0 * eh[1], a[2] - s0 * eh[2]};
        double d = sqrt(f[0] * f[0] + f[1] * f[1] + f[2] * f[2]);
        if (d <= 1e-13 * le) continue;
        double cr[3] = {a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]};
        double sgn = (cr[0] * nn[0] + cr[1] * nn[1] + cr[2] * nn[2]) >= 0.0 ? 1.0 : -1.0;
        span += sgn * (atan2(s1, d) - atan2(s0, d));
        // angle psi from the edge normal, substituted tan(psi) = sinh(w): rho = d cosh(w),
        // dpsi = dw / cosh(w); this grades the panels logarithmically along edges that are long
        // compared with their distance d from x_p, where the integrand varies fastest
        const double w0 = asinh(s0 / d), w1 = asinh(s1 / d);
        const int NPAN = tri_panels(w1 - w0, kr);
        double hw = 0.5 * (w1 - w0) / NPAN;
        for (int pan = 0; pan < NPAN; ++pan) {
            double mid = w0 + (2 * pan + 1) * hw;
            for (int q = 0; q < 8; ++q) {
                double ww = mid + hw * GL8X[q];
                double ch = cosh(ww);
                double w = sgn * hw * GL8W[q] / ch;
                double rho = d * ch;
                double R = sqrt(rho * rho + h * h);
                double dR = R - ah;
                // z = k dR from its half angle: sin z = 2 s c and 1 - cos z = 2 s^2 (no cancellation
                // at small z); the radial L integral is e^{ik|h|} (sin z + i (1 - cos z)) / k and
                // e^{ikR} = e^{ik|h|} e^{iz}, the common factor e^{ik|h|} taken once at the end
                double s, c;
                sincos_red(0.5 * k * dR, s, c);
                const double sz = 2.0 * s * c, omc = 2.0 * s * s;
                Lacc = cadd(Lacc, cmk(w * sz, w * omc));
                Macc = cadd(Macc, cscale(cmk(1.0 - omc, sz), w / R));
            }
        }
    }
    double sh, ch;
    sincos(k * ah, &sh, &ch);
    double2 eh_ = cmk(ch, sh);
    Lout = cscale(cmul(eh_, Lacc), 1.0 / (4.0 * FMM_PI * k));
    if (h == 0.0) {
        Mout = cmk(0, 0);
    } else {
        double sgh = h > 0 ? 1.0 : -1.0;
        Mout = cadd(cscale(cmul(eh_, Macc), -h / (4.0 * FMM_PI)), cscale(eh_, sgh * span / (4.0 * FMM_PI)));
    }
}

// L' and M' in the same way: the edge integrals by Gauss panels with s = d sinh(w) (d = distance from x
// to the edge's line, ds = r dw).
__device__ void tri_gauss_n(const double *x, const double *nx, const double *v, double k, float kr, int self,
                            double2 &L, double2 &M, double2 &Lp, double2 &Mp) {
    tri_gauss(x, v, k, kr, self, L, M);
    double e1[3] = {v[3] - v[0], v[4] - v[1], v[5] - v[2]};
    double e2[3] = {v[6] - v[0], v[7] - v[1], v[8] - v[2]};
    double nn[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2], e1[0] * e2[1] - e1[1] * e2[0]};
    double nl = sqrt(nn[0] * nn[0] + nn[1] * nn[1] + nn[2] * nn[2]);
    for (int q = 0; q < 3; ++q) nn[q] /= nl;
    const double nxn = nx[0] * nn[0] + nx[1] * nn[1] + nx[2] * nn[2];
    double2 lp = cscale(M, -nxn), mp = cscale(L, k * k * nxn);
    for (int e = 0; e < 3; ++e) {
        const int eb = (e + 1) % 3;
        const double a[3] = {v[3 * e], v[3 * e + 1], v[3 * e + 2]}, b[3] = {v[3 * eb], v[3 * eb + 1], v[3 * eb + 2]};
        double tau[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
        const double le = sqrt(tau[0] * tau[0] + tau[1] * tau[1] + tau[2] * tau[2]);
        for (int q = 0; q < 3; ++q) tau[q] /= le;
        const double nu[3] = {tau[1] * nn[2] - tau[2] * nn[1], tau[2] * nn[0] - tau[0] * nn[2], tau[0] * nn[1] - tau[1] * nn[0]};
        const double tn[3] = {tau[1] * nx[2] - tau[2] * nx[1], tau[2] * nx[0] - tau[0] * nx[2], tau[0] * nx[1] - tau[1] * nx[0]};
        const double ax[3] = {a[0] - x[0], a[1] - x[1], a[2] - x[2]};
        const double s0 = ax[0] * tau[0] + ax[1] * tau[1] + ax[2] * tau[2], s1 = s0 + le;
        const double fx[3] = {ax[0] - s0 * tau[0], ax[1] - s0 * tau[1], ax[2] - s0 * tau[2]};  // f - x
        const double d = sqrt(fx[0] * fx[0] + fx[1] * fx[1] + fx[2] * fx[2]);
        const double ce = fx[0] * tn[0] + fx[1] * tn[1] + fx[2] * tn[2];
        const double cnu = nx[0] * nu[0] + nx[1] * nu[1] + nx[2] * nu[2];
        double2 I0 = cmk(0, 0), I2 = cmk(0, 0);
        if (d > 1e-13 * le) {
            const double w0 = asinh(s0 / d), w1 = asinh(s1 / d);
            const int NPAN = tri_panels(w1 - w0, kr);
            const double hw = 0.5 * (w1 - w0) / NPAN;
            for (int pan = 0; pan < NPAN; ++pan) {
                const double mid = w0 + (2 * pan + 1) * hw;
                for (int q = 0; q < 8; ++q) {
                    const double r = d * cosh(mid + hw * GL8X[q]);
                    const double wt = hw * GL8W[q] * r;  // ds = r dw
                    double sn, cs;
                    sincos(k * r, &sn, &cs);
                    const double2 G = cmk(cs / (4.0 * FMM_PI * r), sn / (4.0 * FMM_PI * r));
                    I0 = cadd(I0, cscale(G, wt));
                    I2 = cadd(I2, cscale(cmul(G, cmk(-1.0, k * r)), wt / (r * r)));
                }
            }
        } else if (s0 * s1 > 0.0) {
            // x on the edge's line beyond its ends: c_e = 0, and panels in w = log|s| for I0
            const double w0 = log(fmin(fabs(s0), fabs(s1))), w1 = log(fmax(fabs(s0), fabs(s1)));
            const int NPAN = tri_panels(w1 - w0, kr);
            const double hw = 0.5 * (w1 - w0) / NPAN;
            for (int pan = 0; pan < NPAN; ++pan) {
                const double mid = w0 + (2 * pan + 1) * hw;
                for (int q = 0; q < 8; ++q) {
                    double sn, cs;
                    sincos(k * exp(mid + hw * GL8X[q]), &sn, &cs);
                    I0 = cadd(I0, cscale(cmk(cs, sn), hw * GL8W[q] / (4.0 * FMM_PI)));
                }
            }
        } else {
            // x on the edge itself (the integral diverges): plain panels in s
            const int NPAN = 8;
            const double hs = 0.5 * (s1 - s0) / NPAN;
            for (int pan = 0; pan < NPAN; ++pan) {
                const double mid = s0 + (2 * pan + 1) * hs;
                for (int q = 0; q < 8; ++q) {
                    const double r = fabs(mid + hs * GL8X[q]);
                    double sn, cs;
                    sincos(k * r, &sn, &cs);
                    I0 = cadd(I0, cscale(cmk(cs, sn), hs * GL8W[q] / (4.0 * FMM_PI * r)));
                }
            }
        }
        lp = csub(lp, cscale(I0, cnu));
        mp = cadd(mp, cscale(I2, ce));
    }
    Lp = self ? cmk(0, 0) : lp;
    Mp = mp;
}

// distances of the triangle's vertices; the largest is that of its farthest point
__device__ inline double tri_radii(const double *x, const double *v, double *r) {
    for (int i = 0; i < 3; ++i) {
        const double dx = v[3 * i] - x[0], dy = v[3 * i + 1] - x[1], dz = v[3 * i + 2] - x[2];
        r[i] = sqrt(dx * dx + dy * dy + dz * dz);
    }
    return fmax(r[0], fmax(r[1], r[2]));
}
__device__ inline void tri_integrals(const double *x, const double *v, double k, int self, double2 &L, double2 &M) {
    double r[3];
    const double rmax = tri_radii(x, v, r);
    double2 Lp, Mp;
    if (k * rmax <= TRI_SERIES_KR) tri_series<false>(x, nullptr, v, k, self, rmax, r, L, M, Lp, Mp);
    else tri_gauss(x, v, k, (float)(k * rmax), self, L, M);
}
__device__ inline void tri_integrals_n(const double *x, const double *nx, const double *v, double k, int self,
                                       double2 &L, double2 &M, double2 &Lp, double2 &Mp) {
    double r[3];
    const double rmax = tri_radii(x, v, r);
    if (k * rmax <= TRI_SERIES_KR) tri_series<true>(x, nx, v, k, self, rmax, r, L, M, Lp, Mp);
    else tri_gauss_n(x, nx, v, k, (float)(k * rmax), self, L, M, Lp, Mp);
}

__global__ void __launch_bounds__(128) k_near_quad_n(int64_t nnz, const int32_t *rowv, const int32_t *col, const double4 *ec,
                              const double4 *en, const double *ev, double k, double2 *Lpv, double2 *Mpv) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    int i = rowv[e], j = col[e];
    double4 ci = ec[i], ni = en[i];
    double x[3] = {ci.x, ci.y, ci.z}, nx[3] = {ni.x, ni.y, ni.z}, v[9];
    for (int q = 0; q < 9; ++q) v[q] = ev[9 * (int64_t)j + q];
    double2 L, M, Lp, Mp;
    tri_integrals_n(x, nx, v, k, i == j, L, M, Lp, Mp);
    Lpv[e] = Lp;
    Mpv[e] = Mp;
}

// ------------------------------------------------------------------ near-field table
__global__ void k_near_count(int64_t n, const int32_t *leaf_of, const int32_t *leaf_start, const int32_t *nbr_start,
                             const int32_t *nbr_list, const double4 *ec, double rc2, int32_t *cnt) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double4 ci = ec[i];
    int b = leaf_of[i], c = 0;
    for (int q = nbr_start[b]; q < nbr_start[b + 1]; ++q) {
        int sb = nbr_list[q];
        for (int j = leaf_start[sb]; j < leaf_start[sb + 1]; ++j) {
            double4 cj = ec[j];
            if (j == i || dist2_exact(ci.x, ci.y, ci.z, cj.x, cj.y, cj.z) < rc2) ++c;
        }
    }
    cnt[i] = c;
}

__global__ void k_near_fill(int64_t n, const int32_t *leaf_of, const int32_t *leaf_start, const int32_t *nbr_start,
                            const int32_t *nbr_list, const double4 *ec, double rc2, const int32_t *start,
                            int32_t *rowv, int32_t *col) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double4 ci = ec[i];
    int b = leaf_of[i], o = start[i];
    for (int q = nbr_start[b]; q < nbr_start[b + 1]; ++q) {
        int sb = nbr_list[q];
        for (int j = leaf_start[sb]; j < leaf_start[sb + 1]; ++j) {
            double4 cj = ec[j];
            if (j == i || dist2_exact(ci.x, ci.y, ci.z, cj.x, cj.y, cj.z) < rc2) {
                rowv[o] = (int32_t)i;
                col[o++] = j;
            }
        }
    }
}

__global__ void __launch_bounds__(128) k_near_quad(int64_t nnz, const int32_t *rowv, const int32_t *col, const double4 *ec, const double *ev,
                            double k, double2 *Lv, double2 *Mv) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    int i = rowv[e], j = col[e];
    double4 ci = ec[i];
    double x[3] = {ci.x, ci.y, ci.z}, v[9];
    for (int q = 0; q < 9; ++q) v[q] = ev[9 * (int64_t)j + q];
    double2 L, M;
    tri_integrals(x, v, k, i == j, L, M);
    Lv[e] = L;
    Mv[e] = M;
}

// ------------------------------------------------------------------ densities
// sigma_i = -i k beta_i x_i, mu_i = x_i (sorted order; x in caller order)
// nr right-hand sides: x is nr x N in caller order; sigma/mu interleaved, [i * nr + r] in tree order
__global__ void k_densities(int64_t n, int nr, const int32_t *perm, const double2 *x, const double2 *beta, double k,
                            double2 *sigma, double2 *mu) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * nr) return;
    const int64_t i = e / nr;
    const int r = (int)(e - i * nr);
    double2 xi = x[(int64_t)r * n + perm[i]];
    double2 bx = cmul(beta[i], xi);
    sigma[e] = cmk(k * bx.y, -k * bx.x);  // -i k (beta x)
    mu[e] = xi;
}

// gamma_i = -dpsi_in/dn + i k beta psi_in at centroid i for nr monopoles of amplitude amp at rs (Eq. sp7),
// the vectors interleaved
__global__ void k_gamma(int64_t n, int nr, const double4 *ec, const double4 *en, const double2 *beta, double k,
                        Monopoles src, double2 *sigma, double2 *mu) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double4 c = ec[i], nv = en[i];
    double2 ikb = cmk(-k * beta[i].y, k * beta[i].x);          // i k beta
    for (int q = 0; q < nr; ++q) {
        double dx = c.x - src.rs[q][0], dy = c.y - src.rs[q][1], dz = c.z - src.rs[q][2];
        double r = sqrt(dx * dx + dy * dy + dz * dz);
        double s, co;
        sincos(k * r, &s, &co);
        double2 G = cmul(src.amp[q], cmk(co / (4 * FMM_PI * r), s / (4 * FMM_PI * r)));
        double proj = (dx * nv.x + dy * nv.y + dz * nv.z) / (r * r);
        double2 dG = cscale(cmul(G, cmk(-1.0, k * r)), proj);  // G (ikr - 1) (x - rs).n / r^2
        sigma[i * nr + q] = csub(cmul(ikb, G), dG);
        mu[i * nr + q] = cmk(0, 0);
    }
}

// ------------------------------------------------------------------ pair-kernel helpers
// 1/sqrt(d) for a positive, normal d: the hardware estimate y (relative error below 1e-7) and one
// third-order step, y (1 + e/2 + 3 e^2/8) with e = 1 - d y^2: two instructions fewer than two Newton
// steps, within the same ulp
__device__ inline double rsq_nr(double d) {
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-d * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// cos and sin of 2 pi i / 128
constexpr int EIKR_N = 128;
__device__ const double2 EIKR_TAB[EIKR_N] = {
    {1.0, 0.0}, {0.9987954562051724, 0.049067674327418015},
    {0.9951847266721969, 0.0980171403295606}, {0.989176509964781, 0.14673047445536175},
    {0.9807852804032304, 0.19509032201612828}, {0.970031253194544, 0.2429801799032639},
    {0.9569403357322088, 0.2902846772544624}, {0.9415440651830208, 0.33688985339222005},
    {0.9238795325112867, 0.3826834323650898}, {0.9039892931234433, 0.4275550934302821},
    {0.881921264348355, 0.47139673682599764}, {0.8577286100002721, 0.5141027441932218},
    {0.8314696123025452, 0.5555702330196022}, {0.8032075314806449, 0.5956993044924334},
    {0.773010453362737, 0.6343932841636455}, {0.7409511253549591, 0.6715589548470184},
    {0.7071067811865476, 0.7071067811865476}, {0.6715589548470184, 0.7409511253549591},
    {0.6343932841636455, 0.773010453362737}, {0.5956993044924334, 0.8032075314806449},
    {0.5555702330196022, 0.8314696123025452}, {0.5141027441932218, 0.8577286100002721},
    {0.47139673682599764, 0.881921264348355}, {0.4275550934302821, 0.9039892931234433},
    {0.3826834323650898, 0.9238795325112867}, {0.33688985339222005, 0.9415440651830208},
    {0.2902846772544624, 0.9569403357322088}, {0.2429801799032639, 0.970031253194544},
    {0.19509032201612828, 0.9807852804032304}, {0.14673047445536175, 0.989176509964781},
    {0.0980171403295606, 0.9951847266721969}, {0.049067674327418015, 0.9987954562051724},
    {0.0, 1.0}, {-0.049067674327418015, 0.9987954562051724},
    {-0.0980171403295606, 0.9951847266721969}, {-0.14673047445536175, 0.989176509964781},
    {-0.19509032201612828, 0.9807852804032304}, {-0.2429801799032639, 0.970031253194544},
    {-0.2902846772544624, 0.9569403357322088}, {-0.33688985339222005, 0.9415440651830208},
    {-0.3826834323650898, 0.9238795325112867}, {-0.4275550934302821, 0.9039892931234433},
    {-0.47139673682599764, 0.881921264348355}, {-0.5141027441932218, 0.8577286100002721},
    {-0.5555702330196022, 0.8314696123025452}, {-0.5956993044924334, 0.8032075314806449},
    {-0.6343932841636455, 0.773010453362737}, {-0.6715589548470184, 0.7409511253549591},
    {-0.7071067811865476, 0.7071067811865476}, {-0.7409511253549591, 0.6715589548470184},
    {-0.773010453362737, 0.6343932841636455}, {-0.8032075314806449, 0.5956993044924334},
    {-0.8314696123025452, 0.5555702330196022}, {-0.8577286100002721, 0.5141027441932218},
    {-0.881921264348355, 0.47139673682599764}, {-0.9039892931234433, 0.4275550934302821},
    {-0.9238795325112867, 0.3826834323650898}, {-0.9415440651830208, 0.33688985339222005},
    {-0.9569403357322088, 0.2902846772544624}, {-0.970031253194544, 0.2429801799032639},
    {-0.9807852804032304, 0.19509032201612828}, {-0.989176509964781, 0.14673047445536175},
    {-0.9951847266721969, 0.0980171403295606}, {-0.9987954562051724, 0.049067674327418015},
    {-1.0, 0.0}, {-0.9987954562051724, -0.049067674327418015},
    {-0.9951847266721969, -0.0980171403295606}, {-0.989176509964781, -0.14673047445536175},
    {-0.9807852804032304, -0.19509032201612828}, {-0.970031253194544, -0.2429801799032639},
    {-0.9569403357322088, -0.2902846772544624}, {-0.9415440651830208, -0.33688985339222005},
    {-0.9238795325112867, -0.3826834323650898}, {-0.9039892931234433, -0.4275550934302821},
    {-0.881921264348355, -0.47139673682599764}, {-0.8577286100002721, -0.5141027441932218},
    {-0.8314696123025452, -0.5555702330196022}, {-0.8032075314806449, -0.5956993044924334},
    {-0.773010453362737, -0.6343932841636455}, {-0.7409511253549591, -0.6715589548470184},
    {-0.7071067811865476, -0.7071067811865476}, {-0.6715589548470184, -0.7409511253549591},
    {-0.6343932841636455, -0.773010453362737}, {-0.5956993044924334, -0.8032075314806449},
    {-0.5555702330196022, -0.8314696123025452}, {-0.5141027441932218, -0.8577286100002721},
    {-0.47139673682599764, -0.881921264348355}, {-0.4275550934302821, -0.9039892931234433},
    {-0.3826834323650898, -0.9238795325112867}, {-0.33688985339222005, -0.9415440651830208},
    {-0.2902846772544624, -0.9569403357322088}, {-0.2429801799032639, -0.970031253194544},
    {-0.19509032201612828, -0.9807852804032304}, {-0.14673047445536175, -0.989176509964781},
    {-0.0980171403295606, -0.9951847266721969}, {-0.049067674327418015, -0.9987954562051724},
    {0.0, -1.0}, {0.049067674327418015, -0.9987954562051724},
    {0.0980171403295606, -0.9951847266721969}, {0.14673047445536175, -0.989176509964781},
    {0.19509032201612828, -0.9807852804032304}, {0.2429801799032639, -0.970031253194544},
    {0.2902846772544624, -0.9569403357322088}, {0.33688985339222005, -0.9415440651830208},
    {0.3826834323650898, -0.9238795325112867}, {0.4275550934302821, -0.9039892931234433},
    {0.47139673682599764, -0.881921264348355}, {0.5141027441932218, -0.8577286100002721},
    {0.5555702330196022, -0.8314696123025452}, {0.5956993044924334, -0.8032075314806449},
    {0.6343932841636455, -0.773010453362737}, {0.6715589548470184, -0.7409511253549591},
    {0.7071067811865476, -0.7071067811865476}, {0.7409511253549591, -0.6715589548470184},
    {0.773010453362737, -0.6343932841636455}, {0.8032075314806449, -0.5956993044924334},
    {0.8314696123025452, -0.5555702330196022}, {0.8577286100002721, -0.5141027441932218},
    {0.881921264348355, -0.47139673682599764}, {0.9039892931234433, -0.4275550934302821},
    {0.9238795325112867, -0.3826834323650898}, {0.9415440651830208, -0.33688985339222005},
    {0.9569403357322088, -0.2902846772544624}, {0.970031253194544, -0.2429801799032639},
    {0.9807852804032304, -0.19509032201612828}, {0.989176509964781, -0.14673047445536175},
    {0.9951847266721969, -0.0980171403295606}, {0.9987954562051724, -0.049067674327418015},
};
// the table in LDS, by the first 128 threads of the workgroup
__device__ inline void eikr_stage(double2 *tab, int tid) {
    if (tid < EIKR_N) tab[tid] = EIKR_TAB[tid];
}
// e^{ikr}, kk = k 128 / (2 pi) as a sum of two doubles (eikr_scale): r kk is split into the nearest
// integer n (the low bits of r kk + 1.5 2^52) and a remainder f, |f| <= 1/2; e^{2 pi i n / 128} comes
// from the table in LDS and e^{2 pi i f / 128} from the Taylor polynomials through f^7 and f^6
// (truncation below 2e-17).  About 20 instructions, against about 45 for a Cody-Waite reduction by
// pi/2 and polynomials through degree 17 with their quadrant selects, and more accurate: k r is not
// rounded before the reduction.  Absolute error against 113-bit values, worst of 400,000 draws: 2.1e-16
// for every k r in 0.01..90,000 (the reduction of the rounded product: 2.2e-16 below 1, 9.8e-16 in
// 1..10, 5.7e-14 in 100..1,000).  Needs k r < 2^46 (truncation numbers up to 1,000 bound k r by 1e7
// inside a room).
__device__ inline void eikr(double r, double2 kk, const double2 *tab, double &c, double &s) {
    const double m = fma(r, kk.x, 6755399441055744.0);
    const int i = __double2loint(m) & (EIKR_N - 1);
    const double f = fma(r, kk.y, fma(r, kk.x, 6755399441055744.0 - m));
    const double t = 2.0 * FMM_PI / EIKR_N, t2 = t * t;
    const double w = f * f;
    const double sn = fma(fma(fma(-t * t2 * t2 * t2 / 5040.0, w, t * t2 * t2 / 120.0), w, -t * t2 / 6.0), w, t) * f;
    const double cm = fma(fma(-t2 * t2 * t2 / 720.0, w, t2 * t2 / 24.0), w, -0.5 * t2) * w;  // cos - 1
    const double2 e = tab[i];
    c = fma(-e.y, sn, fma(e.x, cm, e.x));
    s = fma(e.x, sn, fma(e.y, cm, e.y));
}

// ------------------------------------------------------------------ P2P + near table
// y_i = sum_{j in neighbour leaves, |c_i - c_j| >= r_c} [G q_j + dG/dn_y w_j] + sum_near [L sigma + M mu]
// with q_j = A_j sigma_j, w_j = A_j mu_j, and (NRM) the normal derivative at i of the same layers,
// yn_i, from the L', M' near entries and the kernel's derivatives.
//
// One workgroup of 256 per target leaf and split of its sources.  Bound by FP64 vector instructions
// (about 60 per pair), so the layout keeps lanes busy and instructions few:
//  - the neighbour leaves' sources form one list (their ranges end to end), and tiles of it are
//    staged in LDS whole, whatever the leaves' sizes;
//  - a lane takes two targets, so that every source read from LDS serves two pairs; TP lanes cover
//    the leaf and S = floor(256 / TP) lane groups take every S-th source of a tile (leaves hold
//    17-48 targets mostly: 94-100 % of the lanes busy); the groups' sums are added in LDS;
//  - pairs closer than r_c (and the self pair) are left to the near table by a zero 1/r, without a
//    branch.
// With few leaves (nsplit > 1) the source list is cut into nsplit pieces, one workgroup each, so
// that a small room still fills the device; piece g writes its own sums at y + g n NR, which L2P adds
// in order.  Measured against one wavefront per leaf, one target per lane and the polynomial sincos
// (FP64, one vector): 2,664 elements 255 -> 13.6 us, 90,972 241 -> 73 us, 1M L-room 1.20 -> 0.67 ms
// (5.4e11 pairs/s); with normal derivatives 2,664 elements 431 -> 19.5 us, 90,972 412 -> 140 us.
// Mixed-precision products take it too: the vector units issue FP64 as fast as FP32, and the pairs in
// FP32 (its accurate sincos, compensated sums, one wavefront per leaf) took four vectors of 90,972
// elements 276 us where this takes 146, of 612,540 elements 690 and 632.
constexpr int P2P_WG = 256, P2P_T = 2;
// lanes per group TP and groups S of a leaf of nt targets, for the number of passes over the sources
// P (the fewest possible, or up to three more) with the least lane work P / S; a further pass
// stages the sources again and has to save 2 % of it.  Four lanes weigh the four candidates.
__device__ inline void p2p_shape(int nt, int tid, int &TP, int &S) {
    const int P = (nt + P2P_WG * P2P_T - 1) / (P2P_WG * P2P_T) + (tid & 3);
    int tp = (nt + P2P_T * P - 1) / (P2P_T * P), sg = P2P_WG / tp;
    float cost = (float)P / (float)sg * (1.0f + 0.02f * (tid & 3));
    for (int d = 1; d < 4; d <<= 1) {
        const float oc = __shfl_xor(cost, d, 4);
        const int ot = __shfl_xor(tp, d, 4), os = __shfl_xor(sg, d, 4);
        if (oc < cost || (oc == cost && os < sg)) {
            cost = oc;
            tp = ot;
            sg = os;
        }
    }
    TP = __builtin_amdgcn_readfirstlane(tp);
    S = __builtin_amdgcn_readfirstlane(sg);
}

// source tiles: per source (x, y), (z, n_x), (n_y, n_z), then NR (q), NR (w) as double2
template <int NR> constexpr int p2p_tile() { return NR >= 4 ? 128 : 256; }

template <int NR, bool NRM>
__global__ void __launch_bounds__(P2P_WG) __attribute__((amdgpu_waves_per_eu(4)))
k_p2p(int nleaf, const int32_t *leaf_start, const int32_t *nbr_start, const int32_t *nbr_list, int all_leaves,
      int nsplit, const double4 *ec, const double4 *en, const double2 *sigma, const double2 *mu, double k, double2 kk,
      double rc2, const int32_t *near_start, const int32_t *near_col, const double2 *nL, const double2 *nM,
      const double2 *nLp, const double2 *nMp, double2 *y, double2 *yn) {
    constexpr int T = P2P_T, TS = p2p_tile<NR>(), F = 3 + 2 * NR, NA = NRM ? 2 * NR : NR;
    constexpr int BUF = TS * F > P2P_WG * T * NA ? TS * F : P2P_WG * T * NA;
    const int b = blockIdx.x / nsplit, g = blockIdx.x - b * nsplit, tid = threadIdx.x;
    __shared__ double2 tab[EIKR_N], buf[BUF];
    __shared__ int rs[32], cum[33];
    const int ts = leaf_start[b], te = leaf_start[b + 1];
    int nrng = 1;
    if (all_leaves) {  // all-pairs product: the one range of every element
        if (tid == 0) {
            rs[0] = 0;
            cum[0] = 0;
            cum[1] = leaf_start[nleaf];
        }
    } else {
        const int nb0 = nbr_start[b];
        nrng = nbr_start[b + 1] - nb0;  // at most 27
        if (tid < 32) {
            int c = 0;
            if (tid < nrng) {
                const int sb = nbr_list[nb0 + tid], ss = leaf_start[sb];
                rs[tid] = ss;
                c = leaf_start[sb + 1] - ss;
            }
            for (int d = 1; d < 32; d <<= 1) {
                const int o = __shfl_up(c, d, 32);
                if (tid >= d) c += o;
            }
            cum[tid + 1] = c;
            if (tid == 0) cum[0] = 0;
        }
    }
    eikr_stage(tab, tid);
    __syncthreads();
    // this workgroup's piece of the source list
    int lo = 0, hi = cum[nrng];
    if (nsplit > 1) {
        const unsigned tot = hi, piece = (tot + nsplit - 1) / nsplit;
        lo = (int)min(tot, g * piece);
        hi = (int)min(tot, (g + 1) * piece);
    }
    int TP, S;
    p2p_shape(te - ts, tid, TP, S);
    const int h = tid / TP, l = tid - h * TP;
    const double inv4pi = 1.0 / (4.0 * FMM_PI);
    const int64_t n = leaf_start[nleaf];
    for (int t0 = ts; t0 < te; t0 += TP * T) {
        // a lane's targets: the second one repeats the first (unused) where the leaf ends
        int t[T];
        bool act[T];
        double4 ct[T], nt[T];
        double2 acc[T][NR], accn[T][NR];
#pragma unroll
        for (int u = 0; u < T; ++u) {
            t[u] = t0 + l + u * TP;
            act[u] = t[u] < te && h < S;
            const int tt = t[u] < te ? t[u] : ts;
            ct[u] = ec[tt];
            if (NRM) nt[u] = en[tt];
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[u][r] = accn[u][r] = cmk(0, 0);
        }
        for (int j0 = lo; j0 < hi; j0 += TS) {
            __syncthreads();
            const int idx = j0 + tid;
            if (tid < TS && idx < hi) {
                int q = 0;
#pragma unroll
                for (int d = 16; d > 0; d >>= 1)
                    if (q + d < nrng && cum[q + d] <= idx) q += d;
                const int j = rs[q] + (idx - cum[q]);
                const double4 c = ec[j], nv = en[j];
                double2 *o = buf + tid * F;
                o[0] = cmk(c.x, c.y);
                o[1] = cmk(c.z, nv.x);
                o[2] = cmk(nv.y, nv.z);
                const double wgt = c.w * inv4pi;
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    o[3 + r] = cscale(sigma[(int64_t)j * NR + r], wgt);
                    o[3 + NR + r] = cscale(mu[(int64_t)j * NR + r], wgt);
                }
            }
            __syncthreads();
            const int cnt = min(TS, hi - j0);
            if (h < S && act[0])
                for (int jj = h; jj < cnt; jj += S) {
                    const double2 *o = buf + jj * F;
                    const double2 xy = o[0], zn = o[1], nn2 = o[2];
#pragma unroll
                    for (int u = 0; u < T; ++u) {
                        const double d2 = dist2_exact(ct[u].x, ct[u].y, ct[u].z, xy.x, xy.y, zn.x);
                        const double dx = xy.x - ct[u].x, dy = xy.y - ct[u].y, dz = zn.x - ct[u].z;
                        const double ir = d2 < rc2 ? 0.0 : rsq_nr(d2), r = d2 * ir, ir2 = ir * ir, kr = k * r;
                        double s, c;
                        eikr(r, kk, tab, c, s);
                        const double2 G = cmk(c * ir, s * ir);
                        const double a1 = (dx * zn.y + dy * nn2.x + dz * nn2.y) * ir2;  // (y-x).n / r^2
                        double a2 = 0, kx = 0, ky = 0;
                        if (NRM) {
                            // K = G [a1 a2 (3 - 3ikr - k^2 r^2) - (n_x.n_y / r^2)(ikr - 1)], a2 = -(y-x).n_x / r^2
                            a2 = -(dx * nt[u].x + dy * nt[u].y + dz * nt[u].z) * ir2;
                            const double bb = (nt[u].x * zn.y + nt[u].y * nn2.x + nt[u].z * nn2.y) * ir2, mm = a1 * a2;
                            kx = fma(mm, fma(-kr, kr, 3.0), bb);
                            ky = -kr * fma(3.0, mm, bb);
                        }
#pragma unroll
                        for (int rr = 0; rr < NR; ++rr) {
                            const double2 q = o[3 + rr], w = o[3 + NR + rr];
                            // G (q + (ikr - 1) a1 w)
                            const double2 v = cmk(fma(-a1, fma(kr, w.y, w.x), q.x), fma(-a1, fma(-kr, w.x, w.y), q.y));
                            acc[u][rr] = cfma(G, v, acc[u][rr]);
                            if (NRM) {  // G ((ikr - 1) a2 q) + K w
                                const double2 z = cmk(fma(-a2, fma(kr, q.y, q.x), fma(kx, w.x, -ky * w.y)),
                                                      fma(-a2, fma(-kr, q.x, q.y), fma(kx, w.y, ky * w.x)));
                                accn[u][rr] = cfma(G, z, accn[u][rr]);
                            }
                        }
                    }
                }
        }
#pragma unroll
        for (int u = 0; u < T; ++u)
            if (act[u])
                for (int e = near_start[t[u]] + h + S * g; e < near_start[t[u] + 1]; e += S * nsplit) {
                    const int64_t j = near_col[e];
                    const double2 lv = nL[e], mv = nM[e];
#pragma unroll
                    for (int rr = 0; rr < NR; ++rr) {
                        const double2 sg = sigma[j * NR + rr], m_ = mu[j * NR + rr];
                        acc[u][rr] = cfma(mv, m_, cfma(lv, sg, acc[u][rr]));
                        if (NRM) accn[u][rr] = cfma(nMp[e], m_, cfma(nLp[e], sg, accn[u][rr]));
                    }
                }
        // add the groups' sums: every step folds the upper half of the groups onto the lower
        for (int m = S; m > 1;) {
            const int half = (m + 1) / 2;
            __syncthreads();
            if (h >= half && h < m)
#pragma unroll
                for (int u = 0; u < T; ++u)
#pragma unroll
                    for (int rr = 0; rr < NR; ++rr) {
                        buf[((h - half) * TP + l) * (T * NA) + u * NA + rr] = acc[u][rr];
                        if (NRM) buf[((h - half) * TP + l) * (T * NA) + u * NA + NR + rr] = accn[u][rr];
                    }
            __syncthreads();
            if (h < m - half)
#pragma unroll
                for (int u = 0; u < T; ++u)
#pragma unroll
                    for (int rr = 0; rr < NR; ++rr) {
                        acc[u][rr] = cadd(acc[u][rr], buf[(h * TP + l) * (T * NA) + u * NA + rr]);
                        if (NRM) accn[u][rr] = cadd(accn[u][rr], buf[(h * TP + l) * (T * NA) + u * NA + NR + rr]);
                    }
            m = half;
        }
        if (h == 0)
#pragma unroll
            for (int u = 0; u < T; ++u)
                if (act[u])
#pragma unroll
                    for (int rr = 0; rr < NR; ++rr) {
                        y[(g * n + t[u]) * NR + rr] = acc[u][rr];
                        if (NRM) yn[(g * n + t[u]) * NR + rr] = accn[u][rr];
                    }
    }
}

__global__ void k_zero8(int64_t n, uint64_t *p) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

__global__ void k_cvt_d2f(int64_t n, const double2 *a, float2 *b) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = make_float2((float)a[i].x, (float)a[i].y);
}
__global__ void k_cvt_real_d2f(int64_t n, const double *a, float *b) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (float)a[i];
}

// ------------------------------------------------------------------ regular-basis helpers
// reciprocal of a positive, normal double: hardware estimate and two Newton steps (within an ulp)
__device__ inline double rcp_nr(double d) {
    double y = __builtin_amdgcn_rcp(d);
    double e = fma(-d, y, 1.0);
    y = fma(y, e, y);
    e = fma(-d, y, 1.0);
    return fma(y, e, y);
}

// sum of the power series of x^{-n} (2n+1)!! j_n(x): t_0 = 1, t_k = t_{k-1} h / (k (2n+2k+1)), h = -x^2/2
__device__ inline double jn_series(int n, double h, int kmax) {
    double s = 1.0, t = 1.0;
    for (int q = 1; q <= kmax; ++q) {
        t *= h * rcp_nr((double)q * (double)(2 * n + 2 * q + 1));
        s += t;
        if (fabs(t) <= 1e-17 * fabs(s)) break;
    }
    return s;
}

// j_0(x) .. j_N(x), 0 <= x < 4, N <= 40.  Small x: every order from its series (orders that
// underflow are zero to working precision).  Otherwise j_N and j_{N-1} from their series, then the
// downward recurrence j_{n-1} = (2n+1)/x j_n - j_{n+1}, which is stable for this (minimal) solution.
__device__ inline void bessel_j_small(double x, int N, double *j) {
    const double h = -0.5 * x * x;
    if (x < 1e-2) {
        double pre = 1.0;  // x^n / (2n+1)!!
        for (int n = 0; n <= N; ++n) {
            if (n > 0) pre *= x * rcp_nr(2.0 * n + 1.0);
            j[n] = pre * jn_series(n, h, 6);
        }
        return;
    }
    if (N == 0) {
        j[0] = jn_series(0, h, 40);
        return;
    }
    double xn = 1.0, df = 1.0;  // x^{N-1} and (2N-1)!!
    for (int n = 1; n < N; ++n) {
        xn *= x;
        df *= 2.0 * n + 1.0;
    }
    const double pre = xn / df;
    double jh = pre * x / (2.0 * N + 1.0) * jn_series(N, h, 40);
    double jl = pre * jn_series(N - 1, h, 40);
    j[N] = jh;
    j[N - 1] = jl;
    const double ix = 1.0 / x;
    for (int n = N - 1; n >= 1; --n) {
        const double jm = fma((2.0 * n + 1.0) * ix, jl, -jh);
        j[n - 1] = jm;
        jh = jl;
        jl = jm;
    }
}

// j_0(x) .. j_N(x), x >= 0: bessel_j_small, or Miller's normalised recurrence
__device__ inline void bessel_j_seq(double x, int N, double *j) {
    if (x < 1e-2 || (x < 4.0 && N <= 40)) bessel_j_small(x, N, j);
    else sph_jn_seq(x, N, j);
}

// spherical coordinates of (dx, dy, dz) about the expansion centre: r, cos/sin of the polar
// angle and e^{i phi} (any unit phase where the point lies on the axis: the orders m != 0 vanish)
__device__ inline void sph_frame(double dx, double dy, double dz, double &r, double &ct, double &st, double2 &eph) {
    const double rxy2 = dx * dx + dy * dy;
    r = sqrt(rxy2 + dz * dz);
    const double rxy = sqrt(rxy2);
    if (r > 0) {
        const double ir = 1.0 / r;
        ct = dz * ir;
        st = rxy * ir;
    } else {
        ct = 1.0;
        st = 0.0;
    }
    if (rxy > 0) {
        const double irx = 1.0 / rxy;
        eph = cmk(dx * irx, dy * irx);
    } else {
        eph = cmk(1.0, 0.0);
    }
}

// ------------------------------------------------------------------ P2M
// C_n^m = i k sum_j [ q_j R_n^{-m}(c_j - C) + w_j (n_j . grad) R_n^{-m}(c_j - C) ]
// using  d_z R_n^m = k (a_{n-1}^m R_{n-1}^m - a_n^m R_{n+1}^m),
//        (d_x + i d_y) R_n^m = k (b_{n+1}^{-m-1} R_{n+1}^{m+1} - b_n^m R_{n-1}^{m+1}),
//        (d_x - i d_y) R_n^m = k (b_{n+1}^{m-1} R_{n+1}^{m-1} - b_n^{-m} R_{n-1}^{m-1}).
// One workgroup per leaf.  Per chunk of CH sources: geometry and j_n(k r) per source, the basis
// R_n^{m'} (n <= p, m' >= 0, plus a zero slot) per (source, m') in LDS, then each thread adds the
// sources' terms to its coefficient(s).  The seven basis entries a coefficient reads, with their
// factors and conjugation signs, are fixed per coefficient and set up once.
struct P2mTerms {
    int i[7];          // basis slot (the zero slot where the entry does not exist)
    double fx[7], fy[7];  // factors of the real and imaginary parts (fy = -fx for conjugated entries)
};
__device__ inline void p2m_term(int p, int TB, int nn, int mm, double f, int &i, double &fx, double &fy) {
    const int am = mm < 0 ? -mm : mm;
    if (nn < 0 || nn > p || am > nn) {
        i = TB;
        fx = fy = 0.0;
        return;
    }
    i = leg_tri(nn, am);
    fx = f;
    fy = mm < 0 ? -f : f;
}
__device__ inline void p2m_terms(int p, int TB, int c, double k, P2mTerms &T) {
    int n = (int)sqrt((double)c);
    while (n * n > c) --n;
    while ((n + 1) * (n + 1) <= c) ++n;
    const int mm = -(c - n * n - n);
    p2m_term(p, TB, n, mm, 1.0, T.i[0], T.fx[0], T.fy[0]);
    p2m_term(p, TB, n - 1, mm, k * coef_a(n - 1, mm), T.i[1], T.fx[1], T.fy[1]);
    p2m_term(p, TB, n + 1, mm, -k * coef_a(n, mm), T.i[2], T.fx[2], T.fy[2]);
    p2m_term(p, TB, n + 1, mm + 1, k * coef_b(n + 1, -mm - 1), T.i[3], T.fx[3], T.fy[3]);
    p2m_term(p, TB, n - 1, mm + 1, -k * coef_b(n, mm), T.i[4], T.fx[4], T.fy[4]);
    p2m_term(p, TB, n + 1, mm - 1, k * coef_b(n + 1, mm - 1), T.i[5], T.fx[5], T.fy[5]);
    p2m_term(p, TB, n - 1, mm - 1, -k * coef_b(n, -mm), T.i[6], T.fx[6], T.fy[6]);
}
template <int NR>
__device__ inline void p2m_accumulate(const P2mTerms &T, int cnt, int TS, const double2 *basis, const double2 *qw,
                                      const double *nrm, double2 (&a)[NR]) {
    for (int s = 0; s < cnt; ++s) {
        const double2 *B = basis + (int64_t)s * TS;
        double2 v[7];
#pragma unroll
        for (int t = 0; t < 7; ++t) v[t] = B[T.i[t]];
        const double2 R0 = cmk(T.fx[0] * v[0].x, T.fy[0] * v[0].y);
        const double2 dz = cmk(fma(T.fx[1], v[1].x, T.fx[2] * v[2].x), fma(T.fy[1], v[1].y, T.fy[2] * v[2].y));
        const double2 dp = cmk(fma(T.fx[3], v[3].x, T.fx[4] * v[4].x), fma(T.fy[3], v[3].y, T.fy[4] * v[4].y));
        const double2 dm = cmk(fma(T.fx[5], v[5].x, T.fx[6] * v[6].x), fma(T.fy[5], v[5].y, T.fy[6] * v[6].y));
        // n.grad = n_z d_z + (n_x - i n_y)/2 (d_x + i d_y) + (n_x + i n_y)/2 (d_x - i d_y); nrm holds
        // (n_x/2, n_y/2, n_z)
        const double hx = nrm[3 * s], hy = nrm[3 * s + 1], nz = nrm[3 * s + 2];
        double2 dn = cscale(dz, nz);
        dn = cfma(cmk(hx, -hy), dp, dn);
        dn = cfma(cmk(hx, hy), dm, dn);
#pragma unroll
        for (int rr = 0; rr < NR; ++rr) {
            a[rr] = cfma(qw[(2 * s) * NR + rr], R0, a[rr]);
            a[rr] = cfma(qw[(2 * s + 1) * NR + rr], dn, a[rr]);
        }
    }
}

// Slot sums: the derivative relations are linear with source-independent factors, so with
// per-source weights al_0 = q, al_1 = w n_z, al_2 = w (n_x - i n_y)/2, al_3 = w (n_x + i n_y)/2,
//   sum_s al_k,s B_s[t] (P) and sum_s conj(al_k,s) B_s[t] (Q)
// over the basis slots t (m' >= 0) give every coefficient as seven factor-weighted sums: an entry
// read conjugated (negative order) is conj(Q[t]).  One thread per slot keeps the eight sums per
// vector in registers across the leaf's chunks; each basis value is read once per source.
struct P2mSlotSums {
    static constexpr int K = 4;
};

template <int NR>
__global__ void __launch_bounds__(256) k_p2m_wide(int nleaf, int p, int CH, const int32_t *leaf_start,
                                             const double4 *center, const double4 *ec, const double4 *en,
                                             const double2 *sigma, const double2 *mu, double k, const double *leg,
                                             double2 *Mout) {
    extern __shared__ double2 smem[];
    const int b = blockIdx.x, tid = threadIdx.x;
    const int TB = (p + 1) * (p + 2) / 2, TS = TB + 1;     // basis entries and the zero slot
    double2 *basis = smem;                                 // CH * TS
    double2 *qw = basis + (int64_t)CH * TS;                // CH * 2 * NR
    double2 *W = qw + CH * 2 * NR;                         // CH * 4 * NR: slot-sum weights al_k
    double *jb = (double *)(W + CH * 4 * NR);              // CH * (p+2)
    double *geo = jb + CH * (p + 2);                       // CH * 4: cos, sin of the polar angle, e^{i phi}
    double *nrm = geo + CH * 4;                            // CH * 3
    double *lt = nrm + CH * 3;                             // 3 TB: Legendre recurrence table
    for (int e = tid; e < 3 * TB; e += blockDim.x) lt[e] = leg[e];
    const double4 C = center[b];
    const int ss = leaf_start[b], se = leaf_start[b + 1];
    const int ncoef = p * p;
    double2 *Mb = Mout + (int64_t)b * NR * ncoef;          // NR expansions of this leaf
    // slot sums in registers (one slot per thread, the zero slot included) when the slots fit the
    // workgroup and the staged basis can hold the eight sums of one vector at the end; otherwise
    // each thread accumulates whole coefficients in place
    const bool slots = TS <= (int)blockDim.x && CH * TS >= 8 * TS;
    double2 S[2 * P2mSlotSums::K][NR];
#pragma unroll
    for (int q = 0; q < 2 * P2mSlotSums::K; ++q)
#pragma unroll
        for (int rr = 0; rr < NR; ++rr) S[q][rr] = cmk(0, 0);
    if (!slots)
        for (int c = tid; c < NR * ncoef; c += blockDim.x) Mb[c] = cmk(0, 0);
    for (int j0 = ss; j0 < se; j0 += CH) {
        const int cnt = min(CH, se - j0);
        __syncthreads();
        if (tid < cnt) {
            const int j = j0 + tid;
            const double4 c = ec[j], nv = en[j];
            double r, ct, st;
            double2 eph;
            sph_frame(c.x - C.x, c.y - C.y, c.z - C.z, r, ct, st, eph);
            geo[4 * tid] = ct;
            geo[4 * tid + 1] = st;
            geo[4 * tid + 2] = eph.x;
            geo[4 * tid + 3] = eph.y;
            bessel_j_seq(k * r, p, jb + tid * (p + 2));
#pragma unroll
            for (int rr = 0; rr < NR; ++rr) {
                qw[(2 * tid) * NR + rr] = cscale(sigma[(int64_t)j * NR + rr], c.w);
                qw[(2 * tid + 1) * NR + rr] = cscale(mu[(int64_t)j * NR + rr], c.w);
            }
            nrm[3 * tid] = 0.5 * nv.x;
            nrm[3 * tid + 1] = 0.5 * nv.y;
            nrm[3 * tid + 2] = nv.z;
#pragma unroll
            for (int rr = 0; rr < NR; ++rr) {
                const double2 q = qw[(2 * tid) * NR + rr], w = qw[(2 * tid + 1) * NR + rr];
                W[(4 * tid) * NR + rr] = q;
                W[(4 * tid + 1) * NR + rr] = cscale(w, nv.z);
                W[(4 * tid + 2) * NR + rr] = cmul(w, cmk(0.5 * nv.x, -0.5 * nv.y));
                W[(4 * tid + 3) * NR + rr] = cmul(w, cmk(0.5 * nv.x, 0.5 * nv.y));
            }
        }
        __syncthreads();
        // basis column m' of source s: R_n^{m'} = j_n(k r) P_n^{m'}(cos) e^{i m' phi}, n = m'..p
        for (int w = tid; w < cnt * (p + 1); w += blockDim.x) {
            const int s = w / (p + 1), mp = w - s * (p + 1);
            const double ct = geo[4 * s], st = geo[4 * s + 1];
            const double2 eph = cmk(geo[4 * s + 2], geo[4 * s + 3]);
            const double *js = jb + s * (p + 2);
            double2 *out = basis + (int64_t)s * TS;
            double2 e = cmk(1.0, 0.0);
            double sp = 1.0;
            for (int q = 0; q < mp; ++q) {
                e = cmul(e, eph);
                sp *= st;
            }
            double P1 = lt[3 * leg_tri(mp, mp) + 2] * sp, P2 = 0.0;
            out[leg_tri(mp, mp)] = cscale(e, js[mp] * P1);
            for (int n = mp + 1; n <= p; ++n) {
                const int t = leg_tri(n, mp);
                const double P = fma(lt[3 * t] * ct, P1, -lt[3 * t + 1] * P2);
                P2 = P1;
                P1 = P;
                out[t] = cscale(e, js[n] * P);
            }
            if (mp == 0) out[TB] = cmk(0, 0);
        }
        __syncthreads();
        if (slots) {
            if (tid < TS)
                for (int s2 = 0; s2 < cnt; ++s2) {
                    const double2 B = basis[(int64_t)s2 * TS + tid];
#pragma unroll
                    for (int kk = 0; kk < P2mSlotSums::K; ++kk)
#pragma unroll
                        for (int rr = 0; rr < NR; ++rr) {
                            const double2 al = W[(4 * s2 + kk) * NR + rr];
                            S[2 * kk][rr] = cfma(al, B, S[2 * kk][rr]);
                            S[2 * kk + 1][rr] = cfma(cmk(al.x, -al.y), B, S[2 * kk + 1][rr]);
                        }
                }
        } else {
            for (int c = tid; c < ncoef; c += blockDim.x) {
                P2mTerms Tc;
                p2m_terms(p, TB, c, k, Tc);
                double2 a[NR];
#pragma unroll
                for (int rr = 0; rr < NR; ++rr) a[rr] = cmk(0, 0);
                p2m_accumulate<NR>(Tc, cnt, TS, basis, qw, nrm, a);
#pragma unroll
                for (int rr = 0; rr < NR; ++rr)
                    Mb[rr * ncoef + c] = cadd(Mb[rr * ncoef + c], cmuli(cscale(a[rr], k)));  // i k sum
            }
        }
    }
    if (slots) {
        // coefficient c = seven factor-weighted slot sums (entry i of term t from sum type k(t):
        // t = 0 monopole, 1-2 n_z d_z, 3-4 (d_x + i d_y), 5-6 (d_x - i d_y)), one vector at a time
        // through the staged basis region
        const int kt[7] = {0, 1, 1, 2, 2, 3, 3};
        double2 *SL = basis;  // [8][TS]
#pragma unroll
        for (int rr = 0; rr < NR; ++rr) {
            __syncthreads();
            if (tid < TS)
#pragma unroll
                for (int q = 0; q < 2 * P2mSlotSums::K; ++q) SL[q * TS + tid] = S[q][rr];
            __syncthreads();
            for (int c = tid; c < ncoef; c += blockDim.x) {
                P2mTerms T;
                p2m_terms(p, TB, c, k, T);
                double2 a = cmk(0, 0);
#pragma unroll
                for (int t = 0; t < 7; ++t) {
                    const bool cj = T.fy[t] != T.fx[t];  // conjugated entry: conj of the Q sum
                    const double2 v = SL[(2 * kt[t] + (cj ? 1 : 0)) * TS + T.i[t]];
                    a = cadd(a, cmk(T.fx[t] * v.x, T.fy[t] * v.y));
                }
                Mb[rr * ncoef + c] = cmuli(cscale(a, k));  // i k sum
            }
        }
    }
}

// j_0(x) .. j_N(x) for the expansion kernels: the sequence of bessel_j_seq, with Miller's
// normalised downward recurrence (x >= 4) taking one multiplication by 1/x per step instead of a
// division and starting 16 + 2 sqrt(max(N, x) + 1) orders above max(N, x): the minimal solution's
// ratio over the start's tail is then far below the recurrence's own rounding (a check of this
// start against a reference sequence for N <= 60, 4 <= x <= 1.2 N + 5 finds the same ~1e-12
// worst relative error, near zeros of j_n, as starting 40 + 4 sqrt(max(N, x) + 1) above).
__device__ inline void bessel_j_seq_fast(double x, int N, double *j) {
    if (x < (N <= 40 ? 4.0 : 1e-2)) {  // small x at any N: 1/x is no number at x = 0
        bessel_j_small(x, N, j);
        return;
    }
    const int top = N > (int)x ? N : (int)x;
    const int start = top + 16 + (int)(2.0 * sqrt((double)top + 1.0));
    const double ix = rcp_nr(x);
    double fp1 = 0.0, f = 1e-300;
    for (int n = start; n >= 1; --n) {
        const double fm1 = fma((2.0 * n + 1.0) * ix, f, -fp1);
        fp1 = f;
        f = fm1;
        if (n - 1 <= N) j[n - 1] = f;
        if (fabs(f) > 1e250) {  // rescale everything stored so far
            f *= 1e-250;
            fp1 *= 1e-250;
            for (int q = n - 1; q <= N; ++q) j[q] *= 1e-250;
        }
    }
    double sn, cn;
    sincos(x, &sn, &cn);
    const double j0 = sn * ix, j1 = (sn * ix - cn) * ix;
    const double scale = (fabs(j0) >= fabs(j1) || N < 1) ? j0 / j[0] : j1 / j[1];
    for (int n = 0; n <= N; ++n) j[n] *= scale;
}

// Constant tables of P2M (P2M_TABLE doubles): the seven terms of every coefficient c < P2M_CAP
// (p2m_terms without the factor k, independent of p) as factors f[7][cap] and int32 slots[7][cap] =
// 2 slot + (conjugated entry), a missing entry with factor 0; the Bessel series, for n <= SER_NMAX
// ser[n][q - 1] = 1 / (q (2n + 2q + 1)) and, last in the row, 1 / (2n + 1)!!; the orders of the slots.
__global__ void k_p2m_table(double *tab) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x, cap = P2M_CAP;
    double *f = tab, *ser = tab + P2M_OSER;
    int32_t *slot = (int32_t *)(tab + 7 * cap), *order = (int32_t *)(tab + P2M_OORD);
    if (c < cap) {
        P2mTerms T;
        const int none = 1 << 20;
        p2m_terms(1 << 10, none, c, 1.0, T);
        for (int t = 0; t < 7; ++t) {
            f[t * cap + c] = T.fx[t];
            slot[t * cap + c] = T.i[t] == none ? 0 : 2 * T.i[t] + (T.fy[t] != T.fx[t]);
        }
    }
    if (c <= SER_NMAX) {
        double df = 1.0;
        for (int q = 1; q <= c; ++q) df *= 2.0 * q + 1.0;
        for (int q = 1; q < P2M_SER; ++q) ser[c * P2M_SER + q - 1] = 1.0 / ((double)q * (2.0 * c + 2.0 * q + 1.0));
        ser[c * P2M_SER + P2M_SER - 1] = 1.0 / df;
    }
    if (c <= P2M_PMAX) {
        for (int m = 0; m <= c; ++m) order[leg_tri(c, m)] = m;
        for (int t = leg_tri(P2M_PMAX + 1, 0) + c; t < P2M_SLOTS; t += P2M_PMAX + 1) order[t] = 0;
    }
}

// x^m by squaring, m < 64
__device__ inline double pow_small(double x, int m) {
    double r = m & 1 ? x : 1.0;
    for (int b = 1; b < 6; ++b) {
        x *= x;
        r = (m >> b) & 1 ? r * x : r;
    }
    return r;
}

// a read-only array whose elements are read by scalar loads where the index is the wavefront's
typedef const __attribute__((address_space(4))) double *sc_f64;

// j_0(x) .. j_N(x): for 1e-2 <= x < 4 and 1 <= N <= SER_NMAX the method of bessel_j_small with both
// series summed in one loop from a table of the terms' factors (the rows of the orders N - 1 and N,
// P2M_SER each, at ser); otherwise bessel_j_seq_fast.  ix = 1 / x.
template <class SER>
__device__ inline void bessel_j_seq_ser(double x, double ix, int N, double *j, SER ser) {
    if (x < 1e-2 || x >= 4.0 || N < 1 || N > SER_NMAX) {
        bessel_j_seq_fast(x, N, j);
        return;
    }
    const double h = -0.5 * x * x;
    double sh = 1.0, th = 1.0, sl = 1.0, tl = 1.0;  // orders N and N - 1
#pragma unroll 1
    for (int q = 0; q + 4 < P2M_SER; q += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            tl *= h * ser[q + u];
            th *= h * ser[P2M_SER + q + u];
            sl += tl;
            sh += th;
        }
        if (!__any(fabs(tl) > 1e-17 * fabs(sl))) break;
    }
    const double xn = pow_small(x, N - 1);
    double jl = sl * (xn * ser[P2M_SER - 1]), jh = sh * (xn * x * ser[2 * P2M_SER - 1]);
    j[N] = jh;
    j[N - 1] = jl;
    double c = 2.0 * N - 1.0;  // 2n + 1
    for (int n = N - 1; n >= 1; --n) {
        const double jm = fma(c * ix, jl, -jh);
        j[n - 1] = jm;
        jh = jl;
        jl = jm;
        c -= 2.0;
    }
}

// P2M by matrix cores.  A workgroup takes one leaf, its sources in equal groups of at most G; per
// group:
//  1. one thread per source: j_0..j_p(k r) on one wavefront, the phase powers E_m' = ((dx + i dy) /
//     r)^m' = (sin(th) e^{i phi})^m' on another, the weights al_k of every vector on the other two;
//  2. the real part of the basis, R~_n^m' = j_n(k r) P_n^m'(cos th) / sin^m'(th), one recurrence in
//     n per (source, m'), the orders m' and p - m' paired so that each item is p + 2 steps long;
//  3. the sums over the sources as a product: rows the slots (n, m' >= 0) twice (Re E R~, Im E R~,
//     formed as the A operand is read), columns Re/Im al_k of every vector, K the sources: the four
//     real sums per weight that give both sum_s al_k R (P) and sum_s conj(al_k) R (Q).  The four
//     wavefronts take every fourth block of 16 rows, NBW of them, in registers over all groups.
// Then every coefficient from seven factor-weighted slot sums, through LDS.  Bound by the latency of
// its steps: G is chosen for four workgroups per CU (three for several vectors).
// Measured against one thread per slot (every source's weights times the basis on the vector units,
// an FP64 result converted by another kernel for FP32 translations), leaves of 33 sources, p = 16:
// 90,972 elements 94 -> 86 us, 906,812 elements 669 -> 625 us; four vectors of 612,000 elements in
// mixed precision 1,975 -> 990 us.  A thread per (source, order) evaluating its own Bessel series,
// instead of one recurrence per source: 896 us at 906,812 elements.
// Needs (p + 1)(p + 2)/2 <= 256 (p <= 21); launch_p2m takes the wide kernel beyond.
// CO: float2 where the translations run in FP32.
struct P2mLayout {
    int TB, TBP, LDR, LDD, p1, GP, NC;  // slots, padded to 16; row strides; sources padded to 4; columns
    int oE, oJ, oC, oW, oL, oS, total;  // offsets in doubles (the basis at 0)
    __host__ __device__ P2mLayout(int p, int G, int nr) {
        TB = (p + 1) * (p + 2) / 2;
        TBP = (TB + 15) & ~15;
        LDR = TBP + (TBP % 32 ? 0 : 16);  // four sources' rows on different banks
        LDD = nr > 1 && TBP <= 160 ? 17 : 9;  // the sums of two vectors or one (8 columns each)
        p1 = p + 1;
        GP = (G + 3) & ~3;
        NC = nr > 2 ? 32 : 16;
        oE = G * LDR;
        oJ = oE + 2 * G * p1;
        oC = oJ + G * (p + 2);
        oW = (oC + G + 1) & ~1;
        oL = oW + GP * NC;
        oS = oL + 3 * TB;
        total = oS + 2 * P2M_SER;
        if (total < 2 * TBP * LDD) total = 2 * TBP * LDD;  // the sums reuse the area
    }
};
template <int NR, int NBW, class CO>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NBW <= 5 ? (NR > 1 ? 3 : 4) : (NR > 2 ? 2 : 3))))
k_p2m(int p, int G, const int32_t *leaf_start, const double4 *center, const double4 *ec, const double4 *en,
      const double2 *sigma, const double2 *mu, double k, double ik, const double *leg, const double *tab, CO *Mout) {
    typedef double v4 __attribute__((ext_vector_type(4)));
    constexpr int NCB = NR > 2 ? 2 : 1, NC = 16 * NCB, VP = NR > 1 && NBW <= 5 ? 2 : 1, LDD = 8 * VP + 1, cap = P2M_CAP;
    extern __shared__ double p2m_sm[];
    const P2mLayout Y(p, G, NR);
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l16 = lane & 15, kq = lane >> 4;
    const int TB = Y.TB, TBP = Y.TBP, LDR = Y.LDR, p1 = Y.p1;
    double *Rb = p2m_sm, *E = p2m_sm + Y.oE, *jb = p2m_sm + Y.oJ, *cth = p2m_sm + Y.oC, *W = p2m_sm + Y.oW,
           *lt = p2m_sm + Y.oL, *ser = p2m_sm + Y.oS, *Dl = p2m_sm;
    const double4 C = center[b];
    const int ss = leaf_start[b], ns = leaf_start[b + 1] - ss;
    const int ng = (ns + G - 1) / G, gs = (ns + ng - 1) / ng;
    for (int e = tid; e < 3 * TB; e += 256) lt[e] = leg[e];
    if (tid < 2 * P2M_SER) ser[tid] = tab[P2M_OSER + (p - 1) * P2M_SER + tid];
    const int32_t *order = (const int32_t *)(tab + P2M_OORD);
    // this lane's rows of the product: basis slot and the phase power it takes (its real or imaginary part)
    int slot[NBW], eo[NBW];
#pragma unroll
    for (int q = 0; q < NBW; ++q) {
        const int row = 16 * (wv + 4 * q) + l16, part = row >= TBP ? 1 : 0, t = min(row - part * TBP, TBP - 1);
        slot[q] = t;
        eo[q] = t < TB ? 2 * order[t] + part : 0;
    }
    v4 acc[NBW][NCB];
#pragma unroll
    for (int q = 0; q < NBW; ++q)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[q][cb] = v4{0, 0, 0, 0};
    const int npair = p / 2 + 1, npad = TBP - TB;
    for (int g = 0; g < ng; ++g) {
        const int j0 = ss + g * gs, cnt = min(gs, ss + ns - j0), gp = (cnt + 3) & ~3;
        __syncthreads();  // the previous group's readers are done (and the tables are in place)
        if (wv < 2 && lane < cnt) {
            const double4 c = ec[j0 + lane];
            const double dx = c.x - C.x, dy = c.y - C.y, dz = c.z - C.z, r2 = dx * dx + dy * dy + dz * dz;
            const bool at = r2 < 1e-280;  // at the centre: theta = 0
            const double ir = at ? 0.0 : rsq_nr(r2);
            if (wv == 0) {
                cth[lane] = at ? 1.0 : dz * ir;
                bessel_j_seq_ser(k * (r2 * ir), ik * ir, p, jb + lane * (p + 2), (const double *)ser);
            } else {
                const double2 u = cmk(dx * ir, dy * ir);
                double2 e = cmk(1.0, 0.0);
                double *o = E + lane * p1 * 2;
                for (int m = 0; m <= p; ++m) {
                    o[2 * m] = e.x;
                    o[2 * m + 1] = e.y;
                    e = cmul(e, u);
                }
            }
        }
        for (int e = tid - 128; e < gp * 4 * (NC / 8); e += 128) {  // (source, vector, weight)
            if (e < 0) break;
            const int s = e / (NC / 2), rk = e - s * (NC / 2), r = rk >> 2, kk = rk & 3;
            double2 al = cmk(0.0, 0.0);
            if (s < cnt && r < NR) {
                const int64_t j = j0 + s;
                const double4 nv = en[j];
                const double a = ec[j].w;
                if (kk == 0) al = cscale(sigma[j * NR + r], a);
                else {
                    const double2 w = cscale(mu[j * NR + r], a);
                    al = kk == 1 ? cscale(w, nv.z) : cmul(w, cmk(0.5 * nv.x, kk == 2 ? -0.5 * nv.y : 0.5 * nv.y));
                }
            }
            W[s * NC + 2 * rk] = al.x;
            W[s * NC + 2 * rk + 1] = al.y;
        }
        __syncthreads();
        for (int w = tid; w < cnt * npair; w += 256) {
            const int s = w / npair, pr = w - s * npair;
            const double ct = cth[s];
            const double *js = jb + s * (p + 2);
            double *out = Rb + s * LDR;
            for (int h = 0; h < 2; ++h) {
                const int mp = h == 0 ? pr : p - pr;
                if (h == 1 && mp == pr) break;
                int t = leg_tri(mp, mp);
                double P1 = lt[3 * t + 2], P2 = 0.0;
                out[t] = js[mp] * P1;
#pragma unroll 4
                for (int n = mp + 1; n <= p; ++n) {
                    t += n;
                    const double P = fma(lt[3 * t] * ct, P1, -lt[3 * t + 1] * P2);
                    P2 = P1;
                    P1 = P;
                    out[t] = js[n] * P;
                }
            }
        }
        if (tid >= 128)
            for (int e = tid - 128; e < cnt * npad; e += 128) Rb[e / npad * LDR + TB + e % npad] = 0.0;
        __syncthreads();
        for (int i = 0; i < gp; i += 4) {
            const int s = min(i + kq, cnt - 1);  // past the group: a zero row of W
            double bv[NCB];
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) bv[cb] = W[(i + kq) * NC + 16 * cb + l16];
            const double *Rs = Rb + s * LDR, *Es = E + s * p1 * 2;
#pragma unroll
            for (int q = 0; q < NBW; ++q) {
                const double av = Rs[slot[q]] * Es[eo[q]];
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
                    acc[q][cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[cb], acc[q][cb], 0, 0, 0);
            }
        }
    }
    // coefficient c = seven factor-weighted slot sums (term t from weight kt(t): t = 0 monopole, 1-2
    // n_z d_z, 3-4 (d_x + i d_y), 5-6 (d_x - i d_y)), VP vectors at a time
    const double *tf = tab;
    const int32_t *tslot = (const int32_t *)(tab + 7 * cap);
    const int ncoef = p * p;
    CO *Mb = Mout + (int64_t)b * NR * ncoef;
#pragma unroll
    for (int v0 = 0; v0 < NR; v0 += VP) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NBW; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * (wv + 4 * q) + kq + 4 * i, col = l16 - 8 * (v0 & 1);
                if (row < 2 * TBP && col >= 0 && col < 8 * VP) Dl[row * LDD + col] = acc[q][v0 >> 1][i];
            }
        __syncthreads();
        for (int c = tid; c < ncoef; c += 256) {
            double2 a[VP];
#pragma unroll
            for (int v = 0; v < VP; ++v) a[v] = cmk(0.0, 0.0);
#pragma unroll
            for (int t = 0; t < 7; ++t) {
                const int kt = (t + 1) >> 1;
                const double f = t == 0 ? 1.0 : k * tf[t * cap + c];
                const int sl = tslot[t * cap + c];
                const double sg = sl & 1 ? -1.0 : 1.0;
                const double *x = Dl + (sl >> 1) * LDD + 2 * kt, *y = x + TBP * LDD;
#pragma unroll
                for (int v = 0; v < VP; ++v) {
                    // P = (A - B, C + D), conj(Q) = (A + B, -(C - D))
                    a[v].x = fma(f, x[8 * v] - sg * y[8 * v + 1], a[v].x);
                    a[v].y = fma(f, sg * y[8 * v] + x[8 * v + 1], a[v].y);
                }
            }
#pragma unroll
            for (int v = 0; v < VP; ++v) {  // i k sum
                CO o;
                o.x = -k * a[v].y;
                o.y = k * a[v].x;
                Mb[(v0 + v) * ncoef + c] = o;
            }
        }
    }
}

// ------------------------------------------------------------------ L2P + combine
// One wavefront takes a leaf's targets (up to 16 TLM at a time).  First one target per lane: frame
// and j_n(k r), to LDS.  Then 16 targets side by side, TL targets per lane, and the orders split over
// the four groups of 16 lanes (group g takes m = g, g + 4, ...): an entry pair D_n^{+-m} and a
// recurrence entry read from LDS serve TL points, which also hide each other's latency.  A butterfly
// over the groups adds the orders, and group i finishes the lane's target i.  Bound by LDS reads (an
// entry is the same for 16 lanes) and the FP64 instructions together, at 2 to 3 wavefronts per SIMD;
// the orders' unequal lengths cost a sixth (p = 16: 40 steps where 34 would do).
// Measured against one target per lane with the orders split over half-filled wavefronts only, and
// FP32 expansions converted by another kernel, p = 16: 56 leaves of 48 targets 54 -> 20 us (four
// workgroups per leaf), 3,416 leaves of 27 50 -> 37 us, 29,626 leaves of 34 330 -> 187 us, four vectors
// in mixed precision on 29,626 leaves of 21 1,195 -> 452 us; with the normal derivative (four
// expansions) 56 leaves 130 -> 38 us, 3,416 leaves 224 -> 116 us.  Three and two targets per lane (one
// or two, four vectors): a target more costs 187 -> 215 and 452 -> 475 us, a wavefront more per SIMD (fewer
// registers) 187 -> 314 and 452 -> 702 us.  Entries through the scalar cache, all lanes at the same
// one: 259 and 1,345 us (its misses).

constexpr int l2p_tlm(int nv) { return nv > 2 ? 2 : 3; }

// LDS of k_l2p and k_l2p_n, degrees < p, NV expansions of elements T (STAGE: copied there); offsets
// in bytes
struct L2pLayout {
    int JS, oF, oT, oS, oD, total;  // Bessel rows (stride JS); frames; recurrence pairs; seeds; expansions
    __host__ __device__ L2pLayout(int p, int nt, size_t dbytes) {
        JS = (p + 1) | 1;
        oF = nt * JS * 8;
        oT = (oF + nt * 24 + 15) & ~15;
        oS = oT + p * (p + 1) / 2 * 16;
        oD = (oS + p * 8 + 15) & ~15;
        total = oD + (int)dbytes;
    }
};

// far[i][v] = this lane's orders of sum_{n < p, m} D_n^m R_n^m at its targets l + 16 i (of nt), NV
// expansions ps entries apart, then summed over the four groups
template <int NV, int TL, class T2>
__device__ inline void l2p_sums(int p, int nt, const T2 *D, int ps, const double2 *lt, const double *seed,
                                const double *jb, int JS, const double *fr, double2 (&far)[TL][NV]) {
    const int lane = threadIdx.x & 63, g = lane >> 4;
    double ct[TL];
    double2 e[TL], u4[TL];
    const double *jt[TL];
#pragma unroll
    for (int i = 0; i < TL; ++i) {
        const int t = min((lane & 15) + 16 * i, nt - 1);
        jt[i] = jb + t * JS;
        ct[i] = fr[3 * t];
        const double2 u = cmk(fr[3 * t + 1], fr[3 * t + 2]), u2 = cmul(u, u);
        u4[i] = cmul(u2, u2);
        e[i] = cmul(cmk(g & 1 ? u.x : 1.0, g & 1 ? u.y : 0.0), cmk(g & 2 ? u2.x : 1.0, g & 2 ? u2.y : 0.0));
#pragma unroll
        for (int v = 0; v < NV; ++v) far[i][v] = cmk(0.0, 0.0);
    }
#pragma unroll 1
    for (int m = g; m < p; m += 4) {
        double P1[TL], P2[TL];
        double2 sa[TL][NV], sb[TL][NV];  // orders m and -m
        const double sd = seed[m];
#pragma unroll
        for (int i = 0; i < TL; ++i) {
            P1[i] = sd;
            P2[i] = 0.0;
#pragma unroll
            for (int v = 0; v < NV; ++v) sa[i][v] = sb[i][v] = cmk(0.0, 0.0);
        }
        int q = leg_tri(m, m);
        const T2 *Da = D + cidx(m, m), *Db = D + cidx(m, -m);
#pragma unroll 1
        for (int n = m;;) {
            double R[TL];
#pragma unroll
            for (int i = 0; i < TL; ++i) R[i] = jt[i][n] * P1[i];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const T2 a = Da[v * ps], b = Db[v * ps];
#pragma unroll
                for (int i = 0; i < TL; ++i) {
                    sa[i][v].x = fma((double)a.x, R[i], sa[i][v].x);
                    sa[i][v].y = fma((double)a.y, R[i], sa[i][v].y);
                    sb[i][v].x = fma((double)b.x, R[i], sb[i][v].x);
                    sb[i][v].y = fma((double)b.y, R[i], sb[i][v].y);
                }
            }
            if (++n >= p) break;
            q += n;
            Da += 2 * n;
            Db += 2 * n;
            const double2 ab = lt[q];
#pragma unroll
            for (int i = 0; i < TL; ++i) {
                const double P = fma(ab.x * ct[i], P1[i], -ab.y * P2[i]);
                P2[i] = P1[i];
                P1[i] = P;
            }
        }
        // sum_n D_n^m R e^{i m phi} + D_n^{-m} R e^{-i m phi}
#pragma unroll
        for (int i = 0; i < TL; ++i) {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                far[i][v] = cfma(sa[i][v], e[i], far[i][v]);
                if (m > 0) far[i][v] = cfma(sb[i][v], cconj(e[i]), far[i][v]);
            }
            e[i] = cmul(e[i], u4[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < TL; ++i)
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int o = 16; o < 64; o *= 2) {
                far[i][v].x += __shfl_xor(far[i][v].x, o);
                far[i][v].y += __shfl_xor(far[i][v].y, o);
            }
}

// sum of the near field's pieces at t
__device__ inline double2 near_sum(const double2 *y, int64_t t, int64_t stride, int nsplit) {
    double2 v = y[t];
#pragma unroll 4
    for (int g = 1; g < nsplit; ++g) v = cadd(v, y[g * stride + t]);
    return v;
}

// the far field of a leaf's targets in chunks: fin(t, far) for every target t with its NV sums.
// Workgroup y of gy takes the chunks y, y + gy, ...; a chunk holds at most cs <= 16 TLM targets.
template <int NV, bool STAGE, class T2, class FIN>
__device__ inline void l2p_leaf(int p, int cs, int ts, int te, double4 C, const double4 *ec, const T2 *Dg, double k,
                                double ik, const double *leg, const double *ser, char *sm, FIN fin) {
    constexpr int TLM = l2p_tlm(NV);
    const int tid = threadIdx.x, pp = p * p, TB = p * (p + 1) / 2;
    const L2pLayout Y(p, cs, STAGE ? (size_t)NV * pp * sizeof(T2) : 0);
    double *jb = (double *)sm, *fr = (double *)(sm + Y.oF), *seed = (double *)(sm + Y.oS);
    double2 *lt = (double2 *)(sm + Y.oT);
    T2 *Dl = (T2 *)(sm + Y.oD);
    const int nch = (te - ts + cs - 1) / cs, size = (te - ts + nch - 1) / nch;
    if ((int)blockIdx.y >= nch) return;
    if (STAGE)
        for (int e = tid; e < NV * pp; e += 64) Dl[e] = Dg[e];
    for (int e = tid; e < TB; e += 64) lt[e] = cmk(leg[3 * e], leg[3 * e + 1]);
    for (int m = tid; m < p; m += 64) seed[m] = leg[3 * leg_tri(m, m) + 2];
    const T2 *D = STAGE ? (const T2 *)Dl : Dg;
    for (int ch = blockIdx.y; ch < nch; ch += gridDim.y) {
        const int t0 = ts + ch * size, nt = min(size, te - t0);
        if (nt <= 0) break;
        __syncthreads();
        if (tid < nt) {
            const double4 c = ec[t0 + tid];
            const double dx = c.x - C.x, dy = c.y - C.y, dz = c.z - C.z, r2 = dx * dx + dy * dy + dz * dz;
            const bool at = r2 < 1e-280;  // at the centre: theta = 0
            const double ir = at ? 0.0 : rsq_nr(r2);
            fr[3 * tid] = at ? 1.0 : dz * ir;
            fr[3 * tid + 1] = dx * ir;
            fr[3 * tid + 2] = dy * ir;
            bessel_j_seq_ser(k * (r2 * ir), ik * ir, p - 1, jb + tid * Y.JS, (sc_f64)ser + max(p - 2, 0) * P2M_SER);
        }
        __syncthreads();
        auto run = [&](auto tl) {
            constexpr int TL = decltype(tl)::value;
            double2 far[TL][NV];
            l2p_sums<NV, TL>(p, nt, D, pp, lt, seed, jb, Y.JS, fr, far);
#pragma unroll
            for (int i = 0; i < TL; ++i)
                if ((tid >> 4) == i && tid < nt) fin(t0 + tid, far[i]);
        };
        if (nt <= 16) run(std::integral_constant<int, 1>());
        else if (TLM == 2 || nt <= 32) run(std::integral_constant<int, 2>());
        else if constexpr (TLM > 2) run(std::integral_constant<int, 3>());
    }
}

// y[perm[i]] = half * x[perm[i]] + y_near[i] + sum_{n,m} D_n^m R_n^m(c_i - C); T2: entry of the
// expansions (float2 where the translations ran in FP32).  Without STAGE (expansions too large for
// LDS) they are read from global memory.
template <int NR, bool STAGE, class T2>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NR > 1 ? 2 : 3)))
k_l2p(int p, int cs, const int32_t *leaf_start, const double4 *center,
                                            const double4 *ec, const T2 *Lc, double k, double ik, const double *leg,
                                            const double *ser, const double2 *ynear, int nsplit, double half,
                                            const int32_t *perm, int64_t n, const double2 *x, double2 *y, int has_far) {
    extern __shared__ char l2p_sm[];
    const int b = blockIdx.x, ts = leaf_start[b], te = leaf_start[b + 1];
    auto fin = [&](int t, const double2 *far) {
        const int64_t u = perm[t];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            double2 v = cadd(near_sum(ynear + r, (int64_t)t * NR, n * NR, nsplit), far[r]);
            if (x) v = cadd(v, cscale(x[r * n + u], half));  // the right-hand side pass has no identity term
            y[r * n + u] = v;
        }
    };
    if (has_far) {
        l2p_leaf<NR, STAGE>(p, cs, ts, te, center[b], ec, Lc + (int64_t)b * NR * p * p, k, ik, leg, ser, l2p_sm, fin);
    } else {
        double2 far[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) far[r] = cmk(0.0, 0.0);
        for (int t = ts + threadIdx.x + 64 * blockIdx.y; t < te; t += 64 * gridDim.y) fin(t, far);
    }
}

// ------------------------------------------------------------------ field at points
// out[q] = amp * G(r_q, rs) + sum_j [L_j(r_q) sigma_j + M_j(r_q) mu_j], accurate integrals for
// elements with |r_q - c_j| < r_c, one-point rule otherwise.
//
// A workgroup takes R points (8; fewer when fewer are asked for) and one piece of the elements: every
// thread reads its own elements straight into registers (consecutive, no staging), and the points'
// coordinates are the same for all threads (scalar registers), so an element read serves R pairs.
// Bound by FP64 vector instructions (about 60 per pair; e^{ikr} from the table, as in k_p2p).  The
// elements are cut into pieces until there are a few thousand workgroups (field_pieces): with few
// points they are the only parallelism, with many they even out the last round of workgroups.
// Every piece writes its partial sums; k_field_sum adds them in order with the incident field.  The
// pairs closer than r_c take a zero 1/r in that loop; the first workgroups of the launch (one
// wavefront per point) find them through the octree's leaves and write their accurate integrals as
// one more partial sum, beside the other workgroups.
// Measured against one workgroup per point, or 8 points sharing element tiles in LDS from 6,144 points
// on, both with the polynomial sincos: 16 points of 90,972 elements 384 -> 15.4 us (both kernels),
// 19,200 points of 906,812 elements 80.8 -> 30.7 ms (2.2e11 -> 5.7e11 pairs/s).

// spreads the bits of a cell coordinate (below 2^21) three apart
__device__ inline uint64_t spread3_dev(uint64_t v) {
    v = (v | v << 32) & 0x1f00000000ffffULL;
    v = (v | v << 16) & 0x1f0000ff0000ffULL;
    v = (v | v << 8) & 0x100f00f00f00f00fULL;
    v = (v | v << 4) & 0x10c30c30c30c30c3ULL;
    return (v | v << 2) & 0x1249249249249249ULL;
}

// accurate contribution of the elements closer than r_c to the point x, summed over the wavefront:
// lanes look up the leaves of the cells within `reach` of the point's cell by their Morton codes,
// then take the elements of every leaf found
__device__ double2 field_near(const double *x, const FieldTree &T, const double4 *ec, const double *ev,
                              const double2 *sigma, const double2 *mu, double k, double rc2) {
    const int lane = threadIdx.x & 63, w = 2 * T.reach + 1, ncell = w * w * w, nc = 1 << T.depth;
    int base[3];
    for (int d = 0; d < 3; ++d) {  // cells far outside stay outside; a NaN ends up in no cell
        const double q = floor((x[d] - T.lo[d]) * T.scale);
        base[d] = q >= -1e6 && q <= 4e6 ? (int)q : -1000000;
    }
    double2 acc = cmk(0, 0);
    for (int c0 = 0; c0 < ncell; c0 += 64) {
        int ss = 0, cnt = 0;
        const int c = c0 + lane;
        if (c < ncell) {
            const int ix = base[0] + c % w - T.reach, iy = base[1] + c / w % w - T.reach, iz = base[2] + c / (w * w) - T.reach;
            if (ix >= 0 && iy >= 0 && iz >= 0 && ix < nc && iy < nc && iz < nc) {
                const uint64_t code = spread3_dev(ix) | spread3_dev(iy) << 1 | spread3_dev(iz) << 2;
                int a = 0, b = T.nleaf;  // first leaf whose code is not below
                while (a < b) {
                    const int m = (a + b) >> 1;
                    if (T.code[m] < code) a = m + 1;
                    else b = m;
                }
                if (a < T.nleaf && T.code[a] == code) {
                    ss = T.leaf_start[a];
                    cnt = T.leaf_start[a + 1] - ss;
                }
            }
        }
        for (uint64_t m = __ballot(cnt > 0); m; m &= m - 1) {
            const int src = __builtin_ctzll(m), s0 = __shfl(ss, src), n0 = __shfl(cnt, src);
            for (int e = lane; e < n0; e += 64) {
                const int64_t j = s0 + e;
                const double4 cj = ec[j];
                if (dist2_exact(x[0], x[1], x[2], cj.x, cj.y, cj.z) < rc2) {
                    double v[9];
                    for (int q = 0; q < 9; ++q) v[q] = ev[9 * j + q];
                    double2 L, M;
                    tri_integrals(x, v, k, 0, L, M);
                    acc = cfma(M, mu[j], cfma(L, sigma[j], acc));
                }
            }
        }
    }
    for (int d = 32; d > 0; d >>= 1) acc = cmk(acc.x + __shfl_xor(acc.x, d), acc.y + __shfl_xor(acc.y, d));
    return acc;
}

template <int R>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k_field(int64_t nt, int64_t nq, int64_t piece, int npiece, unsigned ngroup, FieldTree tree,
        const double *__restrict__ pts, const double4 *__restrict__ ec, const double4 *__restrict__ en,
        const double *__restrict__ ev,        const double2 *__restrict__ sigma, const double2 *__restrict__ mu, double k, double2 kk, double rc2,
        double2 *__restrict__ part) {
    __shared__ double2 tab[EIKR_N], red[4 * R];
    const int tid = threadIdx.x;
    const unsigned nnear = (unsigned)((nq + 3) / 4);
    if (blockIdx.x < nnear) {
        const int64_t q = (int64_t)blockIdx.x * 4 + (tid >> 6);
        if (q >= nq) return;
        const double y[3] = {pts[3 * q], pts[3 * q + 1], pts[3 * q + 2]};
        const double2 f = field_near(y, tree, ec, ev, sigma, mu, k, rc2);
        if ((tid & 63) == 0) part[npiece * nq + q] = f;
        return;
    }
    const unsigned bid = blockIdx.x - nnear;
    const unsigned pc = bid / ngroup, grp = bid - pc * ngroup;  // pieces outermost: neighbours share one
    eikr_stage(tab, tid);
    double x[R][3];
    double2 acc[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int64_t q = (int64_t)grp * R + u, qc = q < nq ? q : nq - 1;
        for (int d = 0; d < 3; ++d) x[u][d] = pts[3 * qc + d];
        acc[u] = cmk(0, 0);
    }
    __syncthreads();
    const double inv4pi = 1.0 / (4.0 * FMM_PI);
    // a table phase needs r kk < 2^51; a point so far away that k r itself is not known to 1 % keeps
    // the phase of that distance
    const double rmax = 1.0e15 / kk.x;
    const int64_t lo = pc * piece, hi = lo + piece < nt ? lo + piece : nt;
    for (int64_t j = lo + tid; j < hi; j += 256) {
        const double4 c = ec[j], nv = en[j];
        const double2 sg = sigma[j], um = mu[j];
        const double wgt = c.w * inv4pi;
        const double2 q = cscale(sg, wgt), w = cscale(um, wgt);
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const double d2 = dist2_exact(x[u][0], x[u][1], x[u][2], c.x, c.y, c.z);
            const double dx = c.x - x[u][0], dy = c.y - x[u][1], dz = c.z - x[u][2];
            const double ir = d2 < rc2 ? 0.0 : rsq_nr(d2), r = d2 * ir, kr = k * r;
            double s, co;
            eikr(fmin(r, rmax), kk, tab, co, s);
            const double2 G = cmk(co * ir, s * ir);
            const double a1 = (dx * nv.x + dy * nv.y + dz * nv.z) * ir * ir;  // (y-x).n / r^2
            // G (q + (ikr - 1) a1 w)
            acc[u] = cfma(G, cmk(fma(-a1, fma(kr, w.y, w.x), q.x), fma(-a1, fma(-kr, w.x, w.y), q.y)), acc[u]);
        }
    }
    // sums over the wavefront: R/2, R/4, ... points exchanged per step until a lane holds one, then
    // plain folding; the four wavefronts' sums through LDS
    const int lane = tid & 63;
    int who = 0;
#pragma unroll
    for (int d = 32, h = R / 2; d > 0; d >>= 1, h >>= 1) {
        if (h > 0) {
            const bool up = (lane & d) != 0;
#pragma unroll
            for (int u = 0; u < h; ++u) {
                const double2 give = up ? acc[u] : acc[u + h], keep = up ? acc[u + h] : acc[u];
                acc[u] = cmk(keep.x + __shfl_xor(give.x, d), keep.y + __shfl_xor(give.y, d));
            }
            who += up ? h : 0;
        } else {
            acc[0] = cmk(acc[0].x + __shfl_xor(acc[0].x, d), acc[0].y + __shfl_xor(acc[0].y, d));
        }
    }
    if ((lane & (64 / R - 1)) == 0) red[(tid >> 6) * R + who] = acc[0];
    __syncthreads();
    const int64_t q = (int64_t)grp * R + tid;
    if (tid < R && q < nq)
        part[pc * nq + q] = cadd(cadd(red[tid], red[R + tid]), cadd(red[2 * R + tid], red[3 * R + tid]));
}

// one wavefront per point: the pieces' sums and the incident field
__global__ void __launch_bounds__(256) k_field_sum(int64_t nq, int npiece, const double *pts, double k, double sx,
                                                   double sy, double sz, double2 amp, const double2 *part,
                                                   double2 *out) {
    const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (q >= nq) return;
    double2 a = cmk(0, 0);
    for (int g = lane; g <= npiece; g += 64) a = cadd(a, part[g * nq + q]);  // the last: the near pairs
    for (int d = 32; d > 0; d >>= 1) a = cmk(a.x + __shfl_xor(a.x, d), a.y + __shfl_xor(a.y, d));
    if (lane == 0) {
        const double dx = pts[3 * q] - sx, dy = pts[3 * q + 1] - sy, dz = pts[3 * q + 2] - sz;
        const double r = sqrt(dx * dx + dy * dy + dz * dz), inv4pi = 1.0 / (4.0 * FMM_PI);
        double s, co;
        sincos(k * r, &s, &co);
        out[q] = cadd(a, cmul(amp, cmk(co / r * inv4pi, s / r * inv4pi)));
    }
}

// ------------------------------------------------------------------ indirect formulation (Eq. ibem5)
// Unknowns x = (psi-, psi+), N each in caller order.  Both block rows need the same layer
// densities s = -i k (beta- psi- + beta+ psi+) (single layer) and m = psi- - psi+ (double layer):
//   row 1 = (psi- + psi+)/2 + L[s] + M[m],   row 2 = i k (beta- psi- - beta+ psi+)/2 + L'[s] + M'[m],
// so one FMM pass evaluates the potential and its normal derivative at every collocation point.

// g- = -dpsi_in/dn + i k beta- psi_in, g+ = dpsi_in/dn + i k beta+ psi_in (tree order)
__global__ void k_gamma_pm(int64_t n, const double4 *ec, const double4 *en, const double2 *bm, const double2 *bp,
                           double k, double sx, double sy, double sz, double2 amp, double2 *gm, double2 *gp) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double4 c = ec[i], nv = en[i];
    double dx = c.x - sx, dy = c.y - sy, dz = c.z - sz;
    double r = sqrt(dx * dx + dy * dy + dz * dz);
    double s, co;
    sincos(k * r, &s, &co);
    double2 G = cmul(amp, cmk(co / (4 * FMM_PI * r), s / (4 * FMM_PI * r)));
    double proj = (dx * nv.x + dy * nv.y + dz * nv.z) / (r * r);
    double2 dG = cscale(cmul(G, cmk(-1.0, k * r)), proj);  // dpsi_in/dn
    gm[i] = csub(cmul(cmk(-k * bm[i].y, k * bm[i].x), G), dG);
    gp[i] = cadd(cmul(cmk(-k * bp[i].y, k * bp[i].x), G), dG);
}

__global__ void k_densities_ind(int64_t n, const int32_t *perm, const double2 *x, const double2 *bm,
                                const double2 *bp, double k, double2 *sigma, double2 *mu) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    const double2 pm = x[u], pp = x[n + u];
    const double2 t = cadd(cmul(bm[i], pm), cmul(bp[i], pp));
    sigma[i] = cmk(k * t.y, -k * t.x);  // -i k (beta- psi- + beta+ psi+)
    mu[i] = csub(pm, pp);
}

// densities of the receiver formula (Eq. ibem1, ibem4): sigma = g- + g+ + i k (beta- psi- +
// beta+ psi+), mu = psi+ - psi-
__global__ void k_field_dens_ind(int64_t n, const int32_t *perm, const double2 *x, const double2 *gm,
                                 const double2 *gp, const double2 *bm, const double2 *bp, double k, double2 *sigma,
                                 double2 *mu) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    const double2 pm = x[u], pp = x[n + u];
    const double2 t = cadd(cmul(bm[i], pm), cmul(bp[i], pp));
    sigma[i] = cadd(cadd(gm[i], gp[i]), cmk(-k * t.y, k * t.x));
    mu[i] = csub(pp, pm);
}

// Densities of the receiver formula from the surface unknown x (caller order), in tree order, with
// the incident field of a monopole of amplitude amp at s evaluated at each centroid (Eq. sp6-sp7):
//   form 0, unknown psi_sc (Eq. dbem4 and the combined form): sigma = gamma + i k beta x,
//           mu = -x (Eq. dbem1), gamma = -dpsi_in/dn + i k beta psi_in;
//   form 1, unknown v = dpsi_sc/dn (Eq. dbem5): sigma = v, mu = -psi_sc = -(v - gamma)/(i k beta);
//   form 3, unknowns (psi-, psi+) (Eq. ibem5): sigma = g- + g+ + i k (beta- psi- + beta+ psi+),
//           mu = psi+ - psi- (Eq. ibem1, ibem4), g-+ = -+ dpsi_in/dn + i k beta-+ psi_in.
__global__ void k_field_dens(int64_t n, int form, const int32_t *perm, const double2 *x, const double4 *ec,
                             const double4 *en, const double2 *bm, const double2 *bp, double k, double sx, double sy,
                             double sz, double2 amp, double2 *sigma, double2 *mu) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double4 c = ec[i], nv = en[i];
    const double dx = c.x - sx, dy = c.y - sy, dz = c.z - sz;
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    double s, co;
    sincos(k * r, &s, &co);
    const double2 G = cmul(amp, cmk(co / (4 * FMM_PI * r), s / (4 * FMM_PI * r)));
    const double proj = (dx * nv.x + dy * nv.y + dz * nv.z) / (r * r);
    const double2 dG = cscale(cmul(G, cmk(-1.0, k * r)), proj);  // dpsi_in/dn
    const int64_t u = perm[i];
    const double2 ikbm = cmk(-k * bm[i].y, k * bm[i].x);
    const double2 gm = csub(cmul(ikbm, G), dG);
    if (form == 3) {
        const double2 ikbp = cmk(-k * bp[i].y, k * bp[i].x);
        const double2 gp = cadd(cmul(ikbp, G), dG);
        const double2 pm = x[u], pp = x[n + u];
        sigma[i] = cadd(cadd(gm, gp), cadd(cmul(ikbm, pm), cmul(ikbp, pp)));
        mu[i] = csub(pp, pm);
    } else if (form == 1) {
        const double2 v = x[u];
        sigma[i] = v;
        mu[i] = cscale(cdiv(csub(v, gm), ikbm), -1.0);
    } else {
        const double2 xi = x[u];
        sigma[i] = cadd(gm, cmul(ikbm, xi));
        mu[i] = cscale(xi, -1.0);
    }
}

// row 2 of the right-hand side gets (g+ - g-)/2
__global__ void k_rhs_ind_local(int64_t n, const int32_t *perm, const double2 *gm, const double2 *gp, double2 *b) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    b[n + u] = cadd(b[n + u], cscale(csub(gp[i], gm[i]), 0.5));
}

// Eq. (dbem5), unknown v = dpsi_sc/dn (caller order): densities sigma = -i k v, mu = zeta v with
// zeta = 1/beta (tree order); the product is v/2 + beta (L[sigma] + M[mu]).
__global__ void k_densities_dpsi(int64_t n, const int32_t *perm, const double2 *v, const double2 *beta, double k,
                                 double2 *sigma, double2 *mu) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 vi = v[perm[i]];
    sigma[i] = cmk(k * vi.y, -k * vi.x);  // -i k v
    mu[i] = cdiv(vi, beta[i]);
}
// y = half h + beta P (h, P, y caller order; beta tree order): the product (h = v) and the
// right-hand side (h = gamma in caller order)
__global__ void k_dpsi_combine(int64_t n, const int32_t *perm, const double2 *h, const double2 *beta, const double2 *P,
                               double2 *y) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    y[u] = cadd(cscale(h[u], 0.5), cmul(beta[i], P[u]));
}
// right-hand side densities of Eq. (dbem5): gamma (in sigma, tree order) -> gamma in caller order,
// mu = zeta gamma, sigma = 0
__global__ void k_rhs_dpsi_dens(int64_t n, const int32_t *perm, const double2 *beta, double2 *sigma, double2 *mu,
                                double2 *gam_caller) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double2 g = sigma[i];
    gam_caller[perm[i]] = g;
    mu[i] = cdiv(g, beta[i]);
    sigma[i] = cmk(0, 0);
}
// z = v * beta (inv = 0) or v / beta (inv = 1), caller order
__global__ void k_scale_beta(int64_t n, const int32_t *perm, const double2 *beta, int inv, const double2 *v,
                             double2 *z) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    z[u] = inv ? cdiv(v[u], beta[i]) : cmul(v[u], beta[i]);
}

// Combined (Burton-Miller) direct equation: Eq. (dbem3) plus alpha times its normal derivative
// (Section 3.2 jump relations; v = dpsi/dn = gamma + i k beta psi).  From the potential P and the
// normal derivative Q of the layers sigma = -i k beta x, mu = x (caller order, pq[0..n) and
// pq[n..2n)):  y = x/2 + (alpha i k / 2) beta x + P + alpha Q.
__global__ void k_bm_combine(int64_t n, const int32_t *perm, const double2 *x, const double2 *beta, double k,
                             double2 alpha, const double2 *pq, double2 *y) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    const double2 xu = x[u];
    const double2 half_aikb = cscale(cmul(alpha, cmuli(beta[i])), 0.5 * k);  // alpha i k beta / 2
    double2 v = cadd(cscale(xu, 0.5), cmul(half_aikb, xu));
    v = cadd(v, pq[u]);
    y[u] = cadd(v, cmul(alpha, pq[n + u]));
}

// Right-hand side of the combined equation: b = P + alpha (Q - gamma / 2), (P, Q) of the layer
// sigma = gamma (gamma in tree order).
__global__ void k_bm_rhs(int64_t n, const int32_t *perm, const double2 *gam, double2 alpha, const double2 *pq,
                         double2 *b) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    b[u] = cadd(pq[u], cmul(alpha, csub(pq[n + u], cscale(gam[i], 0.5))));
}

// derivative local expansions of a leaf (degree p + 1) from its local expansion D (degree p):
//   d_z R_n^m = k (a_{n-1}^m R_{n-1}^m - a_n^m R_{n+1}^m), etc. (the P2M recurrences), collected
//   per output coefficient (n, m)
template <class T>
__device__ inline double2 dget_nm(const T *D, int p, int n, int m) {
    if (n < 0 || n >= p || (m < 0 ? -m : m) > n) return cmk(0, 0);
    const T d = D[cidx(n, m)];
    return cmk(d.x, d.y);
}
// E: per leaf D itself (its degree p zero), then the z, + and - derivatives, (p + 1)^2 entries each
template <class T>
__global__ void k_local_derivs(int64_t nleaf, int p, const T *D, double k, double2 *E) {
    const int64_t b = blockIdx.x;
    const int q1 = (p + 1) * (p + 1);
    const T *Db = D + b * p * p;
    E += b * 4 * q1;
    for (int c = threadIdx.x; c < q1; c += blockDim.x) {
        int n = (int)sqrt((double)c);
        while (n * n > c) --n;
        while ((n + 1) * (n + 1) <= c) ++n;
        const int m = c - n * n - n;
        const double2 z = csub(cscale(dget_nm(Db, p, n + 1, m), coef_a(n, m)), cscale(dget_nm(Db, p, n - 1, m), coef_a(n - 1, m)));
        const double2 pl = csub(cscale(dget_nm(Db, p, n - 1, m - 1), coef_b(n, -m)),
                                cscale(dget_nm(Db, p, n + 1, m - 1), coef_b(n + 1, m - 1)));
        const double2 mi = csub(cscale(dget_nm(Db, p, n - 1, m + 1), coef_b(n, m)),
                                cscale(dget_nm(Db, p, n + 1, m + 1), coef_b(n + 1, -m - 1)));
        E[c] = dget_nm(Db, p, n, m);
        E[q1 + c] = cscale(z, k);
        E[2 * q1 + c] = cscale(pl, k);
        E[3 * q1 + c] = cscale(mi, k);
    }
}

// potential and normal derivative at the targets from the expansions E of k_local_derivs (degree
// p + 1), plus the near part and the local terms of both block rows; the split of k_l2p
template <bool STAGE>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
k_l2p_n(int p, int cs, const int32_t *leaf_start, const double4 *center,
                                              const double4 *ec, const double4 *en, const double2 *E, double k,
                                              double ik, const double *leg, const double *ser, const double2 *ynear,
                                              const double2 *ynearn, int nsplit, const int32_t *perm, int64_t n,
                                              const double2 *x, const double2 *bm, const double2 *bp, double2 *y,
                                              int has_far) {
    extern __shared__ char l2p_sm[];
    const int b = blockIdx.x, ts = leaf_start[b], te = leaf_start[b + 1], q1 = (p + 1) * (p + 1);
    auto fin = [&](int t, const double2 *f) {  // f: potential, d_z, d_x + i d_y, d_x - i d_y
        const double4 nt = en[t];
        // n.grad = n_z d_z + (n_x - i n_y)/2 (d_x + i d_y) + (n_x + i n_y)/2 (d_x - i d_y)
        double2 farn = cscale(f[1], nt.z);
        farn = cadd(farn, cmul(cmk(0.5 * nt.x, -0.5 * nt.y), f[2]));
        farn = cadd(farn, cmul(cmk(0.5 * nt.x, 0.5 * nt.y), f[3]));
        const int64_t u = perm[t];
        double2 v1 = cadd(near_sum(ynear, t, n, nsplit), f[0]), v2 = cadd(near_sum(ynearn, t, n, nsplit), farn);
        if (x) {
            const double2 pm = x[u], pp = x[n + u];
            v1 = cadd(v1, cscale(cadd(pm, pp), 0.5));
            // i k (beta- psi- - beta+ psi+) / 2
            const double2 t2 = csub(cmul(bm[t], pm), cmul(bp[t], pp));
            v2 = cadd(v2, cmk(-0.5 * k * t2.y, 0.5 * k * t2.x));
        }
        y[u] = v1;
        y[n + u] = v2;
    };
    if (has_far) {
        l2p_leaf<4, STAGE>(p + 1, cs, ts, te, center[b], ec, E + (int64_t)b * 4 * q1, k, ik, leg, ser, l2p_sm, fin);
    } else {
        const double2 f[4] = {cmk(0, 0), cmk(0, 0), cmk(0, 0), cmk(0, 0)};
        for (int t = ts + threadIdx.x + 64 * blockIdx.y; t < te; t += 64 * gridDim.y) fin(t, f);
    }
}

// 2x2 diagonal blocks of the indirect operator (local terms and self entries) and their inverses:
//   [ 1/2 - i k beta- L_ii          1/2 - i k beta+ L_ii  ]
//   [ i k beta-/2 + M'_ii          -i k beta+/2 - M'_ii   ]      (M_ii = L'_ii = 0)
__global__ void k_diag2_inv(int64_t n, const int32_t *near_start, const int32_t *near_col, const double2 *nL,
                            const double2 *nMp, const double2 *bm, const double2 *bp, double k, double shift,
                            double2 *inv) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2 L = cmk(0, 0), Mp = cmk(0, 0);
    for (int e = near_start[i]; e < near_start[i + 1]; ++e)
        if (near_col[e] == i) {
            L = nL[e];
            Mp = nMp[e];
        }
    const double2 ik = cmk(0, k);
    const double2 a = cadd(cmk(0.5 + shift, 0), cscale(cmul(cmul(ik, bm[i]), L), -1.0));
    const double2 b = csub(cmk(0.5, 0), cmul(cmul(ik, bp[i]), L));
    const double2 c = cadd(cscale(cmul(ik, bm[i]), 0.5), Mp);
    const double2 d = csub(cadd(cscale(cmul(ik, bp[i]), -0.5), cmk(shift, 0)), Mp);
    const double2 det = csub(cmul(a, d), cmul(b, c));
    inv[4 * i] = cdiv(d, det);
    inv[4 * i + 1] = cdiv(cscale(b, -1.0), det);
    inv[4 * i + 2] = cdiv(cscale(c, -1.0), det);
    inv[4 * i + 3] = cdiv(a, det);
}

// z = blockdiag(inv) v on (psi-, psi+) pairs (caller order; inv in tree order)
__global__ void k_mul_diag2(int64_t n, const int32_t *perm, const double2 *inv, const double2 *v, double2 *z) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t u = perm[i];
    const double2 a = v[u], b = v[n + u];
    z[u] = cadd(cmul(inv[4 * i], a), cmul(inv[4 * i + 1], b));
    z[n + u] = cadd(cmul(inv[4 * i + 2], a), cmul(inv[4 * i + 3], b));
}

// ------------------------------------------------------------------ launchers (RHS count 1, 2, 4)
#define FMM_NR_DISPATCH(nr, CALL)                                             \
    switch (nr) {                                                             \
    case 1: CALL(1); break;                                                   \
    case 2: CALL(2); break;                                                   \
    case 4: CALL(4); break;                                                   \
    default: throw FmmError(-1, "right-hand-side chunk must be 1, 2 or 4");  \
    }

// e^{ikr} by table steps: k 128 / (2 pi) as a sum of two doubles
static double2 eikr_scale(double k) {
    const long double v = (long double)k * (EIKR_N / (2.0L * 3.14159265358979323846264338327950288L));
    const double hi = (double)v;
    return make_double2(hi, (double)(v - (long double)hi));
}

// pieces of every leaf's source list in the near field: enough workgroups for every CU to hold
// its eight (2,048), at most 16 sums for L2P to add.  56 leaves (2,664 elements): 29.6 us whole,
// 13.6 us in 16 pieces, 16.8 us in 32; the 2,700 leaves of 90,972 elements gain nothing from pieces.
int p2p_splits_of(int nleaf) { return std::max(1, std::min(16, ceil_div(2048, std::max(1, nleaf)))); }

void launch_p2p(int nr, int nleaf, int nsplit, const int32_t *leaf_start, const int32_t *nbr_start,
                const int32_t *nbr_list, int all_leaves, const double4 *ec, const double4 *en, const double2 *sigma,
                const double2 *mu, double k, double rc2, const int32_t *near_start, const int32_t *near_col,
                const double2 *nL, const double2 *nM, double2 *y, hipStream_t st) {
#define P2P_CALL(R)                                                                                               \
    k_p2p<R, false><<<nleaf * nsplit, P2P_WG, 0, st>>>(nleaf, leaf_start, nbr_start, nbr_list, all_leaves, nsplit, ec, \
                                                       en, sigma, mu, k, eikr_scale(k), rc2, near_start, near_col, nL, \
                                                       nM, nullptr, nullptr, y, nullptr)
    FMM_NR_DISPATCH(nr, P2P_CALL)
#undef P2P_CALL
    LAUNCH_OK();
}

// potential y and normal derivative yn of one vector
void launch_p2p_n(int nleaf, int nsplit, const int32_t *leaf_start, const int32_t *nbr_start, const int32_t *nbr_list,
                  int all_leaves, const double4 *ec, const double4 *en, const double2 *sigma, const double2 *mu,
                  double k, double rc2, const int32_t *near_start, const int32_t *near_col, const double2 *nL,
                  const double2 *nM, const double2 *nLp, const double2 *nMp, double2 *y, double2 *yn, hipStream_t st) {
    k_p2p<1, true><<<nleaf * nsplit, P2P_WG, 0, st>>>(nleaf, leaf_start, nbr_start, nbr_list, all_leaves, nsplit, ec,
                                                      en, sigma, mu, k, eikr_scale(k), rc2, near_start, near_col, nL,
                                                      nM, nLp, nMp, y, yn);
    LAUNCH_OK();
}

// Points per workgroup and pieces of the elements for nq points: enough pieces for FIELD_WGS
// workgroups, none below 256 elements, and no more partial sums than FIELD_PART (the near pairs'
// among them).
static void field_shape(int64_t nt, int64_t nq, int &R, int64_t &piece, int &npiece) {
    R = nq >= 5 ? 8 : nq >= 3 ? 4 : (int)nq;
    const int64_t groups = (nq + R - 1) / R;
    int64_t np = std::min<int64_t>((nt + 255) / 256, (FIELD_WGS + groups - 1) / groups);
    np = std::max<int64_t>(1, std::min(np, FIELD_PART / nq - 1));
    piece = (((nt + np - 1) / np + 255) / 256) * 256;
    npiece = (int)((nt + piece - 1) / piece);
}

// part: FIELD_PART partial sums
void launch_field(int64_t nt, int64_t nr, const FieldTree &tree, const double *pts, const double4 *ec,
                  const double4 *en, const double *ev, const double2 *sigma, const double2 *mu, double k, double rc2,
                  const double *rs, double2 amp, double2 *part, double2 *out, hipStream_t st) {
    for (int64_t q0 = 0; q0 < nr; q0 += FIELD_PART / 2) {
        const int64_t nq = std::min<int64_t>(nr - q0, FIELD_PART / 2);
        int R, np;
        int64_t piece;
        field_shape(nt, nq, R, piece, np);
        const unsigned ng = (unsigned)ceil_div(nq, R);
#define FIELD_CALL(RR)                                                                                                \
    k_field<RR><<<ceil_div(nq, 4) + ng * np, 256, 0, st>>>(nt, nq, piece, np, ng, tree, pts + 3 * q0, ec, en, ev, sigma, \
                                                           mu, k, eikr_scale(k), rc2, part)
        switch (R) {
        case 1: FIELD_CALL(1); break;
        case 2: FIELD_CALL(2); break;
        case 4: FIELD_CALL(4); break;
        default: FIELD_CALL(8);
        }
#undef FIELD_CALL
        LAUNCH_OK();
        k_field_sum<<<ceil_div(nq, 4), 256, 0, st>>>(nq, np, pts + 3 * q0, k, rs[0], rs[1], rs[2], amp, part, out + q0);
        LAUNCH_OK();
    }
}

size_t p2m_stage_bytes(int nr, int p) {
    const int TB = (p + 1) * (p + 2) / 2;
    return (size_t)(TB + 1) * 16 + (size_t)nr * 96 + (size_t)(p + 2) * 8 + 56;  // per staged source
}
size_t p2m_fixed_bytes(int p) { return (size_t)3 * (p + 1) * (p + 2) / 2 * sizeof(double); }

static bool p2m_slot_ok(int p) { return (p + 1) * (p + 2) / 2 <= P2M_SLOTS; }
// the largest group of sources with four (one vector) or three workgroups per CU (the registers
// allow no more: three instead of four costs one vector 625 -> 694 us, four instead of three costs
// four vectors 990 -> 1,414 us); with two leaves per CU or fewer up to 64 KB (56 leaves: 27 -> 23 us, and
// no less with every source of a leaf in one group)
static int p2m_group(int nr, int p, int nleaf, size_t &sh) {
    int G = 64;
    const size_t room = nleaf <= 512 ? 65536 : 163840 / (nr > 1 ? 3 : 4);
    while (G > 4 && P2mLayout(p, G, nr).total * sizeof(double) > room) --G;
    sh = P2mLayout(p, G, nr).total * sizeof(double);
    return G;
}
bool p2m_writes_fp32(int p) { return p2m_slot_ok(p); }
void build_p2m_table(double *tab, hipStream_t st) {
    k_p2m_table<<<ceil_div(P2M_CAP, 64), 64, 0, st>>>(tab);
    LAUNCH_OK();
}

bool p2m_fits(int nr, int p) {
    if (p2m_slot_ok(p)) {
        size_t sh;
        p2m_group(nr, p, 1, sh);
        return sh <= 65536;
    }
    return p2m_stage_bytes(nr, p) + p2m_fixed_bytes(p) <= 60000;
}

// Mout: the multipoles; M32 instead (FP32, Mout unused) where p2m_writes_fp32(p)
void launch_p2m(int nr, int nleaf, int p, const int32_t *leaf_start, const double4 *center, const double4 *ec,
                const double4 *en, const double2 *sigma, const double2 *mu, double k, const double *leg,
                const double *tab, double2 *Mout, float2 *M32, hipStream_t st) {
    if (nleaf <= 0) return;
    if (p2m_slot_ok(p)) {
        size_t sh;
        const int G = p2m_group(nr, p, nleaf, sh);
        const int nbw = (P2mLayout(p, G, nr).TBP / 8 + 3) / 4;  // 16-row blocks per wavefront
#define P2M_CALL2(R, B)                                                                                               \
    if (M32) k_p2m<R, B, float2><<<nleaf, 256, sh, st>>>(p, G, leaf_start, center, ec, en, sigma, mu, k, 1.0 / k, leg, \
                                                         tab, M32);                                                   \
    else k_p2m<R, B, double2><<<nleaf, 256, sh, st>>>(p, G, leaf_start, center, ec, en, sigma, mu, k, 1.0 / k, leg,    \
                                                      tab, Mout)
#define P2M_CALL(R)                 \
    if (nbw <= 5) { P2M_CALL2(R, 5); } \
    else { P2M_CALL2(R, 8); }
        FMM_NR_DISPATCH(nr, P2M_CALL)
#undef P2M_CALL
#undef P2M_CALL2
    } else {
        const size_t per = p2m_stage_bytes(nr, p), fixed = p2m_fixed_bytes(p);
        const int CH = (int)std::max<size_t>(1, std::min<size_t>(32, (60000 - fixed) / per));
        const size_t sh = (size_t)CH * per + fixed;
#define P2M_CALL(R) \
    k_p2m_wide<R><<<nleaf, 256, sh, st>>>(nleaf, p, CH, leaf_start, center, ec, en, sigma, mu, k, leg, Mout)
        FMM_NR_DISPATCH(nr, P2M_CALL)
#undef P2M_CALL
    }
    LAUNCH_OK();
}

// targets of a chunk and workgroups of a leaf: with fewer leaves than L2P_FEW (two per CU) there is room
// for four workgroups per leaf, of 16 targets at a time
static dim3 l2p_grid(int nv, int nleaf, int &cs) {
    const bool few = nleaf < L2P_FEW;
    cs = few ? 16 : 16 * l2p_tlm(nv);
    return dim3(nleaf, few ? 4 : 1);
}
constexpr size_t L2P_STAGE = 48 * 1024;  // LDS up to which the expansions are staged

// Lc: the local expansions; L32 instead where the translations ran in FP32; tab: build_p2m_table's
void launch_l2p(int nr, int nleaf, int p, const int32_t *leaf_start, const double4 *center, const double4 *ec,
                const double2 *Lc, const float2 *L32, double k, const double *leg, const double *tab,
                const double2 *ynear, int nsplit, double half, const int32_t *perm, int64_t n, const double2 *x,
                double2 *y, int has_far, hipStream_t st) {
    if (nleaf <= 0) return;
    int cs;
    const dim3 grid = l2p_grid(nr, nleaf, cs);
    const size_t dbytes = (size_t)nr * p * p * (L32 ? sizeof(float2) : sizeof(double2));
    const bool stage = L2pLayout(p, cs, dbytes).total <= (int)L2P_STAGE;
    const size_t sh = L2pLayout(p, cs, stage ? dbytes : 0).total;
#define L2P_CALL2(R, T, D)                                                                                              \
    if (stage) k_l2p<R, true, T><<<grid, 64, sh, st>>>(p, cs, leaf_start, center, ec, D, k, 1.0 / k, leg, tab + P2M_OSER, \
                                                       ynear, nsplit, half, perm, n, x, y, has_far);                    \
    else k_l2p<R, false, T><<<grid, 64, sh, st>>>(p, cs, leaf_start, center, ec, D, k, 1.0 / k, leg, tab + P2M_OSER,     \
                                                  ynear, nsplit, half, perm, n, x, y, has_far)
#define L2P_CALL(R)                               \
    if (L32) { L2P_CALL2(R, float2, L32); }       \
    else { L2P_CALL2(R, double2, Lc); }
    FMM_NR_DISPATCH(nr, L2P_CALL)
#undef L2P_CALL
#undef L2P_CALL2
    LAUNCH_OK();
}

// potential and normal derivative of local expansions; E: 4 (p + 1)^2 entries per leaf of scratch
void launch_l2p_n(int nleaf, int p, const int32_t *leaf_start, const double4 *center, const double4 *ec,
                  const double4 *en, const double2 *Lc, const float2 *L32, double2 *E, double k, const double *leg,
                  const double *tab, const double2 *ynear, const double2 *ynearn, int nsplit, const int32_t *perm,
                  int64_t n, const double2 *x, const double2 *bm, const double2 *bp, double2 *y, int has_far,
                  hipStream_t st) {
    if (nleaf <= 0) return;
    if (has_far) {
        if (L32) k_local_derivs<<<nleaf, 256, 0, st>>>(nleaf, p, L32, k, E);
        else k_local_derivs<<<nleaf, 256, 0, st>>>(nleaf, p, Lc, k, E);
        LAUNCH_OK();
    }
    int cs;
    const dim3 grid = l2p_grid(4, nleaf, cs);
    const size_t dbytes = (size_t)4 * (p + 1) * (p + 1) * sizeof(double2);
    const bool stage = L2pLayout(p + 1, cs, dbytes).total <= (int)L2P_STAGE;
    const size_t sh = L2pLayout(p + 1, cs, stage ? dbytes : 0).total;
#define L2P_CALL(S)                                                                                                    \
    k_l2p_n<S><<<grid, 64, sh, st>>>(p, cs, leaf_start, center, ec, en, E, k, 1.0 / k, leg, tab + P2M_OSER, ynear, ynearn, \
                                     nsplit, perm, n, x, bm, bp, y, has_far)
    if (stage) L2P_CALL(true);
    else L2P_CALL(false);
#undef L2P_CALL
    LAUNCH_OK();
}

}  // namespace fmm

// Device building blocks shared by the HIP kernels: the Philox4x32-10 draw
// keyed by (packet, event, block), phase functions and their samplers
// (Sect. 3), direction rotation, the spherical / slab cell traversal
// (Sect. 2) and the opacity-table interpolation (Sect. 7).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "mcrt_internal.hpp"

namespace mcrt {
namespace dev {

constexpr double kPi = 3.14159265358979323846;
constexpr double kH = 6.62607015e-27;
constexpr double kC = 2.99792458e10;
constexpr double kKB = 1.380649e-16;

// ---------------------------------------------------------------- RNG
// Philox4x32-10 (Salmon et al. 2011): counter (packet lo, packet hi, event,
// block), key (seed lo, seed hi ^ tag).
struct U2 {
    double a, b;
};

__device__ __forceinline__ U2 draw(uint64_t seed, uint32_t tag, uint64_t packet, uint32_t event,
                                   uint32_t block)
{
    uint32_t c0 = (uint32_t)packet, c1 = (uint32_t)(packet >> 32), c2 = event, c3 = block;
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32) ^ tag;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
        uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
        uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    U2 u;
    uint64_t ma = ((uint64_t)c0 << 20) | (uint64_t)(c1 >> 12);
    uint64_t mb = ((uint64_t)c2 << 20) | (uint64_t)(c3 >> 12);
    u.a = ((double)ma + 0.5) * (1.0 / 4503599627370496.0);
    u.b = ((double)mb + 0.5) * (1.0 / 4503599627370496.0);
    return u;
}

// ---------------------------------------------------------------- phase functions
__device__ __forceinline__ double p_rayleigh(double mu) { return 0.75 * (1.0 + mu * mu); }

__device__ __forceinline__ double p_hg(double mu, double g)
{
    if (fabs(g) < 1e-6) return 1.0;
    double den = 1.0 + g * g - 2.0 * g * mu;
    return (1.0 - g * g) / (den * sqrt(den));
}

// Rayleigh: Cardano root of mu^3 + 3 mu = 2 (4 zeta - 2), the inverse of the
// CDF (mu^3 + 3 mu + 4)/8 of the normalised phase function.
__device__ __forceinline__ double sample_rayleigh(double z)
{
    double q = 4.0 * z - 2.0;
    double u = cbrt(q + sqrt(q * q + 1.0));
    double mu = u - 1.0 / u;
    return fmin(fmax(mu, -1.0), 1.0);
}

__device__ __forceinline__ double sample_hg(double z, double g)
{
    double mu;
    if (fabs(g) < 1e-6) {
        mu = 2.0 * z - 1.0;
    } else {
        double t = (1.0 - g * g) / (1.0 - g + 2.0 * g * z);
        mu = (1.0 + g * g - t * t) / (2.0 * g);
    }
    return fmin(fmax(mu, -1.0), 1.0);
}

__device__ __forceinline__ void rotate_dir(double& dx, double& dy, double& dz, double mu, double psi)
{
    double st = sqrt(fmax(1.0 - mu * mu, 0.0));
    double cp = cos(psi), sp = sin(psi);
    double nx, ny, nz;
    if (fabs(dz) < 0.99999) {
        double t = sqrt(1.0 - dz * dz);
        nx = st * (dx * dz * cp - dy * sp) / t + dx * mu;
        ny = st * (dy * dz * cp + dx * sp) / t + dy * mu;
        nz = -st * cp * t + dz * mu;
    } else {
        double sgn = dz >= 0.0 ? 1.0 : -1.0;
        nx = st * cp;
        ny = st * sp;
        nz = sgn * mu;
    }
    double n = sqrt(nx * nx + ny * ny + nz * nz);
    dx = nx / n;
    dy = ny / n;
    dz = nz / n;
}

// ------------------------------------------------------ Draine phase function
// Draine's hybrid HG-Rayleigh function (Sect. 3, aerosol scattering) is
// P_HG(G) (1 + alpha mu^2) / (1 + alpha (1 + 2 G^2)/3); its mean cosine
// G (1 + alpha (3 + 2 G^2)/5) / (1 + alpha (1 + 2 G^2)/3) rises from -1 to 1
// on [-1, 1], so the G of a cloud with asymmetry factor g is found by
// bisection to the last bit (alpha = 0: HG, G = g).
__host__ __device__ inline double draine_G(double g, double alpha)
{
    if (alpha == 0.0) return g;
    double lo = -1.0, hi = 1.0;
    for (int it = 0; it < 200; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid == lo || mid == hi) break;
        const double m = mid * (1.0 + alpha * (3.0 + 2.0 * mid * mid) / 5.0) /
                         (1.0 + alpha * (1.0 + 2.0 * mid * mid) / 3.0);
        if (m < g) lo = mid;
        else hi = mid;
    }
    return 0.5 * (lo + hi);
}

// ------------------------------------------------------ forced interaction
// Optical depth of a forced flight over a path of depth tp (0 < tp < inf)
// from zeta, and the weight factor e^{-tau}/q(tau) of its density q on
// [0, tp]: kind 1 forced scattering q = e^{-tau}/(1 - e^{-tp}); kind 2
// path-length stretching q = l e^{-l tau}/(1 - e^{-l tp}), l = 1/(1 + tp);
// kind 3 their equal mixture, the component picked by zc < 1/2.
__host__ __device__ inline double forced_tau(int kind, double tp, double zeta, double zc, double& wf)
{
    const double pf = -expm1(-tp);
    const double l = 1.0 / (1.0 + tp);
    const double pl = -expm1(-l * tp);
    const bool stretch = kind == 2 || (kind == 3 && !(zc < 0.5));
    const double tau = stretch ? -log1p(-zeta * pl) / l : -log1p(-zeta * pf);
    if (kind == 1) {
        wf = pf;
    } else if (kind == 2) {
        wf = exp(-tau) * pl / (l * exp(-l * tau));
    } else {
        const double q = 0.5 * exp(-tau) / pf + 0.5 * l * exp(-l * tau) / pl;
        wf = exp(-tau) / q;
    }
    return tau;
}

// ------------------------------------------------- stellar limb darkening
// I(mu)/I(1) of the stellar disk at zenith cosine mu (Sect. 5.1.1): laws
// 0 none, 1 linear, 2 quadratic, 3 square-root, 4 logarithmic,
// 5 exponential, 6 power-2; and the weight of the stellar light behind the
// sky-plane point (y, z) of the planet's frame, which lies at (ty + y,
// tz + z) on the stellar disk (zero off the disk).
__host__ __device__ inline double limb_law(int law, double c1, double c2, double mu)
{
    const double x = 1.0 - mu;
    if (law == 1) return 1.0 - c1 * x;
    if (law == 2) return 1.0 - c1 * x - c2 * x * x;
    if (law == 3) return 1.0 - c1 * x - c2 * (1.0 - sqrt(mu));
    if (law == 4) return 1.0 - c1 * x - c2 * (mu > 0.0 ? mu * log(mu) : 0.0);
    if (law == 5) return 1.0 - c1 * x - c2 / (1.0 - exp(mu));
    if (law == 6) return 1.0 - c1 * (1.0 - pow(mu, c2));
    return 1.0;
}

__host__ __device__ inline double limb_weight(const LimbDark& ld, double y, double z)
{
    if (ld.law == 0) return 1.0;
    const double sy = ld.ty + y, sz = ld.tz + z;
    const double q = (sy * sy + sz * sz) / (ld.r_star * ld.r_star);
    return q < 1.0 ? limb_law(ld.law, ld.c1, ld.c2, sqrt(1.0 - q)) : 0.0;
}

// ---------------------------------------------------------------- geometry
__host__ __device__ __forceinline__ int find_edge(const double* e, int n, double x)
{
    // largest m in [0, n-1] with e[m] <= x, 0 if none (edges increasing)
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (e[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__host__ __device__ __forceinline__ void locate_column(const GridDev& g, double x, double y, double z, int& i, int& j)
{
    j = find_edge(g.lat, g.nlat, atan2(z, sqrt(x * x + y * y)));
    i = find_edge(g.lon, g.nlon, atan2(y, x));
}

// ---------------------------------------------------------------- opacity interpolation
struct Bracket {
    int i0, i1;
    double t;
};

__device__ __forceinline__ Bracket bracket(const double* gx, int n, double x)
{
    Bracket b;
    if (n == 1) {
        b.i0 = 0; b.i1 = 0; b.t = 0.0;
        return b;
    }
    if (x <= gx[0]) {
        b.i0 = 0; b.i1 = 1; b.t = 0.0;
        return b;
    }
    if (x >= gx[n - 1]) {
        b.i0 = n - 2; b.i1 = n - 1; b.t = 1.0;
        return b;
    }
    int m = find_edge(gx, n - 1, x);
    b.i0 = m;
    b.i1 = m + 1;
    b.t = (x - gx[m]) / (gx[m + 1] - gx[m]);
    return b;
}

// ln-kappa bilinear in (T, ln P); a -inf (zero kappa) corner with positive
// weight gives zero.  lnk(iT, iP) read through the accessor.
template <typename F>
__device__ __forceinline__ double interp_tp(F lnk, const Bracket& bt, const Bracket& bp)
{
    double t = bt.t, u = bp.t;
    double w0 = (1.0 - t) * (1.0 - u), w1 = (1.0 - t) * u, w2 = t * (1.0 - u), w3 = t * u;
    double acc = 0.0;
    if (w0 > 0.0) { double l = lnk(bt.i0, bp.i0); if (isinf(l)) return 0.0; acc = acc + w0 * l; }
    if (w1 > 0.0) { double l = lnk(bt.i0, bp.i1); if (isinf(l)) return 0.0; acc = acc + w1 * l; }
    if (w2 > 0.0) { double l = lnk(bt.i1, bp.i0); if (isinf(l)) return 0.0; acc = acc + w2 * l; }
    if (w3 > 0.0) { double l = lnk(bt.i1, bp.i1); if (isinf(l)) return 0.0; acc = acc + w3 * l; }
    return exp(acc);
}

// Doppler shift of cell c's table position for light along o (Sect. 7):
// ln(lambda_eff / lambda) by its velocity towards the observer, in table steps.
__device__ __forceinline__ double los_shift(const GridDev& g, int c, double ox, double oy, double oz, double dlnlam)
{
    int i = c % g.nlon, j = (c / g.nlon) % g.nlat, k = c / (g.nlon * g.nlat);
    double rc = 0.5 * (g.r[k] + g.r[k + 1]);
    double th = 0.5 * (g.lat[j] + g.lat[j + 1]);
    double ph = 0.5 * (g.lon[i] + g.lon[i + 1]);
    double sth = sin(th), cth = cos(th), sph = sin(ph), cph = cos(ph);
    double eE0 = -sph, eE1 = cph, eE2 = 0.0;
    double eN0 = -sth * cph, eN1 = -sth * sph, eN2 = cth;
    double eR0 = cth * cph, eR1 = cth * sph, eR2 = sth;
    double uu = g.u ? (double)g.u[c] : 0.0, vv = g.v ? (double)g.v[c] : 0.0, ww = g.w ? (double)g.w[c] : 0.0;
    double ue = uu + g.omega_rot * rc * cth;
    double v0 = ue * eE0 + vv * eN0 + ww * eR0;
    double v1 = ue * eE1 + vv * eN1 + ww * eR1;
    double v2 = ue * eE2 + vv * eN2 + ww * eR2;
    double vlos = -(v0 * ox + v1 * oy + v2 * oz);
    return log1p(-vlos / kC) / dlnlam;
}

// Arithmetic of a walk.  The exact form rounds every product and sum on its
// own and divides and takes roots correctly rounded, as the FP64 oracle; the
// fast form, taken by the FP32-mixed transport, contracts a product and a sum
// into one multiply-add.  A packet's path amplifies a last-bit difference of
// a crossing at every interaction in thick, patchy clouds, so each form's
// operations are part of what it computes and stay as they are.
template <bool FAST>
__host__ __device__ __forceinline__ double wk_mad(double a, double b, double c)
{
    if constexpr (FAST) return fma(a, b, c);
    else return a * b + c;
}

// a / b from the hardware reciprocal (good to about 5e-8 on gfx950): Newton
// steps and a residual correction.  One step (fast form) is within an ulp of
// the rounded quotient; two (exact form) are the steps by which the library's
// division rounds correctly, without its scaling of the ends of the exponent
// range, which the operands of a walk (lengths of ~1e9 cm, their squares and
// differences, direction cosines, extinctions) do not reach.  b = 0 gives a
// NaN, which callers discard.
template <bool FAST>
__host__ __device__ __forceinline__ double wk_div(double a, double b)
{
#if defined(__HIP_DEVICE_COMPILE__) || defined(MCRT_EMULATE_RCP)
    double r = __builtin_amdgcn_rcp(b);
    r = fma(r, fma(-b, r, 1.0), r);
    if constexpr (!FAST) r = fma(r, fma(-b, r, 1.0), r);
    const double qt = a * r;
    return fma(fma(-b, qt, a), r, qt);
#else
    return a / b;
#endif
}

// Square root of x (0 for x <= 0) from the hardware reciprocal square root
// y ~ 1/sqrt(x) by Goldschmidt's iteration (g = x y, h = y/2, r = 1/2 - h g,
// g <- g + g r, h <- h + h r) and corrections g <- g + (x - g^2) h: one within
// an ulp (fast form), two correctly rounded (exact form; as the library's
// root, again without its range scaling).
template <bool FAST>
__host__ __device__ __forceinline__ double wk_sqrt(double x)
{
#if defined(__HIP_DEVICE_COMPILE__) || defined(MCRT_EMULATE_RCP)
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    if constexpr (!FAST) g = fma(fma(-g, g, x), h, g);
    return x > 0.0 ? g : 0.0;
#else
    return x > 0.0 ? sqrt(x) : 0.0;
#endif
}

// min and max of two non-NaN doubles, one instruction (the library's forms
// first quiet their operands)
__host__ __device__ __forceinline__ double wk_min(double a, double b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
#else
    return a < b ? a : b;
#endif
}
__host__ __device__ __forceinline__ double wk_max(double a, double b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
#else
    return a > b ? a : b;
#endif
}

// ---------------------------------------------------------------- walker
// Straight-line walk through the cells from an origin p0 along unit d.  Every
// face surface is met at fixed ray parameters t, so positions are never
// advanced step by step (p(t) = p0 + t d: no drift).  Of each kind of face
// only the next one along the walk is kept, because a straight line meets
// them in a known order:
//   shells     inward while its nearest point to the centre is ahead and the
//              next inner sphere is met, then outward for good; the sphere
//              crossed last on the way in is the first one met on the way out
//              (its far root is kept);
//   planes     the longitude grows or shrinks all along a line (the sign of
//              px dy - py dx), so one edge per cell can be met;
//   cones      sin(lat) = z / r has one extremum along a line and tends to
//              dz.  With P the line's nearest point to the centre, q2 = |P|^2
//              and M = Pz^2 + q2 dz^2, the extremum is a maximum for Pz > 0
//              and its sin^2(lat) is M / q2.  While it is ahead and reaches
//              the edge in front (M >= s^2 q2, s the edge's sine), or with no
//              extremum ahead if dz lies beyond s, that edge is next;
//              otherwise, after the extremum, the edge behind if dz lies
//              beyond that.
// So a step is a minimum of three parameters, and a crossing recomputes the
// one it used: one square root and one division for whatever kinds of face
// the lanes of a wave cross.  Ties go to the shell, the cone, the plane.  A
// slab's walk has shells only.
//
// What it replaced kept both roots of both cones, both planes and both shells
// of the cell (nine parameters) and chose among them at every step.
struct Walker {
    double px, py, pz;  // origin
    double dx, dy, dz;  // unit direction
    double t;           // distance walked from the origin
    double B0, C0;      // p0 . d, |p0|^2 (spherical)
    double ts, tc, tp;  // next shell, cone and plane (INFINITY = none)
    double far;         // while inward: the far root of the sphere at ts
    int i, j, k;
    int dk, dj, di;     // +-1: ts is the outer or inner shell, tc the upper or lower cone, longitude grows or shrinks
    int eq;             // WE_ bits
};
enum {
    WE_ROW = 1,      // the walk just entered a row at GridDev::eq_edge: wk_row_roots sets tc
    WE_FROM_LO = 2,  // ... through the row's lower edge
    WE_FROM_HI = 4   // ... through its upper edge
};

// The geometry a walk is compiled for: spherical, slab, or the grid's own.
enum { GEO_SPHERE = 0, GEO_SLAB = 1, GEO_ANY = 2 };
template <int GEO>
__host__ __device__ __forceinline__ bool wk_slab(const GridDev& g)
{
    if constexpr (GEO == GEO_ANY) return g.geom == 1;
    else return GEO == GEO_SLAB;
}

// v, negated where the top bit of m is set (m = -1 or 1: a sign).
__host__ __device__ __forceinline__ double wk_flip(double v, int m)
{
    return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, v) ^ ((uint64_t)((uint32_t)m & 0x80000000u) << 32));
}

// The face table's entry e (a 32-bit offset from one uniform base).
__host__ __device__ __forceinline__ double2 wk_face(const GridDev& g, int e)
{
    return *(const double2*)((const char*)g.faces + (uint32_t)e * (uint32_t)sizeof(double2));
}

// The outer (out) or inner radius of layer k.
__host__ __device__ __forceinline__ double wk_edge(const GridDev& g, int k, bool out)
{
    return *(const double*)((const char*)g.faces + ((uint32_t)k * 16u + (out ? 8u : 0u)));
}

__host__ __device__ __forceinline__ int wk_cell(const GridDev& g, const Walker& w) { return (w.k * g.nlat + w.j) * g.nlon + w.i; }

// The latitude edge a walk in row j meets next, rising (dj = 1) or falling
// (-1) in latitude; sl, su: the sines of the row's edges (a pole, which is no
// face, counts as +-2: beyond reach).  A falling walk is taken mirrored at the
// equator, so both are one rising case.  upper: it is edge j + 1, met while
// the latitude rises (edge j: while it falls); met: there is one.
struct ConePick {
    double s;
    bool met, upper;
};
__host__ __device__ __forceinline__ ConePick wk_cone_pick(const Walker& w, double q2, double Pz, int dj, double sl, double su)
{
    ConePick p;
    const bool up = dj > 0;
    const double M = fma(Pz, Pz, (q2 * w.dz) * w.dz);
    const double sf = up ? su : sl, sb = up ? sl : su;  // the edges in front and behind
    const double mz = wk_flip(w.dz, dj);
    const bool turn = wk_flip(Pz, dj) > 0.0;  // the extremum is ahead
    const double reach = turn ? fma(-(sf * sf), q2, M) : mz - wk_flip(sf, dj);
    const bool front = reach > 0.0;
    const bool back = !front & turn & (mz < wk_flip(sb, dj));
    p.s = front ? sf : sb;
    p.met = front | back;
    p.upper = up == front;
    return p;
}

// Whether row j lies at the edge whose cone cannot be told from the equator.
__host__ __device__ __forceinline__ bool wk_at_eq(const GridDev& g, int j) { return j == g.eq_edge || j + 1 == g.eq_edge; }

// Coefficients of the latitude cone z^2 cos^2(lat) = (x^2 + y^2) sin^2(lat)
// along p0 + t d: a t^2 + 2 b t + c = 0.  The exact form evaluates them as
// written; the fast form uses cos^2 + sin^2 = 1 and |d| = 1, i.e.
// a = dz^2 - sin^2, b = pz dz - (p0.d) sin^2, c = pz^2 - |p0|^2 sin^2.
template <bool FAST>
__host__ __device__ __forceinline__ void wk_cone_coef(const Walker& w, double s, double c2, double& a, double& b, double& c)
{
    const double s2 = s * s;
    if constexpr (FAST) {
        a = fma(w.dz, w.dz, -s2);
        b = fma(w.pz, w.dz, -(w.B0 * s2));
        c = fma(w.pz, w.pz, -(w.C0 * s2));
    } else {
        a = w.dz * w.dz * c2 - (w.dx * w.dx + w.dy * w.dy) * s2;
        b = w.pz * w.dz * c2 - (w.px * w.dx + w.py * w.dy) * s2;
        c = w.pz * w.pz * c2 - (w.px * w.px + w.py * w.py) * s2;
    }
}

// Root of a face as a quotient: num * (1 / den) in the fast form, num / den
// in the exact one.
template <bool FAST>
__host__ __device__ __forceinline__ double wk_root(double num, double den)
{
    if constexpr (FAST) return num * wk_div<true>(1.0, den);
    else return wk_div<false>(num, den);
}

// The root at which the picked edge is met, q/a (first) or c/q of the cone's
// quadratic with q = -(b + sign(b) sqrt(disc)), as a quotient: of
// (-b -+ sqrt(disc)) / a the one of + sign(s) is met rising.  A parabolic cone
// (a = 0) has one root and the equator (s = 0) is the plane z = 0.
template <bool FAST>
__host__ __device__ __forceinline__ void wk_cone_root(const Walker& w, const ConePick& p, double a, double b, double c,
                                                      double sq, double& num, double& den)
{
    const bool bp = b >= 0.0;
    const bool first = (bp != (p.s > 0.0)) == p.upper;
    const double q = -(b + (bp ? sq : -sq));
    if constexpr (FAST) {
        num = first ? q * q : c * a;
        den = a * q;
    } else {
        num = first ? q : c;
        den = first ? a : q;
    }
    if ((p.s == 0.0) | (a == 0.0)) {
        num = p.s == 0.0 ? -w.pz : -c;
        den = p.s == 0.0 ? w.dz : 2.0 * b;
    }
}

// cos^2 of the picked latitude edge (read by the exact form only)
template <bool FAST>
__host__ __device__ __forceinline__ double wk_cos2(const GridDev& g, const Walker& w, const ConePick& p)
{
    if constexpr (FAST) return 0.0;
    else return g.lat_c2[w.j + (p.upper ? 1 : 0)];
}

// Start of a walk at (px, py, pz) in cell (i, j, k) along unit d.
template <bool FAST, int GEO = GEO_ANY>
__host__ __device__ __forceinline__ void wk_start(const GridDev& g, Walker& w, double px, double py, double pz,
                                                  double dx, double dy, double dz, int i, int j, int k)
{
    w.px = px; w.py = py; w.pz = pz;
    w.dx = dx; w.dy = dy; w.dz = dz;
    w.t = 0.0;
    w.i = i; w.j = j; w.k = k;
    w.tc = w.tp = INFINITY;
    w.far = 0.0;
    w.eq = 0;
    const double2 fr = wk_face(g, k);
    if (wk_slab<GEO>(g)) {
        w.B0 = w.C0 = 0.0;
        w.dk = dz > 0.0 ? 1 : -1;
        w.dj = w.di = 1;
        const double x = wk_div<FAST>((dz > 0.0 ? fr.y : fr.x) - pz, dz);
        w.ts = dz != 0.0 ? wk_max(x, 0.0) : INFINITY;
        return;
    }
    const bool east = px * dy - py * dx > 0.0;
    const double2 fc = wk_face(g, g.lat_base + j);
    const double2 fp = wk_face(g, g.lon_base + i + (east ? 1 : 0));
    const double B = px * dx + py * dy + pz * dz;
    const double C0 = px * px + py * py + pz * pz;
    w.B0 = B;
    // the inner sphere where the walk goes inward and meets it, else the outer one
    const double Ci = wk_mad<FAST>(-fr.x, fr.x, C0), Di = wk_mad<FAST>(B, B, -Ci);
    const double Co = wk_mad<FAST>(-fr.y, fr.y, C0), Do = wk_mad<FAST>(B, B, -Co);
    const bool inward = (B < 0.0) & (Di >= 0.0);
    const double sq = wk_sqrt<FAST>(inward ? Di : Do);
    const double q = B <= 0.0 ? -B + sq : B + sq;
    const double x = wk_div<FAST>(inward ? Ci : -Co, q);
    w.ts = wk_max((inward | (B > 0.0)) ? x : q, 0.0);
    w.far = q;
    w.dk = inward ? -1 : 1;
    w.di = east ? 1 : -1;
    // q2 >= Pz^2, but of a line through the centre both are rounding noise (some
    // 1e-15 |p0|^2) and q2 would come out negative as often as not, which puts
    // edges within reach, the poles among them.  Such a line is taken to pass the
    // centre at 1e-7 |p0|: with Pz^2 <= 2 q2 no pole is ever picked
    // (Pz^2 + q2 (dz^2 - 4) < 0).
    w.C0 = wk_max(C0, fma(B, B, 1e-14 * C0));
    const double q2 = fma(-B, B, w.C0), Pz = fma(-B, dz, pz);
    // (rising or falling: the sign of d sin(lat) / dt)
    const ConePick p = wk_cone_pick(w, q2, Pz, fma(dz, q2, -(Pz * B)) > 0.0 ? 1 : -1, fc.x, fc.y);
    w.dj = p.upper ? 1 : -1;
    double num, den, a, b, c;
    wk_cone_coef<FAST>(w, p.s, wk_cos2<FAST>(g, w, p), a, b, c);
    wk_cone_root<FAST>(w, p, a, b, c, wk_sqrt<FAST>(wk_mad<FAST>(b, b, -(a * c))), num, den);
    double r;
    if constexpr (FAST) r = ((p.s == 0.0) | (a == 0.0)) ? wk_div<true>(num, den) : wk_root<true>(num, den);
    else r = wk_root<false>(num, den);
    w.tc = (p.met & (den != 0.0)) ? wk_max(r, 0.0) : INFINITY;
    if (g.eq_edge > 0 && wk_at_eq(g, j)) w.eq = WE_ROW;
    if (g.nlon > 1) {
        const double nx = -fp.x, ny = fp.y;
        const double dn = wk_mad<FAST>(dx, nx, dy * ny);
        const double v = wk_div<FAST>(-wk_mad<FAST>(px, nx, py * ny), dn);
        w.tp = (east ? dn > 0.0 : dn < 0.0) ? wk_max(v, 0.0) : INFINITY;
    }
}

// Parameter of the next crossing and the kind of its face: a shell, else a
// cone, else a plane (none: no face ahead, only in a slab).
struct CrossKind {
    double t;
    bool shell, cone, none;
};
template <int GEO = GEO_ANY>
__host__ __device__ __forceinline__ CrossKind wk_next(const Walker& w)
{
    CrossKind x;
    if constexpr (GEO == GEO_SLAB) {
        x.t = w.ts;
        x.shell = true;
        x.cone = false;
    } else {
        x.t = wk_min(wk_min(w.ts, w.tc), w.tp);
        x.shell = w.ts <= x.t;
        x.cone = !x.shell & (w.tc <= x.t);
    }
    x.none = GEO != GEO_SPHERE && !(x.t < INFINITY);
    return x;
}

// The face-table values a crossing reads, loaded by wk_cross_begin so that a
// caller can issue other loads before the crossing's arithmetic in
// wk_cross_end waits for them.
struct CrossIn {
    double2 f;
    bool inside;
};

// Index update and table load of a crossing (of a face), without branches.
template <int GEO = GEO_ANY>
__host__ __device__ __forceinline__ CrossIn wk_cross_begin(const GridDev& g, Walker& w, const CrossKind& x)
{
    CrossIn in;
    w.t = x.t;
    if constexpr (GEO == GEO_SLAB) {
        w.k += w.dk;
        in.inside = (unsigned)w.k < (unsigned)g.nlay;
        in.f = wk_face(g, in.inside ? w.k : 0);
        return in;
    }
    int ni = w.i + w.di;
    ni = ni == g.nlon ? 0 : (ni < 0 ? g.nlon - 1 : ni);
    w.k += x.shell ? w.dk : 0;
    w.j += x.cone ? w.dj : 0;
    w.i = (x.shell | x.cone) ? w.i : ni;
    in.inside = (unsigned)w.k < (unsigned)g.nlay;
    const int er = in.inside ? w.k : 0, ec = g.lat_base + w.j, ep = g.lon_base + w.i + (w.di > 0 ? 1 : 0);
    in.f = wk_face(g, x.shell ? er : (x.cone ? ec : ep));
    return in;
}

// The next shell of a ray (a walk whose end nothing is made of: peel-off) that
// has just crossed one into a layer of edge R ahead: its roots lie at -+sqrt(R^2
// - q2) from the ray's nearest point (q2: that point's distance from the centre,
// squared), which needs no division.  The difference loses some 1e-13 of a
// layer's thickness, which a packet's path would amplify and an optical depth
// does not.  sq: the root (0 where there is none).
__host__ __device__ __forceinline__ double wk_ray_q2(const Walker& w) { return fma(-w.B0, w.B0, w.C0); }
__host__ __device__ __forceinline__ void wk_ray_shell(Walker& w, double D, double sq)
{
    const bool out = w.dk > 0, miss = !out & !(D >= 0.0);
    const double v = miss ? w.t + w.B0 : sq;
    w.ts = wk_max(wk_flip(v, w.dk) - w.B0, w.t);
    w.dk = miss ? 1 : w.dk;
}

// The face that replaces the one just crossed.  RAYS: the walk may be a ray.
template <bool FAST, int GEO = GEO_ANY, bool RAYS = false>
__host__ __device__ __forceinline__ void wk_cross_end(const GridDev& g, Walker& w, const CrossKind& x, const CrossIn& in,
                                                      bool ray = false)
{
    const bool outward = w.dk > 0;
    const double R = outward ? in.f.y : in.f.x;
    if (wk_slab<GEO>(g)) {
        w.ts = wk_max(wk_div<FAST>(R - w.pz, w.dz), w.t);
        return;
    }
    // shell: t^2 + 2 B0 t + c; cone: ca t^2 + 2 cb t + cc
    const double c = wk_mad<FAST>(-R, R, w.C0);
    double D = wk_mad<FAST>(w.B0, w.B0, -c);
    if (RAYS && ray) D = fma(R, R, -wk_ray_q2(w));
    double ca, cb, cc;
    ConePick p;
    if (x.cone) {
        const int dj = w.dj;
        p = wk_cone_pick(w, fma(-w.B0, w.B0, w.C0), fma(-w.B0, w.dz, w.pz), dj, in.f.x, in.f.y);
        w.dj = p.upper ? 1 : -1;
        if (g.eq_edge > 0 && wk_at_eq(g, w.j)) w.eq = WE_ROW | (dj > 0 ? WE_FROM_LO : WE_FROM_HI);
        wk_cone_coef<FAST>(w, p.s, wk_cos2<FAST>(g, w, p), ca, cb, cc);
        D = wk_mad<FAST>(cb, cb, -(ca * cc));
    }
    const double sq = wk_sqrt<FAST>(D);
    // the shell's root: with m = |B0| + sqrt(D), the far one of a sphere whose
    // nearest point is still ahead is m, any other next one c / m up to sign
    const double m = fabs(w.B0) + sq;
    const bool past = w.B0 > 0.0, mfar = outward & !past;
    double num = past ? -c : c, den = m;
    if constexpr (FAST) num = mfar ? m * m : num;
    bool met = true;
    if (x.cone) {
        wk_cone_root<FAST>(w, p, ca, cb, cc, sq, num, den);
        met = p.met;
    } else if (!x.shell) {
        const double nx = -in.f.x, ny = in.f.y;
        den = wk_mad<FAST>(w.dx, nx, w.dy * ny);
        num = -wk_mad<FAST>(w.px, nx, w.py * ny);
        met = wk_flip(den, w.di) > 0.0;
    }
    const bool finite = den != 0.0;
    double r = wk_root<FAST>(num, den);
    if (RAYS && x.shell && ray) {
        wk_ray_shell(w, D, sq);
    } else if (x.shell) {
        if constexpr (!FAST) r = mfar ? m : r;
        const bool hit = outward | ((D >= 0.0) & ((r >= w.t) | (c < 0.0)));
        w.ts = wk_max(hit ? (finite ? r : 0.0) : w.far, w.t);
        w.dk = hit ? w.dk : 1;
        w.far = m;
    } else {
        const double v = (met & finite) ? wk_max(r, w.t) : INFINITY;
        w.tc = x.cone ? v : w.tc;
        w.tp = x.cone ? w.tp : v;
    }
}

// tc of a walk that has just entered a row at the edge eq_edge.  Where an edge
// lies within rounding of the equator without being it (sin^2 < 1e-16), its
// two cone roots are one to rounding and which nappe each lies on is decided
// by rounding, so that edge may be met once, twice or not at all.  The
// results of such grids are those of taking, of the roots of both edges that
// fall on their nappe, the first one ahead (past 1e-9 of the radius for the
// edge just crossed).
template <bool FAST>
__host__ __device__ __forceinline__ void wk_row_roots(const GridDev& g, Walker& w)
{
    const double tol = 1e-9 * g.faces[g.nlay - 1].y;
    const double2 f = wk_face(g, g.lat_base + w.j);
    double best = INFINITY;
    bool upper = false;
    for (int e = 0; e < 2; ++e) {
        const int je = w.j + e;
        if (je == 0 || je == g.nlat) continue;
        const double s = e ? f.y : f.x;  // (not a pole here)
        double a, b, c;
        wk_cone_coef<FAST>(w, s, FAST ? 0.0 : g.lat_c2[je], a, b, c);
        const double disc = wk_mad<FAST>(b, b, -(a * c));
        if (!(disc >= 0.0) || a == 0.0) continue;
        const double sq = wk_sqrt<FAST>(disc);
        const double q = -(b + (b >= 0.0 ? sq : -sq));
        double x0 = 0.0, x1 = INFINITY;
        if (q != 0.0) {
            x0 = FAST ? wk_root<FAST>(q * q, a * q) : wk_root<FAST>(q, a);
            x1 = FAST ? wk_root<FAST>(c * a, a * q) : wk_root<FAST>(c, q);
        }
        const double lo = (w.eq & (e ? WE_FROM_HI : WE_FROM_LO)) ? w.t + tol : w.t;
        for (int m = 0; m < 2; ++m) {
            const double x = m ? x1 : x0, z = wk_mad<FAST>(x, w.dz, w.pz);
            if (x < INFINITY && x >= lo && (s > 0.0 ? z > 0.0 : z < 0.0) && x < best) {
                best = x;
                upper = e == 1;
            }
        }
    }
    w.tc = best;
    w.dj = upper ? 1 : -1;
    w.eq = 0;
}

}  // namespace dev
}  // namespace mcrt

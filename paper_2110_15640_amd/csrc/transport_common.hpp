// Device code shared by the kernels of the packet transport (transport.hip:
// flights and peel-off rays in one kernel; flight.hip: in two): lane states,
// the step of a walk, scattering.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "device_common.hpp"
#include "mcrt_internal.hpp"

namespace mcrt {
namespace {
using namespace dev;

constexpr int kTPB = 256;

// Lane modes; the walking ones come first: a flight, a peel-off ray, or the
// probe of a forced interaction (the optical depth to the grid's edge along
// the packet direction).
enum { M_FLIGHT = 0, M_PEEL = 1, M_PROBE = 2, M_EVENT = 3, M_DEAD = 4, M_BIRTH = 5, M_IDLE = 6 };
// Observer-field values outside the observer range: the walk that ended was a
// probe, or the next flight's optical depth is already chosen.
constexpr int kProbeDone = 15, kTauSet = 14;
enum { E_INTERACT = 0, E_ESCAPE = 1, E_SURFACE = 2, E_LOST = 3, E_PEEL_DONE = 4 };
// Birth record of a packet, kept in the counter columns of its row until the
// packet dies: position, direction, weight, packed cell (i | j << 11 | k << 21)
// (-1: nothing emits), then the index of the solve whose optics it uses;
// with a Lambert floor, the weight the floor has absorbed so far; with
// forced interactions, the unscattered fractions booked so far to the floor
// (B_SURF) and to escape (B_FESC).
enum { B_X = 0, B_Y, B_Z, B_DX, B_DY, B_DZ, B_W, B_CELL, B_SOLVE, B_SURF, B_FESC };

__host__ __device__ __forceinline__ unsigned long long pack_ijk(int i, int j, int k)
{
    return (unsigned long long)i | ((unsigned long long)j << 11) | ((unsigned long long)k << 21);
}

// A bit field [sh, sh + w) of a packed LDS word, used like an int.
struct Bits {
    uint32_t* p;
    int sh;
    uint32_t m;
    __device__ operator int() const { return (int)((*p >> sh) & m); }
    __device__ Bits& operator=(int v)
    {
        *p = (*p & ~(m << sh)) | (((uint32_t)v & m) << sh);
        return *this;
    }
    __device__ Bits& operator+=(int v) { return *this = (int)*this + v; }
};

// floor(total * x / kXcds) without overflow.
__device__ __forceinline__ unsigned long long chunk_edge(unsigned long long total, int x)
{
    return (total / kXcds) * (unsigned long long)x + (total % kXcds) * (unsigned long long)x / kXcds;
}

template <bool MIXED>
__device__ __forceinline__ double ld(const void* p, int c)
{
    // per-cell optical properties live in global memory: load through the
    // global address space (a global, not a flat, load)
    typedef const __attribute__((address_space(1))) float gfloat;
    typedef const __attribute__((address_space(1))) double gdouble;
    if (MIXED) return (double)((gfloat*)p)[c];
    return ((gdouble*)p)[c];
}

// The stored type of the optical properties.
template <bool MIXED>
using Prop = typename std::conditional<MIXED, float, double>::type;

// A grid of the launch's table through the scalar cache (i uniform across the
// wave; the table is not written while a kernel runs).
__device__ __forceinline__ GridDev uniform_grid(const GridDev* grids, int i)
{
    static_assert(sizeof(GridDev) % 8 == 0, "whole words");
    typedef const __attribute__((address_space(4))) uint64_t* Words;
    const Words p = (Words)(uintptr_t)(grids + __builtin_amdgcn_readfirstlane(i));
    uint64_t w[sizeof(GridDev) / 8];
#pragma unroll
    for (int k = 0; k < (int)(sizeof(GridDev) / 8); ++k) w[k] = p[k];
    GridDev g;
    __builtin_memcpy(&g, w, sizeof g);
    return g;
}

// Runs f on the grid of a lane's walk.  Of launches on several grids nearly all
// waves hold walks on one of them (their packets follow each other in a solve):
// those read its shape through the scalar cache instead of per lane at each
// step: 200 solves on 128 x 64 x 50 cells, mixed, take 44.4 ms by per-lane
// reads, 41.3 by these, 34.6 by the kernels of one grid.
template <bool MULTI, class F>
__device__ __forceinline__ void on_grid(const GridDev& g1, const GridDev* grids, int lgrid, bool active, F f)
{
    if constexpr (!MULTI) {
        f(g1);
    } else {
        const unsigned long long act = __ballot(active);
        const int ug = act != 0 ? __shfl(lgrid, __ffsll(act) - 1) : 0;
        if (__ballot(active && lgrid != ug) == 0) f(uniform_grid(grids, ug));
        else f(grids[lgrid]);
    }
}

// One cell of a walk.  Flights and peel-off rays share the exit search, the
// extinction gather and the crossing (a single inlined copy of each, so that
// a wave holding both kinds executes them once); they differ only in how the
// optical depth is used and in when the walk stops.  ae: the extinction of
// the walk's cell, gathered when the cell was entered (wk_start's first cell:
// by the caller), so that a step's end and the next one's start cover the
// gather's latency.
template <bool MIXED, bool EXT, int GEO, bool RAYS, class LaneT>
__device__ __forceinline__ void walk_step(LaneT& L, const GridDev& g, const void* aext, const void* aabs,
                                          Prop<MIXED>& ae, const BatchArgs& A)
{
    const CrossKind x = wk_next<GEO>(L.w);
    const double s = x.t - L.w.t;
    const bool flight = L.mode == M_FLIGHT;
    double a = (double)ae;
    if constexpr (EXT) {
        if (A.absorption == 1 && flight) {  // continuous absorption: tau counts scattering only
            const double aa = ld<MIXED>(aabs, wk_cell(g, L.w));
            a = a - aa;
            const bool ends = (a > 0.0) & (L.tau < a * s);
            if (ends | !x.none) {
                const double ds = ends ? wk_div<MIXED>(L.tau, a) : s;
                const double wn = L.W * exp(-aa * ds);
                L.w_abs = L.w_abs + (L.W - wn);
                L.W = wn;
            }
        }
    }
    const bool hit = flight & (a > 0.0) & (L.tau < a * s);
    if (hit | x.none) {
        L.ncross += L.ncw;
        L.mode = M_EVENT;
        if (hit) {  // at t + tau / a (tau is the depth left on entering the cell)
            const double ti = L.w.t + wk_div<MIXED>(L.tau, a);
            L.sx() = wk_mad<MIXED>(ti, L.w.dx, L.w.px);
            L.sy() = wk_mad<MIXED>(ti, L.w.dy, L.w.py);
            L.sz() = wk_mad<MIXED>(ti, L.w.dz, L.w.pz);
            L.set_cell(L.w.i, L.w.j, L.w.k);
        }
        if (!flight) L.tau = INFINITY;
        L.ev = hit ? E_INTERACT : (flight ? E_LOST : E_PEEL_DONE);
        return;
    }
    const CrossIn in = wk_cross_begin<GEO>(g, L.w, x);
    ae = (Prop<MIXED>)ld<MIXED>(aext, in.inside ? wk_cell(g, L.w) : 0);
    L.tau = wk_mad<MIXED>(flight ? -a : a, s, L.tau);
    L.ncw++;
    const bool capped = L.ncw >= g.max_cross;
    // a probe runs to the edge of the grid, the floor included; a peel-off
    // ray stops beyond tau_peel_max or on the planet
    const bool probe = EXT && L.mode == M_PROBE;
    const bool dark = !flight & !probe & (L.tau > A.tau_peel_max);
    if (!in.inside | capped | dark) {
        if (flight) L.ev = !in.inside ? (L.w.k >= g.nlay ? E_ESCAPE : E_SURFACE) : E_LOST;
        else L.ev = E_PEEL_DONE;
        if (!flight && (in.inside || (L.w.k < 0 && !probe) || dark)) L.tau = INFINITY;
        L.ncross += L.ncw;
        L.mode = M_EVENT;
        return;
    }
    wk_cross_end<MIXED, GEO, RAYS>(g, L.w, x, in, L.mode == M_PEEL);
}

// Pending actions of a lane after an event; each is executed at exactly one
// place in the kernel loop so its code (and register demand) appears once.
enum { A_NONE = 0, A_PEEL = 1, A_FLIGHT = 2, A_SCATTER = 3, A_FINISH = 4 };

// Survival weight update, scattering angle, rotation, roulette, event cap.
// A reflection by the Lambert floor takes the same steps: its albedo is A_s,
// its absorbed share goes to the floor, and its polar cosine about the
// normal (held as the packet direction) is sqrt(zeta), block 1, slot a.
// om, pg, gc: the optical properties of the event's cell.
template <bool MIXED, bool EXT, class LaneT>
__device__ __forceinline__ int scatter(LaneT& L, const BatchArgs& A, const SolveDev& S, double om, double pg, double gc)
{
    const unsigned long long q = L.gid() - S.pbase;
    const bool sf = EXT && L.surf();
    if (sf) {
        om = A.surface_albedo;
        pg = gc = 0.0;
        double* b = A.rows + L.gid() * (unsigned long long)A.row_w + A.n_out;
        b[B_SURF] = b[B_SURF] + L.W * (1.0 - om);
        L.W = L.W * om;
    } else if (A.absorption != 1) {
        L.w_abs += L.W * (1.0 - om);
        L.W = L.W * om;
    }
    const double usel = draw(A.seed, S.tag, q, L.e(), 0).b;  // scatterer choice of this event
    U2 u1 = draw(A.seed, S.tag, q, L.e(), 1);
    // two-term HG clouds: the forward lobe g with weight 1 - (g/2)^2 or the
    // backward lobe -g/2, chosen by block 2, slot b of the event
    double globe = gc;
    if (A.cloud_phase == 1 && !sf && !(usel < pg)) {
        const double g2 = -0.5 * gc, a = 1.0 - g2 * g2;
        globe = draw(A.seed, S.tag, q, L.e(), 2).b < a ? gc : g2;
    }
    // Draine clouds (g_cld holds G): rejection from HG(G), candidate 0 from
    // block 1, slot a with acceptance block 2, slot b; candidate k >= 1 from
    // block 2 + k; at most 32 candidates
    const bool draine = EXT && A.cloud_phase == 2 && !sf && !(usel < pg);
    if (MIXED) {
        float z = fminf((float)u1.a, 0.99999994f);
        float mu;
        float g32 = (float)globe;
        auto hgs = [g32](float zz) {
            if (fabsf(g32) < 1e-6f) return 2.0f * zz - 1.0f;
            const float t = (1.0f - g32 * g32) / (1.0f - g32 + 2.0f * g32 * zz);
            return (1.0f + g32 * g32 - t * t) / (2.0f * g32);
        };
        if (sf) {
            mu = sqrtf(z);
        } else if ((float)usel < (float)pg) {
            float qq = 4.0f * z - 2.0f;
            float u = cbrtf(qq + sqrtf(qq * qq + 1.0f));
            mu = u - 1.0f / u;
        } else {
            mu = hgs(z);
        }
        if (draine) {
            const float al = (float)A.draine_alpha;
            float zc = (float)draw(A.seed, S.tag, q, L.e(), 2).b;
            for (int k = 1; k < 32 && !(zc * (1.0f + al) < 1.0f + al * mu * mu); ++k) {
                const U2 cd = draw(A.seed, S.tag, q, L.e(), 2 + k);
                mu = hgs(fminf((float)cd.a, 0.99999994f));
                zc = (float)cd.b;
            }
        }
        mu = fminf(fmaxf(mu, -1.0f), 1.0f);
        float st = sqrtf(fmaxf(1.0f - mu * mu, 0.0f));
        float sp, cp;
        __sincosf((float)(2.0 * kPi) * (float)u1.b, &sp, &cp);
        float dx = (float)L.sdx(), dy = (float)L.sdy(), dz = (float)L.sdz();
        float nx, ny, nz;
        if (fabsf(dz) < 0.99999f) {
            float t = sqrtf(1.0f - dz * dz);
            float it = 1.0f / t;
            nx = st * (dx * dz * cp - dy * sp) * it + dx * mu;
            ny = st * (dy * dz * cp + dx * sp) * it + dy * mu;
            nz = -st * cp * t + dz * mu;
        } else {
            float sgn = dz >= 0.0f ? 1.0f : -1.0f;
            nx = st * cp;
            ny = st * sp;
            nz = sgn * mu;
        }
        // renormalised in FP64 (the traversal takes |d| = 1): one refined
        // reciprocal square root and three products
        double ddx = nx, ddy = ny, ddz = nz;
        const double nn = fma(ddx, ddx, fma(ddy, ddy, ddz * ddz));
        double y = __builtin_amdgcn_rsq(nn);
        y = y * fma(-0.5 * nn, y * y, 1.5);
        y = y * fma(-0.5 * nn, y * y, 1.5);
        L.sdx() = ddx * y;
        L.sdy() = ddy * y;
        L.sdz() = ddz * y;
    } else {
        double mu = sf ? sqrt(u1.a) : ((usel < pg) ? sample_rayleigh(u1.a) : sample_hg(u1.a, globe));
        if (draine) {
            const double al = A.draine_alpha;
            double zc = draw(A.seed, S.tag, q, L.e(), 2).b;
            for (int k = 1; k < 32 && !(zc * (1.0 + al) < 1.0 + al * mu * mu); ++k) {
                const U2 cd = draw(A.seed, S.tag, q, L.e(), 2 + k);
                mu = sample_hg(cd.a, globe);
                zc = cd.b;
            }
        }
        rotate_dir(L.sdx(), L.sdy(), L.sdz(), mu, 2.0 * kPi * u1.b);
    }
    if (L.W < A.rr_threshold * L.W0()) {
        U2 u2 = draw(A.seed, S.tag, q, L.e(), 2);
        if (u2.a < A.rr_survive) {
            double wn = L.W / A.rr_survive;
            L.w_rr() -= (wn - L.W);
            L.W = wn;
        } else {
            L.w_rr() += L.W;
            L.W = 0.0;
            L.ev = -1;
            return A_FINISH;
        }
    }
    if ((long long)L.e() >= A.max_events) {
        L.ncapped() += 1;
        L.ev = K_CAP;
        return A_FINISH;
    }
    L.e() += 1;
    return A_FLIGHT;
}

// The phase-function weight of a ray at cosine mu of its event, times 1/(4 pi).
template <bool MIXED>
__device__ __forceinline__ double peel_weight(const BatchArgs& A, double w, double mu, double pg, double gc)
{
    // normalised mixture of the Rayleigh and cloud phase functions toward the
    // observer, weighted by the gas scattering probability
    if (MIXED) {
        const float m = (float)mu, pgf = (float)pg, gcf = (float)gc;
        const float pr = 0.75f * (1.0f + m * m);
        auto hgf = [m](float gg) {
            if (!(fabsf(gg) >= 1e-6f)) return 1.0f;
            const float den = 1.0f + gg * gg - 2.0f * gg * m;
            return (1.0f - gg * gg) / (den * sqrtf(den));
        };
        float ph;
        if (A.cloud_phase == 1) {
            const float g2 = -0.5f * gcf, af = 1.0f - g2 * g2;
            ph = af * hgf(gcf) + (1.0f - af) * hgf(g2);
        } else if (A.cloud_phase == 2) {  // Draine (gcf is G)
            const float al = (float)A.draine_alpha;
            ph = hgf(gcf) * (1.0f + al * m * m) / (1.0f + al * (1.0f + 2.0f * gcf * gcf) / 3.0f);
        } else {
            ph = hgf(gcf);
        }
        const float theta = (pgf * pr + (1.0f - pgf) * ph) * (float)(0.25 / kPi);
        return (double)((float)w * theta);
    }
    double pc;
    if (A.cloud_phase == 1) {
        const double g2 = -0.5 * gc, a = 1.0 - g2 * g2;
        pc = a * p_hg(mu, gc) + (1.0 - a) * p_hg(mu, g2);
    } else if (A.cloud_phase == 2) {  // Draine (gc is G)
        const double al = A.draine_alpha;
        pc = p_hg(mu, gc) * (1.0 + al * mu * mu) / (1.0 + al * (1.0 + 2.0 * gc * gc) / 3.0);
    } else {
        pc = p_hg(mu, gc);
    }
    const double theta = (pg * p_rayleigh(mu) + (1.0 - pg) * pc) / (4.0 * kPi);
    return w * theta;
}

// Pixel of a sky-plane coordinate x on npix pixels over [-half, half].
__device__ __forceinline__ int pixel_of(double x, double half, int npix)
{
    const int q = (int)floor((x + half) / (2.0 * half) * (double)npix);
    return q < 0 ? 0 : (q >= npix ? npix - 1 : q);
}

// The counter columns of a finished packet's row; `kind` says where its
// remaining weight went.  EXT (here and below): the kernel form with the
// Lambert floor, Draine clouds, forced interactions, continuous absorption
// and multiple-scattering transmission; without it that code is compiled out.
template <bool EXT, class LaneT>
__device__ __forceinline__ void finish_counters(LaneT& L, const BatchArgs& A, int kind)
{
    double* row = A.rows + L.gid() * (unsigned long long)A.row_w + A.n_out;
    if (EXT) {
        // weight booked before the end: absorbed by a Lambert floor (which
        // never ends a packet) or the unscattered fractions of forced flights
        const double wsurf = (A.surface_albedo > 0.0 || A.forced) ? row[B_SURF] : 0.0;
        const double wesc = A.forced ? row[B_FESC] : 0.0;
        row[K_ESC] = kind == K_ESC ? wesc + L.W : wesc;
        row[K_SURF] = kind == K_SURF ? wsurf + L.W : wsurf;
    } else {
        row[K_ESC] = kind == K_ESC ? L.W : 0.0;
        row[K_SURF] = kind == K_SURF ? L.W : 0.0;
    }
    row[K_ABS] = L.w_abs;
    row[K_RR] = L.w_rr();
    row[K_CAP] = kind == K_CAP ? L.W : 0.0;
    row[K_LOST] = kind == K_LOST ? L.W : 0.0;
    row[K_NINT] = (double)L.nint();
    row[K_NCROSS] = (double)L.ncross;
    row[K_NCAPPED] = (double)L.ncapped();
    row[K_NLOST] = (double)L.nlost();
    row[K_W0] = L.W0();
    L.mode = M_DEAD;
}

// A wave's next share of a range kept in kXcds counters (`stride` elements
// apart), one per XCD: adds n to one that lies below its limit (lim in lane x
// for counter x) and returns its index and the value before, or -1.  The
// wave's own XCD's first (blocks are dealt to the XCDs round-robin); once that
// is used up (own = false from then on) lane x reads counter x, all at once
// and past the L2 (whose copy another XCD's additions leave stale), and only
// one that has something left is added to: 4,096 waves adding to eight used up
// counters in one cache line took 0.5 ms at the end of every launch.  Every
// lane of the wave calls it.
template <typename T>
__device__ __forceinline__ int take_share(T* c, int stride, T lim, T n, int lane, bool& own, T& before)
{
    int x = (int)(blockIdx.x % kXcds);
    for (;;) {
        if (!own) {
            T v = lim;
            if (lane < kXcds) v = __hip_atomic_load(c + lane * stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned open = (unsigned)(__ballot(v < lim) & ((1ull << kXcds) - 1ull));
            if (open == 0) return -1;
            const int x0 = (int)(blockIdx.x % kXcds);
            const unsigned rot = (open >> x0 | open << (kXcds - x0)) & ((1u << kXcds) - 1u);
            x = (x0 + __ffs(rot) - 1) % kXcds;
        }
        T b = 0;
        if (lane == 0) b = atomicAdd(c + x * stride, n);
        before = __shfl(b, 0);
        if (before < __shfl(lim, x)) return x;
        own = false;
    }
}

// The next packets of a wave's reservoir [next, end), refilled from the
// launch's dispensers `batch` at a time: the packet range is split into one
// contiguous chunk per XCD, so each XCD's L2 holds the optics of its own
// solves; a wave whose chunk is drained helps the next ones.  false: drained.
__device__ __forceinline__ bool refill(const BatchArgs& A, int lane, bool& own, unsigned long long& next,
                                       unsigned long long& end)
{
    const unsigned long long mine = lane < kXcds ? chunk_edge(A.total, lane + 1) : 0ull;
    unsigned long long b;
    const int x = take_share(A.counter, A.ctr_stride, mine, (unsigned long long)A.batch, lane, own, b);
    if (x < 0) return false;
    const unsigned long long lim = __shfl(mine, x);
    next = b;
    end = b + (unsigned long long)A.batch < lim ? b + A.batch : lim;
    return true;
}

// Index of the solve that owns global packet gid (last solve with begin <= gid).
__device__ __forceinline__ int solve_of(const BatchArgs& A, unsigned long long gid)
{
    int lo = 0, hi = A.n_solves - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (A.solves[mid].begin <= gid) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

}  // namespace
}  // namespace mcrt

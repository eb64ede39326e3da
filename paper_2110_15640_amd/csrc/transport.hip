// K4: persistent packet transport with wavefront-level regeneration.
//
// Every lane of a wave64 carries one photon packet (Sect. 2: packets are
// emitted or injected, sample an optical depth, move sub-grid through the
// spherical cells, interact, scatter or are absorbed, and are peeled off
// toward every observer at each emission and interaction, Sect. 4.6).
// Flights and peel-off rays are both walks through the grid, so the
// cell-exit computation runs for all walking lanes together; the rarer
// events (interaction, end of a peel-off, death, birth) are handled only
// when at least ev_threshold lanes wait on one, or when no lane walks.
// Lanes whose packet has terminated take the next packet index from the
// wave's reservoir, refilled from a global dispenser, so the grid drains
// without tail imbalance and many (spectral point, g) solves share a launch.
//
// Per packet the kernel writes one row: the peel-off sums F_o toward each
// observer, then the bookkeeping counters.  A fixed-order reduction over the
// rows forms the tallies, so results are deterministic and identical whether
// a solve runs alone or inside a batch.
//
// Precision: FP64 keeps everything in double.  MIXED gathers float optical
// properties and evaluates phase functions, scattering angles, the direction
// rotation and the peel-off attenuation in float; positions, the directions
// the traversal uses, exit distances, optical depths and tallies stay double.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <math.h>
#include <stdint.h>

#include "transport_common.hpp"

namespace mcrt {
namespace {
using namespace dev;

// Per-lane state that the cell walk does not touch lives in LDS (one slot
// per lane, structure of arrays) so the registers hold only the walking ray;
// small fields are packed into 32-bit words.  The packet's peel-off sums
// accumulate in LDS too and reach memory once, with its whole row.
struct ColdLDS {
    double sx[kTPB], sy[kTPB], sz[kTPB];      // event point
    double sdx[kTPB], sdy[kTPB], sdz[kTPB];   // packet direction
    double W0[kTPB], w_rr[kTPB];
    unsigned long long gid[kTPB];
    uint32_t ijk[kTPB];   // event cell: i | j << 11 | k << 21
    uint32_t st[kTPB];    // observer:4 | birth:1 | smode:1 | 3 unused | capped:1 | lost:1 | surface:1 | solve:20
    uint32_t e[kTPB];
    int nint[kTPB];
};

struct Lane {
    Walker w;      // the walking ray (flight or peel-off)
    double tau;    // flight: optical depth left; peel-off: accumulated
    double W, w_abs;
    int ncw;       // crossings of the current walk
    int ncross;
    int mode, ev;
    // cold state in LDS, accessed through these references
    ColdLDS* C;
    double* F;     // peel-off sums, F[o * kTPB + t]
    int t;
    __device__ double& sx() { return C->sx[t]; }
    __device__ double& sy() { return C->sy[t]; }
    __device__ double& sz() { return C->sz[t]; }
    __device__ double& sdx() { return C->sdx[t]; }
    __device__ double& sdy() { return C->sdy[t]; }
    __device__ double& sdz() { return C->sdz[t]; }
    __device__ double& W0() { return C->W0[t]; }
    __device__ double& w_rr() { return C->w_rr[t]; }
    __device__ unsigned long long& gid() { return C->gid[t]; }
    __device__ uint32_t& e() { return C->e[t]; }
    __device__ int& nint() { return C->nint[t]; }
    __device__ double& Fo(int o) { return F[o * kTPB + t]; }
    __device__ Bits o() { return Bits{&C->st[t], 0, 0xFu}; }
    __device__ Bits birth() { return Bits{&C->st[t], 4, 0x1u}; }
    __device__ Bits smode() { return Bits{&C->st[t], 5, 0x1u}; }
    __device__ Bits ncapped() { return Bits{&C->st[t], 9, 0x1u}; }
    __device__ Bits nlost() { return Bits{&C->st[t], 10, 0x1u}; }
    __device__ Bits surf() { return Bits{&C->st[t], 11, 0x1u}; }  // the event is a reflection by the floor
    __device__ int solve() { return (int)(C->st[t] >> 12); }
    __device__ void set_solve(int s) { Bits{&C->st[t], 12, 0xFFFFFu} = s; }
    __device__ int si() { return (int)(C->ijk[t] & 0x7FFu); }
    __device__ int sj() { return (int)((C->ijk[t] >> 11) & 0x3FFu); }
    __device__ int sk() { return (int)(C->ijk[t] >> 21); }
    __device__ void set_cell(int i, int j, int k) { C->ijk[t] = (uint32_t)i | ((uint32_t)j << 11) | ((uint32_t)k << 21); }
    __device__ int cell(const GridDev& g) { return (sk() * g.nlat + sj()) * g.nlon + si(); }
};

// Write the packet's row: its peel-off sums, then the counters.
template <bool EXT>
__device__ __forceinline__ void finish_packet(Lane& L, const BatchArgs& A, int kind)
{
    double* row = A.rows + L.gid() * (unsigned long long)A.row_w;
    for (int o = 0; o < A.n_out; ++o) row[o] = (EXT && A.trans_ms) ? L.W0() - L.Fo(o) : L.Fo(o);
    finish_counters<EXT>(L, A, kind);
}

__device__ __forceinline__ void observer(Lane& L, const BatchArgs& A, const double* sobs, double& ox, double& oy,
                                         double& oz)
{
    if (A.n_obs == 0) {  // slab backscatter: minus the incidence direction of the birth record
        const double* b = A.rows + L.gid() * (unsigned long long)A.row_w + A.n_out;
        ox = -b[B_DX];
        oy = 0.0;
        oz = -b[B_DZ];
    } else {
        const double* ob = sobs + L.smode() * (3 * kMaxObs);
        ox = ob[3 * L.o()];
        oy = ob[3 * L.o() + 1];
        oz = ob[3 * L.o() + 2];
    }
}

// Start the lane's next walk from its event point: a flight along the
// packet direction (optical depth drawn from the event's block 0, slot a,
// unless a forced interaction chose it), a peel-off ray toward the current
// observer, or, before a forced flight, the probe along the packet
// direction.  All use one inlined walker start, so a wave starting several
// kinds runs it once.
template <bool MIXED, bool EXT>
__device__ __forceinline__ void start_walk(Lane& L, const GridDev& g, const BatchArgs& A, const double* sobs,
                                           bool flight)
{
    double dx, dy, dz;
    if constexpr (!EXT) {
        if (flight) {
            const SolveDev& S = A.solves[L.solve()];
            U2 u = draw(A.seed, S.tag, L.gid() - S.pbase, L.e(), 0);
            L.tau = -log(u.a);
            dx = L.sdx();
            dy = L.sdy();
            dz = L.sdz();
        } else {
            observer(L, A, sobs, dx, dy, dz);
            L.tau = 0.0;
        }
        wk_start<MIXED>(g, L.w, L.sx(), L.sy(), L.sz(), dx, dy, dz, L.si(), L.sj(), L.sk());
        L.ncw = 0;
        L.mode = flight ? M_FLIGHT : M_PEEL;
        if (!flight && g.geom == 1 && !(dz > 0.0)) {  // a slab peel-off ray that never reaches the top
            L.tau = INFINITY;
            L.mode = M_EVENT;
            L.ev = E_PEEL_DONE;
        }
    } else {
        int kind = flight ? M_FLIGHT : M_PEEL;
        if (flight && A.forced != 0 && L.o() != kTauSet && (A.forced_first == 0 || L.e() == 1)) kind = M_PROBE;
        if (kind == M_FLIGHT) {
            if (A.forced != 0 && L.o() == kTauSet) {
                L.o() = 0;
            } else {
                const SolveDev& S = A.solves[L.solve()];
                U2 u = draw(A.seed, S.tag, L.gid() - S.pbase, L.e(), 0);
                L.tau = -log(u.a);
            }
        } else {
            L.tau = 0.0;
        }
        if (kind == M_PEEL) {
            observer(L, A, sobs, dx, dy, dz);
        } else {
            dx = L.sdx();
            dy = L.sdy();
            dz = L.sdz();
        }
        if (kind == M_PROBE) L.o() = kProbeDone;
        wk_start<MIXED>(g, L.w, L.sx(), L.sy(), L.sz(), dx, dy, dz, L.si(), L.sj(), L.sk());
        L.ncw = 0;
        L.mode = kind;
        // a slab peel-off ray that never reaches the top, or a floor peel-off
        // ray below the horizon (the floor's normal is the packet direction then)
        const bool dark = kind == M_PEEL && ((g.geom == 1 && !(dz > 0.0)) ||
                                             (L.surf() && !(L.sdx() * dx + L.sdy() * dy + L.sdz() * dz > 0.0)));
        if (dark) {
            L.tau = INFINITY;
            L.mode = M_EVENT;
            L.ev = E_PEEL_DONE;
        }
    }
}

// Bookkeeping of one event; returns the action that follows.  L.ev carries
// the counter that receives the final weight when the action is A_FINISH.
template <bool MIXED, bool EXT>
__device__ __forceinline__ int handle_event(Lane& L, const GridDev& g, const BatchArgs& A)
{
    const SolveDev& S = A.solves[L.solve()];
    if (EXT && L.ev == E_PEEL_DONE && L.o() == kProbeDone) {
        // forced interaction: with the path's optical depth tp known, the
        // flight's tau comes from a density on [0, tp], the weight takes the
        // factor e^{-tau}/q(tau) and the unscattered fraction W e^{-tp} is
        // booked where the path ends (nothing is forced when tp is 0 or
        // infinite: a walk failure or the crossing cap)
        const double tp = L.tau;
        const unsigned long long q = L.gid() - S.pbase;
        const U2 u = draw(A.seed, S.tag, q, L.e(), 0);
        double tau = -log(u.a);
        if (tp > 0.0 && tp < INFINITY) {
            double wf;
            tau = forced_tau(A.forced, tp, u.a, draw(A.seed, S.tag, q, L.e(), 34).a, wf);
            double* b = A.rows + L.gid() * (unsigned long long)A.row_w + A.n_out;
            const int slot = L.w.k < 0 ? B_SURF : B_FESC;
            b[slot] = b[slot] + L.W * exp(-tp);
            L.W = L.W * wf;
        }
        L.tau = tau;
        L.o() = kTauSet;
        return A_FLIGHT;
    }
    if (L.ev == E_PEEL_DONE) {
        double f;
        // attenuation e^{-tau} in FP32 in the mixed form, as for the scattered peel-offs below
        const double att = MIXED ? (double)(L.tau < INFINITY ? __expf(-(float)L.tau) : 0.0f) : exp(-L.tau);
        if (L.birth()) {  // emission point (isotropic), or a transmission chord's direct light
            f = (EXT && A.trans_ms) ? L.W * att : L.W * att / (4.0 * kPi);
        } else if (EXT && L.surf()) {  // Lambert floor: W A_s max(n.o, 0)/pi e^{-tau}, n held as the direction
            const double mu = L.sdx() * L.w.dx + L.sdy() * L.w.dy + L.sdz() * L.w.dz;
            f = mu > 0.0 ? L.W * A.surface_albedo * (mu / kPi) * att : 0.0;
        } else {
            // normalised mixture of the Rayleigh and cloud phase functions
            // toward the observer, weighted by the gas scattering probability
            const int c = L.cell(g);
            const double om = ld<MIXED>(S.omega, c), pg = ld<MIXED>(S.p_gas, c), gc = ld<MIXED>(S.g_cld, c);
            if (MIXED) {
                float mu = (float)(L.sdx() * L.w.dx + L.sdy() * L.w.dy + L.sdz() * L.w.dz);
                float pgf = (float)pg, gcf = (float)gc;
                float pr = 0.75f * (1.0f + mu * mu);
                auto hgf = [mu](float gg) {
                    if (!(fabsf(gg) >= 1e-6f)) return 1.0f;
                    const float den = 1.0f + gg * gg - 2.0f * gg * mu;
                    return (1.0f - gg * gg) / (den * sqrtf(den));
                };
                float ph;
                if (A.cloud_phase == 1) {
                    const float g2 = -0.5f * gcf, af = 1.0f - g2 * g2;
                    ph = af * hgf(gcf) + (1.0f - af) * hgf(g2);
                } else if (EXT && A.cloud_phase == 2) {  // Draine (gcf is G)
                    const float al = (float)A.draine_alpha;
                    ph = hgf(gcf) * (1.0f + al * mu * mu) / (1.0f + al * (1.0f + 2.0f * gcf * gcf) / 3.0f);
                } else {
                    ph = hgf(gcf);
                }
                float theta = (pgf * pr + (1.0f - pgf) * ph) * (float)(0.25 / kPi);
                float w = A.absorption == 1 ? (float)L.W : (float)(L.W * om);
                f = (double)(w * theta * (float)att);
            } else {
                double mu = L.sdx() * L.w.dx + L.sdy() * L.w.dy + L.sdz() * L.w.dz;
                double pc;
                if (A.cloud_phase == 1) {
                    const double g2 = -0.5 * gc, a = 1.0 - g2 * g2;
                    pc = a * p_hg(mu, gc) + (1.0 - a) * p_hg(mu, g2);
                } else if (EXT && A.cloud_phase == 2) {  // Draine (gc is G)
                    const double al = A.draine_alpha;
                    pc = p_hg(mu, gc) * (1.0 + al * mu * mu) / (1.0 + al * (1.0 + 2.0 * gc * gc) / 3.0);
                } else {
                    pc = p_hg(mu, gc);
                }
                double theta = (pg * p_rayleigh(mu) + (1.0 - pg) * pc) / (4.0 * kPi);
                f = A.absorption == 1 ? L.W * theta * att : L.W * om * theta * att;
            }
        }
        // scattered light of a transmission packet: per steradian, over the
        // stellar beam's solid angle (peel_w = 1 otherwise)
        if (EXT && !L.birth()) f = f * A.peel_w;
        L.Fo(L.o()) += f;
        if ((S.cf || S.img) && f > 0.0) {
            const double sc = f * (S.cf_ltot ? S.cf_w * *S.cf_ltot : S.cf_w);
            if (S.cf) {  // contribution function: the event's cell, thermal or scattered part
                const int ncell = g.nlon * g.nlat * g.nlay;
                const int c = L.cell(g);
                unsafeAtomicAdd(S.cf + ((size_t)L.o() * 2 + (L.birth() ? 0 : 1)) * ncell + c, sc);
            }
            if (S.img) {  // image: the event point on the observer's sky plane
                const double* eh = A.img_axes + 6 * L.o();
                const double u = L.sx() * eh[0] + L.sy() * eh[1] + L.sz() * eh[2];
                const double v = L.sx() * eh[3] + L.sy() * eh[4] + L.sz() * eh[5];
                const int col = pixel_of(u, A.img_half, A.npix), row = pixel_of(v, A.img_half, A.npix);
                unsafeAtomicAdd(S.img + ((size_t)L.o() * A.npix + row) * A.npix + col, sc);
            }
        }
        L.o() += 1;
        if (L.o() < A.n_out) return A_PEEL;
        if (L.birth()) {
            L.birth() = 0;
            if (!A.scattering) {
                L.ev = K_ESC;
                return A_FINISH;
            }
            L.e() = 1;
            return A_FLIGHT;
        }
        return A_SCATTER;
    }
    if (L.ev == E_INTERACT) {
        L.nint() += 1;
        L.o() = 0;
        L.birth() = 0;
        if (EXT) L.surf() = 0;
        return A_PEEL;
    }
    if (EXT && L.ev == E_SURFACE && A.surface_albedo > 0.0) {
        // the floor reflects: an event on the surface of the lowest cell,
        // entered through its inner face; until the reflection the packet
        // direction holds the floor's outward normal (radial on a sphere, +z
        // in a slab)
        L.nint() += 1;
        const double x = L.w.px + L.w.t * L.w.dx, y = L.w.py + L.w.t * L.w.dy;
        const double z = g.geom == 1 ? g.r[0] : L.w.pz + L.w.t * L.w.dz;
        L.sx() = x;
        L.sy() = y;
        L.sz() = z;
        if (g.geom == 1) {
            L.sdx() = 0.0;
            L.sdy() = 0.0;
            L.sdz() = 1.0;
        } else {
            const double rr = sqrt(x * x + y * y + z * z);
            L.sdx() = x / rr;
            L.sdy() = y / rr;
            L.sdz() = z / rr;
        }
        L.set_cell(L.w.i, L.w.j, 0);
        L.o() = 0;
        L.birth() = 0;
        L.surf() = 1;
        return A_PEEL;
    }
    if (L.ev == E_LOST) L.nlost() += 1;
    L.ev = L.ev == E_ESCAPE ? K_ESC : (L.ev == E_SURFACE ? K_SURF : K_LOST);
    return A_FINISH;
}

// K4a: births of every packet of a batch (albedo: uniform on the top disk or
// the slab's incidence; emission: cell from the biased CDF, uniform position in
// its volume, isotropic direction, weight (L_i/L_tot)/q_i), one thread each.
//
// blk_sv >= 0: the solve every packet of the calling block belongs to (found
// once per block); tab: when that solve is an emission solve with a fixed g,
// 256 samples of its CDF, tab[m] = cdf[(m ncell) >> 8], which narrow the
// search for the birth cell to the range between two samples (same cell as
// the search over the whole CDF: see below).
template <bool MULTI>
__device__ __forceinline__ void birth_record(const GridDev& g1, const BatchArgs& A, unsigned long long gid, double* b,
                                             int blk_sv, const double* tab)
{
    int sv = blk_sv >= 0 ? blk_sv : solve_of(A, gid);
    const GridDev& g = MULTI ? A.grids[A.solves[sv].grid] : g1;
    const double r_toa = g.r[g.nlay];
    const unsigned long long q = gid - A.solves[sv].pbase;
    const uint32_t tag = A.solves[sv].tag;
    double wmul = 1.0;
    if (A.solves[sv].gs_n > 0) {
        // per-packet g-ordinate: p(g) = w_g (albedo) or w_g L_g / sum(w L)
        // (emission); sampled from q(g) (1: p, 2: uniform, 3: (p + 1/N_g)/2)
        // with the smallest g whose cumulative weight exceeds u times the total
        const SolveDev& H = A.solves[sv];
        const int ng = H.gs_n, scheme = H.gs_scheme;
        double ptot = 0.0;
        for (int h = 0; h < ng; ++h) ptot += H.ltot ? H.gs_w[h] * *A.solves[sv + h].ltot : H.gs_w[h];
        if (!(ptot > 0.0)) {  // nothing emits in any g-ordinate
            b[B_W] = 0.0;
            b[B_CELL] = -1.0;
            b[B_SOLVE] = (double)sv;
            return;
        }
        double qtot = 0.0;
        for (int h = 0; h < ng; ++h) {
            const double raw = H.ltot ? H.gs_w[h] * *A.solves[sv + h].ltot : H.gs_w[h];
            qtot += scheme == 1 ? raw : (scheme == 2 ? 1.0 : 0.5 * (raw / ptot) + 0.5 / ng);
        }
        const double target = draw(A.seed, tag, q, 0, 3).a * qtot;
        double cum = 0.0;
        int gi = ng - 1;
        double pg = 0.0, qg = 0.0;
        for (int h = 0; h < ng; ++h) {
            const double raw = H.ltot ? H.gs_w[h] * *A.solves[sv + h].ltot : H.gs_w[h];
            const double qh = scheme == 1 ? raw : (scheme == 2 ? 1.0 : 0.5 * (raw / ptot) + 0.5 / ng);
            cum += qh;
            if (cum > target) {
                gi = h;
                pg = raw / ptot;
                qg = qh;
                break;
            }
            if (h == ng - 1) {
                pg = raw / ptot;
                qg = qh;
            }
        }
        wmul = scheme == 1 ? 1.0 : (scheme == 2 ? pg * ng : pg / qg);
        sv += gi;
    }
    const SolveDev& S = A.solves[sv];
    b[B_SOLVE] = (double)sv;
    if (S.mode == 0) {
        U2 u = draw(A.seed, tag, q, 0, 0);
        if (g.geom == 1) {
            double mu0 = A.mu0 > 0.0 ? A.mu0 : sqrt(1.0 - u.a);
            b[B_X] = 0.0; b[B_Y] = 0.0; b[B_Z] = g.r[g.nlay];
            b[B_DX] = sqrt(fmax(1.0 - mu0 * mu0, 0.0)); b[B_DY] = 0.0; b[B_DZ] = -mu0;
            b[B_CELL] = (double)pack_ijk(0, 0, g.nlay - 1);
        } else {
            double rho = r_toa * sqrt(u.a);
            double a = 2.0 * kPi * u.b;
            double y = rho * cos(a), z = rho * sin(a);
            double x = sqrt(fmax(r_toa * r_toa - y * y - z * z, 0.0));
            int i, j;
            locate_column(g, x, y, z, i, j);
            b[B_X] = x; b[B_Y] = y; b[B_Z] = z;
            b[B_DX] = -1.0; b[B_DY] = 0.0; b[B_DZ] = 0.0;
            b[B_CELL] = (double)pack_ijk(i, j, g.nlay - 1);
        }
        b[B_W] = wmul;
        return;
    }
    if (S.mode == 2) {
        // transmission: a random point of the annulus R0 <= bi <= R_TOA, the
        // stellar beam along -x, weight bi times the limb-darkening fraction
        U2 u = draw(A.seed, tag, q, 0, 0);
        const double r0 = g.r[0];
        const double bi = r0 + u.a * (r_toa - r0);
        const double al = 2.0 * kPi * u.b;
        const double x = sqrt(fmax(r_toa * r_toa - bi * bi, 0.0)), y = bi * cos(al), z = bi * sin(al);
        int i, j;
        locate_column(g, x, y, z, i, j);
        b[B_X] = x; b[B_Y] = y; b[B_Z] = z;
        b[B_DX] = -1.0; b[B_DY] = 0.0; b[B_DZ] = 0.0;
        b[B_CELL] = (double)pack_ijk(i, j, g.nlay - 1);
        b[B_W] = bi * limb_weight(A.ld, y, z) * wmul;
        return;
    }
    const int ncell = g.nlon * g.nlat * g.nlay;
    const double tot = S.cdf[ncell - 1];
    if (!(tot > 0.0)) {  // nothing emits
        b[B_W] = 0.0;
        b[B_CELL] = -1.0;
        return;
    }
    U2 u0 = draw(A.seed, tag, q, 0, 0);
    U2 u1 = draw(A.seed, tag, q, 0, 1);
    U2 u2 = draw(A.seed, tag, q, 0, 2);
    double target = u0.a * tot;
    int lo = 0, hi = ncell - 1;  // smallest c with cdf[c] > target (else ncell - 1)
    if (tab != nullptr && sv == blk_sv) {
        // m = the first sample above target; the cell lies after sample m - 1
        // (every cdf value up to it is <= target) and at or before sample m
        // (its value is > target); past the last sample, up to ncell - 1
        int a = 0, z = 256;
        while (a < z) {
            const int mid = (a + z) >> 1;
            if (tab[mid] > target) z = mid;
            else a = mid + 1;
        }
        lo = a == 0 ? 0 : (int)(((unsigned long long)(a - 1) * (unsigned)ncell) >> 8) + 1;
        hi = a == 256 ? ncell - 1 : (int)(((unsigned long long)a * (unsigned)ncell) >> 8);
    }
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (S.cdf[mid] > target) hi = mid;
        else lo = mid + 1;
    }
    int c = lo < ncell ? lo : ncell - 1;
    int i = c % g.nlon, j = (c / g.nlon) % g.nlat, k = c / (g.nlon * g.nlat);
    double rk = g.r[k], rk1 = g.r[k + 1];
    double rk3 = rk * rk * rk;
    double rk13 = rk1 * rk1 * rk1;
    double r = cbrt(rk3 + u0.b * (rk13 - rk3));
    double sl0 = g.lat_sin[j], sl1 = g.lat_sin[j + 1];
    double sl = sl0 + u1.a * (sl1 - sl0);
    double cl = sqrt(fmax(1.0 - sl * sl, 0.0));
    double lon = g.lon[i] + u1.b * (g.lon[i + 1] - g.lon[i]);
    b[B_X] = r * cl * cos(lon);
    b[B_Y] = r * cl * sin(lon);
    b[B_Z] = r * sl;
    double mu = 2.0 * u2.a - 1.0;
    double sp = sqrt(fmax(1.0 - mu * mu, 0.0));
    double psi = 2.0 * kPi * u2.b;
    b[B_DX] = sp * cos(psi);
    b[B_DY] = sp * sin(psi);
    b[B_DZ] = mu;
    b[B_W] = S.wbirth[c] * wmul;
    b[B_CELL] = (double)pack_ijk(i, j, k);
}

// The records of a block's packets are built in LDS and its rows written
// as one contiguous range (peel-off columns as zeros): coalesced stores of
// whole lines instead of 72 B pieces of 120 B rows.  Dynamic LDS: 256 CDF
// samples, then 256 rows of row_w doubles (row_w = n_obs + kNCounters <= 19,
// sized at launch, so a narrow row leaves room for more resident blocks).
template <bool MULTI>
__global__ void __launch_bounds__(256) k_births(GridDev g1, BatchArgs A)
{
    extern __shared__ double births_lds[];
    double* tab = births_lds;
    double* sh = births_lds + 256;
    __shared__ int blk[2];  // the block's solve (-1: several), and whether tab holds its CDF samples
    const int w = A.row_w;
    const unsigned long long r0 = (unsigned long long)blockIdx.x * 256;
    const unsigned long long left = A.total - r0;
    if (threadIdx.x == 0) {
        const int sv = solve_of(A, r0);
        const SolveDev& S = A.solves[sv];
        const unsigned long long last = r0 + (left < 256 ? left : 256) - 1;
        const bool one = r0 >= S.begin && last < S.begin + S.n;
        blk[0] = one ? sv : -1;
        blk[1] = one && S.mode == 1 && S.gs_n == 0;
    }
    __syncthreads();
    const int blk_sv = blk[0];
    const bool use_tab = blk[1] != 0;
    if (use_tab) {
        const SolveDev& S = A.solves[blk_sv];
        const GridDev& g = MULTI ? A.grids[S.grid] : g1;
        const unsigned ncell = (unsigned)(g.nlon * g.nlat * g.nlay);
        tab[threadIdx.x] = S.cdf[((unsigned long long)threadIdx.x * ncell) >> 8];
    }
    double* mine = sh + threadIdx.x * w;
    for (int c = 0; c < w; ++c) mine[c] = 0.0;
    __syncthreads();
    const unsigned long long gid = r0 + threadIdx.x;
    if (gid < A.total) birth_record<MULTI>(g1, A, gid, mine + A.n_out, blk_sv, use_tab ? tab : nullptr);
    __syncthreads();
    const int n = (int)(left < 256 ? left : 256) * w;
    double* dst = A.rows + r0 * (unsigned long long)w;
    for (int x = threadIdx.x; x < n; x += 256) dst[x] = sh[x];
    if (A.head && gid < A.total) {
        A.head[gid] = kNoRecord;
        A.peel_cross[gid] = 0u;
    }
}

// New packet L.gid: load its birth record and return the first action (a
// flight for albedo, the emission-point peel-off, or finish if none emits).
template <bool EXT>
__device__ __forceinline__ int birth(Lane& L, const BatchArgs& A)
{
    const double* b = A.rows + L.gid() * (unsigned long long)A.row_w + A.n_out;
    if (EXT) {
        double* bw = A.rows + L.gid() * (unsigned long long)A.row_w + A.n_out;
        if (A.surface_albedo > 0.0 || A.forced) bw[B_SURF] = 0.0;
        if (A.forced) bw[B_FESC] = 0.0;
    }
    const int sv = (int)b[B_SOLVE];
    const SolveDev& S = A.solves[sv];
    L.C->st[L.t] = 0u;
    L.set_solve(sv);
    L.smode() = S.mode == 1;  // the emission observer set; albedo and transmission use the other
    for (int o = 0; o < A.n_out; ++o) L.Fo(o) = 0.0;
    L.w_abs = 0.0;
    L.w_rr() = 0.0;
    L.ncross = 0;
    L.nint() = 0;
    L.e() = 1;
    const double cw = b[B_CELL];
    L.W = b[B_W];
    L.W0() = L.W;
    if (cw < 0.0) {
        L.ev = -1;
        return A_FINISH;
    }
    L.C->ijk[L.t] = (uint32_t)cw;
    L.sx() = b[B_X]; L.sy() = b[B_Y]; L.sz() = b[B_Z];
    L.sdx() = b[B_DX]; L.sdy() = b[B_DY]; L.sdz() = b[B_DZ];
    if (S.mode == 0) return A_FLIGHT;
    L.birth() = 1;
    return A_PEEL;
}

// Registers: 101 VGPRs (mixed) or 119 (FP64; on several grids 103 and 121), the
// extended forms 116 to 125, none spilled, so four blocks of four waves are
// resident per CU.
template <bool MIXED, bool MULTI, bool EXT>
__global__ void __launch_bounds__(kTPB, 4) k_transport_persistent(GridDev g1, BatchArgs A)
{
    __shared__ double sobs[2 * 3 * kMaxObs];
    __shared__ ColdLDS cold;
    extern __shared__ double Fsh[];  // [n_out][kTPB]
    if (threadIdx.x < 2 * 3 * kMaxObs) sobs[threadIdx.x] = A.obs[threadIdx.x / (3 * kMaxObs)][threadIdx.x % (3 * kMaxObs)];
    __syncthreads();
    int lgrid = 0;  // grid of the lane's packet (multi-grid launches)
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    unsigned long long res_next = 0, res_end = 0;
    bool exhausted = false, own = true;
    Lane L;
    L.C = &cold;
    L.F = Fsh;
    L.t = threadIdx.x;
    L.mode = M_DEAD;
    cold.st[threadIdx.x] = 0u;
    const void* aext = nullptr;
    const void* aabs = nullptr;
    Prop<MIXED> ae = 0;  // the extinction of the walk's cell
    for (;;) {
        const GridDev& g = MULTI ? A.grids[lgrid] : g1;
        if (L.mode <= M_PROBE && g.eq_edge > 0 && L.w.eq != 0) wk_row_roots<MIXED>(g, L.w);
        if (L.mode <= M_PROBE) walk_step<MIXED, EXT, GEO_ANY, true>(L, g, aext, aabs, ae, A);
        unsigned long long evm = __ballot(L.mode == M_EVENT);
        unsigned long long walking = __ballot(L.mode <= M_PROBE);
        if (__popcll(evm) < A.ev_threshold && walking != 0) continue;
        int act = A_NONE;
        if (L.mode == M_EVENT) act = handle_event<MIXED, EXT>(L, g, A);
        if (act == A_SCATTER) {
            const SolveDev& S = A.solves[L.solve()];
            const int c = L.cell(g);
            act = scatter<MIXED, EXT>(L, A, S, ld<MIXED>(S.omega, c), ld<MIXED>(S.p_gas, c), ld<MIXED>(S.g_cld, c));
        }
        for (int pass = 0; pass < 2; ++pass) {
            if (act == A_FINISH) {
                finish_packet<EXT>(L, A, L.ev);
                act = A_NONE;
            }
            if (pass == 1) break;
            // regeneration: dead lanes take the next packets of the reservoir
            unsigned long long dead = __ballot(L.mode == M_DEAD);
            while (dead != 0) {
                if (res_next >= res_end) {
                    if (exhausted || !refill(A, lane, own, res_next, res_end)) {
                        exhausted = true;
                        break;
                    }
                }
                unsigned long long avail = res_end - res_next;
                int cnt = __popcll(dead);
                int take = (unsigned long long)cnt < avail ? cnt : (int)avail;
                int rank = __popcll(dead & below);
                if (L.mode == M_DEAD && rank < take) {
                    L.gid() = res_next + (unsigned long long)rank;
                    L.mode = M_BIRTH;
                }
                res_next += (unsigned long long)take;
                dead = __ballot(L.mode == M_DEAD);
            }
            if (L.mode == M_DEAD && exhausted) L.mode = M_IDLE;
            if (L.mode == M_BIRTH) {
                if (MULTI) lgrid = A.solves[solve_of(A, L.gid())].grid;
                act = birth<EXT>(L, A);
                const SolveDev& S = A.solves[L.solve()];  // the solve the birth record chose
                aext = S.a_ext;
                aabs = S.a_abs;
            }
        }
        const GridDev& ga = MULTI ? A.grids[lgrid] : g1;
        if (act == A_FLIGHT || act == A_PEEL) {
            ae = (Prop<MIXED>)ld<MIXED>(aext, L.cell(ga));
            start_walk<MIXED, EXT>(L, ga, A, sobs, act == A_FLIGHT);
        }
        if (__ballot(L.mode != M_IDLE) == 0) break;
    }
}

// Fixed-order reduction of the packet rows of every solve: block (chunk, s)
// sums rows [chunk*kChunk, (chunk+1)*kChunk) of solve s into
// partials[s][chunk][2*n_out + kNCounters]; then one block per (s, column)
// sums the chunks.  Optional copy of F to a packet dump.
//
// Thread t of a chunk block owns column t % w of the rows t / w, t / w + R,
// ... (w the row width, R = 1024 / w rows per pass), so each pass of the
// block reads R whole rows as one contiguous, coalesced range, four passes'
// loads in flight; the R per-thread sums of a column are then added by eight
// threads and theirs by one.  Latency-bound where solves are small: 40 solves of
// 40000 packets 104 us with 256 threads and one load at a time, 40 here; 16
// of 1000 21 and 10.
constexpr int kChunk = 4096;
constexpr int kRT = 256, kPT = 1024, kPJ = 8;

__global__ void __launch_bounds__(kPT) k_rows_partial(BatchArgs A, double* __restrict__ partials, int chunks,
                                                      double* __restrict__ dump)
{
    __shared__ double sh[2 * kPT];
    const int s = blockIdx.y;
    const SolveDev& S = A.solves[s];
    const unsigned long long begin = S.begin, n = S.n;
    const int w = A.row_w;  // n_out peel-off sums + the counters
    const int R = kPT / w;
    const int t = threadIdx.x;
    const int c = t % w, r0 = t / w;
    const unsigned long long q0 = (unsigned long long)blockIdx.x * kChunk;
    const unsigned long long qe = q0 + kChunk < n ? q0 + kChunk : n;
    const double* rows = A.rows + begin * (unsigned long long)w + c;
    // the rows of a split launch hold F itself also for transmission, and the
    // crossings of the flights only
    const bool more = A.head && c == A.n_out + K_NCROSS, from_w0 = A.head && A.trans_ms && c < A.n_out;
    double acc = 0.0, acc2 = 0.0;
    if (r0 < R) {
        for (unsigned long long q = q0 + r0; q < qe; q += 4 * R) {
            double v[4], x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned long long p = q + (unsigned)(u * R) < qe ? q + (unsigned)(u * R) : q;
                v[u] = rows[p * (unsigned long long)w];
                x[u] = 0.0;
                if (more) x[u] = (double)A.peel_cross[begin + p];
                if (from_w0) x[u] = rows[p * (unsigned long long)w + A.n_out + K_W0 - c];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned long long p = q + (unsigned)(u * R);
                if (p >= qe) break;
                const double y = more ? v[u] + x[u] : (from_w0 ? x[u] - v[u] : v[u]);
                acc = acc + y;
                acc2 = acc2 + y * y;
                if (dump && c < A.n_out) dump[(begin + p) * (unsigned long long)A.n_out + c] = y;
            }
        }
    }
    sh[t] = acc;
    sh[kPT + t] = acc2;
    __syncthreads();
    double tot = 0.0, tot2 = 0.0;
    if (r0 < kPJ) {
        for (int j = r0; j < R; j += kPJ) {
            tot = tot + sh[c + j * w];
            tot2 = tot2 + sh[kPT + c + j * w];
        }
    }
    __syncthreads();
    sh[t] = tot;
    sh[kPT + t] = tot2;
    __syncthreads();
    if (t < w) {
        for (int j = 1; j < kPJ; ++j) {
            tot = tot + sh[t + j * w];
            tot2 = tot2 + sh[kPT + t + j * w];
        }
        const int pw = 2 * A.n_out + kNCounters;
        double* out = partials + ((size_t)s * chunks + blockIdx.x) * pw;
        if (t < A.n_out) {
            out[2 * t] = tot;
            out[2 * t + 1] = tot2;
        } else {
            out[2 * A.n_out + (t - A.n_out)] = tot;
        }
    }
}

__global__ void __launch_bounds__(kRT) k_rows_final(const double* __restrict__ partials, int chunks, int pw,
                                                    double* __restrict__ sums, int sums_w)
{
    __shared__ double sh[kRT];
    __shared__ double shc[kRT];
    const int s = blockIdx.y, col = blockIdx.x;
    double acc = 0.0, comp = 0.0;
    for (int c = threadIdx.x; c < chunks; c += kRT) {
        double x = partials[((size_t)s * chunks + c) * pw + col];
        double t = acc + x;
        comp = comp + (fabs(acc) >= fabs(x) ? ((acc - t) + x) : ((x - t) + acc));
        acc = t;
    }
    sh[threadIdx.x] = acc;
    shc[threadIdx.x] = comp;
    __syncthreads();
    for (int st = kRT / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) {
            double a = sh[threadIdx.x], b = sh[threadIdx.x + st];
            double t = a + b;
            double e = fabs(a) >= fabs(b) ? ((a - t) + b) : ((b - t) + a);
            sh[threadIdx.x] = t;
            shc[threadIdx.x] = shc[threadIdx.x] + shc[threadIdx.x + st] + e;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[(size_t)s * sums_w + col] = sh[0] + shc[0];
}

__global__ void k_fill_u64(unsigned long long* p, unsigned long long v)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

// Packet dispensers of a launch: counter x starts at the first packet of
// chunk x = [edge(x), edge(x + 1)), edge(x) = floor(total * x / kXcds).
__global__ void k_init_dispensers(unsigned long long* c, int stride, unsigned long long total)
{
    if (blockIdx.x == 0 && threadIdx.x < kXcds) c[threadIdx.x * stride] = chunk_edge(total, (int)threadIdx.x);
}

// Fill n doubles (a kernel, so that recorded graphs hold no memset nodes).
__global__ void __launch_bounds__(256) k_fill_f64(double* __restrict__ p, size_t n, double v)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = v;
}

}  // namespace

void launch_births(const GridDev& g, const BatchArgs& a, bool multi, hipStream_t stream)
{
    dim3 grid((unsigned)((a.total + 255) / 256));
    const size_t lds = (size_t)(256 + 256 * a.row_w) * sizeof(double);  // <= 40 KB
    if (multi) hipLaunchKernelGGL(k_births<true>, grid, dim3(256), lds, stream, g, a);
    else hipLaunchKernelGGL(k_births<false>, grid, dim3(256), lds, stream, g, a);
}

void launch_transport_persistent(const GridDev& g, const BatchArgs& a, bool mixed, bool multi, int blocks,
                                 hipStream_t stream)
{
    if (a.slab) {
        launch_slab(g, a, mixed, blocks, stream);
        return;
    }
    // the extended form only when a launch uses one of its features
    const bool ext = a.surface_albedo > 0.0 || a.cloud_phase == 2 || a.forced != 0 || a.trans_ms != 0 ||
                     a.absorption == 1;
    const size_t lds = (size_t)a.n_out * kTPB * sizeof(double);
#define MCRT_K4(MX, MU)                                                                                              \
    if (ext) hipLaunchKernelGGL((k_transport_persistent<MX, MU, true>), dim3(blocks), dim3(kTPB), lds, stream, g, a); \
    else hipLaunchKernelGGL((k_transport_persistent<MX, MU, false>), dim3(blocks), dim3(kTPB), lds, stream, g, a);
    if (mixed && multi) { MCRT_K4(true, true) }
    else if (mixed) { MCRT_K4(true, false) }
    else if (multi) { MCRT_K4(false, true) }
    else { MCRT_K4(false, false) }
#undef MCRT_K4
}

int reduce_rows_chunks(unsigned long long max_n) { return (int)((max_n + kChunk - 1) / kChunk); }

void launch_reduce_rows(const BatchArgs& a, int n_solves, double* partials, int chunks, double* sums, int sums_w,
                        double* dump, hipStream_t stream)
{
    const int pw = 2 * a.n_out + kNCounters;
    hipLaunchKernelGGL(k_rows_partial, dim3(chunks, n_solves), dim3(kPT), 0, stream, a, partials, chunks, dump);
    hipLaunchKernelGGL(k_rows_final, dim3(pw, n_solves), dim3(kRT), 0, stream, partials, chunks, pw, sums, sums_w);
}

void launch_fill_u64(unsigned long long* p, unsigned long long v, hipStream_t stream)
{
    hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(64), 0, stream, p, v);
}

void launch_init_dispensers(unsigned long long* counters, int stride, unsigned long long total, hipStream_t stream)
{
    hipLaunchKernelGGL(k_init_dispensers, dim3(1), dim3(64), 0, stream, counters, stride, total);
}

void launch_fill_f64(double* p, size_t n, double v, hipStream_t stream)
{
    if (n == 0) return;
    const size_t blocks = std::min<size_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)blocks), dim3(256), 0, stream, p, n, v);
}

}  // namespace mcrt

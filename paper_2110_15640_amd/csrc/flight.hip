// K4 in two kernels: packet flights, and the peel-off rays of their events.
//
// One packet per lane, as in transport.hip, but an event only appends a record
// (point, direction, weight) and the packet flies on; the peel-off rays of all
// records, n_obs per event, are then walked by a second kernel, one ray per
// lane, and a third adds each packet's contributions to its row in the order
// of its events.  What this changes: a packet's chain of dependent walks holds
// its flights alone (a peel-off runs to the edge of the grid, tens of cells;
// in a thick medium a flight crosses a few), so the end of a launch, where a
// few packets with hundreds of events are left, and launches of few packets
// are an order shorter; and rays fill every lane all the time, since a lane
// whose ray ends takes the next of any packet.
//
// The records live in a fixed number of slots, one region per XCD, which waves
// take in chunks: counters that every wave of the device adds to are worth few
// additions (one per
// event pass and per 64 rays, in one cache line, made the 25 x 8 x 1e5 emission
// solve 0.39 s instead of 0.046).  A lane
// that finds them full parks its packet; the host then repeats the three
// kernels until no lane is parked.  A packet's contributions are added in the
// order of its events whatever the rounds, so results do not depend on them,
// and are bit for bit those of transport.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <math.h>
#include <stdint.h>

#include "transport_common.hpp"

namespace mcrt {
namespace {
using namespace dev;

// An event that peels off.  Written and read as 16-byte words.
template <bool MIXED>
struct alignas(16) EvRec {
    double x, y, z;      // event point (slab backscatter: x and y hold the observer's direction)
    double nx, ny, nz;   // packet direction before the event (floor: its normal)
    double w;            // weight: W omega, W A_s of a floor event, W of a birth
    Prop<MIXED> pg, gc;  // gas probability and asymmetry of the cell
    uint32_t ijk;        // cell: i | j << 11 | k << 21
    uint32_t so;         // solve | kind << 20 | observer set << 22
};
enum { R_SCATTER = 0, R_BIRTH = 1, R_FLOOR = 2, R_NONE = 3 };  // R_NONE: a slot left empty

constexpr int E_PENDING = 5;  // a resumed packet whose event has no record yet
constexpr int M_PARKED = 7;
constexpr int A_RECORD = 5;

struct FlightLDS {
    double W0[kTPB], w_rr[kTPB];
    uint32_t gid[kTPB];
    uint32_t ijk[kTPB];   // event cell: i | j << 11 | k << 21
    uint32_t st[kTPB];    // forced state:4 | birth:1 | smode:1 | 3 unused | capped:1 | lost:1 | surface:1 | solve:20
    uint32_t e[kTPB];
    uint32_t last[kTPB];  // the packet's last record since the kernels were last launched
    int nint[kTPB];
};

struct FLane {
    Walker w;  // the flight; its origin and direction are the packet's
    double tau;
    double W, w_abs;
    int ncw;
    int ncross;
    int mode, ev;
    FlightLDS* C;
    int t;
    __device__ double& sx() { return w.px; }
    __device__ double& sy() { return w.py; }
    __device__ double& sz() { return w.pz; }
    __device__ double& sdx() { return w.dx; }
    __device__ double& sdy() { return w.dy; }
    __device__ double& sdz() { return w.dz; }
    __device__ double& W0() { return C->W0[t]; }
    __device__ double& w_rr() { return C->w_rr[t]; }
    __device__ unsigned long long gid() { return C->gid[t]; }
    __device__ uint32_t& e() { return C->e[t]; }
    __device__ int& nint() { return C->nint[t]; }
    __device__ Bits o() { return Bits{&C->st[t], 0, 0xFu}; }
    __device__ Bits birth() { return Bits{&C->st[t], 4, 0x1u}; }
    __device__ Bits smode() { return Bits{&C->st[t], 5, 0x1u}; }
    __device__ Bits ncapped() { return Bits{&C->st[t], 9, 0x1u}; }
    __device__ Bits nlost() { return Bits{&C->st[t], 10, 0x1u}; }
    __device__ Bits surf() { return Bits{&C->st[t], 11, 0x1u}; }
    __device__ int solve() { return (int)(C->st[t] >> 12); }
    __device__ void set_solve(int s) { Bits{&C->st[t], 12, 0xFFFFFu} = s; }
    __device__ int si() { return (int)(C->ijk[t] & 0x7FFu); }
    __device__ int sj() { return (int)((C->ijk[t] >> 11) & 0x3FFu); }
    __device__ int sk() { return (int)(C->ijk[t] >> 21); }
    __device__ void set_cell(int i, int j, int k) { C->ijk[t] = (uint32_t)i | ((uint32_t)j << 11) | ((uint32_t)k << 21); }
    __device__ int cell(const GridDev& g) { return (sk() * g.nlat + sj()) * g.nlon + si(); }
};

// New packet: its birth record, as in transport.hip; returns the first action.
template <bool EXT>
__device__ __forceinline__ int birth(FLane& L, const BatchArgs& A)
{
    double* b = A.rows + L.gid() * (unsigned long long)A.row_w + A.n_out;
    if (EXT) {
        if (A.surface_albedo > 0.0 || A.forced) b[B_SURF] = 0.0;
        if (A.forced) b[B_FESC] = 0.0;
    }
    const int sv = (int)b[B_SOLVE];
    L.C->st[L.t] = 0u;
    L.set_solve(sv);
    const int smode = A.solves[sv].mode;
    L.smode() = smode == 1;
    L.w_abs = 0.0;
    L.w_rr() = 0.0;
    L.ncross = 0;
    L.nint() = 0;
    L.e() = 1;
    L.C->last[L.t] = kNoRecord;
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
    if (smode == 0) return A_FLIGHT;
    L.birth() = 1;
    return A_RECORD;
}

// Bookkeeping of a flight's end; returns the action that follows (L.ev: the
// counter that receives the final weight when that is A_FINISH).
template <bool EXT>
__device__ __forceinline__ int flight_event(FLane& L, const GridDev& g, const BatchArgs& A)
{
    if (EXT && L.ev == E_PEEL_DONE) {
        // a forced interaction's probe: with the path's optical depth tp
        // known, the flight's tau comes from a density on [0, tp], the weight
        // takes the factor e^{-tau}/q(tau) and the unscattered fraction
        // W e^{-tp} is booked where the path ends
        const SolveDev& S = A.solves[L.solve()];
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
    if (L.ev == E_PENDING) return A_RECORD;
    if (L.ev == E_INTERACT) {
        L.nint() += 1;
        if (EXT) L.surf() = 0;
        return A_RECORD;
    }
    if (EXT && L.ev == E_SURFACE && A.surface_albedo > 0.0) {
        // the floor reflects: an event on the surface of the lowest cell; the
        // packet direction holds the floor's outward normal until then
        L.nint() += 1;
        const double x = L.w.px + L.w.t * L.w.dx, y = L.w.py + L.w.t * L.w.dy;
        const double z = g.geom == 1 ? g.r[0] : L.w.pz + L.w.t * L.w.dz;
        L.set_cell(L.w.i, L.w.j, 0);
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
        L.surf() = 1;
        return A_RECORD;
    }
    if (L.ev == E_LOST) L.nlost() += 1;
    L.ev = L.ev == E_ESCAPE ? K_ESC : (L.ev == E_SURFACE ? K_SURF : K_LOST);
    return A_FINISH;
}

// The packet's next flight (its optical depth from the event's block 0, slot
// a, unless a forced interaction chose it) or the probe before a forced one.
template <bool MIXED, bool EXT, int GEO>
__device__ __forceinline__ void start_flight(FLane& L, const GridDev& g, const BatchArgs& A)
{
    int kind = M_FLIGHT;
    bool drawn = false;
    if constexpr (EXT) {
        drawn = A.forced != 0 && L.o() == kTauSet;
        if (A.forced != 0 && !drawn && (A.forced_first == 0 || L.e() == 1)) kind = M_PROBE;
        if (A.forced != 0) L.o() = kind == M_PROBE ? kProbeDone : 0;
    }
    if (kind == M_PROBE) {
        L.tau = 0.0;
    } else if (!drawn) {
        const SolveDev& S = A.solves[L.solve()];
        L.tau = -log(draw(A.seed, S.tag, L.gid() - S.pbase, L.e(), 0).a);
    }
    wk_start<MIXED, GEO>(g, L.w, L.w.px, L.w.py, L.w.pz, L.w.dx, L.w.dy, L.w.dz, L.si(), L.sj(), L.sk());
    L.ncw = 0;
    L.mode = kind;
}

// LF (here and for the rays): the face table of the launch's one grid lies in LDS
// (up to kLdsFaces entries), so that a step waits for no load but the last one's
// extinction.
constexpr int kLdsFaces = 1024;
template <bool LF>
__device__ __forceinline__ GridDev lds_grid(const GridDev& g1, double2* faces)
{
    GridDev g = g1;
    if constexpr (LF) {
        for (int e = threadIdx.x; e <= g1.lon_base + g1.nlon; e += kTPB) faces[e] = g1.faces[e];
        __syncthreads();
        g.faces = faces;
    }
    return g;
}

template <bool MIXED, bool MULTI, bool EXT, int GEO, bool LF>
__global__ void __launch_bounds__(kTPB, 4) k_flight(GridDev g0, BatchArgs A, PeelArgs Q)
{
    __shared__ FlightLDS cold;
    extern __shared__ double2 faces[];
    const GridDev g1 = lds_grid<LF>(g0, faces);
    int lgrid = 0;
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    unsigned long long res_next = 0, res_end = 0;
    bool exhausted = false, own = true;
    uint32_t rec_next = 0, rec_end = 0;  // the wave's chunk of records
    bool full = false, rec_own = true;   // no region has a chunk left; its own has
    FLane L;
    L.C = &cold;
    L.t = threadIdx.x;
    L.mode = lane < A.lanes ? M_DEAD : M_IDLE;
    cold.st[threadIdx.x] = 0u;
    const void* aext = nullptr;
    const void* aabs = nullptr;
    Prop<MIXED> ae = 0;
    const int slot = blockIdx.x * kTPB + threadIdx.x;
    if (Q.resume) {  // the packets the wave had taken but not started
        res_next = Q.park_u[7 * (size_t)Q.n_lanes + slot - lane];
        res_end = Q.park_u[8 * (size_t)Q.n_lanes + slot - lane];
    }
    if (Q.resume && Q.park_u[slot] != 0u) {
        const double* d = Q.park_d + slot;
        const uint32_t* u = Q.park_u + slot;
        const size_t n = (size_t)Q.n_lanes;
        L.sx() = d[0]; L.sy() = d[n]; L.sz() = d[2 * n];
        L.sdx() = d[3 * n]; L.sdy() = d[4 * n]; L.sdz() = d[5 * n];
        L.W = d[6 * n]; L.w_abs = d[7 * n]; L.W0() = d[8 * n]; L.w_rr() = d[9 * n];
        cold.gid[L.t] = u[n]; cold.ijk[L.t] = u[2 * n]; cold.st[L.t] = u[3 * n]; cold.e[L.t] = u[4 * n];
        L.nint() = (int)u[5 * n]; L.ncross = (int)u[6 * n];
        cold.last[L.t] = kNoRecord;
        L.mode = M_EVENT;
        L.ev = E_PENDING;
        const SolveDev& S = A.solves[L.solve()];
        aext = S.a_ext;
        aabs = S.a_abs;
        if (MULTI) lgrid = S.grid;
    }
    for (;;) {
        on_grid<MULTI>(g1, A.grids, lgrid, L.mode <= M_PROBE, [&](const GridDev& g) {
            if (GEO != GEO_SLAB && L.mode <= M_PROBE && g.eq_edge > 0 && L.w.eq != 0) wk_row_roots<MIXED>(g, L.w);
            if (L.mode <= M_PROBE) walk_step<MIXED, EXT, GEO, false>(L, g, aext, aabs, ae, A);
        });
        const GridDev& g = MULTI ? A.grids[lgrid] : g1;
        const unsigned long long walking = __ballot(L.mode <= M_PROBE);
        const unsigned long long waits = __ballot(L.mode == M_EVENT || (L.mode == M_DEAD && !exhausted));
        // ev_threshold of 64 lanes, in proportion where fewer carry packets
        if (64 * __popcll(waits) < A.ev_threshold * __popcll(waits | walking) && walking != 0) continue;
        int act = A_NONE;
        if (L.mode == M_EVENT) act = flight_event<EXT>(L, g, A);
        if (act == A_FINISH) {
            finish_counters<EXT>(L, A, L.ev);
            act = A_NONE;
        }
        // dead lanes take the next packets
        unsigned long long dead = __ballot(L.mode == M_DEAD);
        while (dead != 0) {
            if (res_next >= res_end) {
                if (exhausted || !refill(A, lane, own, res_next, res_end)) {
                    exhausted = true;
                    break;
                }
            }
            const unsigned long long avail = res_end - res_next;
            const int cnt = __popcll(dead);
            const int take = (unsigned long long)cnt < avail ? cnt : (int)avail;
            const int rank = __popcll(dead & below);
            if (L.mode == M_DEAD && rank < take) {
                cold.gid[L.t] = (uint32_t)(res_next + (unsigned long long)rank);
                L.mode = M_BIRTH;
            }
            res_next += (unsigned long long)take;
            dead = __ballot(L.mode == M_DEAD);
        }
        if (L.mode == M_DEAD && exhausted) L.mode = M_IDLE;
        if (L.mode == M_BIRTH) {
            act = birth<EXT>(L, A);
            const SolveDev& S = A.solves[L.solve()];
            aext = S.a_ext;
            aabs = S.a_abs;
            if (MULTI) lgrid = S.grid;
        }
        const GridDev& ga = MULTI ? A.grids[lgrid] : g1;
        // records: the wave's events take consecutive slots of a region that has room
        const unsigned long long want = __ballot(act == A_RECORD);
        if (want != 0) {
            const uint32_t n = (uint32_t)__popcll(want), rank = (uint32_t)__popcll(want & below);
            uint32_t r = kNoRecord;
            for (uint32_t given = 0; given < n;) {
                if (rec_next == rec_end) {
                    uint32_t base = kNoRecord, at;
                    const int x = full ? -1 : take_share(Q.ctl, kCtrStride, Q.cap, Q.chunk, lane, rec_own, at);
                    if (x >= 0) base = (uint32_t)x * Q.cap + at;
                    if (base == kNoRecord) {
                        full = true;
                        break;
                    }
                    rec_next = base;
                    rec_end = base + Q.chunk;
                }
                const uint32_t take = n - given < rec_end - rec_next ? n - given : rec_end - rec_next;
                if (act == A_RECORD && rank >= given && rank < given + take) r = rec_next + rank - given;
                rec_next += take;
                given += take;
            }
            if (act == A_RECORD) {
                if (r != kNoRecord) {
                    const SolveDev& S = A.solves[L.solve()];
                    const bool born = L.birth() != 0;
                    const bool floor = EXT && !born && L.surf();
                    double om = 1.0, pg = 0.0, gc = 0.0;
                    if (!born && !floor) {
                        const int c = L.cell(ga);
                        om = ld<MIXED>(S.omega, c);
                        pg = ld<MIXED>(S.p_gas, c);
                        gc = ld<MIXED>(S.g_cld, c);
                    }
                    EvRec<MIXED> v;
                    v.x = L.sx(); v.y = L.sy(); v.z = L.sz();
                    v.nx = L.sdx(); v.ny = L.sdy(); v.nz = L.sdz();
                    if (A.n_obs == 0) {  // slab backscatter: minus the incidence direction of the birth record
                        const double* b = A.rows + L.gid() * (unsigned long long)A.row_w + A.n_out;
                        v.x = -b[B_DX];
                        v.y = -b[B_DZ];
                    }
                    v.w = born ? L.W
                               : (floor ? L.W * A.surface_albedo : (EXT && A.absorption == 1 ? L.W : L.W * om));
                    v.pg = (Prop<MIXED>)pg;
                    v.gc = (Prop<MIXED>)gc;
                    v.ijk = cold.ijk[L.t];
                    v.so = (uint32_t)L.solve() | (uint32_t)(born ? R_BIRTH : (floor ? R_FLOOR : R_SCATTER)) << 20 |
                           (uint32_t)(int)L.smode() << 22;
                    ((EvRec<MIXED>*)Q.rec)[r] = v;
                    Q.next[r] = kNoRecord;
                    const uint32_t prev = cold.last[L.t];
                    if (prev == kNoRecord) A.head[cold.gid[L.t]] = r;
                    else Q.next[prev] = r;
                    cold.last[L.t] = r;
                    if (born) {
                        L.birth() = 0;
                        L.e() = 1;
                        L.ev = K_ESC;
                        act = A.scattering ? A_FLIGHT : A_FINISH;
                    } else {
                        act = scatter<MIXED, EXT>(L, A, S, om, pg, gc);
                    }
                } else {
                    act = A_NONE;
                    L.mode = M_PARKED;
                }
            }
        }
        if (act == A_FINISH) finish_counters<EXT>(L, A, L.ev);
        if (act == A_FLIGHT) {
            ae = (Prop<MIXED>)ld<MIXED>(aext, L.cell(ga));
            start_flight<MIXED, EXT, GEO>(L, ga, A);
        }
        if (__ballot(L.mode != M_IDLE && L.mode != M_PARKED) == 0) break;
    }
    for (uint32_t q = rec_next + lane; q < rec_end; q += 64) ((EvRec<MIXED>*)Q.rec)[q].so = (uint32_t)R_NONE << 20;
    const bool parked = L.mode == M_PARKED;
    double* d = Q.park_d + slot;
    uint32_t* u = Q.park_u + slot;
    const size_t n = (size_t)Q.n_lanes;
    u[0] = parked ? 1u : 0u;
    u[7 * n] = (uint32_t)res_next;
    u[8 * n] = (uint32_t)res_end;
    if (parked) {
        d[0] = L.sx(); d[n] = L.sy(); d[2 * n] = L.sz();
        d[3 * n] = L.sdx(); d[4 * n] = L.sdy(); d[5 * n] = L.sdz();
        d[6 * n] = L.W; d[7 * n] = L.w_abs; d[8 * n] = L.W0(); d[9 * n] = L.w_rr();
        u[n] = cold.gid[L.t]; u[2 * n] = cold.ijk[L.t]; u[3 * n] = cold.st[L.t]; u[4 * n] = cold.e[L.t];
        u[5 * n] = (uint32_t)L.nint(); u[6 * n] = (uint32_t)L.ncross;
    }
    const unsigned long long left = __ballot(parked);
    if (lane == 0 && left != 0) atomicAdd(Q.ctl + 2 * kXcds * kCtrStride, (uint32_t)__popcll(left));
}

// One peel-off ray per lane: ray q of region x is observer q % n_out of its
// record q / n_out, taken by waves of the region's XCD first (whose L2 holds the optics the region's flights used).
enum { P_IDLE = 0, P_WALK = 1, P_ANGLE = 2, P_DONE = 3 };
// Lanes without a ray that trigger the handing out of new ones: a start costs
// about two steps.  8: 50.5 ms, 16: 46.1, 24: 45.9, 32: 47.3 (25 x 8 x 1e5 emission packets, mixed)
constexpr int kPeelThreshold = 24, kAngleThreshold = 16, kShellSteps = 3;

template <bool MIXED, bool MULTI, int GEO, bool LF>
__global__ void __launch_bounds__(kTPB, MULTI ? 4 : 5) k_peel(GridDev g0, BatchArgs A, PeelArgs Q)
{
    __shared__ double sobs[2 * 3 * kMaxObs];
    extern __shared__ double2 faces[];
    if (threadIdx.x < 2 * 3 * kMaxObs) sobs[threadIdx.x] = A.obs[threadIdx.x / (3 * kMaxObs)][threadIdx.x % (3 * kMaxObs)];
    const GridDev g1 = lds_grid<LF>(g0, faces);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const EvRec<MIXED>* recs = (const EvRec<MIXED>*)Q.rec;
    const uint32_t n_out = (uint32_t)A.n_out;
    int state = P_IDLE, lgrid = 0, ncw = 0, kind = 0, solve = 0, cell = 0;
    Walker w;
    double tau = 0.0, wt = 0.0, q2 = 0.0;
    uint32_t fi = 0;  // the ray's place in Q.out
    Prop<MIXED> ae = 0;
    const void* aext = nullptr;
    uint32_t res_next = 0, res_end = 0, region = 0;  // the wave's rays
    bool more = true;                                // a region may have rays left
    uint32_t rays = 0;                               // lane x: those of region x
    if (lane < kXcds) {
        const uint32_t n = Q.ctl[lane * kCtrStride];
        rays = (n < Q.cap ? n : Q.cap) * n_out;
    }
    bool own = true;
    // an eighth of a wave's part of its XCD's rays at once
    uint32_t share = __shfl(rays, (int)(blockIdx.x % kXcds)) / (gridDim.x / kXcds * (kTPB / 64) * 8u + 1u) & ~63u;
    if (share < 64u) share = 64u;
    for (;;) {
        unsigned long long walking;
        on_grid<MULTI>(g1, A.grids, lgrid, state == P_WALK || state == P_ANGLE, [&](const GridDev& g) {
            const int ncol = g.nlat * g.nlon;
            // a ray ends at the top; beyond tau_peel_max, on the planet or after too
            // many cells nothing of it arrives
            auto through = [&](double t, double a, bool inside) {
                tau = wk_mad<MIXED>(a, t - w.t, tau);
                w.t = t;
                ncw++;
                const bool dark = tau > A.tau_peel_max;
                const bool end = !inside | dark | (ncw >= g.max_cross);
                if (end) {
                    if (dark | inside | (w.k < 0)) tau = INFINITY;
                    state = P_DONE;
                }
                return !end;
            };
#pragma unroll
            for (int m = 0; m < kShellSteps; ++m) {
                if (state != P_WALK) continue;
                if (GEO != GEO_SLAB && wk_min(w.tc, w.tp) < w.ts) {
                    state = P_ANGLE;
                } else {
                    const bool out = w.dk > 0;
                    w.k += w.dk;
                    cell += out ? ncol : -ncol;
                    const bool inside = (unsigned)w.k < (unsigned)g.nlay;
                    const double a = (double)ae;
                    const double R = wk_edge(g, inside ? w.k : 0, out);
                    ae = (Prop<MIXED>)ld<MIXED>(aext, inside ? cell : 0);
                    if (through(w.ts, a, inside)) {
                        if constexpr (GEO == GEO_SLAB) {
                            w.ts = wk_max(wk_div<MIXED>(R - w.pz, w.dz), w.t);
                        } else {
                            const double D = fma(R, R, -q2);
                            wk_ray_shell(w, D, wk_sqrt<MIXED>(D));
                        }
                    }
                }
            }
            walking = __ballot(state == P_WALK);
            if constexpr (GEO != GEO_SLAB) {
                const unsigned long long angle = __ballot(state == P_ANGLE);
                if (angle != 0 && (walking == 0 || __popcll(angle) >= (more ? kAngleThreshold : 1))) {
                    if (state == P_ANGLE) {
                        CrossKind x;
                        x.t = wk_min(w.tc, w.tp);
                        x.shell = x.none = false;
                        x.cone = w.tc <= x.t;
                        const double a = (double)ae, t0 = w.t;
                        const CrossIn in = wk_cross_begin<GEO>(g, w, x);
                        w.t = t0;
                        cell = wk_cell(g, w);
                        ae = (Prop<MIXED>)ld<MIXED>(aext, cell);
                        if (through(x.t, a, true)) {
                            wk_cross_end<MIXED, GEO>(g, w, x, in);
                            if (g.eq_edge > 0 && w.eq != 0) wk_row_roots<MIXED>(g, w);
                            state = P_WALK;
                        }
                    }
                    walking = __ballot(state == P_WALK);
                }
                walking |= __ballot(state == P_ANGLE);
            }
        });
        const GridDev& g = MULTI ? A.grids[lgrid] : g1;
        if (walking != 0 && ((!more && res_next >= res_end) || 64 - __popcll(walking) < kPeelThreshold)) continue;
        if (state == P_DONE) {
            state = P_IDLE;
            double f;
            if (MIXED) {
                const float att = tau < INFINITY ? __expf(-(float)tau) : 0.0f;
                if (kind == R_SCATTER) f = (double)((float)wt * att);
                else f = kind == R_BIRTH && !A.trans_ms ? wt * (double)att / (4.0 * kPi) : wt * (double)att;
            } else {
                const double att = exp(-tau);
                f = kind == R_BIRTH && !A.trans_ms ? wt * att / (4.0 * kPi) : wt * att;
            }
            // scattered light of a transmission packet: per steradian, over the
            // stellar beam's solid angle (peel_w = 1 otherwise)
            if (kind != R_BIRTH) f = f * A.peel_w;
            Q.out[fi].f = f;
            Q.out[fi].nx = (uint32_t)ncw;
            const SolveDev& S = A.solves[solve];
            if ((S.cf || S.img) && f > 0.0) {
                const uint32_t o = fi % n_out, ijk = recs[fi / n_out].ijk;
                const double sc = f * (S.cf_ltot ? S.cf_w * *S.cf_ltot : S.cf_w);
                if (S.cf) {  // contribution function: the event's cell, thermal or scattered part
                    const int ncell = g.nlon * g.nlat * g.nlay;
                    const int c = ((int)(ijk >> 21) * g.nlat + (int)((ijk >> 11) & 0x3FFu)) * g.nlon + (int)(ijk & 0x7FFu);
                    unsafeAtomicAdd(S.cf + ((size_t)o * 2 + (kind == R_BIRTH ? 0 : 1)) * ncell + c, sc);
                }
                if (S.img) {  // image: the event point on the observer's sky plane
                    const double* eh = A.img_axes + 6 * o;
                    const double u = w.px * eh[0] + w.py * eh[1] + w.pz * eh[2];
                    const double v = w.px * eh[3] + w.py * eh[4] + w.pz * eh[5];
                    const int col = pixel_of(u, A.img_half, A.npix), row = pixel_of(v, A.img_half, A.npix);
                    unsafeAtomicAdd(S.img + ((size_t)o * A.npix + row) * A.npix + col, sc);
                }
            }
        }
        // idle lanes take the next rays
        bool fresh = false;
        unsigned long long idle = __ballot(state == P_IDLE);
        while (idle != 0) {
            if (res_next >= res_end) {
                uint32_t at = 0;
                const int x = more ? take_share(Q.ctl + kXcds * kCtrStride, kCtrStride, rays, share, lane, own, at) : -1;
                if (x < 0) {
                    more = false;
                    break;
                }
                region = (uint32_t)x;
                const uint32_t lim = __shfl(rays, x);
                res_next = at;
                res_end = at + share < lim ? at + share : lim;
            }
            const uint32_t avail = res_end - res_next;
            const uint32_t cnt = (uint32_t)__popcll(idle);
            const uint32_t take = cnt < avail ? cnt : avail;
            const uint32_t rank = (uint32_t)__popcll(idle & below);
            if (state == P_IDLE && rank < take) {
                fi = region * Q.cap * n_out + res_next + rank;
                state = P_WALK;  // (unless the record is empty)
                fresh = true;
            }
            res_next += take;
            idle = __ballot(state == P_IDLE);
        }
        if (fresh) {
            const uint32_t r = fi / n_out, o = fi - r * n_out;
            const EvRec<MIXED> v = recs[r];
            kind = (int)((v.so >> 20) & 3u);
            if (kind == R_NONE) {
                state = P_IDLE;
            } else {
                solve = (int)(v.so & 0xFFFFFu);
                const SolveDev& S = A.solves[solve];
                aext = S.a_ext;
                if (MULTI) lgrid = S.grid;
                const GridDev& gs = MULTI ? A.grids[lgrid] : g1;
                double dx, dy, dz, px = v.x, py = v.y;
                if (A.n_obs == 0) {
                    dx = v.x;
                    dy = 0.0;
                    dz = v.y;
                    px = py = 0.0;
                } else {
                    const double* ob = sobs + ((v.so >> 22) & 1u) * (3 * kMaxObs) + 3 * o;
                    dx = ob[0];
                    dy = ob[1];
                    dz = ob[2];
                }
                const double mu = v.nx * dx + v.ny * dy + v.nz * dz;
                // a slab ray that never reaches the top, a floor ray below the horizon
                const bool dark = (GEO == GEO_SLAB && !(dz > 0.0)) || (kind == R_FLOOR && !(mu > 0.0));
                if (kind == R_BIRTH) wt = v.w;
                else if (kind == R_FLOOR) wt = mu > 0.0 ? v.w * (mu / kPi) : 0.0;
                else wt = peel_weight<MIXED>(A, v.w, mu, (double)v.pg, (double)v.gc);
                tau = 0.0;
                ncw = 0;
                const int i = (int)(v.ijk & 0x7FFu), j = (int)((v.ijk >> 11) & 0x3FFu), k = (int)(v.ijk >> 21);
                cell = (k * gs.nlat + j) * gs.nlon + i;
                ae = (Prop<MIXED>)ld<MIXED>(aext, cell);
                wk_start<MIXED, GEO>(gs, w, px, py, v.z, dx, dy, dz, i, j, k);
                q2 = wk_ray_q2(w);
                if (GEO != GEO_SLAB && gs.eq_edge > 0 && w.eq != 0) wk_row_roots<MIXED>(gs, w);
                if (dark) {
                    tau = INFINITY;
                    state = P_DONE;
                }
            }
        }
        if (__ballot(state != P_IDLE) == 0 && !more && res_next >= res_end) break;
    }
}

// Adds the contributions of each packet's records to its row, in the order of
// its events, and its rays' crossings to peel_cross.
__global__ void __launch_bounds__(256) k_peel_sum(BatchArgs A, PeelArgs Q)
{
    const unsigned long long q = (unsigned long long)blockIdx.x * 256 + threadIdx.x;
    if (q >= A.total) return;
    uint32_t r = A.head[q];
    if (r == kNoRecord) return;
    A.head[q] = kNoRecord;
    double* row = A.rows + q * (unsigned long long)A.row_w;
    double F[kMaxObs];
    uint32_t nx = 0;
#pragma unroll
    for (int o = 0; o < kMaxObs; ++o)
        if (o < A.n_out) F[o] = row[o];
    while (r != kNoRecord) {
        const PeelOut* out = Q.out + (size_t)r * A.n_out;
        PeelOut x[kMaxObs];
#pragma unroll
        for (int o = 0; o < kMaxObs; ++o)
            if (o < A.n_out) x[o] = out[o];
        r = Q.next[r];
#pragma unroll
        for (int o = 0; o < kMaxObs; ++o)
            if (o < A.n_out) {
                F[o] += x[o].f;
                nx += x[o].nx;
            }
    }
#pragma unroll
    for (int o = 0; o < kMaxObs; ++o)
        if (o < A.n_out) row[o] = F[o];
    A.peel_cross[q] += nx;
}

__global__ void k_peel_reset(PeelArgs Q)
{
    if (threadIdx.x <= 2 * kXcds) Q.ctl[threadIdx.x * kCtrStride] = 0u;
}

}  // namespace

size_t peel_record_bytes(bool mixed) { return mixed ? sizeof(EvRec<true>) : sizeof(EvRec<false>); }

void launch_peel_reset(const PeelArgs& q, hipStream_t stream)
{
    hipLaunchKernelGGL(k_peel_reset, dim3(1), dim3(64), 0, stream, q);
}

void launch_flight(const GridDev& g, const BatchArgs& a, const PeelArgs& q, bool mixed, bool multi, int blocks,
                   hipStream_t stream)
{
    const bool ext = a.surface_albedo > 0.0 || a.cloud_phase == 2 || a.forced != 0 || a.trans_ms != 0 ||
                     a.absorption == 1;
    // (slabs come without a grid table)
    const int geo = multi ? GEO_SPHERE : g.geom;
    const bool lf = !multi && g.lon_base + g.nlon < kLdsFaces;
    const size_t lds = lf ? sizeof(double2) * (g.lon_base + g.nlon + 1) : 0;
#define MCRT_K(MX, MU, EX, GE, LF) \
    hipLaunchKernelGGL((k_flight<MX, MU, EX, GE, LF>), dim3(blocks), dim3(kTPB), lds, stream, g, a, q)
#define MCRT_KX(MX, MU, GE, LF)                \
    do {                                       \
        if (ext) MCRT_K(MX, MU, true, GE, LF); \
        else MCRT_K(MX, MU, false, GE, LF);    \
    } while (0)
#define MCRT_KL(MX, GE)                       \
    do {                                      \
        if (lf) MCRT_KX(MX, false, GE, true); \
        else MCRT_KX(MX, false, GE, false);   \
    } while (0)
    if (geo == GEO_SLAB) {
        if (mixed) MCRT_KL(true, GEO_SLAB);
        else MCRT_KL(false, GEO_SLAB);
    } else if (multi) {
        if (mixed) MCRT_KX(true, true, GEO_SPHERE, false);
        else MCRT_KX(false, true, GEO_SPHERE, false);
    } else {
        if (mixed) MCRT_KL(true, GEO_SPHERE);
        else MCRT_KL(false, GEO_SPHERE);
    }
#undef MCRT_KL
#undef MCRT_KX
#undef MCRT_K
}

void launch_peel(const GridDev& g, const BatchArgs& a, const PeelArgs& q, bool mixed, bool multi, int blocks,
                 hipStream_t stream)
{
    const bool lf = !multi && g.lon_base + g.nlon < kLdsFaces;
    const size_t lds = lf ? sizeof(double2) * (g.lon_base + g.nlon + 1) : 0;
    const int geo = multi ? GEO_SPHERE : g.geom;
#define MCRT_K(MX, MU, GE, LF) hipLaunchKernelGGL((k_peel<MX, MU, GE, LF>), dim3(blocks), dim3(kTPB), lds, stream, g, a, q)
#define MCRT_KL(MX, GE)                      \
    do {                                     \
        if (lf) MCRT_K(MX, false, GE, true); \
        else MCRT_K(MX, false, GE, false);   \
    } while (0)
    if (geo == GEO_SLAB) {
        if (mixed) MCRT_KL(true, GEO_SLAB);
        else MCRT_KL(false, GEO_SLAB);
    } else if (multi) {
        if (mixed) MCRT_K(true, true, GEO_SPHERE, false);
        else MCRT_K(false, true, GEO_SPHERE, false);
    } else {
        if (mixed) MCRT_KL(true, GEO_SPHERE);
        else MCRT_KL(false, GEO_SPHERE);
    }
#undef MCRT_KL
#undef MCRT_K
}

void launch_peel_sum(const BatchArgs& a, const PeelArgs& q, hipStream_t stream)
{
    hipLaunchKernelGGL(k_peel_sum, dim3((unsigned)((a.total + 255) / 256)), dim3(256), 0, stream, a, q);
}

}  // namespace mcrt

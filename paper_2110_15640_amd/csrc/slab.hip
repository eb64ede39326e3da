// Scattered light of a plane-parallel slab, for gfx950 (CDNA4, wave64).
//
// In a slab the path of a packet needs no walk: with the optical depth from the
// top at every layer's edge tabulated, a flight of optical depth tau along mu
// leads from depth t to t - mu tau, whose layer a search finds, and the depth
// towards an observer is t / mu_o.  The layers in between are counted, not
// crossed.  One persistent kernel does whole packets, with no records and no
// rays, an event of all 64 lanes at a time.  A call of ten wavelengths x 1e5
// packets on 50 layers in FP64 takes 0.74 ms, this kernel 0.63 of it, where
// flights and rays that walk took 1.81; of 1000 packets of one wavelength 0.28
// (0.19) for 0.32: the chain of events of the longest packet.  (The FP64 forms
// have 128 VGPRs and 16 to 21 spilled, the mixed ones 117 to 123 and none.)
// Depths are counted from the top, where their differences
// matter: an event's depth is as good as its position was.  (Lambert floors, Draine clouds,
// forced interactions and continuous absorption, images and contribution
// functions need the positions along a flight and take the general kernels.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <math.h>
#include <stdint.h>

#include "transport_common.hpp"

namespace mcrt {
namespace {
using namespace dev;

// depth[m]: optical depth from the top to the lower edge of the m-th layer from
// the top, one thread per solve (tens of layers; their loads go eight at a time).
template <bool MIXED>
__global__ void __launch_bounds__(64) k_slab_depth(GridDev g, const SolveDev* __restrict__ solves, int n)
{
    const int s = blockIdx.x * 64 + threadIdx.x;
    if (s >= n) return;
    const void* a = solves[s].a_ext;
    double* out = solves[s].depth;
    double t = 0.0;
    for (int m0 = 0; m0 < g.nlay; m0 += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = g.nlay - 1 - m0 - u;
            x[u] = k >= 0 ? ld<MIXED>(a, k) * (g.r[k + 1] - g.r[k]) : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (m0 + u < g.nlay) out[m0 + u] = t = t + x[u];
    }
}

// What scatter() and finish_counters() see of a lane's packet.
struct SLane {
    double dx, dy, dz;
    double W, w_abs, w0, wrr;
    unsigned long long id;
    uint32_t ev_no;
    int n_int, ncross, capped, lost, sv;
    int mode, ev;
    __device__ double& sdx() { return dx; }
    __device__ double& sdy() { return dy; }
    __device__ double& sdz() { return dz; }
    __device__ double& W0() { return w0; }
    __device__ double& w_rr() { return wrr; }
    __device__ unsigned long long gid() { return id; }
    __device__ uint32_t& e() { return ev_no; }
    __device__ int& nint() { return n_int; }
    __device__ int& ncapped() { return capped; }
    __device__ int& nlost() { return lost; }
    __device__ int surf() { return 0; }
};

// First m in [lo, n) with t < d[m]; n if there is none.
__device__ __forceinline__ int first_above(const double* d, int lo, int n, double t)
{
    int hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (t < d[mid]) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// An event waits for one load after another, so what it reads lies in LDS where
// the launch's tables fit: TAB = 4 depth, omega, P_gas and g, 1 depth, 0 none.
constexpr int kSlabTable = 2048;  // doubles in all

template <bool MIXED, int TAB>
__global__ void __launch_bounds__(kTPB, 4) k_slab(GridDev g, BatchArgs A)
{
    extern __shared__ double Fs[];  // [n_out][kTPB]: the lanes' contributions; then the tables
    const int nlay = g.nlay, ntab = A.n_solves * nlay;
    double* table = Fs + A.n_out * kTPB;
    if constexpr (TAB > 0) {
        for (int x = threadIdx.x; x < ntab; x += kTPB) {
            const SolveDev& S = A.solves[x / nlay];
            const int c = x % nlay;
            table[x] = S.depth[c];
            if (TAB == 4) {
                table[ntab + x] = ld<MIXED>(S.omega, nlay - 1 - c);
                table[2 * ntab + x] = ld<MIXED>(S.p_gas, nlay - 1 - c);
                table[3 * ntab + x] = ld<MIXED>(S.g_cld, nlay - 1 - c);
            }
        }
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    unsigned long long res_next = 0, res_end = 0;
    bool exhausted = false, own = true;
    double* F = Fs + threadIdx.x;
    SLane L;
    L.mode = lane < A.lanes ? M_DEAD : M_IDLE;
    double t = 0.0, ox = 0.0, oz = 0.0;  // depth from the top; the backscatter direction
    int m = 0;                           // its layer, from the top
    SolveDev S{};                        // (tag and pbase are read)
    for (;;) {
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
                L.id = res_next + (unsigned long long)rank;
                L.mode = M_BIRTH;
            }
            res_next += (unsigned long long)take;
            dead = __ballot(L.mode == M_DEAD);
        }
        if (L.mode == M_DEAD) L.mode = M_IDLE;
        if (__ballot(L.mode != M_IDLE) == 0) break;
        if (L.mode == M_BIRTH) {  // its birth record, as the general kernels'
            const double* b = A.rows + L.id * (unsigned long long)A.row_w + A.n_out;
            L.sv = (int)b[B_SOLVE];
            S.tag = A.solves[L.sv].tag;
            S.pbase = A.solves[L.sv].pbase;
            L.W = L.w0 = b[B_W];
            L.dx = b[B_DX]; L.dy = b[B_DY]; L.dz = b[B_DZ];
            ox = -L.dx;
            oz = -L.dz;
            L.w_abs = L.wrr = 0.0;
            L.ncross = L.n_int = L.capped = L.lost = 0;
            L.ev_no = 1;
            t = 0.0;
            m = 0;
            for (int o = 0; o < A.n_out; ++o) F[o * kTPB] = 0.0;
            L.mode = M_FLIGHT;
            if (b[B_CELL] < 0.0) {
                L.ev = -1;
                finish_counters<false>(L, A, L.ev);
                for (int o = 0; o < A.n_out; ++o) A.rows[L.id * (unsigned long long)A.row_w + o] = 0.0;
            }
        }
        if (L.mode != M_FLIGHT) continue;
        const double* d;
        if constexpr (TAB > 0) d = table + L.sv * nlay;
        else d = A.solves[L.sv].depth;
        // the flight
        const double tau = -log(draw(A.seed, S.tag, L.id - S.pbase, L.ev_no, 0).a);
        t = t - L.dz * tau;
        const int m0 = m;
        int act = A_NONE;
        if (t < 0.0) {
            L.ncross += m0 + 1;
            L.ev = K_ESC;
            act = A_FINISH;
        } else {
            if (L.dz > 0.0) m = first_above(d, 0, m0, t);
            else if (L.dz < 0.0) m = first_above(d, m0, nlay, t);
            L.ncross += L.dz > 0.0 ? m0 - m : m - m0;
            if (m == nlay) {
                L.ev = K_SURF;
                act = A_FINISH;
            } else if (!(t < d[m])) {  // (no extinction along a level flight)
                L.lost += 1;
                L.ev = K_LOST;
                act = A_FINISH;
            }
        }
        if (act == A_NONE) {  // an interaction: peel off towards the observers, then scatter
            double om, pg, gc;
            if constexpr (TAB == 4) {
                om = d[ntab + m];
                pg = d[2 * ntab + m];
                gc = d[3 * ntab + m];
            } else {
                const SolveDev& P = A.solves[L.sv];
                om = ld<MIXED>(P.omega, nlay - 1 - m);
                pg = ld<MIXED>(P.p_gas, nlay - 1 - m);
                gc = ld<MIXED>(P.g_cld, nlay - 1 - m);
            }
            L.n_int += 1;
            const double w = L.W * om;
            for (int o = 0; o < A.n_out; ++o) {
                double vx = ox, vy = 0.0, vz = oz;
                if (A.n_obs != 0) {
                    vx = A.obs[0][3 * o];
                    vy = A.obs[0][3 * o + 1];
                    vz = A.obs[0][3 * o + 2];
                }
                if (!(vz > 0.0)) continue;  // never reaches the top
                const double to = wk_div<MIXED>(t, vz);
                if (to > A.tau_peel_max) {  // dark: the crossings until it is beyond the limit
                    // the nearest edge above from which on the depth passed is more than the limit
                    const double lim = t - A.tau_peel_max * vz;
                    int lo = 0, hi = m;  // edges 0 .. m at depths 0, d[0] .. d[m - 1]
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (d[mid - 1] < lim) lo = mid;
                        else hi = mid - 1;
                    }
                    L.ncross += m + 1 - lo;
                    continue;
                }
                L.ncross += m + 1;
                const double mu = L.dx * vx + L.dy * vy + L.dz * vz;
                const double wt = peel_weight<MIXED>(A, w, mu, (double)(Prop<MIXED>)pg, (double)(Prop<MIXED>)gc);
                double f;
                if (MIXED) f = (double)((float)wt * __expf(-(float)to));
                else f = wt * exp(-to);
                F[o * kTPB] += f * A.peel_w;
            }
            act = scatter<MIXED, false>(L, A, S, om, pg, gc);
        }
        if (act == A_FINISH) {
            double* row = A.rows + L.id * (unsigned long long)A.row_w;
            for (int o = 0; o < A.n_out; ++o) row[o] = F[o * kTPB];
            finish_counters<false>(L, A, L.ev);
        }
    }
}

}  // namespace

void launch_slab(const GridDev& g, const BatchArgs& a, bool mixed, int blocks, hipStream_t stream)
{
    const unsigned nb = (unsigned)((a.n_solves + 63) / 64);
    if (mixed) hipLaunchKernelGGL(k_slab_depth<true>, dim3(nb), dim3(64), 0, stream, g, a.solves, a.n_solves);
    else hipLaunchKernelGGL(k_slab_depth<false>, dim3(nb), dim3(64), 0, stream, g, a.solves, a.n_solves);
    const unsigned long long waves = (a.total + a.lanes - 1) / a.lanes;
    const int grid = (int)std::min<unsigned long long>((unsigned long long)blocks, (waves + 3) / 4);
    const long long ntab = (long long)a.n_solves * g.nlay;
    const int tab = 4 * ntab <= kSlabTable ? 4 : (ntab <= kSlabTable ? 1 : 0);
    const size_t lds = ((size_t)a.n_out * kTPB + tab * ntab) * sizeof(double);
#define MCRT_K(MX, TAB) hipLaunchKernelGGL((k_slab<MX, TAB>), dim3(grid), dim3(kTPB), lds, stream, g, a)
    if (mixed) {
        if (tab == 4) MCRT_K(true, 4);
        else if (tab == 1) MCRT_K(true, 1);
        else MCRT_K(true, 0);
    } else {
        if (tab == 4) MCRT_K(false, 4);
        else if (tab == 1) MCRT_K(false, 1);
        else MCRT_K(false, 0);
    }
#undef MCRT_K
}

}  // namespace mcrt

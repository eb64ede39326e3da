// Batched preparation of the (spectral point, g) solves of one transport
// launch: every stage is a single launch over all solve slots (blockIdx.y =
// slot), so a batch of hundreds of solves costs a handful of launches.
//   optics  K1/K2: per cell, the ck gather or the Doppler-shifted hi-res gather
//                  (Sect. 7) to alpha_ext, alpha_abs, omega, P_gas, g (FP64, and
//                  FP32 copies for the mixed form);
//   sources K3:    per column, L_i = 4 pi V_i alpha_abs B_lambda(T_i) with the
//                  tau_vert cut (Sect. 5.3, Sect. 4.6); per slot L_tot and
//                  N_emit; hybrid bias q_i (Sect. 4.3), birth weights and the
//                  inclusive FP64 CDF of q.
// The arithmetic per cell and the reduction / scan blocking are those of the
// single-solve kernels, so results do not depend on the batch size.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "device_common.hpp"
#include "mcrt_internal.hpp"

namespace mcrt {
namespace {
using namespace dev;

constexpr int kScanPer = 8;
constexpr int kScanBlock = 256 * kScanPer;

// B_lambda(T); lam5 = pow(lam_cm, 5.0).
__device__ __forceinline__ double planck_bl(double lam_cm, double lam5, double T)
{
    double x = kH * kC / (lam_cm * kKB * T);
    return 2.0 * kH * kC * kC / lam5 / expm1(x);
}

__device__ __forceinline__ double hires_kappa_at(const double* __restrict__ lnk_tpl, int nlam, int nP,
                                                 const Bracket& bt, const Bracket& bp, int n, double shift)
{
    double x = (double)n + shift;
    int n0;
    double fr;
    if (nlam == 1) { n0 = 0; fr = 0.0; }
    else if (x <= 0.0) { n0 = 0; fr = 0.0; }
    else if (x >= (double)(nlam - 1)) { n0 = nlam - 2; fr = 1.0; }
    else { n0 = (int)floor(x); fr = x - (double)n0; }
    double k0 = interp_tp([&](int a, int b) { return lnk_tpl[((size_t)a * nP + b) * nlam + n0]; }, bt, bp);
    if (nlam == 1) return k0;
    double k1 = interp_tp([&](int a, int b) { return lnk_tpl[((size_t)a * nP + b) * nlam + n0 + 1]; }, bt, bp);
    return (1.0 - fr) * k0 + fr * k1;
}

// Optics of a cell for `per` slots: its brackets in the opacity table (a
// logarithm and two searches) are found once for them.  The FP64 form's
// transport reads all five properties in FP64, the mixed form's only their FP32
// copies: there FP64 extinction is kept for the emission sources alone.  Those
// start here (L_i, in cdf).  Bound by the bytes written (of 200 mixed slots of
// 128 x 64 x 50 cells 2.9 GB in 0.95 ms; one slot a thread and all properties in
// both types: 4.9 GB in 1.4 ms, and 0.5 ms for L_i by columns).
constexpr int kOpticsSlots = 8;  // slots of a thread, at most
__global__ void __launch_bounds__(256) k_prep_optics(GridDev g, int ncell, const PrepSlot* __restrict__ slots,
                                                     int nslots, int per, int hires, int nT, int nP,
                                                     const double* __restrict__ T_grid,
                                                     const double* __restrict__ lnP_grid,
                                                     const double* __restrict__ lnk_tpl, int nlam,
                                                     const double* __restrict__ shift, int draine, double alpha)
{
    __shared__ double lam5[kOpticsSlots];
    const int s0 = blockIdx.y * per, s1 = min(nslots, s0 + per);
    if ((int)threadIdx.x < s1 - s0) lam5[threadIdx.x] = pow(slots[s0 + threadIdx.x].lam_cm, 5.0);
    __syncthreads();
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncell) return;
    const Bracket bt = bracket(T_grid, nT, (double)g.T[c]);
    const Bracket bp = bracket(lnP_grid, nP, log((double)g.P[c]));
    const double rho = g.rho[c];
    const double ks = g.cld_ksca ? (double)g.cld_ksca[c] : 0.0;
    const double ka = g.cld_kabs ? (double)g.cld_kabs[c] : 0.0;
    const int ncol = g.nlon * g.nlat, k = c / ncol, j = (c - k * ncol) / g.nlon, i = c - k * ncol - j * g.nlon;
    const double dsl = g.lat_sin[j + 1] - g.lat_sin[j];
    const double dph = g.lon[i + 1] - g.lon[i];
    const double vol = g.vol_r[k] * dsl * dph;
    double gc = 0.0;
    if (!hires) {
        gc = g.cld_g ? (double)g.cld_g[c] : 0.0;
        if (draine) gc = draine_G(gc, alpha);  // Draine clouds carry G in place of g
    }
    for (int sl = s0; sl < s1; ++sl) {
        const PrepSlot S = slots[sl];
        double ae, aa, om, pg;
        if (!hires) {
            const double* tab = S.lnk;
            double kg = interp_tp([&](int a, int b) { return tab[a * nP + b]; }, bt, bp);
            double kab = kg + ka;
            double ksc = S.k_ray + ks;
            double kext = kab + ksc;
            ae = rho * kext;
            aa = rho * kab;
            om = kext > 0.0 ? ksc / kext : 0.0;
            pg = ksc > 0.0 ? S.k_ray / ksc : 1.0;
        } else {
            double kl = hires_kappa_at(lnk_tpl, nlam, nP, bt, bp, S.n, shift ? shift[c] : 0.0);
            double kext = kl + S.k_ray;
            ae = rho * kext;
            aa = rho * kl;
            om = kext > 0.0 ? S.k_ray / kext : 0.0;
            pg = 1.0;
        }
        if (!S.optf) {
            double* o = S.opt;
            o[c] = ae;
            o[ncell + c] = aa;
            o[2 * (size_t)ncell + c] = om;
            o[3 * (size_t)ncell + c] = pg;
            o[4 * (size_t)ncell + c] = gc;
        } else {
            float* f = S.optf;
            f[c] = (float)ae;
            f[ncell + c] = (float)aa;
            f[2 * (size_t)ncell + c] = (float)om;
            f[3 * (size_t)ncell + c] = (float)pg;
            f[4 * (size_t)ncell + c] = (float)gc;
            if (S.cdf) S.opt[c] = ae;
        }
        if (S.cdf) S.cdf[c] = 4.0 * kPi * vol * aa * planck_bl(S.lam_cm, lam5[sl - s0], (double)g.T[c]);
    }
}

// L per cell into the slot's cdf array (the first stage of the CDF).
__global__ void __launch_bounds__(256) k_prep_L(GridDev g, const PrepSlot* __restrict__ slots, double tau_vert)
{
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    if (col >= g.nlon * g.nlat) return;
    const PrepSlot S = slots[blockIdx.y];
    const double* a_ext = S.opt;
    double* L = S.cdf;
    const int i = col % g.nlon, j = col / g.nlon;
    double tau = 0.0;
    // (eight layers' loads in flight)
    for (int k0 = g.nlay - 1; k0 >= 0; k0 -= 8) {
        double a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = k0 >= u ? a_ext[((k0 - u) * g.nlat + j) * g.nlon + i] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 - u;
            if (k < 0) break;
            if (tau > tau_vert) L[(k * g.nlat + j) * g.nlon + i] = 0.0;
            tau = tau + a[u] * (g.r[k + 1] - g.r[k]);
        }
    }
}

// (sum L, count L > 0) per 256 cells -> part[slot][block][2]
__global__ void __launch_bounds__(256) k_prep_sumL(const PrepSlot* __restrict__ slots, int n, double* __restrict__ part)
{
    __shared__ double sh[2][256];
    const PrepSlot S = slots[blockIdx.y];
    const int c = blockIdx.x * 256 + threadIdx.x, t = threadIdx.x;
    const double v = c < n ? S.cdf[c] : 0.0;
    sh[0][t] = v;
    sh[1][t] = (c < n && v > 0.0) ? 1.0 : 0.0;
    __syncthreads();
    if (t >= 128) return;
    // waves 0 and 1: the two sums, each a tree of 128, 64, .. 1 apart
    const double* x = sh[t >> 6];
    const int l = t & 63;
    double s = (x[l] + x[l + 128]) + (x[l + 64] + x[l + 192]);
    for (int o = 32; o > 0; o >>= 1) s = s + __shfl_down(s, o);
    if (l == 0) part[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 2 + (t >> 6)] = s;
}

// Neumaier-compensated sum of the block partials -> slot stats (L_tot, N_emit).
__global__ void __launch_bounds__(256) k_prep_stats(const PrepSlot* __restrict__ slots, const double* __restrict__ part,
                                                    int nb)
{
    __shared__ double sh[256];
    __shared__ double shc[256];
    const PrepSlot S = slots[blockIdx.y];
    const int col = blockIdx.x;
    double s = 0.0, comp = 0.0;
    for (int r = threadIdx.x; r < nb; r += 256) {
        double x = part[((size_t)blockIdx.y * nb + r) * 2 + col];
        double t = s + x;
        if (fabs(s) >= fabs(x)) comp = comp + ((s - t) + x);
        else comp = comp + ((x - t) + s);
        s = t;
    }
    sh[threadIdx.x] = s;
    shc[threadIdx.x] = comp;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) {
            double a = sh[threadIdx.x], b = sh[threadIdx.x + st];
            double t = a + b;
            double e = (fabs(a) >= fabs(b)) ? ((a - t) + b) : ((b - t) + a);
            sh[threadIdx.x] = t;
            shc[threadIdx.x] = shc[threadIdx.x] + shc[threadIdx.x + st] + e;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) S.stats[col] = sh[0] + shc[0];
}

// q_i and the birth weights (L_i / L_tot) / q_i of L_i (in cdf), and in its place
// the inclusive scan of q_i: runs of 8 per thread, a Hillis-Steele scan over the
// 256 thread totals, block totals scanned by one block per slot, then the block
// offsets added.
__global__ void __launch_bounds__(256) k_prep_scan_local(const PrepSlot* __restrict__ slots, int n,
                                                         double xi, double* __restrict__ blocksum)
{
    // (thread t scans elements 8 t .. 8 t + 7; they pass through LDS so that
    // memory is read and written in whole lines)
    __shared__ double sh[256];
    __shared__ double el[kScanBlock + kScanBlock / kScanPer];
    const PrepSlot S = slots[blockIdx.y];
    double* io = S.cdf;
    const double Ltot = S.stats[0], nemit = S.stats[1];
    const int base = blockIdx.x * kScanBlock;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        const int e = q * 256 + threadIdx.x;
        const double Lc = base + e < n ? io[base + e] : 0.0;
        double x = 0.0;
        if (Lc > 0.0) x = (1.0 - xi) * Lc / Ltot + xi / nemit;
        if (base + e < n) S.wbirth[base + e] = (Lc > 0.0) ? (Lc / Ltot) / x : 0.0;
        el[e + e / kScanPer] = x;
    }
    __syncthreads();
    double* mine = el + threadIdx.x * (kScanPer + 1);
    double run = 0.0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        run = run + mine[q];
        mine[q] = run;
    }
    sh[threadIdx.x] = run;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        double v = (int)threadIdx.x >= off ? sh[threadIdx.x - off] : 0.0;
        __syncthreads();
        sh[threadIdx.x] = sh[threadIdx.x] + v;
        __syncthreads();
    }
    const double pre = threadIdx.x > 0 ? sh[threadIdx.x - 1] : 0.0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) mine[q] = pre + mine[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
        const int e = q * 256 + threadIdx.x;
        if (base + e < n) io[base + e] = el[e + e / kScanPer];
    }
    if (threadIdx.x == 255) blocksum[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = sh[255];
}

__global__ void __launch_bounds__(256) k_prep_scan_blocksums(double* __restrict__ blocksum, int nb)
{
    __shared__ double sh[256];
    double* bs = blocksum + (size_t)blockIdx.y * nb;
    const int per = (nb + 255) / 256;
    const int b0 = threadIdx.x * per;
    double run = 0.0;
    for (int q = 0; q < per; ++q)
        if (b0 + q < nb) run = run + bs[b0 + q];
    sh[threadIdx.x] = run;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        double v = (int)threadIdx.x >= off ? sh[threadIdx.x - off] : 0.0;
        __syncthreads();
        sh[threadIdx.x] = sh[threadIdx.x] + v;
        __syncthreads();
    }
    double acc = threadIdx.x > 0 ? sh[threadIdx.x - 1] : 0.0;
    for (int q = 0; q < per; ++q) {
        if (b0 + q < nb) {
            double x = bs[b0 + q];
            bs[b0 + q] = acc;
            acc = acc + x;
        }
    }
}

__global__ void __launch_bounds__(256) k_prep_scan_add(const PrepSlot* __restrict__ slots, int n,
                                                       const double* __restrict__ blocksum, int nb)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= n) return;
    const int b = c / kScanBlock;
    if (b > 0) {
        double* io = slots[blockIdx.y].cdf;
        io[c] = blocksum[(size_t)blockIdx.y * nb + b] + io[c];
    }
}

inline unsigned nb(long long n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

size_t prep_scratch_doubles(int ncell, int nslots)
{
    return (size_t)nslots * (2 * (size_t)nb(ncell, 256) + nb(ncell, kScanBlock)) + 16;
}

void launch_prep_optics(const GridDev& g, int ncell, const PrepSlot* slots, int nslots, int hires, int nT, int nP,
                        const double* T_grid, const double* lnP_grid, const double* lnk_tpl, int nlam,
                        const double* shift, int draine, double alpha, hipStream_t stream)
{
    // up to eight slots a thread, of launches that leave eight blocks a CU
    const unsigned blocks = nb(ncell, 256);
    const int per = std::min(std::max((int)((long long)blocks * nslots / 2048), 1), kOpticsSlots);
    hipLaunchKernelGGL(k_prep_optics, dim3(blocks, nb(nslots, per)), dim3(256), 0, stream, g, ncell, slots, nslots, per, hires,
                       nT, nP, T_grid, lnP_grid, lnk_tpl, nlam, shift, draine, alpha);
}

void launch_prep_sources(const GridDev& g, int ncell, const PrepSlot* slots, int nslots, double tau_vert, double xi,
                         double* scratch, hipStream_t stream)
{
    const unsigned ncol = nb(g.nlon * g.nlat, 256), b256 = nb(ncell, 256), bs = nb(ncell, kScanBlock);
    double* lpart = scratch;
    double* bsum = lpart + (size_t)nslots * 2 * b256;
    hipLaunchKernelGGL(k_prep_L, dim3(ncol, nslots), dim3(256), 0, stream, g, slots, tau_vert);
    hipLaunchKernelGGL(k_prep_sumL, dim3(b256, nslots), dim3(256), 0, stream, slots, ncell, lpart);
    hipLaunchKernelGGL(k_prep_stats, dim3(2, nslots), dim3(256), 0, stream, slots, lpart, (int)b256);
    hipLaunchKernelGGL(k_prep_scan_local, dim3(bs, nslots), dim3(256), 0, stream, slots, ncell, xi, bsum);
    if (bs > 1) {
        hipLaunchKernelGGL(k_prep_scan_blocksums, dim3(1, nslots), dim3(256), 0, stream, bsum, (int)bs);
        hipLaunchKernelGGL(k_prep_scan_add, dim3(b256, nslots), dim3(256), 0, stream, slots, ncell, bsum, (int)bs);
    }
}

}  // namespace mcrt

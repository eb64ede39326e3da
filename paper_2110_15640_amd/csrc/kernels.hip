// HIP kernels on a grid's cells for gfx950 (CDNA4, wave64): the line-of-sight
// Doppler shifts of line-by-line tables (Sect. 7, v_LOS and lambda_eff) and the
// checks of borrowed grids.  (Optics and emission sources: prep.hip; transport:
// transport.hip and flight.hip; transmission: chords.hip.)
//
// All FP64 arithmetic is written in the order of its definition and built
// with -ffp-contract=off so that results equal an independent FP64 CPU
// evaluation up to the last-bit differences of the math library.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "device_common.hpp"
#include "mcrt_internal.hpp"

namespace mcrt {
namespace {
using namespace dev;

// ---------------------------------------------------------------- K2
__global__ void __launch_bounds__(256) k_doppler_shift(GridDev g, double ox, double oy, double oz,
                                                       double dlnlam, double* __restrict__ shift)
{
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    int ncell = g.nlon * g.nlat * g.nlay;
    if (c >= ncell) return;
    shift[c] = los_shift(g, c, ox, oy, oz, dlnlam);
}

// ------------------------------------------------- borrowed grid checks
// The validation of host grids, done where borrowed device arrays live:
// every cell sets the bits of the checks it fails (atomic OR on one word).
__global__ void __launch_bounds__(256) k_check_cells(const float* __restrict__ T, const float* __restrict__ P,
                                                     const double* __restrict__ rho, const float* __restrict__ u,
                                                     const float* __restrict__ v, const float* __restrict__ w,
                                                     const float* __restrict__ cs, const float* __restrict__ ca,
                                                     const float* __restrict__ cg, size_t n, int* __restrict__ bad)
{
    int f = 0;
    for (size_t c = (size_t)blockIdx.x * 256 + threadIdx.x; c < n; c += (size_t)gridDim.x * 256) {
        if (!(isfinite(T[c]) && T[c] > 0.0f)) f |= 1;
        if (!(isfinite(P[c]) && P[c] > 0.0f)) f |= 2;
        if (!(isfinite(rho[c]) && rho[c] >= 0.0)) f |= 4;
        if ((u && !isfinite(u[c])) || (v && !isfinite(v[c])) || (w && !isfinite(w[c]))) f |= 8;
        if (cs && !(isfinite(cs[c]) && cs[c] >= 0.0f && isfinite(ca[c]) && ca[c] >= 0.0f)) f |= 16;
        if (cg && !(fabsf(cg[c]) < 1.0f)) f |= 32;
    }
    if (f) atomicOr(bad, f);
}

inline int nblk(long long n, int b) { return (int)((n + b - 1) / b); }

}  // namespace

// ---------------------------------------------------------------- launchers
void launch_doppler_shift(const GridDev& g, double ox, double oy, double oz, double dlnlam, double* shift,
                          hipStream_t stream)
{
    int ncell = g.nlon * g.nlat * g.nlay;
    hipLaunchKernelGGL(k_doppler_shift, dim3(nblk(ncell, 256)), dim3(256), 0, stream, g, ox, oy, oz, dlnlam, shift);
}

void launch_check_cells(const float* T, const float* P, const double* rho, const float* u, const float* v,
                        const float* w, const float* cs, const float* ca, const float* cg, size_t n, int* bad,
                        hipStream_t stream)
{
    const unsigned blocks = (unsigned)std::min<size_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_check_cells, dim3(blocks), dim3(256), 0, stream, T, P, rho, u, v, w, cs, ca, cg, n, bad);
}

}  // namespace mcrt

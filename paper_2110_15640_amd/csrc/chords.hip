// Transmission (Sect. 5.1) by groups of chords, for gfx950 (CDNA4, wave64): the
// optical depths of 16 neighbouring chords (8 impact parameters x
// 2 limb angles) are one small matrix product,
//
//   tau[chord][wavelength] = sum over cells of length[chord][cell] alpha[cell][wavelength],
//
// over the union of the cells that the 16 cross.  Neighbouring chords cross
// mostly the same cells (5 to 9 of the 16 share one on grids of 90 x 46 x 53
// to 64 x 32 x 50 with 1 degree between angles), so an extinction row is
// fetched once for them, and the product runs on the matrix cores in FP64.
//
//   k_chord_walk    the chords' cells and lengths, one walk per chord
//   k_chord_group   the distinct cells of each group, in order of first use
//   k_chord_scan*   places of the groups' rows and of the crossed cells
//   k_cell_rows     each crossed cell's place in the opacity table
//   k_chord_rows    the groups' length matrices
//   k_ck_rows       the solve's ck tables, row fastest
//   k_row_alpha     extinction of the crossed cells for 64 rows of the spectrum
//   k_group_tau     optical depths and tallies
//   k_group_sums*   tallies over the groups, in a fixed order
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "device_common.hpp"
#include "mcrt_internal.hpp"

namespace mcrt {
namespace {
using namespace dev;

constexpr int kGB = 8, kGA = 2;      // impact parameters x limb angles of a group
constexpr int kGC = kGB * kGA;       // its chords
static_assert(kGC == 16, "the matrix instruction takes 16 rows");

// Place of step n of a group's chord c in the walks' arrays: a wave's 64 chords
// (4 groups) are next to each other, so its writes are contiguous.
__device__ __forceinline__ size_t strip(int group, int c, int n, int cap)
{
    return ((size_t)(group >> 2) * cap + n) * 64 + (group & 3) * kGC + c;
}

// ---------------------------------------------------------------- geometry
// One thread per chord, by the transport's walk in its exact form; one pass
// into strips of `cap` steps (what a straight line can cross): 110 us on a 64 x
// 32 x 50 grid with 256 x 360 chords, where a count and a fill pass by per-face
// root finding took 274 + 305.  A wave holds 4 groups; its time is the serial
// chain of its longest chord.  Bit 31 of a cell tells the outgoing half of the
// chord, on which a cell crossed on the way in counts anew: within a half the
// distance from the centre is monotonic and no cell is met twice.
template <typename R>
__global__ void __launch_bounds__(64) k_chord_walk(GridDev g, int n_b, int n_alpha, uint64_t seed, uint32_t tag, ChordDev q,
                                                   LimbDark ld)
{
    for (size_t w = (size_t)blockIdx.x * 64 + threadIdx.x; w < (size_t)q.n_flag_words; w += (size_t)gridDim.x * 64)
        ((uint4*)q.touched)[w] = uint4{0, 0, 0, 0};
    const int t = blockIdx.x * 64 + threadIdx.x;
    const int group = t / kGC, c = t % kGC;
    if (group >= q.n_group) return;
    const int ib = ((q.g0 + group) % q.nbg) * kGB + c % kGB, ia = ((q.g0 + group) / q.nbg) * kGA + c / kGB;
    int n = 0;
    double wb = 0.0;
    uint32_t ok = 1;
    if (ib < n_b && ia < n_alpha) {
        const U2 u = draw(seed, tag, (uint64_t)ib * n_alpha + ia, 0, 0);
        const double r0 = g.r[0], rt = g.r[g.nlay];
        const double b = r0 + ((double)ib + u.a) * (rt - r0) / (double)n_b;
        const double al = 2.0 * kPi * ((double)ia + u.b) / (double)n_alpha;
        const double px = sqrt(fmax(rt * rt - b * b, 0.0)), py = b * cos(al), pz = b * sin(al);
        int i, j;
        locate_column(g, px, py, pz, i, j);
        // the chord's weight: b times the limb-darkening fraction of the
        // stellar light behind it
        wb = b * limb_weight(ld, py, pz);
        Walker w;
        wk_start<false, GEO_SPHERE>(g, w, px, py, pz, -1.0, 0.0, 0.0, i, j, g.nlay - 1);
        R* len = (R*)q.seg_len;
        ok = 0;
        while (n < q.cap) {
            if (g.eq_edge > 0 && w.eq != 0) wk_row_roots<false>(g, w);
            const CrossKind x = wk_next<GEO_SPHERE>(w);
            if (!(x.t < INFINITY)) break;
            const size_t o = strip(group, c, n, q.cap);
            q.seg_cell[o] = (uint32_t)wk_cell(g, w) | (px - w.t > 0.0 ? 0u : 0x80000000u);
            len[o] = (R)(x.t - w.t);
            ++n;
            const CrossIn in = wk_cross_begin<GEO_SPHERE>(g, w, x);
            if (!in.inside) {
                ok = w.k >= g.nlay;
                break;
            }
            wk_cross_end<false, GEO_SPHERE>(g, w, x, in);
            if (n == q.cap && q.cap < q.cap_max) n = q.cap + 1;  // the strip does not hold them
        }
    }
    q.chord_n[t] = (uint32_t)n;
    q.chord_b[t] = wb;
    q.chord_ok[t] = ok;
}

// The distinct cells of a group's chords, numbered by their first use (in
// order of step, then chord): cells are entered in a hash table in LDS with the
// smallest segment number that names them, which no order of the threads
// changes.  Long chords are taken kGroupSteps steps at a time (the table then
// cannot fill up); a cell met again in a later part gets another row.
constexpr int kGroupSteps = 160, kHash = 4096;
constexpr int kGroupIter = kGroupSteps * kGC / 256;

__global__ void __launch_bounds__(256) k_chord_group(ChordDev q)
{
    __shared__ uint32_t key[kHash], first[kHash];
    __shared__ int cnt[kGC];
    __shared__ int wcnt[kGroupIter * 4];
    const int group = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < kGC) cnt[tid] = (int)q.chord_n[group * kGC + tid];
    __syncthreads();
    int most = 0, segs = 0;
    bool over = false;
    for (int c = 0; c < kGC; ++c) {
        over |= cnt[c] > q.cap;
        segs += cnt[c];
        most = cnt[c] > most ? cnt[c] : most;
    }
    if (over) {  // the batch is repeated with longer strips
        if (tid == 0) q.group_n[group] = uint2{kChordOver, 0};
        return;
    }
    const int c = tid % kGC;
    int base = 0;
    for (int n0 = 0; n0 < most; n0 += kGroupSteps) {
        for (int h = tid; h < kHash; h += 256) key[h] = first[h] = 0xffffffffu;
        __syncthreads();
        uint32_t hs[kGroupIter], cell[kGroupIter];
#pragma unroll
        for (int it = 0; it < kGroupIter; ++it) {
            const int s = it * 256 + tid, n = n0 + s / kGC;
            hs[it] = 0xffffffffu;
            if (n >= cnt[c]) continue;
            cell[it] = q.seg_cell[strip(group, c, n, q.cap)];
            uint32_t h = (cell[it] * 2654435761u) >> 20;
            static_assert(kHash == 1 << 12, "hash width");
            for (;;) {
                const uint32_t was = atomicCAS(&key[h], 0xffffffffu, cell[it]);
                if (was == 0xffffffffu || was == cell[it]) break;
                h = (h + 1) & (kHash - 1);
            }
            atomicMin(&first[h], (uint32_t)s);
            hs[it] = h;
        }
        __syncthreads();
        uint32_t mine = 0;
#pragma unroll
        for (int it = 0; it < kGroupIter; ++it) {
            const bool f = hs[it] != 0xffffffffu && first[hs[it]] == (uint32_t)(it * 256 + tid);
            const unsigned long long m = __ballot(f);
            mine |= f ? 1u << it : 0u;
            if (lane == 0) wcnt[it * 4 + wave] = __popcll(m);
        }
        __syncthreads();
        int run = base, at = 0;
#pragma unroll
        for (int it = 0; it < kGroupIter; ++it) {
            for (; at < it * 4 + wave; ++at) run += wcnt[at];
            const bool f = mine >> it & 1;
            const unsigned long long m = __ballot(f);
            if (f) key[hs[it]] = (uint32_t)(run + __popcll(m & ((1ull << lane) - 1)));  // the cell's row
        }
        for (; at < kGroupIter * 4; ++at) run += wcnt[at];
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kGroupIter; ++it) {
            if (hs[it] == 0xffffffffu) continue;
            const bool f = mine >> it & 1;
            q.seg_row[strip(group, c, n0 + (it * 256 + tid) / kGC, q.cap)] = key[hs[it]] | (f ? 0x80000000u : 0u);
            if (f) q.touched[cell[it] & 0x7fffffffu] = 1;
        }
        base = run;
        __syncthreads();
    }
    if (tid == 0) q.group_n[group] = uint2{(uint32_t)base, (uint32_t)segs};
}

// Exclusive prefix sums, in two launches, of the crossed cells (their place
// among the crossed) and of the groups' rows, in whole quads (the matrix
// instruction's depth).  Blocks [0, n_fblk) take 4096 cells each, the rest 256
// groups each; totals: rows, cells, segments, groups not held.
__device__ __forceinline__ unsigned long long block_sum(unsigned long long v, unsigned long long* sh)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return sh[0] + sh[1] + sh[2] + sh[3];
}
__device__ __forceinline__ uint32_t quads(uint32_t rows) { return (rows + 3) & ~3u; }

__global__ void __launch_bounds__(256) k_chord_scan_sums(ChordDev q)
{
    __shared__ unsigned long long sh[4];
    const int tid = threadIdx.x;
    unsigned long long a = 0, b = 0, c = 0;
    if ((int)blockIdx.x < q.n_fblk) {
        const int w = blockIdx.x * 256 + tid;
        if (w < q.n_flag_words) {
            const uint4 v = ((const uint4*)q.touched)[w];
            a = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
        }
    } else {
        const int gr = ((int)blockIdx.x - q.n_fblk) * 256 + tid;
        if (gr < q.n_group) {
            const uint2 n = q.group_n[gr];
            if (n.x == kChordOver) c = 1;
            else {
                a = quads(n.x);
                b = n.y;
            }
        }
    }
    a = block_sum(a, sh);
    b = block_sum(b, sh);
    c = block_sum(c, sh);
    if (tid == 0) {
        q.bsum[3 * blockIdx.x] = a;
        q.bsum[3 * blockIdx.x + 1] = b;
        q.bsum[3 * blockIdx.x + 2] = c;
    }
}

__global__ void __launch_bounds__(256) k_chord_scan_apply(ChordDev q)
{
    __shared__ unsigned long long sh[4];
    __shared__ uint32_t ws[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, blk = blockIdx.x;
    const bool flags = blk < q.n_fblk;
    const int b0 = flags ? 0 : q.n_fblk, last = flags ? q.n_fblk - 1 : (int)gridDim.x - 1;
    unsigned long long before = 0, segs = 0, over = 0;
    for (int b = b0 + tid; b < blk; b += 256) before += q.bsum[3 * b];
    before = block_sum(before, sh);
    if (blk == last && !flags) {
        for (int b = b0 + tid; b <= last; b += 256) {
            segs += q.bsum[3 * b + 1];
            over += q.bsum[3 * b + 2];
        }
        segs = block_sum(segs, sh);
        over = block_sum(over, sh);
    }
    uint32_t v[16];
    uint32_t mine = 0;
    const int w = blk * 256 + tid, gr = (blk - q.n_fblk) * 256 + tid;
    if (flags) {
        uint4 f = uint4{0, 0, 0, 0};
        if (w < q.n_flag_words) f = ((const uint4*)q.touched)[w];
        const uint32_t x[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            v[e] = x[e / 4] >> (8 * (e % 4)) & 1;
            mine += v[e];
        }
    } else if (gr < q.n_group && q.group_n[gr].x != kChordOver) {
        mine = quads(q.group_n[gr].x);
    }
    uint32_t inc = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) ws[wave] = inc;
    __syncthreads();
    uint32_t at = (uint32_t)before + inc - mine;
    for (int k = 0; k < wave; ++k) at += ws[k];
    if (flags) {
        uint32_t a = at;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (v[e]) q.comp[(size_t)w * 16 + e] = a;
            a += v[e];
        }
    } else if (gr < q.n_group) {
        q.group_at[gr] = at;
    }
    if (blk == last && tid == 255) {
        if (flags) q.totals[1] = at + mine;
        else {
            q.totals[0] = before + ws[0] + ws[1] + ws[2] + ws[3];
            q.totals[2] = segs;
            q.totals[3] = over;
        }
    }
}

// The groups' length matrices: row (cell) fastest over the 16 chords.  Each
// entry is one segment's length (see the halves above), added to a zero.
template <typename R>
__global__ void __launch_bounds__(256) k_chord_rows(ChordDev q)
{
    const int group = blockIdx.x, tid = threadIdx.x, c = tid % kGC;
    const size_t r0 = q.group_at[group];
    const uint32_t n = q.group_n[group].x, n4 = quads(n);
    R* len = (R*)q.row_len + r0 * kGC;
    const R* sl = (const R*)q.seg_len;
    for (uint32_t e = tid; e < n4 * kGC; e += 256) len[e] = (R)0;
    if (tid < 4 && n + tid < n4) q.row_cell[r0 + n + tid] = 0;  // (a row of no length)
    __syncthreads();
    const int steps = (int)q.chord_n[group * kGC + c];
    for (int s = tid / kGC; s < steps; s += 256 / kGC) {
        const size_t o = strip(group, c, s, q.cap);
        const uint32_t w = q.seg_row[o], row = w & 0x7fffffffu;
        unsafeAtomicAdd(&len[row * kGC + c], sl[o]);
        if (w >> 31) q.row_cell[r0 + row] = q.comp[q.seg_cell[o] & 0x7fffffffu];
    }
}

// ---------------------------------------------------------------- extinction
// A crossed cell's place in the opacity table: its four (T, ln P) corners and
// their weights in the type in which ln kappa is summed.
template <typename W, bool HIRES>
__global__ void __launch_bounds__(256) k_cell_rows(GridDev g, int ncell, ChordDev q, int nT, int nP,
                                                   const double* __restrict__ T_grid, const double* __restrict__ lnP_grid,
                                                   double dlnlam, CellRow<W>* __restrict__ out)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= ncell || !q.touched[c]) return;
    const Bracket bt = bracket(T_grid, nT, (double)g.T[c]);
    const Bracket bp = bracket(lnP_grid, nP, log((double)g.P[c]));
    const W t = (W)bt.t, u = (W)bp.t, one = (W)1;
    CellRow<W> r;
    r.row[0] = bt.i0 * nP + bp.i0;
    r.row[1] = bt.i0 * nP + bp.i1;
    r.row[2] = bt.i1 * nP + bp.i0;
    r.row[3] = bt.i1 * nP + bp.i1;
    r.w[0] = (one - t) * (one - u);
    r.w[1] = (one - t) * u;
    r.w[2] = t * (one - u);
    r.w[3] = t * u;
    int used = r.row[0];  // a corner with weight
#pragma unroll
    for (int k = 0; k < 4; ++k) used = r.w[k] > (W)0 ? r.row[k] : used;
#pragma unroll
    for (int k = 0; k < 4; ++k) r.row[k] = r.w[k] > (W)0 ? r.row[k] : used;
    r.rho = g.rho[c];
    r.shift = HIRES ? los_shift(g, c, -1.0, 0.0, 0.0, dlnlam) : 0.0;
    r.ks = g.cld_ksca ? g.cld_ksca[c] : 0.0f;
    r.ka = g.cld_kabs ? g.cld_kabs[c] : 0.0f;
    out[q.comp[c]] = r;
}

// The ck tables of nrow of the solve's rows from row0, row fastest in blocks of 64: a cell's 64
// values at a corner are then contiguous.
__global__ void __launch_bounds__(256) k_ck_rows(const double* __restrict__ lnk, int ng_tab, int ntp,
                                                 const int* __restrict__ specs, int ng, int row0, int nrow,
                                                 const double* __restrict__ k_ray, double* __restrict__ tab,
                                                 double* __restrict__ kray_row)
{
    const int s = threadIdx.x & 63, r = row0 + min((int)blockIdx.x * 64 + s, nrow - 1);
    const int spec = specs[r / ng];
    const double* src = lnk + ((size_t)spec * ng_tab + r % ng) * ntp;
    double* dst = tab + (size_t)blockIdx.x * ntp * 64;
    for (int e = blockIdx.y * 4 + (threadIdx.x >> 6); e < ntp; e += gridDim.y * 4) dst[(size_t)e * 64 + s] = src[e];
    if (blockIdx.y == 0 && threadIdx.x < 64) kray_row[(size_t)blockIdx.x * 64 + s] = k_ray[spec];
}

// Table position n + shift split into the lower neighbour n0 and the
// fraction fr, clamped at the table ends.
__device__ __forceinline__ void hires_pos(int nlam, int n, double shift, int& n0, double& fr)
{
    const double x = wk_min(wk_max((double)n + shift, 0.0), (double)(nlam - 1));
    n0 = min((int)x, nlam > 1 ? nlam - 2 : 0);
    fr = x - (double)n0;
}

// kappa = exp(sum of w l).  l is finite or -inf; a corner with weight and -inf
// gives zero.  (A corner without weight stands for one with weight, k_cell_rows,
// so 0 times -inf, the only NaN here, is that case too.)
template <typename W>
__device__ __forceinline__ W corner_sum(const W* l, const CellRow<W>& q)
{
    W acc = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if constexpr (sizeof(W) == 4) acc = fmaf(q.w[k], l[k], acc);
        else acc = acc + q.w[k] * l[k];
    }
    W e;
    if constexpr (sizeof(W) == 4) e = __expf(acc);
    else e = exp(acc);
    return acc == acc ? e : (W)0;
}

template <typename R>
__device__ __forceinline__ R below_inf(double a)
{
    // lengths of zero multiply it: the largest finite value in place of
    // infinity is as opaque and leaves them zero
    const R big = sizeof(R) == 4 ? (R)3.4028234663852886e38 : (R)1.7976931348623157e308;
    const R r = (R)a;
    return r > big ? big : r;
}

// alpha[cell][slot] of the crossed cells for up to 64 rows of the spectrum.
// A wave takes kRowCells cells, lanes over the slots; a cell's corners and
// weights are then uniform and come through the scalar cache.  Line by line
// tables are shifted by each cell's velocity and interpolated linearly between
// the two table wavelengths around a slot's: the upper one is the next lane's
// lower one whenever that lane has the next table wavelength, so each kappa is
// evaluated once; for the last slot they are evaluated beforehand, one cell per
// lane.  Lanes past the last slot repeat it.
// 30 us for 64 rows of the 223000 crossed cells of a 128 x 64 x 60 grid in FP32,
// two thirds of it vector instructions (50 a cell); every cell of that grid with
// each value evaluated twice took 210.
constexpr int kRowCells = 8;

template <typename R, typename W, bool HIRES>
__global__ void __launch_bounds__(256) k_row_alpha(const CellRow<W>* __restrict__ cells, int n_cells,
                                                   const W* __restrict__ tab, int nlam, const double* __restrict__ k_ray,
                                                   const int* __restrict__ nlist, int nslot, int stride,
                                                   R* __restrict__ alpha)
{
    const int lane = threadIdx.x & 63;
    const int c0 = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6))) * kRowCells;
    if (c0 >= n_cells) return;
    const int s = lane < nslot ? lane : nslot - 1;
    const int n = HIRES ? nlist[s] : s;
    const double kr = k_ray[n];
    const int d = HIRES && nlam > 1 ? 1 : 0;
    const bool end = lane >= nslot - 1;
    W k_end = 0;
    if (HIRES && d) {
        const CellRow<W>& q = cells[min(c0 + (lane & (kRowCells - 1)), n_cells - 1)];
        int n0;
        double fr;
        hires_pos(nlam, nlist[nslot - 1], q.shift, n0, fr);
        W l[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) l[k] = tab[(size_t)q.row[k] * nlam + (unsigned)(n0 + 1)];
        k_end = corner_sum<W>(l, q);
    }
    constexpr int U = 4;  // cells whose loads are in flight together
#pragma unroll
    for (int u0 = 0; u0 < kRowCells; u0 += U) {
        W l[U][4];
        int n0[U];
        double fr[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const CellRow<W>& q = cells[min(c0 + u0 + u, n_cells - 1)];
            if constexpr (HIRES) hires_pos(nlam, n, q.shift, n0[u], fr[u]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const W* row = tab + (size_t)q.row[k] * (HIRES ? nlam : 64);
                l[u][k] = row[(unsigned)(HIRES ? n0[u] : s)];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u0 + u;
            if (c >= n_cells) break;
            const CellRow<W>& q = cells[c];
            const W k0 = corner_sum<W>(l[u], q);
            double kext;
            if constexpr (HIRES) {
                double kl = (double)k0;
                if (d) {
                    W k1 = __shfl_down(k0, 1);
                    const bool take = __shfl_down(n0[u], 1) == n0[u] + 1;
                    const W ke = __shfl(k_end, u0 + u);
                    k1 = end ? ke : k1;
                    if (!end && !take) {
                        W m[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) m[k] = tab[(size_t)q.row[k] * nlam + (unsigned)(n0[u] + 1)];
                        k1 = corner_sum<W>(m, q);
                    }
                    if constexpr (sizeof(W) == 4) {
                        const float f = (float)fr[u];
                        kl = (double)fmaf(f, k1, (1.0f - f) * k0);
                    } else {
                        kl = (1.0 - fr[u]) * k0 + fr[u] * k1;
                    }
                }
                kext = kl + kr;
            } else {
                kext = (k0 + (double)q.ka) + (kr + (double)q.ks);
            }
            R* row = alpha + (size_t)c * stride;
            if (lane < stride) row[(unsigned)lane] = below_inf<R>(q.rho * kext);
        }
    }
}

// ---------------------------------------------------------------- optical depths
typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int kTauBlocks = 2;   // 16-slot blocks of a wave (of 16 slots in all: 1)
constexpr int kTauBytes = 64;   // bytes of extinction that a lane has in flight
constexpr int kRuns = 16;       // runs of groups of each XCD
template <typename R, int NB>
struct __attribute__((aligned(sizeof(R) * NB))) RowVec {
    R v[NB];
};

// One group's optical depths by FP64 matrix instructions of 16 chords x 16
// slots x 4 cells, and its sums of (1 - e^-tau) b and of their squares.  A wave
// takes 16 NB slots of a group (lane & 15 holds NB neighbouring ones) and all
// of its cells, so nothing is shared between waves and the accumulators stay
// small enough for eight waves a SIMD: a group has few cells (some 200, at the
// poles 800) and the time goes on waiting for their rows.  Of a 128 x 64 x 60
// grid's 256 x 360 chords and 64 rows in FP32 the matrix instructions alone are
// 34 us, and the kernel takes 88 (a wave per segment's row, without groups:
// 420).  One or four blocks a wave instead of two, and four waves that
// share a group's cells, are 10 to 15 % slower there; twice the loads in flight
// are no faster.
template <typename R, int NB>
__global__ void __launch_bounds__(256) k_group_tau(ChordDev q, const R* __restrict__ alpha, int stride,
                                                   double* __restrict__ part)
{
    const int lane = threadIdx.x & 63, n = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // XCD x takes runs x, x + 8, ... of kRuns x 8 runs of the groups, which
    // follow the limb angle: the cells of an angle are then read into one L2
    // only, and each XCD has its share of the poles, whose chords cross more
    // cells (of the 256 x 360 chords on 128 x 64 x 60 cells the largest share is
    // 1.05 of the mean; with one run each 1.29)
    const int parts = stride / (16 * NB);  // waves of a group
    const int n_blk = (q.n_group * parts + 3) / 4, per = (n_blk + kRuns * kXcds - 1) / (kRuns * kXcds);
    const int turn = (int)blockIdx.x / kXcds;
    const int blk = ((turn / per) * kXcds + (int)blockIdx.x % kXcds) * per + turn % per;
    const int id = blk * 4 + wave, group = id / parts;
    if (group >= q.n_group) return;
    const int s0 = (id % parts) * (16 * NB) + n * NB;
    const size_t r0 = q.group_at[group];
    const int nq = (int)(quads(q.group_n[group].x) / 4);
    const uint32_t* __restrict__ rc = q.row_cell + r0 + kq;
    const R* __restrict__ rl = (const R*)q.row_len + r0 * kGC + lane;
    const R* __restrict__ al = alpha + s0;
    // register r of an accumulator holds chord 4 r + kq
    double wb[4];
    bool ok[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        wb[r] = q.chord_b[group * kGC + 4 * r + kq];
        ok[r] = q.chord_ok[group * kGC + 4 * r + kq] != 0;
    }
    d4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = d4{0.0, 0.0, 0.0, 0.0};
    // U quads at a time, their loads in flight together (a quad past the end
    // repeats the last one with length zero); the cells of the next U are
    // fetched before the products
    constexpr int U = kTauBytes / (NB * (int)sizeof(R));
    uint32_t cell[U];
    auto cells = [&](int at) {
#pragma unroll
        for (int u = 0; u < U; ++u) cell[u] = rc[(unsigned)min(at + u, nq - 1) * 4];
    };
    if (nq > 0) cells(0);
    for (int i = 0; i < nq; i += U) {
        R len[U];
        RowVec<R, NB> a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = *(const RowVec<R, NB>*)(al + (size_t)cell[u] * stride);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const R x = rl[(unsigned)min(i + u, nq - 1) * 64];
            len[u] = i + u < nq ? x : (R)0;
        }
        cells(i + U);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < NB; ++b)
                acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)len[u], (double)a[u].v[b], acc[b], 0, 0, 0);
    }
    double* out = part + (size_t)group * (2 * stride) + s0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        double s1 = 0.0, s2 = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double v = (1.0 - (ok[r] ? exp(-acc[b][r]) : 0.0)) * wb[r];
            s1 = s1 + v;
            s2 = s2 + v * v;
        }
        for (int o = 16; o < 64; o <<= 1) {
            s1 = s1 + __shfl_xor(s1, o);
            s2 = s2 + __shfl_xor(s2, o);
        }
        if (kq == 0) {
            out[b] = s1;
            out[stride + b] = s2;
        }
    }
}

// ---------------------------------------------------------------- tallies
// Neumaier-compensated sum and its correction, over a fixed order.
__device__ __forceinline__ void comp_add(double& s, double& c, double x, double xc)
{
    const double t = s + x;
    c = c + ((fabs(s) >= fabs(x) ? (s - t) + x : (x - t) + s) + xc);
    s = t;
}

// Chunk sums of each column over groups [64 blockIdx.x, + 64): threads over the
// columns, and over every k-th group, eight loads in flight in each.
constexpr int kSumThreads = 512;
__global__ void __launch_bounds__(kSumThreads) k_group_sums(const double* __restrict__ part, int n_group, int width,
                                                            double2* __restrict__ out)
{
    __shared__ double2 sh[kSumThreads];
    const int col = threadIdx.x % width, k = threadIdx.x / width, nk = kSumThreads / width;
    const int g1 = min(n_group, ((int)blockIdx.x + 1) * kGroupChunk);
    double s = 0.0, c = 0.0;
    for (int gr = blockIdx.x * kGroupChunk + k; gr < g1; gr += 8 * nk) {
        double x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = gr + e * nk < g1 ? part[(size_t)(gr + e * nk) * width + col] : 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) comp_add(s, c, x[e], 0.0);
    }
    sh[threadIdx.x] = double2{s, c};
    __syncthreads();
    if (k == 0) {
        for (int e = 1; e < nk; ++e) comp_add(s, c, sh[e * width + col].x, sh[e * width + col].y);
        out[(size_t)blockIdx.x * 128 + col] = double2{s, c};
    }
}

// All blocks of rows at once: the sum of each row's chunks.
__global__ void __launch_bounds__(64) k_group_final(const double2* __restrict__ chunks, int n_chunk, int nrow,
                                                    double* __restrict__ sums)
{
    const int blk = blockIdx.x, j = blockIdx.y, s = threadIdx.x;
    const int nslot = min(64, nrow - blk * 64);
    if (s >= nslot) return;
    const double2* src = chunks + (size_t)blk * n_chunk * 128 + j * chord_stride(nslot) + s;
    double a = 0.0, c = 0.0;
    for (int e = 0; e < n_chunk; e += 8) {
        double2 x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = e + u < n_chunk ? src[(size_t)(e + u) * 128] : double2{0.0, 0.0};
#pragma unroll
        for (int u = 0; u < 8; ++u) comp_add(a, c, x[u].x, x[u].y);
    }
    sums[2 * ((size_t)blk * 64 + s) + j] = a + c;
}

inline int nblk(long long n, int b) { return (int)((n + b - 1) / b); }

}  // namespace

// ---------------------------------------------------------------- launchers
void chord_shape(ChordDev& q, const GridDev& g, int ncell, int n_b, int n_alpha)
{
    q = ChordDev{};
    q.nbg = nblk(n_b, kGB);
    q.n_total = q.nbg * nblk(n_alpha, kGA);
    // a straight line meets every shell and cone at most twice and every half plane once
    q.cap = 2 * g.nlay + 2 * g.nlat + g.nlon + 8;
    q.cap_max = 64 * (g.nlay + g.nlat + g.nlon) + 64;
    chord_batch(q, 0, q.n_total);
    q.n_flag_words = nblk(ncell, 16);
    q.n_fblk = nblk(q.n_flag_words, 256);
}
void chord_batch(ChordDev& q, int g0, int n_group)
{
    q.g0 = g0;
    q.n_group = n_group;
    q.n_wave = nblk(n_group, 64 / kGC);
}
int chord_scan_blocks(const ChordDev& q) { return q.n_fblk + nblk(q.n_group, 256); }

template <typename R>
void launch_chord_geometry(const GridDev& g, int n_b, int n_alpha, uint64_t seed, uint32_t tag, const ChordDev& q,
                           const LimbDark& ld, hipStream_t stream)
{
    hipLaunchKernelGGL(k_chord_walk<R>, dim3(q.n_wave), dim3(64), 0, stream, g, n_b, n_alpha, seed, tag, q, ld);
    hipLaunchKernelGGL(k_chord_group, dim3(q.n_group), dim3(256), 0, stream, q);
    hipLaunchKernelGGL(k_chord_scan_sums, dim3(chord_scan_blocks(q)), dim3(256), 0, stream, q);
    hipLaunchKernelGGL(k_chord_scan_apply, dim3(chord_scan_blocks(q)), dim3(256), 0, stream, q);
}
template void launch_chord_geometry<double>(const GridDev&, int, int, uint64_t, uint32_t, const ChordDev&, const LimbDark&,
                                            hipStream_t);
template void launch_chord_geometry<float>(const GridDev&, int, int, uint64_t, uint32_t, const ChordDev&, const LimbDark&,
                                           hipStream_t);

template <typename R>
void launch_chord_rows(const ChordDev& q, hipStream_t stream)
{
    hipLaunchKernelGGL(k_chord_rows<R>, dim3(q.n_group), dim3(256), 0, stream, q);
}
template void launch_chord_rows<double>(const ChordDev&, hipStream_t);
template void launch_chord_rows<float>(const ChordDev&, hipStream_t);

template <typename W>
void launch_cell_rows(const GridDev& g, int ncell, const ChordDev& q, bool hires, int nT, int nP, const double* T_grid,
                      const double* lnP_grid, double dlnlam, CellRow<W>* out, hipStream_t stream)
{
    if (hires)
        hipLaunchKernelGGL((k_cell_rows<W, true>), dim3(nblk(ncell, 256)), dim3(256), 0, stream, g, ncell, q, nT, nP, T_grid,
                           lnP_grid, dlnlam, out);
    else
        hipLaunchKernelGGL((k_cell_rows<W, false>), dim3(nblk(ncell, 256)), dim3(256), 0, stream, g, ncell, q, nT, nP, T_grid,
                           lnP_grid, dlnlam, out);
}
template void launch_cell_rows<double>(const GridDev&, int, const ChordDev&, bool, int, int, const double*, const double*,
                                       double, CellRow<double>*, hipStream_t);
template void launch_cell_rows<float>(const GridDev&, int, const ChordDev&, bool, int, int, const double*, const double*,
                                      double, CellRow<float>*, hipStream_t);

void launch_ck_rows(const double* lnk, int ng_tab, int ntp, const int* specs, int ng, int row0, int nrow, const double* k_ray,
                    double* tab, double* kray_row, hipStream_t stream)
{
    hipLaunchKernelGGL(k_ck_rows, dim3(nblk(nrow, 64), std::min(nblk(ntp, 4), 64)), dim3(256), 0, stream, lnk, ng_tab, ntp, specs,
                       ng, row0, nrow, k_ray, tab, kray_row);
}

template <typename R, typename W>
void launch_row_alpha(const CellRow<W>* cells, int n_cells, bool hires, const W* tab, int nlam, const double* k_ray,
                      const int* nlist, int nslot, R* alpha, hipStream_t stream)
{
    const dim3 grid(nblk(n_cells, 4 * kRowCells)), block(256);
    const int stride = chord_stride(nslot);
    if constexpr (sizeof(W) == sizeof(R)) {
        if (hires) {
            hipLaunchKernelGGL((k_row_alpha<R, W, true>), grid, block, 0, stream, cells, n_cells, tab, nlam, k_ray, nlist, nslot,
                               stride, alpha);
            return;
        }
    }
    if constexpr (sizeof(W) == sizeof(double))
        hipLaunchKernelGGL((k_row_alpha<R, W, false>), grid, block, 0, stream, cells, n_cells, tab, nlam, k_ray, nlist, nslot,
                           stride, alpha);
}
template void launch_row_alpha<double, double>(const CellRow<double>*, int, bool, const double*, int, const double*, const int*,
                                               int, double*, hipStream_t);
template void launch_row_alpha<float, double>(const CellRow<double>*, int, bool, const double*, int, const double*, const int*,
                                              int, float*, hipStream_t);
template void launch_row_alpha<float, float>(const CellRow<float>*, int, bool, const float*, int, const double*, const int*, int,
                                             float*, hipStream_t);

template <typename R>
void launch_group_tau(const ChordDev& q, const R* alpha, int nslot, double* part, hipStream_t stream)
{
    const int stride = chord_stride(nslot);
    const int nb = std::min(stride / 16, kTauBlocks);
    const int n_blk = nblk((long long)q.n_group * (stride / (16 * nb)), 4);
    const dim3 grid(nblk(n_blk, kRuns * kXcds) * kRuns * kXcds), block(256);
    if (nb == kTauBlocks) hipLaunchKernelGGL((k_group_tau<R, kTauBlocks>), grid, block, 0, stream, q, alpha, stride, part);
    else hipLaunchKernelGGL((k_group_tau<R, 1>), grid, block, 0, stream, q, alpha, stride, part);
}
template void launch_group_tau<double>(const ChordDev&, const double*, int, double*, hipStream_t);
template void launch_group_tau<float>(const ChordDev&, const float*, int, double*, hipStream_t);

void launch_group_sums(const double* part, int n_group, int nslot, double* chunks, hipStream_t stream)
{
    hipLaunchKernelGGL(k_group_sums, dim3(nblk(n_group, kGroupChunk)), dim3(kSumThreads), 0, stream, part, n_group,
                       2 * chord_stride(nslot), (double2*)chunks);
}

void launch_group_final(const double* chunks, int n_chunk, int nrow, double* sums, hipStream_t stream)
{
    hipLaunchKernelGGL(k_group_final, dim3(nblk(nrow, 64), 2), dim3(64), 0, stream, (const double2*)chunks, n_chunk, nrow, sums);
}

}  // namespace mcrt

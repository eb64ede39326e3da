// Internal structures shared by the host runtime (api.cpp) and the HIP
// kernels (kernels.hip).  Device pointers only; plain data.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mcrt {

constexpr int kMaxObs = 8;
constexpr int kMaxSolvesPerLaunch = 1 << 20;  // solve index field of the transport's packed lane state
constexpr int kXcds = 8;                      // packet dispensers per launch, one per XCD
constexpr int kCtrStride = 32;                // words between counters that all waves share (cache lines of their own)
constexpr int kNCounters = 11;
enum Counter { K_ESC = 0, K_SURF, K_ABS, K_RR, K_CAP, K_LOST, K_NINT, K_NCROSS, K_NCAPPED, K_NLOST, K_W0 };

// Geometry of one resident grid.  The trigonometric edge tables are computed
// once at upload on the host.
struct GridDev {
    int geom;  // 0 spherical, 1 slab
    int nlon, nlat, nlay;
    int max_cross;
    const double* r;       // [nlay+1]
    const double* lat;     // [nlat+1]
    const double* lat_c2;  // cos^2(lat edge)
    const double* lat_sin; // sin(lat edge)
    const double* lon;     // [nlon+1]
    const double* vol_r;   // (r_{k+1}^3 - r_k^3)/3 [nlay]
    // the edge values a crossing reads, in one array so that one base and a
    // per-lane offset reach any of them with one 16-byte load: the layer's
    // (r[k], r[k + 1]) at k; (sin lat[j], sin lat[j + 1]) of row j at
    // lat_base + j (-2 and 2 at the poles); (sin, cos) of longitude edge e (edge nlon = edge 0) at
    // lon_base + e
    const double2* faces;
    int lat_base, lon_base;
    int eq_edge;  // latitude edge within rounding of the equator but not on it (0 = none)
    const float* T;
    const float* P;
    const double* rho;
    const float* u;
    const float* v;
    const float* w;
    const float* cld_ksca;
    const float* cld_kabs;
    const float* cld_g;
    double omega_rot;
};

// One (spectral point, g) solve inside a persistent transport launch.
// Optical-property arrays are double (FP64) or float (MIXED).
struct SolveDev {
    const void* a_ext;
    const void* a_abs;
    const void* omega;
    const void* p_gas;
    const void* g_cld;
    const double* cdf;     // emission only
    const double* wbirth;  // emission only
    unsigned long long begin;  // global index of the solve's first packet
    unsigned long long n;      // packets of the solve
    unsigned long long pbase;  // packet id 0 of the random stream (begin, or the band's first packet)
    uint32_t tag;
    int mode;  // 0 albedo, 1 emission
    int grid;  // index into BatchArgs.grids (multi-grid launches)
    // per-event tallies, each scaled by cf_w * (*cf_ltot if set):
    // contribution functions cf[(observer * 2 + part) * ncell + cell] and
    // images img[(observer * npix + row) * npix + column] (null = off)
    double* cf;
    double* img;
    double cf_w;
    const double* cf_ltot;
    // per-packet g-ordinate sampling: on the first solve of a band, the number
    // of g-ordinates (the band's solves follow it) and the scheme
    // (1 unbiased, 2 uniform, 3 composite); 0 = fixed-g solve
    int gs_n;
    int gs_scheme;
    const double* gs_w;    // g-ordinate weights of the table
    const double* ltot;    // emission: L_tot of this solve (written by the preparation)
    double* depth;         // slab launches: optical depth from the top, [nlay]
};

// Stellar limb darkening of transmission chords and packets: law (0 none,
// 1 linear, 2 quadratic, 3 square-root, 4 logarithmic, 5 exponential,
// 6 power-2), its coefficients, the planet centre on the stellar disk (sky
// plane, cm) and the stellar radius.
struct LimbDark {
    int law;
    double c1, c2;
    double ty, tz;
    double r_star;
};

struct BatchArgs {
    const SolveDev* solves;
    int n_solves;
    const GridDev* grids;  // per-solve grids of a multi-grid launch (else unused)
    unsigned long long total;     // packets over all solves
    unsigned long long* counter;  // kXcds packet dispensers (one chunk of the packets each)
    int ctr_stride;               // elements between them (cache lines of their own where scratch allows)
    double* rows;                 // [total][row_w]: F per observer, then counters
    int row_w;
    uint64_t seed;
    int scattering;
    int absorption;
    int n_obs;
    int n_out;
    long long max_events;
    double rr_threshold;
    double rr_survive;
    double tau_peel_max;
    double mu0;
    double r_toa;
    double obs[2][3 * kMaxObs];  // observer directions for albedo [0] and emission [1] solves
    int slab;          // scattered light of a slab without what slab.hip leaves to the general kernels
    int batch;         // packets a wave takes from the dispenser at once
    int lanes;         // lanes of a wave that carry packets (split launches)
    int ev_threshold;  // waiting lanes that trigger event handling
    int cloud_phase;   // 0 Henyey-Greenstein, 1 two-term Henyey-Greenstein, 2 Draine (g_cld holds G)
    double draine_alpha;
    double surface_albedo;  // 0: the lower boundary absorbs; > 0: Lambert albedo of the floor
    // transmission with multiple scattering: births on the annulus, the birth
    // peel-off is the direct light (no 1/4pi), later peel-offs are scaled by
    // peel_w (the stellar beam's solid angle; 1 otherwise), and a packet's
    // row holds W0 - F
    int trans_ms;
    double peel_w;
    int forced;        // forced interaction: 0 off, 1 forced scattering, 2 path-length stretching, 3 hybrid
    int forced_first;  // 1: only a packet's first flight
    LimbDark ld;
    // images: npix x npix pixels over [-img_half, img_half]^2 of each
    // observer's sky plane, horizontal / vertical unit vectors per observer
    int npix;
    double img_half;
    double img_axes[6 * kMaxObs];
    // split launches: each packet's first peel-off record (null: peel-offs run inside the transport)
    uint32_t* head;
    uint32_t* peel_cross;  // and the crossings of its peel-off rays so far
};

// Scratch of a split launch (flight.hip): flights append a record per event
// that peels off, a second kernel walks the peel-off rays of all records, a
// third adds their contributions to the packets' rows in the order of events.
constexpr uint32_t kNoRecord = 0xFFFFFFFFu;
// What a record's ray towards one observer gives: its contribution and number of
// crossings.  One cache line holds those of four observers.
struct alignas(16) PeelOut {
    double f;
    uint32_t nx;
};
struct PeelArgs {
    void* rec;        // records, one region per XCD
    uint32_t* head;   // BatchArgs.head and peel_cross
    uint32_t* peel_cross;
    uint32_t* next;   // the packet's next record
    PeelOut* out;     // [record][n_out]: the rays
    uint32_t cap;     // records per region (a multiple of chunk)
    uint32_t chunk;   // records a wave takes at once
    uint32_t* ctl;    // counters a cache line apart: records and dispensed rays per region, parked lanes
    double* park_d;   // lanes that found the regions full: their packets (resumed by the next round)
    uint32_t* park_u;
    int n_lanes;      // lanes of the flight kernel (the same in every round of a launch)
    int resume;       // not the first round
    int scarce;       // fewer records than packets usually need: further rounds are likely
};
constexpr int kPeelCtl = (2 * kXcds + 1) * kCtrStride;
constexpr int kParkD = 10, kParkU = 9;
size_t peel_record_bytes(bool mixed);
void launch_peel_reset(const PeelArgs& q, hipStream_t stream);
void launch_flight(const GridDev& g, const BatchArgs& a, const PeelArgs& q, bool mixed, bool multi, int blocks,
                   hipStream_t stream);
void launch_peel(const GridDev& g, const BatchArgs& a, const PeelArgs& q, bool mixed, bool multi, int blocks,
                 hipStream_t stream);
void launch_peel_sum(const BatchArgs& a, const PeelArgs& q, hipStream_t stream);

// One solve slot of a batched preparation.
struct PrepSlot {
    const double* lnk;  // ck: ln kappa slice [T][P] of (band, g)
    double k_ray;       // Rayleigh opacity at the spectral point
    int n;              // hi-res: table wavelength index
    double lam_cm;      // emission: wavelength of B_lambda
    double* opt;        // FP64 optics: alpha_ext, alpha_abs, omega, P_gas, g (ncell each)
    float* optf;        // FP32 copies (mixed form) or null
    double* cdf;        // emission: L, then q, then the inclusive CDF
    double* wbirth;     // emission: (L_i/L_tot)/q_i
    double* stats;      // emission: (L_tot, N_emit)
};

void launch_prep_optics(const GridDev& g, int ncell, const PrepSlot* slots, int nslots, int hires, int nT,
                        int nP, const double* T_grid, const double* lnP_grid, const double* lnk_tpl, int nlam,
                        const double* shift, int draine, double alpha, hipStream_t stream);
void launch_prep_sources(const GridDev& g, int ncell, const PrepSlot* slots, int nslots, double tau_vert,
                         double xi, double* scratch, hipStream_t stream);
size_t prep_scratch_doubles(int ncell, int nslots);

void launch_slab(const GridDev& g, const BatchArgs& a, bool mixed, int blocks, hipStream_t stream);
void launch_transport_persistent(const GridDev& g, const BatchArgs& a, bool mixed, bool multi, int blocks,
                                 hipStream_t stream);
void launch_reduce_rows(const BatchArgs& a, int n_solves, double* partials, int chunks, double* sums, int sums_w,
                        double* dump, hipStream_t stream);
int reduce_rows_chunks(unsigned long long max_n);
void launch_fill_u64(unsigned long long* p, unsigned long long v, hipStream_t stream);
void launch_init_dispensers(unsigned long long* counters, int stride, unsigned long long total, hipStream_t stream);
void launch_fill_f64(double* p, size_t n, double v, hipStream_t stream);
void launch_births(const GridDev& g, const BatchArgs& a, bool multi, hipStream_t stream);

// Launchers (kernels.hip).  All run on `stream`; none synchronises.
void launch_doppler_shift(const GridDev& g, double ox, double oy, double oz, double dlnlam,
                          double* shift, hipStream_t stream);
// Transmission chords in groups of 16 (chords.hip).  A launch takes the n_group
// groups from g0; their arrays count from there, and a chord's slot in them is
// 16 group + its place in the group.
constexpr uint32_t kChordOver = 0xffffffffu;  // a group with a chord that its strip does not hold
constexpr int kGroupChunk = 64;               // groups of one chunk of the tallies
struct ChordDev {
    int nbg, n_total;            // groups along the impact parameter, in all
    int g0, n_group, n_wave;     // groups of the launch and waves of their walk
    int cap, cap_max;            // steps that a chord's strip holds; steps after which a chord is given up
    int n_flag_words, n_fblk;    // 16-byte words of touched, and their blocks in the scans
    uint32_t* seg_cell;          // [n_wave][cap][64] cell, bit 31: outgoing half
    uint32_t* seg_row;           // ... row within the group, bit 31: the row's first segment
    void* seg_len;               // ... length, FP64 or FP32
    uint32_t* chord_n;           // per chord slot: steps (> cap: more than the strip holds)
    double* chord_b;             // ... weight
    uint32_t* chord_ok;          // ... 0: opaque
    uint8_t* touched;            // per cell: crossed by a chord
    uint32_t* comp;              // per crossed cell: its place among the crossed
    uint2* group_n;              // per group: rows, segments
    uint32_t* group_at;          // ... its first row
    unsigned long long* bsum;    // scan blocks' sums, 3 each
    unsigned long long* totals;  // rows, crossed cells, segments, groups not held
    uint32_t* row_cell;          // per row: place of its cell among the crossed
    void* row_len;               // per row: 16 lengths
};
// W: type in which ln kappa is summed.
template <typename W>
struct CellRow {
    int row[4];  // T, P corners in the table
    W w[4];      // their weights
    double rho, shift;
    float ks, ka;  // cloud scattering and absorption
};
// Slots of an extinction row: the next of 16, 32, 64.
__host__ __device__ inline int chord_stride(int nslot) { return nslot <= 16 ? 16 : nslot <= 32 ? 32 : 64; }
void chord_shape(ChordDev& q, const GridDev& g, int ncell, int n_b, int n_alpha);
void chord_batch(ChordDev& q, int g0, int n_group);
int chord_scan_blocks(const ChordDev& q);
template <typename R>
void launch_chord_geometry(const GridDev& g, int n_b, int n_alpha, uint64_t seed, uint32_t tag, const ChordDev& q,
                           const LimbDark& ld, hipStream_t stream);
template <typename R>
void launch_chord_rows(const ChordDev& q, hipStream_t stream);
template <typename W>
void launch_cell_rows(const GridDev& g, int ncell, const ChordDev& q, bool hires, int nT, int nP, const double* T_grid,
                      const double* lnP_grid, double dlnlam, CellRow<W>* out, hipStream_t stream);
void launch_ck_rows(const double* lnk, int ng_tab, int ntp, const int* specs, int ng, int row0, int nrow, const double* k_ray,
                    double* tab, double* kray_row, hipStream_t stream);
template <typename R, typename W>
void launch_row_alpha(const CellRow<W>* cells, int n_cells, bool hires, const W* tab, int nlam, const double* k_ray,
                      const int* nlist, int nslot, R* alpha, hipStream_t stream);
template <typename R>
void launch_group_tau(const ChordDev& q, const R* alpha, int nslot, double* part, hipStream_t stream);
// The chunks' sums of the part of n_group groups from a chunk's first one.
void launch_group_sums(const double* part, int n_group, int nslot, double* chunks, hipStream_t stream);
void launch_group_final(const double* chunks, int n_chunk, int nrow, double* sums, hipStream_t stream);

}  // namespace mcrt

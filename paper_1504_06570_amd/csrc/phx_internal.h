// Internal layout shared by the host API (phx_api.cpp) and the HIP kernels (phx_trace.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/phx.h"

namespace phx {

constexpr int kNZern = 12;  // Noll Z4..Z15
constexpr int kThreads = 256;   // workgroup size of every trace kernel
constexpr int kSedGuide = 1024;   // guide entries per SED for the wavelength search
constexpr int kNZernPoly = 15;  // monomials u^a v^b, a + b <= 4

// One surface as the kernels read it.  The element frame maps to the global frame by
// g = R q + t (R row-major); kSurfMoved unset means R = identity and t = (0, 0, z_vertex).  The first
// 64 bytes hold what every passage of the optics kernel needs, the next 64 the aspheric
// coefficients: one scalar load each.
enum : uint32_t {
    kSurfMoved = 1u << 0,
    kSurfMirror = 1u << 1,      // reflects (else it refracts; the detector refracts into silicon)
    kSurfGlass = 1u << 2,       // the medium behind it is glass
    kSurfGlassIn = 1u << 3,     // the ray arrives through glass (else vacuum)
    kSurfEven = 1u << 4,        // even aspheric terms only
    kSurfGeneral = 1u << 5,     // an odd aspheric term is present
    kSurfZernike = 1u << 6,
    kSurfPlane = 1u << 7,       // curvature 0 and no aspheric term
};
struct alignas(64) DevSurface {
    uint32_t bits;
    int32_t coating;
    double c, kappa1;      // curvature, 1 + kappa
    double kc2;            // (1 + kappa) c^2
    double r_in2, r_out2;  // squared aperture radii
    double tz;             // t[2]
    const float* coat;     // transmission table of its coating [n_s][n_lam], or null
    double alpha[8];       // alpha_3 .. alpha_10
    double R[9];
    double t[3];
    double r_in, r_out;
    int32_t kind, medium;
    int32_t group;         // rigid-body perturbation group (0 = fixed)
    int32_t pad;
    double z_vertex;       // nominal vertex height (the group transform acts about a pivot)
    double pad2[7];
};
static_assert(sizeof(DevSurface) == 320, "two 64-byte blocks of scalar loads, then the rest");

struct DevSource {
    double xi, eta, nz;
    double lambda_lo, lambda_span, redshift1;
    double sersic_n, sersic_bn, sersic_a, sersic_b, cos_pa, sin_pa;
    int32_t kind, sed;
    uint64_t n_photons;
};

// Per-photon physics beyond the core path, as the kernels use it (derived from phx_physics).
struct DevPhysics {
    double airmass;                  // sec z
    double tau0, gamma;              // aerosol tau = tau0 (lambda / 500 nm)^gamma
    double disp_tanz, disp_cx, disp_cy;  // tan z and the direction of the shift in (n_x, n_y)
    double disp_pt, disp_w;          // Filippenko pressure-temperature factor, water factor
    double disp_b0, disp_s0;         // standard-air bracket and 1/lambda0^2 (um^-2) at lambda0
    double dome_sigma;
    double halo_f, halo_n, halo_r0;
    double halo_e, halo_fq, halo_inv_m;  // 1 - n/2, proposal CDF at x_max, 2^(1 - n/2)
    double dead;
    int32_t vanes, pad;
    double vane_c[8], vane_s[8];     // unit vector of each vane
    double vane_hw, vane_r0, vane_r1, vane_z0, vane_z1, vane_zm, vane_w;
    // second kick: per-layer phase variance above kappa_crit and exp(-variance); the wavenumber
    // CDF through A(kappa) = (kappa^2 + kappa0^2)^(-5/6): A0 = A(kappa_crit), dA = A0 - A(kappa_max)
    double kick_s2[PHX_MAX_LAYERS], kick_p0[PHX_MAX_LAYERS];
    double kick_A0, kick_dA, kick_k02;
    // field diffusion: sigma^2 at depths k dmax / n_sig2 below the entrance, k = 0..n_sig2
    const double* sig2;
    double sig2_inv_step, sig2_dmax;
    int32_t n_sig2, sig2_pad;
};
constexpr int kSig2Cells = 131072;   // cells of 0.75 nm over 98 um: sigma within 2e-14 m

// Everything the trace kernel reads that does not change between launches with the same loads.
struct DevParams {
    int32_t n_surf, nx, ny, n_layers;
    int32_t n_scales, screen_n, n_coat, n_s;
    int32_t n_lam, sed_k, has_glass, pad;
    alignas(64) DevSurface surf[PHX_MAX_SURF];
    double zern[kNZernPoly];   // Zernike deformation of surface 0 as monomial coefficients
    double zern_inv_r;
    double zern_basis[kNZern][kNZernPoly];  // Noll Z4..Z15 as monomial coefficients
    double group_pivot[3][3];
    double group_cs[3][4];     // cos t_x, sin t_x, cos t_y, sin t_y of each group's rotation
    double pupil_r_in, pupil_r_out;
    double z_start, obsc_z, obsc_r;
    double obsc_s;             // smallest s with sqrt(s) >= obsc_r
    double sell_b[3], sell_c[3];
    double chip_x0, chip_y0, pixel;
    double t_si, sigma_max;
    // Rajkanan constants at the device temperature (section 2.4.2)
    double eg[2], egd, absorb[2], emit[2];
    double inv_absorb[2], inv_emit[2];
    // coatings: uniform grid in s = sin^2(theta) and wavelength
    double inv_s_step, lam0, inv_dlam;
    int32_t cull_order[PHX_MAX_SURF]; // coated surfaces, most selective coating first
    // pre-roll escape test per wavelength column: a conversion word at or above esc_thr[il]
    // cannot mean a certain escape (a quick filter; the exact test follows below it); null: off
    const uint32_t* esc_thr;
    int32_t esc_col0;          // first column whose esc_thr is not 0 (n_lam when none)
    int32_t esc_pad;
    int32_t n_cull;
    int32_t ghost_cull_limit;  // first coated refracting surface (n_surf if none): with ghosts the
                               // pre-roll tests only coated surfaces ahead of it
    const float* coat;       // [n_coat][n_s][n_lam]
    const float* coat_r;     // [n_coat][n_s][n_lam] reflection probability (ghosts), or null
    const int64_t* coat_thr; // [n_coat][n_lam]: pre-roll threshold of wavelength column pair
                             // (il, il + 1): the largest roulette word w whose uniform
                             // (w + 1/2) 2^-32 does not exceed the larger of the two columns'
                             // maxima over s (plus 1e-12); -1 when every word exceeds it
    // atmosphere
    double height[PHX_MAX_LAYERS];
    double wind[PHX_MAX_LAYERS][2];
    double inv_pix[PHX_MAX_SCALES];
    double lambda_ref;
    const float4* grad;      // [L][S][N][N][2]: per cell (i, j) the gradients (g_x, g_y) at
                             // (i, j), (i+1, j) then (i, j+1), (i+1, j+1): one 32-byte record
                             // holds a bilinear footprint
    // sources
    const DevSource* src;
    const double* sed_cdf;   // [n_sed][sed_k + 1]
    const double* sed_edges; // [sed_k + 1]
    const uint16_t* sed_guide; // [n_sed][kSedGuide + 1]: guide[j] = the first bin k with
                               // CDF[k + 1] > j / kSedGuide (guide[kSedGuide] = sed_k - 1)
    DevPhysics ph;
};

// Per-launch arguments.
struct Launch {
    uint32_t seed, flags;
    int32_t src_begin, n_src;      // sources [src_begin, src_begin + n_src)
    uint64_t photon_begin;
    uint64_t uniform_count;        // > 0: every source traces this many photons
    const uint64_t* prefix;        // else: exclusive prefix of per-source counts [n_src + 1]
    const int32_t* src_guide;      // with prefix: src_guide[b] = the source holding flattened
                                   // photon b << guide_shift ([blocks + 1], last = n_src - 1)
    uint32_t guide_shift, guide_pad;
    uint64_t total;
    double exposure, pupil_margin;
    uint32_t* image;
    unsigned long long* stats;
    unsigned long long* moments;
    phx_event* events;
    uint64_t event_stride;
    int32_t any_sersic;            // an extended source is in the range
    int32_t any_zernike;           // the first surface carries a Zernike deformation
    // pre-roll geometric cull: a pupil sample at radius r with r^2 < cull_r2_lo or
    // r^2 > cull_r2_hi cannot
    // reach the primary's clear aperture (its atmospheric displacement is bounded)
    double cull_r2_lo, cull_r2_hi;
};

// Scratch of the staged trace: the launch's photon range is processed in chunks; per chunk the
// photons to trace (offsets within the chunk), their number, and the start-plane state of every
// traced photon (kStateFields doubles each, structure of arrays; p_z is the start plane's height).
constexpr uint64_t kChunk = 1ull << 26;
constexpr int kStateFields = 6;
// One chunk of a launch: photons [begin, begin + len) of the flattened launch index, and the order
// in which the photons to trace are listed: as they come, sorted (by pupil sector, by whether they can pass
// the most selective coating, by time; see sort_scatter), or by that class alone.  A chunk inside one source's range names it (src: index relative to
// the launch's first source, first: the flattened index of that source's first photon); src = -1
// for a chunk that spans several sources.
constexpr int kListAsIs = 0, kListSort = 1, kListClass = 2;
struct ChunkSpan {
    uint64_t begin, len, first;
    int32_t sort, src;
};
struct Workspace {
    uint32_t* survivors;       // [buffers][chunk]
    unsigned int* counts;      // [n_chunks]
    uint64_t n_chunks;
    double* state;             // [buffers][kStateFields][chunk]
    uint64_t chunk;
    unsigned long long* tiles; // [n_chunks][2] tile counters of the dynamic schedule
    // sorted chunks only
    uint32_t* seg;             // [buffers][chunk] listed photons of each range, in photon order
    uint32_t* seg_n;           // [buffers][max_ranges(chunk)] photons listed per range
    uint32_t* hist;            // [kSortGroups][kSortKeys] photons per key and sort group, then
                               // their prefixes over the groups; then [kSortKeys] totals
    uint32_t* sect;            // [n_chunks][16]: where each pupil sector's photons start, or
                               // the counter of a list by class
    const ChunkSpan* plan;     // host array: the launch's chunks in order
    uint64_t n_plan;
    int buffers;               // lists and states hold this many chunks (1 or 2)
    double* ghost_list = nullptr;          // [kGhostFields][ghost_cap] ghost starts of a chunk
    uint64_t ghost_cap = 0;                 // (with ghosts: at least ghost_entries)
    unsigned long long* ghost_ctr = nullptr; // [2] entries listed, entries claimed
};
// Photons per pre-roll range (one workgroup's unit): 4096 amortise the range's barriers and keep
// the two stages' lanes full; a small chunk takes smaller ranges so that they cover the compute
// units (the pre-roll of 2e4 photons in 5 ranges of 4096 took 31 us, in 79 of 256 it takes 8).  Whole
// traces of one star with ranges of 256 / 1024 / 4096, in us: 2e4 photons 70 / 72 / 87, 1e5 77 / 77 / 96, 5e5
// 111 / 94 / 108, 6e5 118 / 97 / 110, 2.2e6 220 / 195 / 205, 4e6 330 / 291 / 293, 8e6 575 / 493 / 490.
constexpr int range_log2(uint64_t len) { return len >= (1ull << 22) ? 12 : len >= (1ull << 19) ? 10 : 8; }
constexpr uint64_t range_count(uint64_t len) {
    return (len + (1ull << range_log2(len)) - 1) >> range_log2(len);
}
constexpr uint64_t max_ranges(uint64_t chunk) {
    const uint64_t full = (chunk >> 12) + 1;
    return full > 4096 ? full : 4096;   // 2^22 photons in ranges of 1024
}
// The sort's keys and groups of ranges.
constexpr int kSortKeyBits = 10;         // pupil sector (8) x class (2) x time bucket (64)
constexpr int kSortKeys = 1 << kSortKeyBits;
constexpr uint32_t kSortClass = 64;      // the class bit of a key
constexpr int kSectors = 8;              // one per die
constexpr uint64_t kSortGroups = 512;    // groups at most
// log2 of the ranges per group: at least one for each of a group's eight wavefronts.  Groups of
// 32 ranges left most compute units without one in a chunk of 1e7 photons; more groups than 512 gain
// nothing alone, and beside the optics stage cost 1e8 photons of 1e4 sources 5.75 -> 6.03 ms.
constexpr int sort_group_log2(uint64_t n_ranges) {
    int lg = 3;
    while (((n_ranges + (1ull << lg) - 1) >> lg) > kSortGroups) ++lg;
    return lg;
}
// Workspace of phx_trace_noalloc: a file-scope device array of kScratchBytes on each GPU (its
// address is looked up once per device when a context is created), carved into the buffers of
// one chunk of at most 2^kNoAllocChunkLog2 photons (one buffer set: no pipeline), the per-chunk
// counters of at most kNoAllocMaxChunks chunks, and the prefix table and source guide of at
// most kNoAllocMaxSources sources (built on the device).  Offsets in bytes, each 256-aligned.
constexpr int kNoAllocChunkLog2 = 19;
constexpr uint64_t kNoAllocMaxChunks = 16384;
constexpr int kNoAllocMaxSources = 65536;
constexpr uint64_t kNoAllocGuideMax = 8ull * kNoAllocMaxSources + 2;   // guide blocks + 1
constexpr uint64_t kScratchBytes = 40ull << 20;
struct ScratchLayout {
    uint64_t survivors, state, counts, tiles, prefix, guide, end;
};
constexpr uint64_t align256(uint64_t x) { return (x + 255) & ~uint64_t(255); }
constexpr ScratchLayout scratch_layout() {
    const uint64_t chunk = 1ull << kNoAllocChunkLog2;
    ScratchLayout s{};
    s.survivors = 0;
    s.state = align256(s.survivors + chunk * 4);
    s.counts = align256(s.state + kStateFields * chunk * 8);
    s.tiles = align256(s.counts + kNoAllocMaxChunks * 4);
    s.prefix = align256(s.tiles + 2 * kNoAllocMaxChunks * 8);
    s.guide = align256(s.prefix + (kNoAllocMaxSources + 1) * 8);
    s.end = align256(s.guide + kNoAllocGuideMax * 4);
    return s;
}
static_assert(scratch_layout().end <= kScratchBytes, "no-allocation workspace exceeds the scratch");
// Device address of this GPU's scratch array (the calling thread's current device must be
// `device`); looked up once per device and cached.
hipError_t scratch_address(int device, void** out);
// Exclusive prefix of the photon counts of sources [src_begin, src_begin + n_src) into
// prefix[0 .. n_src] and the photon-block guide (Launch::src_guide) guide[0 .. n_blocks] for
// blocks of 2^shift photons, computed on the device from the source table.
hipError_t launch_prefix(const DevSource* src, int src_begin, int n_src, uint64_t* prefix,
                         int32_t* guide, uint64_t n_blocks, uint32_t shift, hipStream_t stream);

// 8-byte fields of one entry of the ghost list (the optics kernel's ghost starts of a chunk).
constexpr int kGhostFields = 14;

// Second stream and events for pipelining chunks (aux null: everything on the caller's stream).
struct Pipe {
    hipStream_t aux = nullptr;   // pre-roll and optics stages
    hipEvent_t* ev = nullptr;    // at least 3 n_chunks + 1 events
    uint64_t n_ev = 0;
};
// Launch shape (tunable): workgroups of the pre-roll per compute unit, workgroups of the sky and optics
// stages (in fours for the static schedule: stage_groups), and the schedule of the
// sky and optics stages (static grid-stride, or tiles of kTileIters x 256 photons taken from a
// device counter).
struct LaunchConfig {
    int generate_per_cu = 16;
    int front_per_cu = 48;
    int back_per_cu = 2;
    int dynamic = 0;
    int pipeline = 1;
};
constexpr int kTileIters = 8;
// Workgroups of the sky or optics stage per compute unit.  The static schedule takes the setting in fours: by
// default the optics stage then is queued twice as deep as it is resident (4 workgroups per compute
// unit) and the sky stage holds about one tile per workgroup, so that compute units which finish
// early, or share theirs with the other stage, take fewer of them: 1e9 photons 37.2 ms with 4 and 48
// workgroups, 35.5 with 8 and 192; 3e7 without the pre-roll 7.8 and 7.1.  The dynamic schedule takes it as
// it is: its wavefronts balance by their claims, and each workgroup more is an atomic more on the one
// counter, to find the work done (1e6 photons 0.38 ms with fours, 0.32 without; 1e8 on two streams 6.98 and
// 5.55).
constexpr int kGroupsPerUnit = 4;
constexpr int stage_groups(const LaunchConfig& cfg, int per_cu) {
    return cfg.dynamic ? per_cu : kGroupsPerUnit * per_cu;
}
// Workgroups of the optics stage for len photons, in tiles of 256: all of them where each gets two tiles at
// least, else half of them: one tile hardly pays for a workgroup's pixel window, which is cleared and added
// to the image.  All / half / a quarter of 2048, in us: 4.3e5 photons through the paraboloid 40 / 33 / 32,
// 1e6 59 / 48 / 51, 4e6 119 / 113 / 134; 1e6 through the full stack 413 / 386 / 413; 1.8e6 from 441 sources
// through the telescope 251 / 279 / 326.
constexpr uint64_t optics_groups(const LaunchConfig& cfg, int n_cu, uint64_t len) {
    const uint64_t tiles = (len + kThreads - 1) / kThreads, width = (uint64_t)n_cu * cfg.back_per_cu;
    const uint64_t most = (uint64_t)n_cu * stage_groups(cfg, cfg.back_per_cu);
    const uint64_t g = tiles >= 2 * most || most == width ? most : most / 2;
    return g < tiles ? g : tiles;
}
// Flags that select the sky and optics kernels carrying the per-photon physics beyond the core
// path (the other instantiations hold none of its code).
constexpr uint32_t kFrontExtra = PHX_F_DISPERSION | PHX_F_DOME | PHX_F_HALO | PHX_F_SECOND_KICK;
constexpr uint32_t kBackExtra = PHX_F_AEROSOL | PHX_F_SPIDER | PHX_F_GHOSTS;

// Ghost list: a wavefront of the sequential pass with at least kGhostUnits units to trace reserves
// kGhostReserve entries at a time (at least 64), one with fewer the entries that it appends; a
// wavefront of the branch pass takes kGhostClaim at a time, in turn while the list holds at most
// kGhostDealt of them per wavefront, else from a counter (an atomic on one address takes 25 ns, and each of
// the wavefronts needs one to find the list empty: 1e4 photons 395 us with the counter, 229 in
// turn; 3e7 9.8 ms with it, 10.3 in turn, where the branches' lengths balance).  The list holds an entry
// for each photon of a chunk and the entries that the wavefronts leave unused.
constexpr uint64_t kGhostReserve = 128, kGhostUnits = 4, kGhostClaim = 64, kGhostDealt = 4;
constexpr uint64_t ghost_entries(uint64_t chunk, int n_cu, int back_per_cu) {
    const uint64_t launched = (uint64_t)n_cu * kGroupsPerUnit * back_per_cu * (kThreads / 64);   // at most
    const uint64_t filled = chunk / 64 + kThreads / 64;   // no more workgroups than units of work
    return chunk + kGhostReserve * (launched < filled ? launched : filled);
}

// Optional per-kernel timing: events recorded before/after each kernel launch.
struct Timing {
    bool on = false;
    // event pairs per kernel kind (0 generate, 1 front, 2 back, 3 the sort),
    // appended per chunk
    void (*record)(void* self, int kind, int edge, hipStream_t stream) = nullptr;
    void* self = nullptr;
};

hipError_t launch_trace(const DevParams* dparams, const Launch& L, const Workspace& W, int n_cu,
                        const LaunchConfig& cfg, hipStream_t stream, const Pipe& pipe,
                        const Timing& T);
// Adjoint of the per-source moments (pathwise derivative, decisions frozen).  Per-lane
// accumulators: the ten rigid-body parameters, then the fifteen monomial coefficients of the
// primary's deformation (mapped to Zernike amplitudes by the final reduction).
constexpr int kAdj = 10 + kNZernPoly;
constexpr int kTapeFields = 7;   // per surface: hit point (3), incoming direction (3), path length
struct Adjoint {
    const double* seed;      // [n_src][8]: gx, gy, gxx, gyy, gxy, mean x, mean y, unused
    double* partial;         // [rows][kAdj], one row per (chunk, workgroup)
    double* tape;            // [n_surf * kTapeFields][tape_stride]
    uint64_t tape_stride;    // threads of one adjoint launch
    double* jac;             // optional [slots][2][PHX_N_THETA]
    uint64_t jac_stride, jac_cap;
    int per_cu;              // workgroups per compute unit of the adjoint kernel
};

hipError_t launch_adjoint(const DevParams* dparams, const Launch& L, const Workspace& W, int n_cu,
                          const LaunchConfig& cfg, const Adjoint& A, double* colsum, double* grad,
                          hipStream_t stream, const Pipe& pipe, const Timing& T);
// One readout of a sensor image (phx_readout): parameters, the input electrons and the
// buffers of each step (device pointers).
struct ReadoutThr {
    uint32_t a0, a1;    // a draw's word above a0 is a delay, above a1 one of two slots or more
    double p0;          // probability of no delay
};
struct ReadoutJob {
    phx_readout_params p;
    const uint32_t* in;
    int32_t nx, ny;
    uint32_t* work;     // [ny][nx] after bleeding, dark current and defects
    uint32_t* par;      // [amp][sh + over_y][sw] after the parallel transfers
    uint32_t* ser;      // [amp][sh + over_y][sw + over_x] after the serial transfers
    uint16_t* out;      // [amp][sh + over_y][sw + over_x] ADU
    uint32_t* heavy;    // packets with many electrons, handled by whole wavefronts
                        // [max(ny nx, amp (sh + over_y) sw)]
    uint32_t* heavy_count;   // [2] of the parallel and the serial transfers
    ReadoutThr* thr;    // [sh + sw] of the transfer counts 1..sh (parallel) and 1..sw (serial)
};
hipError_t launch_readout(const ReadoutJob& J, hipStream_t stream);

// Per-source (n, mean x, mean y, Ixx, Iyy, Ixy) from moment words [n_src][PHX_MOMENT_WORDS]
// into out [n_src][6], each rounded once from exact integer arithmetic (phx_moments).
hipError_t launch_moments(const unsigned long long* words, int n_src, double* out,
                          hipStream_t stream);
// The adjoint's cotangent coefficients [n_src][8] from the moment words and a loss gradient
// dmom [n_src][5] with respect to (mean x, mean y, Ixx, Iyy, Ixy).
hipError_t launch_seeds(const unsigned long long* words, int n_src, const double* dmom,
                        double* seed, hipStream_t stream);

hipError_t launch_gradients(const float* opd, float4* grad, int n_layers, int n_scales, int n,
                            const double* pixel, unsigned int* gmax, hipStream_t stream);

}  // namespace phx

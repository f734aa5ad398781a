// Internal plan object of the collision library and the device launch interface.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "dgfs.h"

namespace dgfs {

// Launch geometry of the fused gain kernel for one velocity resolution N:
// CH   chunks of the output grid along x (each work item owns x-indices = c mod CH),
// CZ   thread groups sharing each y/z pencil of the chunk (group g keeps the outputs
//      with index = g mod CZ); CZ = 0: the shifted fields are formed on the matrix cores
//      (gain_mfma.hip).
struct GainGeometry {
    int CH;
    int CZ;
};

// The default: the first compiled geometry, skipping the matrix-core ones (CZ = 0: FP32
// VHS plans of the circular form) unless matrix_ok.
bool gain_geometry(int N, int precision, GainGeometry* g, bool matrix_ok = true);
// A call of few nodes spreads the directions of its gain items over the chip, one
// workgroup per (item, direction), and sums them in a second kernel (gain.hpp).  An item runs
// its class's directions one after the other, so a call whose items do not fill the chip takes
// the longest class's time whatever its size; the split takes the time of all directions over
// the chip, about 1.5 times theirs in full rounds (no kept x-transforms, and the terms, one
// value per point and direction, go through memory).  So what counts is the call's items in
// units of the longest class's, n = nb nrho CH dirs / longest, against the workgroups that the
// chip runs together: `most` is where the two forms cost the same.  With one workgroup per CU
// (`single`) the unsplit form takes whole rounds of 256, and just past the first one the split
// is ahead again, up to 2 most.  Calls in us, together / split, by n (one species, M = 12 unless
// said; two species have classes of two lengths):
//   FP32 N = 16 (1,1): 248 51/44, 448 60/59, 848 84/88; two species 560 119/108, 672 122/121;
//     M = 24 600 198/184, 848 229/254, 1000 233/293;
//   FP32 N = 24 (3,1): 288 83/66, 612 107/100, 684 108/108, 864 116/126; two species 576 175/157;
//     M = 24 612 322/299, 864 347/393;  (3,2): 360 76/75, 504 79/90, 612 110/103, 864 133/132,
//     two species 576 175/166;  (3,4): 360 84/83, 504 87/101;  (3,3): 360 110/88, 864 201/166;
//     (1,1) single: 204 115/114, 252 118/131, 300 202/168, 504 208/236;
//   FP32 N = 32 (2,1) single: 96 118/95, 160 121/115, 192 123/132, 256 126/152, 288 211/180,
//     384 211/217; two species 128 208/164, 192 216/219, 256 221/271; M = 24 160 365/323,
//     256 370/490;  (4,1): 320 134/121, 384 135/134, 448 137/149;  (4,2): 384 170/131;
//   FP64 N = 16 (1,1): 200 66/61, 352 89/88, 400 89/94; two species 272 129/116, 336 130/135;
//     M = 24 304 253/216, 400 255/276;
//   FP64 N = 24 (3,2) single: 108 77/69, 144 79/77, 216 81/97, 288 136/120, 360 139/141; two
//     species 144 127/118, 216 142/160; M = 24 144 202/193, 216 204/263;
//   FP64 N = 32 (4,2) single: 128 127/103, 192 137/136, 256 139/157, 320 234/200, 448 233/253;
//     two species 128 232/174, 256 248/277; M = 24 128 351/278, 192 366/403, 320 702/627.
// Above N = 32 the split is not compiled: a two-species node fills the chip (N = 48: 432 items at
// 24 radial points; N = 64: 16 or 32 chunks of each), one species at N = 48 does not (72 to 150
// items) and runs its directions one after the other.
struct SplitRule {
    int most;
    bool single;
};
inline SplitRule split_rule(int N, int precision, const GainGeometry& geo) {
    const int g = 10 * geo.CH + geo.CZ;
    if (N > 32 || geo.CZ == 0) return {0, false};
    if (precision != 0) return N == 16 ? SplitRule{320, false} : N == 24 ? SplitRule{150, true} : SplitRule{192, true};
    if (N == 16) return {g == 11 ? 600 : g == 21 ? 900 : 960, false};
    if (N == 24) return g == 11 ? SplitRule{240, true} : SplitRule{g == 34 ? 380 : g == 33 ? 960 : 640, false};
    return g == 21 ? SplitRule{160, true} : SplitRule{400, false};
}
// The most bytes of terms held at once: a call with more spreads the radial points in groups,
// one pair of launches each, of as many as fit.  Each group still has more workgroups than the
// chip runs together (256 MiB are 1024 FP64 or 2048 FP32 fields at N = 32), so the groups cost
// launches alone: three FP64 nodes at N = 32, M = 24 (302 MB) 400 us in one group, 392 in two;
// 17 FP32 nodes at N = 24, M = 24 (271 MB) 287 and 294 us.
constexpr size_t split_bytes = size_t(256) << 20;
// Bytes per (node, species) of the matrix-core gain's prepared input (N = 32): f split into
// FP16 hi and lo, the alternating x-sum plane split likewise, and 64 FP32 scalars.
constexpr size_t mfma_prep_bytes = (2 * 32768 + 2048) * 2 + 64 * 4;
int tile_candidates(int N, int precision, GainGeometry* out, int max);  // compiled geometries

// One "gain class": the S_q field sum_p w A_p B_p with A = f^i shifted by +a rho sigma_p,
// B = f^j shifted by -b rho sigma_p.  With an antipodal design one class serves both
// orderings of an unlike pair, and a like pair needs only half of the directions.
//
// With a VSS kernel the kernel mode depends on sigma, so the directions are not summed:
// a class holds one direction, whose complex product S is transformed whole, and the
// sphere weight goes into the kernel-mode tables.
struct GainClass {
    int i, j;
    double a, b;
    int ndir;        // directions of this class
    int dir_offset;  // first global direction index in the phase tables
    double weight;   // sphere weight per direction (4 pi / M, doubled for a halved like pair; 1 for VSS)
    std::vector<int> dirs;  // design point of each direction
};

struct PairParams {
    double a, b, gamma, C, R, alpha;
    std::vector<double> rho, wrho;
};

// Device-side integer descriptors (all int32):
//   class:  i, j, ndir, dir_offset
//   slot:   species, gain_begin, gain_count, loss_begin, loss_count
//   gain term: class, F table
//   loss term: species j, G table
struct SlotSet {
    int nslots = 0;
    std::vector<int> slots, gterms, lterms;
    std::vector<int> cuses;  // per class: (slot, F table) of its first and second use, -1 if none
    size_t off_slots = 0, off_gterms = 0, off_lterms = 0, off_cuses = 0;  // byte offsets in the device block
};

}  // namespace dgfs

struct dgfs_plan {
    int s = 0, N = 0, M = 0, nrho = 0, precision = 0;
    double L = 0;               // box half-width (the widest box with species-specific grids)
    std::vector<double> mass;
    std::vector<double> Ls;     // [s] half-width of each species' grid
    std::vector<unsigned char> mask;  // [s*s] ordered pairs evaluated by this plan
    dgfs::GainGeometry geo{};
    std::vector<double> sigma;  // design, [M][3]
    bool antipodal = false;
    bool vss = false;           // some pair has alpha > 1: sigma-dependent kernel-mode tables
    std::vector<dgfs::PairParams> pair;  // [s*s]
    std::vector<dgfs::GainClass> classes;
    int total_dirs = 0, fresh_dirs = 0;  // fresh: with another sigma_x than the one before in its class
    int nftab = 0, ngtab = 0, K2 = 0;
    dgfs::SlotSet sum_slots, pair_slots;

    int device = 0;
    void* dev = nullptr;  // one block holding every table
    size_t dev_bytes = 0;
    // byte offsets of the tables in `dev`
    size_t off_kx = 0, off_yz = 0, off_nyq = 0, off_F = 0, off_G = 0, off_tw = 0, off_cls = 0, off_wdir = 0, off_ord = 0, off_xs = 0;
    // matrix-core gain (geometry CZ = 0): split-FP16 shift-matrix operands and Nyquist
    // coefficients per (direction, rho, field)
    size_t off_mtab = 0, off_msc = 0;
    size_t off_minv = 0;  // (s+4)^2 doubles, inverse Gram matrix of the invariants
    // plain per-point FP64 path (FP64 plans only): phases [s*s][nrho][M][2][3][N], F [s*s][nrho][K2]
    size_t off_plain_ph = 0, off_plain_F = 0;

    // Species-specific grids: one single-grid sub-plan per distinct pair box L_ij, each
    // evaluating the ordered pairs whose wider box it is.  Empty for a single-grid plan.
    struct GridPart {
        dgfs_plan* plan = nullptr;
        double L = 0;
        std::vector<int> species;         // global index of each local species
        std::vector<long long> t_in;      // byte offset in `dev` of the map own grid -> L, or -1
        std::vector<long long> t_out;     // byte offset in `dev` of the map L -> own grid, or -1
    };
    std::vector<GridPart> parts;

    // Dealiased form (linear convolution): the companion plan on the 3N/2 grid whose
    // tables the padded gain and loss use; this plan keeps the conservation tables.
    dgfs_plan* inner = nullptr;

    size_t elem() const { return precision == DGFS_FP64 ? sizeof(double) : sizeof(float); }
    size_t n3() const { return size_t(N) * N * N; }
    // workspace bytes per node, and the alignment slack added once per call
    size_t ws_per_node(bool pairs) const;
    size_t ws_slack() const { return parts.empty() ? 4 * 256 : 12 * 256; }
    // what a pass over `batch` nodes needs in either mode, and the plain FP64 path for one node
    size_t ws_required(int64_t batch) const;
    // bytes beyond those with which a call of nb nodes spreads its gain directions over the
    // chip (gain.hpp), at most dgfs::split_bytes; 0 where it does not
    size_t ws_split(int64_t nb) const;
    // bytes beyond ws_required(batch) with which every call of up to `batch` nodes finds room
    // for that
    size_t ws_spread(int64_t batch) const;
};

namespace dgfs {
// Device memory of a call: at least ws_per_node() per node (and the alignment slack), and
// what the caller gave beyond that.
struct Scratch {
    void* p;
    size_t bytes;
};
// Launch the full collide pipeline for nb nodes on `stream`.
// ev: NULL, or 6 events recorded at the stage boundaries of the slice.
hipError_t launch_collide(const dgfs_plan& p, const void* f, void* Q, int64_t nb, Scratch ws,
                          bool pairs, hipStream_t stream, hipEvent_t* ev);
// The dealiased pipeline (vss_24.hip: N = 16, dealias_36.hip: N = 24, vss_48.hip: N = 32,
// dealias_72.hip: N = 48).
hipError_t run_dealias_16(const dgfs_plan& outer, const dgfs_plan& inner, const void* f, void* Q, int nb, void* ws,
                          bool pairs, hipStream_t st, hipEvent_t* ev);
hipError_t run_dealias_24(const dgfs_plan& outer, const dgfs_plan& inner, const void* f, void* Q, int nb, void* ws,
                          bool pairs, hipStream_t st, hipEvent_t* ev);
hipError_t run_dealias_32(const dgfs_plan& outer, const dgfs_plan& inner, const void* f, void* Q, int nb, void* ws,
                          bool pairs, hipStream_t st, hipEvent_t* ev);
hipError_t run_dealias_48(const dgfs_plan& outer, const dgfs_plan& inner, const void* f, void* Q, int nb, void* ws,
                          bool pairs, hipStream_t st, hipEvent_t* ev);
// out != NULL: out = projection of Q (FP64); fstate != NULL: fstate += dt * projection.
hipError_t launch_conserve(const dgfs_plan& p, const void* Q, double* out, void* fstate, double dt, int64_t nb,
                           hipStream_t stream);
// Copy (Tm == NULL) or interpolate (Tm = [N][N] one-dimensional map, applied along each
// axis) nb fields of N^3 values with per-node strides (in elements), storing or adding.
// tmp: 2 nb N^3 values of scratch.
hipError_t launch_move(const dgfs_plan& p, const void* in, int64_t in_stride, void* out, int64_t out_stride,
                       const void* Tm, int64_t nb, bool accumulate, void* tmp, hipStream_t stream);
// out = a x + b y over n values of the plan precision.
hipError_t launch_axpby(const dgfs_plan& p, const void* x, const void* y, void* out, double a, double b, int64_t n,
                        hipStream_t stream);
// Workspace bytes per node of the dealiased pipeline on an N-grid plan (NI = 3N/2):
// f_hat on N, the padded f_hat and the complex interpolant on NI, the class partials on
// NI, the loss spectra on NI and the kept modes on N.
inline size_t dealias_ws_per_node(size_t elem, int N, int s, int ncls, int nrho, int nslots) {
    const size_t c = 2 * elem, N3 = size_t(N) * N * N, NI = size_t(3 * N / 2), NI3 = NI * NI * NI;
    return c * (size_t(s) * N3 + 2 * size_t(s) * NI3 + size_t(ncls) * nrho * NI3 + size_t(nslots) * NI3 +
                size_t(nslots) * N3) + 7 * 256;
}
// dgfs_collide with the caller's workspace (api.cpp): the batch runs in slices of as many
// nodes as ws_bytes holds.
dgfs_status collide_with_workspace(const dgfs_plan* plan, const void* f, void* Q, int64_t batch, void* ws,
                                   size_t ws_bytes, void* stream);
// Record the error text returned by dgfs_last_error and return st (api.cpp).
dgfs_status set_error(dgfs_status st, const std::string& msg);
// Plain per-point FP64 path (plain.hip).
size_t plain_ws_bytes(const dgfs_plan& p);
hipError_t launch_collide_plain(const dgfs_plan& p, const double* f, double* Q, int64_t nb, void* ws,
                                hipStream_t stream);
}  // namespace dgfs

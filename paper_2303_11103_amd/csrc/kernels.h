// Launch interface between the C ABI (api.hip) and the kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "device.h"
#include "layout.h"

namespace rt {

constexpr int kTraceBlock = 512;  // block size of the shoot-and-bounce kernels
constexpr uint64_t kEmptyKey = ~0ull;
constexpr int kQueueRegions = 64;
// The region counters sit 64 bytes apart: every wave's append is a
// device-scope atomic performed past the L2, and counters that share a line
// contend with each other.
constexpr int kCounterStride = 16;  // 32-bit words between two region counters

struct DevScene {
    const Node* nodes;
    const Tri* tris;
    const Shade* shades;
    const Face* faces;
    const int32_t* face_tris;
    int32_t num_faces;
    int32_t nt;
    int32_t num_nodes;
    int32_t stack_need;  // worst-case traversal stack entries of the tree
    const int32_t* leaf_of_input;  // [nt] leaf-order index of each input triangle
    const Wedge* wedges;           // [num_wedges] diffraction wedges
    int32_t num_wedges;
};

struct SbrArgs {
    DevScene sc;
    int64_t num_rays;   // lattice size N
    int64_t begin, stride;
    int64_t count;      // traced rays (positions 0..count-1)
    int64_t pos0, chunk; // positions handled by this launch sequence: [pos0, pos0 + chunk)
    Bands perm;         // order of the positions
    double tmin;
    uint64_t scat_seed;  // SplitMix64 seed of the diffuse-scattering draws
    double tx[3];
    Antenna tx_ant, rx_ant;
    // coverage
    double gx0, gy0, gcell, gz;
    int32_t gnx, gny;
    float wscale;       // (lambda/4pi)^2 (4pi/N) / cell^2
    float* gain;
    uint32_t* hits;
    int32_t merge;      // the first two bounces merge a wave's deposits per cell
    // queues
    int32_t depth, max_depth;
    // The queues are split into kQueueRegions regions of region_cap rays; a
    // wave appends its survivors to region (wave % kQueueRegions) through
    // that region's counter, which spreads the queue atomics over 64 addresses.
    const void* in;
    // [kQueueRegions * kCounterStride]: word 0 of a region counts its rays, word 1
    // the rays its waves dropped before a last bounce (they add to the depth's count)
    const uint32_t* in_count;
    void* out;
    uint32_t* out_count;        // [kQueueRegions * kCounterStride]
    int64_t region_cap;
    uint64_t* stats;    // [max_depth + 1] traced rays per depth (nullable)
    uint64_t* work;     // stats mode: [4][max_depth + 1] rays, inner-node visits, child-box tests, triangle tests
    // record mode
    int32_t* rec_tri;
    double* rec_t;
    // candidate mode
    uint64_t* table;
    uint64_t table_mask;
    uint32_t* overflow;
    // reception-sphere mode: receivers binned on an xy grid (each receiver in
    // every cell within r_ins of it, CSR lists), the heights they span widened
    // by r_ins, and the set of (receiver, prefix slot) pairs
    const double* rx;            // [nrx][3]
    const int32_t* cell_start;   // [rnx * rny + 1]
    const int32_t* cell_rx;
    double rgx0, rgy0, rgcell;
    int32_t rgnx, rgny;
    double rz_lo, rz_hi, rx_zmin, rx_zmax;  // the receivers' heights with and without r_ins
    double sphere_k;             // kappa sqrt(4 pi / N): sphere radius per metre of path
    uint64_t* pairs;
    uint64_t pairs_mask;
    uint32_t* pairs_overflow;
};

// kModeSphere: rays carry their face sequence and path length; segments after
// the first reflection record (receiver, sequence) pairs within the spheres.
enum : int { kModeCoverage = 1, kModeRecord = 2, kModeCandidates = 4, kModeStats = 8, kModeSphere = 16 };
// Bytes of a live ray's queue record between two bounces, read and written
// coalesced by consecutive lanes.  All hold o[3], d[3] (fp64), then
//   maps: E[6] (complex field per axis), face of the last reflection, lattice
//     position j (ray index = begin + j stride): 80;
//   records, candidates: face of the last reflection, prefix-table slot of the
//     face sequence (-1 none), j, padding: 64;
//   reception spheres: path length (float), the face sequence at 24 bits a face
//     (its last is the face of the last reflection): 64, with a fifth face 80.
// With 96 bytes and the field's arithmetic in every mode, the paths of 10^8
// rays through a city took 28.3 instead of 26.6 ms and the gradient of a map of
// 10^7 rays 1.44 instead of 1.34 ms; a map of 10^8 rays of the city takes 21.9
// ms with 96 bytes and 21.2 with 80.
__host__ __device__ constexpr int64_t sbr_ray_bytes(int mode, int faces) {
    return (mode & kModeCoverage) || ((mode & kModeSphere) && faces > 4) ? 80 : 64;
}
constexpr int kSphereMaxDepth = 5;       // faces packed 24 bits each into 128 bits
constexpr int32_t kSphereMaxFaces = 1 << 24;

// Rays one queue region must hold for a bounce launch of `grid` blocks over
// at most `chunk` rays: the waves of a region (every kQueueRegions-th) times
// their grid-stride iterations times 64 lanes.
int64_t sbr_region_capacity(int64_t chunk, int grid);
hipError_t launch_sbr_bounce(const SbrArgs& a, const MatTable& mats, int mode, int grid, hipStream_t s);
hipError_t launch_fib_dirs(int64_t N, int64_t begin, int64_t stride, int64_t count, double* out, hipStream_t s);
hipError_t launch_finalize_db(const float* gain, float* db, int64_t n, hipStream_t s);
// Zeroes p[k][0 .. words[k]) (32-bit words) of all arrays in one launch.
struct ClearArgs {
    void* p[4];
    int64_t words[4];
};
hipError_t launch_clear(const ClearArgs& a, hipStream_t s);
// p[0 .. n) = v (32-bit words), as a kernel (usable inside captured graphs).
hipError_t launch_fill_u32(void* p, uint32_t v, size_t n, hipStream_t s);

// ---------------------------------------------------------------- paths
struct Cand {
    int32_t depth;
    int32_t faces[8];
};

struct PathArgs {
    DevScene sc;
    double freq, lambda;
    double tx[3];
    Antenna tx_ant;
    const double* rx;        // [nrx][3]
    const Antenna* rx_ant;   // [nrx]
    int32_t nrx;
    const Cand* cands;
    const uint32_t* ncand;   // device count
    const int32_t* pair_rx;  // reception-sphere mode: receiver of candidate j (null: every receiver)
    int32_t max_depth;
    int32_t P;               // slots per rx
    uint32_t* counts;        // [nrx] paths found
    // unsorted path records
    float* a;      // [nrx][P][2]
    float* T;      // [nrx][P][8]
    float* tau;    // [nrx][P]
    float* aod;    // [nrx][P][2]
    float* aoa;    // [nrx][P][2]
    int32_t* depth;   // [nrx][P]
    int32_t* faces;   // [nrx][P][FD]
    int32_t fd;       // faces stride = max(max_depth, 1)
};

hipError_t launch_paths_power(const float* a, const int32_t* depth, int64_t n, int P, double* power, hipStream_t s);
hipError_t launch_extract_pairs(const uint64_t* pairs, uint64_t pairs_cap, const uint64_t* table, Cand* out,
                                int32_t* out_rx, uint32_t* count, uint32_t max_out, hipStream_t s);
hipError_t launch_extract_candidates(const uint64_t* table, uint64_t cap, int32_t max_depth, Cand* out,
                                     uint32_t* count, uint32_t max_out, hipStream_t s);
// Image method over `items` (receiver, candidate) pairs, `chunk` at a time (all of
// a chunk may have a path); scratch: image_scratch(chunk) bytes.
constexpr int64_t kImageChunk = int64_t(1) << 22;
size_t image_scratch(int64_t chunk);
hipError_t launch_image_paths(const PathArgs& a, const MatTable& mats, int64_t items, int64_t chunk, void* scratch,
                              hipStream_t s);
// First-order diffraction: the valid (receiver, wedge) paths into the unsorted
// records of a (depth = 1, faces[0] = wedge id, fd = 1).  `chunk` receivers at a
// time, their pairs at most `most` (or one receiver's), in two queues: pairs that
// pass the filter and pairs whose legs are clear.  For street receivers of a city
// 2% and 1 in 8,000 do, of a street canyon 16% pass the filter, so beyond
// kDiffWholePairs pairs the queues have room for a quarter and an eighth (200 MB
// for 2^27 pairs, where all would take 1.07 GB; smaller chunks cost a launch's
// tail each: 1024 receivers x 129,768 wedges at 2^27, 2^26, 2^25 pairs 0.96, 1.12,
// 1.37 ms).  If that does not do, some receiver's count is 2^31: the paths are not
// whole, and the plan diffraction_sure has room for every pair.
constexpr int64_t kDiffQueuePairs = int64_t(1) << 27, kDiffWholePairs = int64_t(1) << 22;
struct DiffPlan {
    int64_t chunk, filtered, clear;
};
DiffPlan diffraction_plan(int64_t nrx, int64_t num_wedges, int64_t most);
DiffPlan diffraction_sure(const DiffPlan& p, int64_t num_wedges);
size_t diffraction_scratch(const DiffPlan& p);
hipError_t launch_diffraction_paths(const PathArgs& a, const MatTable& mats, const DiffPlan& plan, void* scratch,
                                    hipStream_t s);
// Diffraction part of a coverage map: gain[c] += sum over wedges of |a|^2 of the
// diffracted path from tx to the centre of cell c (one thread per cell).
hipError_t launch_coverage_diffraction(const DevScene& sc, const MatTable& mats, double lambda, const double* tx,
                                      const Antenna& txa, const Antenna& rxa, double gx0, double gy0, double gcell,
                                      double gz, int32_t gnx, int32_t gny, float* gain, hipStream_t s);
hipError_t launch_sort_paths(const PathArgs& a, int32_t nrx, float* a_out, float* T_out, float* tau_out,
                             float* aod_out, float* aoa_out, int32_t* depth_out, int32_t* faces_out,
                             int32_t* num_paths_out, hipStream_t s);

// Diffusely scattered paths: scattering points of a chunk of lattice rays,
// [ray][depth] (128 bytes).
struct alignas(16) ScatPoint {
    double p[3];    // the hit point
    double n[3];    // unit normal facing the incident ray
    double g[8];    // 2x2 complex G: (perp, par) from departure (theta, phi), times S w r_{perp,par}
    double s;       // ray length from the transmitter
    double pad;
};
static_assert(sizeof(ScatPoint) == 128, "scattering point size");

// What the visibility test needs of a scattering hit (64 bytes).
struct alignas(16) ScatHit {
    double p[3], n[3];
    int32_t face;
    int32_t rec;    // its record, ray * max_depth + depth
    int32_t pad[2];
};
static_assert(sizeof(ScatHit) == 64, "scattering hit size");

struct ScatArgs {
    Bands perm;          // order in which a chunk's rays are traced
    DevScene sc;
    int64_t num_rays, begin, stride;
    int64_t pos0, n;          // lattice positions [pos0, pos0 + n) of this chunk
    int32_t max_depth, nrx;
    double tmin, lambda;
    double tx[3];
    Antenna tx_ant;
    const double* rx;         // [nrx][3]
    const Antenna* rx_ant;    // [nrx]
    ScatPoint* points;        // [n][max_depth], written where the hit scatters
    int32_t* hit;             // [n][max_depth] 2 face + (1 where S > 0), -1: no hit
    ScatHit* hits;            // [n * max_depth] dense list of the scattering hits
    uint32_t* num_hits;       // its length
    int64_t nrec_pad;         // n * max_depth rounded up to a multiple of 64
    uint64_t* masks;          // [nrx][nrec_pad / 64] visibility bits
    uint32_t* prefix;         // [nrx][nrec_pad / 64] visible records before each word (this chunk)
    int64_t* first;           // [nrx] paths of the earlier chunks
    int64_t* base;            // [nrx] paths so far (after the last chunk: the counts)
    int64_t P;                // slots per receiver
    float* a;                 // [nrx][P][2]
    float* T;                 // [nrx][P][8]
    float* tau;               // [nrx][P]
    float* aod;               // [nrx][P][2]
    float* aoa;               // [nrx][P][2]
    int32_t* depth;           // [nrx][P]
    int64_t* ray;             // [nrx][P]
    int32_t* faces;           // [nrx][P][fd]
    int32_t fd;               // max_depth
};
// All passes of one chunk; base must hold the counts of the earlier chunks (zero
// before the first).
hipError_t launch_scatter_chunk(const ScatArgs& a, const MatTable& mats, hipStream_t s);
// Empty-slot values for the slots at or after every receiver's final count.
hipError_t launch_scatter_tail(const ScatArgs& a, hipStream_t s);

struct GradArgs {
    DevScene sc;
    double freq, lambda;
    double tx[3];
    double yaw, pitch, roll;
    int32_t tx_pattern, tx_pol;
    const double* rx;
    const Antenna* rx_ant;
    int32_t nrx, P, fd;
    const int32_t* depth;   // [nrx][P]
    const int32_t* faces;   // [nrx][P][fd]
    const double* dL_dP;    // [nrx] (used when coef_adj is null)
    const double* coef_adj; // [nrx][P][2] complex adjoint g of each path's coefficient (nullable)
    double* grad;           // [2 nm + 5]
    int32_t nm;
};
hipError_t launch_power_grad(const GradArgs& a, const MatTable& mats, hipStream_t s);

// Channel frequency responses of paths (synthetic arrays, Doppler, OFDM).
struct CfrArgs {
    int64_t npairs;           // ntx * nrx
    int32_t nrx, P;
    const float* a;           // [npairs][P][2]
    const float* tau;         // [npairs][P]
    const float* aod;         // [npairs][P][2] (theta, phi)
    const float* aoa;
    const int32_t* depth;     // [npairs][P], < 0 for an empty slot
    double freq, lambda, spacing, fs;
    int32_t K, T, nt_el, nr_el;
    const double* tx_el;      // [nt_el][3] element offsets [m] (dev)
    const double* rx_el;      // [nr_el][3]
    const double* v_tx;       // [ntx][3] velocities [m/s] (dev)
    const double* v_rx;       // [nrx][3]
    float* H;                 // [npairs][T][nr_el][nt_el][K][2]
    int64_t total;            // entries of H
};
hipError_t launch_cfr(const CfrArgs& c, hipStream_t s);
// scratch: cfr_adjoint_scratch(c) bytes of partial sums, 16-byte aligned; without,
// a kernel that needs none (a sine per output and path).
size_t cfr_adjoint_scratch(const CfrArgs& c);
hipError_t launch_cfr_adjoint(const CfrArgs& c, const float* G, double* g, void* scratch, hipStream_t s);

// Coverage-map gradient: replay of recorded rays with field tangents.
constexpr int kCovMaxMat = 4;                 // materials with tangents
struct CovGradArgs {
    DevScene sc;
    int64_t num_rays, begin, stride, count;
    int32_t max_depth;
    int32_t nm;
    int32_t scatters;         // some material has diffuse reflections
    double tx[3];
    double R[9], Ryaw[9], Rpitch[9];  // tx orientation and its derivatives
    int32_t tx_pattern, tx_pol;
    int32_t gnx, gny;
    Antenna rx_ant;
    double gx0, gy0, gcell, gz;
    double wscale;            // (lambda/4pi)^2 (4pi/N) / cell^2
    double omega;             // 2 pi f
    uint64_t scat_seed;       // draws of diffuse scattering (as in the forward kernel)
    const uint8_t* region;    // [gny][gnx] (nullable: every cell)
    const int32_t* hit_tri;   // [max_depth+1][count] input triangle ids (-1 miss, -2 terminated)
    const double* hit_t;      // [max_depth+1][count]
    double* out;              // [2 nm + 3]: region sum, d/d(eps_r, sigma) per material, d/d yaw, d/d pitch
};
// Rays taken at a time, and the device memory their queue needs (all may be
// marked: 8 bytes a ray, 134 MB at most; 10^7 rays in chunks of 2^22 take 288
// instead of 259 us).  Without scratch, one kernel that needs none (and no chunks).
constexpr int64_t kCovChunk = int64_t(1) << 24;
size_t coverage_grad_scratch(int64_t rays, int num_cu);
hipError_t launch_coverage_grad(const CovGradArgs& a, const MatTable& mats, int num_cu, int64_t chunk, void* scratch,
                                hipStream_t s);

}  // namespace rt

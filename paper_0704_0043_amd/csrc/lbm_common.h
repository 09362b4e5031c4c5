// Structures shared by the host runtime (lbm.cpp) and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm.h"

namespace lbm {

enum { kD1Q3 = 1, kD2Q9 = 2 };
enum { kPoly = 0, kEntropic = 1 };
// Delta S form of a kernel; kExactHom: exact, with the exact homothety in some
// domain (the root solve's registers would halve the occupancy of the others)
enum { kExact = 0, kQuad = 1, kExactHom = 2 };
enum { kPeriodic = 0, kCavity = 1, kTube = 2 };
enum { kLimTrim = 1, kLimMedian = 2, kLimEnsThresh = 4, kLimEnsSmooth = 8, kLimEnsRational = 16,
       kLimEnsBudget = 32, kLimPos = 64,
       // internal: trimming limited to the top_k largest Delta S' (a second-pass
       // limiter; the domain's kLimTrim bit is cleared on the device)
       kLimTopK = 128, kLimEns = 4 | 8 | 16 | 32 | 128 };
enum { kLBGK = 0, kELBM = 1 };
enum { kF64 = 0, kF32 = 1, kF16 = 2, kBF16 = 3 };

enum : unsigned { kMaskTrim = 1, kMaskMedian = 2, kMaskNonpos = 4, kMaskNotFluid = 8, kMaskEns = 16, kMaskPos = 32 };
// kFlagAllTiles makes the second pass walk every tile, as if each had a
// candidate; only the tuner sets it, to time that pass's full work.
// kFlagStats: the step's sums will be read (the last step of a captured
// sequence or of a call, and every step with an ensemble-dependent limiter).
enum : unsigned { kFlagRecord = 1, kFlagEntropy = 2, kFlagAllTiles = 4, kFlagStats = 8 };

constexpr int kThreads = 256;      // workgroup size of the step kernels (= D2Q9 tile width)
constexpr int kWave = 64;          // wavefront size (CDNA)
constexpr int kMaxTileH = 64;      // rows per D2Q9 tile
constexpr int kNStat = 16;         // FP64 values per tile partial

// partial / stats slot layout (FP64 each)
enum {
    kSMass = 0,   // sum of rho - shift (the shift is added back on the host)
    kSJx, kSJy,
    kSDpre, kSDpost, kSMax, kSLim, kSEnt,
    kSTrim, kSFilt, kSNonpos, kSNonfin, kSFluid,
    kSUnused,
    kSEns,        // nodes an ensemble-dependent limiter moved
    kSPos         // nodes the positivity rule moved (limiter, or ELBM without a root)
};

// per-domain ensemble values of the current step (device array of kNEns doubles)
enum { kEMean = 0, kEThresh, kESmoothA, kEBudget, kETopk, kNEns };

// Entropy-budget threshold (eq. EntThresh) by radix selection over the bit
// patterns of the non-negative Delta S' values, most significant digit
// first.  Each level histograms one digit of the values whose higher digits
// equal the prefix chosen so far.  A bucket holds values of one binary
// exponent, so its sum is kept exactly as the integer sum of the
// significands: the histogram does not depend on the order of the additions,
// and neither does the threshold.
constexpr int kBudgetBuckets = 2048;
enum { kSelectBudget = 1, kSelectTopK = 2 };   // which selections a step runs
struct BudgetState {
    unsigned long long prefix;   // digits chosen so far
    double budget;               // delta_0 [1 - (2 beta - 1)^2] sum Delta S'
    double s_above, c_above;     // sum and count of the values above the chosen bucket
    int level, done;
};
struct BudgetBucket {
    unsigned long long n, lo, hi;   // count; significand sum = hi 2^64 + lo
};
// key digits: FP64 keys 11 bits (the exponent), 11, 11, 10, 10, 10; FP32 keys
// 11 bits (the exponent and 3 significand bits), 10, 10
__host__ __device__ constexpr int budget_levels(bool dbl) { return dbl ? 6 : 3; }
__host__ __device__ constexpr int budget_lo(bool dbl, int level)
{
    return dbl ? (level == 0 ? 52 : level == 1 ? 41 : level == 2 ? 30 : level == 3 ? 20 : level == 4 ? 10 : 0)
               : (level == 0 ? 20 : level == 1 ? 10 : 0);
}
__host__ __device__ constexpr int budget_hi(bool dbl, int level)   // one past the digit's top bit
{
    return level == 0 ? (dbl ? 63 : 31) : budget_lo(dbl, level - 1);
}

// Which kinds of domains need a second pass: ones whose every node it forms
// (k_form2d), ones where it moves the nodes a limiter hits.
enum { kDenseSome = 1, kSparseSome = 2 };

// Per-domain parameters, device visible.  Pointers are device pointers.
struct DomainDev {
    void* buf[2];           // population planes (storage type), A and B
    long long plane;        // elements per population plane
    int nx, ny;
    double c;               // 2 beta - 1
    double shift;           // rho0 for shifted storage, 0 for FP64
    double delta_trim, delta_median;
    double rho0, lid_ux;
    int limiter, trim_mode, median_mode;
    int diffusive;          // cavity walls: 0 on-node bounce-back + equilibrium lid, 1 diffusive Maxwell
    int collision;          // kLBGK or kELBM
    int dense;              // the smooth or rational factor (LBGK): every node's limited state is formed
                            // by k_form2d, the collision kernel stores Delta S' only
    int homothety;          // 1: homothety targets reached exactly with the exact Delta S
    long long top_k;        // kLimTopK: trimming at the top_k largest finite Delta S' only
    int probe_x, probe_y, probe_cap;
    float* probe;           // [probe_cap][2]
    unsigned char* mask;    // [ny*nx] when recording
    double* dS;             // [ny*nx] when recording
    int tile_first, tile_count;   // this domain's range in the tile table
    double ens_c, ens_k, delta_ens;   // ensemble limiter parameters
    double* ens;                  // [kNEns]: E(Delta S') and the thresholds of this step
    void* phibuf;                 // D1Q3 with ensemble limiters: phi applied by the first pass
    unsigned inv_nx;              // ceil(2^32 / nx) (nx >= 64 only), see row_of_node
    int part_first;               // D2Q9: this domain's first collision partial (one per workgroup)
    int group_first, group_count; // this domain's range of collision-partial groups
    BudgetState* bstate;          // budget threshold: search state (budget limiter only)
    BudgetBucket* bhist;          // [kBudgetBuckets], left zero between levels
    double* stats;          // [kNStat + 1]: last finalised sums, then the step index
    void* dsbuf;            // [ny*nx] Delta S' of the last collision (arithmetic type), median only
};

constexpr int kXcds = 8;   // MI355X: 8 accelerator dies, each with its own L2

// Workgroup b is dispatched to XCD b % 8.  Tiles are numbered in spatial
// order (domain, row chunk, column strip); XCD x takes one contiguous range
// of that order so neighbouring tiles share an L2.  This maps a block id to
// its spatial tile index (a bijection on [0, T)).
__host__ __device__ inline int xcd_spatial(int b, int T)
{
    const int x = b % kXcds, j = b / kXcds;
    const int q = T / kXcds, r = T % kXcds;
    return x * q + (x < r ? x : r) + j;
}

// One work item (one workgroup) of the second pass, the fused step, the tile
// kernel or the D1Q3 step: columns [x0, x1) and rows [y0, y1) of one domain.
struct Tile {
    int domain, x0, x1, y0, y1;
};

// Output sites of one D1Q3 workgroup: with the halo of the longest launch
// (k1DMaxSteps, reach 1; half of it, reach 2) four waves, one per SIMD, and
// with that of a single step three whole ones.  A wave alone is a
// chain of latencies; a fifth wave shares a SIMD and delays the barrier (254
// sites on 320 threads: 400 steps of 800 sites 959 us against 914, and of
// 200000 sites, which then take fewer turns on the CUs, 3207 against 2028).
constexpr int k1DWidth = 188;

// D1Q3 steps of one launch.  A workgroup computes its k1DWidth sites with a
// halo that each further step eats `reach` sites of on either side (1, with
// the median filter 2).
constexpr int k1DMaxSteps = 33;
constexpr int k1DMaxThreads = 320;
inline int threads1d(int reach, int steps) { return (k1DWidth + 2 * reach * steps + kWave - 1) / kWave * kWave; }
static_assert(k1DWidth + 4 * k1DMaxSteps <= k1DMaxThreads, "the halo of the longest launch fits");

// The D2Q9 collision kernel walks a domain's nodes in row-major order, kThreads
// consecutive nodes per workgroup, whatever the rows: every store (and every
// load without a shift) of a wave is one aligned piece, the last workgroup of
// the domain alone is short, and the grid streams through a narrow band of
// rows.  Workgroup `first` of domain `domain` takes the nodes from
// first * kThreads.
struct Block {
    int domain, first;
};
inline int blocks_of(int nx, int ny) { return int(((long long)nx * ny + kThreads - 1) / kThreads); }

// Row of node n by the reciprocal ceil(2^32 / nx): the product is at most one
// too large.
__host__ __device__ inline int row_of_node(unsigned n, int nx, unsigned inv_nx)
{
    const unsigned r = unsigned(((unsigned long long)n * inv_nx) >> 32);
    return int(r * unsigned(nx) > n ? r - 1 : r);
}
inline unsigned inverse_nx(int nx) { return nx > 1 ? unsigned(((1ull << 32) + nx - 1) / nx) : 0u; }

// Collision partials (and the nodes) summed together for the stats and
// E(Delta S'), the nodes [n0, n1) of a domain: kGroupParts workgroups of the
// D2Q9 kernel, one D1Q3 tile.
constexpr int kGroupParts = 64;
struct Group {
    int domain, n0, n1;
};
__host__ __device__ inline Group group_entry2d(int domain, int n, int i)
{
    constexpr int w = kGroupParts * kThreads;
    return Group{domain, i * w, (i + 1) * w < n ? (i + 1) * w : n};
}
inline int groups_of(int nx, int ny) { return (blocks_of(nx, ny) + kGroupParts - 1) / kGroupParts; }

// Columns lbm_tile_config reports for the collision workgroups (of 256
// consecutive nodes): with `narrow` 64 or 128 for a domain that narrow, else 256.
inline int seg_width(int nx, int narrow)
{
    return (narrow && nx <= 64) ? 64 : ((narrow && nx <= 128) ? 128 : kThreads);
}

// Entry i of a domain's work tables (host and device build them alike):
// D2Q9 tiles of kThreads columns by th rows in spatial order (row chunk, then
// column strip); D1Q3 tiles of k1DWidth sites.
__host__ __device__ inline Tile tile_entry2d(int domain, int nx, int ny, int th, int i)
{
    const int strips = (nx + kThreads - 1) / kThreads;
    const int r = i / strips, x0 = (i - r * strips) * kThreads;
    return Tile{domain, x0, x0 + kThreads < nx ? x0 + kThreads : nx, r * th, r * th + th < ny ? r * th + th : ny};
}
__host__ __device__ inline Tile tile_entry1d(int domain, int nx, int i)
{
    const int x0 = i * k1DWidth;
    return Tile{domain, x0, x0 + k1DWidth < nx ? x0 + k1DWidth : nx, 0, 1};
}
__host__ __device__ inline int tiles_of(int lattice, int nx, int ny, int th)
{
    return lattice == kD2Q9 ? ((nx + kThreads - 1) / kThreads) * ((ny + th - 1) / th) : (nx + k1DWidth - 1) / k1DWidth;
}

// The fused D2Q9 step (collision and median filter in one pass): each wave
// computes 64 adjacent columns and keeps the 62 inner ones (the two outer
// lanes supply the stencil's neighbours), so a workgroup of four waves owns
// kFusedWidth columns of a tile of th rows (plus one halo row above and
// below, computed for their Delta S' only).
constexpr int kFusedCols = kWave - 2;
constexpr int kFusedWidth = (kThreads / kWave) * kFusedCols;
__host__ __device__ inline int fused_tiles_of(int nx, int ny, int th)
{
    return ((nx + kFusedWidth - 1) / kFusedWidth) * ((ny + th - 1) / th);
}
__host__ __device__ inline Tile fused_tile_entry(int domain, int nx, int ny, int th, int i)
{
    const int strips = (nx + kFusedWidth - 1) / kFusedWidth;
    const int r = i / strips, x0 = (i - r * strips) * kFusedWidth;
    return Tile{domain, x0, x0 + kFusedWidth < nx ? x0 + kFusedWidth : nx, r * th, r * th + th < ny ? r * th + th : ny};
}

// Tiles of bw x bh nodes of the small-domain kernel (k_block2d)
__host__ __device__ inline int block_tiles_of(int nx, int ny, int bw, int bh)
{
    return ((nx + bw - 1) / bw) * ((ny + bh - 1) / bh);
}
__host__ __device__ inline Tile block_tile_entry(int domain, int nx, int ny, int bw, int bh, int i)
{
    const int cols = (nx + bw - 1) / bw;
    const int r = i / cols, x0 = (i - r * cols) * bw, y0 = r * bh;
    return Tile{domain, x0, x0 + bw < nx ? x0 + bw : nx, y0, y0 + bh < ny ? y0 + bh : ny};
}

struct StepArgs {
    const DomainDev* dom;
    const Tile* tiles;      // spatial order (domain, row chunk, column strip)
    int ntiles;             // the D2Q9 median pass (and D1Q3) has one workgroup per tile
    int ndomains;
    int parity;             // read buf[parity], write buf[1 - parity]
    unsigned flags;
    double* partials;       // [2 sets][pstride][kNStat]: FP64 stats of a step, set 0 (collision)
                            // per group, set 1 (second pass) per tile; what reads them is queued
                            // before the next step
    const Group* groups;    // the collision-partial groups: fixed, so that the set-0 sums (and
                            // E(Delta S')) do not depend on the tile height
    int ngroups;
    int pstride;            // slots per set in `partials` (>= ntiles, ngroups)
    int median_pass;        // 1 if a second pass (median and/or ensemble limiters) writes set 1
    int dense;              // kDense* of the domains
    int fused = 0;          // 1: the fused step kernel (2: the small-domain kernel) runs alone over
                            // `tiles` (its own) and writes every partial to set 1
    int block_w = 0, block_h = 0;   // small-domain kernel: nodes of a tile
    int ens_pass;           // 1 if some domain has an ensemble-dependent limiter
    int elbm;               // 1 with ELBM collisions (all domains)
    int budget;             // kSelect* of the domains: budget threshold, top-k trimming
    const Block* blocks;    // D2Q9 collision workgroups of several domains; null for one (block b is
                            // workgroup b of the domain)
    int nblocks;            // the D2Q9 collision grid has nblocks blocks
    double* blockpart;      // [nblocks][kNStat]: collision partials of a step with kFlagStats
    unsigned* above;        // [nblocks]: byte w is 1 when wave w of the block (64 consecutive nodes) holds
                            // a median candidate (Delta S' > delta_median) and stored its Delta S'
    long long* counter;     // [2] step index by parity
    int reach = 1;          // D1Q3: sites a step's result depends on, on either side
    int in_place = 0;       // after LBGK too the second pass rescales the stored states (in_place)
    int collide_lds = 0, fused_lds = 0;   // bytes of LDS that a workgroup of the collision and of the fused
                            // step without sums holds idle (collide_lds, fused_lds)
    int steps = 1;          // D1Q3 and the small-domain kernel: steps of this launch
};

// Allocation-free stepping (lbm_step_static): bytes of the per-GPU static
// device array that holds everything but the caller's population buffers.
constexpr size_t kStaticScratchBytes = LBM_STATIC_SCRATCH_BYTES;
// its address on `device` (looked up once per device; `device` must be current)
hipError_t static_scratch(int device, char** ptr);
hipError_t launch_static_setup(const DomainDev& dd, int lattice, DomainDev* dom, Tile* tiles, int ntiles, int th,
                               int block_w, Group* groups, int ngroups, long long* counter, hipStream_t s);
hipError_t launch_static_stats(const DomainDev* dom, double shift_mass, double* out, hipStream_t s);

// Launchers (one per storage type / lattice), defined in the .hip files.
// kernel 0: collision kernel (LBGK); kernel 2: the same with the ELBM collision;
// kernel 1: the second pass (median filter, ensemble factors; after kernel 0 or 2);
// kernel 3: the fused step (LBGK, trimming, positivity and median filter);
// kernel 4: the second pass of the dense domains (after kernel 0);
// kernel 5: whole steps of small domains (LBGK, trimming, positivity and median filter)
hipError_t launch_step2d(int storage, int qe, int ds, int bc, const StepArgs& a, int kernel, hipStream_t s);
// kernel 0: D1Q3 step (LBGK); kernel 2: the same with ELBM; kernel 1: D1Q3 ensemble pass
hipError_t launch_step1d(int storage, int qe, int ds, int bc, const StepArgs& a, int kernel, hipStream_t s);
// E(Delta S') and ensemble thresholds of the step just run (before the second pass)
hipError_t launch_ens_prepare(const StepArgs& a, hipStream_t s);
// the budget threshold of the step just run (after launch_ens_prepare)
hipError_t launch_budget(int storage, int bc, const StepArgs& a, hipStream_t s);
hipError_t launch_finalize(const StepArgs& a, long long steps_done, hipStream_t s);
// nodes moved by the median filter in the step just run -> out[0]
hipError_t launch_filtered_count(const StepArgs& a, double* out, hipStream_t s);
hipError_t launch_init_f(int lattice, int qe, const double* rho, const double* u, double* f, int nx, int ny,
                         hipStream_t s);
hipError_t launch_scatter(int storage, int lattice, int bc, const double* f, void* buf, long long plane, int nx,
                          int ny, double shift, hipStream_t s);
hipError_t launch_gather(int storage, int lattice, int bc, const void* buf, long long plane, double* f, int nx,
                         int ny, double shift, int want_f, double* rho, double* u, hipStream_t s);
hipError_t launch_read(const void* ring, void* out, int words, int first, int cap, hipStream_t s);

}  // namespace lbm

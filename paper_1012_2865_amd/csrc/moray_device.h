// Internal layout shared by the host runtime and the HIP kernels of the
// adaptive ray tracer. Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

namespace moray {

constexpr int kMaxLevel = 29;
constexpr int kLevels = kMaxLevel + 2;
constexpr int kWave = 64;
constexpr int kTraceBlock = 256;
constexpr int kFinalBlock = 256;
constexpr int kFinalCellsPerThread = 4;
constexpr unsigned long long kReserveMax = 64;    // next-level queue slots (of 4 rays) a wave reserves per atomic
// Time-dependent rays: a wave reserves the halt list's records in blocks of
// kHaltBlock; the records of its last block that it does not fill are empty,
// with the level kHaltHole (above every HEALPix level, so they sort last).
// The list's one counter takes an atomic per block from every wave of the
// device: a steady step of the 128^3 workload (c dt_P = 32 cells) takes 5.69 ms
// with blocks of 64 records, 5.60 with 128 and 5.58 with 256, at the price of
// up to 255 empty records per wave and launch in the list and its sort.
constexpr int kHaltBlock = 256;
constexpr int kHaltHole = 31;
static_assert(kLevels <= kHaltHole, "empty halt records need a level above every real one");
constexpr uint32_t kNoTree = 0xffffffffu;      // tree of an empty queue slot
constexpr int kDropRanges = 16;                // tree ranges one queue filter pass removes (serving)
constexpr uint32_t kNoSlot = 0xffffffffu;      // empty cache entry
constexpr int kPack = 4;                       // most energy groups of a source one ray carries
constexpr double kHydrogenMassG = 1.6735575e-24;   // mass of a hydrogen atom, g
constexpr double kLightCms = 2.99792458e10;        // speed of light, cm/s
// One uniform grid patch of one problem, in the batch-wide cell numbering.
struct GridDev {
  int nx, ny, nz;
  int ox, oy, oz;          // lower corner in root cells (children), 0 for roots
  int is_child;            // 0: root (unit scale), 1: 2x-refined child of the root
  int problem;
  long long cell_off;      // first cell of this grid in the batch-wide numbering
  double dx_cm;            // local cell width
  const float* n_h;        // device copies (or caller device memory) of the inputs
  const float* x_hi;
  double* out_kph;         // where finalize writes this grid's k_ph and heating
  double* out_heat;
  double* out_acc;         // radiation-pressure acceleration: component k of local cell i at
                           // out_acc[k * (problem's cells) + i]; NULL when not asked for
};

// kAccSums: the absorbed rate, one plane per group.
// kAccMoments (rays carry several groups): the absorbed rate summed over the
//   groups, then the absorbed rate times (E - E_ion) summed over them; one plane.
// kAccThin (optically-thin approximation): the absorbed rate, then the deposits
//   of thin rays in cells that hold their source (nothing removed); one plane per group.
// kAccRadp (radiation pressure asked for): the absorbed rate, then the three
//   components of the absorbed momentum rate; one plane per group.
constexpr int kAccSums = 0, kAccMoments = 1, kAccThin = 2, kAccRadp = 3;

struct ProblemDev {
  int root_grid;           // index of the root grid in the grid table
  int n_groups;
  long long cell_off;      // first cell of the problem
  long long n_cells;       // cells of all its grids
  long long acc_off;       // its first accumulator
  int eexc_off;            // first of its n_groups (E - E_ion) values in erg
  // Accumulators: acc_planes records of acc_stride float64 sums per cell, record p of cell c at
  // acc_off + acc_stride * (p*n_cells + (c - cell_off)). acc_mode says what a record holds:
  int acc_mode = kAccSums;
  int acc_stride = 1;
  int acc_planes = 1;
  // optically-thin approximation: the mark of the problem's (source, group) tree t (tree table
  // index tree_first + t) on cell c is the byte mark[mark_off + t*n_cells + (c - cell_off)], t < mark_trees
  int mark_trees = 0;      // 0: the problem does not use the approximation
  int tree_first = 0;      // its first tree in the tree table (its trees are consecutive)
  long long mark_off = 0;
};

// One ray tree: the rays of one source that carry a pack of n_grp consecutive
// energy groups (1 to kPack of them), with the shape of its problem's root
// grid so a ray can start without another table lookup. All groups of a pack
// share the rays' geometry, which depends on the source alone; each keeps its
// own photon rate and ends by itself. Entries of absent groups (n_grp and
// beyond) hold P0 = -1, the mark of a group that has ended.
struct TreeDev {
  double sx, sy, sz;       // source position, root cells
  double P0[kPack];        // photon rate of one seed ray, per group
  double pmin0[kPack];     // p_min_frac * P0 (quartered per level below the seeds)
  double sigma64[kPack];   // cross-section, cm^2
  double eexc[kPack];      // E - E_ion, erg (0 where the problem's records have no second moment)
  long long acc_slot;      // accumulator of cell c (batch numbering) is acc[acc_slot + (c << acc_shift)]
  double split_r;          // sqrt(12 / (4 pi phi_c)): a ray of level l splits beyond 2^l times this many
                           // local cells; infinite when the problem never splits
  int level_init;
  int level_max;
  int gen0;                // launch generation of the tree's seed rays: a ray of generation g is at
                           // HEALPix level level_init + (g - gen0)
  int root_grid;           // grid-table index of the problem's root grid
  int rnx, rny, rnz;       // its shape
  long long rcell_off;     // its first cell
  double four_pi_phi_c;    // 4 pi phi_c of its problem
  int problem;
  int covering;            // scale deposits into the accumulators by the covering factor
  int n_grp;               // groups of the pack
  uint32_t stat0;          // statistics of its first group (those of the others follow)
  uint32_t acc_shift = 0;  // log2 of its problem's acc_stride
  double mom_scale;        // E_ph / c of the (one) group (erg s/cm), 0 without radiation pressure
  double r_halt = __builtin_huge_val();   // time-dependent rays: radius (root cells) where the
                                          // tree's rays halt in this step
  // optically-thin approximation (tau_thin > 0; one group per tree)
  double tau_thin = 0.0;   // a ray is thin in a cell while its optical depth on leaving it is below this
  double four_pi_phi_thin; // 4 pi min(1, phi_c): the split threshold of thin rays
  double split_r_thin;     // split_r for min(1, phi_c)
  long long mark_base;     // its mark on cell c (batch numbering) is the byte mark[mark_base + c]
  double thin_coef;        // sigma Ndot_g / (4 pi dx_root^2): the thin rate at r root cells is thin_coef / r^2
};

// Statistics of one (source, group).
struct SgStats {
  double esc_P;            // escaped photon rate
  double trunc_P;          // photon rate left in truncated rays
  unsigned long long segs, splits, n_esc, n_trunc;
  unsigned long long thin_segs;   // of segs, those of optically thin rays
};

// A level queue is split into up to kSegMax segments of seg_cap slots, each
// with its own write counter, and its rays into as many parts, each with its own
// claim counter, so the same-address atomics that
// reserve and claim rays spread over many addresses (a float64 or integer
// atomic on one address serialises at the memory side).
constexpr int kSegMax = 64;
constexpr int kHaltSpread = 8;

// Rays of a unit of a level of `all` rays (see the trace kernel), launched with
// `waves` waves: `chunk`, or where the level holds no more than one such unit a wave
// an equal share in whole rays per lane. Units are counted in 32 bits, and a level
// may hold any number of seeds: `chunk` grows where there would be 2^30 units and
// more (two trees whose seeds are of level 14, in units of one ray: 6.4e9).
__host__ __device__ inline unsigned unit_rays(unsigned long long all, unsigned chunk, unsigned waves) {
  if (all <= (unsigned long long)chunk * waves) {
    const unsigned long long lanes = (unsigned long long)waves * kWave;
    return (unsigned)((all + lanes - 1) / lanes) * kWave;
  }
  const unsigned least = (unsigned)(all >> 30) + 1u;
  return chunk < least ? least : chunk;
}

// Blocks of a trace launch: those the context asks for, but no more than the
// kernel keeps resident, `per_cu` on each of `num_cu` compute units. A wave
// starts with its share of the level, so a block that waits for another's place
// holds its share back.
inline int launch_blocks(int asked, int per_cu, int num_cu) {
  const long long resident = (long long)per_cu * num_cu;
  return resident < asked ? (int)resident : asked;
}

struct Counters {
  unsigned long long count[kLevels][kSegMax];   // slots written to each segment of each level queue
  unsigned int err;                             // bit flags, see kErr*
  unsigned int pad;
  unsigned long long halt_count;                // time-dependent rays halted in this step
  // per HEALPix level, the rays that halted in this step and the photons they hold;
  // a wave adds to one of kHaltSpread places (the memory side performs the atomics
  // of one line one after the other)
  struct alignas(64) Halted {
    double P;
    unsigned long long rays;
  } halted[kLevels][kHaltSpread];
  // Units of each part of a level claimed beyond those dealt at its launch's start
  // (see the trace kernel), 64 bytes apart: the memory side performs the atomics of
  // one line one after the other, and waves that run out together claim together.
  struct alignas(64) Head {
    unsigned long long n;
  } head[kLevels][kSegMax];
};
// the part the host reads, and that it reads after a time-dependent step
constexpr size_t kCountersRead = offsetof(Counters, halted), kCountersReadTd = offsetof(Counters, head);

constexpr unsigned kErrOverflow = 1u;
constexpr unsigned kErrBadInput = 2u;
constexpr unsigned kErrInternal = 8u;

// Level queue, structure of arrays. A slot holds a ray of the level above that
// split; its four children (pixels 4p .. 4p+3, a quarter of the photon rates
// each) are formed when they are claimed: ray index i of a segment is child
// i & 3 of slot i >> 2. The photon rates are one plane per group of the pack,
// pstride apart; a group that has ended holds a negative rate. The radius is
// float64 in both precision modes so a child starts exactly where its
// parent's exit distance put it. The halt lists of time-dependent rays use
// the same arrays for single rays.
struct RayQueue {
  uint64_t* pix;
  uint32_t* tree;
  double* r;
  double* P;
  unsigned long long pstride;
};

template <typename R>
struct TraceArgs {
  const GridDev* grids;
  const TreeDev* trees;
  const R* kappa;          // n_H x_HI dx_root per leaf cell; -(child+1) on covered root cells
  double* acc;             // accumulators (see ProblemDev)
  RayQueue in, out;                    // nseg segments of seg_cap slots each
  unsigned long long seg_cap;
  int nseg;                            // segments per level queue: a power of two
  Counters* ctr;
  SgStats* stats;
  int gen;                             // launch generation (the HEALPix level in a one-shot solve)
  int cin, cout;                       // counter rows of the input and output queues
  int seed_level;                      // HEALPix level of the seed rays of this launch
  int seed_begin, seed_end;            // trees seeded in this launch
  int chunk;                           // rays of a unit, at most
  unsigned max_steps;                  // hard cap on cells per ray (never reached)
  unsigned long long reserve;          // next-level slots a wave reserves at once
  // time-dependent rays: where rays halted in this step go (halt_cap records; level in halt_lev),
  // and the ones halted in the previous step that are of this launch's level: records
  // held[held_order[held_first + i]], i < n_held
  RayQueue halt;
  int* halt_lev;
  unsigned long long halt_cap;
  RayQueue held;
  const uint32_t* held_order;
  unsigned long long held_first, n_held;
  uint8_t* mark;                       // optically-thin marks (see ProblemDev), or NULL
  const double* kappa64;               // float kernels with the optically-thin approximation: the
                                       // columns in float64 (same layout as kappa), else NULL
};

// One finalize block: cells [first, first + count) of one grid.
struct FinalBlock {
  int grid;
  int count;
  long long first;
};

}  // namespace moray

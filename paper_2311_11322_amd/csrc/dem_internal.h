// dem_internal.h -- device-side layout of the DEM step (gfx950).
//
// Every kernel covers a *batch* of independent systems ("piles").  Each pile
// owns its device buffers; a device-resident table of PileDev entries holds
// their pointers, and static work lists map each launch block to
// (pile, first element).  A standalone system is a batch of one pile.
//
// Layout in HBM: structure-of-arrays, FP64, 3-vectors stored component-major
// ([3][n]) so that consecutive lanes read consecutive addresses.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dem {

constexpr int kBlock = 256;        // threads per block (4 wave64)
constexpr int kHist = 7;           // spring history per contact: xi_t[3], xi_r[3], xi_q
constexpr int kHistRow = 8;        // doubles a contact's history takes: one 64 B row
constexpr int kScanItems = 8;      // elements per thread in the batched scan
constexpr int kScanChunk = kBlock * kScanItems;
constexpr int kScanSingleItems = 4;   // segments of at most this many chunks: one-launch scan
constexpr int kRunLds = 16;        // contact ids per sphere the search keeps in LDS
constexpr int kMaxBig = 64;        // big spheres per pile searched separately
constexpr int kBigRun = 2048;      // contacts per run of a big sphere (LDS sort)
constexpr int kMom = 40;           // per tree node: M, c[3], sum m e, sum m e^2, traceless
                                   // Q2[6], Q3[10], Q4[15], 3 unused
constexpr int kRaw = 32;           // per tree node: raw M2[6], M3[10], M4[15], 1 unused

// status bits of a pile (device-written)
constexpr int kStCapacity = 1;
constexpr int kStUnstable = 2;
constexpr int kStStopped = 4;      // the stop rule fired (bulk radius grown by stop_growth)

// per-block partials of the sphere set for the cell grid: bbox min[3],
// max[3], mass moments sum m, sum m r[3], and sum m |r - c|^2 about a
// reference point c (aggregate 0's centre) for the bulk radius
constexpr int kBbox = 11;

// modes of one pass through the step graph
constexpr int kModeStep = 0;       // kick, drift, rotate, evaluate, kick
constexpr int kModeInit = 1;       // evaluate at t0 only (no motion, no kick)

// Contact model constants shared by every pile of a batch.
struct ContactParams {
  double dt;
  double k_n, k_t, k_r, k_q;
  double mu_s, mu_r, mu_t;
  double damp_n, damp_t;     // -2 ln(eps) / sqrt(pi^2 + ln^2 eps): C = damp * sqrt(k mu)
  double max_overlap_frac;   // <= 0: no check
};

// Cells of a pile.
struct CellGrid {
  double lo[3];              // origin of cell (0,0,0)
  double cell;               // cell side (>= largest sphere diameter)
  double inv_cell;
  int32_t nc[3];             // cells per axis
  int32_t nbits[3];          // key bits per axis (sum 3 * bits)
};

// What the spheres of an evaluation as a whole determine, and the cells of the
// evaluations at both parities, written on the device every step.
struct Grid {
  CellGrid c[2];
  double com[3];             // centre of mass of the pile (spin-up forcing)
  double t;                  // time of this evaluation
  double R_bulk;             // bulk radius sqrt(5/3 <|r - com|^2>_m) of this evaluation
  double wall_d[6];          // plane offset of each wall at time t
  double wall_v[6][3];       // velocity of each wall at time t
};

// Sorted-slot records read by the contact search: one 32 B load for the
// geometry and one 8 B load for the identity of each candidate.
struct alignas(32) SortedGeom {
  double x, y, z, s;
};
struct alignas(8) SortedId {
  int32_t agg;
  uint32_t id;
};

// Source record of gravity: centre, mass, softening half-length.
struct alignas(64) Rec64 {
  double x, y, z, m, e, p0, p1, p2;
};

struct PileDev {
  // sizes (host-set)
  int32_t na, ns;
  int32_t cap_pairs;         // capacity of each contact list (upper and lower)
  int32_t bits;              // cell table is (1 << bits)^3 cells
  int32_t periodic;
  int32_t g_tile;            // gravity tile (slots per tile)
  int32_t g_nt;              // gravity tiles
  int32_t g_form;            // 1: symmetric super-tile pairs; 2: per-target
  int32_t g_np;              // partial-sum rows: tiles x segments, super-tiles, or source splits
  int32_t g_m0;              // pairs of single tiles: tiles from g_m0 on are cut, as sources,
  int32_t g_segs;            // into g_segs segments (rows g_m0 + (J - g_m0) g_segs + s)
  int32_t g_half;            // 1: as targets a tile J is two halves (reactions in rows 2J, 2J + 1)
  int32_t n_rblk;            // reconstruct blocks (bbox partials)
  int32_t n_periodic;        // cells per axis of a periodic pile
  int32_t member_scan;       // 1: reduction finds members by scanning all spheres
  int32_t member_read;       // 0 automatic, 1 direct, 2 staged through LDS
  double box;                // periodic cube side
  double G, soft_frac, spin_dw;
  double stop_growth;        // > 0: stop (kStStopped) once R_bulk >= stop_growth * R0
  double R0;                 // bulk radius the stop rule compares with (device-set at the
                             // first evaluation with the rule on)
  double cell_min;           // cell side lower bound: largest diameter of the non-big spheres
  // spheres with radius > s_cut ("big", at most kMaxBig) are not binned: they
  // sit in one extra cell after the Morton cells and are searched by a block
  // each; s_small is the largest radius of the others
  double s_cut, s_small;
  int32_t n_big;
  int32_t given;             // 1: sphere positions and velocities are given (no rigid bodies
                             // to reconstruct them from; stateless test hooks)
  int32_t fused;             // 1: the whole step runs in one workgroup (k_fused); the staged
                             // kernels launched over every pile skip it
  // 1 (no gravity): cell keys are row-major and the spheres are binned on the
  // cells of the evaluation before, so that moving and binning are one launch;
  // no result depends on the cells or on the order inside them.  0: Morton keys
  // on the cells of this evaluation, whose order gravity sums follow.
  int32_t rows;
  // uniform field and container walls (host-set)
  int32_t n_walls;
  int32_t pad3;
  double gfield[3];
  double wall[6][4];         // unit normal (into the domain), offset
  double wall_amp[6][3];     // rigid sinusoidal displacement amplitude
  double wall_omega, wall_phase;
  // tree gravity (host-set)
  int32_t tree;              // 1: tree instead of the direct sum
  int32_t tree_leaf;         // nodes of at most this many spheres act as pairs
  double theta;              // opening angle
  int32_t tree_order;        // highest multipole order: 2 or 4
  int32_t pad5;
  double* tmom;              // [sum_l 8^l][kMom] node moments, level l at (8^l - 1) / 7
  double* traw;              // [sum_l 8^l][kRaw] raw moments about each node's centre of mass
  double* tpart;             // [64][3][ns] tree sum per level-2 subtree, by sorted slot
  double* tbox;              // [ceil(ns / 64)][6] bounding box (min xyz, max xyz) of each group

  // device-updated bookkeeping
  int32_t parity;            // which half of each ping-pong pair is current
  int32_t status;            // kSt* bits; a failed pile is frozen
  int64_t step;              // steps completed
  int64_t fail_step;         // step index at which it failed
  uint32_t n_pairs;          // contacts of the last evaluation
  uint32_t pad0;

  // point-mass perturber, ping-pong by parity (state lives in the table)
  int32_t pert_on;
  int32_t pad1;
  double pert_M;
  double pert_r[2][3], pert_v[2][3], pert_a[2][3];
  double* ppart;             // [ceil(ns / 64)][3] sums of the perturber's pull over 64 slots

  // aggregate constants (written once by the set-up kernel)
  int32_t* first;            // [na] first member sphere
  int32_t* count;            // [na]
  double* M;                 // [na]
  double* I;                 // [3][na] principal moments
  // aggregate state, ping-pong [2]
  double* rA[2];             // [3][na]
  double* vA[2];
  double* aA[2];
  double* NA[2];
  double* q[2];              // [4][na]
  double* wb[2];             // [3][na]
  double* wA;                // [3][na] spin in space frame (this step)

  // sphere constants (set-up)
  double* b;                 // [3][ns] body offsets
  double* s;                 // [ns] radius
  double* m;                 // [ns] mass
  int32_t* agg;              // [ns] aggregate of each sphere
  // sphere per-step
  double* r;                 // [3][ns]
  double* v;                 // [3][ns]
  double* F;                 // [3][ns] contact force (gravity is added by the reduction)
  double* tau;               // [3][ns] contact torque about the centre
  uint32_t* key;             // [ns] cell key (row-major, or Morton with gravity)
  uint32_t* sidx;            // [ns] sphere at sorted slot (piles with gravity)
  uint32_t* num;             // [ns] arrival number of sphere i in its cell
  uint32_t* sidx_raw;        // [ns] sphere at slot, in arrival order (piles with gravity)
  SortedGeom* xg;            // [ns] sorted x, y, z, radius (search)
  SortedId* sid;             // [ns] sorted aggregate id and sphere id
  void* jrec;                // gravity records in sorted order (64 B, FP64)
  void* jrec32;              // FP32 per-target form: 32 B records relative to their tile's anchor
  double* ganchor;           // [g_nt][4] that form's FP64 anchor of each tile
  void* gpart;               // [g_np][3][ns] partial sums (sorted slots)
  double* gacc;              // [3][ns] gravity force G m_i sum_j (by sphere id)
  double* bpart;             // [n_rblk][kBbox] bbox min/max + mass moments
  Grid* grid;
  uint32_t* cell_cnt;        // [cells]
  uint32_t* cell_start;      // [cells + 1]
  // contacts listed so far by the search of this evaluation: upper in the
  // high word, lower in the low (reset with the cell grid; on a line of its
  // own, as every block of the search adds to it)
  // and, beside it, the blocks of the member reduction that are done
  unsigned long long* runs;
  uint2* up_run[2];          // [ns] first entry and length of sphere i's contacts (i, j > i)
  uint2* lo_run;             // [ns] the same of its contacts (j, i), j < i
  uint32_t* cnt_up;          // [ns] upper run lengths, or NULL (stateless searches only)
  uint32_t* pair_j[2];       // [cap] partners j of the upper runs, each run sorted
  double* hist[2];           // [cap][kHistRow] spring history beside pair_j
  uint32_t* lo_nbr;          // [cap] lower neighbour ids, each run sorted
};

// One block of a per-element kernel: pile p, elements base .. base+255.
struct WorkItem {
  int32_t pile;
  int32_t base;
};

// One block of the pair kernel: the targets from slot i0 on (one tile) against
// the sources in slots [j0, j1) of the same or a later tile, per of them for each
// wave.  The targets' sums go to row row_t of the partial sums, the sources'
// reactions to row row_r (row_r < 0: sources of the targets' own tile, ordered
// pairs one way).
struct GravPair {
  int32_t pile;
  int32_t i0, j0, j1;
  int32_t row_t, row_r;
  int32_t per, pad;
};

// One block of the super-tile kernel: the super-tile pair (ti, tj), ti <= tj,
// of a pile; in the per-target form, target group ti and source split tj.
struct GravItem {
  int32_t pile;
  int32_t ti, tj;
  int32_t pad;
};

// One segment of the batched exclusive scan (out[n] receives the total).
struct ScanSeg {
  uint32_t* in;
  uint32_t* out;
  int32_t n;
  int32_t item0;             // first work item of this segment
  int32_t n_items;
  int32_t pad;
};

struct ScanItem {
  int32_t seg;
  int32_t chunk;             // chunk index inside the segment
};

// ---------------------------------------------------------------------------
// launchers (each defined next to its kernels)
// ---------------------------------------------------------------------------
void launch_setup(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk,
                  const double* pos_in, const double* vel_in, const double* spin_in);
// bin: piles of row-major cells are binned too, on the cells they carry
void launch_move(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk,
                 ContactParams cp, int mode, bool bin);
// Cells of this evaluation (and, in piles that carry them, of the next) of the
// listed piles (plist NULL: the first n).
void launch_grid(hipStream_t st, const PileDev* piles, const int32_t* plist, int n, int mode,
                 double dt);
void launch_bin(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk);
// Sorted copies of piles without gravity, in arrival order inside a cell.
void launch_place(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk);
// Piles with gravity: slots in arrival order, then ordered by id and copied.
void launch_scatter(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk);
void launch_cell_sort(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk);
void launch_search(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk);
void launch_search_big(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk);
void launch_forces(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk,
                   ContactParams cp, int precision);
// Gravity: the per-slot combine covers every pile (the tree's included); the
// pair, super-tile and per-target kernels run once per tile size present in
// the batch.  records: the FP32 records of the piles in the per-target form.
void launch_gravity_records(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk);
void launch_gravity_pairs(hipStream_t st, const PileDev* piles, const GravPair* gp, int nitems,
                          int precision, bool softened, int tile);
// Whole tiles as targets of the piles that are cut in halves (GravPlan::half; FP64).
void launch_gravity_whole(hipStream_t st, const PileDev* piles, const GravPair* gp, int nitems,
                          bool softened);
// Piles of more than kGravSlots tiles: super-tiles of several tiles.
void launch_gravity_tiles(hipStream_t st, const PileDev* piles, const GravItem* gl, int nitems,
                          int precision, bool softened, int tile);
void launch_gravity_split(hipStream_t st, const PileDev* piles, const GravItem* gl, int nitems,
                          int precision, bool softened, int tile);
// Targets per lane of the per-target kernel for a precision and tile size
// (a target group is 64 x that many slots).
int gravity_split_ipt(int precision, int tile);
void launch_gravity_combine(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk,
                            int precision);
// Supported tile sizes for a precision (the large piles' default first);
// returns the count.
int gravity_tiles(int precision, int* tiles);
// How the exact sum of a pile in the pair form is cut into blocks: its tile (the
// given one, or chosen by the number of spheres when tile is 0) and, for piles of
// at most kGravSlots tiles, the segments into which tiles from m0 on are cut as
// sources, or (FP64) whether tiles of kHalvedTile may be taken as two halves as targets.
struct GravPlan {
  int tile, segs, m0;
  bool half;
};
constexpr int kHalvedTile = 512;
// Waves of a block of the pair kernel, which share its sources, for a tile size.
constexpr int grav_pair_waves(int tile) { return tile < 256 ? tile / 64 : 4; }
GravPlan gravity_plan(int precision, int64_t ns, int tile);
// Tile sizes the pair kernel is built for: the supported ones and smaller.
constexpr int kGravTileSizes = 6;
// Aggregates in one launch from which the member reduction stages its
// members through LDS (below it, direct member reads are faster: few waves,
// and the members stay in L2 between a wave's member iterations).
constexpr int64_t kReduceStageMin = 131072;
// Super-tiles of the pair form of the exact gravity sum (at most this many
// partial sums per sphere: a super-tile is ceil(tiles / kGravSlots) tiles),
// source splits of the per-target form, and the size of the pair form's
// partial sums above which a system takes the per-target form by default.
constexpr int kGravSlots = 256;
constexpr int kGravSplits = 16;
// Targets per lane of the per-target kernel at most (measured at 125k
// spheres: FP64 2, 4, 8 took 10.5, 10.8, 11.0 ms; FP32 4, 8, 16 took 6.7,
// 6.7, 6.4 ms).
constexpr int kSplitIpt64 = 2, kSplitIpt32 = 16;
constexpr int64_t kSymPartialMax = int64_t(64) << 30;
// Spheres in one search launch from which each sphere gets one lane instead
// of eight.
constexpr int64_t kSearchLargeLaunch = 32768;
// finish: the last block of a pile ends its step (else launch_finish does)
void launch_reduce(hipStream_t st, PileDev* piles, const WorkItem* wl, int nblk, ContactParams cp,
                   int mode, bool stage, bool finish);
// Blocks of one pile in the reduction up to which its last block ends the step.
constexpr int kFinishInReduce = 64;
void launch_finish(hipStream_t st, PileDev* piles, int n_piles, int mode, double dt);
// any_order[0], [1]: some tree pile of multipole order 2, 4
// leaf_levels: bit l set when level l is some pile's finest
void launch_tree(hipStream_t st, const PileDev* piles, WorkItem* const* wl_level,
                 const int* n_level, unsigned leaf_levels, const WorkItem* wl_sph, int n_sph_blk,
                 const bool* any_order);
void launch_fill_u32(hipStream_t st, uint32_t* p, uint32_t value, int64_t n);
void launch_clear(hipStream_t st, const PileDev& h, int64_t cells);
// Fields of a state read-out: component-major src [comps][n] to row-major dst
// [n][comps].  add: a second array added to src; spin: src is the orientation,
// add the body-frame spin, and dst gets the space-frame spin.
struct ReadField {
  const double* src;
  const double* add;
  double* dst;
  int64_t n;
  int32_t comps, spin, block0;
};
constexpr int kReadFields = 14;
struct ReadList {
  ReadField f[kReadFields];
  int n;
};
void launch_read(hipStream_t st, ReadList& list);
// The n contacts of a pile in canonical order: keys (i << 32) | j and the
// history [n][kHist], through offset [ns].
void launch_read_pairs(hipStream_t st, const PileDev& h, uint32_t* offset, uint64_t* keys,
                       double* hist);
// n contacts' history [n][kHist] to rows [n][kHistRow].
void launch_history_rows(hipStream_t st, const double* packed, double* rows, int64_t n);
// The whole step of each listed pile in one workgroup: part 1 the stages
// before gravity, part 2 those after it, part 3 all (no gravity); that many steps.
void launch_fused(hipStream_t st, const PileDev* piles, const int32_t* plist, int n,
                  ContactParams cp, int mode, int part, int precision, int steps);
// Steps of one launch of k_fused without gravity: a launch apart costs about 8 us
// beside a step's 17 (97 spheres); the bound keeps a launch to some milliseconds (57 us
// a step at 400 spheres, 366 us at 2,350), piles of more than kFusedLong spheres get
// fewer steps in proportion.
constexpr int kFusedSteps = 64;
constexpr int kFusedLong = 512;
// Piles of at most this many spheres run the fused step unless tuned
// otherwise: one workgroup tests every pair of them itself, the staged step
// uses the chip (measured per step, fused and staged: 97 spheres 18.8 and 38.2
// us, 256 spheres 34.5 and 43.0, 300 spheres 45.8 and 43.5).
constexpr int64_t kFusedAutoMax = 256;
// Counts are returned to zero.  grids: that many listed piles get the cells of
// their next evaluation from the same launch.
struct ScanGrids {
  PileDev* piles;
  const int32_t* plist;
  int n, mode;
  double dt;
};
void launch_scan(hipStream_t st, const ScanSeg* segs, int n_segs, const ScanItem* items,
                 int n_items, uint32_t* item_sums, int max_seg_items, ScanGrids grids);

// What the search without allocation reports: the largest radius (bit pattern
// of a positive double, ordered like an unsigned integer), a flag for invalid
// input, the pile's status and its counter of contacts.
struct NoAllocOut {
  unsigned long long max_r_bits, runs;
  uint32_t bad;
  int32_t status;
};
// Its table entry, work list and scan segments (cell counts; contacts per
// sphere), filled in on the device.
struct NoAllocLists {
  NoAllocOut* out;
  PileDev* entry;
  WorkItem* wl;
  ScanSeg *seg_cells, *seg_keys;
  ScanItem *item_cells, *item_keys;
  uint32_t *sums_cells, *sums_keys;
  ScanSeg cells, keys;
  int n_blk;
};
void launch_noalloc(hipStream_t st, const PileDev& h, const NoAllocLists& q, const double* pos,
                    const double* radius, uint64_t* keys, int64_t cap);

// Cells per axis of a periodic cube of side L: as many as fit with a side of
// at least cell_min (with a relative margin against rounding), at least one,
// and no more than the key holds.
__host__ __device__ inline int periodic_cells(double L, double cell_min, int bits) {
  const double ratio = L / (cell_min * (1.0 + 1e-12));
  const double n = ratio >= 1.0 ? fmin(floor(ratio), (double)(1 << bits)) : 1.0;
  return (int)n;
}

// ---------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ void cross3(const double a[3], const double b[3], double c[3]) {
  const double x = a[1] * b[2] - a[2] * b[1];
  const double y = a[2] * b[0] - a[0] * b[2];
  const double z = a[0] * b[1] - a[1] * b[0];
  c[0] = x;
  c[1] = y;
  c[2] = z;
}

__device__ __forceinline__ double dot3(const double a[3], const double b[3]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// Rotation matrix (body -> space, row-major) of quaternion (w, x, y, z),
// the unit-quaternion formula applied to q as given.
__device__ __forceinline__ void quat_rot(const double q[4], double R[9]) {
  const double w = q[0], x = q[1], y = q[2], z = q[3];
  R[0] = 1.0 - 2.0 * (y * y + z * z);
  R[1] = 2.0 * (x * y - w * z);
  R[2] = 2.0 * (x * z + w * y);
  R[3] = 2.0 * (x * y + w * z);
  R[4] = 1.0 - 2.0 * (x * x + z * z);
  R[5] = 2.0 * (y * z - w * x);
  R[6] = 2.0 * (x * z - w * y);
  R[7] = 2.0 * (y * z + w * x);
  R[8] = 1.0 - 2.0 * (x * x + y * y);
}

__device__ __forceinline__ void rot_apply(const double R[9], const double a[3], double c[3]) {
  c[0] = R[0] * a[0] + R[1] * a[1] + R[2] * a[2];
  c[1] = R[3] * a[0] + R[4] * a[1] + R[5] * a[2];
  c[2] = R[6] * a[0] + R[7] * a[1] + R[8] * a[2];
}

__device__ __forceinline__ void rot_apply_T(const double R[9], const double a[3], double c[3]) {
  c[0] = R[0] * a[0] + R[3] * a[1] + R[6] * a[2];
  c[1] = R[1] * a[0] + R[4] * a[1] + R[7] * a[2];
  c[2] = R[2] * a[0] + R[5] * a[1] + R[8] * a[2];
}

// Spread the low 10 bits of v to every third bit.
__device__ __forceinline__ uint32_t spread3(uint32_t v) {
  v &= 0x3ffu;
  v = (v | (v << 16)) & 0x030000ffu;
  v = (v | (v << 8)) & 0x0300f00fu;
  v = (v | (v << 4)) & 0x030c30c3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

__device__ __forceinline__ uint32_t morton3(uint32_t x, uint32_t y, uint32_t z) {
  return spread3(x) | (spread3(y) << 1) | (spread3(z) << 2);
}

// Morton cell key for per-axis bit counts b: with m = min(b), the Morton code of
// the low m bits of each coordinate (a block of 2^m cells per axis), then the
// block's row-major index above it -- a bijection onto [0, 2^(bx+by+bz)),
// and the plain Morton code when the counts are equal.
__device__ __forceinline__ uint32_t morton_key(int cx, int cy, int cz, const int32_t nbits[3]) {
  const int m = min(nbits[0], min(nbits[1], nbits[2]));
  const uint32_t lo = (1u << m) - 1u;
  const uint32_t blk = ((uint32_t)cx >> m) + (((uint32_t)cy >> m) << (nbits[0] - m)) +
                       (((uint32_t)cz >> m) << (nbits[0] + nbits[1] - 2 * m));
  return morton3((uint32_t)cx & lo, (uint32_t)cy & lo, (uint32_t)cz & lo) | (blk << (3 * m));
}

// Cell coordinate of a position on one axis.  Periodic piles wrap the
// coordinate into [0, L) first (sphere centres are not wrapped; only the
// aggregate centres are).
__device__ __forceinline__ int cell_coord(double x, double lo, double inv_cell, int n,
                                          int periodic, double L) {
  if (periodic) {
    if (x >= L) x -= L;
    else if (x < 0.0) x += L;
  }
  // clamped before the conversion: a sphere far outside the grid falls into
  // its outermost cell
  const double c = fmin(fmax(floor((x - lo) * inv_cell), 0.0), (double)(n - 1));
  return (int)c;
}

// The pile's status as another thread or block may have set it in this launch.
__device__ __forceinline__ int status_of(const PileDev& P) {
  return __hip_atomic_load(&P.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  This bijection of [0, n) gives XCD x (blocks b with b % 8 == x) one
// contiguous range of logical blocks, so spatially adjacent work shares an
// L2 instead of being fetched by every XCD.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_block(int b, int n) {
  const int x = b % kXcds, r = b / kXcds, q = n / kXcds, rem = n % kXcds;
  return x < rem ? x * (q + 1) + r : rem * (q + 1) + (x - rem) * q + r;
}

// A product and a sum, each rounded on its own: compiled without
// contraction, so no fused multiply-add forms across them where they are
// inlined (a plain a * b + c may become one).
__device__ __forceinline__ double rn_mul(double a, double b) {
#pragma clang fp contract(off)
  return a * b;
}
__device__ __forceinline__ double rn_add(double a, double b) {
#pragma clang fp contract(off)
  return a + b;
}

// Signed distance of a point from wall w at the evaluation time (plane
// offset d_t = Grid::wall_d[w]), rounded step by step (no fused
// multiply-add) so that the contact decision is reproducible:
// ((n_x x + n_y y) + n_z z) - d_t.
__device__ __forceinline__ double wall_gap(const PileDev& P, int w, double d_t, double x, double y,
                                           double z) {
  const double* n = P.wall[w];
  const double s = rn_add(rn_add(rn_mul(n[0], x), rn_mul(n[1], y)), rn_mul(n[2], z));
  return rn_add(s, -d_t);
}

}  // namespace dem

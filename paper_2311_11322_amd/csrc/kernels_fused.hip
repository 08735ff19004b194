// kernels_fused.hip -- the whole step of a pile in one workgroup.
//
// For piles small enough that the staged step (one launch per stage, each
// over every pile of a batch) is bound by launch latency, one workgroup of
// kFusedThreads threads runs every stage of its pile in order, separated by
// workgroup barriers: kick/drift/rotate, member reconstruction, cell grid,
// binning and counting sort, contact search, per-sphere contact forces,
// member reduction and end-of-step bookkeeping.  Many piles run as
// many workgroups of one launch.  Gravity, when the pile has it, stays with
// the batched tile kernels (it would not fit one compute unit): the launch
// then covers the stages before gravity (part 1) and a second launch those
// after it (part 2); without gravity one launch (part 3) is the whole step.
//
// Every element is handled by the same device functions as in the staged
// kernels (step_body.h, step_contact.h, step_force.h), so the arithmetic of
// each element is the same; only the pile's centre of mass and bulk radius
// are summed in another order (block partials of another shape).
#include "step_body.h"
#include "step_contact.h"
#include "step_force.h"

namespace dem {

namespace {

constexpr int kFusedThreads = 512;
constexpr int kFusedWaves = kFusedThreads / 64;
constexpr int kFusedLanes = kLanesSmall;          // lanes per sphere in the search
constexpr int kFusedGroups = kFusedThreads / kFusedLanes;
constexpr int kPairThreads = kFusedThreads - 64;  // of the search without cells
constexpr int kPairsMax = kPairThreads;           // its spheres at most
constexpr int kFusedSpheres = kFusedThreads;      // spheres whose contacts are taken together

// Between stages: a workgroup barrier.  All waves of the workgroup run on
// one compute unit and share its first-level cache, so the barrier's
// workgroup-scope release and acquire make every global write of a stage
// visible to the next; a device-scope fence would also write the second-level
// cache back to memory at every stage.  Values changed by atomics (the
// status) are read with atomic loads, from the second level.
__device__ __forceinline__ void stage_sync() { __syncthreads(); }

// Exclusive prefix sum of in[0, n) into out[0, n) and the total into out[n], in
// returned to zero, by the whole workgroup: each thread scans one contiguous run, the run
// totals are scanned across the workgroup.  Integer sums: any order gives
// the same result.
__device__ void block_scan(uint32_t* __restrict__ in, uint32_t* __restrict__ out, int n,
                           uint32_t* sh /* [kFusedWaves + 1] */) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (n + kFusedThreads - 1) / kFusedThreads;
  const int b0 = min(n, tid * per), b1 = min(n, b0 + per);
  uint32_t sum = 0;
  for (int k = b0; k < b1; ++k) sum += in[k];
  uint32_t x = sum;                       // inclusive scan inside the wave
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off);
    if (lane >= off) x += y;
  }
  if (lane == 63) sh[wave] = x;
  __syncthreads();
  uint32_t before = 0, total = 0;
  for (int w = 0; w < kFusedWaves; ++w) {
    const uint32_t t = sh[w];
    if (w < wave) before += t;
    total += t;
  }
  uint32_t run = before + x - sum;
  for (int k = b0; k < b1; ++k) {
    const uint32_t v = in[k];
    in[k] = 0u;
    out[k] = run;
    run += v;
  }
  if (tid == 0) out[n] = total;
  __syncthreads();                        // sh is reused by the next scan
}

// The search of every sphere: lane groups over the sorted slots, each taking
// room for its runs from the workgroup's counter, then the big spheres with the
// whole workgroup.  total: LDS, the number of contacts listed so far.
__device__ void search_all(PileDev& P, SearchLds<kFusedLanes, kFusedThreads>& sh,
                           unsigned long long* total, uint32_t* big_up, uint32_t* big_lo,
                           uint32_t* big_fill) {
  const int tid = threadIdx.x, grp = tid / kFusedLanes, lane = tid % kFusedLanes;
  const unsigned long long cap = (unsigned long long)P.cap_pairs;
  for (int k = grp; k < P.ns - P.n_big; k += kFusedGroups) {
    const uint32_t i = P.sid[k].id;
    uint32_t nup, nlo;
    find_slot(P, k, i, grp, lane, sh, nup, nlo);
    unsigned long long at = 0;
    if (lane == 0)
      at = atomicAdd(total, ((unsigned long long)nup << 32) | (unsigned long long)nlo);
    at = __shfl(at, (tid & 63) - lane);
    if ((at >> 32) + nup <= cap && (at & 0xffffffffull) + nlo <= cap)
      store_runs(P, k, i, grp, lane, sh, nup, nlo, (uint32_t)(at >> 32), (uint32_t)at);
    else if (lane == 0)
      atomicOr(&P.status, kStCapacity);
  }
  stage_sync();
  if (tid == 0) *P.runs = *total;
  stage_sync();
  for (int kb = 0; kb < P.n_big; ++kb) {
    search_big_one(P, kb, tid, kFusedThreads, tid == 0 ? status_of(P) : 0, big_up, big_lo, big_fill);
    stage_sync();                         // runs written, the LDS read
  }
}

// The spheres of a pile searched without cells, and the contacts found.
struct PairsLds {
  SortedGeom x[kPairsMax];
  int32_t agg[kPairsMax];
  uint32_t fill[kPairsMax][2];
  uint32_t buf[kPairsMax][kRunLds];
};

// The search of a small pile without gravity: every pair of its spheres once,
// from LDS, by the waves but the last, which works out the pile's moments
// meanwhile.  A sphere's threads test it against the spheres at every L-th
// distance in the ring of ids, each half the ring; a contact goes to the ids of
// both its spheres.  By cells (moments, cells, binning, scan, placing, search) the
// search is a chain of barriers and dependent loads: 18.0 us of a step of 97
// spheres and 36 us of 250, now 5.2 (the moments) and 20.7 (FP64 rate: 75 ns
// for a wave's 64 tests).
// Called by the whole workgroup with sh.x, sh.agg and cleared sh.fill in place.
__device__ __forceinline__ void search_pairs(PileDev& P, PairsLds& sh, unsigned long long* total,
                             const double cref[3]) {
  const int ns = P.ns, tid = threadIdx.x, nxt = P.parity ^ 1;
  const int periodic = P.periodic;
  const double box = P.box;
  if (tid >= kPairThreads) {
    const int lane = tid - kPairThreads;
    double acc[kBbox];
    bbox_identity(acc);
    for (int i = lane; i < ns; i += 64) {
      const SortedGeom g = sh.x[i];
      double one[kBbox];
      moments_one(P, i, g.x, g.y, g.z, cref, one);
      bbox_combine(acc, one);
    }
    bbox_wave(acc);
    grid_from_vals(P, acc, lane, kCellsNow);
  }
  int lg = 0;                                     // 2^lg threads of one wave per sphere
  while (lg < 6 && (ns << (lg + 1)) <= kPairThreads) ++lg;
  const int L = 1 << lg, i = tid >> lg, lane = tid & (L - 1);
  const bool active = tid < kPairThreads && i < ns;
  SortedGeom me{};
  int ai = 0;
  // the contact test without branches, so that tests overlap: the number of boxes
  // to shift by (-1, 0, 1; every wave has pairs across a face) times the box is
  // exact, so the shifted distance is rounded once, as in touching
  const double far = periodic ? 0.5 * box : INFINITY, shift = periodic ? box : 0.0;
  auto image = [&](double d) { return fma((double)((int)(d < -far) - (int)(d > far)), shift, d); };
  auto meets = [&](int j) {
    const SortedGeom o = sh.x[j];
    return (sh.agg[j] != ai) & touching(image(o.x - me.x), image(o.y - me.y), image(o.z - me.z),
                                        me.s + o.s, 0, 0.0);
  };
  auto enter_up = [&](int a, int b) {
    const uint32_t pos = atomicAdd(&sh.fill[a][0], 1u);
    if (pos < (uint32_t)kRunLds) sh.buf[a][pos] = (uint32_t)b;
  };
  auto enter = [&](int j) {
    const int a = min(i, j), b = max(i, j);
    enter_up(a, b);
    const uint32_t pos = atomicAdd(&sh.fill[b][1], 1u);
    if (pos < (uint32_t)kRunLds) sh.buf[b][kRunLds - 1 - pos] = (uint32_t)a;
  };
  if (active) {
    me = sh.x[i];
    ai = sh.agg[i];
    const int half = (ns - 1) / 2;
    for (int d0 = 1 + lane; d0 <= half; d0 += 8 * L) {
      uint32_t met = 0;
      auto other = [&](int u) {
        const int j = i + min(d0 + u * L, half);
        return j < ns ? j : j - ns;
      };
#pragma unroll
      for (int u = 0; u < 8; ++u)
        met |= (uint32_t)(meets(other(u)) & (d0 + u * L <= half)) << u;
      for (; met != 0; met &= met - 1) enter(other(__builtin_ctz(met)));
    }
    // an even ring's opposite sphere, from the first half alone
    if ((ns & 1) == 0 && lane == 0 && i < ns / 2 && meets(i + ns / 2)) enter(i + ns / 2);
    for (int w = lane; w < P.n_walls; w += L)
      if (wall_gap(P, w, P.grid->wall_d[w], me.x, me.y, me.z) < me.s) enter_up(i, ns + w);
  }
  __syncthreads();
  if (!active) return;
  const uint32_t nup = sh.fill[i][0], nlo = sh.fill[i][1];
  unsigned long long at = 0;
  if (lane == 0) at = atomicAdd(total, ((unsigned long long)nup << 32) | (unsigned long long)nlo);
  at = __shfl(at, (tid & 63) - lane);
  const uint32_t u0 = (uint32_t)(at >> 32), l0 = (uint32_t)at;
  const unsigned long long cap = (unsigned long long)P.cap_pairs;
  if ((unsigned long long)u0 + nup > cap || (unsigned long long)l0 + nlo > cap) {
    if (lane == 0) atomicOr(&P.status, kStCapacity);
    return;
  }
  uint32_t* up_out = P.pair_j[nxt] + u0;
  uint32_t* lo_out = P.lo_nbr + l0;
  if (lane == 0) {
    P.up_run[nxt][i] = make_uint2(u0, nup);
    P.lo_run[i] = make_uint2(l0, nlo);
  }
  if (nup + nlo > (uint32_t)kRunLds) {
    // more contacts than the LDS keeps: once more, in order
    if (lane != 0) return;
    for (int j = 0; j < ns; ++j)
      if (meets(j)) *(j < i ? lo_out++ : up_out++) = (uint32_t)j;
    for (int w = 0; w < P.n_walls; ++w)
      if (wall_gap(P, w, P.grid->wall_d[w], me.x, me.y, me.z) < me.s) *up_out++ = (uint32_t)(ns + w);
    return;
  }
  put_run<1>(sh.buf[i], nup, lane, L, up_out);
  put_run<1>(sh.buf[i] + (kRunLds - nlo), nlo, lane, L, lo_out);
}

template <typename T>
__global__ __launch_bounds__(kFusedThreads) void k_fused(PileDev* __restrict__ piles,
                                                         const int32_t* __restrict__ plist,
                                                         ContactParams cp, int mode, int part,
                                                         int steps) {
  // the search and the forces take turns in this one
  __shared__ union {
    PairsLds pairs;
    struct {
      SearchLds<kFusedLanes, kFusedThreads> lanes;
      uint32_t big_up[kBigRun], big_lo[kBigRun], big_fill[4];
    } cells;
    ForceLds<kFusedThreads, kFusedSpheres> force;
  } sh;
  __shared__ unsigned long long run_total;
  __shared__ double red[kFusedWaves][kBbox];
  __shared__ uint32_t scan_sh[kFusedWaves + 1];
  __shared__ MoveLds<kFusedThreads> move_sh;
  PileDev& P = piles[plist[blockIdx.x]];
  const int tid = threadIdx.x;
  const bool pairs = P.rows != 0 && P.ns <= kPairsMax;
  for (int step = 0; step < steps; ++step) {
    bool ok = status_of(P) == 0;            // a failed pile stays frozen
    if (part & 1) {
      if (ok) {
        // kick, drift and rotate every aggregate; members, and the bounding box
        // and mass moments of the pile
        double acc[kBbox], cref[3];
        bbox_identity(acc);
        bbox_ref(P, cref);
        if (tid == 0) run_total = 0ull;
        if ((tid >> 6) == kFusedWaves - 1) walls_at(P, tid & 63, mode, cp.dt);
        for (int base = 0; base < P.ns; base += kFusedThreads) {
          double one[kBbox];
          bbox_identity(one);
          move_block<kFusedThreads>(P, base, cp, mode, move_sh, cref, one);
          if (pairs && tid < P.ns) {
            sh.pairs.x[tid] = SortedGeom{one[0], one[1], one[2], P.s[tid]};
            sh.pairs.agg[tid] = P.agg[tid];
            sh.pairs.fill[tid][0] = sh.pairs.fill[tid][1] = 0u;
          }
          bbox_combine(acc, one);
          if (base + kFusedThreads < P.ns) stage_sync();      // move_sh is written again
        }
        if (pairs) {
          stage_sync();
          search_pairs(P, sh.pairs, &run_total, cref);
          stage_sync();
          if (tid == 0) *P.runs = run_total;
        } else {
          bbox_wave(acc);
          if ((tid & 63) == 0)
            for (int k = 0; k < kBbox; ++k) red[tid >> 6][k] = acc[k];
          stage_sync();
          if (tid < 64) {
            for (int w = 1; w < kFusedWaves; ++w) bbox_combine(acc, red[w]);
            grid_from_vals(P, acc, tid, kCellsNow);
          }
          stage_sync();
        }
        ok = status_of(P) == 0;
      }
      if (ok && !pairs) {
        // counting sort of the cell keys
        for (int i = tid; i < P.ns; i += kFusedThreads) bin_one(P, i);
        stage_sync();
        block_scan(P.cell_cnt, P.cell_start, (1 << (3 * P.bits)) + 1, scan_sh);
        stage_sync();
        if (P.rows) {
          for (int i = tid; i < P.ns; i += kFusedThreads) place_one(P, i);
        } else {
          for (int i = tid; i < P.ns; i += kFusedThreads) scatter_one(P, i);
          stage_sync();
          for (int k = tid; k < P.ns; k += kFusedThreads) cell_sort_one(P, k);
        }
        stage_sync();
        // contact search (the counter was cleared before the last barriers)
        search_all(P, sh.cells.lanes, &run_total, sh.cells.big_up, sh.cells.big_lo,
                   sh.cells.big_fill);
        ok = status_of(P) == 0;
      }
      if (ok) {
        // contact forces with the spring history
        const PairCtx<T> c = pair_ctx<T>(P, cp);
        bool bad = false;
        for (int i = 0; i < P.ns; i += kFusedSpheres)
          forces_group<T, kFusedThreads, kFusedSpheres>(P, c, cp, i, sh.force, bad);
        if (bad) atomicOr(&P.status, kStUnstable);
        stage_sync();
        ok = status_of(P) == 0;
      }
    }
    if (part & 2) {
      if (ok) {
        const int na = P.na, nxt = P.parity ^ 1;
        for (int A = tid; A < na; A += kFusedThreads) {
          double q[4], R[9];
          for (int k = 0; k < 4; ++k) q[k] = P.q[nxt][k * na + A];
          quat_rot(q, R);
          double FA[3] = {0.0, 0.0, 0.0}, NA[3] = {0.0, 0.0, 0.0};
          if (P.member_scan != 0) reduce_members_scan(P, A, R, FA, NA);
          else reduce_members_direct(P, A, R, FA, NA);
          reduce_tail(P, A, R, FA, NA, cp, mode);
        }
        stage_sync();
      }
      if (tid < 64) finish_one(P, tid, mode, cp.dt, !ok);
    }
    if (step + 1 < steps) stage_sync();     // the entry as the end of the step left it
  }
}

}  // namespace

void launch_fused(hipStream_t st, const PileDev* piles, const int32_t* plist, int n, ContactParams cp,
                  int mode, int part, int precision, int steps) {
  if (n <= 0) return;
  PileDev* p = const_cast<PileDev*>(piles);
  if (precision == 1)
    hipLaunchKernelGGL(k_fused<float>, dim3(n), dim3(kFusedThreads), 0, st, p, plist, cp, mode,
                       part, steps);
  else
    hipLaunchKernelGGL(k_fused<double>, dim3(n), dim3(kFusedThreads), 0, st, p, plist, cp, mode,
                       part, steps);
}

}  // namespace dem

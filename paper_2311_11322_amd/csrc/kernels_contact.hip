// kernels_contact.hip -- cell-list binning, contact search that skips pairs
// inside one aggregate, and the per-contact soft-sphere force with spring
// history (Sec. 2.1, 2.2.4 and 2.2.5 of the paper; lever arm Eq. 8, contact-point
// torque Eq. 9).
//
// Binning is a counting sort on cell keys: integer atomics build the per-cell
// counts, a batched exclusive scan turns them into cell ranges, and the spheres
// are placed there.  Without gravity any order inside a cell will do, so the
// number that its atomic returned places a sphere; with gravity the slots set
// the order of the force sums, and ranking each sphere by id within its cell
// makes it deterministic.
// The search scans the 27 neighbouring cells of every sphere (a group of
// lanes per sphere, blocks mapped to XCDs by region); each sphere lists
// its contacts with higher ids (the canonical upper list) and with lower ids
// (the lower list) as one sorted run each, so sphere by sphere the contacts
// come out in canonical (i, j) order without a global sort and without float
// atomics.
#include "step_contact.h"

namespace dem {

namespace {

__global__ __launch_bounds__(kBlock) void k_bin(const PileDev* __restrict__ piles,
                                                const WorkItem* __restrict__ wl) {
  const WorkItem w = wl[xcd_block(blockIdx.x, gridDim.x)];
  const PileDev& P = piles[w.pile];
  const int i = w.base + threadIdx.x;
  if (i >= P.ns || P.status != 0) return;
  bin_one(P, i);
}

__global__ __launch_bounds__(kBlock) void k_place(const PileDev* __restrict__ piles,
                                                  const WorkItem* __restrict__ wl) {
  const WorkItem w = wl[xcd_block(blockIdx.x, gridDim.x)];
  const PileDev& P = piles[w.pile];
  const int i = w.base + threadIdx.x;
  if (i >= P.ns || P.status != 0) return;
  place_one(P, i);
}

__global__ __launch_bounds__(kBlock) void k_scatter(const PileDev* __restrict__ piles,
                                                    const WorkItem* __restrict__ wl) {
  const WorkItem w = wl[xcd_block(blockIdx.x, gridDim.x)];
  const PileDev& P = piles[w.pile];
  const int i = w.base + threadIdx.x;
  if (i >= P.ns || P.status != 0) return;
  scatter_one(P, i);
}

// Order each cell's spheres by id and write their sorted copies
// (cell_sort_one).
__global__ __launch_bounds__(kBlock) void k_cell_sort(const PileDev* __restrict__ piles,
                                                      const WorkItem* __restrict__ wl) {
  const WorkItem w = wl[xcd_block(blockIdx.x, gridDim.x)];
  const PileDev& P = piles[w.pile];
  const int k = w.base + threadIdx.x;
  if (k >= P.ns || P.status != 0) return;
  cell_sort_one(P, k);
}

// L lanes per sorted slot.  Every lane tests the spheres of its share of
// the 27 neighbouring cells that belong to another aggregate, and its share
// of the walls; the contacts with j > i (upper) and j < i (lower) stay in LDS
// until the block knows how many it has.  One atomic then takes room for all
// of them in the pile's lists, and every sphere's runs are written there, sorted
// by id.  (As count, scan of the counts and write it took two launches more:
// 21.8 -> 12.0 us for 6,400 spheres, 200 -> 131 us for a 1M-sphere lattice.)
template <int L, int NT>
__global__ __launch_bounds__(NT, 5) void k_search(PileDev* __restrict__ piles,
                                               const WorkItem* __restrict__ wl) {
  constexpr int kGroups = NT / L;                // spheres per block
  constexpr int kWaves = NT / 64;
  __shared__ SearchLds<L, NT> sh;
  __shared__ uint32_t wsum[kWaves][2], at[3];
  static_assert(kGroups <= kBlock, "a block's spheres lie in one work item");
  constexpr int kPer = kBlock / kGroups;         // blocks per work item
  const int blk = xcd_block(blockIdx.x, gridDim.x);
  const WorkItem w = wl[blk / kPer];
  PileDev& P = piles[w.pile];
  const int grp = threadIdx.x / L, lane = threadIdx.x % L;
  const int wave = threadIdx.x >> 6, l64 = threadIdx.x & 63;
  const int k = w.base + (blk % kPer) * kGroups + grp;
  // big spheres: k_search_big.  The status may change meanwhile (another block
  // finds the lists full): a wave that reads a failure lists nothing, and the
  // block goes on to its barriers.
  const bool active = k < P.ns - P.n_big && searching(P, P.status);   // uniform over the lane group
  uint32_t nup = 0, nlo = 0, i = 0;
  if (active) {
    i = P.sid[k].id;
    find_slot<L, NT>(P, k, i, grp, lane, sh, nup, nlo);
  }
  // prefix sums over the wave's groups (a group's first lane counts)
  uint32_t pu = lane == 0 ? nup : 0u, pl = lane == 0 ? nlo : 0u;
  for (int off = L; off < 64; off <<= 1) {
    const uint32_t u = __shfl_up(pu, off), l = __shfl_up(pl, off);
    if (l64 >= off) {
      pu += u;
      pl += l;
    }
  }
  if (l64 == 64 - L) {
    wsum[wave][0] = pu;
    wsum[wave][1] = pl;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t tu = 0, tl = 0, u0 = 0, l0 = 0;
    for (int q = 0; q < kWaves; ++q) {
      tu += wsum[q][0];
      tl += wsum[q][1];
    }
    at[2] = (tu | tl) == 0u || take_runs(P, tu, tl, u0, l0) ? 1u : 0u;
    at[0] = u0;
    at[1] = l0;
  }
  __syncthreads();
  if (at[2] == 0u || !active) return;
  uint32_t u0 = at[0], l0 = at[1];
  for (int q = 0; q < wave; ++q) {
    u0 += wsum[q][0];
    l0 += wsum[q][1];
  }
  // the group's offset inside its wave, from its first lane
  const int first = l64 - lane;
  u0 += __shfl(pu, first) - nup;
  l0 += __shfl(pl, first) - nlo;
  store_runs<L, NT>(P, k, i, grp, lane, sh, nup, nlo, u0, l0);
}

// One block per big sphere (the k-th, by id, sits at slot ns - n_big + k):
// its threads split the cells within reach of any other sphere and the big
// spheres' cell.
__global__ __launch_bounds__(kBlock) void k_search_big(PileDev* __restrict__ piles,
                                                       const WorkItem* __restrict__ wl) {
  __shared__ uint32_t buf_up[kBigRun];
  __shared__ uint32_t buf_lo[kBigRun];
  __shared__ uint32_t fill[4];
  const WorkItem w = wl[blockIdx.x];
  PileDev& P = piles[w.pile];
  search_big_one(P, w.base, threadIdx.x, kBlock, P.status, buf_up, buf_lo, fill);
}

}  // namespace

void launch_bin(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk) {
  if (nblk <= 0) return;
  hipLaunchKernelGGL(k_bin, dim3(nblk), dim3(kBlock), 0, st, piles, wl);
}
void launch_place(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk) {
  if (nblk <= 0) return;
  hipLaunchKernelGGL(k_place, dim3(nblk), dim3(kBlock), 0, st, piles, wl);
}
void launch_scatter(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk) {
  if (nblk <= 0) return;
  hipLaunchKernelGGL(k_scatter, dim3(nblk), dim3(kBlock), 0, st, piles, wl);
}
void launch_cell_sort(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk) {
  if (nblk <= 0) return;
  hipLaunchKernelGGL(k_cell_sort, dim3(nblk), dim3(kBlock), 0, st, piles, wl);
}
void launch_search_big(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk) {
  hipLaunchKernelGGL(k_search_big, dim3(nblk), dim3(kBlock), 0, st, const_cast<PileDev*>(piles),
                     wl);
}
void launch_search(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk) {
  // Small launches are bound by the chain of loads of one sphere, which eight
  // lanes split; large ones by the loads in all, which one lane per sphere
  // keeps fewest (1M-sphere lattice: 131 us with one lane, 159 with two, 229
  // with four).  A block covers 64 or 256 spheres: every block adds to one
  // counter, 12 ns each.
  PileDev* p = const_cast<PileDev*>(piles);
  if ((int64_t)nblk * kBlock >= kSearchLargeLaunch)
    hipLaunchKernelGGL((k_search<kLanesLarge, 256>), dim3(nblk * kLanesLarge), dim3(256), 0, st, p,
                       wl);
  else
    hipLaunchKernelGGL((k_search<kLanesSmall, 512>), dim3(nblk * kLanesSmall / 2), dim3(512), 0, st,
                       p, wl);
}

}  // namespace dem

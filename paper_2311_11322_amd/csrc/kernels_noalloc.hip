// kernels_noalloc.hip -- the stateless contact search on device arrays without
// allocation: its own stages around those of the step (binning, scan, placing,
// search).  Everything the host would have to read back in between -- whether
// the input is valid, the largest radius, whether there are contacts -- stays
// on the device, and the launches follow each other without it; the host reads
// one small block at the end.  (With the table, work lists and segments copied
// from the host, the radius read back and the contacts counted before the keys:
// 165 us for 20,011 spheres, 93 this way.)
#include "step_body.h"
#include "step_contact.h"

namespace dem {

namespace {

// Zero cell counts, an empty result, and by the first block the table entry,
// work list and scan segments.
__global__ __launch_bounds__(kBlock) void k_noalloc_setup(PileDev h, NoAllocLists q) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < q.cells.n) q.cells.in[i] = 0u;
  if (i < q.n_blk) q.wl[i] = WorkItem{0, i * kBlock};
  if (i < q.cells.n_items) q.item_cells[i] = ScanItem{0, i};
  if (i < q.keys.n_items) q.item_keys[i] = ScanItem{0, i};
  if (i == 0) {
    *q.out = NoAllocOut{};
    *q.seg_cells = q.cells;
    *q.seg_keys = q.keys;
    *q.entry = h;
  }
}

// One thread per sphere: row-major device positions into the search's
// component-major array; radius and position checks; largest radius; the
// bounding-box partials of the block.
__global__ __launch_bounds__(kBlock) void k_noalloc_ingest(const double* __restrict__ pos,
                                                           const double* __restrict__ rad,
                                                           const PileDev* __restrict__ entry,
                                                           NoAllocOut* __restrict__ out) {
  __shared__ double red[kBlock / 64][kBbox], top[kBlock / 64];
  const PileDev& P = *entry;
  const int n = P.ns, i = blockIdx.x * kBlock + threadIdx.x;
  double smax = 0.0, vals[kBbox];
  bbox_identity(vals);
  bool bad = false;
  if (i < n) {
    const double x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2], s = rad[i];
    P.r[i] = x;
    P.r[n + i] = y;
    P.r[2 * n + i] = z;
    given_vals(x, y, z, vals);
    bad = !(isfinite(x) && isfinite(y) && isfinite(z) && isfinite(s) && s > 0.0);
    smax = bad ? 0.0 : s;
  }
  for (int off = 32; off > 0; off >>= 1) smax = fmax(smax, __shfl_xor(smax, off));
  const bool any_bad = __any(bad);
  bbox_wave(vals);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    if (any_bad) atomicOr(&out->bad, 1u);
    top[wave] = smax;
    for (int k = 0; k < kBbox; ++k) red[wave][k] = vals[k];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < kBlock / 64; ++w) {
    bbox_combine(vals, red[w]);
    smax = fmax(smax, top[w]);
  }
  // one atomic per block: atomics on one address take 12 ns each
  if (smax > 0.0) atomicMax(&out->max_r_bits, (unsigned long long)__double_as_longlong(smax));
  for (int k = 0; k < kBbox; ++k) P.bpart[(size_t)blockIdx.x * kBbox + k] = vals[k];
}

// One block: cells of the largest diameter and the grid; invalid input fails
// the pile, so that the stages after this do nothing.
__global__ __launch_bounds__(kBlock) void k_noalloc_grid(PileDev* __restrict__ entry,
                                                         const NoAllocOut* __restrict__ out) {
  __shared__ GridLds sh;
  PileDev& P = *entry;
  if (out->bad != 0u) {
    if (threadIdx.x == 0) {
      P.status = kStUnstable;
      *P.runs = 0ull;
    }
    return;
  }
  if (threadIdx.x == 0) {
    const double smax = __longlong_as_double((long long)out->max_r_bits);
    P.cell_min = 2.0 * smax;
    P.s_small = smax;
    if (P.periodic) P.n_periodic = periodic_cells(P.box, 2.0 * smax, P.bits);
  }
  __syncthreads();
  grid_block(P, kModeInit, 1.0, kCellsNow, sh);
}

// One thread per sphere: its upper run as canonical keys, up to cap in all; and
// what the host reads.
__global__ __launch_bounds__(kBlock) void k_noalloc_keys(const PileDev* __restrict__ entry,
                                                         const uint32_t* __restrict__ off,
                                                         uint64_t* __restrict__ keys, int64_t cap,
                                                         NoAllocOut* __restrict__ out) {
  const PileDev& P = *entry;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i == 0) {
    out->status = P.status;
    out->runs = *P.runs;
  }
  if (i >= P.ns || P.status != 0 || cap == 0) return;
  const uint2 r = P.up_run[P.parity ^ 1][i];
  const uint32_t* __restrict__ pj = P.pair_j[P.parity ^ 1];
  for (int64_t e = 0, p = off[i]; e < r.y && p < cap; ++e, ++p)
    keys[p] = (uint64_t(i) << 32) | pj[r.x + e];
}

}  // namespace

void launch_noalloc(hipStream_t st, const PileDev& h, const NoAllocLists& q, const double* pos,
                    const double* radius, uint64_t* keys, int64_t cap) {
  const int rows = std::max(q.cells.n, q.n_blk);
  hipLaunchKernelGGL(k_noalloc_setup, dim3((rows + kBlock - 1) / kBlock), dim3(kBlock), 0, st, h, q);
  hipLaunchKernelGGL(k_noalloc_ingest, dim3(q.n_blk), dim3(kBlock), 0, st, pos, radius, q.entry,
                     q.out);
  hipLaunchKernelGGL(k_noalloc_grid, dim3(1), dim3(kBlock), 0, st, q.entry, q.out);
  launch_bin(st, q.entry, q.wl, q.n_blk);
  launch_scan(st, q.seg_cells, 1, q.item_cells, q.cells.n_items, q.sums_cells, q.cells.n_items,
              ScanGrids{});
  launch_place(st, q.entry, q.wl, q.n_blk);
  launch_search(st, q.entry, q.wl, q.n_blk);
  if (cap > 0)
    launch_scan(st, q.seg_keys, 1, q.item_keys, q.keys.n_items, q.sums_keys, q.keys.n_items,
                ScanGrids{});
  hipLaunchKernelGGL(k_noalloc_keys, dim3(q.n_blk), dim3(kBlock), 0, st, q.entry, q.keys.out, keys,
                     cap, q.out);
}

}  // namespace dem

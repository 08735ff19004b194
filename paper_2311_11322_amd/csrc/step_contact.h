// step_contact.h -- per-element device functions of the contact search:
// cell binning (counting sort of cell keys; with gravity rank by id in a cell),
// and the search that skips pairs inside one aggregate (the 27 neighbouring
// cells of a sphere split among a group of lanes; big spheres searched
// apart).  Included by the staged kernels and by the fused per-pile step.
//
// Paper references: contacts between spheres of different aggregates only
// (Sec. 2.2); the contact model acts on spheres in contact (Sec. 2.1).
#pragma once
#include "dem_internal.h"

namespace dem {

namespace {

// Cell of a sphere on the pile's current grid.
__device__ __forceinline__ void sphere_cell(const PileDev& P, const CellGrid& g, double x, double y,
                                            double z, int c[3]) {
  c[0] = cell_coord(x, g.lo[0], g.inv_cell, g.nc[0], P.periodic, P.box);
  c[1] = cell_coord(y, g.lo[1], g.inv_cell, g.nc[1], P.periodic, P.box);
  c[2] = cell_coord(z, g.lo[2], g.inv_cell, g.nc[2], P.periodic, P.box);
}

// Key of a cell: row-major in a pile without gravity, so that the search reads
// a row of neighbours as one range; Morton in a pile with gravity, whose tiles
// and tree nodes are runs of neighbouring cells.
__device__ __forceinline__ uint32_t cell_key(const PileDev& P, const CellGrid& g, int cx, int cy,
                                             int cz) {
  return P.rows ? (uint32_t)((cz * g.nc[1] + cy) * g.nc[0] + cx)
                : morton_key(cx, cy, cz, g.nbits);
}

// Cell key of a sphere with radius s at (x, y, z): the big spheres' cell comes
// after all the others.
__device__ __forceinline__ uint32_t sphere_key(const PileDev& P, const CellGrid& g, double x,
                                               double y, double z, double s) {
  if (P.n_big > 0 && s > P.s_cut) return 1u << (3 * P.bits);
  int c[3];
  sphere_cell(P, g, x, y, z, c);
  return cell_key(P, g, c[0], c[1], c[2]);
}

// Cell key of sphere i and its arrival number in the cell (integer atomics on
// the cell counts).
__device__ __forceinline__ void bin_one(const PileDev& P, int i) {
  const int ns = P.ns;
  const uint32_t key = sphere_key(P, P.grid->c[P.parity], P.r[i], P.r[ns + i], P.r[2 * ns + i],
                                  P.n_big > 0 ? P.s[i] : 0.0);
  P.key[i] = key;
  P.num[i] = atomicAdd(&P.cell_cnt[key], 1u);
}

// The sorted copies of sphere i at slot d: packed records for the search and, in
// a pile with gravity, its source record and id.
__device__ __forceinline__ void place_sphere(const PileDev& P, uint32_t i, uint32_t d) {
  const int ns = P.ns;
  const double x = P.r[i], y = P.r[ns + i], z = P.r[2 * ns + i], s = P.s[i];
  if (P.G != 0.0) {
    const double e = 0.5 * P.soft_frac * s;
    P.sidx[d] = i;
    ((Rec64*)P.jrec)[d] = Rec64{x, y, z, P.m[i], e, 0.0, 0.0, 0.0};
  }
  P.xg[d] = SortedGeom{x, y, z, s};
  P.sid[d] = SortedId{P.agg[i], i};
}

// Place sphere i, in arrival order inside its cell (piles without gravity: no
// result depends on that order).
__device__ __forceinline__ void place_one(const PileDev& P, int i) {
  place_sphere(P, (uint32_t)i, P.cell_start[P.key[i]] + P.num[i]);
}

// Enter sphere i in its cell's range, in arrival order.
__device__ __forceinline__ void scatter_one(const PileDev& P, int i) {
  P.sidx_raw[P.cell_start[P.key[i]] + P.num[i]] = (uint32_t)i;
}

// Order one cell's spheres by id, independent of arrival order: the sphere at
// raw slot k goes to its cell's start plus its rank (the number of smaller ids
// in the cell).
__device__ __forceinline__ void cell_sort_one(const PileDev& P, int k) {
  const uint32_t* __restrict__ raw = P.sidx_raw;
  const uint32_t i = raw[k];
  const uint32_t key = P.key[i];
  const uint32_t s0 = P.cell_start[key], s1 = P.cell_start[key + 1];
  uint32_t r = 0;
  for (uint32_t t = s0; t < s1; ++t) r += raw[t] < i;
  place_sphere(P, i, s0 + r);
}

// Contact test exactly as written d^2 = (dx*dx + dy*dy) + dz*dz < S*S, each
// product and sum rounded separately (no fused multiply-add), with the
// minimum-image correction per axis in a periodic cube.
__device__ __forceinline__ bool touching(double dx, double dy, double dz, double S, int periodic,
                                         double L) {
  const double hL = 0.5 * L;
  // one test for the three axes: few candidates lie across a face
  if (periodic && fmax(fmax(fabs(dx), fabs(dy)), fabs(dz)) > hL) {
    if (dx > hL) dx -= L;
    else if (dx < -hL) dx += L;
    if (dy > hL) dy -= L;
    else if (dy < -hL) dy += L;
    if (dz > hL) dz -= L;
    else if (dz < -hL) dz += L;
  }
  const double d2 = rn_add(rn_add(rn_mul(dx, dx), rn_mul(dy, dy)), rn_mul(dz, dz));
  return d2 < rn_mul(S, S);
}

// The search gives each sphere a group of L lanes of one wave; the lanes
// split the 27 neighbouring cells (and the walls) between them, so a
// sphere's dependent cell-range and candidate loads run L-wide.  Eight lanes
// keep the dependent chains short where few spheres cannot fill the chip; one
// lane per sphere issues the fewest instructions where many can.
constexpr int kLanesSmall = 8;            // launches of few spheres
constexpr int kLanesLarge = 1;            // launches of many

// Sorts a short run of ids in global memory (insertion).
__device__ __forceinline__ void sort_run(uint32_t* __restrict__ a, uint32_t n) {
  for (uint32_t x = 1; x < n; ++x) {
    const uint32_t v = a[x];
    uint32_t y = x;
    while (y > 0 && a[y - 1] > v) {
      a[y] = a[y - 1];
      --y;
    }
    a[y] = v;
  }
}

// Calls emit(j) for every contact partner j of the sphere at sorted slot k
// that falls to this lane of its group: the spheres of the lane's share of the
// 27 neighbouring cells that touch it and belong to another aggregate, the big
// spheres, and the walls (partners ns + w).
template <int Lanes, typename Emit>
__device__ __forceinline__ void search_partners(const PileDev& P, int k, int lane, Emit emit) {
  const int ns = P.ns;
  const SortedGeom* __restrict__ xg = P.xg;
  const SortedId* __restrict__ sid = P.sid;
  const CellGrid& g = P.grid->c[P.parity];
  const uint32_t* __restrict__ cstart = P.cell_start;
  const SortedGeom mg = xg[k];
  const double x = mg.x, y = mg.y, z = mg.z, si = mg.s;
  const int ai = sid[k].agg;
  const int periodic = P.periodic;
  const double L = P.box;
  int c[3];
  sphere_cell(P, g, x, y, z, c);
  const int nx = g.nc[0], ny = g.nc[1], nz = g.nc[2];   // periodic piles: all the same
  // neighbouring cells along an axis: c-1..c+1, or every cell when a
  // periodic axis has fewer than three (so no cell is visited twice)
  const bool all = periodic && nx < 3;
  // the o-th (0..2) neighbour of coordinate c on an axis of n cells
  auto nb = [&](int cc, int o, int n, bool& ok) {
    int v = all ? o : cc + o - 1;
    if (periodic && !all) v += v < 0 ? n : (v >= n ? -n : 0);
    ok = ok && v >= 0 && v < n;
    return v;
  };
  // candidates t0 .. t1 - 1, kAhead of them loaded together
  constexpr uint32_t kAhead = Lanes == 1 ? 2 : 1;
  auto scan = [&](uint32_t t0, uint32_t t1) {
    for (uint32_t t = t0; t < t1; t += kAhead) {
      SortedId o[kAhead];
      SortedGeom cg[kAhead];
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u) {
        const uint32_t v = min(t + u, t1 - 1);
        o[u] = sid[v];
        cg[u] = xg[v];
      }
#pragma unroll
      for (uint32_t u = 0; u < kAhead; ++u) {
        // not one of this aggregate (the sphere itself among them)
        if (t + u < t1 && o[u].agg != ai &&
            touching(cg[u].x - x, cg[u].y - y, cg[u].z - z, si + cg[u].s, periodic, L))
          emit(o[u].id);
      }
    }
  };
  if (P.rows) {
    // row-major cells: the neighbours of a row (y, z) are one range of slots,
    // and one more cell where the row wraps
    constexpr int kR = (9 + Lanes - 1) / Lanes;
    const int x0 = all ? 0 : max(c[0] - 1, 0), x1 = all ? nx - 1 : min(c[0] + 1, nx - 1);
    const int xw = periodic && !all ? (c[0] == 0 ? nx - 1 : (c[0] == nx - 1 ? 0 : -1)) : -1;
    uint32_t rs[kR], re[kR], row[kR];
#pragma unroll
    for (int q = 0; q < kR; ++q) {
      const int d = lane + q * Lanes;
      bool ok = d < 9;
      const int cy = nb(c[1], d % 3, ny, ok), cz = nb(c[2], d / 3, nz, ok);
      row[q] = ok ? (uint32_t)(cz * ny + cy) * (uint32_t)nx : 0xffffffffu;
      rs[q] = ok ? cstart[row[q] + x0] : 0u;
      re[q] = ok ? cstart[row[q] + x1 + 1] : 0u;
    }
#pragma unroll
    for (int q = 0; q < kR; ++q) {
      scan(rs[q], re[q]);
      if (xw >= 0 && row[q] != 0xffffffffu) scan(cstart[row[q] + xw], cstart[row[q] + xw + 1]);
    }
  } else {
    constexpr int kSlots = (27 + Lanes - 1) / Lanes;     // cells per lane
    constexpr int kStep = kSlots < 9 ? kSlots : 9;       // ranges loaded together
    for (int q0 = 0; q0 < kSlots; q0 += kStep) {
      uint32_t rs[kStep], re[kStep];
#pragma unroll
      for (int q = 0; q < kStep; ++q) {
        const int d = lane + (q0 + q) * Lanes;
        bool ok = d < 27;
        const int cx = nb(c[0], d % 3, nx, ok), cy = nb(c[1], (d / 3) % 3, ny, ok),
                  cz = nb(c[2], d / 9, nz, ok);
        const uint32_t key = ok ? morton_key(cx, cy, cz, g.nbits) : 0u;
        rs[q] = ok ? cstart[key] : 0u;
        re[q] = ok ? cstart[key + 1] : 0u;
      }
#pragma unroll
      for (int q = 0; q < kStep; ++q) scan(rs[q], re[q]);
    }
  }
  if (P.n_big > 0) {
    const uint32_t bk = 1u << (3 * P.bits);
    for (uint32_t t = cstart[bk] + lane, t1 = cstart[bk + 1]; t < t1; t += Lanes) scan(t, t + 1);
  }
  // walls are partners ns + w, after every sphere partner
  for (int w = lane; w < P.n_walls; w += Lanes)
    if (wall_gap(P, w, P.grid->wall_d[w], x, y, z) < si) emit((uint32_t)(ns + w));
}

// A lane group's part of the LDS of a search by NT threads: kRunLds ids, which
// the lanes of a group keep together, or apart by NT when every lane is its own
// group (then consecutive lanes touch consecutive banks), and two counters.
template <int Lanes, int NT>
struct SearchLds {
  static constexpr int kGroups = NT / Lanes;
  static constexpr int kStride = Lanes == 1 ? NT : 1;
  uint32_t buf[kGroups * kRunLds];
  uint32_t fill[Lanes == 1 ? 1 : kGroups][2];
  __device__ uint32_t* ids(int grp) { return buf + (Lanes == 1 ? grp : grp * kRunLds); }
};

// Finds the contacts of the sphere at slot k: nup contacts with j > i (upper)
// and nlo with j < i (lower), the upper ids from the front of the group's ids
// and the lower from their back while they fit kRunLds entries together.  The
// group's LDS is visible to all its lanes on return.
template <int Lanes, int NT>
__device__ __forceinline__ void find_slot(const PileDev& P, int k, uint32_t i, int grp, int lane,
                                          SearchLds<Lanes, NT>& sh, uint32_t& nup, uint32_t& nlo) {
  uint32_t* buf = sh.ids(grp);
  constexpr int st = SearchLds<Lanes, NT>::kStride;
  // the two ends may meet when there are more than kRunLds: not used then
  if constexpr (Lanes == 1) {
    uint32_t u = 0, l = 0;
    search_partners<1>(P, k, 0, [&](uint32_t j) {
      const bool up = j > i;
      const uint32_t pos = up ? u : l;
      if (pos < (uint32_t)kRunLds) buf[(up ? pos : kRunLds - 1 - pos) * st] = j;
      u += up ? 1u : 0u;
      l += up ? 0u : 1u;
    });
    nup = u;
    nlo = l;
  } else {
    uint32_t* fill = sh.fill[grp];
    if (lane == 0) {
      fill[0] = 0u;
      fill[1] = 0u;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    search_partners<Lanes>(P, k, lane, [&](uint32_t j) {
      const bool up = j > i;
      const uint32_t pos = atomicAdd(&fill[up ? 0 : 1], 1u);
      if (pos < (uint32_t)kRunLds) buf[up ? pos : kRunLds - 1 - pos] = j;
    });
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    nup = fill[0];
    nlo = fill[1];
  }
}

// Runs too long for the group's ids: found again by the group's first lane
// alone, written in arrival order and sorted in place (rare: more than kRunLds
// contacts of one sphere).
__device__ __forceinline__ void store_long_runs(const PileDev& P, int k, uint32_t i, uint32_t nup,
                                             uint32_t nlo, uint32_t u0, uint32_t l0) {
  uint32_t* up_out = P.pair_j[P.parity ^ 1] + u0;
  uint32_t* lo_out = P.lo_nbr + l0;
  uint32_t u = 0, l = 0;
  search_partners<1>(P, k, 0, [&](uint32_t j) {
    if (j > i) up_out[u++] = j;
    else lo_out[l++] = j;
  });
  sort_run(up_out, nup);
  sort_run(lo_out, nlo);
}

// Writes the n ids b[0], b[St], .. to out, sorted: ids in a run are distinct, so
// an entry's rank is the number of smaller entries.  Lane of a group of lanes.
template <int St>
__device__ __forceinline__ void put_run(const uint32_t* b, uint32_t n, int lane, int lanes,
                                        uint32_t* out) {
  for (uint32_t e = lane; e < n; e += lanes) {
    const uint32_t v = b[e * St];
    uint32_t r = 0;
    for (uint32_t f = 0; f < n; ++f) r += b[f * St] < v;
    out[r] = v;
  }
}

// Stores the runs found by find_slot at u0 (upper) and l0 (lower), each sorted.
template <int Lanes, int NT>
__device__ __forceinline__ void store_runs(const PileDev& P, int k, uint32_t i, int grp, int lane,
                                           SearchLds<Lanes, NT>& sh, uint32_t nup, uint32_t nlo,
                                           uint32_t u0, uint32_t l0) {
  constexpr int st = SearchLds<Lanes, NT>::kStride;
  const int nxt = P.parity ^ 1;
  if (lane == 0) {
    P.up_run[nxt][i] = make_uint2(u0, nup);
    P.lo_run[i] = make_uint2(l0, nlo);
    if (P.cnt_up) P.cnt_up[i] = nup;
  }
  if (nup + nlo > (uint32_t)kRunLds) {
    if (lane == 0) store_long_runs(P, k, i, nup, nlo, u0, l0);
    return;
  }
  const uint32_t* buf = sh.ids(grp);
  put_run<st>(buf, nup, lane, Lanes, P.pair_j[nxt] + u0);
  put_run<st>(buf + (kRunLds - nlo) * st, nlo, lane, Lanes, P.lo_nbr + l0);
}

// Whether the search of a pile of status st goes on.  A failed pile's does not; but
// a stateless search (given positions) whose lists are full goes on counting, so that
// it reports how many contacts there are.
__device__ __forceinline__ bool searching(const PileDev& P, int st) {
  return st == 0 || (st == kStCapacity && (P.given || P.na == 0));
}

// Room for nup upper and nlo lower contacts in the pile's lists: the first
// entries, taken in arrival order (the order of the runs in the lists decides
// no result; read-outs go by sphere).  False, and a capacity failure, when
// either list is full.
__device__ __forceinline__ bool take_runs(PileDev& P, uint32_t nup, uint32_t nlo, uint32_t& u0,
                                          uint32_t& l0) {
  const unsigned long long at =
      atomicAdd(P.runs, ((unsigned long long)nup << 32) | (unsigned long long)nlo);
  u0 = (uint32_t)(at >> 32);
  l0 = (uint32_t)at;
  const unsigned long long cap = (unsigned long long)P.cap_pairs;
  if ((unsigned long long)u0 + nup <= cap && (unsigned long long)l0 + nlo <= cap) return true;
  atomicOr(&P.status, kStCapacity);
  return false;
}

// The kb-th big sphere of the pile (at slot ns - n_big + kb), searched by
// nthreads threads of one block (tid the thread's index, st the first one's reading
// of the status; LDS buf_up, buf_lo of kBigRun entries and fill[4]; every thread of the
// block calls this):
// they split the cells within reach of any other sphere and the big
// spheres' cell, gather both runs in LDS, rank-sort them and store them.  A
// run longer than kBigRun is counted, and a capacity failure.
__device__ __forceinline__ void search_big_one(PileDev& P, int kb, int tid, int nthreads,
                                               int st, uint32_t* buf_up, uint32_t* buf_lo,
                                               uint32_t* fill) {
  // one read of the status for the whole block (another block of this pile
  // may set it meanwhile), so that every thread takes the same path
  if (tid == 0) fill[0] = searching(P, st) ? 0u : 1u;
  __syncthreads();
  const bool failed = fill[0] != 0u;
  __syncthreads();
  if (failed) return;
  const int ns = P.ns, nxt = P.parity ^ 1;
  const int k = ns - P.n_big + kb;
  const SortedId me = P.sid[k];
  const SortedGeom mg = P.xg[k];
  const uint32_t i = me.id;
  const double x = mg.x, y = mg.y, z = mg.z, si = mg.s;
  const int ai = me.agg;
  if (tid == 0) {
    fill[0] = 0u;
    fill[1] = 0u;
  }
  __syncthreads();
  const SortedGeom* __restrict__ xg = P.xg;
  const SortedId* __restrict__ sid = P.sid;
  const uint32_t* __restrict__ cstart = P.cell_start;
  const int periodic = P.periodic;
  const double L = P.box;
  const CellGrid& g = P.grid->c[P.parity];
  int c[3];
  sphere_cell(P, g, x, y, z, c);
  // reach in cells of any partner: (s_i + s_small) / cell, plus one for rounding
  const int R = (int)ceil((si + P.s_small) * g.inv_cell) + 1;
  int start[3], cnt[3];
  for (int a = 0; a < 3; ++a) {
    const int n = g.nc[a];
    if (periodic) {
      if (2 * R + 1 >= n) {
        start[a] = 0;
        cnt[a] = n;
      } else {
        start[a] = c[a] - R;
        cnt[a] = 2 * R + 1;
      }
    } else {
      const int lo = c[a] - R < 0 ? 0 : c[a] - R;
      const int hi = c[a] + R > n - 1 ? n - 1 : c[a] + R;
      start[a] = lo;
      cnt[a] = hi - lo + 1;
    }
  }
  auto test = [&](uint32_t t) {
    const SortedId o = sid[t];
    if (o.agg == ai) return;
    const SortedGeom cg = xg[t];
    if (!touching(cg.x - x, cg.y - y, cg.z - z, si + cg.s, periodic, L)) return;
    const bool up = o.id > i;
    const uint32_t pos = atomicAdd(&fill[up ? 0 : 1], 1u);
    if (pos < (uint32_t)kBigRun) (up ? buf_up : buf_lo)[pos] = o.id;
  };
  const int total = cnt[0] * cnt[1] * cnt[2];
  for (int u = tid; u < total; u += nthreads) {
    int cx = start[0] + u % cnt[0];
    int cy = start[1] + (u / cnt[0]) % cnt[1];
    int cz = start[2] + u / (cnt[0] * cnt[1]);
    if (periodic) {
      const int n = g.nc[0];
      cx += cx < 0 ? n : (cx >= n ? -n : 0);
      cy += cy < 0 ? n : (cy >= n ? -n : 0);
      cz += cz < 0 ? n : (cz >= n ? -n : 0);
    }
    const uint32_t key = cell_key(P, g, cx, cy, cz);
    for (uint32_t t = cstart[key], t1 = cstart[key + 1]; t < t1; ++t) test(t);
  }
  const uint32_t bk = 1u << (3 * P.bits);
  for (uint32_t t = cstart[bk] + tid; t < cstart[bk + 1]; t += nthreads) test(t);
  for (int wi_ = tid; wi_ < P.n_walls; wi_ += nthreads) {
    if (wall_gap(P, wi_, P.grid->wall_d[wi_], x, y, z) < si) {
      const uint32_t pos = atomicAdd(&fill[0], 1u);
      if (pos < (uint32_t)kBigRun) buf_up[pos] = (uint32_t)(ns + wi_);
    }
  }
  __syncthreads();
  const uint32_t run_up = fill[0], run_lo = fill[1];
  if (tid == 0) {
    const bool fits = run_up <= (uint32_t)kBigRun && run_lo <= (uint32_t)kBigRun;
    if (!fits) atomicOr(&P.status, kStCapacity);
    uint32_t u0, l0;
    const bool ok = take_runs(P, run_up, run_lo, u0, l0) && fits;
    fill[2] = ok ? u0 : 0xffffffffu;
    fill[3] = l0;
    if (ok) {
      P.up_run[nxt][i] = make_uint2(u0, run_up);
      P.lo_run[i] = make_uint2(l0, run_lo);
      if (P.cnt_up) P.cnt_up[i] = run_up;
    }
  }
  __syncthreads();
  if (fill[2] == 0xffffffffu) return;
  uint32_t* up_out = P.pair_j[nxt] + fill[2];
  uint32_t* lo_out = P.lo_nbr + fill[3];
  for (uint32_t e = tid; e < run_up; e += nthreads) {
    const uint32_t v = buf_up[e];
    uint32_t r = 0;
    for (uint32_t f = 0; f < run_up; ++f) r += buf_up[f] < v;
    up_out[r] = v;
  }
  for (uint32_t e = tid; e < run_lo; e += nthreads) {
    const uint32_t v = buf_lo[e];
    uint32_t r = 0;
    for (uint32_t f = 0; f < run_lo; ++f) r += buf_lo[f] < v;
    lo_out[r] = v;
  }
}

}  // namespace

}  // namespace dem

// kernels_gravity.hip -- softened all-pairs self-gravity (Eq. 4 of the
// paper, with Plummer softening eps_ij = soft_frac (s_i + s_j) / 2).
//
// Spheres are taken in cell-sorted (Morton) order and cut into tiles of B
// slots.  A pile of at most kGravSlots tiles runs k_grav_pairs: one block per
// pair of tiles (I, J >= I), or per segment of J, so every unordered pair of spheres
// is evaluated once (Newton's third law), by up to four waves that share the sources:
//  * each lane holds IPT = B / 64 targets in registers, with their sums;
//  * the sources enter 64 at a time, one per lane, together with a reaction
//    accumulator, and rotate one lane per step (DPP wave_ror:1), so that after
//    64 steps every source has met every target of the wave and is back in
//    its own lane holding its complete reaction sum;
//  * sources of the targets' own tile rotate without a reaction (ordered
//    pairs, one way);
//  * the waves' sums of a target are added in LDS, in order.
// Each block stores its targets' sums in the row of its sources (tile or segment)
// and its sources' reactions in the row of its targets' tile; the combine kernel
// adds a sphere's rows in a fixed order, so the result is deterministic and
// independent of other piles.
//
// A larger pile runs k_grav_tiles: its tiles are grouped into at most
// kGravSlots super-tiles of `span` consecutive tiles and one wave takes one
// super-tile pair (SI, SJ), SI <= SJ, tile pair by tile pair: the targets of
// I keep their sums over all J of SJ, and a source's lane adds its reaction to
// the source's running sum over the tiles of SI.  The partial sums take at
// most kGravSlots x 3 values per sphere.
//
// FP64 form: rsqrt from the hardware estimate y0 and one first-order
// correction folded into the cube: r^-3 = y0^3 (1 + 3e/2), e = 1 - r^2 y0^2.
// FP32-force form: coordinates relative to an FP64 anchor, the first sphere of
// the target tile, subtracted in FP64 from the FP64 records as a block loads
// them; FP32 partial sums, FP64 across them.  (The per-target form reads FP32
// records relative to their own tile's anchor instead.)
#include "gravity_common.h"

#include <algorithm>

namespace dem {

namespace {

// FP32 per-target form, one thread per sorted slot: the sphere's record
// relative to its tile's anchor (the tile's first sphere).
__global__ __launch_bounds__(kBlock) void k_grav_records(const PileDev* __restrict__ piles,
                                                         const WorkItem* __restrict__ wl) {
  const WorkItem w = wl[blockIdx.x];
  const PileDev& P = piles[w.pile];
  const int k = w.base + threadIdx.x;
  if (k >= P.ns || P.status != 0 || P.g_form != 2 || P.tree) return;
  const int a = (k / P.g_tile) * P.g_tile;
  const Rec64 f = ((const Rec64*)P.jrec)[k], o = ((const Rec64*)P.jrec)[a];
  ((Rec32*)P.jrec32)[k] = Rec32{(float)(f.x - o.x), (float)(f.y - o.y), (float)(f.z - o.z),
                                (float)f.m, (float)f.e, 0.f, 0.f, 0.f};
  if (k == a) {
    double* an = P.ganchor + (size_t)(k / P.g_tile) * 4;
    an[0] = o.x;
    an[1] = o.y;
    an[2] = o.z;
    an[3] = 0.0;
  }
}

// A source or target of the pair kernels: the record's centre less the
// anchor (FP32 form; the FP64 form takes the centre as it is), its softening
// half-length and its mass.
template <typename T>
struct Src {
  T x, y, z, m, e;
};
template <typename T>
__device__ __forceinline__ Src<T> relative(const Rec64& r, const double an[3]) {
  if (sizeof(T) == 4)
    return Src<T>{(T)(r.x - an[0]), (T)(r.y - an[1]), (T)(r.z - an[2]), (T)r.m, (T)r.e};
  return Src<T>{(T)r.x, (T)r.y, (T)r.z, (T)r.m, (T)r.e};
}

// 64 sources, one per lane, led once around the wave past every lane's IPT
// targets; with REACT each source's reaction sum comes back in (bx, by, bz), one for
// each of G groups of a lane's targets.
template <typename T, int IPT, bool SOFT, bool REACT, int G = 1>
__device__ __forceinline__ void ring(Src<T> s, const T (&xi)[IPT], const T (&yi)[IPT],
                                     const T (&zi)[IPT], const T (&ei)[IPT], const T (&mi)[IPT],
                                     T (&ax)[IPT], T (&ay)[IPT], T (&az)[IPT], double c15,
                                     T (&bx)[G], T (&by)[G], T (&bz)[G]) {
#pragma unroll
  for (int h = 0; h < G; ++h) bx[h] = by[h] = bz[h] = 0;
  for (int step = 0; step < 64; ++step) {
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
      // a sphere met by itself (own tile) contributes nothing: d = 0, and
      // r^-3 = 0 when unsoftened
      const T dx = s.x - xi[u], dy = s.y - yi[u], dz = s.z - zi[u];
      const T t = ei[u] + s.e;
      const T r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, t * t)));
      const T c3 = inv_cube<SOFT>(r2, c15);
      const T wi = s.m * c3;
      ax[u] = fma(wi, dx, ax[u]);
      ay[u] = fma(wi, dy, ay[u]);
      az[u] = fma(wi, dz, az[u]);
      if (REACT) {
        const T wj = mi[u] * c3;
        constexpr int P = IPT / G;
        bx[u / P] = fma(wj, dx, bx[u / P]);
        by[u / P] = fma(wj, dy, by[u / P]);
        bz[u / P] = fma(wj, dz, bz[u / P]);
      }
    }
    s.x = ror1(s.x);
    s.y = ror1(s.y);
    s.z = ror1(s.z);
    s.m = ror1(s.m);
    s.e = ror1(s.e);
    if (REACT) {
#pragma unroll
      for (int h = 0; h < G; ++h) {
        bx[h] = ror1(bx[h]);
        by[h] = ror1(by[h]);
        bz[h] = ror1(bz[h]);
      }
    }
  }
}

// Waves per SIMD the compiler may plan for.  FP64 with 8 targets per lane runs
// at two waves per SIMD whatever the schedule; saying so lets the compiler
// issue the eight inverse square roots together (measured 1.5 % faster at 125k
// spheres than its three-wave schedule).
#define GRAV_WAVES(T, IPT) \
  __attribute__((amdgpu_waves_per_eu(1, (sizeof(T) == 8 && IPT == 8) ? 2 : 8)))

// One block per (target tile, source tile or segment of it).  Bound by the FP64
// (FP32) instruction rate of `ring`: a pair of tiles of 512 takes one compute unit
// 56 us (28 us).  Up to four waves share the sources, because a row of partial sums
// then serves all of them: with one wave per block a small pile needed a row for
// every 64 or 128 sources to fill the chip, and an engine that fills it anyway spent
// its gain, and more, on writing and reading those rows.  Gravity stage, FP64, by one
// wave for a whole pair of 512 / one for 64 to 256 sources, a row each / so: 25 piles
// of 16,000 spheres 2.59 / 2.77 / 2.59 ms in tiles of 512 (2.70 in the plan's 256), one
// of 13,001 231 / 102 / 91 us, one of 124,958 6017 / 5999 / 6032 us.
//
// G = 2: the reactions from the two halves of the targets' tile in a row each, as two
// blocks of half the targets store them, to the bit: a launch that has few blocks
// takes the halves, a full one the whole tiles (rebuild in dem_host.hip).
template <typename T, int IPT, bool SOFT, int G>
__global__ __launch_bounds__(64 * grav_pair_waves(64 * IPT)) GRAV_WAVES(T, IPT) void k_grav_pairs(
    const PileDev* __restrict__ piles, const GravPair* __restrict__ gp) {
  constexpr int B = 64 * IPT, W = grav_pair_waves(64 * IPT);
  __shared__ T sums[W][3][B];
  __shared__ int failed[W];
  const GravPair it = gp[blockIdx.x];
  const PileDev& P = piles[it.pile];
  const int ns = P.ns, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // The search and the contact forces run beside this and may set the status: each
  // wave takes what it reads to the block's barrier, and none leaves before.
  const int st = P.status;
  const Rec64* __restrict__ rec = (const Rec64*)P.jrec;
  double c15;
  series_coeffs(c15);
  T* __restrict__ part = (T*)P.gpart;
  double an[3] = {0.0, 0.0, 0.0};
  if (sizeof(T) == 4) {
    const ConstRec64 cr = (ConstRec64)P.jrec;
    an[0] = cr[it.i0].x;
    an[1] = cr[it.i0].y;
    an[2] = cr[it.i0].z;
  }
  T xi[IPT], yi[IPT], zi[IPT], ei[IPT], mi[IPT], ax[IPT], ay[IPT], az[IPT];
#pragma unroll
  for (int u = 0; u < IPT; ++u) {
    const int k = it.i0 + u * 64 + lane;
    const Src<T> r = relative<T>(rec[min(k, ns - 1)], an);
    xi[u] = r.x;
    yi[u] = r.y;
    zi[u] = r.z;
    ei[u] = r.e;
    mi[u] = k < ns ? r.m : (T)0;
    ax[u] = ay[u] = az[u] = (T)0;
  }
  // the wave's sources; none in a short last tile's last waves
  const int j0 = it.j0 + wv * it.per, j1 = st != 0 ? j0 : min(j0 + it.per, it.j1);
  // with few targets per lane a round of 64 sources is short, so the next 64
  // are loaded while the current ones go round
  constexpr bool kAhead = IPT < 8;
  Rec64 next = rec[min(j0 + lane, it.j1 - 1)];
  for (int jc = j0; jc < j1; jc += 64) {
    const int jx = jc + lane;
    Src<T> s = relative<T>(next, an);
    if (jx >= j1) s.m = (T)0;
    if (kAhead) next = rec[min(jx + 64, it.j1 - 1)];
    T bx[G], by[G], bz[G];
    if (it.row_r < 0) {
      ring<T, IPT, SOFT, false, G>(s, xi, yi, zi, ei, mi, ax, ay, az, c15, bx, by, bz);
    } else {
      ring<T, IPT, SOFT, true, G>(s, xi, yi, zi, ei, mi, ax, ay, az, c15, bx, by, bz);
      if (jx < j1) {
#pragma unroll
        for (int h = 0; h < G; ++h) {
          T* q = part + (size_t)(it.row_r + h) * 3 * ns + jx;
          q[0] = -bx[h];
          q[ns] = -by[h];
          q[2 * (size_t)ns] = -bz[h];
        }
      }
    }
    if (!kAhead) next = rec[min(jx + 64, it.j1 - 1)];
  }
  T* __restrict__ row = part + (size_t)it.row_t * 3 * ns + it.i0;
  const int n = min(B, ns - it.i0);
#pragma unroll
  for (int u = 0; u < IPT; ++u) {
    sums[wv][0][u * 64 + lane] = ax[u];
    sums[wv][1][u * 64 + lane] = ay[u];
    sums[wv][2][u * 64 + lane] = az[u];
  }
  if (lane == 0) failed[wv] = st;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < W; ++w)
    if (failed[w] != 0) return;
#pragma unroll
  for (int c = 0; c < 3; ++c)
    for (int k = threadIdx.x; k < n; k += 64 * W) {
      double g = (double)sums[0][c][k];
#pragma unroll
      for (int w = 1; w < W; ++w) g += (double)sums[w][c][k];
      row[(size_t)c * ns + k] = (T)g;
    }
}

template <typename T, int IPT, bool SOFT>
__global__ __launch_bounds__(64) GRAV_WAVES(T, IPT) void k_grav_tiles(
    const PileDev* __restrict__ piles, const GravItem* __restrict__ gl) {
  constexpr int B = 64 * IPT;
  const GravItem it = gl[blockIdx.x];
  const PileDev& P = piles[it.pile];
  if (P.status != 0) return;
  const int ns = P.ns, nt = P.g_nt, lane = threadIdx.x;
  const int span = (nt + kGravSlots - 1) / kGravSlots;     // tiles per super-tile
  const int si = it.ti, sj = it.tj;
  const int I0 = si * span, I1 = min(I0 + span, nt);
  const int J0 = sj * span, J1 = min(J0 + span, nt);
  const bool diag_item = si == sj;
  const Rec64* __restrict__ rec = (const Rec64*)P.jrec;
  double c15;
  series_coeffs(c15);
  T* __restrict__ part = (T*)P.gpart;

  for (int I = I0; I < I1; ++I) {
    const int i0 = I * B;
    double an[3] = {0.0, 0.0, 0.0};
    if (sizeof(T) == 4) {
      const ConstRec64 cr = (ConstRec64)P.jrec;
      an[0] = cr[i0].x;
      an[1] = cr[i0].y;
      an[2] = cr[i0].z;
    }
    T xi[IPT], yi[IPT], zi[IPT], ei[IPT], mi[IPT], ax[IPT], ay[IPT], az[IPT];
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
      const int k = i0 + u * 64 + lane;
      const Src<T> r = relative<T>(rec[min(k, ns - 1)], an);
      xi[u] = r.x;
      yi[u] = r.y;
      zi[u] = r.z;
      ei[u] = r.e;
      mi[u] = k < ns ? r.m : (T)0;
      ax[u] = ay[u] = az[u] = (T)0;
    }
    for (int J = diag_item ? I : J0; J < J1; ++J) {
      const int j0 = J * B, j1 = min(j0 + B, ns);
      for (int jc = j0; jc < j1; jc += 64) {
        const int jx = jc + lane;
        Src<T> s = relative<T>(rec[min(jx, j1 - 1)], an);
        if (jx >= j1) s.m = (T)0;
        T b[3][1];
        T &bx = b[0][0], &by = b[1][0], &bz = b[2][0];
        if (J == I) {
          ring<T, IPT, SOFT, false>(s, xi, yi, zi, ei, mi, ax, ay, az, c15, b[0], b[1], b[2]);
          continue;
        }
        ring<T, IPT, SOFT, true>(s, xi, yi, zi, ei, mi, ax, ay, az, c15, b[0], b[1], b[2]);
        // add to the source's reaction sum over the tiles of SI so far (which
        // this same lane stored)
        if (jx < j1) {
          T* q = part + (size_t)si * 3 * ns + jx;
          const bool first = I == I0;
          q[0] = first ? -bx : q[0] - bx;
          q[ns] = first ? -by : q[ns] - by;
          q[2 * (size_t)ns] = first ? -bz : q[2 * (size_t)ns] - bz;
        }
      }
    }
    // targets of tile I store under super-tile sj; on a diagonal item that
    // slot already holds the reactions from the tiles before I
    const bool add = diag_item && I > I0;
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
      const int k = i0 + u * 64 + lane;
      if (k < ns) {
        T* q = part + (size_t)sj * 3 * ns + k;
        q[0] = add ? q[0] + ax[u] : ax[u];
        q[ns] = add ? q[ns] + ay[u] : ay[u];
        q[2 * (size_t)ns] = add ? q[2 * (size_t)ns] + az[u] : az[u];
      }
    }
  }
}

// The per-target form (O(N) partial sums): one wave per (target group,
// source split s), a target group being 64 x IPT consecutive slots inside
// one tile (IPT per lane, fewer than a tile holds, so that the launch has
// enough waves).  Split s covers a run of consecutive source tiles; the
// wave's lanes hold the group's targets and walk every source of the run by
// a uniform index (scalar loads), evaluating each ordered pair once from the
// target's side, so no reaction is carried and each sphere receives one
// partial per split.  Twice the pair evaluations of the pair form, for 16
// partial sums per sphere.
template <typename T, int IPT, bool SOFT>
__global__ __launch_bounds__(64) void k_grav_split(const PileDev* __restrict__ piles,
                                                   const GravItem* __restrict__ gl) {
  constexpr int G = 64 * IPT;
  constexpr bool F32 = sizeof(T) == 4;
  const GravItem it = gl[blockIdx.x];
  const PileDev& P = piles[it.pile];
  if (P.status != 0) return;
  const int ns = P.ns, nt = P.g_nt, B = P.g_tile, lane = threadIdx.x;
  const int span = (nt + kGravSplits - 1) / kGravSplits;  // source tiles per split
  const int t0 = it.tj * span, t1 = min(t0 + span, nt);
  const int i0 = it.ti * G;
  const int ti = i0 / B;                                   // the targets' tile
  double c15;
  series_coeffs(c15);

  T xi[IPT], yi[IPT], zi[IPT], ei[IPT], ax[IPT], ay[IPT], az[IPT];
#pragma unroll
  for (int u = 0; u < IPT; ++u) {
    const int k = i0 + u * 64 + lane;
    const int kk = k < ns ? k : ns - 1;
    if (F32) {
      const Rec32 r = ((const Rec32*)P.jrec32)[kk];
      xi[u] = (T)r.x;
      yi[u] = (T)r.y;
      zi[u] = (T)r.z;
      ei[u] = (T)r.e;
    } else {
      const Rec64 r = ((const Rec64*)P.jrec)[kk];
      xi[u] = (T)r.x;
      yi[u] = (T)r.y;
      zi[u] = (T)r.z;
      ei[u] = (T)r.e;
    }
    ax[u] = ay[u] = az[u] = (T)0;
  }
  for (int tj = t0; tj < t1; ++tj) {
    // FP32 form: targets relative to source tile J's anchor,
    // (x_i - A_I) - (A_J - A_I), the offset formed in FP64
    T xs[IPT], ys[IPT], zs[IPT];
    T sx = 0, sy = 0, sz = 0;
    if (F32) {
      const double* aI = P.ganchor + (size_t)ti * 4;
      const double* aJ = P.ganchor + (size_t)tj * 4;
      sx = (T)(aJ[0] - aI[0]);
      sy = (T)(aJ[1] - aI[1]);
      sz = (T)(aJ[2] - aI[2]);
    }
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
      xs[u] = xi[u] - sx;
      ys[u] = yi[u] - sy;
      zs[u] = zi[u] - sz;
    }
    const int j0 = tj * B, j1 = min(j0 + B, ns);
    for (int j = j0; j < j1; ++j) {
      T xj, yj, zj, mj, ej;
      if (F32) {
        const ConstRec32 cr = (ConstRec32)P.jrec32;
        xj = cr[j].x;
        yj = cr[j].y;
        zj = cr[j].z;
        mj = cr[j].m;
        ej = cr[j].e;
      } else {
        const ConstRec64 cr = (ConstRec64)P.jrec;
        xj = (T)cr[j].x;
        yj = (T)cr[j].y;
        zj = (T)cr[j].z;
        mj = (T)cr[j].m;
        ej = (T)cr[j].e;
      }
      // the sphere itself contributes nothing: d = 0 (and r^-3 = 0 when
      // unsoftened)
#pragma unroll
      for (int u = 0; u < IPT; ++u) {
        const T dx = xj - xs[u], dy = yj - ys[u], dz = zj - zs[u];
        const T t = ei[u] + ej;
        const T r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, t * t)));
        const T w = mj * inv_cube<SOFT>(r2, c15);
        ax[u] = fma(w, dx, ax[u]);
        ay[u] = fma(w, dy, ay[u]);
        az[u] = fma(w, dz, az[u]);
      }
    }
  }
  T* __restrict__ part = (T*)P.gpart;
#pragma unroll
  for (int u = 0; u < IPT; ++u) {
    const int k = i0 + u * 64 + lane;
    if (k < ns) {
      part[((size_t)it.tj * 3 + 0) * ns + k] = ax[u];
      part[((size_t)it.tj * 3 + 1) * ns + k] = ay[u];
      part[((size_t)it.tj * 3 + 2) * ns + k] = az[u];
    }
  }
}

// Sum of the partials of slot k over its rows q0 <= q < q1, in row order, FP64.
// The rows of a slot are every row below m0, then the first of segs rows b times,
// and every row after those.  Eight rows' loads are in flight.
template <typename T>
__device__ __forceinline__ void sum_rows(const T* __restrict__ part, size_t ns, int k, int q0,
                                         int q1, int m0, int b, int segs, double g[3]) {
  auto row = [&](int q) {
    return q < m0 ? q : (q < m0 + b ? m0 + (q - m0) * segs : b * (segs - 1) + q);
  };
  int q = q0;
  for (; q + 8 <= q1; q += 8) {
    T v[8][3];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int c = 0; c < 3; ++c) v[u][c] = part[((size_t)row(q + u) * 3 + c) * ns + k];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int c = 0; c < 3; ++c) g[c] += (double)v[u][c];
  }
  for (; q < q1; ++q)
    for (int c = 0; c < 3; ++c) g[c] += (double)part[((size_t)row(q) * 3 + c) * ns + k];
}

// 64 sorted slots per block, four threads per slot: each adds a quarter of the
// slot's rows -- per tile, super-tile, source split, or level-2 subtree of the
// tree -- and the four sums are added in order, FP64.
// (One thread per slot with three loads in flight took 5.3 us for 3 rows of
// 3,000 spheres and 11.5 us for 26 rows of 13,001, a chain of memory
// latencies.)  The gravity force G m_i sum is stored under the sphere's id.  With a
// perturber, its unsoftened pull G m_i M d/|d|^3 is added and each block
// stores the sum of its spheres' pulls (the reaction, reduced in a fixed order
// at the end of the step).
__global__ __launch_bounds__(kBlock) void k_grav_combine(const PileDev* __restrict__ piles,
                                                         const WorkItem* __restrict__ wl,
                                                         int precision) {
  __shared__ double red[4][3][64];
  __shared__ int failed[4];
  const WorkItem w = wl[blockIdx.x >> 2];
  const int base = w.base + (int)(blockIdx.x & 3) * 64;
  const PileDev& P = piles[w.pile];
  const int ns = P.ns;
  if (P.G == 0.0 || base >= ns) return;                    // uniform over the block
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // the search and the contact forces run beside this and may set the status:
  // each wave takes what it reads to the barrier, and the first decides by all
  const int st = P.status;
  if (lane == 0) failed[wv] = st;
  const int k = base + lane;
  double g[3] = {0.0, 0.0, 0.0};
  if (k < ns && st == 0) {
    // whole tiles below g_m0, the first row of each cut tile before the slot's own (the
    // reaction of that tile's targets), and every row from its own tile on; halves:
    // two reactions of each tile before its own, then one row per tile
    const int t = P.tree || P.g_segs == 1 ? 0 : k / P.g_tile;
    const int m0 = P.g_half ? 2 * t : P.g_m0, segs = P.g_segs;
    const int b = P.g_half ? P.g_np : max(0, t - m0);
    const int n = P.tree ? kTreeParts : (P.g_half ? P.g_nt + t : P.g_np - b * (segs - 1));
    const int q0 = n * wv / 4, q1 = n * (wv + 1) / 4;
    if (P.tree) sum_rows<double>(P.tpart, ns, k, q0, q1, n, 0, 1, g);
    else if (precision == 1) sum_rows<float>((const float*)P.gpart, ns, k, q0, q1, m0, b, segs, g);
    else sum_rows<double>((const double*)P.gpart, ns, k, q0, q1, m0, b, segs, g);
  }
  for (int c = 0; c < 3; ++c) red[wv][c][lane] = g[c];
  __syncthreads();
  if (wv != 0 || (failed[0] | failed[1] | failed[2] | failed[3]) != 0) return;
  double pull[3] = {0.0, 0.0, 0.0};
  if (k < ns) {
    for (int c = 0; c < 3; ++c)
      g[c] = ((red[0][c][lane] + red[1][c][lane]) + red[2][c][lane]) + red[3][c][lane];
    const uint32_t i = P.sidx[k];
    const Rec64 r = ((const Rec64*)P.jrec)[k];
    const double gm = P.G * r.m;
    for (int c = 0; c < 3; ++c) g[c] *= gm;
    if (P.pert_on) {
      const int nxt = P.parity ^ 1;
      const double d[3] = {P.pert_r[nxt][0] - r.x, P.pert_r[nxt][1] - r.y, P.pert_r[nxt][2] - r.z};
      const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
      const double f = gm * P.pert_M / (r2 * sqrt(r2));
      for (int c = 0; c < 3; ++c) {
        pull[c] = f * d[c];
        g[c] += pull[c];
      }
    }
    for (int c = 0; c < 3; ++c) P.gacc[c * ns + i] = g[c];
  }
  if (!P.pert_on) return;
  for (int off = 32; off > 0; off >>= 1)
    for (int c = 0; c < 3; ++c) pull[c] += __shfl_xor(pull[c], off);
  if (lane == 0)
    for (int c = 0; c < 3; ++c) P.ppart[(base / 64) * 3 + c] = pull[c];
}

}  // namespace

int gravity_tiles(int precision, int* tiles) {
  // default first: the fastest at 125k spheres on MI355X (measured)
  if (precision == 1) {
    tiles[0] = 64 * 16;
    tiles[1] = 64 * 8;
    tiles[2] = 64 * 4;
  } else {
    tiles[0] = 64 * 8;
    tiles[1] = 64 * 4;
    tiles[2] = 64 * 2;
  }
  return 3;
}

// Targets per lane amortise the sources' rotation (8 moves of 32 bits a step in
// FP32, 16 in FP64), and a tile needs a row of partial sums, so the tile grows with
// the pile as far as its blocks still fill the 256 compute units evenly: a block is
// one compute unit's, and the launch lasts as long as the unit with the most.  Step
// of one pile in us, FP64 by tiles of 128 / 192 / 256 / 512: 2,000 spheres 76 / 78 /
// 81 / 119, 3,500 85 / 82 / 85 / 121, 6,000 98 / 101 / 100 / 124, 9,000 122 / 124 /
// 116 / 127; by 256 / 512 whole / in halves as targets: 10,500 (231 blocks of 512, one
// round) 144 / 126 / -, 11,500 154 / 173 / 149, 13,001 161 / 174 / 158, 16,000 191 /
// 223 / 203, 20,000 - / 274 / 255; FP32: 2,000 75 / 76 / 76 / 108, 3,500
// 81 / 79 / 80 / 111, 8,000 104 / 100 / 98 / 105; by 512 / 768 / 1024: 40,000 455 /
// 491 / 562, 70,000 1208 / 1177 / 1257, 124,958 3491 / - / 3513.  An engine that fills
// the chip takes any of them, the larger the better above some 4,000 spheres, because
// of the rows: 256 piles of 500-20,000 in FP64, with 256 / halves / 512 above 11,264
// spheres 7.12 / 7.00 / 6.91 ms, 25 piles of 16,000 in FP32, 256 / 512, 1.94 / 1.65;
// 20 of 20,000 in FP64, halves / 512, 3.67 / 3.52, hence whole tiles past 18,432.
//
// A source tile is cut in segments (a row each) while that halves the one round of
// blocks, or where a few blocks beyond one or two rounds would double or half as much
// again the time: FP32, 12,000 spheres (300 blocks of 512) 137 -> 120 us, 16,000 (528)
// 168 -> 143; 14,500 (435) 139 either way.  In tiles of 1024 the last two, in
// quarters, end the launch evenly (124,958 spheres, FP32, gravity stage 3393 -> 3338
// us).  A given tile keeps its size and is cut by the same rule.
GravPlan gravity_plan(int precision, int64_t ns, int tile) {
  GravPlan p{tile, 1, 0, false};
  if (tile <= 0) {
    if (ns <= 2500) p.tile = 128;
    else if (ns <= 4200) p.tile = 192;
    else if (precision == 0) p.tile = ns <= 9500 ? 256 : 512;
    else p.tile = ns <= 8000 ? 256 : (ns <= 45000 ? 512 : (ns <= 98304 ? 768 : 1024));
    if (precision == 0 && ns > 22 * kHalvedTile && ns <= 18432) {
      p.half = true;
      p.segs = 2;
      return p;
    }
  }
  constexpr int64_t kUnits = 256;
  const int64_t nt = (ns + p.tile - 1) / p.tile, pairs = nt * (nt + 1) / 2;
  const int per = p.tile / grav_pair_waves(p.tile);    // sources of a wave, uncut
  if (pairs < 4 * kUnits) {
    for (int64_t b = pairs; per / p.segs % 128 == 0; b *= 2) {
      const bool uneven = b > kUnits && b < kUnits * 5 / 2 && b % kUnits < kUnits * 3 / 4;
      if (2 * b > kUnits && !uneven) break;
      p.segs *= 2;
    }
  } else if (p.tile == 1024) {
    p.segs = 4;
    p.m0 = (int)nt - 2;
  }
  if (p.segs == 1) p.m0 = (int)nt;
  return p;
}

void launch_gravity_records(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk) {
  hipLaunchKernelGGL(k_grav_records, dim3(nblk), dim3(kBlock), 0, st, piles, wl);
}

template <typename T, int IPT, int G = 1>
static void pairs_launch(hipStream_t st, const PileDev* piles, const GravPair* gp, int n,
                         bool soft) {
  if (soft)
    hipLaunchKernelGGL((k_grav_pairs<T, IPT, true, G>), dim3(n), dim3(64 * grav_pair_waves(64 * IPT)), 0, st,
                       piles, gp);
  else
    hipLaunchKernelGGL((k_grav_pairs<T, IPT, false, G>), dim3(n), dim3(64 * grav_pair_waves(64 * IPT)), 0, st,
                       piles, gp);
}

void launch_gravity_pairs(hipStream_t st, const PileDev* piles, const GravPair* gp, int nitems,
                          int precision, bool softened, int tile) {
  if (nitems <= 0) return;
  const int ipt = tile / 64;
  if (precision == 1) {
    if (ipt == 2) pairs_launch<float, 2>(st, piles, gp, nitems, softened);
    else if (ipt == 3) pairs_launch<float, 3>(st, piles, gp, nitems, softened);
    else if (ipt == 4) pairs_launch<float, 4>(st, piles, gp, nitems, softened);
    else if (ipt == 8) pairs_launch<float, 8>(st, piles, gp, nitems, softened);
    else if (ipt == 12) pairs_launch<float, 12>(st, piles, gp, nitems, softened);
    else pairs_launch<float, 16>(st, piles, gp, nitems, softened);
  } else {
    if (ipt == 2) pairs_launch<double, 2>(st, piles, gp, nitems, softened);
    else if (ipt == 3) pairs_launch<double, 3>(st, piles, gp, nitems, softened);
    else if (ipt == 4) pairs_launch<double, 4>(st, piles, gp, nitems, softened);
    else pairs_launch<double, 8>(st, piles, gp, nitems, softened);
  }
}

void launch_gravity_whole(hipStream_t st, const PileDev* piles, const GravPair* gp, int nitems,
                          bool softened) {
  if (nitems > 0) pairs_launch<double, kHalvedTile / 64, 2>(st, piles, gp, nitems, softened);
}

template <typename T, int IPT>
static void tiles_launch(hipStream_t st, const PileDev* piles, const GravItem* gl, int n,
                         bool soft) {
  if (soft)
    hipLaunchKernelGGL((k_grav_tiles<T, IPT, true>), dim3(n), dim3(64), 0, st, piles, gl);
  else
    hipLaunchKernelGGL((k_grav_tiles<T, IPT, false>), dim3(n), dim3(64), 0, st, piles, gl);
}

void launch_gravity_tiles(hipStream_t st, const PileDev* piles, const GravItem* gl, int nitems,
                          int precision, bool softened, int tile) {
  if (nitems <= 0) return;
  const int ipt = tile / 64;
  if (precision == 1) {
    if (ipt == 4) tiles_launch<float, 4>(st, piles, gl, nitems, softened);
    else if (ipt == 16) tiles_launch<float, 16>(st, piles, gl, nitems, softened);
    else tiles_launch<float, 8>(st, piles, gl, nitems, softened);
  } else {
    if (ipt == 2) tiles_launch<double, 2>(st, piles, gl, nitems, softened);
    else if (ipt == 8) tiles_launch<double, 8>(st, piles, gl, nitems, softened);
    else tiles_launch<double, 4>(st, piles, gl, nitems, softened);
  }
}

template <typename T, int IPT>
static void split_launch(hipStream_t st, const PileDev* piles, const GravItem* gl, int n, bool soft) {
  if (soft)
    hipLaunchKernelGGL((k_grav_split<T, IPT, true>), dim3(n), dim3(64), 0, st, piles, gl);
  else
    hipLaunchKernelGGL((k_grav_split<T, IPT, false>), dim3(n), dim3(64), 0, st, piles, gl);
}

int gravity_split_ipt(int precision, int tile) {
  // targets per lane of the per-target kernel: at most kSplitIpt64 (FP64) or
  // kSplitIpt32 (FP32), and never more than one tile holds
  const int cap = precision == 1 ? kSplitIpt32 : kSplitIpt64;
  return std::min(tile / 64, cap);
}

void launch_gravity_split(hipStream_t st, const PileDev* piles, const GravItem* gl, int nitems,
                          int precision, bool softened, int tile) {
  if (nitems <= 0) return;
  const int ipt = gravity_split_ipt(precision, tile);
  if (precision == 1) {
    if (ipt == 4) split_launch<float, 4>(st, piles, gl, nitems, softened);
    else if (ipt == 16) split_launch<float, 16>(st, piles, gl, nitems, softened);
    else split_launch<float, 8>(st, piles, gl, nitems, softened);
  } else {
    if (ipt == 2) split_launch<double, 2>(st, piles, gl, nitems, softened);
    else if (ipt == 8) split_launch<double, 8>(st, piles, gl, nitems, softened);
    else split_launch<double, 4>(st, piles, gl, nitems, softened);
  }
}

void launch_gravity_combine(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk,
                            int precision) {
  hipLaunchKernelGGL(k_grav_combine, dim3(nblk * 4), dim3(kBlock), 0, st, piles, wl, precision);
}

}  // namespace dem

// step_force.h -- the soft-sphere contact forces of one sphere, with the
// spring history carried from the previous step (Sec. 2.1: spring-dashpot
// normal and tangential forces, static friction, rolling and twisting
// friction, history kept while the contact lasts; Sec. 2.2.4: forces act at
// the contact point, lever arm of Eq. 8, torque of Eq. 9).  Included by the
// staged force kernel and by the fused per-pile step.
//
// Geometry (separation, distance, overlap) is always FP64; the force
// arithmetic runs in T (double, or float for the FP32-force form).  A wall
// is partner ns + w: infinite mass, no spin, moving rigidly; its reaction
// goes nowhere.
#pragma once
#include "dem_internal.h"

namespace dem {

namespace {

// Every floating-point operation of the contact model is rounded on its own
// (no fused multiply-add): a contact is evaluated by both of its spheres, in
// different places of the code, and both must see the same force.
template <typename T>
struct V3 {
  T x, y, z;
};

template <typename T>
__device__ __forceinline__ V3<T> mk(T x, T y, T z) {
  return V3<T>{x, y, z};
}
template <typename T>
__device__ __forceinline__ V3<T> operator+(V3<T> a, V3<T> b) {
#pragma clang fp contract(off)
  return mk(a.x + b.x, a.y + b.y, a.z + b.z);
}
template <typename T>
__device__ __forceinline__ V3<T> operator-(V3<T> a, V3<T> b) {
#pragma clang fp contract(off)
  return mk(a.x - b.x, a.y - b.y, a.z - b.z);
}
template <typename T>
__device__ __forceinline__ V3<T> operator*(T s, V3<T> a) {
#pragma clang fp contract(off)
  return mk(s * a.x, s * a.y, s * a.z);
}
template <typename T>
__device__ __forceinline__ T dotv(V3<T> a, V3<T> b) {
#pragma clang fp contract(off)
  return a.x * b.x + a.y * b.y + a.z * b.z;
}
template <typename T>
__device__ __forceinline__ V3<T> crossv(V3<T> a, V3<T> b) {
#pragma clang fp contract(off)
  return mk(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
template <typename T>
__device__ __forceinline__ T normv(V3<T> a) {
  return sqrt(dotv(a, a));
}

// Rescale a spring so that k |xi| does not exceed the friction limit.
template <typename T>
__device__ __forceinline__ V3<T> cap_spring(V3<T> xi, T k, T limit, bool* capped) {
#pragma clang fp contract(off)
  const T mag = normv(xi);
  if (k * mag > limit) {
    *capped = true;
    return (limit / (k * mag)) * xi;
  }
  *capped = false;
  return xi;
}

// What every contact of a pile's step reads from its table entry.
template <typename T>
struct PairCtx {
  int ns, na;
  const uint2* __restrict__ up_run;
  const uint32_t* __restrict__ new_j;
  const uint2* __restrict__ old_run;
  const uint32_t* __restrict__ old_j;
  const double* __restrict__ old_h;
  double* __restrict__ new_h;
  int periodic;
  double L;
  T h, kn, kt, kr, kq;
};

template <typename T>
__device__ __forceinline__ PairCtx<T> pair_ctx(const PileDev& P, const ContactParams& cp) {
  PairCtx<T> c;
  const int cur = P.parity, nxt = cur ^ 1;
  c.ns = P.ns;
  c.na = P.na;
  c.up_run = P.up_run[nxt];
  c.new_j = P.pair_j[nxt];
  c.old_run = P.up_run[cur];
  c.old_j = P.pair_j[cur];
  c.old_h = P.hist[cur];
  c.new_h = P.hist[nxt];
  c.periodic = P.periodic;
  c.L = P.box;
  c.h = (T)cp.dt;
  c.kn = (T)cp.k_n;
  c.kt = (T)cp.k_t;
  c.kr = (T)cp.k_r;
  c.kq = (T)cp.k_q;
  return c;
}

// What the force needs of one sphere of a contact: centre, radius, its
// aggregate's mass, the sphere's velocity and the aggregate's spin.
template <typename T>
struct Body {
  double x, y, z, s, M;
  V3<T> v, w;
};

template <typename T>
__device__ __forceinline__ Body<T> load_body(const PileDev& P, uint32_t i, int ns, int na) {
  Body<T> b;
  b.x = P.r[i];
  b.y = P.r[ns + i];
  b.z = P.r[2 * ns + i];
  b.s = P.s[i];
  const int A = P.agg[i];
  b.v = mk<T>(P.v[i], P.v[ns + i], P.v[2 * ns + i]);
  b.w = mk<T>(P.wA[A], P.wA[na + A], P.wA[2 * na + A]);
  b.M = P.M[A];
  return b;
}

// A contact's history is one aligned 64-byte row, moved as four 16-byte vectors:
// the sphere that finds it in another sphere's run touches one line for it
// instead of one per component.
__device__ __forceinline__ void load_row(const double* __restrict__ h, uint32_t p,
                                         double row[kHistRow]) {
  const double2* __restrict__ s = reinterpret_cast<const double2*>(h + (size_t)p * kHistRow);
#pragma unroll
  for (int k = 0; k < kHistRow / 2; ++k) {
    const double2 v = s[k];
    row[2 * k] = v.x;
    row[2 * k + 1] = v.y;
  }
}
__device__ __forceinline__ void store_row(double* __restrict__ h, uint32_t p,
                                          const double row[kHistRow]) {
  double2* __restrict__ d = reinterpret_cast<double2*>(h + (size_t)p * kHistRow);
#pragma unroll
  for (int k = 0; k < kHistRow / 2; ++k) d[k] = make_double2(row[2 * k], row[2 * k + 1]);
}

// Spring history of contact (a, b) from the previous step, searched in a's
// previous (sorted) upper run; zero for a new contact.  The first four
// keys are loaded together, so the usual short run costs one round of loads,
// not a chain.
template <typename T>
__device__ __forceinline__ void find_hist(const PairCtx<T>& c, uint32_t a, uint32_t b,
                                          T hs[kHist]) {
  const uint2 run = c.old_run[a];
  const uint32_t o = run.x, n = run.y, o1 = o + n;
  uint32_t kk[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) kk[u] = (uint32_t)u < n ? c.old_j[o + u] : 0xffffffffu;
  int pos = -1;
#pragma unroll
  for (int u = 3; u >= 0; --u)
    if (kk[u] == b) pos = u;
  uint32_t p = o + (uint32_t)pos;
  if (pos < 0 && n > 4u) {
    p = o + 4u;
    while (p < o1 && c.old_j[p] < b) ++p;
    if (!(p < o1 && c.old_j[p] == b)) p = o1;
  } else if (pos < 0) {
    p = o1;
  }
  if (p < o1) {
    double row[kHistRow];
    load_row(c.old_h, p, row);
    for (int k = 0; k < kHist; ++k) hs[k] = (T)row[k];
  } else {
    for (int k = 0; k < kHist; ++k) hs[k] = (T)0;
  }
}

// Force on a, torques on a and b about their centres, and the new spring
// history of one contact (a, b), a < b.
template <typename T>
struct ContactOut {
  V3<T> F, Ta, Tb;
  T hn[kHist];
  double delta, s_min;
};

// The contact model for normal n (from a towards b), overlap delta, lever
// arms la, lb along n, reduced mass mu, effective radius Rab, and the two
// bodies' velocities and spins at their centres.
template <typename T>
__device__ __forceinline__ void contact_model(const PairCtx<T>& c, const ContactParams& cp,
                                              V3<T> n, double delta_d, double la_d, double lb_d,
                                              double mu, double Rab_d, V3<T> va, V3<T> wa,
                                              V3<T> vb, V3<T> wb, const T hs[kHist],
                                              ContactOut<T>& out) {
#pragma clang fp contract(off)
  const T h = c.h, kn = c.kn, kt = c.kt, kr = c.kr, kq = c.kq;
  const T delta = (T)delta_d;
  const T li = (T)la_d;
  const T lj = (T)lb_d;
  // velocity of each body's material point at the contact point
  const V3<T> arm_i = li * n;
  const V3<T> arm_j = ((T)-1) * (lj * n);
  const V3<T> u = (vb + crossv(wb, arm_j)) - (va + crossv(wa, arm_i));
  const T un = dotv(u, n);
  const V3<T> ut = u - un * n;
  // dashpots from the restitution coefficients, aggregate reduced mass
  const T Cn = (T)(cp.damp_n * sqrt(cp.k_n * mu));
  const T Ct = (T)(cp.damp_t * sqrt(cp.k_t * mu));
  const T fn = -kn * delta + Cn * un;              // along n, on a
  T fN = kn * delta - Cn * un;                     // repulsive load for the caps
  fN = fN > (T)0 ? fN : (T)0;

  // sliding: spring on the tangent plane, static-friction cap
  V3<T> xt = mk(hs[0], hs[1], hs[2]);
  xt = xt - dotv(xt, n) * n;
  xt = xt + h * ut;
  bool slid;
  xt = cap_spring(xt, kt, (T)cp.mu_s * fN, &slid);
  const V3<T> FT = slid ? kt * xt : kt * xt + Ct * ut;

  // rolling and twisting: springs on the relative spin of the two bodies
  const T Rij = (T)Rab_d;
  const V3<T> dw = wb - wa;
  V3<T> xr = mk(hs[3], hs[4], hs[5]);
  xr = (xr - dotv(xr, n) * n) + (h * Rij) * crossv(dw, n);
  bool tmp;
  xr = cap_spring(xr, kr, (T)cp.mu_r * fN, &tmp);
  const V3<T> tau_r = Rij * crossv(n, kr * xr);
  T xq = hs[6] + h * Rij * dotv(dw, n);
  const T xq_lim = (T)cp.mu_t * fN;
  if (kq * fabs(xq) > xq_lim) xq = xq * (xq_lim / (kq * fabs(xq)));
  const V3<T> tau_q = (Rij * kq * xq) * n;

  out.F = fn * n + FT;
  out.Ta = crossv(arm_i, out.F) + tau_r + tau_q;
  out.Tb = crossv(arm_j, ((T)-1) * out.F) - tau_r - tau_q;
  out.hn[0] = xt.x;
  out.hn[1] = xt.y;
  out.hn[2] = xt.z;
  out.hn[3] = xr.x;
  out.hn[4] = xr.y;
  out.hn[5] = xr.z;
  out.hn[6] = xq;
}

// Contact of spheres a < b: separation by the minimum image, distance
// formed as the contact search forms it, contact point at la from a.
template <typename T>
__device__ __forceinline__ void sphere_contact(const PairCtx<T>& c, const ContactParams& cp,
                                               const Body<T>& a, const Body<T>& b,
                                               const T hs[kHist], ContactOut<T>& out) {
#pragma clang fp contract(off)
  double dx = b.x - a.x, dy = b.y - a.y, dz = b.z - a.z;
  if (c.periodic) {
    const double L = c.L, hL = 0.5 * L;
    if (dx > hL) dx -= L;
    else if (dx < -hL) dx += L;
    if (dy > hL) dy -= L;
    else if (dy < -hL) dy += L;
    if (dz > hL) dz -= L;
    else if (dz < -hL) dz += L;
  }
  // |d| from d^2 = (dx*dx + dy*dy) + dz*dz rounded step by step (no fused
  // multiply-add)
  const double dist =
      sqrt(rn_add(rn_add(rn_mul(dx, dx), rn_mul(dy, dy)), rn_mul(dz, dz)));
  const double si = a.s, sj = b.s;
  const double delta_d = (si + sj) - dist;
  const double li_d = (si * si - sj * sj + dist * dist) / (2.0 * dist);
  const double lj_d = dist - li_d;
  const double inv_d = 1.0 / dist;
  const V3<T> n = mk<T>(dx * inv_d, dy * inv_d, dz * inv_d);
  const double mu = a.M * b.M / (a.M + b.M);
  const double Rij_d = si * sj / (si + sj);
  contact_model<T>(c, cp, n, delta_d, li_d, lj_d, mu, Rij_d, a.v, a.w, b.v, b.w, hs, out);
  out.delta = delta_d;
  out.s_min = fmin(si, sj);
}

// Contact of sphere a with wall w: infinite mass, no spin; the contact
// point is the foot of the perpendicular and the normal points from the
// sphere into the wall.
template <typename T>
__device__ __forceinline__ void wall_contact(const PileDev& P, const PairCtx<T>& c,
                                             const ContactParams& cp, const Body<T>& a, int w,
                                             const T hs[kHist], ContactOut<T>& out) {
#pragma clang fp contract(off)
  const Grid& g = *P.grid;
  const double gap = wall_gap(P, w, g.wall_d[w], a.x, a.y, a.z);
  const V3<T> n = mk<T>((T)-P.wall[w][0], (T)-P.wall[w][1], (T)-P.wall[w][2]);
  const double delta_d = a.s - gap;
  const V3<T> vw = mk<T>((T)g.wall_v[w][0], (T)g.wall_v[w][1], (T)g.wall_v[w][2]);
  const V3<T> zero = mk<T>((T)0, (T)0, (T)0);
  contact_model<T>(c, cp, n, delta_d, gap, 0.0, a.M, a.s, a.v, a.w, vw, zero, hs, out);
  out.delta = delta_d;
  out.s_min = a.s;
}

// Shared memory of forces_group: the contacts' first index per sphere, and the
// force and torque of one round of contacts on the sphere they belong to.
template <int NT, int S>
struct ForceLds {
  uint32_t start[S + 1], lo0[S], up0[S], nlo[S], wave[S / 64];
  double res[6][NT];
};

// Spheres base .. base + S - 1 (S a multiple of 64, up to the pile's last) by
// the NT threads of a block: the force and torque of all their contacts, summed
// in canonical contact order -- contacts (j, i) with j < i by increasing j,
// then (i, j) by increasing j (walls last) -- into F and tau; the new spring
// history of their upper contacts.
//
// The contacts of the S spheres are numbered in that order and dealt to the
// threads one each, NT per round: a contact is a chain of dependent loads (its
// partner, the partner's aggregate, the previous run, the history) and some
// 700 FP64 instructions, so a thread that took its sphere's contacts in turn
// made the kernel as long as the sphere with the most of them.  Each contact
// leaves its force and torque on its sphere in LDS and one thread per sphere
// and axis adds them in order.  Measured, FP64, thread per sphere -> per
// contact: settled box of 6,400 spheres 32.4 -> 9.5 us (latency); 1M-sphere
// lattice, five contacts each, 275 -> 251 us (memory: consecutive threads hold
// consecutive upper contacts, so history reads and writes coalesce).
//
// A contact is evaluated by both of its spheres, with the same operands in the
// same order, so both see the same force; its lower sphere writes the history
// and checks it (sets bad on a non-finite force or an overlap beyond the limit).
// Every thread of the block calls this.
template <typename T, int NT, int S>
__device__ __forceinline__ void forces_group(const PileDev& P, const PairCtx<T>& c,
                                             const ContactParams& cp, int base,
                                             ForceLds<NT, S>& sh, bool& bad) {
  static_assert(S % 64 == 0 && (S & (S - 1)) == 0 && S <= NT, "a wave per 64 spheres, a search by halves");
  constexpr int K = (3 * S + NT - 1) / NT;   // sums (sphere, axis) of a thread
  const int ns = c.ns, na = c.na, tid = threadIdx.x;
  const int n = min(S, ns - base);
  if (tid < S) {
    // numbers of contacts, and their prefix sum
    const int i = base + tid;
    uint32_t nc = 0;
    if (tid < n) {
      const uint2 lo = P.lo_run[i], up = c.up_run[i];
      sh.lo0[tid] = lo.x;
      sh.up0[tid] = up.x;
      sh.nlo[tid] = lo.y;
      nc = lo.y + up.y;
    }
    uint32_t x = nc;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(x, off);
      if ((tid & 63) >= off) x += y;
    }
    sh.start[tid] = x - nc;
    if ((tid & 63) == 63) sh.wave[tid >> 6] = x;
  }
  __syncthreads();
  uint32_t total = 0;
  if constexpr (S == 64) {
    total = sh.wave[0];
    if (tid == 0) sh.start[S] = total;
  } else {
    uint32_t before = 0;
    for (int w = 0; w < S / 64; ++w) {
      if (w < tid >> 6) before += sh.wave[w];
      total += sh.wave[w];
    }
    if (tid < S) sh.start[tid] += before;
    if (tid == 0) sh.start[S] = total;
    __syncthreads();
  }
  double f[K] = {}, t[K] = {};
  for (uint32_t r0 = 0; r0 < total; r0 += NT) {
    const uint32_t e = r0 + (uint32_t)tid;
    if (e < total) {
      // the last sphere whose contacts start at or before e
      int l = 0;
#pragma unroll
      for (int w = S / 2; w > 0; w >>= 1)
        if (sh.start[l + w] <= e) l += w;
      const uint32_t i = (uint32_t)(base + l), k = e - sh.start[l], nlo = sh.nlo[l];
      const bool lower = k < nlo;
      const uint32_t p = sh.up0[l] + (k - nlo);            // upper contacts only
      const uint32_t j = lower ? P.lo_nbr[sh.lo0[l] + k] : c.new_j[p];
      const uint32_t a = lower ? j : i, b = lower ? i : j;
      T hs[kHist];
      ContactOut<T> r;
      const Body<T> ba = load_body<T>(P, a, ns, na);
      if (b < (uint32_t)ns) {
        const Body<T> bb = load_body<T>(P, b, ns, na);
        find_hist<T>(c, a, b, hs);
        sphere_contact<T>(c, cp, ba, bb, hs, r);
      } else {
        find_hist<T>(c, a, b, hs);
        wall_contact<T>(P, c, cp, ba, (int)(b - (uint32_t)ns), hs, r);
      }
      if (!lower) {
        double row[kHistRow];
        for (int q = 0; q < kHist; ++q) row[q] = (double)r.hn[q];
        row[kHist] = 0.0;
        store_row(c.new_h, p, row);
        if (!isfinite((double)r.F.x) || !isfinite((double)r.F.y) || !isfinite((double)r.F.z))
          bad = true;
        if (cp.max_overlap_frac > 0.0 && r.delta > cp.max_overlap_frac * r.s_min) bad = true;
      }
      sh.res[0][tid] = lower ? -(double)r.F.x : (double)r.F.x;
      sh.res[1][tid] = lower ? -(double)r.F.y : (double)r.F.y;
      sh.res[2][tid] = lower ? -(double)r.F.z : (double)r.F.z;
      sh.res[3][tid] = lower ? (double)r.Tb.x : (double)r.Ta.x;
      sh.res[4][tid] = lower ? (double)r.Tb.y : (double)r.Ta.y;
      sh.res[5][tid] = lower ? (double)r.Tb.z : (double)r.Ta.z;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const int ls = (tid + u * NT) % S, ax = (tid + u * NT) / S;
      if (ax >= 3) continue;
      const uint32_t e0 = max(sh.start[ls], r0), e1 = min(sh.start[ls + 1], r0 + (uint32_t)NT);
      for (uint32_t q = e0; q < e1; ++q) {
        f[u] += sh.res[ax][q - r0];
        t[u] += sh.res[3 + ax][q - r0];
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const int ls = (tid + u * NT) % S, ax = (tid + u * NT) / S;
    if (ax < 3 && ls < n) {
      P.F[ax * ns + base + ls] = f[u];
      P.tau[ax * ns + base + ls] = t[u];
    }
  }
  __syncthreads();                       // sh is free for the next group
}

}  // namespace

}  // namespace dem

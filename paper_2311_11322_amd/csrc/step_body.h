// step_body.h -- per-element device functions of the rigid-body part of a
// step: the fifth-order rotation step, kick/drift/rotate of one aggregate,
// member reconstruction, the per-pile cell grid from reduced partials, the
// member reduction (GetAccelAndTorque, which adds each sphere's gravity force
// to its contact force) and the end-of-step bookkeeping.  Included by the staged
// kernels and by the fused per-pile step, so both do the same arithmetic.
//
// Paper references: leapfrog for centres of mass and a fifth-order
// Runge-Kutta step for orientation and spin (Sec. 2.1-2.2); predicted member
// velocity (Eq. 3); aggregate acceleration and torque (Eqs. 5-7, 9).
#pragma once
#include "dem_internal.h"

namespace dem {

namespace {

// ---------------------------------------------------------------------------
// rotation: Euler's equations with quaternion kinematics, Cash-Karp RK5
// ---------------------------------------------------------------------------

// y = (q0..q3, w1..w3); body-frame principal moments I; torque N fixed in
// the space frame.  dq/dt = q (x) (0, w) / 2; I dw/dt = R^T N - w x (I w).
__device__ __forceinline__ void euler_deriv(const double y[7], const double I[3],
                                            const double N[3], double f[7]) {
  double R[9], Nb[3];
  quat_rot(y, R);
  rot_apply_T(R, N, Nb);
  const double w = y[0], x = y[1], yy = y[2], z = y[3];
  const double o1 = y[4], o2 = y[5], o3 = y[6];
  f[0] = 0.5 * (-x * o1 - yy * o2 - z * o3);
  f[1] = 0.5 * (w * o1 + yy * o3 - z * o2);
  f[2] = 0.5 * (w * o2 + z * o1 - x * o3);
  f[3] = 0.5 * (w * o3 + x * o2 - yy * o1);
  f[4] = (Nb[0] - (I[2] - I[1]) * o2 * o3) / I[0];
  f[5] = (Nb[1] - (I[0] - I[2]) * o3 * o1) / I[1];
  f[6] = (Nb[2] - (I[1] - I[0]) * o1 * o2) / I[2];
}

// Cash & Karp (1990) fifth-order weights and stage matrix.
__constant__ double ck_a[6][5] = {
    {0.0, 0.0, 0.0, 0.0, 0.0},
    {1.0 / 5.0, 0.0, 0.0, 0.0, 0.0},
    {3.0 / 40.0, 9.0 / 40.0, 0.0, 0.0, 0.0},
    {3.0 / 10.0, -9.0 / 10.0, 6.0 / 5.0, 0.0, 0.0},
    {-11.0 / 54.0, 5.0 / 2.0, -70.0 / 27.0, 35.0 / 27.0, 0.0},
    {1631.0 / 55296.0, 175.0 / 512.0, 575.0 / 13824.0, 44275.0 / 110592.0, 253.0 / 4096.0}};
__constant__ double ck_b[6] = {37.0 / 378.0, 0.0, 250.0 / 621.0, 125.0 / 594.0, 0.0,
                               512.0 / 1771.0};

__device__ void rk5_rotate(double y[7], const double I[3], const double N[3], double h) {
  double k[6][7];
  for (int st = 0; st < 6; ++st) {
    double ys[7];
    for (int c = 0; c < 7; ++c) {
      double acc = 0.0;
      for (int j = 0; j < st; ++j) acc += ck_a[st][j] * k[j][c];
      ys[c] = y[c] + h * acc;
    }
    euler_deriv(ys, I, N, k[st]);
  }
  for (int c = 0; c < 7; ++c) {
    double acc = 0.0;
    for (int st = 0; st < 6; ++st) acc += ck_b[st] * k[st][c];
    y[c] = y[c] + h * acc;
  }
  const double inv = 1.0 / sqrt(y[0] * y[0] + y[1] * y[1] + y[2] * y[2] + y[3] * y[3]);
  for (int c = 0; c < 4; ++c) y[c] *= inv;
}

// What a member's reconstruction needs of its aggregate after the drift: the new
// centre, orientation and space-frame spin, and the predicted centre velocity.
struct Moved {
  double r[3], q[4], w[3], vpred[3];
};

// One aggregate.  Step mode: v_A += h/2 a_A, r_A += h v_A (wrapped in a
// periodic cube), one RK5 step of (q, w_b) with the last torque.  Returns the
// new state with the space-frame spin w_A = R w_b and the predicted
// centre-of-mass velocity v_A + h/2 a_A (first bracket of Eq. 3) and, with
// store, writes it.  Init mode copies the state unchanged (evaluation at t0).
__device__ __forceinline__ Moved move_one(PileDev& P, int A, const ContactParams& cp, int mode,
                                          bool store) {
  const int na = P.na, cur = P.parity, nxt = cur ^ 1;
  const double h = cp.dt;
  double v[3], a[3], y[7];
  Moved m;
  for (int k = 0; k < 3; ++k) {
    v[k] = P.vA[cur][k * na + A];
    m.r[k] = P.rA[cur][k * na + A];
    a[k] = P.aA[cur][k * na + A];
  }
  for (int k = 0; k < 4; ++k) y[k] = P.q[cur][k * na + A];
  for (int k = 0; k < 3; ++k) y[4 + k] = P.wb[cur][k * na + A];
  if (mode == kModeStep) {
    for (int k = 0; k < 3; ++k) {
      v[k] += 0.5 * h * a[k];
      m.r[k] += h * v[k];
    }
    if (P.periodic) {
      const double L = P.box;
      for (int k = 0; k < 3; ++k) {
        if (m.r[k] >= L) m.r[k] -= L;
        if (m.r[k] < 0.0) m.r[k] += L;
      }
    }
    const double I[3] = {P.I[A], P.I[na + A], P.I[2 * na + A]};
    const double N[3] = {P.NA[cur][A], P.NA[cur][na + A], P.NA[cur][2 * na + A]};
    rk5_rotate(y, I, N, h);
  }
  double R[9];
  quat_rot(y, R);
  rot_apply(R, &y[4], m.w);
  const double hh = (mode == kModeStep) ? 0.5 * h : 0.0;
  for (int k = 0; k < 3; ++k) m.vpred[k] = v[k] + hh * a[k];
  for (int k = 0; k < 4; ++k) m.q[k] = y[k];
  if (!store) return m;
  for (int k = 0; k < 3; ++k) {
    P.vA[nxt][k * na + A] = v[k];
    P.rA[nxt][k * na + A] = m.r[k];
    P.wA[k * na + A] = m.w[k];
    P.wb[nxt][k * na + A] = y[4 + k];
  }
  for (int k = 0; k < 4; ++k) P.q[nxt][k * na + A] = y[k];
  if (A == 0 && P.pert_on) {
    // the perturber is one more body of the same leapfrog
    for (int k = 0; k < 3; ++k) {
      double pv = P.pert_v[cur][k], pr = P.pert_r[cur][k];
      if (mode == kModeStep) {
        pv += 0.5 * h * P.pert_a[cur][k];
        pr += h * pv;
      }
      P.pert_v[nxt][k] = pv;
      P.pert_r[nxt][k] = pr;
    }
  }
  return m;
}

// Partials of an empty set of spheres: bbox min / max and mass moments.
__device__ __forceinline__ void bbox_identity(double vals[kBbox]) {
  for (int k = 0; k < 3; ++k) {
    vals[k] = INFINITY;
    vals[3 + k] = -INFINITY;
  }
  for (int k = 6; k < kBbox; ++k) vals[k] = 0.0;
}

// Combine partials b into a (min, max, sums).
__device__ __forceinline__ void bbox_combine(double a[kBbox], const double b[kBbox]) {
  for (int k = 0; k < 3; ++k) a[k] = fmin(a[k], b[k]);
  for (int k = 3; k < 6; ++k) a[k] = fmax(a[k], b[k]);
  for (int k = 6; k < kBbox; ++k) a[k] += b[k];
}

// Reference point of the second moment: aggregate 0's centre before the step
// (the origin for a pile of given positions).
__device__ __forceinline__ void bbox_ref(const PileDev& P, double cref[3]) {
  const int na = P.na, cur = P.parity;
  for (int k = 0; k < 3; ++k) cref[k] = (na > 0 && !P.given) ? P.rA[cur][k * na] : 0.0;
}

// Bounding-box contribution of a sphere of a pile whose positions are given
// (stateless hooks).
__device__ __forceinline__ void given_vals(double x, double y, double z, double vals[kBbox]) {
  const double r[3] = {x, y, z};
  for (int k = 0; k < 3; ++k) vals[k] = vals[3 + k] = vals[7 + k] = r[k];
  vals[6] = 1.0;
  vals[10] = 0.0;
}

// Combine the partials of a wave's lanes, in every lane.
__device__ __forceinline__ void bbox_wave(double a[kBbox]) {
  for (int off = 32; off > 0; off >>= 1) {
    double o[kBbox];
    for (int k = 0; k < kBbox; ++k) o[k] = __shfl_xor(a[k], off);
    bbox_combine(a, o);
  }
}

// Bounding-box and mass-moment contributions of sphere i at (x, y, z), second
// moment about cref.
__device__ __forceinline__ void moments_one(const PileDev& P, int i, double x, double y, double z,
                                            const double cref[3], double vals[kBbox]) {
  const double r[3] = {x, y, z}, mi = P.m[i];
  double d2 = 0.0;
  for (int k = 0; k < 3; ++k) {
    vals[k] = r[k];
    vals[3 + k] = r[k];
    vals[7 + k] = mi * r[k];
    d2 += (r[k] - cref[k]) * (r[k] - cref[k]);
  }
  vals[6] = mi;
  vals[10] = mi * d2;
}

// Member reconstruction of sphere i of the aggregate in state (rA, q, wa, vp)
// (SetSpacePos / SetSpaceVel, Eq. 3): r_i = r_A + R b_i, v_i = vpred_A + w_A x
// (R b_i).  Its bounding-box and mass-moment contributions (second moment
// about cref) go into vals.
__device__ __forceinline__ void reconstruct_one(const PileDev& P, int i, const Moved& m,
                                                const double cref[3], double vals[kBbox]) {
  const int ns = P.ns;
  double R[9];
  quat_rot(m.q, R);
  const double bb[3] = {P.b[i], P.b[ns + i], P.b[2 * ns + i]};
  double d[3], wxd[3];
  rot_apply(R, bb, d);
  cross3(m.w, d, wxd);
  double r[3];
  for (int k = 0; k < 3; ++k) {
    r[k] = m.r[k] + d[k];
    P.r[k * ns + i] = r[k];
    P.v[k * ns + i] = m.vpred[k] + wxd[k];
  }
  moments_one(P, i, r[0], r[1], r[2], cref, vals);
}

// The new states of the aggregates of one block's NT spheres, in LDS.
template <int NT>
struct MoveLds {
  double v[13][NT];
};

// Kick, drift and rotation of the aggregates that own spheres base .. base +
// NT - 1, and the reconstruction of those spheres, by a block of NT threads.
// The spheres are grouped by aggregate, so at most NT aggregates take part;
// one whose members lie in several blocks is moved by each of them (the same
// arithmetic) and stored by the block of its first member.  Every thread of the
// block calls this; vals gets this thread's sphere's contribution.
template <int NT>
__device__ __forceinline__ void move_block(PileDev& P, int base, const ContactParams& cp, int mode,
                                           MoveLds<NT>& sh, const double cref[3],
                                           double vals[kBbox]) {
  const int ns = P.ns, tid = threadIdx.x, i = base + tid;
  if (P.na == 0 || P.given) {
    if (i < ns) given_vals(P.r[i], P.r[ns + i], P.r[2 * ns + i], vals);
    return;
  }
  const int a0 = P.agg[base], a1 = P.agg[min(base + NT, ns) - 1];
  if (tid <= a1 - a0) {
    const int A = a0 + tid;
    const Moved m = move_one(P, A, cp, mode, P.first[A] >= base);
    for (int k = 0; k < 3; ++k) {
      sh.v[k][tid] = m.r[k];
      sh.v[3 + k][tid] = m.w[k];
      sh.v[6 + k][tid] = m.vpred[k];
    }
    for (int k = 0; k < 4; ++k) sh.v[9 + k][tid] = m.q[k];
  }
  __syncthreads();
  if (i < ns) {
    const int l = P.agg[i] - a0;
    Moved m;
    for (int k = 0; k < 3; ++k) {
      m.r[k] = sh.v[k][l];
      m.w[k] = sh.v[3 + k][l];
      m.vpred[k] = sh.v[6 + k][l];
    }
    for (int k = 0; k < 4; ++k) m.q[k] = sh.v[9 + k][l];
    reconstruct_one(P, i, m, cref, vals);
  }
}

// Which cells an evaluation's bounding box sets: those of this evaluation (1),
// those of the next (2).
constexpr int kCellsNow = 1, kCellsNext = 2;

// A lane's value in every lane of the wave.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// The pile's centre of mass, bulk radius and stop rule, and the cells named by
// cells, from the reduced partials of all its spheres: by one wave, every lane
// with the same vals.
// Cells are at least one largest-sphere diameter; an open pile's grid spans
// its bounding box, or only the part of it within three rms radii of the
// centre of mass when that is smaller.
__device__ __forceinline__ void grid_from_vals(PileDev& P, const double vals[kBbox], int lane,
                                               int cells) {
  if (lane == 0) *P.runs = 0ull;       // the search of this evaluation starts
  Grid& gr = *P.grid;
  CellGrid g;
  bool finite = true;
  for (int k = 0; k < kBbox; ++k) finite = finite && isfinite(vals[k]);
  if (!finite) {
    if (lane == 0) atomicOr(&P.status, kStUnstable);
    return;
  }
  double com[3];
  for (int k = 0; k < 3; ++k) com[k] = vals[7 + k] / vals[6];
  // second moment about the centre of mass, from the one about the reference
  // point c: <|r - com|^2>_m = <|r - c|^2>_m - |com - c|^2
  double s2;
  {
    double c[3];
    bbox_ref(P, c);
    s2 = vals[10] / vals[6];
    for (int k = 0; k < 3; ++k) s2 -= (com[k] - c[k]) * (com[k] - c[k]);
    s2 = fmax(s2, 0.0);
  }
  const double R_bulk = sqrt(s2 * (5.0 / 3.0));
  if (P.periodic) {
    for (int k = 0; k < 3; ++k) {
      g.nc[k] = P.n_periodic;
      g.nbits[k] = P.bits;
    }
    g.lo[0] = g.lo[1] = g.lo[2] = 0.0;
    g.cell = P.box / (double)P.n_periodic;
  } else {
    double lo[3], hi[3];
    for (int k = 0; k < 3; ++k) {
      lo[k] = vals[k];
      hi[k] = vals[3 + k];
    }
    if (!P.tree && !P.given && P.na > 0) {
      // a few spheres thrown far from the rest would make every cell of a
      // bounding-box grid large and crowd the rest into a few cells; the
      // grid covers three rms radii about the centre of mass instead, and a
      // sphere beyond it falls into an outermost cell (clamping keeps two
      // spheres in contact within one cell of each other on every axis, so
      // the 27-cell search still finds every contact)
      const double h = 3.0 * sqrt(s2) + P.cell_min;
      for (int k = 0; k < 3; ++k) {
        lo[k] = fmax(lo[k], com[k] - h);
        hi[k] = fmax(lo[k], fmin(hi[k], com[k] + h));
      }
    }
    // cube cells; the key's 3 * bits bits go one at a time to the axis whose
    // cells are currently the longest, so an elongated pile (a tall box)
    // gets more cells along its long axis
    double ext[3];
    for (int k = 0; k < 3; ++k) {
      g.lo[k] = lo[k];
      ext[k] = hi[k] - lo[k];
    }
    int b0 = P.bits, b1 = P.bits, b2 = P.bits;
    if (!P.tree) {                       // the tree's pyramid needs a cubic code
      // handing out bits one by one to the axis with the longest cells (below
      // 10 bits, the first axis on a tie) takes the 3 * bits longest of the
      // lengths ext / 2^n, n < 10, of the axes: lane (axis, n) ranks its length
      const int axis = lane / 10, n = lane % 10;
      const double len = lane < 30 ? ldexp(axis == 0 ? ext[0] : (axis == 1 ? ext[1] : ext[2]), -n)
                                   : -1.0;
      int rank = 0;
#pragma unroll
      for (int q = 0; q < 30; ++q) {
        const double o = lane_value(len, q);
        rank += (o > len || (o == len && (q / 10 < axis || (q / 10 == axis && q % 10 < n)))) ? 1 : 0;
      }
      const uint64_t in = __ballot(lane < 30 && rank < 3 * P.bits);
      b0 = __popcll(in & 0x3ffull);
      b1 = __popcll(in & 0xffc00ull);
      b2 = __popcll(in & 0x3ff00000ull);
    }
    const int b[3] = {b0, b1, b2};
    double fit = 0.0;
    for (int k = 0; k < 3; ++k) {
      g.nbits[k] = b[k];
      g.nc[k] = 1 << b[k];
      fit = fmax(fit, ldexp(ext[k] * (1.0 + 1e-12), -b[k]));
    }
    g.cell = fmax(P.cell_min, fit + 1e-300);
  }
  g.inv_cell = 1.0 / g.cell;
  if (lane != 0) return;
  if (cells & kCellsNow) gr.c[P.parity] = g;
  if (cells & kCellsNext) gr.c[P.parity ^ 1] = g;
  for (int k = 0; k < 3; ++k) gr.com[k] = com[k];
  gr.R_bulk = R_bulk;
  if (P.stop_growth > 0.0) {
    // the stop rule: the first evaluation sets the reference radius; an
    // evaluation at or beyond stop_growth times it stops the pile (its step
    // is not committed, like a failure)
    if (!(P.R0 > 0.0)) {
      P.R0 = R_bulk;
    } else if (R_bulk >= P.stop_growth * P.R0) {
      atomicOr(&P.status, kStStopped);
    }
  }
}

// Time of this evaluation (the end of the step being taken, or the current
// time for an evaluation in place) and the walls at that time, wall w by lane
// w of a wave: displaced rigidly by A sin(omega t + phase), moving at
// A omega cos(omega t + phase).
__device__ __forceinline__ void walls_at(const PileDev& P, int lane, int mode, double dt) {
  Grid& g = *P.grid;
  const double t = (double)(P.step + (mode == kModeStep ? 1 : 0)) * dt;
  if (lane == 0) g.t = t;
  if (lane >= 6) return;
  double d = 0.0, v[3] = {0.0, 0.0, 0.0};
  if (lane < P.n_walls) {
    const double ph = rn_add(rn_mul(P.wall_omega, t), P.wall_phase);
    double sn, cs;
    sincos(ph, &sn, &cs);
    const double* n = P.wall[lane];
    const double* A = P.wall_amp[lane];
    const double shift =
        rn_add(rn_add(rn_mul(n[0], A[0]), rn_mul(n[1], A[1])), rn_mul(n[2], A[2]));
    d = rn_add(n[3], rn_mul(shift, sn));
    for (int k = 0; k < 3; ++k) v[k] = rn_mul(rn_mul(A[k], P.wall_omega), cs);
  }
  g.wall_d[lane] = d;
  for (int k = 0; k < 3; ++k) g.wall_v[lane][k] = v[k];
}

// The pile's block partials combined by a block of 256 threads (each thread its
// share in block order, then across the block), and from them its grid
// (grid_from_vals); the walls by another wave meanwhile.
struct GridLds {
  double red[4][kBbox];
};
__device__ __forceinline__ void grid_block(PileDev& P, int mode, double dt, int cells,
                                           GridLds& sh) {
  constexpr int kThreads = 256;
  double vals[kBbox];
  bbox_identity(vals);
  // unrolled so that several partials' loads are in flight (same order)
#pragma unroll 4
  for (int b = threadIdx.x; b < P.n_rblk; b += kThreads) {
    const double* p = P.bpart + (size_t)b * kBbox;
    bbox_combine(vals, p);
  }
  bbox_wave(vals);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0)
    for (int k = 0; k < kBbox; ++k) sh.red[wave][k] = vals[k];
  __syncthreads();
  if (wave == 1) walls_at(P, lane, mode, dt);
  if (wave != 0) return;
  for (int j = 1; j < kThreads / 64; ++j) bbox_combine(vals, sh.red[j]);
  grid_from_vals(P, vals, lane, cells);
}

// Force on sphere i: its contact force plus, in a pile with gravity, its
// gravity force (added last, after the contacts).
__device__ __forceinline__ void sphere_force(const PileDev& P, int i, double f[3]) {
  const int ns = P.ns;
  for (int k = 0; k < 3; ++k) f[k] = P.F[k * ns + i];
  if (P.G != 0.0)
    for (int k = 0; k < 3; ++k) f[k] += P.gacc[k * ns + i];
}

// One member's share of F_A and N_A: f_i and (R b_i) x f_i + tau_i.
__device__ __forceinline__ void add_member(const double R[9], const double f[3],
                                           const double bb[3], const double tau[3], double FA[3],
                                           double NA[3]) {
  double d[3], dxf[3];
  rot_apply(R, bb, d);
  cross3(d, f, dxf);
  for (int k = 0; k < 3; ++k) {
    FA[k] += f[k];
    NA[k] += dxf[k] + tau[k];
  }
}

// Members of aggregate A added in member order, read directly.
__device__ __forceinline__ void reduce_members_direct(const PileDev& P, int A, const double R[9],
                                                      double FA[3], double NA[3]) {
  const int ns = P.ns;
  // unrolled so that two members' loads are in flight (same order of sums)
#pragma unroll 2
  for (int i = P.first[A], i1 = i + P.count[A]; i < i1; ++i) {
    double f[3];
    sphere_force(P, i, f);
    const double bb[3] = {P.b[i], P.b[ns + i], P.b[2 * ns + i]};
    const double tau[3] = {P.tau[i], P.tau[ns + i], P.tau[2 * ns + i]};
    add_member(R, f, bb, tau, FA, NA);
  }
}

// The paper's original member search (ablation): every sphere of the pile
// tested for membership, in order.
__device__ __forceinline__ void reduce_members_scan(const PileDev& P, int A, const double R[9],
                                                    double FA[3], double NA[3]) {
  const int ns = P.ns;
  for (int i = 0; i < ns; ++i) {
    if (P.agg[i] != A) continue;
    double f[3];
    sphere_force(P, i, f);
    const double bb[3] = {P.b[i], P.b[ns + i], P.b[2 * ns + i]};
    const double tau[3] = {P.tau[i], P.tau[ns + i], P.tau[2 * ns + i]};
    add_member(R, f, bb, tau, FA, NA);
  }
}

// a_A = F_A / M + g, N_A; in step mode the closing half kick and the spin-up
// increment about +z through the pile's centre of mass.
__device__ __forceinline__ void reduce_tail(const PileDev& P, int A, const double R[9],
                                            const double FA[3], const double NA[3],
                                            const ContactParams& cp, int mode) {
  const int na = P.na, nxt = P.parity ^ 1;
  const double M = P.M[A];
  double a[3];
  for (int k = 0; k < 3; ++k) {
    a[k] = FA[k] / M + P.gfield[k];      // a uniform field adds no torque
    P.aA[nxt][k * na + A] = a[k];
    P.NA[nxt][k * na + A] = NA[k];
  }
  if (mode == kModeStep) {
    double v[3];
    for (int k = 0; k < 3; ++k) v[k] = P.vA[nxt][k * na + A] + 0.5 * cp.dt * a[k];
    if (P.spin_dw != 0.0) {
      // spin-up: w += dw z-hat about the pile's centre of mass
      const double* com = P.grid->com;
      const double dw = P.spin_dw;
      const double rel[3] = {P.rA[nxt][A] - com[0], P.rA[nxt][na + A] - com[1],
                             P.rA[nxt][2 * na + A] - com[2]};
      const double z[3] = {0.0, 0.0, dw};
      double dv[3], dwb[3];
      cross3(z, rel, dv);
      for (int k = 0; k < 3; ++k) v[k] += dv[k];
      rot_apply_T(R, z, dwb);
      for (int k = 0; k < 3; ++k) P.wb[nxt][k * na + A] += dwb[k];
    }
    for (int k = 0; k < 3; ++k) P.vA[nxt][k * na + A] = v[k];
  }
}

// Per pile, by one wave: commit the step (flip the ping-pong halves) unless the
// pile failed during it, in which case its state stays at the failing step's
// start and the step index is recorded; the perturber's reaction and kick.  failed:
// the pile's status by the caller, as in k_fused the same launch set it by atomics.
__device__ __forceinline__ void finish_one(PileDev& P, int lane, int mode, double dt, bool failed) {
  if (failed) {
    if (lane == 0 && P.fail_step < 0) P.fail_step = P.step;
    return;
  }
  const int nxt = P.parity ^ 1;
  // reaction on the perturber: minus the pull on every sphere, each lane adding
  // its share of the partials in order, then across the lanes
  double f[3] = {0.0, 0.0, 0.0};
  if (P.pert_on) {
    for (int b = lane; b < (P.ns + 63) / 64; b += 64)
      for (int k = 0; k < 3; ++k) f[k] += P.ppart[b * 3 + k];
    for (int off = 32; off > 0; off >>= 1)
      for (int k = 0; k < 3; ++k) f[k] += __shfl_xor(f[k], off);
  }
  if (lane != 0) return;
  if (P.pert_on) {
    // its closing half kick
    for (int k = 0; k < 3; ++k) {
      const double a = -f[k] / P.pert_M;
      P.pert_a[nxt][k] = a;
      if (mode == kModeStep) P.pert_v[nxt][k] += 0.5 * dt * a;
    }
  }
  P.n_pairs = (uint32_t)(__hip_atomic_load(P.runs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32);
  P.parity = nxt;
  if (mode == kModeStep) P.step += 1;
}

}  // namespace

}  // namespace dem

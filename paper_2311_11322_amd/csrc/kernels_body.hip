// kernels_body.hip -- rigid-body kernels: aggregate set-up, kick/drift/rotate,
// member reconstruction, reduction onto aggregates, end-of-step bookkeeping.
//
// Paper references: aggregate mass and centre of mass (Eqs. 1-2); the
// appendix table of aggregate functions (CountPart, GetCOM, GetAxesAndSpin,
// SetBodyPos, SetMassDEM, SetSpacePos/Spin/Vel, GetAccelAndTorque); leapfrog
// for centres of mass and a fifth-order Runge-Kutta step for orientation and
// spin (Sec. 2.1-2.2); predicted member velocity (Eq. 3); aggregate
// acceleration and torque (Eqs. 5-7, 9).
#include "step_body.h"
#include "step_contact.h"

namespace dem {

namespace {

// ---------------------------------------------------------------------------
// set-up of one aggregate
// ---------------------------------------------------------------------------

// Symmetric 3x3 eigen-decomposition by cyclic Jacobi plane rotations.  a is
// overwritten (eigenvalues on the diagonal); columns of V are eigenvectors.
__device__ void jacobi_eig3(double a[3][3], double V[3][3]) {
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) V[i][j] = (i == j) ? 1.0 : 0.0;
  const int P[3] = {0, 0, 1}, Q[3] = {1, 2, 2};
  for (int sweep = 0; sweep < 50; ++sweep) {
    const double off = a[0][1] * a[0][1] + a[0][2] * a[0][2] + a[1][2] * a[1][2];
    const double dia = a[0][0] * a[0][0] + a[1][1] * a[1][1] + a[2][2] * a[2][2];
    if (off == 0.0 || off <= 1e-34 * dia) break;
    for (int k = 0; k < 3; ++k) {
      const int p = P[k], q = Q[k];
      const double apq = a[p][q];
      if (apq == 0.0) continue;
      const double zeta = (a[q][q] - a[p][p]) / (2.0 * apq);
      const double t = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
      const double c = 1.0 / sqrt(1.0 + t * t);
      const double s = t * c;
      a[p][p] -= t * apq;
      a[q][q] += t * apq;
      a[p][q] = a[q][p] = 0.0;
      const int r = 3 - p - q;
      const double arp = a[r][p], arq = a[r][q];
      a[r][p] = a[p][r] = c * arp - s * arq;
      a[r][q] = a[q][r] = s * arp + c * arq;
      for (int i = 0; i < 3; ++i) {
        const double vip = V[i][p], viq = V[i][q];
        V[i][p] = c * vip - s * viq;
        V[i][q] = s * vip + c * viq;
      }
    }
  }
}

// Unit quaternion of a proper rotation matrix (largest-component branch).
__device__ void rot_to_quat(const double R[3][3], double q[4]) {
  const double t0 = R[0][0] + R[1][1] + R[2][2];
  double w, x, y, z;
  if (t0 >= R[0][0] && t0 >= R[1][1] && t0 >= R[2][2]) {
    const double f = 2.0 * sqrt(1.0 + t0);
    w = 0.25 * f;
    x = (R[2][1] - R[1][2]) / f;
    y = (R[0][2] - R[2][0]) / f;
    z = (R[1][0] - R[0][1]) / f;
  } else if (R[0][0] >= R[1][1] && R[0][0] >= R[2][2]) {
    const double f = 2.0 * sqrt(1.0 + R[0][0] - R[1][1] - R[2][2]);
    w = (R[2][1] - R[1][2]) / f;
    x = 0.25 * f;
    y = (R[0][1] + R[1][0]) / f;
    z = (R[0][2] + R[2][0]) / f;
  } else if (R[1][1] >= R[2][2]) {
    const double f = 2.0 * sqrt(1.0 + R[1][1] - R[0][0] - R[2][2]);
    w = (R[0][2] - R[2][0]) / f;
    x = (R[0][1] + R[1][0]) / f;
    y = 0.25 * f;
    z = (R[1][2] + R[2][1]) / f;
  } else {
    const double f = 2.0 * sqrt(1.0 + R[2][2] - R[0][0] - R[1][1]);
    w = (R[1][0] - R[0][1]) / f;
    x = (R[0][2] + R[2][0]) / f;
    y = (R[1][2] + R[2][1]) / f;
    z = 0.25 * f;
  }
  const double inv = 1.0 / sqrt(w * w + x * x + y * y + z * z);
  q[0] = w * inv;
  q[1] = x * inv;
  q[2] = y * inv;
  q[3] = z * inv;
}

// One thread per aggregate: CountPart/GetCOM (Eqs. 1-2), the inertia tensor
// about the centre of mass with each sphere's own 2/5 m s^2, its principal
// axes (GetAxesAndSpin) as a proper rotation and quaternion, body offsets
// (SetBodyPos) and the body-frame spin.  pos_in/vel_in/spin_in are the
// caller's row-major arrays copied to the device.
__global__ __launch_bounds__(kBlock) void k_setup(const PileDev* __restrict__ piles,
                                                  const WorkItem* __restrict__ wl,
                                                  const double* __restrict__ pos_in,
                                                  const double* __restrict__ vel_in,
                                                  const double* __restrict__ spin_in) {
  const WorkItem w = wl[xcd_block(blockIdx.x, gridDim.x)];
  const PileDev& P = piles[w.pile];
  const int A = w.base + threadIdx.x;
  if (A >= P.na) return;
  const int i0 = P.first[A], n = P.count[A];
  double M = 0.0, c[3] = {0.0, 0.0, 0.0};
  for (int i = i0; i < i0 + n; ++i) M += P.m[i];
  for (int i = i0; i < i0 + n; ++i)
    for (int k = 0; k < 3; ++k) c[k] += P.m[i] * pos_in[3 * i + k];
  for (int k = 0; k < 3; ++k) c[k] /= M;
  double T[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
  for (int i = i0; i < i0 + n; ++i) {
    const double d[3] = {pos_in[3 * i] - c[0], pos_in[3 * i + 1] - c[1], pos_in[3 * i + 2] - c[2]};
    const double mi = P.m[i];
    const double tr = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + 0.4 * P.s[i] * P.s[i];
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) T[a][b] += mi * ((a == b ? tr : 0.0) - d[a] * d[b]);
  }
  double V[3][3];
  jacobi_eig3(T, V);
  // right-handed axes
  const double c0[3] = {V[0][0], V[1][0], V[2][0]}, c1[3] = {V[0][1], V[1][1], V[2][1]},
               c2[3] = {V[0][2], V[1][2], V[2][2]};
  double x01[3];
  cross3(c0, c1, x01);
  if (dot3(x01, c2) < 0.0)
    for (int a = 0; a < 3; ++a) V[a][2] = -V[a][2];
  double q[4], R[9];
  rot_to_quat(V, q);
  quat_rot(q, R);
  for (int i = i0; i < i0 + n; ++i) {
    const double d[3] = {pos_in[3 * i] - c[0], pos_in[3 * i + 1] - c[1], pos_in[3 * i + 2] - c[2]};
    double bb[3];
    rot_apply_T(R, d, bb);
    for (int k = 0; k < 3; ++k) P.b[k * P.ns + i] = bb[k];
  }
  const int cur = P.parity;
  P.M[A] = M;
  for (int k = 0; k < 3; ++k) {
    P.I[k * P.na + A] = T[k][k];
    double x = c[k];
    if (P.periodic) {
      const double L = P.box;
      x = x - L * floor(x / L);
      if (x >= L) x -= L;
    }
    P.rA[cur][k * P.na + A] = x;
    P.vA[cur][k * P.na + A] = vel_in ? vel_in[3 * A + k] : 0.0;
    P.aA[cur][k * P.na + A] = 0.0;
    P.NA[cur][k * P.na + A] = 0.0;
  }
  double ws[3] = {0.0, 0.0, 0.0}, wbv[3];
  if (spin_in)
    for (int k = 0; k < 3; ++k) ws[k] = spin_in[3 * A + k];
  rot_apply_T(R, ws, wbv);
  for (int k = 0; k < 3; ++k) P.wb[cur][k * P.na + A] = wbv[k];
  for (int k = 0; k < 4; ++k) P.q[cur][k * P.na + A] = q[k];
}

// ---------------------------------------------------------------------------
// kick, drift, rotation and member reconstruction (SetSpacePos / SetSpaceSpin /
// SetSpaceVel, Eq. 3)
// ---------------------------------------------------------------------------

// One thread per sphere, after the aggregates of the block's spheres have been
// moved (move_block; as two launches, one thread per aggregate and one per
// sphere, it took 12.2 us for 6,400 spheres and takes 9.3).  Each block also
// writes the bounding box and mass moments of its spheres for the per-pile
// grid.  With bin, a pile of row-major cells bins the sphere in the same
// thread, on the cells of the evaluation before: a sphere that has left them
// falls into an outermost cell, which keeps touching spheres in neighbouring
// cells, so the contacts found are the same.
__global__ __launch_bounds__(kBlock) void k_move(PileDev* __restrict__ piles,
                                                 const WorkItem* __restrict__ wl, ContactParams cp,
                                                 int mode, int bin) {
  __shared__ MoveLds<kBlock> sh;
  const WorkItem w = wl[xcd_block(blockIdx.x, gridDim.x)];
  PileDev& P = piles[w.pile];
  if (P.status != 0) return;
  double vals[kBbox];
  bbox_identity(vals);
  double cref[3];
  bbox_ref(P, cref);
  move_block<kBlock>(P, w.base, cp, mode, sh, cref, vals);
  const int i = w.base + (int)threadIdx.x;
  if (bin && P.rows && i < P.ns) {
    const uint32_t key = sphere_key(P, P.grid->c[P.parity], vals[0], vals[1], vals[2],
                                    P.n_big > 0 ? P.s[i] : 0.0);
    P.key[i] = key;
    P.num[i] = atomicAdd(&P.cell_cnt[key], 1u);
  }
  // block reduction (wave shuffles, then across the 4 waves through LDS)
  __shared__ double red[4][kBbox];
  for (int off = 32; off > 0; off >>= 1) {
    for (int k = 0; k < 3; ++k) vals[k] = fmin(vals[k], __shfl_xor(vals[k], off));
    for (int k = 3; k < 6; ++k) vals[k] = fmax(vals[k], __shfl_xor(vals[k], off));
    for (int k = 6; k < kBbox; ++k) vals[k] += __shfl_xor(vals[k], off);
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0)
    for (int k = 0; k < kBbox; ++k) red[wave][k] = vals[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    double* out = P.bpart + (size_t)(w.base / kBlock) * kBbox;
    for (int k = 0; k < kBbox; ++k) {
      double x = red[0][k];
      for (int j = 1; j < 4; ++j) {
        const double y = red[j][k];
        x = (k < 3) ? fmin(x, y) : (k < 6 ? fmax(x, y) : x + y);
      }
      out[k] = x;
    }
  }
}

// One block per listed pile: its grid from the block partials (grid_block).  A
// pile that bins on carried cells gets those of its next evaluation too.
__global__ __launch_bounds__(256) void k_grid(PileDev* __restrict__ piles,
                                              const int32_t* __restrict__ plist, int mode,
                                              double dt) {
  __shared__ GridLds sh;
  PileDev& P = piles[plist ? plist[blockIdx.x] : (int)blockIdx.x];
  if (P.status != 0) return;
  grid_block(P, mode, dt, P.rows ? kCellsNow | kCellsNext : kCellsNow, sh);
}

// ---------------------------------------------------------------------------
// GetAccelAndTorque (Eqs. 5-7, 9) and the closing half kick
// ---------------------------------------------------------------------------

// One thread per aggregate: F_A = sum F_i (F_i a member's contact force,
// plus its gravity force in a pile with gravity), a_A = F_A / M + g,
// N_A = sum [ (R b_i) x F_i + tau_i ] over the members in order, and in step
// mode v_A += h/2 a_A followed by the spin-up increment about +z through the
// pile's centre.  Members are added in member order, read in one of two
// ways with the same arithmetic:
// * direct (launches of few aggregates): each lane reads its members;
// * staged (many aggregates): lanes ~5 spheres apart would re-fetch each
//   line once per member, the lines leaving L2 between a wave's member
//   iterations, so a wave's 64 aggregates -- one contiguous run of
//   spheres -- pass through the wave's LDS slice 64 spheres at a time (one
//   coalesced load per array) and each lane adds the members in the slice.
// The launch chooses (stage: at least kReduceStageMin aggregates) unless the
// pile's tuning fixes one way.
__device__ __forceinline__ void reduce_block(const PileDev& P, const WorkItem& w,
                                             const ContactParams& cp, int mode, int stage,
                                             double (*sh_all)[9][64]) {
  const int na = P.na, ns = P.ns, nxt = P.parity ^ 1;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int a0 = w.base + wv * 64;               // the wave's first aggregate
  if (a0 >= na || P.status != 0) return;         // uniform over the wave
  const int A = a0 + lane;
  const bool own = A < na;
  double (*sh)[64] = sh_all[wv];
  double R[9];
  if (own) {
    double q[4];
    for (int k = 0; k < 4; ++k) q[k] = P.q[nxt][k * na + A];
    quat_rot(q, R);
  }
  double FA[3] = {0.0, 0.0, 0.0}, NA[3] = {0.0, 0.0, 0.0};
  if (P.member_scan != 0) {
    // ablation of the paper's original routines: every sphere of the pile
    // tested for membership, in order
    if (own) reduce_members_scan(P, A, R, FA, NA);
  } else if (P.member_read == 1 || (P.member_read == 0 && !stage)) {
    if (own) reduce_members_direct(P, A, R, FA, NA);
  } else {
    const int a_last = min(a0 + 64, na) - 1;
    const int s0 = P.first[a0], s1 = P.first[a_last] + P.count[a_last];
    const int m0 = own ? P.first[A] : 0, m1 = own ? m0 + P.count[A] : 0;
    // Loads through the global address space: a generic load would also
    // count against the LDS wait counter that the slice reads wait on.  The
    // next slice's nine loads are in flight while the lanes add this one.
    typedef const __attribute__((address_space(1))) double* GlobalD;
    const GlobalD gF = (GlobalD)P.F, gb = (GlobalD)P.b, gt = (GlobalD)P.tau;
    const GlobalD gg = (GlobalD)P.gacc;
    const bool grav = P.G != 0.0;
    double v[9];
    auto fetch = [&](int c) {
      const int t = c + lane;
      if (t < s1)
        for (int k = 0; k < 3; ++k) {
          v[k] = gF[k * ns + t];
          if (grav) v[k] += gg[k * ns + t];     // gravity after the contacts
          v[3 + k] = gb[k * ns + t];
          v[6 + k] = gt[k * ns + t];
        }
    };
    fetch(s0);
    for (int c0 = s0; c0 < s1; c0 += 64) {
      if (c0 + lane < s1)
        for (int k = 0; k < 9; ++k) sh[k][lane] = v[k];
      if (c0 + 64 < s1) fetch(c0 + 64);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      for (int i = max(m0, c0), i1 = min(m1, c0 + 64); i < i1; ++i) {
        const int l = i - c0;
        const double f[3] = {sh[0][l], sh[1][l], sh[2][l]};
        const double bb[3] = {sh[3][l], sh[4][l], sh[5][l]};
        const double tau[3] = {sh[6][l], sh[7][l], sh[8][l]};
        add_member(R, f, bb, tau, FA, NA);
      }
      // every lane has read the slice before the next pass overwrites it
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
  if (!own) return;
  reduce_tail(P, A, R, FA, NA, cp, mode);
}

__global__ __launch_bounds__(kBlock) void k_reduce(PileDev* __restrict__ piles,
                                                   const WorkItem* __restrict__ wl,
                                                   ContactParams cp, int mode, int stage,
                                                   int finish) {
  __shared__ double sh_all[kBlock / 64][9][64];
  __shared__ uint32_t last;
  const WorkItem w = wl[xcd_block(blockIdx.x, gridDim.x)];
  PileDev& P = piles[w.pile];
  reduce_block(P, w, cp, mode, stage, sh_all);
  if (!finish) return;
  // The last block to get here ends the pile's step.  It writes the table
  // entry that the other blocks have finished reading: their count comes after
  // their last use of it.
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t* done = reinterpret_cast<uint32_t*>(P.runs + 1);
    const uint32_t n = (uint32_t)((P.na + kBlock - 1) / kBlock);
    last = atomicAdd(done, 1u) == n - 1u ? 1u : 0u;
    if (last) atomicExch(done, 0u);
  }
  __syncthreads();
  if (last && threadIdx.x < 64) finish_one(P, threadIdx.x, mode, cp.dt, P.status != 0);
}

// One wave per pile: commit the step (flip the ping-pong halves) unless the
// pile failed during it, in which case its state stays at the failing step's
// start and the step index is recorded.
__global__ __launch_bounds__(64) void k_finish(PileDev* __restrict__ piles, int mode, double dt) {
  PileDev& P = piles[blockIdx.x];
  if (P.fused) return;                       // k_fused finishes it
  finish_one(P, threadIdx.x, mode, dt, P.status != 0);
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t value, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

// A state read-out: one thread per row of a field.
__global__ __launch_bounds__(kBlock) void k_read(ReadList list) {
  int q = 0;
  while (q + 1 < list.n && (int)blockIdx.x >= list.f[q + 1].block0) ++q;
  const ReadField f = list.f[q];
  const int64_t n = f.n, i = (int64_t)((int)blockIdx.x - f.block0) * kBlock + threadIdx.x;
  if (i >= n) return;
  double* out = f.dst + i * f.comps;
  if (f.spin) {
    // R(q) w_b, every product and sum rounded
    const double w = f.src[i], x = f.src[n + i], y = f.src[2 * n + i], z = f.src[3 * n + i];
    auto two = [](double a) { return rn_mul(2.0, a); };
    auto mul = [](double a, double b) { return rn_mul(a, b); };
    auto add = [](double a, double b) { return rn_add(a, b); };
    const double R[9] = {add(1.0, -two(add(mul(y, y), mul(z, z)))),
                         two(add(mul(x, y), -mul(w, z))), two(add(mul(x, z), mul(w, y))),
                         two(add(mul(x, y), mul(w, z))), add(1.0, -two(add(mul(x, x), mul(z, z)))),
                         two(add(mul(y, z), -mul(w, x))), two(add(mul(x, z), -mul(w, y))),
                         two(add(mul(y, z), mul(w, x))), add(1.0, -two(add(mul(x, x), mul(y, y))))};
    const double o[3] = {f.add[i], f.add[n + i], f.add[2 * n + i]};
    for (int c = 0; c < 3; ++c)
      out[c] = add(add(mul(R[3 * c], o[0]), mul(R[3 * c + 1], o[1])), mul(R[3 * c + 2], o[2]));
    return;
  }
  for (int c = 0; c < f.comps; ++c) {
    const double v = f.src[c * n + i];
    out[c] = f.add ? v + f.add[c * n + i] : v;
  }
}

// First canonical contact of every sphere: the prefix sum of the lengths of the
// upper runs, by one block (each thread a contiguous share).
constexpr int kOffsetThreads = 1024;
__global__ __launch_bounds__(kOffsetThreads) void k_read_offsets(const uint2* __restrict__ run,
                                                                 int ns,
                                                                 uint32_t* __restrict__ offset) {
  __shared__ uint32_t wsum[kOffsetThreads / 64];
  const int tid = threadIdx.x, per = (ns + kOffsetThreads - 1) / kOffsetThreads;
  const int b0 = min(ns, tid * per), b1 = min(ns, b0 + per);
  uint32_t sum = 0;
  for (int i = b0; i < b1; ++i) sum += run[i].y;
  uint32_t x = sum;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off);
    if ((tid & 63) >= off) x += y;
  }
  if ((tid & 63) == 63) wsum[tid >> 6] = x;
  __syncthreads();
  uint32_t at = x - sum;
  for (int w = 0; w < tid >> 6; ++w) at += wsum[w];
  for (int i = b0; i < b1; ++i) {
    offset[i] = at;
    at += run[i].y;
  }
}

__global__ __launch_bounds__(kBlock) void k_read_pairs(PileDev P, const uint32_t* __restrict__ offset,
                                                       uint64_t* __restrict__ keys,
                                                       double* __restrict__ hist) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= P.ns) return;
  const uint2 run = P.up_run[P.parity][i];
  const uint32_t* __restrict__ pj = P.pair_j[P.parity] + run.x;
  const double* __restrict__ rows = P.hist[P.parity] + (size_t)run.x * kHistRow;
  uint32_t p = offset[i];
  for (uint32_t e = 0; e < run.y; ++e, ++p) {
    keys[p] = ((uint64_t)i << 32) | pj[e];
    for (int c = 0; c < kHist; ++c) hist[(size_t)p * kHist + c] = rows[(size_t)e * kHistRow + c];
  }
}

// One thread per value of a row (the last one is zero).
__global__ __launch_bounds__(kBlock) void k_history_rows(const double* __restrict__ packed,
                                                         double* __restrict__ rows, int64_t n) {
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x, p = t / kHistRow;
  const int c = (int)(t % kHistRow);
  if (p < n) rows[t] = c < kHist ? packed[p * kHist + c] : 0.0;
}

// No contacts and no counts: empty runs of every sphere, zero cell counts.
__global__ void k_clear(PileDev P, int64_t cells) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < P.ns) P.up_run[0][i] = P.up_run[1][i] = P.lo_run[i] = make_uint2(0u, 0u);
  if (i < cells) P.cell_cnt[i] = 0u;
  if (i < 16) P.runs[i] = 0ull;
}

}  // namespace

void launch_setup(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk,
                  const double* pos_in, const double* vel_in, const double* spin_in) {
  hipLaunchKernelGGL(k_setup, dim3(nblk), dim3(kBlock), 0, st, piles, wl, pos_in, vel_in, spin_in);
}

void launch_move(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk,
                 ContactParams cp, int mode, bool bin) {
  hipLaunchKernelGGL(k_move, dim3(nblk), dim3(kBlock), 0, st, const_cast<PileDev*>(piles), wl, cp,
                     mode, (int)bin);
}

void launch_grid(hipStream_t st, const PileDev* piles, const int32_t* plist, int n, int mode,
                 double dt) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_grid, dim3(n), dim3(256), 0, st, const_cast<PileDev*>(piles), plist, mode,
                     dt);
}

void launch_reduce(hipStream_t st, PileDev* piles, const WorkItem* wl, int nblk, ContactParams cp,
                   int mode, bool stage, bool finish) {
  hipLaunchKernelGGL(k_reduce, dim3(nblk), dim3(kBlock), 0, st, piles, wl, cp, mode, (int)stage,
                     (int)finish);
}

void launch_finish(hipStream_t st, PileDev* piles, int n_piles, int mode, double dt) {
  hipLaunchKernelGGL(k_finish, dim3(n_piles), dim3(64), 0, st, piles, mode, dt);
}

void launch_fill_u32(hipStream_t st, uint32_t* p, uint32_t value, int64_t n) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st,
                     p, value, n);
}
void launch_read(hipStream_t st, ReadList& list) {
  int blk = 0;
  for (int q = 0; q < list.n; ++q) {
    list.f[q].block0 = blk;
    blk += (int)((list.f[q].n + kBlock - 1) / kBlock);
  }
  if (blk > 0) hipLaunchKernelGGL(k_read, dim3(blk), dim3(kBlock), 0, st, list);
}
void launch_read_pairs(hipStream_t st, const PileDev& h, uint32_t* offset, uint64_t* keys,
                       double* hist) {
  hipLaunchKernelGGL(k_read_offsets, dim3(1), dim3(kOffsetThreads), 0, st, h.up_run[h.parity], h.ns,
                     offset);
  hipLaunchKernelGGL(k_read_pairs, dim3((h.ns + kBlock - 1) / kBlock), dim3(kBlock), 0, st, h,
                     offset, keys, hist);
}
void launch_history_rows(hipStream_t st, const double* packed, double* rows, int64_t n) {
  const int64_t t = n * kHistRow;
  hipLaunchKernelGGL(k_history_rows, dim3((unsigned)((t + kBlock - 1) / kBlock)), dim3(kBlock), 0, st,
                     packed, rows, n);
}
void launch_clear(hipStream_t st, const PileDev& h, int64_t cells) {
  const int64_t n = std::max<int64_t>(std::max<int64_t>(h.ns, cells), 16);
  hipLaunchKernelGGL(k_clear, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, h,
                     cells);
}

}  // namespace dem

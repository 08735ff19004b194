// kernels_force.hip -- soft-sphere contact forces of every sphere, with the
// spring history carried from the previous step (Sec. 2.1: spring-dashpot
// normal and tangential forces, static friction, rolling and twisting
// friction, history kept while the contact lasts; Sec. 2.2.4: forces act at
// the contact point, lever arm of Eq. 8, torque of Eq. 9).
//
// A block takes kForceSpheres spheres and deals their contacts to its threads
// one each (forces_group in step_force.h); the force and torque of a sphere
// are summed in canonical order: the lower list (j, i), j < i, then the upper
// list (i, j), each by increasing j.  Each contact is evaluated by both of its
// spheres with the same operands in the same order, so the two sums see the same
// force and no per-contact force is stored or read back; the lower sphere
// writes the contact's new spring history.  A wall is partner ns + w:
// infinite mass, no spin, moving rigidly; its reaction goes nowhere.
// Geometry is always FP64; the force arithmetic runs in T (double, or float
// for the FP32-force form).
#include "step_force.h"

namespace dem {

namespace {

constexpr int kForceSpheres = 64;

template <typename T>
__global__ __launch_bounds__(kBlock) void k_forces(PileDev* __restrict__ piles,
                                                   const WorkItem* __restrict__ wl,
                                                   ContactParams cp) {
  constexpr int kPer = kBlock / kForceSpheres;   // blocks per work item
  __shared__ ForceLds<kBlock, kForceSpheres> sh;
  const int blk = xcd_block(blockIdx.x, gridDim.x);
  const WorkItem w = wl[blk / kPer];
  PileDev& P = piles[w.pile];
  const int base = w.base + (blk % kPer) * kForceSpheres;
  if (threadIdx.x == 0) sh.start[0] = (uint32_t)P.status;   // one read for the block
  __syncthreads();
  const bool failed = sh.start[0] != 0u;
  __syncthreads();
  if (base >= P.ns || failed) return;
  const PairCtx<T> c = pair_ctx<T>(P, cp);
  bool bad = false;
  forces_group<T, kBlock, kForceSpheres>(P, c, cp, base, sh, bad);
  if (bad) atomicOr(&P.status, kStUnstable);
}

}  // namespace

void launch_forces(hipStream_t st, const PileDev* piles, const WorkItem* wl, int nblk,
                   ContactParams cp, int precision) {
  PileDev* p = const_cast<PileDev*>(piles);
  const dim3 grid(nblk * (kBlock / kForceSpheres));
  if (precision == 1)
    hipLaunchKernelGGL(k_forces<float>, grid, dim3(kBlock), 0, st, p, wl, cp);
  else
    hipLaunchKernelGGL(k_forces<double>, grid, dim3(kBlock), 0, st, p, wl, cp);
}

}  // namespace dem

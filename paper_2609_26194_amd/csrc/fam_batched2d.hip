// fam_batched2d.hip - the 2D kernels of a batch of meshes (tiles in fam_tiles2d.h):
// workgroups take the items of a work list (instance, first column, first row, rows).
#include "fam_tiles2d.h"

namespace fam {

template <int K, class P, bool PP>
__global__ void FAM_STAGE_ATTR(K, false) stage2d_batched_kernel(StageArgs A, const Inst* __restrict__ insts,
                                                                const int4* __restrict__ work, int nwork) {
  FAM_STAGE_SHARED(K, P::NC, false);
  const P phys = make_phys<P>(A.phys);
  bool bad = false;
  // one item per workgroup: the XCD-aware order (limiter on: heavy items first)
  const bool one_each = (int)gridDim.x == nwork;
#pragma unroll 1
  for (int w = blockIdx.x; w < nwork; w += gridDim.x) {
    // limiter on: items in the order of the previous launch's limiter work
    int wi;
    if constexpr (PP) wi = A.tile_perm[one_each ? heavy_first_slot(w, nwork, A.tile_perm[nwork]) : w];
    else wi = one_each ? xcd_tile(w, nwork) : w;
    wi = __builtin_amdgcn_readfirstlane(wi);   // in scalar registers, and with it the item and its instance
    const int4 it = work[wi];             // (instance, i0, j0, H)
    const Inst in = insts[it.x];
    if (in.done && __builtin_amdgcn_readfirstlane(*in.done)) continue;
    double amx = 0.0, amy = 0.0;
    if constexpr (PP) S.nwork = 0;
    // slot 0 alone: the atomics of a batch already go to as many lines as it has
    // instances, and the reduction of all slots for every item costs more (40
    // meshes of 64^2 to 512^2: 1 %; it also takes scalar registers from the rows)
    stage_tile<K, P, PP, false, false, false>(phys, A, in, it.y, it.z, it.w, S, amx, amy, bad);
    flush_wave_results<false>(amx, amy, false, in.alpha_out, A.flag);
    if constexpr (PP) {
      if (threadIdx.x == 0) A.tile_work[wi] = S.nwork;
    }
  }
  if (__any(bad) && threadIdx.x == 0) atomicOr(A.flag, 1);
}

template <int K, class P>
__global__ void FAM_OE_ATTR oe2d_batched_kernel(OEArgs A, const Inst* __restrict__ insts,
                                                             const int4* __restrict__ work, int nwork) {
  constexpr int SLOTS = P::NC == 1 ? 4 : 3;
  __shared__ Window<3 * P::NC, SLOTS> W;
  __shared__ double t1s[8];
  const P phys = make_phys<P>(A.phys);
  bool bad = false;
  const bool one_each = (int)gridDim.x == nwork;   // then the XCD-aware order
#pragma unroll 1
  for (int w = blockIdx.x; w < nwork; w += gridDim.x) {
    const int4 it = work[__builtin_amdgcn_readfirstlane(one_each ? xcd_tile(w, nwork) : w)];
    const Inst in = insts[it.x];
    if (in.done && __builtin_amdgcn_readfirstlane(*in.done)) continue;
    if (K == 6 && A.k6_table)
      oe_tile<K, P, true, false, SLOTS>(phys, A, in, it.y, it.z, it.w, W, t1s, bad);
    else
      oe_tile<K, P, false, false, SLOTS>(phys, A, in, it.y, it.z, it.w, W, t1s, bad);
  }
  if (__any(bad) && threadIdx.x == 0) atomicOr(A.flag, 1);
}

template <int K, class P>
static void launch_stage2d_b(const StageArgs& A, const Inst* insts, const int4* work, int nwork, int nblocks,
                             hipStream_t s) {
  if (A.pp) {
    hipLaunchKernelGGL((stage2d_batched_kernel<K, P, true>), dim3(nblocks), dim3(LANES), 0, s, A, insts, work,
                       nwork);
    // (renewed after stage 0 only, a step of 40 meshes takes 2 % longer, though a renewal is 6 us)
    if (!starts_at_once(nblocks, nwork, stage_waves(K, P::NC, false)))
      launch_tile_order(A.tile_work, const_cast<int*>(A.tile_perm), nwork, s);
  } else
    hipLaunchKernelGGL((stage2d_batched_kernel<K, P, false>), dim3(nblocks), dim3(LANES), 0, s, A, insts, work,
                       nwork);
}
template <int K, class P>
static void launch_oe2d_b(const OEArgs& A, const Inst* insts, const int4* work, int nwork, int nblocks,
                          hipStream_t s) {
  hipLaunchKernelGGL((oe2d_batched_kernel<K, P>), dim3(nblocks), dim3(LANES), 0, s, A, insts, work, nwork);
}

void launch_stage2d_batched(int k, int sys, const StageArgs& A, const Inst* insts, const int4* work, int nwork,
                            int nblocks, hipStream_t s) {
  FAM_DISPATCH_P(sys, FAM_DISPATCH_K(k, (launch_stage2d_b<KK, PP>(A, insts, work, nwork, nblocks, s))));
}
void launch_oe2d_batched(int k, int sys, const OEArgs& A, const Inst* insts, const int4* work, int nwork,
                         int nblocks, hipStream_t s) {
  FAM_DISPATCH_P(sys, FAM_DISPATCH_K(k, (launch_oe2d_b<KK, PP>(A, insts, work, nwork, nblocks, s))));
}

}  // namespace fam

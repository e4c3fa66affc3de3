// The fused z pass over the lengths of a family in one launch (included by the
// zfused_*_f*.hip units, one per form and precision): 2D batches of patches of
// several sides.  The same work per item as fft_z_kernel, which runs the length
// alone; what it saves is the launches: us per step, launches per length and per
// family: 64 patches with sources FP32 300 -> 272, 128 patches with sources FP64
// 576 -> 544, 200 patches with sources FP32 627 -> 608, 256 patches vacuum 589 ->
// 591 (long launches, nothing to save).  384 points in the family or not: 272 and
// 278, 544 and 554, 608 and 615.
#pragma once

#include "zfused_kernel.hpp"

namespace psatd {
namespace zfused {

namespace {

// LDS (double2) and waves per SIMD that serve every length of the family.
template <typename ST, int SRC, int L>
constexpr int z_lds() {
  using LN = ZLine<ST, 2, SRC, L>;
  static_assert(LN::NT == kFamilyBlock, "one workgroup size in a family");
  return LN::kLds;
}
template <typename ST, int SRC, int FAM>
constexpr int family_lds() {
  int m = 0;
#define PSATD_ZS_LDS(LEN) m = z_lds<ST, SRC, LEN>() > m ? z_lds<ST, SRC, LEN>() : m;
  if (FAM == kPow2) {
    PSATD_Z_POW2(PSATD_ZS_LDS)
  } else {
    PSATD_Z_3POW2(PSATD_ZS_LDS)
  }
  return m;
}
template <typename ST, int SRC, int FAM>
constexpr int family_waves() {
  int n = 2;
#define PSATD_ZS_WAVES(LEN) \
  n = Budget<2, SRC, LEN, sizeof(ST)>::waves < n ? Budget<2, SRC, LEN, sizeof(ST)>::waves : n;
  if (FAM == kPow2) {
    PSATD_Z_POW2(PSATD_ZS_WAVES)
  } else {
    PSATD_Z_3POW2(PSATD_ZS_WAVES)
  }
  return n;
}

template <typename ST, int SRC, int L>
__device__ __forceinline__ void z_item(int set, const PatchDev* P, const WorkItem& wi, ST* ws,
                                       const Physics& ph, double2* lds) {
  ZLine<ST, 2, SRC, L> ln;
  ln.load_twiddles(P->fz.tw, lds);
  if (set == 0) z_set<ST, 2, SRC, L, 0>(ln, P, wi, ws, ph, lds);
  else z_set<ST, 2, SRC, L, 1>(ln, P, wi, ws, ph, lds);
}

template <typename ST, int SRC, int FAM>
__global__ void __launch_bounds__(kFamilyBlock)
    __attribute__((amdgpu_waves_per_eu(family_waves<ST, SRC, FAM>())))
fft_zs_kernel(const PatchDev* __restrict__ patches, const WorkItem* __restrict__ items, int nitems,
              ST* __restrict__ ws, Physics ph) {
  __shared__ double2 lds[family_lds<ST, SRC, FAM>()];
  for (int w = blockIdx.x; w < 2 * nitems; w += gridDim.x) {
    const WorkItem wi = items[w / 2];
    const PatchDev* P = patches + wi.patch;
#define PSATD_ZS_ITEM(LEN) \
  case LEN: z_item<ST, SRC, LEN>(w & 1, P, wi, ws, ph, lds); break;
    if constexpr (FAM == kPow2) {
      switch (P->nz) {
        PSATD_Z_POW2(PSATD_ZS_ITEM)
        default: break;
      }
    } else {
      switch (P->nz) {
        PSATD_Z_3POW2(PSATD_ZS_ITEM)
        default: break;
      }
    }
    __syncthreads();  // the next item may divide the rows among the waves differently
  }
}

template <typename ST, int SRC>
hipError_t launch_zs(int fam, int grid, hipStream_t stream, const PatchDev* p, const WorkItem* it,
                     int n, void* ws, Physics ph) {
  if (fam == kPow2)
    hipLaunchKernelGGL((fft_zs_kernel<ST, SRC, kPow2>), dim3(grid), dim3(kFamilyBlock), 0, stream, p,
                       it, n, static_cast<ST*>(ws), ph);
  else if (fam == k3Pow2)
    hipLaunchKernelGGL((fft_zs_kernel<ST, SRC, k3Pow2>), dim3(grid), dim3(kFamilyBlock), 0, stream, p,
                       it, n, static_cast<ST*>(ws), ph);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

}  // namespace zfused
}  // namespace psatd

#define PSATD_ZS_DEFINE(name, ST, SRC)                                                            \
  namespace psatd {                                                                               \
  namespace zfused {                                                                              \
  hipError_t launch_family_##name(int fam, int grid, hipStream_t stream, const PatchDev* patches, \
                                  const WorkItem* items, int nitems, void* ws, Physics ph) {      \
    return launch_zs<ST, SRC>(fam, grid, stream, patches, items, nitems, ws, ph);                 \
  }                                                                                               \
  int family_lds_##name(int fam) {                                                                \
    return 16 * (fam == kPow2 ? family_lds<ST, SRC, kPow2>() : family_lds<ST, SRC, k3Pow2>());    \
  }                                                                                               \
  }                                                                                               \
  }

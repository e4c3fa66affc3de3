// Fused z passes with compile-time lengths (zfused_*.hip): tiles and launchers.
#pragma once

#include <hip/hip_runtime.h>

#include "bfft.hpp"
#include "groups.hpp"
#include "internal.hpp"
#include "kernels.hpp"

namespace psatd {
namespace zfused {

// Lengths compiled, by group (one translation unit each): 2D forms take all
// of them (FP64 up to 2048), 3D forms those up to 512.
#define PSATD_Z_A(X) X(32) X(36) X(48) X(54) X(64) X(72) X(96) X(108)
#define PSATD_Z_B(X) X(128) X(144) X(162) X(192) X(216)
#define PSATD_Z_C(X) X(256) X(288) X(324) X(384) X(432) X(512)
#define PSATD_Z_D(X) X(576) X(648) X(768) X(864) X(1024) X(1152)
#define PSATD_Z_E(X) X(1296) X(1536) X(1728) X(2048)
#define PSATD_Z_F(X) X(2304) X(3072) X(4096)

// Inputs of a set: the larger of the two polarization sets in 2D.
constexpr int inputs(int dim, int src) {
  if (dim == 2) return !src_has_j(src) ? 3 : (src == kRho ? 7 : 5);
  return !src_has_j(src) ? 6 : (src == kRho ? 11 : 9);
}

// A work item is up to T lines of one patch, transformed by T S threads (both
// sets of a 2D item are work of their own).
template <int L>
struct Tile {
  using SC = bfft::Sched<L, bfft::kFusedZ>;
  static constexpr int round64(int n) { return (n + 63) / 64 * 64; }
  static constexpr int lines() {
    int best = 1;
    for (int t = 1; t * SC::S <= 256; ++t)
      if (t * SC::S * round64(best * SC::S) >= best * SC::S * round64(t * SC::S)) best = t;
    return best;
  }
  static constexpr int T = lines();
  static constexpr int NT = round64(T * SC::S);
};

// What each kernel holds: P modes of every input of its set in storage
// precision.  A wave alone on its SIMD issues an FP64 instruction every 6
// cycles, two together one every 4.8 (measured), so two waves share a SIMD
// where 256 registers each are enough -- with up to HELD_LDS inputs in LDS
// slots of their thread, and without the next input's loads in flight where
// those do not fit.  512^3 rho form (9 inputs in registers, 2 in LDS, no
// prefetch, a few spills): 2.9 ms; one wave with 394 registers: 3.63 ms.  FP64
// takes the second wave only with room to spare: the 2D J form at 512 points
// ran 51.8 us with it (spills) and 32.8 without (2048 x 512).  At 8 points per
// thread that is every FP32 form and the 2D vacuum form in FP64; at 12 points the
// 2D FP32 forms but rho.  The others run one wave per SIMD.
template <int DIM, int SRC, int L, int ELEM>
struct Budget {
  using SC = bfft::Sched<L, bfft::kFusedZ>;
  static constexpr int NIN = inputs(DIM, SRC);
  static constexpr int kTwo = ELEM == 4 ? 264 : 230;  // estimates up to which two waves pay
  // double2 elements of a workgroup's LDS copy of the twiddles
  static constexpr int kCopy = ELEM == 8 ? bfft::shared_offset<SC>(SC::N) : 0;
  // held inputs, the transform, the rest
  static constexpr int regs(int held) { return held * SC::P * ELEM / 2 + 7 * SC::P + 60; }
  static constexpr int lds_wave(int in_lds) {
    return (SC::kRow * 16 * 64 + SC::S - 1) / SC::S + in_lds * SC::P * 64 * 2 * ELEM +
           kCopy * 16 * 64 / Tile<L>::NT;
  }
  // fewest inputs in LDS that leave the others (the outputs among them) within
  // the limit, -1: none
  static constexpr int held_lds(int limit, int waves_per_cu) {
    for (int n = 0; n <= 2 && NIN - n >= (DIM == 2 ? 3 : 6); ++n)
      if (regs(NIN - n) <= limit && lds_wave(n) * waves_per_cu <= 160 * 1024) return n;
    return -1;
  }
  static constexpr bool two = held_lds(kTwo, 8) >= 0;
  static constexpr int one = held_lds(480, 4);
  static constexpr int HELD_LDS = two ? held_lds(kTwo, 8) : (one >= 0 ? one : 0);
  static constexpr bool kPrefetch = !two || regs(NIN - HELD_LDS + 1) <= kTwo;
  static constexpr int waves = two ? 2 : 1;
  // FP64 storage: the twiddles in registers where radices are powers of two and
  // their three per stage fit (2D rho form, 1024 points: 93 us, 98 from LDS), else
  // in LDS (2D J form of 1728 x 1152, 12 points per thread: 145 us, 159 folded and
  // from registers)
  static constexpr bool kHeld = SC::P == 8 && regs(NIN - HELD_LDS) + 36 <= (two ? kTwo : 480);
  static constexpr bfft::Twiddles kTw =
      ELEM == 4 ? bfft::kSquares : (kHeld ? bfft::kTable : bfft::kShared);
  static constexpr int kTwiddles = kTw == bfft::kShared ? kCopy : 0;
};

bool supported(int precision, int ndim, int src, int nz);
int lines_per_item(int nz);  // T
int block(int nz);
int points_per_thread(int nz);
int lds_bytes(int precision, int ndim, int src, int nz);
// Workgroups that give every set of every item its own.
inline int workgroups(int ndim, int nitems) { return ndim == 2 ? 2 * nitems : nitems; }

// One launch covers the items of the patches with this nz.
hipError_t launch(int precision, int ndim, int src, int nz, int grid, hipStream_t stream,
                  const PatchDev* patches, const WorkItem* items, int nitems, void* ws, Physics ph);

// Families of lengths that a 2D plan runs in one launch when it has several of
// a family (fft_zs_kernel): the points per thread, the threads per workgroup
// and so the registers are the same within a family, and a launch per length
// costs about 6 us to fork and join in the step graph.  (One launch for both
// families, and for families of different points per thread in the line
// passes, gave the short lengths the registers of the long ones: 64 x 64
// patches, x pass 69 -> 138 us.)
#define PSATD_Z_POW2(X) X(32) X(64) X(128) X(256) X(512)
#define PSATD_Z_3POW2(X) X(48) X(96) X(192) X(384)
enum Family { kNoFamily = 0, kPow2 = 1, k3Pow2 = 2 };
constexpr int kFamilyBlock = 256;
// The family whose kernel is compiled for this form and takes the length.
int family(int precision, int ndim, int src, int nz);
int family_lds_bytes(int precision, int src, int fam);
// One launch covers the items of the patches with lengths of the family.
hipError_t launch_family(int precision, int src, int fam, int grid, hipStream_t stream,
                         const PatchDev* patches, const WorkItem* items, int nitems, void* ws,
                         Physics ph);
// (one translation unit per form and precision)
#define PSATD_ZS_FORM(name)                                                                        \
  hipError_t launch_family_##name(int fam, int grid, hipStream_t stream, const PatchDev* patches,  \
                                  const WorkItem* items, int nitems, void* ws, Physics ph);        \
  int family_lds_##name(int fam)
PSATD_ZS_FORM(vacuum_f32);
PSATD_ZS_FORM(rho_f32);
PSATD_ZS_FORM(j_f32);
PSATD_ZS_FORM(vacuum_f64);
PSATD_ZS_FORM(rho_f64);
PSATD_ZS_FORM(j_f64);

#define PSATD_Z_GROUP(name)                                                                        \
  hipError_t launch_##name(int precision, int ndim, int src, int nz, int grid, hipStream_t stream, \
                           const PatchDev* patches, const WorkItem* items, int nitems, void* ws,   \
                           Physics ph)
PSATD_Z_GROUP(a);
PSATD_Z_GROUP(b);
PSATD_Z_GROUP(c);
PSATD_Z_GROUP(d);
PSATD_Z_GROUP(e);
PSATD_Z_GROUP(f);

// Which (precision, dimension, form) each length is compiled for.
constexpr bool compiled(int elem, int dim, int src, int L) {
  if (src_is_pstd(src)) return dim == 2 && elem == 4;
  // (3D FP64 rho form at 12 points per thread: 11 inputs do not fit 512 registers)
  if (dim == 3) return L <= 512 && !(elem == 8 && inputs(3, src) * bfft::fused_radices(L).P > 108);
  return elem == 4 || L <= 2048;
}

}  // namespace zfused
}  // namespace psatd

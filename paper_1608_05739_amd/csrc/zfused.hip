// Fused z passes with compile-time lengths: what is compiled, and the dispatch
// to the translation units that hold the kernels.
#include "zfused.hpp"

namespace psatd {
namespace zfused {

namespace {

struct Shape {
  int lines, block, row_bytes;
};
Shape shape(int nz) {
  switch (nz) {
#define PSATD_Z_SHAPE(LEN) \
  case LEN: return Shape{Tile<LEN>::T, Tile<LEN>::NT, Tile<LEN>::T * bfft::Sched<LEN, bfft::kFusedZ>::kRow * 16};
    PSATD_Z_A(PSATD_Z_SHAPE)
    PSATD_Z_B(PSATD_Z_SHAPE)
    PSATD_Z_C(PSATD_Z_SHAPE)
    PSATD_Z_D(PSATD_Z_SHAPE)
    PSATD_Z_E(PSATD_Z_SHAPE)
    PSATD_Z_F(PSATD_Z_SHAPE)
    default: return Shape{0, 0, 0};
  }
}

// LDS of the held inputs and of the twiddles, per form.
template <int DIM, int SRC, int L, int ELEM>
int form_bytes() {
  using BU = Budget<DIM, SRC, L, ELEM>;
  return BU::HELD_LDS * bfft::Sched<L, bfft::kFusedZ>::P * Tile<L>::NT * 2 * ELEM + BU::kTwiddles * 16;
}
template <int DIM, int L, int ELEM>
int slots(int src) {
  switch (src) {
    case kVacuum: return form_bytes<DIM, kVacuum, L, ELEM>();
    case kRho: return form_bytes<DIM, kRho, L, ELEM>();
    case kJForm: return form_bytes<DIM, kJForm, L, ELEM>();
    case kPstdVacuum: return form_bytes<DIM, kPstdVacuum, L, ELEM>();
    default: return form_bytes<DIM, kPstdJ, L, ELEM>();
  }
}
template <int L>
int slots_of(int precision, int ndim, int src) {
  if (ndim == 2) return precision == 0 ? slots<2, L, 4>(src) : slots<2, L, 8>(src);
  return precision == 0 ? slots<3, L, 4>(src) : slots<3, L, 8>(src);
}

}  // namespace

bool supported(int precision, int ndim, int src, int nz) {
  return shape(nz).lines > 0 && compiled(precision == 0 ? 4 : 8, ndim, src, nz);
}
int lines_per_item(int nz) { return shape(nz).lines; }
int block(int nz) { return shape(nz).block; }
int points_per_thread(int nz) { return bfft::fused_radices(nz).P; }
int lds_bytes(int precision, int ndim, int src, int nz) {
  switch (nz) {
#define PSATD_Z_SLOTS(LEN) \
  case LEN: return shape(nz).row_bytes + slots_of<LEN>(precision, ndim, src);
    PSATD_Z_A(PSATD_Z_SLOTS)
    PSATD_Z_B(PSATD_Z_SLOTS)
    PSATD_Z_C(PSATD_Z_SLOTS)
    PSATD_Z_D(PSATD_Z_SLOTS)
    PSATD_Z_E(PSATD_Z_SLOTS)
    PSATD_Z_F(PSATD_Z_SLOTS)
    default: return 0;
  }
}

int family(int precision, int ndim, int src, int nz) {
  if (ndim != 2 || src_is_pstd(src) || !supported(precision, ndim, src, nz)) return kNoFamily;
  switch (nz) {
#define PSATD_Z_FAMILY_LABEL(LEN) case LEN:
    PSATD_Z_POW2(PSATD_Z_FAMILY_LABEL)
    return kPow2;
    PSATD_Z_3POW2(PSATD_Z_FAMILY_LABEL)
    return k3Pow2;
    default: return kNoFamily;
  }
}
int family_lds_bytes(int precision, int src, int fam) {
  switch (src) {
    case kVacuum: return precision == 0 ? family_lds_vacuum_f32(fam) : family_lds_vacuum_f64(fam);
    case kRho: return precision == 0 ? family_lds_rho_f32(fam) : family_lds_rho_f64(fam);
    default: return precision == 0 ? family_lds_j_f32(fam) : family_lds_j_f64(fam);
  }
}
hipError_t launch_family(int precision, int src, int fam, int grid, hipStream_t stream,
                         const PatchDev* patches, const WorkItem* items, int nitems, void* ws,
                         Physics ph) {
  switch (src) {
    case kVacuum:
      return precision == 0
                 ? launch_family_vacuum_f32(fam, grid, stream, patches, items, nitems, ws, ph)
                 : launch_family_vacuum_f64(fam, grid, stream, patches, items, nitems, ws, ph);
    case kRho:
      return precision == 0 ? launch_family_rho_f32(fam, grid, stream, patches, items, nitems, ws, ph)
                            : launch_family_rho_f64(fam, grid, stream, patches, items, nitems, ws, ph);
    case kJForm:
      return precision == 0 ? launch_family_j_f32(fam, grid, stream, patches, items, nitems, ws, ph)
                            : launch_family_j_f64(fam, grid, stream, patches, items, nitems, ws, ph);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch(int precision, int ndim, int src, int nz, int grid, hipStream_t stream,
                  const PatchDev* patches, const WorkItem* items, int nitems, void* ws, Physics ph) {
  switch (nz) {
#define PSATD_Z_LABEL(LEN) case LEN:
    PSATD_Z_A(PSATD_Z_LABEL)
    return launch_a(precision, ndim, src, nz, grid, stream, patches, items, nitems, ws, ph);
    PSATD_Z_B(PSATD_Z_LABEL)
    return launch_b(precision, ndim, src, nz, grid, stream, patches, items, nitems, ws, ph);
    PSATD_Z_C(PSATD_Z_LABEL)
    return launch_c(precision, ndim, src, nz, grid, stream, patches, items, nitems, ws, ph);
    PSATD_Z_D(PSATD_Z_LABEL)
    return launch_d(precision, ndim, src, nz, grid, stream, patches, items, nitems, ws, ph);
    PSATD_Z_E(PSATD_Z_LABEL)
    return launch_e(precision, ndim, src, nz, grid, stream, patches, items, nitems, ws, ph);
    PSATD_Z_F(PSATD_Z_LABEL)
    return launch_f(precision, ndim, src, nz, grid, stream, patches, items, nitems, ws, ph);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace zfused
}  // namespace psatd

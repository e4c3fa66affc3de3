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

// LDS of the held inputs, per form.
template <int DIM, int L, int ELEM>
int slots(int src) {
  int n = 0;
  switch (src) {
    case kVacuum: n = Budget<DIM, kVacuum, L, ELEM>::HELD_LDS; break;
    case kRho: n = Budget<DIM, kRho, L, ELEM>::HELD_LDS; break;
    case kJForm: n = Budget<DIM, kJForm, L, ELEM>::HELD_LDS; break;
    case kPstdVacuum: n = Budget<DIM, kPstdVacuum, L, ELEM>::HELD_LDS; break;
    default: n = Budget<DIM, kPstdJ, L, ELEM>::HELD_LDS; break;
  }
  return n * bfft::Sched<L, bfft::kFusedZ>::P * Tile<L>::NT * 2 * ELEM;
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

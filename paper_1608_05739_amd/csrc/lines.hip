// Line passes with compile-time lengths: what is compiled, and the dispatch to
// the translation units that hold the kernels.
#include "lines.hpp"

namespace psatd {
namespace lines {

namespace {

enum Group { kNone, kSmall, kMid, kLarge, kLong };

Group group_of(int L) {
  switch (L) {
#define PSATD_IN_SMALL(LEN) case LEN: return kSmall;
#define PSATD_IN_MID(LEN) case LEN: return kMid;
#define PSATD_IN_LARGE(LEN) case LEN: return kLarge;
#define PSATD_IN_LONG(LEN) case LEN: return kLong;
    PSATD_LINE_SMALL(PSATD_IN_SMALL)
    PSATD_LINE_MID(PSATD_IN_MID)
    PSATD_LINE_LARGE(PSATD_IN_LARGE)
    PSATD_LINE_LONG(PSATD_IN_LONG)
    default: return kNone;
  }
}

struct Shape {
  int rows, block, lds;
};
template <int L, int ELEM>
Shape shape_of(bool transposing) {
  if (transposing) {
    using T = Tile<L, ELEM, true>;
    return Shape{T::T, T::NT, T::kLds * 16};
  }
  using T = Tile<L, ELEM, false>;
  return Shape{T::T, T::NT, T::kLds * 16};
}
Shape shape(int kind, int precision, int L) {
  const bool tr = kind != kZFwd && kind != kZInv;
  switch (L) {
#define PSATD_SHAPE(LEN) \
  case LEN: return precision == 0 ? shape_of<LEN, 4>(tr) : shape_of<LEN, 8>(tr);
    PSATD_LINE_SMALL(PSATD_SHAPE)
    PSATD_LINE_MID(PSATD_SHAPE)
    PSATD_LINE_LARGE(PSATD_SHAPE)
    PSATD_LINE_LONG(PSATD_SHAPE)
    default: return Shape{0, 0, 0};
  }
}

}  // namespace

bool supported(int, int L) { return group_of(L) != kNone; }
int rows(int kind, int precision, int L) { return shape(kind, precision, L).rows; }
int block(int kind, int precision, int L) { return shape(kind, precision, L).block; }
int lds_bytes(int kind, int precision, int L) { return shape(kind, precision, L).lds; }

hipError_t launch(int kind, int precision, int L, int grid, hipStream_t stream,
                  const PatchDev* patches, const WorkItem* items, int nitems,
                  const FieldPtrs& fields, void* ws) {
  switch (group_of(L)) {
    case kSmall: return launch_small(kind, precision, L, grid, stream, patches, items, nitems, fields, ws);
    case kMid: return launch_mid(kind, precision, L, grid, stream, patches, items, nitems, fields, ws);
    case kLarge: return launch_large(kind, precision, L, grid, stream, patches, items, nitems, fields, ws);
    case kLong: return launch_long(kind, precision, L, grid, stream, patches, items, nitems, fields, ws);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lines
}  // namespace psatd

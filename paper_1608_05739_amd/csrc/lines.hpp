// Line passes with compile-time lengths (lines_*.hip): tiles and launchers.
#pragma once

#include <hip/hip_runtime.h>

#include "bfft.hpp"
#include "internal.hpp"
#include "kernels.hpp"

namespace psatd {
namespace lines {

// Lengths (complex points) the line passes are compiled for, by pass: the x
// passes take L = nx / 2 (even, so that the r2c pairs split evenly), the y
// and z passes the side itself.
#define PSATD_LINE_SMALL(X) X(24) X(32) X(36) X(48) X(54) X(64) X(72) X(96) X(108) X(128)
#define PSATD_LINE_MID(X) X(144) X(162) X(192) X(216) X(256) X(288) X(324) X(384)
#define PSATD_LINE_LARGE(X) X(432) X(486) X(512) X(576) X(648) X(768) X(864) X(1024)
#define PSATD_LINE_LONG(X) X(1152) X(1296) X(1536) X(1728) X(2048)

// A tile is T rows (lines) of one component, transformed by T S threads.  The
// x and y passes transpose: on the strided side of a tile T consecutive
// elements are one run of 8 T (FP32) or 16 T bytes (FP64).  T is 16 or 8 (128
// bytes) as long as two tiles fit a CU's LDS, and is halved until they do:
// neighbouring tiles run on one XCD and complete the lines in its L2, and a
// second tile on the CU is worth more than longer runs.  FP32 x passes of
// grids of 4 M cells with sources, forward / inverse TB/s, two tiles of short runs
// against one of runs twice or four times as long: 648 points (32 bytes) 3.9 / 3.5
// and 2.7 / 2.6; 1152 points (32 bytes) 3.8 / 3.5 and 3.1 / 2.6; 1296 points (16
// bytes) 3.4 / 2.7 and 2.6 / 2.5; 2048 points (16 bytes) 3.4 / 3.5 and 3.3 / 3.0.
// FP64 keeps 64 bytes where one tile fits (2048 points forward: 4.0 TB/s, 2.8 with
// two tiles of 32-byte runs).
template <int L, int ELEM, bool TRANSPOSING>
struct Tile {
  using SC = bfft::Sched<L, ELEM == 8 ? bfft::kLine64 : bfft::kLine32>;
  static constexpr bfft::Twiddles kTw = ELEM == 8 ? bfft::kTable : bfft::kSquares;
  static constexpr int rows() {
    int t = ELEM == 4 ? 16 : 8;
    while (t > 1 && (t * SC::S > 640 || t * SC::kRow * 16 > 80 * 1024)) t /= 2;
    if (TRANSPOSING && ELEM == 8)
      while (t < 4 && 2 * t * SC::S <= 1024 && 2 * t * SC::kRow * 16 <= 160 * 1024) t *= 2;
    while (t * SC::S < 128 && 2 * t * SC::kRow * 16 <= 40 * 1024) t *= 2;  // short lines: two waves
    return t;
  }
  static constexpr int T = rows();
  static constexpr int NT = (T * SC::S + 63) / 64 * 64;  // threads per workgroup
  static constexpr int kLds = T * SC::kRow;              // double2 elements
};

// Is L compiled for the pass kind?  Rows per tile and threads per workgroup.
bool supported(int kind, int L);
int rows(int kind, int precision, int L);
int block(int kind, int precision, int L);
int lds_bytes(int kind, int precision, int L);

// One launch covers the work items of one length: tiles of up to rows()
// consecutive lines inside one run of the spectra layout.
hipError_t launch(int kind, int precision, int L, int grid, hipStream_t stream,
                  const PatchDev* patches, const WorkItem* items, int nitems,
                  const FieldPtrs& fields, void* ws);

// One translation unit per group of lengths (see the lists above).
#define PSATD_LINE_GROUP(name)                                                                     \
  hipError_t launch_##name(int kind, int precision, int L, int grid, hipStream_t stream,           \
                           const PatchDev* patches, const WorkItem* items, int nitems,             \
                           const FieldPtrs& fields, void* ws)
PSATD_LINE_GROUP(small);
PSATD_LINE_GROUP(mid);
PSATD_LINE_GROUP(large);
PSATD_LINE_GROUP(long);

}  // namespace lines
}  // namespace psatd

// The line-pass kernel with compile-time length (included by lines_*.hip).
//
// A workgroup transforms a tile of T rows.  Threads have two mappings:
//   A: S consecutive threads per row -- the contiguous side (rows of a field,
//      lines along y) is loaded and stored along the row;
//   B: T consecutive threads per point index -- the strided side is loaded and
//      stored as runs of T consecutive elements.
// The transposition between them is folded into an exchange of the transform
// (its last one forward, its first one inverse): the rows are written to LDS
// in one mapping and read in the other, so that no staging of the results and
// no pass over LDS of its own is needed.  Layouts (rows r, columns kx):
//   x passes, 2D: spectra [kx][z], row = z; 3D: [z][kx][y], row = z ny + y;
//   y passes: [z][kx][y] <-> [kx][y][z], line = kx nz + z;  z passes: in place.
// Forward x: rows packed as complex c[j] = x[2j] + i x[2j+1] (L = nx / 2),
// transformed, then split into pairs
//   X[k] = e + W^k o,  X[L-k] = conj(e - W^k o),
//   e = (Z[k] + conj Z[L-k]) / 2,  o = -i (Z[k] - conj Z[L-k]) / 2,
// W = exp(-2 pi i / nx), the Nyquist value packed into column 0.  Thread s
// computes the pairs k = s + S m, m < P/2: it needs only the upper half of the
// points of thread S - s, so half of the points cross LDS.  The inverse x pass
// is the mirror image (no 1/N: the update carries it).
//
// Bound: HBM.  Measured against kernels that kept each row in one wave at 8
// points per thread and staged every tile through LDS (512^3 with sources,
// FP32; a large device-to-device copy reaches 4.8 TB/s): x forward 2.98 ->
// 2.35 ms (3.96 -> 5.02 TB/s of rows read and spectra written), x inverse
// 1.57 -> 1.31, y forward 2.48 -> 2.44, y inverse 1.39 -> 1.31 ms.  The old x
// kernels spent 66% of their cycles in LDS and issued 614 VALU instructions
// per 8 points of a wave; 256 points at 16 per thread issue about 400.
// Against the generic kernels: 4096^2 in four 2304^2 boxes 5.56 -> 4.41 ms per
// step, 216 x 96 x 144 vacuum 0.475 -> 0.403 ms.
#pragma once

#include "lines.hpp"

namespace psatd {
namespace lines {

namespace {

template <typename ST>
struct Store;
template <>
struct Store<float> {
  using V = float2;
};
template <>
struct Store<double> {
  using V = double2;
};
__device__ __forceinline__ double2 up(float2 v) { return bfft::c2(v.x, v.y); }
__device__ __forceinline__ double2 up(double2 v) { return v; }
template <typename V>
__device__ __forceinline__ V down(double2 v);
template <>
__device__ __forceinline__ float2 down<float2>(double2 v) {
  return make_float2(static_cast<float>(v.x), static_cast<float>(v.y));
}
template <>
__device__ __forceinline__ double2 down<double2>(double2 v) {
  return v;
}

// Element at a byte offset of a workgroup-uniform base.
template <typename V>
__device__ __forceinline__ V& at(V* base, unsigned byte) {
  return *reinterpret_cast<V*>(reinterpret_cast<char*>(base) + byte);
}
template <typename V>
__device__ __forceinline__ const V& at(const V* base, unsigned byte) {
  return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + byte);
}

// A row of a patch of a decomposition in the global grid (GlobalMap): first
// pair of its row there, and the position of local pair 0 in it.
struct MappedRow {
  long long row;
  int x0, half;
  bool inside;  // an interior row
  __device__ __forceinline__ MappedRow(const PatchDev* P, int r) {
    const GlobalMap& m = P->map;
    int lz, ly;
    udivmod(r, P->ny, lz, ly);
    half = m.gnx / 2;
    row = (static_cast<long long>((m.oz + lz) % m.gnz) * m.gny + (m.oy + ly) % m.gny) * half;
    x0 = m.ox / 2;
    inside = lz >= m.iz0 && lz < m.iz1 && ly >= m.iy0 && ly < m.iy1;
  }
  __device__ __forceinline__ long long pair(int j) const {
    int x = x0 + j;
    while (x >= half) x -= half;
    return row + x;
  }
};

// w exp(-i pi M / P) for M < P / 2, P in {6, 8, 12, 18, 24}
template <int P, int M>
__device__ __forceinline__ double2 half_turn(double2 w) {
  if constexpr (M == 0) {
    return w;
  } else {
    constexpr double c = bfft::cos_72(72 / P * M), s = -bfft::sin_72(72 / P * M);
    static_assert(72 % P == 0 && c <= 1.0, "constant twiddle");
    return bfft::c2(fma(w.x, c, -w.y * s), fma(w.x, s, w.y * c));
  }
}
// (P = 16: multiples of 11.25 degrees, outside the tables)
template <int M>
__device__ __forceinline__ double2 half_turn16(double2 w) {
  constexpr double t[9] = {1.0, 0.98078528040323044913, 0.92387953251128675613,
                           0.83146961230254523708, 0.70710678118654752440, 0.55557023301960222474,
                           0.38268343236508977173, 0.19509032201612826785, 0.0};
  if constexpr (M == 0) return w;
  else return bfft::c2(fma(w.x, t[M], w.y * t[8 - M]), fma(w.y, t[M], -w.x * t[8 - M]));
}
template <int P, int M>
__device__ __forceinline__ double2 post_step(double2 w) {
  if constexpr (P == 16) return half_turn16<M>(w);
  else return half_turn<P, M>(w);
}

// The post-twiddles W^(s + S m) (FWD: -i W^(s + S m) / 2), m < P / 2, of a thread:
// COUNT = 1 keeps that of m = 0 and multiplies it by constants, which rounds once
// more; COUNT = P / 2 holds the table's.
template <int P, int S, int COUNT, bool FWD>
struct Post {
  double2 w[COUNT];
  __device__ __forceinline__ void load(const double2* post, int s) {
#pragma unroll
    for (int m = 0; m < COUNT; ++m) {
      const double2 v = gload(post, s + S * m);
      w[m] = FWD ? bfft::c2(0.5 * v.y, -0.5 * v.x) : v;
    }
  }
  template <int M>
  __device__ __forceinline__ double2 get() const {
    if constexpr (COUNT == 1) return post_step<P, M>(w[0]);
    else return w[M];
  }
};

template <typename ST, int KIND, int L>
struct Line {
  using SC = bfft::Sched<L, sizeof(ST) == 8 ? bfft::kLine64 : bfft::kLine32>;
  using V = typename Store<ST>::V;
  static constexpr bool kX = KIND == kXFwd || KIND == kXInv;
  static constexpr bool kY = KIND == kYFwd || KIND == kYInv;
  static constexpr bool kZ = !kX && !kY;
  static constexpr bool kFwd = KIND == kXFwd || KIND == kYFwd || KIND == kZFwd;
  using TL = Tile<L, sizeof(ST), !kZ>;
  static constexpr int T = TL::T, NT = TL::NT, P = SC::P, S = SC::S, N = SC::N;
  static constexpr int kRow = SC::kRow;
  static constexpr int kHalf = (L / 2) | 1;  // row of the r2c half exchange
  static constexpr bool kFull = NT == T * S;
  static constexpr bfft::Twiddles kTw = TL::kTw;
  static_assert(SC::valid() && SC::separable() && (N >= 2 || kZ), "schedule");
  // FP64 rows of at most 12 points per thread hold the post-twiddles; at 16 and
  // more (which would take 32 registers and more) the transform is exact enough
  // (r2c of 64 values, 1e-16: 1.81 with constants, 1.73 held, 1.77 the generic
  // kernel; of 2048 values 2.5 with constants, 3.4 the generic kernel)
  using PT = Post<P, S, (kX && sizeof(ST) == 8 && P <= 12) ? P / 2 : 1, kFwd>;

  // waves per SIMD that the registers are limited to: at 18 and 24 points per
  // thread the inverse x pass would take 258 registers and run alone on its
  // SIMD (288 points FP32: 2.75 TB/s; 4.4 forward at 232 registers)
  static constexpr int kWaves = P >= 18 ? 2 : (NT + 255) / 256;

  // thread positions: (gA, sA) in mapping A, (gB, sB) in mapping B
  int gA, sA, gB, sB;
  bool live;

  __device__ __forceinline__ Line() {
    const int tid = threadIdx.x;
    live = kFull || tid < T * S;
    const int t = live ? tid : 0;
    gA = t / S;
    sA = t % S;
    gB = t % T;
    sB = t / T;
  }

  // Twiddle bases: the stages before the transposition run in one mapping,
  // the others in the other.
  template <int I>
  static constexpr bool in_b() {
    return !kZ && (kFwd ? I == N - 1 : I == 0);
  }
  bfft::Base<SC, 1, kTw> w1;
  bfft::Base<SC, (N > 2 ? 2 : 1), kTw> w2;
  bfft::Base<SC, (N > 3 ? 3 : 1), kTw> w3;
  __device__ __forceinline__ void load_twiddles(const double2* tw) {
    w1.load(tw, in_b<1>() ? sB : sA);
    if constexpr (N > 2) w2.load(tw, in_b<2>() ? sB : sA);
    if constexpr (N > 3) w3.load(tw, in_b<3>() ? sB : sA);
  }
  template <int I>
  __device__ __forceinline__ void stage(double2 (&v)[P]) const {
    constexpr int SIGN = kFwd ? -1 : 1;
    if constexpr (I == 0) {
      bfft::Base<SC, 0, kTw> none{};
      bfft::stage<SC, 0, SIGN, kTw>(v, none);
    } else if constexpr (I == 1) {
      bfft::stage<SC, 1, SIGN, kTw>(v, w1);
    } else if constexpr (I == 2) {
      bfft::stage<SC, 2, SIGN, kTw>(v, w2);
    } else {
      bfft::stage<SC, 3, SIGN, kTw>(v, w3);
    }
  }
  // exchange I; FROM_B / TO_B: the mappings it is written and read in
  template <int I, bool FROM_B, bool TO_B>
  __device__ __forceinline__ void exchange(double2 (&v)[P], double2* lds) const {
    constexpr bool wave = SC::kWave && kFull && !FROM_B && !TO_B;
    if (live) bfft::put<SC, I>(v, lds + (FROM_B ? gB : gA) * kRow, FROM_B ? sB : sA);
    bfft::sync<wave>();
    bfft::get<SC, I>(v, lds + (TO_B ? gB : gA) * kRow, TO_B ? sB : sA);
    if constexpr (I + 2 < N) bfft::sync<wave || (SC::kWave && kFull && FROM_B)>();
  }
  template <int I>
  __device__ __forceinline__ void transform(double2 (&v)[P], double2* lds) const {
    stage<I>(v);
    if constexpr (I + 1 < N) {
      exchange<I, in_b<I>(), in_b<I + 1>()>(v, lds);
      transform<I + 1>(v, lds);
    }
  }
};

template <typename ST, int KIND, int L>
__global__ void __launch_bounds__((Line<ST, KIND, L>::NT))
    __attribute__((amdgpu_waves_per_eu(Line<ST, KIND, L>::kWaves)))
fft_line_kernel(const PatchDev* __restrict__ patches, const WorkItem* __restrict__ items,
                int nitems, FieldPtrs fields, ST* __restrict__ ws) {
  using LN = Line<ST, KIND, L>;
  using V = typename LN::V;
  constexpr int P = LN::P, S = LN::S, H = P / 2;
  constexpr unsigned E = sizeof(V);
  __shared__ double2 lds[LN::TL::kLds];
  if (static_cast<int>(blockIdx.x) >= nitems) return;
  LN ln;
  typename LN::PT wpost{};
  {
    // every item of the launch has this length, and the tables depend only on it
    const PatchDev* P0 = patches + items[0].patch;
    ln.load_twiddles(LN::kX ? P0->fx.tw : (LN::kY ? P0->fy.tw : P0->fz.tw));
    if constexpr (LN::kX) wpost.load(P0->post, ln.sB);
  }
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const WorkItem wi = items[xcd_local_order(it, nitems)];
    const PatchDev* Pt = patches + wi.patch;
    V* const blk_x = reinterpret_cast<V*>(ws) + Pt->off_spec + wi.comp * Pt->comp_stride;
    V* const blk_z = reinterpret_cast<V*>(ws) + Pt->off_z + wi.comp * Pt->comp_stride;
    // the row of an idle slot of a short tile is a valid one; nothing is stored for it
    const bool actA = ln.live && ln.gA < wi.count, actB = ln.live && ln.gB < wi.count;
    const int rowA = ln.gA < wi.count ? ln.gA : 0, rowB = ln.gB < wi.count ? ln.gB : 0;
    // strided side: element n of row r at base + r + n C
    V* strided = nullptr;
    int C = 0;
    // contiguous side: row r at base + r step
    V* contig = nullptr;
    unsigned step = L * E;
    bool mapped = false;
    if constexpr (LN::kX) {
      C = Pt->ndim == 2 ? Pt->nz : Pt->ny;
      int p, a0;
      udivmod(wi.first, C, p, a0);
      strided = blk_x + static_cast<long long>(p) * Pt->mx * C + a0;
      mapped = Pt->map.on != 0;
      contig = reinterpret_cast<V*>(static_cast<ST*>(field_ptr(fields, wi.comp)) + Pt->off_real);
      if (!mapped) contig += static_cast<long long>(wi.first) * L;
      else contig = reinterpret_cast<V*>(field_ptr(fields, wi.comp));
    } else if constexpr (LN::kY) {
      C = Pt->nz;
      int kx, z0;
      udivmod(wi.first, C, kx, z0);
      contig = blk_x + (static_cast<long long>(z0) * Pt->mx + kx) * L;
      step = static_cast<unsigned>(Pt->mx) * L * E;
      strided = blk_z + static_cast<long long>(kx) * L * C + z0;
    } else {
      contig = blk_z + static_cast<long long>(wi.first) * L;
    }
    const unsigned offA = rowA * step + ln.sA * E;
    const unsigned offB = (rowB + ln.sB * static_cast<unsigned>(C)) * E;
    const unsigned stepB = S * static_cast<unsigned>(C) * E;  // S columns on

    double2 v[P];
    if constexpr (LN::kFwd || LN::kZ) {
      if (LN::kX && mapped) {
        const MappedRow mr(Pt, wi.first + rowA);
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = up(contig[mr.pair(ln.sA + S * m)]);
      } else {
        V raw[P];
#pragma unroll
        for (int m = 0; m < P; ++m) raw[m] = at(contig, offA + S * m * E);
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = up(raw[m]);
      }
    } else if constexpr (KIND == kYInv) {
      V raw[P];
#pragma unroll
      for (int m = 0; m < P; ++m) raw[m] = at(strided, offB + m * stepB);
#pragma unroll
      for (int m = 0; m < P; ++m) v[m] = up(raw[m]);
    } else {
      // x inverse: the pairs X[k], X[L - k] of k = s + S m, m < P / 2 (k = 0:
      // columns 0 and L / 2), and their pre-step
      const unsigned offP = (rowB + (ln.sB == 0 ? L / 2 : L - ln.sB) * static_cast<unsigned>(C)) * E;
      V xa[H], xb[H];
#pragma unroll
      for (int m = 0; m < H; ++m) {
        xa[m] = at(strided, offB + m * stepB);
        xb[m] = at(strided, m == 0 ? offP
                                   : (rowB + (L - S * m - ln.sB) * static_cast<unsigned>(C)) * E);
      }
      double2* const half = lds + ln.gB * LN::kHalf;
      static_for<0, H>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        const double2 a = up(xa[m]), b = up(xb[m]);
        // q = i conj(W^k) (a - conj b);  Z[k] = p + q, Z[L-k] = conj(p - q)
        const double2 w = wpost.template get<m>();
        const double2 p = bfft::c2(a.x + b.x, a.y - b.y), d = bfft::c2(a.x - b.x, a.y + b.y);
        double2 z1 = bfft::c2(fma(-w.x, d.y, fma(w.y, d.x, p.x)), fma(w.x, d.x, fma(w.y, d.y, p.y)));
        double2 z2 = bfft::c2(fma(2.0, p.x, -z1.x), -fma(2.0, p.y, -z1.y));
        if (m == 0 && ln.sB == 0) {  // DC and Nyquist packed; Z[L/2] = 2 conj X[L/2]
          z1 = bfft::c2(a.x + a.y, a.x - a.y);
          z2 = bfft::c2(2.0 * b.x, -2.0 * b.y);
        }
        v[m] = z1;
        const int slot = (m == 0 && ln.sB == 0) ? 0 : L / 2 - S * m - ln.sB;
        if (ln.live) half[slot] = z2;
      });
      __syncthreads();
#pragma unroll
      for (int m = 0; m < H; ++m) v[H + m] = half[ln.sB + S * m];
      __syncthreads();
    }

    ln.template transform<0>(v, lds);

    if constexpr (KIND == kXFwd) {
      // upper half to LDS, the partners back, both halves of every pair stored
      double2* const half = lds + ln.gB * LN::kHalf;
      __syncthreads();
      if (ln.live) {
#pragma unroll
        for (int m = 0; m < H; ++m) half[ln.sB + S * m] = v[H + m];
      }
      __syncthreads();
      const unsigned offP = (rowB + (ln.sB == 0 ? L / 2 : L - ln.sB) * static_cast<unsigned>(C)) * E;
      static_for<0, H>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        const int slot = (m == 0 && ln.sB == 0) ? 0 : L / 2 - S * m - ln.sB;
        const double2 a = v[m], b = half[slot];
        const double2 w = wpost.template get<m>();
        const double2 s = bfft::c2(a.x + b.x, a.y - b.y), d = bfft::c2(a.x - b.x, a.y + b.y);
        double2 x1 = bfft::c2(fma(-w.y, d.y, fma(w.x, d.x, 0.5 * s.x)),
                              fma(w.y, d.x, fma(w.x, d.y, 0.5 * s.y)));
        double2 x2 = bfft::c2(s.x - x1.x, x1.y - s.y);
        if (m == 0 && ln.sB == 0) {
          x1 = bfft::c2(a.x + a.y, a.x - a.y);
          x2 = bfft::c2(b.x, -b.y);
        }
        if (actB) {
          at(strided, offB + m * stepB) = down<V>(x1);
          at(strided, m == 0 ? offP : (rowB + (L - S * m - ln.sB) * static_cast<unsigned>(C)) * E) =
              down<V>(x2);
        }
      });
    } else if constexpr (KIND == kYFwd) {
      if (actB) {
#pragma unroll
        for (int m = 0; m < P; ++m) at(strided, offB + m * stepB) = down<V>(v[m]);
      }
    } else {
      if (LN::kX && mapped) {
        const MappedRow mr(Pt, wi.first + rowA);
        const int ix0 = Pt->map.ix0, ix1 = Pt->map.ix1;
#pragma unroll
        for (int m = 0; m < P; ++m) {
          const int j = ln.sA + S * m;
          if (actA && mr.inside && 2 * j >= ix0 && 2 * j < ix1) contig[mr.pair(j)] = down<V>(v[m]);
        }
      } else if (actA) {
#pragma unroll
        for (int m = 0; m < P; ++m) at(contig, offA + S * m * E) = down<V>(v[m]);
      }
    }
    __syncthreads();  // the LDS rows are reused by the next tile
  }
}

template <typename ST, int KIND, int L>
hipError_t launch_one(int grid, hipStream_t stream, const PatchDev* p, const WorkItem* it, int n,
                      const FieldPtrs& f, void* ws) {
  hipLaunchKernelGGL((fft_line_kernel<ST, KIND, L>), dim3(grid), dim3(Line<ST, KIND, L>::NT), 0,
                     stream, p, it, n, f, static_cast<ST*>(ws));
  return hipGetLastError();
}

template <typename ST, int L>
hipError_t launch_kind(int kind, int grid, hipStream_t stream, const PatchDev* p,
                       const WorkItem* it, int n, const FieldPtrs& f, void* ws) {
  switch (kind) {
    case kXFwd: return launch_one<ST, kXFwd, L>(grid, stream, p, it, n, f, ws);
    case kXInv: return launch_one<ST, kXInv, L>(grid, stream, p, it, n, f, ws);
    case kYFwd: return launch_one<ST, kYFwd, L>(grid, stream, p, it, n, f, ws);
    case kYInv: return launch_one<ST, kYInv, L>(grid, stream, p, it, n, f, ws);
    case kZFwd: return launch_one<ST, kZFwd, L>(grid, stream, p, it, n, f, ws);
    case kZInv: return launch_one<ST, kZInv, L>(grid, stream, p, it, n, f, ws);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

}  // namespace lines
}  // namespace psatd

// The launcher of one group of lengths.
#define PSATD_LINE_CASE(LEN)                                                                       \
  case LEN:                                                                                        \
    return precision == 0 ? launch_kind<float, LEN>(kind, grid, stream, patches, items, nitems,    \
                                                    fields, ws)                                    \
                          : launch_kind<double, LEN>(kind, grid, stream, patches, items, nitems,   \
                                                     fields, ws);
#define PSATD_LINE_DEFINE(name, LIST)                                                              \
  namespace psatd {                                                                                \
  namespace lines {                                                                                \
  PSATD_LINE_GROUP(name) {                                                                         \
    switch (L) {                                                                                   \
      LIST(PSATD_LINE_CASE)                                                                        \
      default: return hipErrorInvalidValue;                                                        \
    }                                                                                              \
  }                                                                                                \
  }                                                                                                \
  }

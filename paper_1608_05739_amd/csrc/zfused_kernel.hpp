// The fused z pass with compile-time length (included by zfused_*.hip).
//
// For T lines at a time: forward FFT along z of every input, the per-mode
// update, inverse FFT of E' and B', all in one kernel; the transformed inputs
// stay with their thread in storage precision, as the generic kernel keeps
// them.  In 2D the two polarization sets are separate work (neighbouring
// workgroups take the two sets of the same lines), in 3D all components
// couple.  In FP32 the inputs are walked in a loop that is not unrolled, so
// that one transform's code and registers serve all of them (unrolled, the 3D
// rho form at 512 points spilled 182 registers: 8.2 ms at 512^3 against 2.8);
// the next input's loads are in flight during a transform where registers
// allow.  Lines of up to 64 threads never leave their wave, so that their
// exchanges need no workgroup barrier.
//
// Bound: the FP64 instructions of the transforms and of the update, at two waves
// per SIMD or one (Budget).  Measured, z pass alone: 512^3 rho form FP32 4.43 ->
// 2.89 ms (2.06 -> 3.16 TB/s; the kernel before accumulated the six outputs input by
// input, rounding each contribution to FP32, at one wave per SIMD); 1152 x 1536
// J form 192 -> 90 us, 216 x 96 x 144 vacuum 235 -> 78 us, 1024^2 rho FP64 99
// -> 51 us, 128 x 192 x 256 rho FP64 470 -> 253 us (the generic kernel before).
#pragma once

#include "update.hpp"
#include "zfused.hpp"

namespace psatd {
namespace zfused {

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

// One complex value per input of a set, input c at a register index that may
// be the (uniform) counter of a loop: each 32-bit part is a vector of N
// registers, so that a write is one indexed move instead of a chain of
// branches with a copy of the whole array on every path.
template <int N, typename ST>
struct Held;
template <int N>
struct Held<N, float> {
  typedef float VN __attribute__((ext_vector_type(N)));
  VN x, y;
  __device__ __forceinline__ void set(int c, double2 v) {
    x[c] = static_cast<float>(v.x);
    y[c] = static_cast<float>(v.y);
  }
  __device__ __forceinline__ double2 get(int c) const { return bfft::c2(x[c], y[c]); }
};
template <int N>
struct Held<N, double> {
  typedef int VN __attribute__((ext_vector_type(N)));
  VN xl, xh, yl, yh;
  __device__ __forceinline__ void set(int c, double2 v) {
    xl[c] = __double2loint(v.x);
    xh[c] = __double2hiint(v.x);
    yl[c] = __double2loint(v.y);
    yh[c] = __double2hiint(v.y);
  }
  __device__ __forceinline__ double2 get(int c) const {
    return bfft::c2(__hiloint2double(xh[c], xl[c]), __hiloint2double(yh[c], yl[c]));
  }
};

template <typename ST, int DIM, int SRC, int L>
struct ZLine {
  using SC = bfft::Sched<L, bfft::kFusedZ>;
  using TL = Tile<L>;
  using BU = Budget<DIM, SRC, L, sizeof(ST)>;
  using V = typename Store<ST>::V;
  static constexpr int P = SC::P, S = SC::S, N = SC::N, T = TL::T, NT = TL::NT;
  static constexpr bool kFull = NT == T * S;
  static constexpr bfft::Twiddles kTw = BU::kTw;
  static constexpr bool kWave = SC::kWave && kFull;
  static constexpr int kSlots = BU::HELD_LDS * P * NT;  // thread slots of held inputs (V)
  // LDS in double2: the rows, the slots, the copy of the twiddles
  static constexpr int kTwiddlesAt = T * SC::kRow + (kSlots * static_cast<int>(sizeof(V)) + 15) / 16;
  static constexpr int kLds = kTwiddlesAt + BU::kTwiddles;
  static_assert(SC::valid() && SC::separable() && N >= 2, "schedule");

  int g, s;
  bool live;
  bfft::Base<SC, 1, kTw> w1;
  bfft::Base<SC, (N > 2 ? 2 : 1), kTw> w2;
  bfft::Base<SC, (N > 3 ? 3 : 1), kTw> w3;
  bfft::Base<SC, (N > 4 ? 4 : 1), kTw> w4;

  __device__ __forceinline__ ZLine() {
    const int tid = threadIdx.x;
    live = kFull || tid < T * S;
    const int t = live ? tid : 0;
    g = t / S;
    s = t % S;
  }
  // (kShared: the copy is written by the whole workgroup, ends with a barrier)
  __device__ __forceinline__ void load_twiddles(const double2* tw, double2* lds) {
    if constexpr (kTw == bfft::kShared) {
      bfft::fill_shared<SC>(lds + kTwiddlesAt, tw, threadIdx.x, NT);
      __syncthreads();
      tw = lds + kTwiddlesAt;
    }
    w1.load(tw, s);
    if constexpr (N > 2) w2.load(tw, s);
    if constexpr (N > 3) w3.load(tw, s);
    if constexpr (N > 4) w4.load(tw, s);
  }
  template <int I, int SIGN>
  __device__ __forceinline__ void stage(double2 (&v)[P]) const {
    if constexpr (I == 0) {
      bfft::Base<SC, 0, kTw> none{};
      bfft::stage<SC, 0, SIGN, kTw>(v, none);
    } else if constexpr (I == 1) {
      bfft::stage<SC, 1, SIGN, kTw>(v, w1);
    } else if constexpr (I == 2) {
      bfft::stage<SC, 2, SIGN, kTw>(v, w2);
    } else if constexpr (I == 3) {
      bfft::stage<SC, 3, SIGN, kTw>(v, w3);
    } else {
      bfft::stage<SC, 4, SIGN, kTw>(v, w4);
    }
  }
  template <int SIGN, int I = 0>
  __device__ __forceinline__ void transform(double2 (&v)[P], double2* lds) const {
    stage<I, SIGN>(v);
    if constexpr (I + 1 < N) {
      double2* const row = lds + g * SC::kRow;
      if (live) bfft::put<SC, I>(v, row, s);
      bfft::sync<kWave>();
      bfft::get<SC, I>(v, row, s);
      bfft::sync<kWave>();
      transform<SIGN, I + 1>(v, lds);
    }
  }
};

// One set (2D: G = 0 or 1) or all components (3D: G = 2) of one item.
template <typename ST, int DIM, int SRC, int L, int G>
__device__ __forceinline__ void z_set(const ZLine<ST, DIM, SRC, L>& ln, const PatchDev* P,
                                      const WorkItem& wi, ST* __restrict__ ws, const Physics& ph,
                                      double2* lds) {
  using LN = ZLine<ST, DIM, SRC, L>;
  using V = typename LN::V;
  using Gr = Group<G, SRC>;
  constexpr int NP = LN::P, S = LN::S, NIN = Gr::nin, NOUT = Gr::nout;
  // the last inputs (charge in the rho form) may stay in LDS
  constexpr int NL = NIN > 3 ? (LN::BU::HELD_LDS < NIN - 3 ? LN::BU::HELD_LDS : NIN - 3) : 0;
  constexpr int NR = NIN - NL;
  // FP32: loops that are not unrolled; FP64, whose values take two registers of
  // an indexed array each (511 spills), as straight code with one transform at a
  // time
  constexpr bool kUnroll = sizeof(ST) == 8;
  V* const slot = reinterpret_cast<V*>(lds + LN::T * LN::SC::kRow) + threadIdx.x;
  V* const base = reinterpret_cast<V*>(ws) + P->off_z + static_cast<long long>(wi.first) * L;
  const bool act = ln.live && ln.g < wi.count;
  const int row = ln.g < wi.count ? ln.g : 0;  // idle threads: a valid line
  const unsigned off = (row * L + ln.s) * static_cast<unsigned>(sizeof(V));
  const long long cs = P->comp_stride;
  auto elem = [&](V* b, int m) -> V& {
    return *reinterpret_cast<V*>(reinterpret_cast<char*>(b) + (off + S * m * static_cast<unsigned>(sizeof(V))));
  };

  Held<NR, ST> held[NP];
  V nxt[NP];
  if constexpr (LN::BU::kPrefetch) {
#pragma unroll
    for (int m = 0; m < NP; ++m) nxt[m] = elem(base + Gr::in[0] * cs, m);
  }
  auto input = [&](auto cc) __attribute__((always_inline)) {
    const int c = cc;
    if constexpr (!LN::BU::kPrefetch) {
      V* const src = base + Gr::in[c] * cs;
#pragma unroll
      for (int m = 0; m < NP; ++m) nxt[m] = elem(src, m);
    }
    double2 v[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) v[m] = up(nxt[m]);
    if (LN::BU::kPrefetch && c + 1 < NIN) {
      V* const src = base + Gr::in[c + 1] * cs;
#pragma unroll
      for (int m = 0; m < NP; ++m) nxt[m] = elem(src, m);
    }
    ln.template transform<-1>(v, lds);
    if (NL == 0 || c < NR) {
#pragma unroll
      for (int m = 0; m < NP; ++m) held[m].set(c, v[m]);
    } else {
#pragma unroll
      for (int m = 0; m < NP; ++m) slot[((c - NR) * NP + m) * LN::NT] = down<V>(v[m]);
    }
  };
  if constexpr (kUnroll) {
    static_for<0, NIN>([&](auto cc) __attribute__((always_inline)) {
      input(cc);
      __builtin_amdgcn_sched_barrier(0);
    });
  } else {
#pragma unroll 1
    for (int c = 0; c < NIN; ++c) input(c);
  }

  // the update of every mode (kx, ky of the line, kz of mode s + S m)
  const int line = wi.first + row;
  double kx, ky = 0.0;
  if constexpr (DIM == 2) {
    kx = gload(P->kx, line);
  } else {
    int ix, iy;
    udivmod(line, P->ny, ix, iy);
    kx = gload(P->kx, ix);
    ky = gload(P->ky, iy);
  }
  double kzv[NP];
#pragma unroll
  for (int m = 0; m < NP; ++m) kzv[m] = gload(P->kz, ln.s + S * m);
  const double dt = P->dt, scale = P->inv_n;
#pragma unroll
  for (int m = 0; m < NP; ++m) {
    __builtin_amdgcn_sched_barrier(0);  // one mode at a time (registers)
    double2 in[11];
    static_for<0, NIN>([&](auto sc) __attribute__((always_inline)) {
      constexpr int k = decltype(sc)::value;
      if constexpr (k < NR) in[k] = held[m].get(k);
      else in[k] = up(slot[((k - NR) * NP + m) * LN::NT]);
    });
    if constexpr (DIM == 2) {
      update_set<ST, G, SRC>(kx, kzv[m], dt, ph.c, ph.eps0, scale, in);
#pragma unroll
      for (int k = 0; k < 3; ++k) held[m].set(k, in[k]);
    } else {
      const double kz = kzv[m];
      const Coef q = psatd_coef<ST>(kx * kx + ky * ky + kz * kz, dt, ph.c, ph.eps0, scale);
      double2 Eo[3], Bo[3];
      update_mode<SRC>(kx, ky, kz, q, ph.c, ph.eps0, dt, in, in + 3, in + 6, in[9], in[10], Eo, Bo);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        held[m].set(k, Eo[k]);
        held[m].set(k + 3, Bo[k]);
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // the outputs back along z, over their inputs
  auto output = [&](auto oc) __attribute__((always_inline)) {
    const int o = oc;
    double2 v[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) v[m] = held[m].get(o);
    ln.template transform<1>(v, lds);
    if (act) {
      V* const dst = base + Gr::in[o] * cs;
#pragma unroll
      for (int m = 0; m < NP; ++m) elem(dst, m) = down<V>(v[m]);
    }
  };
  if constexpr (kUnroll) {
    static_for<0, NOUT>([&](auto oc) __attribute__((always_inline)) {
      output(oc);
      __builtin_amdgcn_sched_barrier(0);
    });
  } else {
#pragma unroll 1
    for (int o = 0; o < NOUT; ++o) output(o);
  }
}

template <typename ST, int DIM, int SRC, int L>
__global__ void __launch_bounds__((ZLine<ST, DIM, SRC, L>::NT))
    __attribute__((amdgpu_waves_per_eu(Budget<DIM, SRC, L, sizeof(ST)>::waves)))
fft_z_kernel(const PatchDev* __restrict__ patches, const WorkItem* __restrict__ items, int nitems,
             ST* __restrict__ ws, Physics ph) {
  using LN = ZLine<ST, DIM, SRC, L>;
  __shared__ double2 lds[LN::kLds];
  constexpr int kSets = DIM == 2 ? 2 : 1;
  const int nwork = kSets * nitems;
  if (static_cast<int>(blockIdx.x) >= nwork) return;
  LN ln;
  ln.load_twiddles(patches[items[0].patch].fz.tw, lds);  // one length per launch
  for (int w = blockIdx.x; w < nwork; w += gridDim.x) {
    const WorkItem wi = items[w / kSets];
    const PatchDev* P = patches + wi.patch;
    if constexpr (DIM == 2) {
      if ((w & 1) == 0) z_set<ST, DIM, SRC, L, 0>(ln, P, wi, ws, ph, lds);
      else z_set<ST, DIM, SRC, L, 1>(ln, P, wi, ws, ph, lds);
    } else {
      z_set<ST, DIM, SRC, L, 2>(ln, P, wi, ws, ph, lds);
    }
  }
}

template <typename ST, int DIM, int SRC, int L>
hipError_t launch_one(int grid, hipStream_t stream, const PatchDev* p, const WorkItem* it, int n,
                      void* ws, Physics ph) {
  if constexpr (compiled(sizeof(ST), DIM, SRC, L)) {
    hipLaunchKernelGGL((fft_z_kernel<ST, DIM, SRC, L>), dim3(grid),
                       dim3(ZLine<ST, DIM, SRC, L>::NT), 0, stream, p, it, n, static_cast<ST*>(ws), ph);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <typename ST, int DIM, int L>
hipError_t launch_src(int src, int grid, hipStream_t stream, const PatchDev* p, const WorkItem* it,
                      int n, void* ws, Physics ph) {
  switch (src) {
    case kVacuum: return launch_one<ST, DIM, kVacuum, L>(grid, stream, p, it, n, ws, ph);
    case kRho: return launch_one<ST, DIM, kRho, L>(grid, stream, p, it, n, ws, ph);
    case kJForm: return launch_one<ST, DIM, kJForm, L>(grid, stream, p, it, n, ws, ph);
    case kPstdVacuum: return launch_one<ST, DIM, kPstdVacuum, L>(grid, stream, p, it, n, ws, ph);
    case kPstdJ: return launch_one<ST, DIM, kPstdJ, L>(grid, stream, p, it, n, ws, ph);
    default: return hipErrorInvalidValue;
  }
}

template <int L>
hipError_t launch_len(int precision, int ndim, int src, int grid, hipStream_t stream,
                      const PatchDev* p, const WorkItem* it, int n, void* ws, Physics ph) {
  if (ndim == 2)
    return precision == 0 ? launch_src<float, 2, L>(src, grid, stream, p, it, n, ws, ph)
                          : launch_src<double, 2, L>(src, grid, stream, p, it, n, ws, ph);
  return precision == 0 ? launch_src<float, 3, L>(src, grid, stream, p, it, n, ws, ph)
                        : launch_src<double, 3, L>(src, grid, stream, p, it, n, ws, ph);
}

}  // namespace

}  // namespace zfused
}  // namespace psatd

#define PSATD_Z_CASE(LEN) \
  case LEN: return launch_len<LEN>(precision, ndim, src, grid, stream, patches, items, nitems, ws, ph);
#define PSATD_Z_DEFINE(name, LIST)   \
  namespace psatd {                  \
  namespace zfused {                 \
  PSATD_Z_GROUP(name) {              \
    switch (nz) {                    \
      LIST(PSATD_Z_CASE)             \
      default: return hipErrorInvalidValue; \
    }                                \
  }                                  \
  }                                  \
  }

// Compile-time FFTs of lines spread over the threads of a workgroup (gfx950).
//
// A line of L = P S points belongs to S threads; thread s holds the points
// s + S m (m < P) in registers.  Each Stockham stage of radix R (R divides P)
// runs P / R butterflies per thread: butterfly t is j = s + S t, it reads
// x[j + q L/R] -- register t + q P/R of the thread --, multiplies by w^q with
// w = exp(SIGN 2 pi i (j mod Ns) / (Ns R)), applies the DFT of length R and
// produces y[(j - j mod Ns) R + j mod Ns + q Ns] (Ns = product of the radices
// before the stage).  Between stages the threads exchange y through LDS and
// read back y[s + S m].  Input and output are in natural order.
//
// What bounds these transforms on this chip, and what follows from it:
// - An FP64 instruction issues every 4 cycles per SIMD, like any other.  The
//   butterflies are radix 2 and 3 steps with the stage twiddle folded in:
//   r = a + w b is four FMAs and a - w b = 2 a - r two more, so that a
//   radix-8 butterfly with its seven twiddles takes 84 operations (108 as
//   seven products, their powers and an untwiddled DFT of 8), a radix-16 one
//   220 (288).
// - LDS: a wave writes 16-byte elements at 13 cycles per instruction whatever
//   the pattern (up to two lanes per bank), and reads them at 4 when the 64
//   lanes are consecutive (measured).  Exchanges are therefore few: 16 points
//   per thread do 256 points in one exchange where 8 points need two.
#pragma once

#include <hip/hip_runtime.h>

#include "fft.hpp"

namespace psatd {
namespace bfft {

#define PSATD_HD __host__ __device__ __forceinline__

// ------------------------------------------------------------------ constants
// cos(pi m / 72) for the multiples that the radices use: 10, 15 and 22.5
// degrees (m = 4, 6 and 9 per step), and 7.5 for the r2c post-twiddles (3), from
// first-quadrant values so that the symmetries hold exactly.
constexpr double cos_72(int m) {
  m %= 144;
  if (m < 0) m += 144;
  if (m > 72) return cos_72(144 - m);
  if (m > 36) return -cos_72(72 - m);
  switch (m) {
    case 0: return 1.0;
    case 3: return 0.99144486137381041114;   // 7.5 degrees
    case 4: return 0.98480775301220805937;   // 10
    case 6: return 0.96592582628906828675;   // 15
    case 8: return 0.93969262078590838405;   // 20
    case 9: return 0.92387953251128675613;   // 22.5
    case 12: return 0.86602540378443864676;  // 30
    case 15: return 0.79335334029123516458;  // 37.5
    case 16: return 0.76604444311897803520;  // 40
    case 18: return 0.70710678118654752440;  // 45
    case 20: return 0.64278760968653932632;  // 50
    case 21: return 0.60876142900872063942;  // 52.5
    case 24: return 0.5;                     // 60
    case 27: return 0.38268343236508977173;  // 67.5
    case 28: return 0.34202014332566873304;  // 70
    case 30: return 0.25881904510252076235;  // 75
    case 32: return 0.17364817766693034885;  // 80
    case 33: return 0.13052619222005159155;  // 82.5
    default: return m == 36 ? 0.0 : 2.0;     // (2: not a value of these radices)
  }
}
constexpr double sin_72(int m) { return cos_72(36 - m); }

constexpr bool unit_circle() {
  for (int m = 0; m < 144; ++m)
    if (m % 4 == 0 || m % 3 == 0) {
      const double r = cos_72(m) * cos_72(m) + sin_72(m) * sin_72(m) - 1.0;
      if (r > 4e-16 || r < -4e-16) return false;
    }
  return true;
}
static_assert(unit_circle() && cos_72(24) == 0.5 && sin_72(12) == 0.5, "cos / sin tables");

// ------------------------------------------------------------------ butterflies
PSATD_HD double2 c2(double x, double y) {
  double2 v;
  v.x = x;
  v.y = y;
  return v;
}
PSATD_HD double2 mul(double2 a, double2 b) {
  return c2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
PSATD_HD double2 sqr(double2 a) {
  const double t = a.x * a.y;
  return c2(fma(a.x, a.x, -a.y * a.y), t + t);
}
// a * exp(SIGN 2 pi i M / N)
template <int N, int M, int SIGN>
PSATD_HD double2 rot(double2 a) {
  constexpr int m = 144 / N * M % 144;
  static_assert(144 % N == 0 && cos_72(m) <= 1.0, "constant twiddle");
  if constexpr (M == 0) {
    return a;
  } else if constexpr (m == 18) {  // 45 degrees: one factor
    constexpr double h = cos_72(18);
    return SIGN > 0 ? c2((a.x - a.y) * h, (a.x + a.y) * h) : c2((a.x + a.y) * h, (a.y - a.x) * h);
  } else {
    constexpr double c = cos_72(m), s = SIGN * sin_72(m);
    return c2(fma(a.x, c, -a.y * s), fma(a.x, s, a.y * c));
  }
}

// a, b <- a + w b, a - w b
PSATD_HD void bfly(double2& a, double2& b, double2 w) {
  const double2 r = c2(fma(-w.y, b.y, fma(w.x, b.x, a.x)), fma(w.y, b.x, fma(w.x, b.y, a.y)));
  b = c2(fma(2.0, a.x, -r.x), fma(2.0, a.y, -r.y));
  a = r;
}
// a, b <- a + SIGN i w b, a - SIGN i w b
template <int SIGN>
PSATD_HD void bfly_i(double2& a, double2& b, double2 w) {
  double2 t = SIGN > 0 ? c2(-b.y, b.x) : c2(b.y, -b.x);
  bfly(a, t, w);
  b = t;
}
PSATD_HD void bfly1(double2& a, double2& b) {
  const double2 d = c2(a.x - b.x, a.y - b.y);
  a = c2(a.x + b.x, a.y + b.y);
  b = d;
}
template <int SIGN>
PSATD_HD void bfly1_i(double2& a, double2& b) {
  double2 t = SIGN > 0 ? c2(-b.y, b.x) : c2(b.y, -b.x);
  bfly1(a, t);
  b = t;
}

// The powers of a twiddle base that a butterfly of radix R uses: 1 and twice
// those of R / 2; 1, 2 for R = 3; 1, 2 and three times those of 3 for R = 9.
constexpr int power_count(int R) { return R == 1 ? 0 : (R == 3 ? 2 : (R == 9 ? 4 : 1 + power_count(R / 2))); }
constexpr int power(int R, int j) {
  if (R % 2 == 0) return j == 0 ? 1 : 2 * power(R / 2, j - 1);
  return j < 2 ? j + 1 : 3 * (j - 1);
}
// The same from the base alone, for FP32 storage: each squaring doubles the
// relative error of the table's rounding, which 2^-24 does not show.
template <int R>
PSATD_HD void powers(double2 u, double2* p) {
  if constexpr (R == 1) {
    return;
  } else if constexpr (R % 2 == 0) {
    p[0] = u;
    if constexpr (R > 2) powers<R / 2>(sqr(u), p + 1);
  } else {
    p[0] = u;
    p[1] = sqr(u);
    if constexpr (R == 9) powers<3>(mul(p[1], u), p + 2);
  }
}

// x0, x1, x2 <- DFT of length 3 of (x0, u x1, u^2 x2) (T) or (x0, x1, x2)
template <int SIGN, bool T>
PSATD_HD void dft3(double2& x0, double2& x1, double2& x2, double2 u, double2 u2) {
  constexpr double h = SIGN * 0.86602540378443864676;
  double2 s, d;
  if constexpr (T) {
    const double2 b = mul(x2, u2);
    s = c2(fma(-u.y, x1.y, fma(u.x, x1.x, b.x)), fma(u.y, x1.x, fma(u.x, x1.y, b.y)));
    d = c2(fma(-2.0, b.x, s.x), fma(-2.0, b.y, s.y));
  } else {
    s = c2(x1.x + x2.x, x1.y + x2.y);
    d = c2(x1.x - x2.x, x1.y - x2.y);
  }
  const double2 m = c2(fma(-0.5, s.x, x0.x), fma(-0.5, s.y, x0.y));
  x0 = c2(x0.x + s.x, x0.y + s.y);
  x1 = c2(fma(-h, d.y, m.x), fma(h, d.x, m.y));
  x2 = c2(fma(h, d.y, m.x), fma(-h, d.x, m.y));
}

// In-place DFT of length R (natural order in and out) of a[q] u^q (T) or a[q]:
// v[k] <- sum_q a[q] u^q exp(SIGN 2 pi i q k / R), p the powers of u.
// Decimation in time: the halves (or thirds) are transforms with base u^2
// (u^3), joined by butterflies with the twiddles u W_R^k.
template <int R, int SIGN, bool T>
PSATD_HD void dft(double2 (&a)[R], const double2* p) {
  if constexpr (R == 1) {
    return;
  } else if constexpr (R == 3) {
    dft3<SIGN, T>(a[0], a[1], a[2], p[0], p[1]);
  } else if constexpr (R % 2 == 1) {
    static_assert(R == 9, "odd radix");
    double2 y[3][3];
    static_for<0, 3>([&](auto rc) __attribute__((always_inline)) {
      constexpr int r = decltype(rc)::value;
      for (int q = 0; q < 3; ++q) y[r][q] = a[r + 3 * q];
      dft<3, SIGN, T>(y[r], p + 2);
    });
    static_for<0, 3>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      if constexpr (!T && k == 0) {
        dft3<SIGN, false>(y[0][0], y[1][0], y[2][0], p[0], p[1]);
      } else {
        constexpr double cs = cos_72(16 * k), sn = SIGN * sin_72(16 * k);
        constexpr double cs2 = cos_72(32 * k), sn2 = SIGN * sin_72(32 * k);
        const double2 w = T ? rot<9, k, SIGN>(p[0]) : c2(cs, sn);
        const double2 w2 = T ? rot<9, 2 * k, SIGN>(p[1]) : c2(cs2, sn2);
        dft3<SIGN, true>(y[0][k], y[1][k], y[2][k], w, w2);
      }
    });
    for (int r = 0; r < 3; ++r)
      for (int k = 0; k < 3; ++k) a[k + 3 * r] = y[r][k];
  } else {
    constexpr int H = R / 2;
    double2 e[H], o[H];
#pragma unroll
    for (int q = 0; q < H; ++q) {
      e[q] = a[2 * q];
      o[q] = a[2 * q + 1];
    }
    dft<H, SIGN, T>(e, p + 1);
    dft<H, SIGN, T>(o, p + 1);
    // twiddles u W_R^k; from k = R / 4 on they repeat with a factor SIGN i
    constexpr int K = R % 4 == 0 ? R / 4 : H;
    static_for<0, K>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      if constexpr (T) {
        const double2 w = rot<R, k, SIGN>(p[0]);
        bfly(e[k], o[k], w);
        if constexpr (K < H) bfly_i<SIGN>(e[k + K], o[k + K], w);
      } else if constexpr (k == 0) {
        bfly1(e[0], o[0]);
        if constexpr (K < H) bfly1_i<SIGN>(e[K], o[K]);
      } else {
        constexpr double cs = cos_72(144 / R * k), sn = SIGN * sin_72(144 / R * k);
        bfly(e[k], o[k], c2(cs, sn));
        if constexpr (K < H) bfly_i<SIGN>(e[k + K], o[k + K], c2(cs, sn));
      }
    });
#pragma unroll
    for (int k = 0; k < H; ++k) {
      a[k] = e[k];
      a[k + H] = o[k];
    }
  }
}

// Where the twiddles of a stage come from.  FP32 storage keeps the base of each
// butterfly and squares it (kSquares).  FP64 storage takes them from the plan's
// table, so that its transforms are not less exact than those of the generic
// kernels, whose stages of at most 8 points multiply powers up: read once and
// held (kTable, the line passes), or read from a copy in LDS (kShared, most fused
// z passes, whose registers hold a set of inputs).  Relative error of a transform
// of Gaussian values, 1e-16, squared / from the table / generic: 192 points 3.4 /
// 1.8 / 2.5, 432 points 3.9 / 2.0 / 2.3, 1024 points 3.3 / 2.3 / 3.3.
enum Twiddles { kSquares, kTable, kShared };

// Radices 6, 12, 18 and 24.  Their butterflies with folded twiddles multiply the
// base by constants of both factors (144 points: 2.2 with folded twiddles from
// the table, 2.0 the generic kernels); FP64 storage multiplies the points by
// their twiddles and transforms them by the prime-factor algorithm, which has no
// twiddles of its own (1.7).  Both forms of a radix-12 butterfly are about 160
// operations.
constexpr bool mixed(int R) { return R % 6 == 0; }

// Of the powers that such a butterfly takes, those below W and the multiples of W
// come from the table and the others are one product each: 8 instead of 23 values
// for 24 points, 5 instead of 11 for 12 (error at 1152 points 2.05 instead of
// 2.00; 2D rho form of 2592 x 768, FP64, fused z pass: 128 us, 131 with all 11
// read from LDS).
constexpr int split(int R) { return R == 18 ? 3 : 4; }  // W

// Twiddles a butterfly of radix R takes, and the power of the base that each is.
constexpr int twiddle_count(int R, Twiddles tw) {
  if (tw == kSquares) return 1;
  if (!mixed(R)) return power_count(R);
  return split(R) - 1 + (R - 1) / split(R);
}
constexpr int twiddle_power(int R, Twiddles tw, int j) {
  if (tw == kSquares || !mixed(R)) return power(R, j);
  return j < split(R) ? j + 1 : split(R) * (j - split(R) + 2);
}
// Twiddle u^q of a mixed radix from those (p).
template <int R, int Q>
PSATD_HD double2 twiddle(const double2* p) {
  constexpr int W = split(R), lo = Q % W, hi = Q / W;
  if constexpr (hi == 0) return p[Q - 1];
  else if constexpr (lo == 0) return p[W - 2 + hi];
  else return mul(p[lo - 1], p[W - 2 + hi]);
}

// In-place DFT of length R = A B, A a power of two and B = 3 or 9, by the
// prime-factor algorithm (Good 1958): input (B i + A j) mod R is element (i, j)
// of a two-dimensional transform, whose element (k mod A, k mod B) is output k.
// Other lengths as dft without twiddles.
template <int R, int SIGN>
PSATD_HD void dft_prime_factor(double2 (&a)[R]) {
  if constexpr (!mixed(R)) {
    dft<R, SIGN, false>(a, nullptr);
  } else {
    constexpr int B = R % 9 == 0 ? 9 : 3, A = R / B;
    double2 y[B][A];
#pragma unroll
    for (int i = 0; i < A; ++i) {
      double2 t[B];
#pragma unroll
      for (int j = 0; j < B; ++j) t[j] = a[(B * i + A * j) % R];
      dft<B, SIGN, false>(t, nullptr);
#pragma unroll
      for (int j = 0; j < B; ++j) y[j][i] = t[j];
    }
#pragma unroll
    for (int j = 0; j < B; ++j) dft<A, SIGN, false>(y[j], nullptr);
#pragma unroll
    for (int k = 0; k < R; ++k) a[k] = y[k % B][k % A];
  }
}

// ------------------------------------------------------------------ schedules
// P points per thread and up to five radices, in the order of the stages.
struct Radices {
  int P, n, r[5];
};

// Schedules of the passes that hold one transform at a time.  Every radix
// divides P.  The last stage has P / R twiddle bases per thread: up to three of
// them are cheaper than a twiddled butterfly of 24 (154 registers against 218
// at 192 = 24.8); from four on the last radix is P (1152 = 24.2.24 holds 2
// bases, 24.24.2 would hold 13).
constexpr Radices line_radices(int L) {
  switch (L) {
    case 24: return {12, 2, {2, 12}};
    case 32: return {8, 2, {4, 8}};
    case 36: return {12, 2, {3, 12}};
    case 48: return {12, 2, {4, 12}};
    case 54: return {18, 2, {18, 3}};
    case 64: return {8, 2, {8, 8}};
    case 72: return {12, 2, {12, 6}};
    case 96: return {24, 2, {12, 8}};
    case 108: return {18, 2, {18, 6}};
    case 128: return {16, 2, {8, 16}};
    case 144: return {12, 2, {12, 12}};
    case 162: return {18, 2, {18, 9}};
    case 192: return {24, 2, {24, 8}};
    case 216: return {18, 3, {6, 2, 18}};
    case 256: return {16, 2, {16, 16}};
    case 288: return {24, 2, {24, 12}};
    case 324: return {18, 2, {18, 18}};
    case 384: return {12, 4, {4, 4, 2, 12}};
    case 432: return {12, 3, {12, 3, 12}};
    case 486: return {18, 3, {9, 3, 18}};
    case 512: return {8, 3, {8, 8, 8}};
    case 576: return {24, 2, {24, 24}};
    case 648: return {12, 4, {6, 3, 3, 12}};
    case 768: return {12, 4, {4, 4, 4, 12}};
    case 864: return {24, 3, {12, 3, 24}};
    case 1024: return {16, 3, {16, 4, 16}};
    case 1152: return {24, 3, {24, 2, 24}};
    case 1296: return {12, 4, {12, 3, 3, 12}};
    case 1536: return {24, 3, {8, 8, 24}};
    case 1728: return {24, 3, {24, 3, 24}};
    case 2048: return {16, 3, {16, 8, 16}};
    default: return {0, 0, {0}};
  }
}

// FP64 storage: the same, except where 18 or 24 points of 16 bytes leave too few
// waves (288 points, x passes of 16 MiB components: 4.3 forward and 3.7 TB/s
// inverse as 24.12, 5.3 and 5.2 as 12.2.12) or spill with the twiddles (1728
// points, x passes of 4.0 M cells: 241 and 175 us as 24.3.24, 191 and 112 as
// 12.12.12; 1152 points 152 and 88 as 24.2.24, 179 and 121 as 12.4.2.12).
constexpr Radices line_radices_f64(int L) {
  switch (L) {
    case 216: return {12, 3, {6, 3, 12}};
    case 288: return {12, 3, {12, 2, 12}};
    case 864: return {12, 3, {12, 6, 12}};
    case 1728: return {12, 3, {12, 12, 12}};
    default: return line_radices(L);
  }
}

// Schedules of the fused z passes, whose threads also hold a set of
// transformed inputs: at most 12 points per thread, and one twiddle base per
// stage (the last radix is P).
constexpr Radices fused_radices(int L) {
  switch (L) {
    case 32: return {8, 2, {4, 8}};
    case 36: return {12, 2, {3, 12}};
    case 48: return {12, 2, {4, 12}};
    case 54: return {6, 3, {3, 3, 6}};
    case 64: return {8, 2, {8, 8}};
    case 72: return {12, 2, {6, 12}};
    case 96: return {12, 3, {4, 2, 12}};
    case 108: return {12, 3, {3, 3, 12}};
    case 128: return {8, 3, {8, 2, 8}};
    case 144: return {12, 2, {12, 12}};
    case 162: return {6, 4, {3, 3, 3, 6}};
    case 192: return {12, 3, {4, 4, 12}};
    case 216: return {12, 3, {6, 3, 12}};
    case 256: return {8, 3, {8, 4, 8}};
    case 288: return {12, 3, {12, 2, 12}};
    case 324: return {6, 4, {6, 3, 3, 6}};
    case 384: return {12, 4, {4, 4, 2, 12}};
    case 432: return {12, 3, {12, 3, 12}};
    case 512: return {8, 3, {8, 8, 8}};
    case 576: return {12, 3, {12, 4, 12}};
    case 648: return {12, 4, {6, 3, 3, 12}};
    case 768: return {12, 4, {4, 4, 4, 12}};
    case 864: return {12, 3, {12, 6, 12}};
    case 1024: return {8, 4, {8, 8, 2, 8}};
    case 1152: return {12, 4, {12, 4, 2, 12}};
    case 1296: return {12, 4, {12, 3, 3, 12}};
    case 1536: return {12, 5, {4, 4, 2, 4, 12}};
    case 1728: return {12, 3, {12, 12, 12}};
    case 2048: return {8, 4, {8, 8, 4, 8}};
    case 2304: return {12, 4, {12, 4, 4, 12}};
    case 3072: return {12, 5, {4, 4, 4, 4, 12}};
    case 4096: return {8, 4, {8, 8, 8, 8}};
    default: return {0, 0, {0}};
  }
}

enum Use { kLine32, kLine64, kFusedZ };

template <int L_, Use USE>
struct Sched {
  static constexpr Radices rd = USE == kFusedZ   ? fused_radices(L_)
                                : USE == kLine64 ? line_radices_f64(L_)
                                                 : line_radices(L_);
  static constexpr int L = L_;
  static constexpr int P = rd.P;       // points per thread
  static constexpr int S = L / P;      // threads per line
  static constexpr int N = rd.n;       // stages
  static constexpr bool kWave = 64 % S == 0;  // a line never leaves its wave
  static constexpr int radix(int i) { return rd.r[i]; }
  static constexpr int ns(int i) {  // product of the radices before stage i
    int n = 1;
    for (int j = 0; j < i; ++j) n *= rd.r[j];
    return n;
  }
  static constexpr bool valid() {
    if (P < 1 || L % P != 0 || ns(N) != L) return false;
    for (int i = 0; i < N; ++i)
      if (P % rd.r[i] != 0) return false;
    return true;
  }
  // Padding of exchange i (after stage i): PAD elements after every D.  The
  // first exchange writes with a stride of its radix: one element after each
  // block of a radix that is a multiple of 4.  Blocks of Ns = 4 elements
  // (R Ns apart) get four.  The others meet at most two lanes per bank, which
  // costs a write nothing.
  static constexpr int pad_d(int i) {
    if (i == 0 && rd.r[0] % 4 == 0) return rd.r[0];
    if (i > 0 && ns(i) == 4 && (S % (4 * rd.r[i]) == 0 || (4 * rd.r[i]) % S == 0)) return 4 * rd.r[i];
    return L;
  }
  static constexpr int pad_n(int i) { return i == 0 ? 1 : 4; }
  static constexpr int pa(int i, int e) { return e + (e / pad_d(i)) * pad_n(i); }
  // elements of a line's LDS row, odd so that rows start in different banks
  static constexpr int row() {
    int m = L;
    for (int i = 0; i + 1 < N; ++i) {
      const int need = pa(i, L - 1) + 1;
      if (need > m) m = need;
    }
    return m | 1;
  }
  static constexpr int kRow = row();
  // Stockham output index of butterfly t, output q, thread s at stage i
  static constexpr PSATD_HD int out(int i, int s, int t, int q) {
    const int R = rd.r[i], n = ns(i);
    const int j = s + S * t, k = j % n;
    return (j - k) * R + k + q * n;
  }
  // The padded reads s + S m are a thread base plus a constant where the
  // padding period divides S or S divides it; the writes of a butterfly stay
  // inside one period by the choice of pad_d.
  static constexpr bool separable() {
    for (int i = 0; i + 1 < N; ++i) {
      const int d = pad_d(i);
      if (d != L && S % d != 0 && d % S != 0) return false;
    }
    return true;
  }
  // padded distance of consecutive outputs of a butterfly
  static constexpr int step(int i) { return pa(i, out(i, 0, 0, 1)) - pa(i, out(i, 0, 0, 0)); }
};

// The thread's twiddle bases of stage I (exp(-2 pi i k / (Ns R)), one per
// butterfly), from the plan's table tw[m] = exp(-2 pi i m / L).
template <typename SC, int I>
PSATD_HD int twiddle_index(int s, int t) {
  return ((s + SC::S * t) % SC::ns(I)) * (SC::L / (SC::ns(I) * SC::radix(I)));
}
// Distinct bases of stage I: butterflies repeat with period Ns / S in t.
template <typename SC, int I>
constexpr int bases() {
  constexpr int ns = SC::ns(I), bpt = SC::P / SC::radix(I);
  if (ns == 1) return 0;
  if (SC::S % ns == 0) return 1;
  if (ns % SC::S == 0) return ns / SC::S < bpt ? ns / SC::S : bpt;
  return bpt;
}
constexpr int at_least_one(int n) { return n > 0 ? n : 1; }

// The thread's twiddles of stage I: get(t, j) is twiddle j of butterfly t.
// Held in registers:
template <typename SC, int I, Twiddles TW>
struct Base {
  static constexpr int kCount = twiddle_count(SC::radix(I), TW);
  static constexpr int kBases = at_least_one(bases<SC, I>());
  double2 w[kBases][kCount];
  PSATD_HD void load(const double2* tw, int s) {
#pragma unroll
    for (int t = 0; t < bases<SC, I>(); ++t) {
      const int i = twiddle_index<SC, I>(s, t);
      static_for<0, kCount>([&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value, e = twiddle_power(SC::radix(I), TW, j);
        w[t][j] = gload(tw, i * e);
      });
    }
  }
  PSATD_HD double2 get(int t, int j) const { return w[t % kBases][j]; }
};

// The LDS copy of every stage's twiddles: twiddle j of the butterflies with
// j mod Ns = k at [j][k], so that neighbouring threads read neighbouring
// elements.  First element of stage I's (I = SC::N: the size).
template <typename SC>
constexpr int shared_offset(int I) {
  int n = 0;
  for (int i = 1; i < I; ++i) n += twiddle_count(SC::radix(i), kShared) * SC::ns(i);
  return n;
}
// Thread `tid` of `nt` writes its part (the caller synchronizes).
template <typename SC, int I = 1>
PSATD_HD void fill_shared(double2* lds, const double2* tw, int tid, int nt) {
  if constexpr (I < SC::N) {
    constexpr int R = SC::radix(I), ns = SC::ns(I), step = SC::L / (ns * R);
    static_for<0, twiddle_count(R, kShared)>([&](auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value, e = step * twiddle_power(R, kShared, j);
      constexpr int first = shared_offset<SC>(I) + j * ns;
      for (int k = tid; k < ns; k += nt) lds[first + k] = gload(tw, k * e);
    });
    fill_shared<SC, I + 1>(lds, tw, tid, nt);
  }
}
template <typename SC, int I>
struct Base<SC, I, kShared> {
  static constexpr int kBases = at_least_one(bases<SC, I>());
  const double2* p[kBases];
  PSATD_HD void load(const double2* lds, int s) {
#pragma unroll
    for (int t = 0; t < bases<SC, I>(); ++t) {
      constexpr int first = shared_offset<SC>(I);
      p[t] = lds + first + (s + SC::S * t) % SC::ns(I);
    }
  }
  PSATD_HD double2 get(int t, int j) const { return p[t % kBases][j * SC::ns(I)]; }
};

// Stage I on the thread's points: v[t + q P/R] is input q of butterfly t, and
// output q after it.
template <typename SC, int I, int SIGN, Twiddles TW>
PSATD_HD void stage(double2 (&v)[SC::P], const Base<SC, I, TW>& tb) {
  constexpr int R = SC::radix(I), BPT = SC::P / R, NPOW = power_count(R);
  constexpr int COUNT = twiddle_count(R, TW);
  constexpr bool products = TW != kSquares && mixed(R);
#pragma unroll
  for (int t = 0; t < BPT; ++t) {
    double2 a[R];
#pragma unroll
    for (int q = 0; q < R; ++q) a[q] = v[t + q * BPT];
    if constexpr (SC::ns(I) > 1) {
      double2 p[COUNT > NPOW ? COUNT : NPOW];
#pragma unroll
      for (int j = 0; j < COUNT; ++j) {
        double2 u = tb.get(t, j);
#if defined(__HIP_DEVICE_COMPILE__)
        // a copy the optimizer cannot see through: the products of the base are
        // formed in each transform, not kept live from one to the next
        if constexpr (TW != kShared) asm volatile("" : "+v"(u.x), "+v"(u.y));
#endif
        if constexpr (SIGN > 0) u.y = -u.y;
        p[j] = u;
      }
      if constexpr (products) {
        static_for<1, R>([&](auto qc) __attribute__((always_inline)) {
          constexpr int q = decltype(qc)::value;
          a[q] = mul(a[q], twiddle<R, q>(p));
        });
        dft_prime_factor<R, SIGN>(a);
      } else {
        if constexpr (TW == kSquares) powers<R>(p[0], p);
        dft<R, SIGN, true>(a, p);
      }
    } else if constexpr (TW != kSquares) {
      dft_prime_factor<R, SIGN>(a);
    } else {
      dft<R, SIGN, false>(a, nullptr);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) v[t + q * BPT] = a[q];
  }
}

// Exchange I: stage I's outputs into the line's LDS row, and the points of
// stage I + 1 out of it.
template <typename SC, int I>
PSATD_HD void put(const double2 (&v)[SC::P], double2* row, int s) {
  constexpr int R = SC::radix(I), BPT = SC::P / R, ns = SC::ns(I);
  static_assert(SC::valid() && SC::separable(), "schedule");
#pragma unroll
  for (int t = 0; t < BPT; ++t) {
    // the block of butterfly t is a constant where Ns divides S or S t
    constexpr bool fixed = SC::S % ns == 0;
    const int b = fixed ? SC::pa(I, SC::out(I, s, 0, 0)) + SC::pa(I, SC::out(I, 0, t, 0)) - SC::pa(I, 0)
                        : SC::pa(I, SC::out(I, s, t, 0));
#pragma unroll
    for (int q = 0; q < R; ++q) row[b + q * SC::step(I)] = v[t + q * BPT];
  }
}
template <typename SC, int I>
PSATD_HD void get(double2 (&v)[SC::P], const double2* row, int s) {
  const int b = SC::pa(I, s);
#pragma unroll
  for (int m = 0; m < SC::P; ++m) v[m] = row[b + SC::pa(I, SC::S * m)];
}

// Wave-level ordering of LDS traffic (a line inside one wave), or the
// workgroup barrier.
template <bool WAVE>
__device__ __forceinline__ void sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

}  // namespace bfft
}  // namespace psatd

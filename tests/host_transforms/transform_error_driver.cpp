// Error of the compile-time transforms (bfft.hpp) of the FP64 passes, run on
// the host: every compiled line length of the line passes and of the fused z
// passes, both signs, with the schedule and the twiddles that the kernels use,
// against a DFT in long double.  Prints "pass length error bound" per case (in
// units of 1e-16) and exits with status 0 only if every error is in its bound.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "lines.hpp"
#include "zfused.hpp"

using namespace psatd;

namespace {

typedef long double real;
const real kPi = acosl(-1.0L);

struct Wide {
  real x, y;
};

std::vector<double2> table(int L) {
  std::vector<double2> t(L);
  for (int m = 0; m < L; ++m) {
    const real a = -2 * kPi * m / L;
    t[m] = make_double2(static_cast<double>(cosl(a)), static_cast<double>(sinl(a)));
  }
  return t;
}

std::vector<Wide> dft(const std::vector<double2>& in, int sign) {
  const int L = static_cast<int>(in.size());
  std::vector<Wide> w(L), out(L);
  for (int m = 0; m < L; ++m) w[m] = Wide{cosl(2 * kPi * m / L), sign * sinl(2 * kPi * m / L)};
  for (int k = 0; k < L; ++k) {
    Wide s{0, 0};
    for (int n = 0, i = 0; n < L; ++n) {
      s.x += w[i].x * in[n].x - w[i].y * in[n].y;
      s.y += w[i].x * in[n].y + w[i].y * in[n].x;
      i += k;
      if (i >= L) i -= L;
    }
    out[k] = s;
  }
  return out;
}

// The stages from I on, thread by thread, through rows laid out as in LDS.
template <typename SC, int I, int SIGN, bfft::Twiddles TW>
void stages(std::vector<double2>& a, const double2* tw) {
  std::vector<double2> row(SC::kRow);
  for (int s = 0; s < SC::S; ++s) {
    double2 v[SC::P];
    for (int m = 0; m < SC::P; ++m) v[m] = a[s + SC::S * m];
    bfft::Base<SC, I, TW> base{};
    if (I > 0) base.load(tw, s);
    bfft::stage<SC, I, SIGN, TW>(v, base);
    if constexpr (I + 1 < SC::N) {
      bfft::put<SC, I>(v, row.data(), s);
    } else {
      for (int m = 0; m < SC::P; ++m) row[s + SC::S * m] = v[m];
    }
  }
  for (int s = 0; s < SC::S; ++s) {
    double2 v[SC::P];
    if constexpr (I + 1 < SC::N) {
      bfft::get<SC, I>(v, row.data(), s);
    } else {
      for (int m = 0; m < SC::P; ++m) v[m] = row[s + SC::S * m];
    }
    for (int m = 0; m < SC::P; ++m) a[s + SC::S * m] = v[m];
  }
  if constexpr (I + 1 < SC::N) stages<SC, I + 1, SIGN, TW>(a, tw);
}

template <typename SC, int SIGN, bfft::Twiddles TW>
real error(std::mt19937_64& gen) {
  std::normal_distribution<double> normal;
  std::vector<double2> tw = table(SC::L), shared;
  if (TW == bfft::kShared) {
    shared.resize(bfft::shared_offset<SC>(SC::N));
    for (int t = 0; t < 64; ++t) bfft::fill_shared<SC>(shared.data(), tw.data(), t, 64);
  }
  real num = 0, den = 0;
  for (int r = 0; r < 4096 / SC::L + 2; ++r) {
    std::vector<double2> a(SC::L);
    for (double2& v : a) v = make_double2(normal(gen), normal(gen));
    const std::vector<Wide> ref = dft(a, SIGN);
    stages<SC, 0, SIGN, TW>(a, TW == bfft::kShared ? shared.data() : tw.data());
    for (int k = 0; k < SC::L; ++k) {
      const real x = a[k].x - ref[k].x, y = a[k].y - ref[k].y;
      num += x * x + y * y;
      den += ref[k].x * ref[k].x + ref[k].y * ref[k].y;
    }
  }
  return sqrtl(num / den);
}

int failed = 0;

template <typename SC, bfft::Twiddles TW>
void check(const char* pass) {
  std::mt19937_64 gen(SC::L);
  // the root-mean-square error of an FFT grows as the root of its stages: 0.75
  // units of rounding per radix-2 stage
  const real bound = 0.76L * 0x1p-53L * sqrtl(log2l(static_cast<real>(SC::L)));
  const real f = error<SC, -1, TW>(gen), b = error<SC, 1, TW>(gen);
  const bool ok = f <= bound && b <= bound;
  if (!ok) ++failed;
  std::printf("%s %d forward %.2Lf inverse %.2Lf bound %.2Lf%s\n", pass, SC::L, f * 1e16L, b * 1e16L,
              bound * 1e16L, ok ? "" : " FAIL");
}

template <int L>
void line() {
  check<bfft::Sched<L, bfft::kLine64>, lines::Tile<L, 8, true>::kTw>("line");
}
// Does a form of the FP64 fused z pass take its twiddles this way?
template <int L, int DIM, bfft::Twiddles TW>
constexpr bool any_form() {
  return (zfused::compiled(8, DIM, kVacuum, L) && zfused::Budget<DIM, kVacuum, L, 8>::kTw == TW) ||
         (zfused::compiled(8, DIM, kRho, L) && zfused::Budget<DIM, kRho, L, 8>::kTw == TW) ||
         (zfused::compiled(8, DIM, kJForm, L) && zfused::Budget<DIM, kJForm, L, 8>::kTw == TW);
}
template <int L, bfft::Twiddles TW>
void fused_with(const char* pass) {
  if constexpr (any_form<L, 2, TW>() || any_form<L, 3, TW>()) check<bfft::Sched<L, bfft::kFusedZ>, TW>(pass);
}
template <int L>
void fused() {
  fused_with<L, bfft::kSquares>("fused, squares");
  fused_with<L, bfft::kTable>("fused, table");
  fused_with<L, bfft::kShared>("fused, LDS");
}

}  // namespace

// PART: the lengths of this program (several, compiled in parallel)
int main() {
#define LINE(LEN) line<LEN>();
#define FUSED(LEN) fused<LEN>();
#if PART == 0
  PSATD_LINE_SMALL(LINE) PSATD_LINE_MID(LINE)
#elif PART == 1
  PSATD_LINE_LARGE(LINE) PSATD_LINE_LONG(LINE)
#elif PART == 2
  PSATD_Z_A(FUSED) PSATD_Z_B(FUSED)
#else
  PSATD_Z_C(FUSED) PSATD_Z_D(FUSED) PSATD_Z_E(FUSED) PSATD_Z_F(FUSED)
#endif
  std::printf("%d failed\n", failed);
  return failed == 0 ? 0 : 1;
}

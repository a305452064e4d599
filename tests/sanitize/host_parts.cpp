// Parts of libfrg's host code against plain forms of themselves (built with g++ under
// AddressSanitizer and UndefinedBehaviorSanitizer, no GPU):
//   - the elimination of a tridiagonal system from both ends (stepper.cpp) against the
//     band LU with partial pivoting and 80-bit residuals, with and without row swaps,
//     odd and even numbers of middle rows, singular systems;
//   - the panels and moments of the radial sums, the nodes of the mass panels and the
//     regulator table (tables.cpp) against 80-bit sums.
// stepper.cpp is included for its internal types.  Exit status 0 and the line "host
// parts ok" mean every check held.
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <random>
#include <vector>

#include "stepper.cpp"

namespace frg {
int fail(int code, const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  std::vfprintf(stderr, fmt, ap);
  va_end(ap);
  std::fputc('\n', stderr);
  return code;
}
void clear_error() {}
double now_s() { return 0.0; }
int check_lpa(const frg_lpa &) { return 0; }
}  // namespace frg

using namespace frg;
typedef long double ld;

static int failures = 0;
#define CHECK(c)                                                             \
  do {                                                                       \
    if (!(c)) {                                                              \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c);   \
      ++failures;                                                            \
    }                                                                        \
  } while (0)

static std::mt19937_64 rng(1);
static double uni(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }

// ------------------------------------------------------------- elimination --
// |b - A x| / (|A| |x|) in the maximum norm, A = I - gamma J in 80 bits.
static ld backward(int64_t n, double gamma, const std::vector<double> &jac,
                   const std::vector<double> &b, const std::vector<double> &x) {
  ld res = 0.0L, norm = 0.0L, xmax = 0.0L;
  for (int64_t i = 0; i < n; ++i) {
    ld r = b[i], row = 0.0L;
    for (int o = -3; o <= 3; ++o) {
      const int64_t j = i + o;
      if (j < 0 || j >= n) continue;
      const ld a = (o == 0 ? 1.0L : 0.0L) - (ld)gamma * jac[(o + 3) * n + i];
      r -= a * x[j];
      row += fabsl(a);
    }
    res = std::max(res, fabsl(r));
    norm = std::max(norm, row);
    xmax = std::max(xmax, fabsl((ld)x[i]));
  }
  return res / (norm * xmax);
}

// Bands of a Jacobian whose rows 1..n-2 are tridiagonal; swaps: off-diagonal entries
// larger than the diagonal ones on some rows, so that both ends pivot.
static std::vector<double> bands(int64_t n, bool swaps) {
  std::vector<double> jac(7 * n, 0.0);
  for (int64_t i = 0; i < n; ++i) {
    const double off = swaps && uni(0, 1) < 0.5 ? 8.0 : 0.4;
    jac[2 * n + i] = i > 0 ? uni(-off, off) : 0.0;
    jac[4 * n + i] = i + 1 < n ? uni(-off, off) : 0.0;
    jac[3 * n + i] = uni(-1, 1) * (swaps ? 1.0 : 0.1);
  }
  jac[5 * n] = uni(-2, 2);
  jac[6 * n] = uni(-2, 2);
  jac[1 * n + n - 1] = uni(-2, 2);
  jac[n - 1] = uni(-2, 2);
  return jac;
}

static void elimination() {
  int swapped[2] = {0, 0};
  for (int64_t n : {32, 33, 40, 41, 127, 1024, 1025})
    for (int rep = 0; rep < 20; ++rep) {
      const bool swaps = rep % 2;
      const double gamma = uni(0.5, 1.5);
      const std::vector<double> jac = bands(n, swaps);
      CHECK(TwoEndedLU::fits(n, jac.data()));
      TwoEndedLU two;
      BandLU band;
      CHECK(two.factor(n, gamma, jac.data()));
      band.assemble(n, gamma, jac.data());
      CHECK(band.factor());
      for (int64_t s = 0; s < two.h; ++s)
        for (int e = 0; e < 2; ++e) swapped[e] += two.sw[s] >> e & 1;
      std::vector<double> b(n), x, y;
      for (double &v : b) v = uni(-1, 1);
      x = y = b;
      two.solve(x.data());
      band.solve(y.data());
      // growth under partial pivoting of such a system is at most 2, and a row takes a
      // few operations: a few units of 1.1e-16
      CHECK(backward(n, gamma, jac, b, x) < 2e-15L);
      CHECK(backward(n, gamma, jac, b, y) < 2e-15L);
    }
  CHECK(swapped[0] > 100 && swapped[1] > 100);
  // what it does not take: short systems, a far band inside, NaN there
  const int64_t n = 64;
  std::vector<double> jac = bands(n, false);
  CHECK(!TwoEndedLU::fits(31, bands(31, false).data()));
  for (int o : {0, 1, 5, 6})
    for (double v : {1e-300, (double)NAN}) {
      std::vector<double> k = jac;
      k[o * n + 17] = v;
      CHECK(!TwoEndedLU::fits(n, k.data()));
    }
  // singular: a zero row at either end, in the middle, and elsewhere; NaN on the diagonal
  for (int64_t at : {(int64_t)0, n - 1, n / 2, (int64_t)9, n - 11}) {
    std::vector<double> k = jac;
    for (int o = 0; o < 7; ++o) k[o * n + at] = 0.0;
    k[3 * n + at] = 1.0;  // 1 - gamma J with gamma = 1
    for (int64_t i : {at - 1, at, at + 1})  // and its column
      if (i >= 0 && i < n) k[(at - i + 3) * n + i] = i == at ? 1.0 : 0.0;
    if (at > 0 && at < 4) k[(at + 3) * n] = 0.0;
    TwoEndedLU two;
    CHECK(!two.factor(n, 1.0, k.data()));
    k[3 * n + at] = NAN;
    CHECK(!two.factor(n, 1.0, k.data()));
  }
}

// ------------------------------------------------------------ radial sums --
static void radial_panels(int d, int reg, int n_r, double q_max) {
  const LpaTable t = build_lpa_table(d, reg, n_r, q_max);
  const std::vector<double> tab = build_fv_panels(t);
  CHECK((int)tab.size() == kFvTable);
  double h_max = 0.0;
  for (int i = 0; i < n_r; ++i) h_max = std::max(h_max, t.data[n_r + i]);
  auto sums = [&](ld x, ld &s1, ld &s2) {
    s1 = s2 = 0.0L;
    for (int i = 0; i < n_r; ++i) {
      const ld g = 1.0L / ((ld)t.data[n_r + i] + x);
      s1 += t.data[i] * g;
      s2 += t.data[i] * g * g;
    }
  };
  ld e1 = 0.0L, e2 = 0.0L, f1, f2;
  for (int p = 0; p < kPanels; ++p)
    for (double w : {0.0, uni(0, 1), 1.0 - 1e-15}) {
      const double lo = std::ldexp(1.0 + (double)(p % kFvPerOctave) / kFvPerOctave,
                                   kPanelLo + p / kFvPerOctave);
      const double width = std::ldexp(1.0 / kFvPerOctave, kPanelLo + p / kFvPerOctave);
      const double x = lo + w * width;
      const ld z = (ld)x - ((ld)lo + 0.5L * width);
      ld P = 0.0L, D = 0.0L;
      for (int k = kFvPoly - 1; k >= 0; --k) {
        D = D * z + P;
        P = P * z + tab[(size_t)p * kFvPoly + k];
      }
      sums(x, f1, f2);
      e1 = std::max(e1, fabsl(P / f1 - 1.0L));
      e2 = std::max(e2, fabsl(-D / f2 - 1.0L));
    }
  // The coefficients' own rounding: 1.11e-16 of the first and 1/33, 1/33^2 .. of that of
  // the next (of s2 twice, three times .. that).  s2 lacks T_11' too, 121 2^-10 33^-10 =
  // 7.7e-17, and its terms from the second on are summed in double: 2/33 of a few
  // 1.1e-16.
  CHECK(e1 < 1.3e-16L);
  CHECK(e2 < 2.4e-16L);
  const double *C = tab.data() + (size_t)kPanels * kFvPoly;
  CHECK((C[0] > 0.0) == (h_max <= std::ldexp(1.0, kFvTailH)));
  if (C[0] > 0.0)
    for (int e : {kPanelHi, kPanelHi + 1, 40, 100, 400}) {
      const ld x = ldexpl(1.0L + (ld)uni(0, 0.999), e), z = 1.0L / x;
      sums(x, f1, f2);
      const ld s1 = z * (C[0] - z * (C[1] - z * (C[2] - z * C[3])));
      const ld s2 = z * z * (C[0] - z * (2.0L * C[1] - z * (3.0L * C[2] - z * 4.0L * C[3])));
      CHECK(fabsl(s1 / f1 - 1.0L) < 1.2e-16L);
      CHECK(fabsl(s2 / f2 - 1.0L) < 1.2e-16L);
    }
}

// -------------------------------------------------------------- mass nodes --
// Barycentric interpolation through the table's nodes of delta^pw times a product of
// poles, at points between, next to and on the nodes.
static void mass_nodes() {
  const std::vector<double> t = build_mass_nodes();
  const int n = kMassNodes;
  CHECK((int)t.size() == 5 * n);
  for (int i = 0; i < n; ++i) {
    CHECK(t[i] > 1.0 && t[i] < 16.0);
    const ld u = (ld)t[n + i] + t[2 * n + i];
    CHECK(fabsl(u - logl((ld)t[i] / 4.0L)) < 1e-18L);
  }
  ld worst = 0.0L;
  for (int rep = 0; rep < 2000; ++rep) {
    const int poles = rep % 2 ? 3 : 4;
    const ld pw = poles / 2.0L;
    ld H[4];
    for (int k = 0; k < poles; ++k) H[k] = rep % 5 ? powl(10.0L, uni(-3, 3)) : (rep % 3 ? 0.0L : 1e6L);
    auto f = [&](ld x) {
      ld v = powl(x, pw);
      for (int k = 0; k < poles; ++k) v /= x + H[k];
      return v;
    };
    const double x = rep % 7 ? 1.0 + 15.0 * uni(0, 1) : t[rep % n] * (1.0 + 1e-12 * uni(-1, 1));
    const ld u = logl((ld)x / 4.0L);
    ld num = 0.0L, den = 0.0L;
    for (int i = 0; i < n; ++i) {
      const ld w = ((ld)t[3 * n + i] + t[4 * n + i]) / (u - ((ld)t[n + i] + t[2 * n + i]));
      num += w * f(t[i]);
      den += w;
    }
    worst = std::max(worst, fabsl(num / den / f(x) - 1.0L));
  }
  // 2.2e-18 of the interpolant; next to a node the difference of u carries the 80-bit
  // rounding of both logarithms, which cancels in the quotient
  CHECK(worst < 1e-17L);
}

// --------------------------------------------------------- regulator table --
static void regulator() {
  const std::vector<double> t = build_regulator_table();
  CHECK((int)t.size() == kRegPanels * kRegCoef);
  ld worst = 0.0L;
  for (int rep = 0; rep < 20000; ++rep) {
    const double y = rep % 4 == 0 ? std::pow(10.0, uni(-12, 3)) : uni(0.0, 45.0);
    uint64_t bits;
    std::memcpy(&bits, &y, 8);
    const uint32_t hi = (uint32_t)(bits >> 32);
    const int k = std::min(std::max((int)(hi >> 17) - kRegBits, 0), kRegPanels - 1);
    double c = 0.0;
    if (k > 0 && k < kRegPanels - 1) {
      bits = (uint64_t)((hi & 0xfffe0000u) | 0x00010000u) << 32;
      std::memcpy(&c, &bits, 8);
    }
    ld h = 0.0L;
    const ld f = (ld)y - c;
    for (int n = kRegCoef - 1; n >= 0; --n) h = h * f + t[k * kRegCoef + n];
    const ld w = -expm1l(-(ld)y);
    // (y - w)/w loses y/2 of itself below 1: its series there
    ld want = ((ld)y - w) / w;
    if (y < 0.25) {
      const ld z = (ld)y * y;
      want = y * 0.5L + z * (1.0L / 12 - z * (1.0L / 720 - z * (1.0L / 30240 - z * (1.0L / 1209600 -
             z * (1.0L / 47900160 - z * (691.0L / 1307674368000.0L))))));
    }
    worst = std::max(worst, fabsl(h / want - 1.0L));
  }
  // the rounding of ten coefficients, whose terms add up to h without much cancelling
  CHECK(worst < 2.2e-16L);
}

int main() {
  elimination();
  for (int reg : {FRG_REG_EXP, FRG_REG_LITIM})
    for (int n_r : {1, 7, 64, 200}) {
      radial_panels(3, reg, n_r, 6.0);
      if (n_r > 7) radial_panels(4, reg, n_r, 1000.0);  // fewer nodes all weigh nothing there
    }
  mass_nodes();
  regulator();
  if (failures) return 1;
  std::printf("host parts ok\n");
  return 0;
}

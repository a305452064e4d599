// Host-side quadrature and regulator tables.
//
// The Gauss-Legendre rule comes from the Golub-Welsch construction: the
// nodes are the eigenvalues of the symmetric tridiagonal Jacobi matrix of
// the Legendre polynomials (zero diagonal, off-diagonal j/sqrt(4j^2-1)),
// found by the implicit QL iteration with Wilkinson-type shifts in 80-bit
// arithmetic and polished by Newton steps on P_n; the weights are
//   w = 2 / ((1 - x^2) P_n'(x)^2),  (1 - x^2) P_n'(x) = n (P_{n-1}(x) - x P_n(x)).
#include <algorithm>
#include <cmath>
#include <vector>

#include "frg_internal.h"

namespace frg {

int gauss_legendre_gw(int n, double *x, double *w) {
  if (n < 1 || n > 4096 || !x || !w) return FRG_E_INVAL;
  std::vector<long double> d(n, 0.0L), e(n, 0.0L);
  for (int j = 1; j < n; ++j) e[j - 1] = j / sqrtl(4.0L * j * j - 1.0L);
  // implicit QL on (d, e): e[i] couples i and i+1
  for (int l = 0; l < n; ++l) {
    for (int iter = 0; iter < 200; ++iter) {
      int m = l;
      for (; m < n - 1; ++m) {
        long double dd = fabsl(d[m]) + fabsl(d[m + 1]);
        if (fabsl(e[m]) + dd == dd) break;
      }
      if (m == l) break;
      long double g = (d[l + 1] - d[l]) / (2.0L * e[l]);
      long double r = hypotl(g, 1.0L);
      g = d[m] - d[l] + e[l] / (g + (g >= 0 ? r : -r));
      long double s = 1.0L, c = 1.0L, p = 0.0L;
      int i = m - 1;
      bool deflated = false;
      for (; i >= l; --i) {
        long double f = s * e[i], b = c * e[i];
        r = hypotl(f, g);
        e[i + 1] = r;
        if (r == 0.0L) {
          d[i + 1] -= p;
          e[m] = 0.0L;
          deflated = true;
          break;
        }
        s = f / r;
        c = g / r;
        g = d[i + 1] - p;
        r = (d[i] - g) * s + 2.0L * c * b;
        p = s * r;
        d[i + 1] = g + p;
        g = c * r - b;
      }
      if (deflated) continue;
      d[l] -= p;
      e[l] = g;
      e[m] = 0.0L;
    }
  }
  std::sort(d.begin(), d.end());
  for (int i = 0; i < n; ++i) {
    // symmetrise: the rule is exactly symmetric about 0
    long double xi = 0.5L * (d[i] - d[n - 1 - i]);
    if (2 * i + 1 == n) xi = 0.0L;
    // P_{n-1}(xi) and P_n(xi) by the three-term recurrence; two Newton
    // corrections of the eigenvalue on P_n remove the QL rounding that the
    // weight formula would amplify near the ends of [-1, 1].
    long double pm = 1.0L, pn = xi;  // P_{n-1}, P_n
    for (int pass = 0; pass < 3; ++pass) {
      long double p0 = 1.0L, p1 = xi;
      for (int j = 1; j < n; ++j) {
        long double p2 = ((2.0L * j + 1.0L) * xi * p1 - j * p0) / (j + 1.0L);
        p0 = p1;
        p1 = p2;
      }
      pm = (n == 1) ? 1.0L : p0;
      pn = (n == 1) ? xi : p1;
      if (pass == 2 || 2 * i + 1 == n) break;
      const long double dpn = n * (xi * pn - pm) / (xi * xi - 1.0L);
      xi -= pn / dpn;
    }
    // w = 2 / ((1 - x^2) P_n'(x)^2) with (1 - x^2) P_n' = n (P_{n-1} - x P_n)
    const long double omx2 = (1.0L - xi) * (1.0L + xi);
    const long double s = n * (pm - xi * pn);
    long double wi = 2.0L * omx2 / (s * s);
    x[i] = (double)xi;
    w[i] = (double)wi;
  }
  return FRG_OK;
}

double omega_sphere(int n) { return 2.0 * std::pow(M_PI, 0.5 * n) / std::tgamma(0.5 * n); }

// h(y) = y/(1 - e^{-y}) - 1, Bernoulli series below 0.1
double h_exp_host(double y) {
  if (y < 0.1) {
    const double y2 = y * y;
    return y * 0.5 + y2 * (1.0 / 12.0 + y2 * (-1.0 / 720.0 + y2 * (1.0 / 30240.0 +
                                  y2 * (-1.0 / 1209600.0 + y2 * (1.0 / 47900160.0)))));
  }
  return y / (-std::expm1(-y)) - 1.0;
}

static double bern(double z) { return z == 0.0 ? 1.0 : z / std::expm1(z); }

double dtR_over_k2_host(int reg, double y) {
  if (reg == FRG_REG_EXP) return 2.0 * bern(y) * bern(-y);
  return y < 1.0 ? 2.0 : 0.0;
}

static double angular_weight_factor(int d, double x) {
  const double z = (1.0 - x) * (1.0 + x);
  double f = 1.0;
  for (int i = 0; i < (d - 3) / 2; ++i) f *= z;
  if ((d - 3) % 2) f *= std::sqrt(z);
  return f;
}

QuadTable build_quad_table(const frg_quad &q) {
  QuadTable t;
  const int nr = q.n_radial, na = q.n_angular;
  t.n_r = nr;
  t.n_a = na;
  t.k2 = q.k * q.k;
  t.inv_k2 = 1.0 / t.k2;
  t.pref = omega_sphere(q.d - 1) / std::pow(2.0 * M_PI, q.d);
  t.q_top = q.q_max;
  t.rmu_max = 0.0;
  t.data.assign(table_doubles(nr, na), 0.0);
  std::vector<double> xr(nr), wr(nr), xa(na), wa(na);
  gauss_legendre_gw(nr, xr.data(), wr.data());
  gauss_legendre_gw(na, xa.data(), wa.data());
  const double Q = (q.reg == FRG_REG_LITIM) ? std::min(q.q_max, q.k) : q.q_max;
  for (int i = 0; i < nr; ++i) {
    const double qi = 0.5 * Q * (1.0 + xr[i]);
    const double wi = 0.5 * Q * wr[i];
    const double s = qi * qi, y = s / t.k2;
    double qp = 1.0;
    for (int e = 0; e < q.d - 1; ++e) qp *= qi;
    t.data[i] = qi;
    t.data[nr + i] = wi * qp * (t.k2 * dtR_over_k2_host(q.reg, y));
    t.data[2 * nr + i] =
        (q.reg == FRG_REG_EXP) ? t.k2 * h_exp_host(y) : std::max(s - t.k2, 0.0);
  }
  for (int j = 0; j < na; ++j) {
    t.data[3 * nr + j] = 1.0 + xa[j];
    const double mu = wa[j] * angular_weight_factor(q.d, xa[j]);
    t.data[3 * nr + na + j] = mu;
    t.data[3 * nr + 2 * na + j] = 1.0 / mu;
    t.rmu_max = std::max(t.rmu_max, 1.0 / mu);
  }
  return t;
}

LpaTable build_lpa_table(int d, int reg, int n_r, double q_max_over_k) {
  LpaTable t;
  t.n_r = n_r;
  t.Cd = omega_sphere(d) / std::pow(2.0 * M_PI, d);
  t.data.assign(2 * n_r, 0.0);
  std::vector<double> xr(n_r), wr(n_r);
  gauss_legendre_gw(n_r, xr.data(), wr.data());
  const double Q = (reg == FRG_REG_LITIM) ? std::min(q_max_over_k, 1.0) : q_max_over_k;
  for (int i = 0; i < n_r; ++i) {
    const double qi = 0.5 * Q * (1.0 + xr[i]);
    const double wi = 0.5 * Q * wr[i];
    const double y = qi * qi;
    double qp = 1.0;
    for (int e = 0; e < d - 1; ++e) qp *= qi;
    t.data[i] = wi * qp * dtR_over_k2_host(reg, y);
    t.data[n_r + i] = (reg == FRG_REG_EXP) ? h_exp_host(y) : std::max(y - 1.0, 0.0);
  }
  // coefficient groups (products in long double; all terms are >= 0)
  const int ng = fv_groups(n_r);
  t.data.resize(2 * (size_t)n_r + (size_t)kFvCoef * ng, 0.0);
  for (int g = 0; g < ng; ++g) {
    long double c[kFvGroup], h[kFvGroup];
    for (int l = 0; l < kFvGroup; ++l) {
      const int i = kFvGroup * g + l;
      c[l] = i < n_r ? t.data[i] : 0.0L;
      h[l] = i < n_r ? t.data[n_r + i] : 1.0L;
    }
    // poly *= (x + hl), coefficients from x^0 up
    auto mul_lin = [](std::vector<long double> &p, long double hl) {
      p.push_back(0.0L);
      for (size_t k = p.size() - 1; k > 0; --k) p[k] = p[k - 1] + hl * p[k];
      p[0] *= hl;
    };
    std::vector<long double> P{1.0L};
    for (int l = 0; l < kFvGroup; ++l) mul_lin(P, h[l]);
    std::vector<long double> N(kFvGroup, 0.0L), M(2 * kFvGroup - 1, 0.0L);
    for (int i = 0; i < kFvGroup; ++i) {
      std::vector<long double> Pi{1.0L};
      for (int l = 0; l < kFvGroup; ++l)
        if (l != i) mul_lin(Pi, h[l]);
      for (int k = 0; k < kFvGroup; ++k) N[k] += c[i] * Pi[k];
      for (int k = 0; k < kFvGroup; ++k)
        for (int k2 = 0; k2 < kFvGroup; ++k2) M[k + k2] += c[i] * Pi[k] * Pi[k2];
    }
    double *dst = t.data.data() + 2 * (size_t)n_r + (size_t)kFvCoef * g;
    for (int k = 0; k < kFvGroup; ++k) dst[k] = (double)P[k];
    for (int k = 0; k < kFvGroup; ++k) dst[kFvGroup + k] = (double)N[k];
    for (int k = 0; k < 2 * kFvGroup - 1; ++k) dst[2 * kFvGroup + k] = (double)M[k];
  }
  return t;
}

// Per panel the Taylor series of s1 about the middle c, terms t_k = (-1)^k sum_i
// c_i w^k/(h_i + c)^(k+1) (w the half-width; w/c = 1/33 at most, so t_k/t_0 <=
// 33^-k), economised: the Chebyshev terms above degree kFvPoly - 1 = 10 are
// dropped (below 66^-11 = 1e-20 of s1; their derivative below 1e-16 of s2 / 2).
std::vector<double> build_fv_panels(const LpaTable &t) {
  constexpr int K = 14, n = kFvPoly;  // Taylor terms, coefficients kept
  // z^k = sum_j b[k][j] T_j(z); T_j = sum_i a[j][i] z^i
  static const auto econ = [] {
    std::vector<std::vector<long double>> a(K, std::vector<long double>(K, 0.0L)), b = a;
    a[0][0] = 1.0L;
    a[1][1] = 1.0L;
    for (int j = 2; j < K; ++j)
      for (int i = 0; i < K; ++i) a[j][i] = (i ? 2.0L * a[j - 1][i - 1] : 0.0L) - a[j - 2][i];
    b[0][0] = 1.0L;
    for (int k = 1; k < K; ++k)  // z T_j = (T_{j+1} + T_{|j-1|})/2
      for (int j = 0; j < k; ++j) {
        b[k][j + 1] += (j ? 0.5L : 1.0L) * b[k - 1][j];
        if (j) b[k][j - 1] += 0.5L * b[k - 1][j];
      }
    std::vector<long double> m(n * K, 0.0L);  // kept coefficient i of z^k
    for (int k = 0; k < K; ++k)
      for (int j = 0; j < n; ++j)
        for (int i = 0; i <= j; ++i) m[i * K + k] += b[k][j] * a[j][i];
    return m;
  }();
  const int n_r = t.n_r;
  std::vector<double> out((size_t)kFvTable);
  for (int p = 0; p < kPanels; ++p) {
    const int e = kPanelLo + p / kFvPerOctave, s = p % kFvPerOctave;
    const long double lo = ldexpl((long double)(kFvPerOctave + s) / kFvPerOctave, e);
    const long double w = ldexpl(0.5L / kFvPerOctave, e), c = lo + w;
    long double tk[K] = {};
    double td[K] = {};  // the terms from 33^-2 on: double is enough
    for (int i = 0; i < n_r; ++i) {
      const long double g = 1.0L / ((long double)t.data[n_r + i] + c), f = -w * g;
      const long double v = (long double)t.data[i] * g, v1 = v * f;
      tk[0] += v;
      tk[1] += v1;
      const double fd = (double)f;
      double vd = (double)v1 * fd;
      for (int k = 2; k < K; ++k, vd *= fd) td[k] += vd;
    }
    for (int k = 2; k < K; ++k) tk[k] = td[k];
    long double wi = 1.0L;
    for (int i = 0; i < n; ++i, wi /= w) {
      long double v = 0.0L;
      for (int k = 0; k < K; ++k) v += econ[i * K + k] * tk[k];
      out[(size_t)p * n + i] = (double)(v * wi);
    }
  }
  double h_max = 0.0;
  for (int i = 0; i < n_r; ++i) h_max = std::fmax(h_max, t.data[n_r + i]);
  if (h_max <= std::ldexp(1.0, kFvTailH))
    for (int m = 0; m < kFvTail; ++m) {
      long double v = 0.0L;
      for (int i = 0; i < n_r; ++i)
        v += (long double)t.data[i] * powl((long double)t.data[n_r + i], m);
      out[(size_t)kPanels * n + m] = (double)v;
    }
  return out;
}

// Angular data of the vertex diagram: [x_j | sqrt(1 - x_j^2) | cos phi_l |
// nu_l], x_j the polar Gauss-Legendre nodes (as in build_quad_table),
// phi_l the Gauss-Legendre nodes on [0, pi] and nu_l = (pi/2) w_l sin^{d-3}(phi_l).
std::vector<double> build_vertex_table(int d, int n_a, int n_phi) {
  std::vector<double> xa(n_a), wa(n_a), xp(n_phi), wp(n_phi);
  gauss_legendre_gw(n_a, xa.data(), wa.data());
  gauss_legendre_gw(n_phi, xp.data(), wp.data());
  std::vector<double> t(2 * n_a + 2 * n_phi);
  for (int j = 0; j < n_a; ++j) {
    t[j] = xa[j];
    t[n_a + j] = std::sqrt((1.0 - xa[j]) * (1.0 + xa[j]));
  }
  for (int l = 0; l < n_phi; ++l) {
    const double f = 0.5 * M_PI * (1.0 + xp[l]);
    t[2 * n_a + l] = std::cos(f);
    t[2 * n_a + n_phi + l] = 0.5 * M_PI * wp[l] * std::pow(std::sin(f), d - 3);
  }
  return t;
}

// Chebyshev nodes of a mass panel in u = ln(x/4), |u| <= ln 4: x_n rounded to
// double, u_n = ln(x_n/4) of the rounded node in two doubles, and the
// barycentric weights of exactly these u_n (up to a common factor), in two
// doubles.
std::vector<double> build_mass_nodes() {
  const int n = kMassNodes;
  std::vector<double> t(5 * n);
  std::vector<long double> u(n);
  const long double pi = 3.14159265358979323846264338327950288L, half = logl(4.0L);
  for (int i = 0; i < n; ++i) {
    const double x = (double)(4.0L * expl(half * cosl(pi * (2 * i + 1) / (2.0L * n))));
    u[i] = logl((long double)x / 4.0L);
    t[i] = x;
    t[n + i] = (double)u[i];
    t[2 * n + i] = (double)(u[i] - (long double)t[n + i]);
  }
  for (int i = 0; i < n; ++i) {
    long double w = 1.0L;
    for (int m = 0; m < n; ++m)
      if (m != i) w *= 0.5L * half / (u[i] - u[m]);  // capacity of the interval: w stays O(1)
    t[3 * n + i] = (double)w;
    t[4 * n + i] = (double)(w - (long double)t[3 * n + i]);
  }
  return t;
}

// Coefficients of h(y) per panel: Chebyshev interpolation in long double
// (degree 9; 8 for h/y in the first panel, so that h keeps its relative
// accuracy there), converted to powers of y - c.  The nearest poles of h lie
// at +-2 pi i, so the truncation is below 2e-18 of h in every panel.
std::vector<double> build_regulator_table() {
  const long double pi = 3.14159265358979323846264338327950288L;
  auto h_of = [](long double y) -> long double {
    if (y < 0.5L) {  // Bernoulli series, |term ratio| < 0.0064
      static const long double b[8] = {1.0L / 12, -1.0L / 720, 1.0L / 30240, -1.0L / 1209600,
                                       1.0L / 47900160, -691.0L / 1307674368000.0L,
                                       1.0L / 74724249600.0L, -3617.0L / 10670622842880000.0L};
      const long double z = y * y;
      long double t = 0.0L;
      for (int n = 7; n >= 0; --n) t = t * z + b[n];
      return 0.5L * y + z * t;
    }
    const long double w = -expm1l(-y);
    return (y - w) / w;
  };
  std::vector<double> t((size_t)kRegPanels * kRegCoef, 0.0);
  for (int k = 0; k < kRegPanels - 1; ++k) {
    long double lo = 0.0L, hi = 0.3125L;
    if (k > 0) {
      const int e = (k + 1) / 8, s = (k + 1) % 8;
      lo = ldexpl(8.0L + s, e - 5);
      hi = ldexpl(9.0L + s, e - 5);
    }
    const int n = k ? kRegCoef : kRegCoef - 1;  // coefficients of h, or of h/y
    const long double c = 0.5L * (lo + hi), w = 0.5L * (hi - lo);
    // Chebyshev coefficients, then powers of v = (y - c)/w
    std::vector<long double> a(n, 0.0L), f(n);
    for (int i = 0; i < n; ++i) {
      const long double y = c + w * cosl(pi * (2 * i + 1) / (2.0L * n));
      f[i] = k ? h_of(y) : h_of(y) / y;
    }
    for (int j = 0; j < n; ++j) {
      for (int i = 0; i < n; ++i) a[j] += f[i] * cosl(pi * j * (2 * i + 1) / (2.0L * n));
      a[j] *= (j ? 2.0L : 1.0L) / n;
    }
    std::vector<long double> p(n, 0.0L), t0(n, 0.0L), t1(n, 0.0L);
    t0[0] = 1.0L;
    if (n > 1) t1[1] = 1.0L;
    for (int j = 0; j < n; ++j) {
      const std::vector<long double> &tj = j == 0 ? t0 : t1;
      for (int i = 0; i < n; ++i) p[i] += a[j] * tj[i];
      if (j >= 1) {  // T_{j+1} = 2 v T_j - T_{j-1}
        std::vector<long double> t2(n, 0.0L);
        for (int i = 0; i < n; ++i) t2[i] = (i ? 2.0L * t1[i - 1] : 0.0L) - t0[i];
        t0 = t1;
        t1 = t2;
      }
    }
    double *dst = t.data() + (size_t)k * kRegCoef;
    if (k) {
      long double s = 1.0L;
      for (int i = 0; i < n; ++i, s /= w) dst[i] = (double)(p[i] * s);
    } else {
      // r(v) = h/y with v = (y - c)/w, in powers of y; h = y r
      std::vector<long double> q(n, 0.0L);
      for (int i = n - 1; i >= 0; --i) {  // q <- q (y - c)/w + p_i
        std::vector<long double> z(n, 0.0L);
        for (int l = 0; l < n; ++l) z[l] = ((l ? q[l - 1] : 0.0L) - c * q[l]) / w;
        z[0] += p[i];
        q = z;
      }
      dst[0] = 0.0;
      for (int i = 0; i < n; ++i) dst[i + 1] = (double)q[i];
    }
  }
  double *last = t.data() + (size_t)(kRegPanels - 1) * kRegCoef;
  last[0] = -1.0;
  last[1] = 1.0;
  return t;
}

void lane_split(int n_r, int n_a, int *R, int *J, int *T, int *U) {
  int r = 1;
  while (r * 2 <= n_r && r * 2 <= kWave) r *= 2;
  *R = r;
  *J = kWave / r;
  *T = (n_r + r - 1) / r;
  *U = (n_a + *J - 1) / *J;
}

}  // namespace frg

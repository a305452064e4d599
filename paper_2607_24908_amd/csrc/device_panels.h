// Radial sums of the local-potential flows on gfx950 from polynomial panels:
//   s1(x) = sum_i chat_i/(hhat_i + x),  s2(x) = sum_i chat_i/(hhat_i + x)^2
// at x = (m^2 + k^2)/k^2 for 2^kPanelLo <= x < 2^kPanelHi (build_fv_panels; the
// table, or a part of it, in LDS or global memory): s1 and its derivative by one Horner pass over 11
// coefficients, within 2.2e-16 and 3.3e-16.  20 FMAs; the 64 nodes of the usual
// table take 64 reciprocals term by term, or 232 FMAs and 8 reciprocals as
// rational groups.
#pragma once

#include "frg_internal.h"

#pragma clang fp contract(off)

namespace frg {
namespace dev {

// Panel of x, counted from that at 2^LO; as an unsigned number below the number of
// panels exactly for x in their range (not for x <= 0, infinities and NaN).
template <int LO>
__device__ __forceinline__ int fv_panel(double x) {
  static_assert(kFvPerOctave == 16, "four mantissa bits select the panel");
  const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32);
  int p = (int)(hi >> 16) - ((1023 + LO) << 4);
  asm("" : "+v"(p));  // the address is p times the panel's size, not a folded base below zero
  return p;
}
// s1[m], s2[m] at x[m] in panel p[m]; s2[0] only for FIRST.  The loads of all
// masses first (those of the last kFvLate coefficients after the first steps, in
// the registers these free), then their Horner chains in step (the compiler's own
// order runs the masses one after the other, each waiting for its loads and for
// itself).
constexpr int kFvLate = 3;
template <int M, bool FIRST>
__device__ __forceinline__ void fv_poly(const double *poly, const double *x, const int *p,
                                        double *s1, double *s2) {
  double q[M][kFvPoly], z[M], P[M], D[M];
  const double *qp[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, x[m]) >> 32);
    const double c = __builtin_bit_cast(
        double, (unsigned long long)((hi & 0xffff0000u) | 0x8000u) << 32);  // its middle
    z[m] = x[m] - c;
    qp[m] = poly + p[m] * kFvPoly;
  }
#pragma unroll
  for (int k = kFvPoly - 1; k >= kFvLate; --k)
#pragma unroll
    for (int m = 0; m < M; ++m) q[m][k] = qp[m][k];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int m = 0; m < M; ++m) {
    P[m] = q[m][kFvPoly - 1];
    D[m] = P[m];
    P[m] = __builtin_fma(P[m], z[m], q[m][kFvPoly - 2]);
  }
#pragma unroll
  for (int k = kFvPoly - 3; k >= 0; --k) {
    if (k == kFvPoly - 5) {
#pragma unroll
      for (int l = kFvLate - 1; l >= 0; --l)
#pragma unroll
        for (int m = 0; m < M; ++m) q[m][l] = qp[m][l];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if (FIRST || m > 0) D[m] = __builtin_fma(D[m], z[m], P[m]);
      P[m] = __builtin_fma(P[m], z[m], q[m][k]);
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      asm volatile("" : "+v"(P[m]));
      if (FIRST || m > 0) asm volatile("" : "+v"(D[m]));
    }
  }
#pragma unroll
  for (int m = 0; m < M; ++m) {
    s1[m] = P[m];
    s2[m] = FIRST || m > 0 ? -D[m] : 0.0;
  }
}

// Whether every x is in a panel of the whole table or, finite, above them all where
// its moments hold; p: their panels.
template <int M>
__device__ __forceinline__ bool fv_covered(const double *table, const double *x, int *p) {
  bool all = table != nullptr;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    p[m] = fv_panel<kPanelLo>(x[m]);
    all &= (unsigned)p[m] < (unsigned)kPanels ||
           (x[m] >= __builtin_ldexp(1.0, kPanelHi) && x[m] < __builtin_inf());
  }
  return all && table[kPanels * kFvPoly] > 0.0;
}
// s1[m], s2[m] at masses that fv_covered accepts: a panel's by fv_poly, the others
// from four moments C_m, s1 = z (C_0 - z (C_1 - z (C_2 - z C_3))), z = 1/x, and s2 =
// -ds1/dx; the terms left out are below 5 (2^(kFvTailH - kPanelHi))^4 = 3e-19.
template <int M, bool FIRST>
__device__ __forceinline__ void fv_table_sums(const double *table, const double *x, const int *p,
                                              double *s1, double *s2) {
  double xc[M];
  int pc[M];
  bool some = false;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const bool in = (unsigned)p[m] < (unsigned)kPanels;
    some |= in;
    xc[m] = in ? x[m] : 1.0;
    pc[m] = in ? p[m] : -kPanelLo * kFvPerOctave;
  }
  if (some) fv_poly<M, FIRST>(table, xc, pc, s1, s2);
  using Const = const __attribute__((address_space(4))) double *;
  const Const C = (Const)(table + kPanels * kFvPoly);
#pragma unroll
  for (int m = 0; m < M; ++m) {
    if ((unsigned)p[m] < (unsigned)kPanels) continue;
    const double z = 1.0 / x[m];
    s1[m] = z * __builtin_fma(-z, __builtin_fma(-z, __builtin_fma(-z, C[3], C[2]), C[1]), C[0]);
    s2[m] = (z * z) * __builtin_fma(-z, __builtin_fma(-z, __builtin_fma(-z, 4.0 * C[3], 3.0 * C[2]),
                                                      2.0 * C[1]), C[0]);
  }
}

}  // namespace dev
}  // namespace frg

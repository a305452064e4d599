// Finite-volume LPA on gfx950: the semi-discrete central scheme of Kurganov
// and Tadmor for d_t u = d_sigma Q, Q = 1/2 F_1(d_sigma u) + (N-1)/2 F_1(u/sigma),
// u = dU/dsigma, with the local Lax-Friedrichs flux on the Goldstone part and
// minmod-limited piecewise-linear states, for n_rows flows at once; the
// three-stage strong-stability-preserving Runge-Kutta stages on the device.
//
// Cells i = 0..n-1 of width ds; interface j = 0..n at sigma_j = j ds between
// cells j-1 and j; ghost cells u_{-1} = -u_0, u_{-2} = -u_1 (u odd in sigma),
// u_n = 2u_{n-1} - u_{n-2}, u_{n+1} = 2u_n - u_{n-1}.  Interface 0 carries the
// flux N/2 F_1(2u_0/ds) (at sigma = 0 the Goldstone mass u/sigma equals
// d_sigma u); interface j >= 1 carries
//   1/2 F_1((u_j - u_{j-1})/ds) + 1/2 (f(u-) + f(u+)) - 1/2 a (u+ - u-),
//   f(u) = (N-1)/2 F_1(u/sigma_j), a = max |f'(u-)|, |f'(u+)|,
//   f'(u) = -(N-1)/2 F_2(u/sigma_j)/sigma_j,
// with u- = u_{j-1} + s_{j-1}/2, u+ = u_j - s_j/2, s_i = minmod(u_i - u_{i-1},
// u_{i+1} - u_i).  F_n(m^2) = C_d k^(d+2-2n) sum_i chat_i/(hhat_i + delta/k^2)^n,
// delta = m^2 + k^2 > 0 (else the flow has left the domain).
#include <hip/hip_runtime.h>

#include <cmath>

#include "frg_internal.h"

#pragma clang fp contract(off)

#include "device_fp64.h"
#include "device_panels.h"

namespace frg {

namespace {

using namespace dev;

__device__ __forceinline__ double minmod(double a, double b) {
  if (a * b <= 0.0) return 0.0;
  return fabs(a) < fabs(b) ? a : b;
}

// alive = 1, t_reached = t_end, domain flag cleared.
__global__ __launch_bounds__(256) void fv_init_kernel(FvArgs a, double t_end) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e == 0) *a.flag = 0;
  if (e < a.n_rows) {
    a.alive[e] = 1;
    a.t_reached[e] = t_end;
  }
}

// Scales of the stage at RG time t with k = lambda e^t: k^2, 1/k^2 and the
// factors of the radial sums in the flux (integer powers by products).  Every
// kernel forms them the same way.
struct FvScale {
  double k2, inv_k2;
  double c1, c2;  // C_d k^d / 2, C_d k^(d-2) / 2
  double g1, g2;  // (N - 1)/2 times them
  double n1, n2;  // N times them
};
__device__ __forceinline__ FvScale fv_scale(const FvArgs &a, double t) {
  const double k = a.lambda * exp(t);
  FvScale sc;
  sc.k2 = k * k;
  sc.inv_k2 = 1.0 / sc.k2;
  double p = 1.0;
  for (int i = 0; i < a.d - 2; ++i) p *= k;
  sc.c2 = 0.5 * a.Cd * p;
  sc.c1 = 0.5 * a.Cd * (p * sc.k2);
  const double g = 0.5 * (double)(a.N - 1);
  sc.g1 = g * sc.c1;
  sc.g2 = g * sc.c2;
  sc.n1 = (double)a.N * sc.c1;
  sc.n2 = (double)a.N * sc.c2;
  return sc;
}

// Ghost cells of one flow behind its last two cells f2, f1.
__device__ __forceinline__ double fv_ghost(double f2, double f1) { return 2.0 * f1 - f2; }

// Cells of the stencil of interface j: u_{j-2}, u_{j-1}, u_j, u_{j+1}.
struct FvCells {
  double LL, L, R, RR;
};
// ... from the cells u[0..n), n >= 2, without ghosts: loaded at clamped indices
// (issued together), the ghost rules applied afterwards by selects.
__device__ __forceinline__ FvCells fv_cells(const double *u, int n, int j) {
  const int nm1 = n - 1;
  auto cl = [&](int i) { return i < 0 ? 0 : (i > nm1 ? nm1 : i); };
  FvCells c{u[cl(j - 2)], u[cl(j - 1)], u[cl(j)], u[cl(j + 1)]};
  const double f1 = j == n ? c.L : c.R, f2 = j == n ? c.LL : c.L;  // u_{n-1}, u_{n-2}
  const double gn = fv_ghost(f2, f1);
  const double gn1 = fv_ghost(f1, gn);
  if (j < 2) c.LL = j == 1 ? -c.L : -c.RR;
  if (j < 1) c.L = -c.R;
  if (j == nm1) c.RR = gn;
  if (j == n) {
    c.R = gn;
    c.RR = gn1;
  }
  return c;
}

// s1 and s2 at M masses without the panels (device_panels.h): for x in [kFvXMin,
// kFvXMax] the coefficient groups, N/P and M/P^2 by Horner with one reciprocal per
// group of eight nodes (the powers of x and the products stay inside the FP64 range
// there); beyond those term by term.  Every term and coefficient is positive and x >
// 0, so neither form cancels.  The masses' chains run in step, coefficients in scalar
// registers (loaded there through the constant address space; the compiler's own FMA
// copies the addend into vector registers first, two moves per coefficient).
constexpr double kFvXMin = 1e-20, kFvXMax = 1e20;
using FvConst = const __attribute__((address_space(4))) double *;

__device__ __forceinline__ double fma_su(double a, double b, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
  return r;
}
template <int M>
__device__ __forceinline__ void fv_radial_far(const double *table, int n_r, const double *x,
                                              double *s1, double *s2) {
  const FvConst tab = (FvConst)table, cf = tab + 2 * n_r;
  bool in[M], some = false, all = true;
  double xc[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    in[m] = x[m] >= kFvXMin && x[m] <= kFvXMax;
    some |= in[m];
    all &= in[m];
    xc[m] = in[m] ? x[m] : 1.0;
    s1[m] = s2[m] = 0.0;
  }
  if (some) {
    const int ng = (n_r + kFvGroup - 1) / kFvGroup;
#pragma unroll 1
    for (int g = 0; g < ng; ++g) {
      const FvConst c = cf + kFvCoef * g;
      double P[M], N[M], Q[M];
#pragma unroll
      for (int m = 0; m < M; ++m) {
        P[m] = xc[m] + c[7];
        N[m] = c[15];
        Q[m] = c[30];
      }
#pragma unroll
      for (int k = 6; k >= 0; --k)
#pragma unroll
        for (int m = 0; m < M; ++m) {
          P[m] = fma_su(P[m], xc[m], c[k]);
          N[m] = fma_su(N[m], xc[m], c[k + 8]);
          Q[m] = fma_su(Q[m], xc[m], c[k + 23]);
        }
#pragma unroll
      for (int k = 22; k >= 16; --k)
#pragma unroll
        for (int m = 0; m < M; ++m) Q[m] = fma_su(Q[m], xc[m], c[k]);
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const double r = rcp64(P[m]);
        s1[m] = __builtin_fma(N[m], r, s1[m]);
        s2[m] = __builtin_fma(Q[m] * r, r, s2[m]);
      }
    }
  }
  if (!all) {
#pragma unroll
    for (int m = 0; m < M; ++m)
      if (!in[m]) s1[m] = s2[m] = 0.0;
#pragma unroll 1
    for (int i = 0; i < n_r; ++i)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const double G = rcp64(tab[n_r + i] + x[m]);
        const double cg = tab[i] * G;
        if (!in[m]) {
          s1[m] += cg;
          s2[m] = __builtin_fma(cg, G, s2[m]);
        }
      }
  }
}

// Flux Q and (LAM) the local bound lam of the step estimate at interface j from
// the cells c of its stencil; isj = 1/sigma_j, 0 for j = 0 (zero), where d_sigma u
// = (u_0 - u_{-1})/ds = 2 u_0/ds is the only mass that enters.  The masses are
// d_sigma u and, for N > 1 (GOLD), the limited states u-/sigma_j and u+/sigma_j;
// bad: one of them has left the domain.  All masses of the interface in one lane,
// so that their panel loads and Horner chains fill each other's latency.  NEAR: the
// panels 2^kFvLo .. 2^kFvHi, at `near`, alone; a mass outside them counts as bad and
// leaves the sums of some panel.  Else the whole table, or the sums without it where a
// mass is in no panel (so is one outside the domain) or there is no table.
struct FvOut {
  double Q, lam;
  bool bad;
};
template <bool GOLD, bool LAM, bool NEAR>
__device__ __forceinline__ FvOut fv_iface(const FvArgs &a, const FvScale &sc, const double *near,
                                          const FvCells &c, double isj, bool zero) {
  constexpr int M = GOLD ? 3 : 1;
  const double ids = a.inv_ds;
  double jump = 0.0, delta[M], x[M], s1[M], s2[M];
  int p[M];
  const double b = c.R - c.L;
  delta[0] = __builtin_fma(b, ids, sc.k2);
  if constexpr (GOLD) {
    const double um = __builtin_fma(0.5, minmod(c.L - c.LL, b), c.L);
    const double up = __builtin_fma(-0.5, minmod(b, c.RR - c.R), c.R);
    jump = up - um;
    delta[1] = __builtin_fma(um, isj, sc.k2);
    delta[2] = __builtin_fma(up, isj, sc.k2);
  }
  FvOut o;
  o.bad = false;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    x[m] = delta[m] * sc.inv_k2;
    if constexpr (NEAR) {
      p[m] = fv_panel<kFvLo>(x[m]);
      o.bad |= (unsigned)p[m] >= (unsigned)kFvPanels;
      p[m] = (int)min((unsigned)p[m], (unsigned)kFvPanels - 1u);
    }
  }
  if constexpr (NEAR) {
    fv_poly<M, LAM>(near, x, p, s1, s2);
  } else if (fv_covered<M>(a.poly, x, p)) {
    fv_table_sums<M, LAM>(a.poly, x, p, s1, s2);
  } else {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const bool bad = !(delta[m] > 0.0);
      o.bad |= bad;
      x[m] = bad ? 1.0 : x[m];
    }
    fv_radial_far<M>(a.tab, a.n_r, x, s1, s2);
  }
  const double q0 = (zero ? sc.n1 : sc.c1) * s1[0];
  o.Q = q0;
  o.lam = LAM ? 2.0 * ((zero ? sc.n2 : sc.c2) * s2[0]) * (ids * ids) : 0.0;
  if constexpr (GOLD) {
    const double ah = sc.g2 * fmax(s2[1], s2[2]) * isj;  // half the larger |f'|; 0 at j = 0
    const double Q = __builtin_fma(-ah, jump, __builtin_fma(sc.g1, s1[1] + s1[2], q0));
    o.Q = zero ? q0 : Q;
    if (LAM) o.lam += 2.0 * ah * ids;
  }
  return o;
}

// 1/sigma_j; 0 for j = 0.
__device__ __forceinline__ double fv_isj(const FvArgs &a, int j) {
  return j > 0 ? a.inv_ds / (double)j : 0.0;
}

// SSP-RK3 stage s (0..2) of one cell: y0 at the start of the step, y the state
// this stage starts from (y0 itself in stage 0), e = y + h L with dq = L ds and
// hids = h/ds; y0 + w (e - y0), w = 1, 1/4, 2/3.  In this form a rounded weight
// scales a small change only: y0/3 + (2/3) e multiplies the state by 1 - 3.7e-17 in
// every step, which over 2000 steps of a flow of 256 cells made 7.1e-14 of the
// solution (2.7e-15 in this form, both against 80-bit arithmetic).
__device__ __forceinline__ double fv_update(int s, double dq, double hids, double y0, double y) {
  const double e = __builtin_fma(hids, dq, y);
  return s == 0 ? e : __builtin_fma(s == 1 ? 0.25 : 2.0 / 3.0, e - y0, y0);
}

// Grid (interface blocks, flows) at the stage time a.t.
__global__ __launch_bounds__(256) void fv_flux_kernel(FvArgs a) {
  const int64_t r = blockIdx.y;
  const int64_t nq = a.n + 1;
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= nq) return;
  double *Q = a.Q + r * nq, *lam = a.lam + r * nq;
  if (!a.alive[r]) {  // workgroup-uniform
    Q[j] = lam[j] = 0.0;
    return;
  }
  const double *u = (a.first ? a.y0 : a.ys) + r * a.n;
  const FvScale sc = fv_scale(a, a.t);
  const FvCells c = fv_cells(u, (int)a.n, (int)j);
  const double isj = fv_isj(a, (int)j);
  const FvOut o = a.N > 1 ? fv_iface<true, true, false>(a, sc, nullptr, c, isj, j == 0)
                          : fv_iface<false, true, false>(a, sc, nullptr, c, isj, j == 0);
  if (o.bad) {
    // the flow ends at the start of this step with its state kept
    a.alive[r] = 0;
    a.t_reached[r] = a.t_n;
    *a.flag = 1;
  }
  Q[j] = o.bad ? 0.0 : o.Q;
  lam[j] = o.bad ? 0.0 : o.lam;
}

// Grid (cell blocks, flows): d_t u_i = (Q_{i+1} - Q_i)/ds and the stage.
__global__ __launch_bounds__(256) void fv_stage_kernel(FvArgs a) {
  const int64_t r = blockIdx.y;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const int64_t e = r * a.n + i;
  if (!a.alive[r]) {
    if (a.stage == 3) a.dudt[e] = __builtin_nan("");
    return;
  }
  const double *Q = a.Q + r * (a.n + 1);
  const double dq = Q[i + 1] - Q[i];
  if (a.stage == 3) {
    a.dudt[e] = dq * a.inv_ds;
  } else {
    const double y0 = a.y0[e], y = a.stage == 0 ? y0 : a.ys[e];
    (a.stage == 2 ? a.y0 : a.ys)[e] = fv_update(a.stage, dq, a.h * a.inv_ds, y0, y);
  }
}

// Steps of one flow by its workgroup, everything in LDS: three state buffers with
// their ghost cells, 1/sigma_j, the polynomial panels and the scales of the next
// kFvScaleSteps steps (formed by all threads at once).  A
// wave takes 64 consecutive interfaces and with them the 63 cells between: each
// lane forms its interface's flux (fv_iface), takes its left neighbour's by a
// lane permutation and updates the cell between the two; the next wave starts
// at this one's last interface, and the last wave ends with interface n, so that
// one wave holds the cells of the ghosts.  One barrier per stage.  The
// per-interface and per-cell arithmetic is that of the flux and stage kernels
// (same bits); no launch per stage.  A step goes from buffer Y over A and B to A,
// so a step that fv_iface finds bad leaves Y, the state of its start.
//
// Bound by the latency of this chain (cells, states, panels, Horner, flux) on
// the one CU of a flow, one wave on most SIMDs: 0.57 us per stage for one wave
// (63 cells), 0.68 for the four of 200 cells and 0.85 for the five of 256 cells, whose panel
// coefficients (84 KB per stage) also share the CU's LDS port.  128 flows of 256
// cells, 64 nodes, N = 4, 2000 steps: 5.2 ms.  With the radial sums as rational
// groups, one lane per mass, four barriers per stage and the scales formed by
// every thread it took 25.9 ms; this kernel's sums with a quad of lanes per
// interface (each lane one mass, two barriers) 8.6 ms, bound by instruction
// issue.  At most 128 VGPRs, so that two workgroups of five waves fit a CU
// (512 flows: 1.20 us per stage; 1.83 at 151 VGPRs with an earlier loop of 1.31).
//
// From the first step with a mass outside the panels in LDS a flow goes on in a loop
// of its own, with the whole table and the sums without it; in one loop they took
// registers of the panels' (0.94 us per stage, 0.85 so). 128 flows of 256 cells there:
// 1.6 us per stage with the masses in the other panels, 1.5 above them all, whatever
// the order of the rule (14 us at 64 nodes and 211 at 1024 by rational groups, one
// mass after the other); 4.8, 16 and 55 us at 64, 256 and 1024 nodes in a context
// that cannot spare the table.
constexpr int kFvScaleSteps = 32;
constexpr int kFvWaveCells = kWave - 1;
constexpr int kFvMaxWaves = 8;

struct FvLds {
  const double *poly;
  double *Y, *A, *B, *isj;
  FvScale *scales;  // [kFvScaleSteps][3]
  int *bad;         // 0 between steps
};
// Steps st .. n_st - 1 of the launch's, up to one that is bad: the step after the
// last good one, whose state is in l.Y.
template <bool GOLD, bool NEAR>
__device__ __forceinline__ int64_t fv_steps(const FvArgs &a, FvLds &l, int64_t s0, int64_t st,
                                            int64_t n_st) {
  const int n = (int)a.n;
  const int tid = threadIdx.x, bs = blockDim.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const double cs[3] = {0.0, 1.0, 0.5};
  const double hids = a.h * a.inv_ds;
  for (; st < n_st; ++st) {
    const int sl = (int)(st % kFvScaleSteps);
    if (sl == 0) {
      for (int k = tid; k < 3 * kFvScaleSteps; k += bs) {
        const double t = (double)(s0 + st + k / 3) * a.h;
        l.scales[k] = fv_scale(a, t + cs[k % 3] * a.h);
      }
      __syncthreads();
    }
    bool bad = false;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const FvScale sc = l.scales[3 * sl + s];
      const double *u = s == 0 ? l.Y : (s == 1 ? l.A : l.B);
      double *dst = s == 1 ? l.B : l.A;
      for (int je = n - wave * kFvWaveCells; je > 0; je -= bs / kWave * kFvWaveCells) {
        const int jl = je - kFvWaveCells + lane;  // je is the wave's last interface
        const int j = max(jl, 0);
        const FvCells c{u[j - 2], u[j - 1], u[j], u[j + 1]};
        const double y0 = s == 0 ? c.L : l.Y[j - 1];
        const FvOut o = fv_iface<GOLD, false, NEAR>(a, sc, l.poly, c, l.isj[j], j == 0);
        bad |= o.bad;
        const double left = dpp_f64<0x138>(o.Q);  // wave_shr 1: the flux of interface j - 1
        const double v = fv_update(s, o.Q - left, hids, y0, c.L);
        const double vl = dpp_f64<0x138>(v);
        if (lane > 0 && jl > 0) {
          dst[j - 1] = v;
          if (j == 1) dst[-1] = -v;
          if (j == n) {
            const double gn = fv_ghost(vl, v);
            dst[n] = gn;
            dst[n + 1] = fv_ghost(v, gn);
          }
        }
      }
      if (s == 2 && bad) *l.bad = 1;
      __syncthreads();
    }
    if (*l.bad) break;  // workgroup-uniform
    double *t = l.Y;
    l.Y = l.A;
    l.A = t;
  }
  return st;
}

// Steps [s0, s0 + n_st) of one flow per workgroup.
template <bool GOLD>
__global__ __launch_bounds__(kFvMaxWaves * kWave, 4) void fv_solve_kernel(FvArgs a, int64_t s0,
                                                                         int64_t n_st) {
  extern __shared__ double lds[];
  const int64_t r = blockIdx.x;
  if (!a.alive[r]) return;  // workgroup-uniform
  const int n = (int)a.n;
  const int tid = threadIdx.x, bs = blockDim.x;
  const int n_poly = a.poly ? kFvPanels * kFvPoly : 0;
  double *poly = lds;
  FvLds l;
  l.poly = poly;
  l.Y = poly + n_poly + 2;  // cells -2 .. n + 1 each
  l.A = l.Y + n + 4;
  l.B = l.A + n + 4;
  l.isj = l.B + n + 2;  // [n + 1]
  l.scales = reinterpret_cast<FvScale *>(l.isj + n + 1);
  l.bad = reinterpret_cast<int *>(l.scales + 3 * kFvScaleSteps);
  const double *y = a.y0 + r * n;
  for (int i = tid; i < n_poly; i += bs) poly[i] = a.poly[kFvFirst * kFvPoly + i];
  for (int i = tid; i < n; i += bs) l.Y[i] = y[i];
  for (int j = tid; j <= n; j += bs) l.isj[j] = fv_isj(a, j);
  if (tid == 0) {
    *l.bad = 0;
    l.Y[-2] = l.A[-2] = l.B[-2] = 0.0;  // read by interface 0, in which it does not enter
    l.Y[-1] = -y[0];
    l.Y[n] = fv_ghost(y[n - 2], y[n - 1]);
    l.Y[n + 1] = fv_ghost(y[n - 1], l.Y[n]);
  }
  int64_t st = 0;
  if (a.poly) st = fv_steps<GOLD, true>(a, l, s0, st, n_st);
  if (st < n_st) {
    __syncthreads();  // the flag is read
    if (tid == 0) *l.bad = 0;
    st = fv_steps<GOLD, false>(a, l, s0, st, n_st);
    if (st < n_st && tid == 0) {
      a.alive[r] = 0;
      a.t_reached[r] = (double)(s0 + st) * a.h;
      *a.flag = 1;
    }
  }
  for (int i = tid; i < n; i += bs) a.y0[r * n + i] = l.Y[i];
}

// One workgroup per flow: step estimate 1 / max_j lam_j.
__global__ __launch_bounds__(256) void fv_dt_kernel(FvArgs a) {
  __shared__ double red[256];
  const int64_t r = blockIdx.x;
  double m = 0.0;
  for (int64_t j = threadIdx.x; j <= a.n; j += blockDim.x) m = fmax(m, a.lam[r * (a.n + 1) + j]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) a.dt[r] = a.alive[r] ? 1.0 / red[0] : __builtin_nan("");
}

}  // namespace

int launch_fv_init(const FvArgs &a, double t_end, void *stream) {
  const int64_t n = a.n_rows > 1 ? a.n_rows : 1;
  hipLaunchKernelGGL(fv_init_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, a, t_end);
  return (int)hipGetLastError();
}

int launch_fv_flux(const FvArgs &a, void *stream) {
  if (a.n_rows <= 0) return 0;
  hipLaunchKernelGGL(fv_flux_kernel, dim3((unsigned)(a.n / 256 + 1), (unsigned)a.n_rows),
                     dim3(256), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

int launch_fv_stage(const FvArgs &a, void *stream) {
  if (a.n_rows <= 0) return 0;
  hipLaunchKernelGGL(fv_stage_kernel, dim3((unsigned)((a.n + 255) / 256), (unsigned)a.n_rows),
                     dim3(256), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

static int64_t fv_solve_lds_bytes(const FvArgs &a) {
  return (int64_t)sizeof(double) *
             ((a.poly ? kFvPanels * kFvPoly : 0) + 3 * (a.n + 4) + a.n + 1) +
         (int64_t)sizeof(FvScale) * 3 * kFvScaleSteps + 16;
}

// One workgroup per flow, or the launches of the flux and stage kernels. With panels
// the first wherever the LDS holds the flow. Without, the sums bound both forms: a
// coefficient group of a wave's masses takes a SIMD about 0.2 us, and the launches
// 8 us per stage beside them, over the whole chip (128 flows of 256 cells, 1024 nodes:
// 55 us per stage by launches, 68 in the workgroup; at 64 nodes 4.8 in the workgroup).
bool fv_solve_fused(const FvArgs &a, int n_cu) {
  if (fv_solve_lds_bytes(a) > kFvSolveLdsMax) return false;
  if (a.poly) return true;
  const int64_t waves = (a.n + kFvWaveCells - 1) / kFvWaveCells, simds = 4 * (int64_t)n_cu;
  const double sum = 0.2 * fv_groups(a.n_r);
  const int64_t mine = ((a.n_rows + n_cu - 1) / n_cu * waves + 3) / 4;
  const int64_t all = (a.n_rows * (a.n / kWave + 1) + simds - 1) / simds;
  return sum * (double)mine <= 8.0 + sum * (double)all;
}

int launch_fv_solve(const FvArgs &a, int64_t s0, int64_t n_st, void *stream) {
  if (a.n_rows <= 0 || n_st <= 0) return 0;
  if (fv_solve_lds_bytes(a) > kFvSolveLdsMax) return (int)hipErrorInvalidValue;
  static const bool once =
      ((void)hipFuncSetAttribute((const void *)&fv_solve_kernel<true>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, kFvSolveLdsMax),
       (void)hipFuncSetAttribute((const void *)&fv_solve_kernel<false>,
                                 hipFuncAttributeMaxDynamicSharedMemorySize, kFvSolveLdsMax),
       (void)hipGetLastError(), true);
  (void)once;
  const int waves = (int)((a.n + kFvWaveCells - 1) / kFvWaveCells);
  hipLaunchKernelGGL(a.N > 1 ? fv_solve_kernel<true> : fv_solve_kernel<false>,
                     dim3((unsigned)a.n_rows), dim3(kWave * (waves < kFvMaxWaves ? waves : kFvMaxWaves)),
                     (size_t)fv_solve_lds_bytes(a), (hipStream_t)stream, a, s0, n_st);
  return (int)hipGetLastError();
}

int launch_fv_dt(const FvArgs &a, void *stream) {
  if (a.n_rows <= 0) return 0;
  hipLaunchKernelGGL(fv_dt_kernel, dim3((unsigned)a.n_rows), dim3(256), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

}  // namespace frg

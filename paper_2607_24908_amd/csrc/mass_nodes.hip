// Mass nodes: tensor grids (momenta x masses) and vertex diagrams with many
// masses, evaluated at a few masses per panel and interpolated (gfx950).
//
// At fixed momenta a diagram is, as a function of delta = m^2 + k^2,
//   f(delta) = sum_k w_k / prod_{e <= E+1} (delta + H_ke),  w_k > 0, H >= 0
// (E + 1 = 3 factors for the two-point diagram, 4 for the vertex): a sum of
// thousands of poles on the negative axis.  In u = ln delta it is analytic in
// the strip |Im u| < pi, so on a panel delta in [c/4, 4c] (half-length ln 4 in
// u) the Chebyshev interpolant of g = f delta^pw (pw = 3/2, 2: the middle of
// the powers that f can follow) through N = 32 nodes has a relative error
// below 2.2e-19 (3 equal poles, the worst case found over their positions) and
// 2.2e-18 (4): ~(N/2)^2 rho^-N with rho = 4.74, the ellipse that touches
// Im u = pi.  Every f is a positive combination of such terms, so the bound
// holds for it too: the interpolant is the discrete sum to far below rounding.
// The panels are fixed (powers of 16 in x = sig delta, the units of the
// coefficient form), so a mass takes the same nodes in every call.
//
// Rounding.  sum_n |l_n g_n / g|^2 stays near one (at most 2.1^2 for three
// poles, reached only at a panel's end with every pole far to one side), so
// the interpolated values carry about the rounding error of the evaluated
// ones; the nodes are exact doubles, and u - u_n is formed as
// log1p((x - x_r)/x_r) + (u_r - u_n) with the node x_r nearest to x, which
// keeps it accurate to a few 1e-18 absolute.
//
// Two launches.  grid_nodes_kernel / vertex_nodes_kernel evaluate every
// momentum at the 32 nodes of each panel that holds a mass (the coefficient form
// on the matrix cores, device_grid.h), and at the masses that lie in no panel
// (outside the domain, or beyond the coefficient form) themselves; where the
// panels' nodes would take as many rounds of a workgroup's waves as the masses, every
// mass is evaluated itself.
// Their last workgroups form the Lagrange rows of the masses meanwhile.
// mass_interp_kernel forms values x Lagrange rows, also on the matrix cores.
//
// Measured (4096 momenta x 512 masses, 128 x 32 nodes, exponential regulator):
// 158 us against 695 us for the direct form; 256 vertex configurations x 512
// masses, 48 x 8 x 16 nodes: 35 against 73 us.  The node kernel (150 us of the
// 158) is bound by the FP64 pipes of the SIMDs, which matrix and vector
// instructions share: 44% of its cycles in matrix instructions (36 per tile, 16
// terms and 64 rows), 34% in vector instructions (regulator values, expansions,
// quotients), the rest at the barriers between the phases of a chunk.
//
// Errors against 64-bit sums, in brackets the direct form's: 4096 x 512 grid, norm
// of the error over that of the results 3.1e-16 (1.9e-16), root mean square of the
// relative errors 2.9e-16 (3.6e-16), largest 1.6e-15 (2.3e-15); vertex 3.3e-16
// (5.2e-16), 3.4e-16 (6.2e-16), 1.5e-15 (4.1e-15).  The grid's norm, of its largest
// results at the smallest masses, is what grew: there the interpolant is a sum of
// 32 products of both signs that exceed the result several times.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "frg_internal.h"

#pragma clang fp contract(off)

#include "device_fp64.h"
#include "device_grid.h"

namespace frg {

namespace {

using namespace dev;

constexpr int N = kMassNodes;
static_assert(N == 32, "one node per lane of a half-wave; 8 per lane group of 16 in the products");

// Panel of x: floor(log16 x) - kMassPanelLo/4 from the exponent bits, -1
// outside [2^kMassPanelLo, 2^kMassPanelHi) (then the mass is evaluated
// itself).  The range lies inside FoldRange of every group size.
__device__ __forceinline__ int panel_of(double x) {
  if (!(x > 0.0)) return -1;  // also NaN
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const int e = (int)(b >> 52) - 1023;
  if (e < kMassPanelLo || e >= kMassPanelHi) return -1;
  return (e - kMassPanelLo) >> 2;
}
// 2^-4p' x, p' = floor(log16 x): x scaled into [1, 16) (exact).
__device__ __forceinline__ double panel_unit(double x, int panel) {
  return __builtin_ldexp(x, -(kMassPanelLo + 4 * panel));
}

// Lagrange rows of kLagTile masses (tile `tile` of the masses): half-wave h,
// lane n the entry l_n of one mass, barycentric
//   l_n = t_n / sum t,  t_n = w_n/(u - u_n),  times (x_n/x)^pw,
// pw = (E + 1)/2, the middle of the powers 0..-(E + 1) that the diagram can
// follow.
// Zero rows for the masses outside every panel.
constexpr int kNodeWaves = 4;
constexpr int kLagTile = kNodeWaves * kWave / N;
template <int E>
__device__ __forceinline__ void lagrange_rows(const GridArgs &g, const MassPlan &m, int64_t tile) {
  const int lane = threadIdx.x & (kWave - 1), n = threadIdx.x & (N - 1);
  const double xn = m.nodes[n], uh = m.nodes[N + n], ul = m.nodes[2 * N + n], wn = m.nodes[3 * N + n],
               wl = m.nodes[4 * N + n];
  const int64_t b = tile * kLagTile + threadIdx.x / N;
  if (b >= g.n_m) return;  // half-wave-uniform, no barrier follows
  double l = 0.0;
  const double xs = g.sig * (g.m2[b] + g.k2);
  const int panel = panel_of(xs);
  if (panel >= 0) {  // half-wave-uniform
    const double x = panel_unit(xs, panel);
    // the node nearest to x (smallest |x - x_n|, lowest n on ties)
    double dist = fabs(x - xn);
    int near = n;
#pragma unroll
    for (int o = N / 2; o >= 1; o >>= 1) {
      const double od = __shfl_xor(dist, o, kWave);
      const int on = __shfl_xor(near, o, kWave);
      if (od < dist || (od == dist && on < near)) {
        dist = od;
        near = on;
      }
    }
    const int src = (lane & ~(N - 1)) + near;
    const double xr = __shfl(xn, src, kWave), urh = __shfl(uh, src, kWave),
                 url = __shfl(ul, src, kWave);
    const double v = log1p((x - xr) / xr);  // x - xr exact
    if (v == 0.0) {
      l = n == near ? 1.0 : 0.0;
    } else {
      // in two doubles (hi, lo) up to the rounding of l: an error of a row is
      // common to every momentum
      const double dh = urh - uh, db = dh - urh;  // u_r - u_n
      const double dl = ((urh - (dh - db)) - (uh + db)) + (url - ul);
      const double eh = v + dh, eb = eh - v;      // u - u_n
      const double el = ((v - (eh - eb)) + (dh - eb)) + dl;
      const double t = wn / eh;
      double S = t, lo = (__builtin_fma(-t, eh, wn) + (wl - t * el)) / eh;
      const double tl = lo;
#pragma unroll
      for (int o = N / 2; o >= 1; o >>= 1) {
        const double y = __shfl_xor(S, o, kWave), ylo = __shfl_xor(lo, o, kWave);
        const double z = S + y, bb = z - S;
        lo = (lo + ylo) + ((S - (z - bb)) + (y - bb));
        S = z;
      }
      const double l0 = t / S;
      const double l1 = (__builtin_fma(-l0, S, t) + (tl - l0 * lo)) / S;
      // (x_n/x)^pw: w + w1
      const double q = xn / x, ql = __builtin_fma(-q, x, xn) / x;
      const double r = E == 2 ? sqrt(q) : q;
      const double rl = E == 2 ? (__builtin_fma(-r, r, q) + ql) / (2.0 * r) : ql;
      const double w = q * r, w1 = __builtin_fma(q, r, -w) + (q * rl + ql * r);
      l = __builtin_fma(l0, w, l0 * w1 + l1 * w);
    }
  }
  m.lag[b * N + n] = l;
}

// Bit p: panel p holds a mass and is interpolated; bit 31: some mass is
// evaluated itself.  Interpolated while the nodes take fewer rounds (kNodeWaves tiles of
// 16) than the masses: 4096 momenta x 131 or 190 masses in three panels, 206 us, against
// 333 and 361 where half as many nodes as masses were asked for.  The same in every
// workgroup (all threads take part; `sh`:
// kNodeWaves words of LDS).
constexpr unsigned kSingles = 1u << 31;
__device__ __forceinline__ unsigned mass_panels(const GridArgs &g, unsigned *sh) {
  unsigned mask = 0;
  for (int b = threadIdx.x; b < (int)g.n_m; b += blockDim.x) {
    const int p = panel_of(g.sig * (g.m2[b] + g.k2));
    mask |= p >= 0 ? 1u << p : kSingles;
  }
#pragma unroll
  for (int o = kWave / 2; o >= 1; o >>= 1) mask |= __shfl_xor(mask, o, kWave);
  if ((threadIdx.x & (kWave - 1)) == 0) sh[threadIdx.x / kWave] = mask;
  __syncthreads();
  mask = 0;
  for (int w = 0; w < (int)(blockDim.x / kWave); ++w) mask |= sh[w];
  mask = __builtin_amdgcn_readfirstlane(mask);
  return mass_rounds(N * __builtin_popcount(mask & ~kSingles)) < mass_rounds((int)g.n_m) ? mask
                                                                                     : kSingles;
}

// Slot of mass x among the interpolated panels, or -1.
__device__ __forceinline__ int slot_of(double x, unsigned panels) {
  const int p = panel_of(x);
  if (p < 0 || !((panels >> p) & 1u)) return -1;
  return __builtin_popcount(panels & ((1u << p) - 1u));
}

// h(y) = y/(1 - e^-y) - 1 of the coefficient build from the table of
// build_regulator_table (ht, in LDS): ten coefficients in f = y - c, the panel
// and its centre c from the exponent and the top three mantissa bits of y; the
// first panel (y < 5/16) and the last (y >= 40: h = y - 1) have c = 0.  One path
// for every y: the series below y = 1 and the exponential above it, of which
// most waves need both, took 76 vector instructions per value against 32.
template <int REG>
__device__ __forceinline__ double h_build(double y, const double *ht) {
  const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, y) >> 32);
  int k = (int)(hi >> 17) - kRegBits;
  k = k < 0 ? 0 : (k > kRegPanels - 1 ? kRegPanels - 1 : k);
  const unsigned ch = (hi & 0xfffe0000u) | 0x00010000u;  // middle of the panel
  const bool mid = k > 0 && k < kRegPanels - 1;
  const double c = mid ? __builtin_bit_cast(double, (unsigned long long)ch << 32) : 0.0;
  const double f = y - c;
  const double2 *t = reinterpret_cast<const double2 *>(ht + k * kRegCoef);
  double h = t[4].y;
  h = __builtin_fma(h, f, t[4].x);
#pragma unroll
  for (int n = 3; n >= 0; --n) {
    h = __builtin_fma(h, f, t[n].y);
    h = __builtin_fma(h, f, t[n].x);
  }
  return h;
}

// sig Hk(s) of the coefficient build.
template <int REG>
__device__ __forceinline__ double hk_build(const GridArgs &g, double s, const double *ht) {
  if constexpr (REG == kExp)
    return (g.sig * g.k2) * h_build<REG>(s * g.inv_k2, ht);
  else
    return g.sig * fmax(s - g.k2, 0.0);
}

// The regulator table into LDS (exponential regulator only).
template <int REG>
__device__ __forceinline__ void stage_regulator(const MassPlan &m, double *ht) {
  if constexpr (REG == kExp)
    for (int i = threadIdx.x; i < kRegPanels * kRegCoef; i += blockDim.x) ht[i] = m.reg[i];
}

// Expand one group from its regulator values in `col` (row k at col[64 k],
// weights mu(k)) and up to three extra linear factors f of P; N is scaled by
// c.  The recurrences of grid_fill_fold.
template <int G, int E, class Mu>
__device__ __forceinline__ void expand_group(double *col, const double *f, double c, Mu mu) {
  double P[G + E + 1], Nc[G];
#pragma unroll
  for (int m = 0; m < G + E + 1; ++m) P[m] = 0.0;
#pragma unroll
  for (int m = 0; m < G; ++m) Nc[m] = 0.0;
  // the next term's reads are issued one term ahead
  double Hn = col[0], wn = mu(0);
#pragma unroll
  for (int k = 0; k < G; ++k) {
    const double H = Hn, w = wn;
    if (k + 1 < G) {
      Hn = col[(k + 1) * kWave];
      wn = mu(k + 1);
    }
    if (k == 0) {
      Nc[0] = w;
      P[1] = 1.0;
      P[0] = H;
    } else {
      // N <- N (x + H) + w P and P <- P (x + H), downwards in place
      Nc[k] = __builtin_fma(w, P[k], Nc[k - 1]);
      P[k + 1] = 1.0;
      P[k] = H + P[k - 1];
#pragma unroll
      for (int m = G - 1; m >= 1; --m)
        if (m < k) {
          Nc[m] = __builtin_fma(w, P[m], __builtin_fma(H, Nc[m], Nc[m - 1]));
          P[m] = __builtin_fma(H, P[m], P[m - 1]);
        }
      Nc[0] = __builtin_fma(w, P[0], H * Nc[0]);
      P[0] = H * P[0];
    }
    // keep the steps in order: left alone the compiler reads every term first
    // and then runs diagonally through the recurrence, 150 doubles live
#pragma unroll
    for (int m = 0; m <= k; ++m) asm volatile("" : "+v"(P[m]), "+v"(Nc[m]));
  }
#pragma unroll
  for (int m = 0; m < G; ++m) col[(G + E + m) * kWave] = c * Nc[m];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int deg = G + r;
    P[deg + 1] = 1.0;
#pragma unroll
    for (int m = G + E - 1; m >= 1; --m)
      if (m <= deg) P[m] = __builtin_fma(f[r], P[m], P[m - 1]);
    P[0] = f[r] * P[0];
#pragma unroll
    for (int m = 0; m < G + E; ++m) asm volatile("" : "+v"(P[m]));
  }
#pragma unroll
  for (int m = 0; m < G + E; ++m) col[m * kWave] = P[m];
}

// The listed masses at one momentum.  The workgroup (four waves) takes the
// table in chunks of kChunk coefficient groups of 64 lane rows: its waves form
// the chunk's regulator values in LDS (fill), two of them expand its groups
// (expand), then every wave evaluates its tiles of 16 masses on the matrix
// cores.  A chunk takes 35 KiB whatever the rule's size, so four workgroups
// share a CU (four waves per SIMD) and while one builds another evaluates.
// A mass sums its chunks in four sums by chunk mod 4, added in order at the end.
// With few momenta the sums are dealt to m.parts (2 or 4) workgroups per
// momentum and stored apart (planes of m.val, added by mass_interp_kernel in the
// same order): the same bits for any number of parts and any list.
// Stored values are in units of g.pref_c (a power of two times g.pref).
// lane_row(gg, l): what the terms of lane row l of group gg share;
// fill(row, k): the regulator value of its term k; expand(gg, col, l):
// expand_group with the group's factors and weights; single(delta): per-term
// lane partial of a mass outside the coefficient form.
// A chunk is built once for up to kMassRegTiles tiles, two per wave with their sums in
// registers (the nodes of four panels, or 128 masses); for more (MANY) the sums are in
// memory, m.spill, one row per workgroup: a pass of the table takes m.pass tiles and
// reads and writes 128 bytes per tile and chunk beside 72 matrix instructions.  The two
// are loops of their own: one for both took 162 us for 157 on 4096 momenta x 512 masses.
// With two tiles per wave for every list, and each chunk built again for the next ones,
// 1024 momenta (128 x 32 nodes) x 512 masses over ten panels took 229 us, 142 so (176
// in the direct form); x 300, not interpolated, 152, 134 so (123).  Lists of 129 to 384
// masses over more than four panels are the ones slower than the direct form, by up to
// 9 % (vertex 256 x 512 over ten panels, 48 x 8 x 16 nodes: 88 us, 73): masses on the
// device cannot be looked at before the launch.
constexpr int kChunk = 2;      // coefficient groups of a chunk
constexpr int kWaveTiles = 2;  // tiles of a wave held in registers
static_assert(kNodeWaves * kWaveTiles == kMassRegTiles && kMassPassTiles <= 32 * kNodeWaves,
              "a wave's tiles of a pass are the bits of a word");
// Tiles of 16: the nodes of the panels, then the masses (those in a panel are passed over).
__device__ __forceinline__ int node_tiles(const GridArgs &g, unsigned panels) {
  return N / 16 * __builtin_popcount(panels & ~kSingles) +
         ((panels & kSingles) ? ((int)g.n_m + 15) / 16 : 0);
}
template <int G, int E, bool MANY, class LaneRow, class Fill, class Expand, class Single>
__device__ __forceinline__ void node_values(const GridArgs &g, const MassPlan &m, double *lC,
                                            int64_t a, int part, unsigned panels,
                                            bool p_ok, bool table, int n_grp, LaneRow lane_row,
                                            Fill fill, Expand expand, Single single) {
  constexpr int kRows = 2 * G + E;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int parts = m.parts;
  const unsigned inside = panels & ~kSingles;
  const int n_node = N * __builtin_popcount(inside);
  const int n_tiles = node_tiles(g, panels);
  const int n_chunks = (n_grp + kChunk - 1) / kChunk;
  const int mine = lane & 15;
  // delta of entry e of the tiles and its place in the row of values; false:
  // nothing to evaluate there
  auto entry = [&](int e, double &d) {
    if (e < n_node) {
      unsigned rest = inside;
      for (int s = e / N; s > 0; --s) rest &= rest - 1u;
      const double x = __builtin_ldexp(m.nodes[e & (N - 1)], kMassPanelLo + 4 * __builtin_ctz(rest));
      d = x / g.sig;  // sig: a power of two
      return true;
    }
    const int b = e - n_node;
    d = b < (int)g.n_m ? g.m2[b] + g.k2 : 1.0;
    return b < (int)g.n_m && slot_of(g.sig * d, inside) < 0;
  };
  int t0 = 0;  // first tile of the pass
  do {
    // x of a lane in tile q of the wave, 1 where the coefficient form has nothing to
    // evaluate; some: it has for a lane
    auto x_of = [&](int q, bool &some) {
      const int t = t0 + kNodeWaves * q + wave;
      double d;
      const bool want = t < n_tiles && entry(16 * t + mine, d);
      const double xs = want ? g.sig * d : 0.0;
      const bool in = table && fold_m_ok<G, E>(xs);
      some = __builtin_amdgcn_ballot_w64(in) != 0;
      return in ? xs : 1.0;
    };
    const int n_q = MANY ? (min(m.pass, n_tiles - t0) - wave + kNodeWaves - 1) / kNodeWaves
                         : kWaveTiles;
    // lane group r = lane / 16 holds sum r of the wave's masses
    double x[kWaveTiles], acc[kWaveTiles];
    bool any[kWaveTiles];
    unsigned todo = 0;  // tiles with something to evaluate
    if constexpr (MANY) {
#pragma unroll 1
      for (int q = 0; q < n_q; ++q) {
        bool some;
        (void)x_of(q, some);
        todo |= some ? 1u << q : 0u;
      }
    } else {
#pragma unroll
      for (int q = 0; q < kWaveTiles; ++q) {
        x[q] = x_of(q, any[q]);
        todo |= any[q];
        acc[q] = 0.0;
      }
    }
    // lane's sum of tile q of the wave in memory
    auto spilled = [&](int q) {
      return m.spill + ((int64_t)blockIdx.x * m.pass + kNodeWaves * q + wave) * kWave + lane;
    };
    // a pass with nodes is built for a momentum inside the coefficient form; one
    // of masses alone if any of them is
    bool build = table && 16 * t0 < n_node;  // workgroup-uniform
    if (table && !build) {
      unsigned *sh = reinterpret_cast<unsigned *>(lC);
      if (lane == 0) sh[wave] = todo;
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kNodeWaves; ++w) build |= sh[w] != 0;
      __syncthreads();
    }
    if (build) {
      for (int c = part; c < n_chunks; c += parts) {
        const int live = min(kChunk, n_grp - c * kChunk);
        __builtin_amdgcn_s_setprio(3);
#pragma unroll 1
        for (int gl = 0; gl < live; ++gl) {
          const auto row = lane_row(c * kChunk + gl, lane);
          double *col = lC + gl * kRows * kWave + lane;
          // the wave's values of the group together: independent chains
          double H[G / kNodeWaves];
#pragma unroll
          for (int r = 0; r < G / kNodeWaves; ++r) H[r] = fill(row, wave + kNodeWaves * r);
#pragma unroll
          for (int r = 0; r < G / kNodeWaves; ++r) col[(wave + kNodeWaves * r) * kWave] = H[r];
        }
        __syncthreads();
        // the expanding waves alternate with the chunk and the momentum, so
        // that the work falls on every SIMD
        const int ew = wave ^ (2 * (((c >> __builtin_ctz(parts)) + (int)a) & 1));
        if (ew < live) expand(c * kChunk + ew, lC + ew * kRows * kWave + lane, lane);
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        // the chunk's part of sum c mod 4 of the masses at xq
        auto chunk_sum = [&](double xq) {
          double v[MfmaShape<G, E>::kP];
          mfma_powers<G, E>(xq, lane, v);
          double tot = 0.0;
#pragma unroll 1
          for (int gl = 0; gl < live; ++gl) {
            const double *grp = lC + gl * kRows * kWave;
            mfma_slice_pair<G, E, true>(grp, lane, v, 0, 1, tot);
            mfma_slice_pair<G, E, true>(grp, lane, v, 2, 3, tot);
          }
          tot = swap_add<32>(tot, tot);
          return swap_add<16>(tot, tot);
        };
        if constexpr (MANY) {
#pragma unroll 1
          for (unsigned left = todo; left; left &= left - 1u) {  // wave-uniform
            const int q = __builtin_ctz(left);
            bool some;
            const double tot = chunk_sum(x_of(q, some));
            double *sum = spilled(q);
            if (lane >> 4 == (c & 3)) *sum = c < 4 ? tot : *sum + tot;
          }
        } else {
#pragma unroll
          for (int q = 0; q < kWaveTiles; ++q) {
            if (!any[q]) continue;  // wave-uniform
            // the powers of x are formed again for each chunk: kept over the
            // build they would cost it its registers
            asm volatile("" : "+v"(x[q]));
            const double tot = chunk_sum(x[q]);
            acc[q] += lane >> 4 == (c & 3) ? tot : 0.0;
          }
        }
        __syncthreads();  // the chunk is consumed
      }
    }
    auto store = [&](int q, double sums) {
      const int t = t0 + kNodeWaves * q + wave;
      if (t >= n_tiles) return;  // wave-uniform
      const int e = 16 * t + mine;
      double d;
      const bool want = entry(e, d);
      const bool ok = p_ok && d > 0.0;
      const bool in = table && ok && fold_m_ok<G, E>(g.sig * d);
      double s[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        s[r] = __shfl(sums, 16 * r + mine, kWave);
        if (!in) s[r] = 0.0;
      }
      if (part == 0) {  // workgroup-uniform
        unsigned long long sm = __builtin_amdgcn_ballot_w64(want && ok && !in && lane < 16);
        while (sm) {  // wave-uniform: masses or momenta outside the coefficient form
          const int k = __builtin_ctzll(sm);
          sm &= sm - 1ull;
          const double one = single(__shfl(d, k, kWave));
          const double w = wave_sum_fold<1>(&one, lane);
          if (mine == k) s[0] = w * (g.pref / g.pref_c);
        }
        if (!ok) s[0] = __builtin_nan("");
      }
      if (lane < 16 && want) {
        if (!ok) *g.flag = 1;
        double *dst = m.val + a * m.ld + e;
        if (parts == 1) {
          *dst = ((s[0] + s[1]) + s[2]) + s[3];
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if ((r & (parts - 1)) == part) dst[r * m.plane] = s[r];
        }
      }
    };
    if constexpr (MANY) {
      // sums of this part that have a chunk
      const int r = lane >> 4;
      const bool has = build && r < n_chunks && (r & (parts - 1)) == part;
#pragma unroll 1
      for (int q = 0; q < n_q; ++q)
        store(q, has && ((todo >> q) & 1u) ? *spilled(q) : 0.0);
    } else {
#pragma unroll
      for (int q = 0; q < kWaveTiles; ++q) store(q, acc[q]);
    }
  } while (MANY && (t0 += m.pass) < n_tiles);
}

// LDS of the node kernels: chunk | regulator table | the rule's tables.

// Workgroups take (momentum, part) pairs in turn.
template <int REG, int G>
__global__ __launch_bounds__(64 * kNodeWaves, 4) void grid_nodes_kernel(GridArgs g, MassPlan m) {
  extern __shared__ double lds[];
  const int n_blocks = (int)gridDim.x - m.n_lag;
  if ((int)blockIdx.x >= n_blocks) {
    lagrange_rows<2>(g, m, (int)blockIdx.x - n_blocks);
    return;
  }
  const int n_r = g.n_r, n_a = g.n_a;
  const FoldShape<G> fs(g.U, g.T);
  double *lC = lds;
  double *ht = lC + kChunk * (2 * G + 2) * kWave;
  const int n_ap = g.J * fs.NG * G;  // angular slots of the lane split: padded with mu = 0
  double *lo = ht + (REG == kExp ? kRegPanels * kRegCoef : 0);  // 1 + x_j (-1 past n_a)
  double *lm = lo + n_ap;            // mu_j
  const unsigned panels = mass_panels(g, reinterpret_cast<unsigned *>(lC));
  if (blockIdx.x == 0 && threadIdx.x == 0) *m.panels = panels;
  stage_regulator<REG>(m, ht);
  for (int j = threadIdx.x; j < n_ap; j += blockDim.x) {
    lo[j] = j < n_a ? g.tab[3 * n_r + j] : -1.0;
    lm[j] = j < n_a ? g.tab[3 * n_r + n_a + j] : 0.0;
  }
  __syncthreads();
  const int64_t n_work = g.n_p * m.parts;
  auto run = [&](auto many) {
    for (int64_t w = blockIdx.x; w < n_work; w += n_blocks) {
      const int64_t a = w >> __builtin_ctz(m.parts);  // parts: 1, 2 or 4
      const int part = (int)w & (m.parts - 1);
      const double p = g.p[a];
      const bool p_ok = p >= 0.0;
      const bool table = p_ok && fold_p_ok<G>(p, g);  // workgroup-uniform
      const int rsh = __builtin_ctz(g.R);
      struct Row {
        double a, b;       // s = a + b (1 + x_j)
        const double *lo;  // 1 + x_j of the row's term 0; term k at lo[J k]
        bool live;
      };
      auto lane_row = [&](int gg, int l) {
        const int t = gg / fs.NG, gi = gg - t * fs.NG;  // scalar
        const int i = (l & (g.R - 1)) + g.R * t;
        const double q = g.tab[min(i, n_r - 1)];
        const double qm = q - p;
        return Row{qm * qm, (2.0 * q) * p, lo + (l >> rsh) + g.J * gi * G, i < n_r};
      };
      auto fill = [&](const Row &r, int k) {
        const double o = r.lo[g.J * k];  // padded terms: 1 + x_j = -1
        const double H = hk_build<REG>(g, fmax(__builtin_fma(r.b, o, r.a), 0.0), ht);
        return r.live && o >= 0.0 ? H : 0.0;
      };
      auto expand = [&](int gg, double *col, int l) {
        const int t = gg / fs.NG, gi = gg - t * fs.NG;
        const int i = (l & (g.R - 1)) + g.R * t, ic = min(i, n_r - 1);
        const double Hq = i < n_r ? g.sig * g.tab[2 * n_r + ic] : 0.0;
        const double c = i < n_r ? g.kap * g.tab[n_r + ic] : 0.0;  // 0: the row adds nothing
        const double f[2] = {Hq, Hq};
        const double *mu = lm + (l >> rsh) + g.J * gi * G;
        expand_group<G, 2>(col, f, c, [&](int k) { return mu[g.J * k]; });
      };
      // every term on its own, for masses or momenta outside the coefficient form
      auto single = [&](double delta) {
        const int l = threadIdx.x & (kWave - 1);
        double total = 0.0;
  #pragma unroll 1
        for (int t = 0; t < g.T; ++t) {
          const int i = (l & (g.R - 1)) + g.R * t, ic = min(i, n_r - 1);
          const double Gq = rcp64(g.tab[2 * n_r + ic] + delta);
          const double A = i < n_r ? (g.tab[n_r + ic] * Gq) * Gq : 0.0;
          double inner = 0.0;
  #pragma unroll 1
          for (int gi = 0; gi < fs.NG; ++gi) {
            const Row r = lane_row(t * fs.NG + gi, l);
  #pragma unroll 1
            for (int k = 0; k < G; ++k) {
              const double mu = lm[(l >> rsh) + g.J * (gi * G + k)];
              if (mu > 0.0) inner = __builtin_fma(mu, rcp64(fill(r, k) / g.sig + delta), inner);
            }
          }
          total = __builtin_fma(A, inner, total);
        }
        return total;
      };
      node_values<G, 2, many.value>(g, m, lC, a, part, panels, p_ok, table, g.T * fs.NG,
                                    lane_row, fill, expand, single);
    }
  };
  if (__builtin_expect(node_tiles(g, panels) <= kMassRegTiles, 1))
    run(std::false_type{});
  else
    run(std::true_type{});
}

// As grid_nodes_kernel for the vertex diagram: lane rows are (radial, polar)
// pairs pi = l + 64 t, groups azimuthal nodes (device_grid.h, vertex section).
template <int REG, int G>
__global__ __launch_bounds__(64 * kNodeWaves, 4) void vertex_nodes_kernel(GridArgs g, MassPlan m) {
  extern __shared__ double lds[];
  const int n_blocks = (int)gridDim.x - m.n_lag;
  if ((int)blockIdx.x >= n_blocks) {
    lagrange_rows<3>(g, m, (int)blockIdx.x - n_blocks);
    return;
  }
  const int n_r = g.n_r, n_a = g.n_a, n_phi = g.n_phi;
  const FoldShape<G, 3> fs(g.U, g.T);
  double *lC = lds;
  double *ht = lC + kChunk * (2 * G + 3) * kWave;
  double *lx = ht + (REG == kExp ? kRegPanels * kRegCoef : 0);  // x_j
  double *lm = lx + n_a;        // mu_j
  double *lsx = lm + n_a;       // sqrt(1 - x_j^2)
  double *lcp = lsx + n_a;      // cos phi_l
  const int n_pp = fs.NG * G;   // azimuthal slots: padded with nu = 0
  double *lnu = lcp + n_pp;     // nu_l
  const unsigned panels = mass_panels(g, reinterpret_cast<unsigned *>(lC));
  if (blockIdx.x == 0 && threadIdx.x == 0) *m.panels = panels;
  stage_regulator<REG>(m, ht);
  for (int idx = threadIdx.x; idx < n_a; idx += blockDim.x) {
    lx[idx] = g.vtab[idx];
    lm[idx] = g.tab[3 * n_r + n_a + idx];
    lsx[idx] = g.vtab[n_a + idx];
  }
  for (int idx = threadIdx.x; idx < n_pp; idx += blockDim.x) {
    lcp[idx] = idx < n_phi ? g.vtab[2 * n_a + idx] : 0.0;
    lnu[idx] = idx < n_phi ? g.vtab[2 * n_a + n_phi + idx] : 0.0;
  }
  __syncthreads();
  const int64_t n_work = g.n_p * m.parts;
  auto run = [&](auto many) {
    for (int64_t w = blockIdx.x; w < n_work; w += n_blocks) {
      const int64_t a = w >> __builtin_ctz(m.parts);  // parts: 1, 2 or 4
      const int part = (int)w & (m.parts - 1);
      const double p1 = g.p[a], p2 = g.p2[a], ct = g.c12[a];
      const bool p_ok = p1 >= 0.0 && p2 >= 0.0 && ct >= -1.0 && ct <= 1.0;
      const double st = p_ok ? sqrt((1.0 - ct) * (1.0 + ct)) : 0.0;
      const bool table = p_ok && fold_p_ok<G, 3>(fmax(p1, p2), g);
      const int n_pairs = n_r * n_a;
      struct Row {
        double q, x, sx;  // q_i, x_j, sqrt(1 - x_j^2) of the lane row's pair
        int az;           // azimuthal node of its term 0
        bool live;
      };
      auto lane_row = [&](int gg, int l) {
        const int t = gg / fs.NG, gi = gg - t * fs.NG;
        const int pi = min(l + kWave * t, n_pairs - 1);
        const int i = pi / n_a, j = pi - i * n_a;
        return Row{g.tab[i], lx[j], lsx[j], gi * G, l + kWave * t < n_pairs};
      };
      auto fill = [&](const Row &r, int k) {
        const int az = r.az + k;
        const double s2 = vertex_s2<REG>(r.q, p2, r.x, r.sx, lcp[az], ct, st);
        const double H = hk_build<REG>(g, s2, ht);
        return r.live && az < n_phi ? H : 0.0;
      };
      auto expand = [&](int gg, double *col, int l) {
        const int t = gg / fs.NG, gi = gg - t * fs.NG;
        const bool vp = l + kWave * t < n_pairs;
        const int pi = min(l + kWave * t, n_pairs - 1);
        const int i = pi / n_a, j = pi - i * n_a;
        const double q = g.tab[i];
        const double s1 = fmax((q * q + p1 * p1) + (2.0 * q) * p1 * lx[j], 0.0);
        const double Hq = vp ? g.sig * g.tab[2 * n_r + i] : 0.0;
        const double f[3] = {Hq, Hq, vp ? hk_build<REG>(g, s1, ht) : 0.0};
        const double c = vp ? (g.kap * g.tab[n_r + i]) * lm[j] : 0.0;  // 0: the row adds nothing
        const double *nu = lnu + gi * G;
        expand_group<G, 3>(col, f, c, [&](int k) { return nu[k]; });
      };
      auto single = [&](double delta) {
        const int l = threadIdx.x & (kWave - 1);
        double total = 0.0;
  #pragma unroll 1
        for (int t = 0; t < g.T; ++t) {
          const bool vp = l + kWave * t < n_pairs;
          const int pi = min(l + kWave * t, n_pairs - 1);
          const int i = pi / n_a, j = pi - i * n_a;
          const double q = g.tab[i];
          const double Gq = rcp64(g.tab[2 * n_r + i] + delta);
          const double A = vp ? (g.tab[n_r + i] * Gq) * Gq : 0.0;
          const double s1 = fmax((q * q + p1 * p1) + (2.0 * q) * p1 * lx[j], 0.0);
          const double G1 = rcp64(hk_build<REG>(g, s1, ht) / g.sig + delta);
          double inner = 0.0;
  #pragma unroll 1
          for (int gi = 0; gi < fs.NG; ++gi) {
            const Row r = lane_row(t * fs.NG + gi, l);
  #pragma unroll 1
            for (int k = 0; k < G; ++k) {
              const double nu = lnu[gi * G + k];
              if (nu > 0.0) inner = __builtin_fma(nu, rcp64(fill(r, k) / g.sig + delta), inner);
            }
          }
          total = __builtin_fma((A * lm[j]) * G1, inner, total);
        }
        return total;
      };
      node_values<G, 3, many.value>(g, m, lC, a, part, panels, p_ok, table, g.T * fs.NG,
                                    lane_row, fill, expand, single);
    }
  };
  if (__builtin_expect(node_tiles(g, panels) <= kMassRegTiles, 1))
    run(std::false_type{});
  else
    run(std::true_type{});
}

// out[a, b] = pref_c sum_n L[b][n] val[a][slot_b N + n] for the masses b of a
// panel, pref_c val[a][entry of b] for the others; val is the sum of its
// planes.  A wave takes 16 masses and 16 momenta: bound by the latency of its
// loads, so one tile per wave and as many waves as there are tiles (four tiles
// in turn took 12.7 us at 4096 x 512 and 18 us at 256 x 512 with four planes).
// Masses of one tile may belong to several panels: one product per panel
// present, the rows of the other masses zero (node values are finite or, for a
// momentum outside the domain, all NaN).
template <int PLANES>
__device__ __forceinline__ double plane_sum(const MassPlan &m, const double *v) {
  double s = v[0];
#pragma unroll
  for (int r = 1; r < PLANES; ++r) s = s + v[r * m.plane];
  return s;
}

template <int PLANES>
__global__ __launch_bounds__(256) void mass_interp_kernel(GridArgs g, MassPlan m) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int col = lane & 15, e = lane >> 4;
  const int64_t b = (int64_t)blockIdx.x * 16 + col;
  const bool vb = b < g.n_m;
  const unsigned panels = *m.panels;
  const int slot = vb ? slot_of(g.sig * (g.m2[b] + g.k2), panels) : -1;
  const int64_t single = N * __builtin_popcount(panels & ~kSingles) + b;  // its entry if slot < 0
  unsigned present = 0;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int sr = __builtin_amdgcn_readlane(slot, r);
    present |= sr >= 0 ? 1u << sr : 0u;
  }
  double L[N / 4];
#pragma unroll
  for (int c = 0; c < N / 4; ++c) L[c] = slot >= 0 ? m.lag[b * N + 8 * e + c] : 0.0;
  const int64_t a0 = ((int64_t)blockIdx.y * 4 + wave) * 16;
  if (a0 >= g.n_p) return;  // wave-uniform
  const int64_t ar = a0 + col < g.n_p ? a0 + col : g.n_p - 1;
  dbl4 D = {0.0, 0.0, 0.0, 0.0};
  for (unsigned todo = present; todo; todo &= todo - 1u) {  // wave-uniform
    const int s = __builtin_ctz(todo);
    const double *va = m.val + ar * m.ld + s * N + 8 * e;
    const bool mine = slot == s;
    double v[N / 4];
#pragma unroll
    for (int c = 0; c < N / 4; ++c) v[c] = plane_sum<PLANES>(m, va + c);
#pragma unroll
    for (int c = 0; c < N / 4; ++c)
      D = __builtin_amdgcn_mfma_f64_16x16x4f64(v[c], mine ? L[c] : 0.0, D, 0, 0, 0);
  }
  if (vb) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t a = a0 + 4 * r + e;
      if (a < g.n_p) {
        const double v = slot >= 0 ? D[r] : plane_sum<PLANES>(m, m.val + a * m.ld + single);
        g.out[a * g.n_m + b] = g.pref_c * v;
      }
    }
  }
}

void allow_lds(const void *fn) {
  (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  (void)hipGetLastError();
}

// Group size: matrix instructions per 16 terms and tile are 2 (8/4 + 1 + 8/4) =
// 10 for groups of 8, 16/4 + 1 + 16/4 = 9 for groups of 16; terms past the row
// are padding.
int mass_nodes_group(const GridArgs &g) {
  const int c8 = ((g.U + 7) / 8) * 5, c16 = ((g.U + 15) / 16) * 9;
  return c8 < c16 ? 8 : 16;
}

template <bool VERTEX, int REG, int G>
void nodes_t(const GridArgs &g, const MassPlan &m, int blocks, int lds, hipStream_t st) {
  const dim3 grid((unsigned)(blocks + m.n_lag)), block(64 * kNodeWaves);
  if constexpr (VERTEX) {
    static const bool once = (allow_lds((const void *)&vertex_nodes_kernel<REG, G>), true);
    (void)once;
    hipLaunchKernelGGL((vertex_nodes_kernel<REG, G>), grid, block, lds, st, g, m);
  } else {
    static const bool once = (allow_lds((const void *)&grid_nodes_kernel<REG, G>), true);
    (void)once;
    hipLaunchKernelGGL((grid_nodes_kernel<REG, G>), grid, block, lds, st, g, m);
  }
}
template <bool VERTEX, int REG>
void nodes_reg(const GridArgs &g, const MassPlan &m, int blocks, int lds, hipStream_t st) {
  if (mass_nodes_group(g) == 16)
    nodes_t<VERTEX, REG, 16>(g, m, blocks, lds, st);
  else
    nodes_t<VERTEX, REG, 8>(g, m, blocks, lds, st);
}

int mass_nodes_lds(const GridArgs &g, int reg, bool vertex) {
  const int G = mass_nodes_group(g), slots = ((g.U + G - 1) / G) * G;
  const int rows = 2 * G + (vertex ? 3 : 2);
  const int small = vertex ? 3 * g.n_a + 2 * slots : 2 * g.J * slots;
  return (int)sizeof(double) *
         (kChunk * rows * kWave + (reg == kExp ? kRegPanels * kRegCoef : 0) + small);
}

}  // namespace

// Workgroups per momentum: four fit a CU, so a momentum is split over two or
// four while that leaves none of them a second one.
int mass_nodes_parts(int64_t n_p, int n_cu) {
  return n_p <= n_cu ? 4 : n_p <= 2 * (int64_t)n_cu ? 2 : 1;
}

int mass_nodes_blocks(int64_t n_p, int parts, int n_cu) {
  return (int)std::min<int64_t>(n_p * parts, 4 * (int64_t)n_cu);
}

int launch_mass_nodes(const GridArgs &g, MassPlan m, int reg, bool vertex, bool first, int n_cu,
                      void *stream) {
  if (g.n_p <= 0 || g.n_m <= 0) return 0;
  m.n_lag = first ? (int)((g.n_m + kLagTile - 1) / kLagTile) : 0;
  hipStream_t st = (hipStream_t)stream;
  const int lds = mass_nodes_lds(g, reg, vertex);
  if (lds > 160 * 1024) return (int)hipErrorInvalidValue;
  const int blocks = mass_nodes_blocks(g.n_p, m.parts, n_cu);
  if (vertex) {
    if (reg == kExp)
      nodes_reg<true, kExp>(g, m, blocks, lds, st);
    else
      nodes_reg<true, kLitim>(g, m, blocks, lds, st);
  } else {
    if (reg == kExp)
      nodes_reg<false, kExp>(g, m, blocks, lds, st);
    else
      nodes_reg<false, kLitim>(g, m, blocks, lds, st);
  }
  const dim3 grid((unsigned)((g.n_m + 15) / 16),
                  (unsigned)((g.n_p + 63) / 64));
  if (m.parts > 1)
    hipLaunchKernelGGL(mass_interp_kernel<4>, grid, dim3(256), 0, st, g, m);
  else
    hipLaunchKernelGGL(mass_interp_kernel<1>, grid, dim3(256), 0, st, g, m);
  return (int)hipGetLastError();
}

}  // namespace frg

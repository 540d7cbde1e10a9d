// Column solve (steps 2-6 of Sec. 3.4 plus the spectral vorticity): one
// wavefront takes 16 (kx, ky) columns, the Chebyshev transforms are matrix
// products on the matrix cores and everything stays in registers.
//
// Rotated frame.  With L along k and T across it, and the along-k quantities
// multiplied by i, every operator of a column is real, so the real and the
// imaginary part of a column are two independent real problems.  With
//   a = i f_L,  U = i u_L,  gamma = i g_T     (g: dipole density)
// the body force f + (1/2) curl g is a - (1/2) gamma', f_T - (1/2) i k g_z +
// (1/2) g_L', f_z + (1/2) k gamma, and
//   p'' - k^2 p = k i F_L + F_z'          (the dipoles drop out: div curl = 0)
//   W'' - k^2 W = (p' - F_z - (1/2) k gamma) / eta
//   U'' - k^2 U = (-k p - i F_L + (1/2) gamma') / eta
//   T'' - k^2 T = -(F_T - (1/2) i k G_z + (1/2) G_L') / eta
// with  g_H, g_0 = 0, 0;  p(H), p(0);  p(H), -p(0) (over 2 eta);  0, 0  in the
// Robin conditions.  Out come U, T, W and omega = (1/2) curl u: omega_L =
// -(1/2) T', i omega_T = (1/2)(k W + U'), omega_z = (1/2) i k T.
//
// Layout.  v_mfma_*_16x16x4 takes B[k][j] from lane j + 16 k and returns
// column j in the four lanes j + 16 g.  A lane loads the complex node values
// of its column j = lane % 16 and of every fourth node, so the real and the
// imaginary parts are the B operands of two products (sets) with no data
// movement.  The rows of the transform matrix are ordered so that lane group
// g gets the coefficients: 0, 1: the lower and upper half of the even ones,
// 2, 3: of the odd ones.  One v_permlane16_swap of the two sets then leaves
// each lane with one parity of one real column,
//   lane = 16 (2 parity + imaginary) + column,  NA coefficients 2 i + parity,
// and the tridiagonal half-systems of the BVPs become plain sequential sweeps
// in registers, the same in every lane (no scans and no lane moves).  What couples the parities (B of a series, sums at the walls) is
// exchanged with v_permlane32_swap.  The inverse transform reads the same
// registers as B operands after the opposite swap, and a lane ends with the
// complex values of its column at four nodes per tile: 128-byte runs per
// plane in FP32, both ways.
//
// z-derivatives on the right-hand sides are taken through B^2 D = B, i.e.
// (f_{m-1} - f_{m+1}) / (2 m): no recurrence over the coefficients.
//
// Bound by several units at once, at two wavefronts per SIMD: vector issue 0.43
// (the FP64 sweeps), matrix cores 0.28, HBM 0.64 of a plain copy at 2176^2, 20
// planes.  Registers, as the compiler reports them for FP32 transforms: none
// spilled up to 20 nodes, up to 32 nodes at most 6 above one wall and 89 to 119
// between two, where the FP64 low-wavenumber copy shares the kernel; for FP64
// transforms at most 6 up to 48 nodes, up to 163 beyond.  Against eight lanes per
// column with segmented scans (and, for FP64 data or Nz > 32, one thread per column
// in scratch), one launch: 2176^2, 20 planes, mixed 3.37 -> 1.62 ms; two walls 4.39
// -> 1.9; 2700^2, 11 planes, forces only 3.34 -> 1.05; 768^2 0.43 -> 0.22; in FP64
// 1.41 -> 0.44; 192^2, Nz = 48, FP64 6.2 -> 0.12.
#include <algorithm>
#include <type_traits>

#include "fcmdp_internal.h"
#include "colmath.h"

// Fused multiply-adds are written out: left to the compiler they would differ
// from one instantiation to another, and a call without torques would not have
// the bits of a call with zero torques.
#pragma clang fp contract(off)

namespace fcmdp {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef double d4v __attribute__((ext_vector_type(4)));

// matrix product of the compute type; row(g, r): the row of D that lane group
// g holds in register r
template <typename D> struct Mat;
template <> struct Mat<float> {
  using acc = f4v;
  static __device__ __forceinline__ acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int r) { return 4 * g + r; }
  static __device__ __forceinline__ int group(int row) { return row >> 2; }
  static __device__ __forceinline__ int reg(int row) { return row & 3; }
};
template <> struct Mat<double> {
  using acc = d4v;
  static __device__ __forceinline__ acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int r) { return 4 * r + g; }
  static __device__ __forceinline__ int group(int row) { return row & 3; }
  static __device__ __forceinline__ int reg(int row) { return row >> 2; }
};

// lanes are four rows of 16: rows 1, 3 of a trade places with rows 0, 2 of b
__device__ __forceinline__ void swap16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b),
                                                  false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap16(double& a, double& b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b),
                                                   false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b),
                                                   false, false);
  a = __hiloint2double(hi[0], lo[0]);
  b = __hiloint2double(hi[1], lo[1]);
}
// Exchange between the halves of the wavefront (up: this lane is one of
// 32-63): lanes 0-31 get x of lane + 32, lanes 32-63 get y of lane - 32.
__device__ __forceinline__ float across(float x, float y, bool up) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y),
                                                  false, false);
  return __uint_as_float(up ? r[0] : r[1]);
}
__device__ __forceinline__ double across(double x, double y, bool up) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(y),
                                                   false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(y),
                                                   false, false);
  return __hiloint2double(up ? hi[0] : hi[1], up ? lo[0] : lo[1]);
}

// 1/x from the hardware estimate and two Newton steps (within an ulp or two
// of the rounded quotient; x is a normal, finite number here).
__device__ __forceinline__ double frcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// Value of lane xor 32, through the LDS crossbar (no vector instruction).
__device__ __forceinline__ float pass(float x, int addr) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(x)));
}
__device__ __forceinline__ double pass(double x, int addr) {
  return __hiloint2double(__builtin_amdgcn_ds_bpermute(addr, __double2hiint(x)),
                          __builtin_amdgcn_ds_bpermute(addr, __double2loint(x)));
}

// Rows of the double antiderivative, m = 2 i + parity >= 2, divided by their
// first entry tl = (H^2/4) / (4 m (m - 1)):
//   (H^2/4)(B^2 f)_m  = tl (d_i - rho d_{i+1}),  d_i = c_{m-2} f_{m-2} - f_m,
//                       rho = (m - 1) / (m + 1)
//   (H^2/4)(B^2 f')_m = tl (4/H)(m - 1)(f_{m-1} - f_{m+1}).
// tl = rho = 0 for m >= N.  The rows of both parities lie in LDS.
// Table rows are read where they are used: the address is opaque to the
// optimiser at every use, so that the reads are neither hoisted out of the
// column loop nor kept in registers from one sweep to the next (the scheduling
// barrier keeps the sweeps from being interleaved for the same reason).
typedef __attribute__((address_space(3))) const double* LdsPtr;
template <int NA> struct RowTab {
  double v[2][5][NA];             // [parity]: rho, tl, m - 1, m^2, m
};
template <int NA> struct Rows {
  LdsPtr p;
  __device__ __forceinline__ double rho(int i) const { return p[i]; }
  __device__ __forceinline__ double tl(int i) const { return p[NA + i]; }
  __device__ __forceinline__ double m1(int i) const { return p[2 * NA + i]; }
  __device__ __forceinline__ double m2(int i) const { return p[3 * NA + i]; }
  __device__ __forceinline__ double n(int i) const { return p[4 * NA + i]; }
};
template <int NA>
__device__ __forceinline__ Rows<NA> fresh(const RowTab<NA>& tab, int off) {
  __builtin_amdgcn_sched_barrier(0);
  LdsPtr p = (LdsPtr)&tab.v[0][0][0] + off;
  asm volatile("" : "+v"(p));
  return Rows<NA>{p};
}

// Coefficients n = 2 i + parity of one real column, NA per lane.
// The tridiagonal half of y - k^2 (H^2/4) B^2 y = R with the dense boundary
// row sum_i e_i y_i = g (e_i = m^2 + kappa), eliminated from the last
// coefficient.  With R_i = k^2 tl_i r_i (the callers form r, scaled so that
// one of its series needs no factor) and al_i = k^2 tl_i / Delta_i:
//   s_i = r_i + rho_i be_{i+1},  be_i = al_i s_i,  y_i = al_i (c y_{i-1} + s_i)
// and c_i = e_i + al_{i+1} c_{i+1} is the weight that y_i carries in
// sum_{j >= i} e_j y_j: five operations per row and right-hand side.
template <int NA> struct HalfOp {
  double al[NA], c[NA];           // entries 1 .. NA - 1
  double ic0;

  __device__ __forceinline__ void prepare(Rows<NA> rows, double k2, double kappa, bool up) {
    double aln = 0.0, cn = 0.0;
#pragma unroll
    for (int i = NA - 1; i >= 1; --i) {
      const double t = k2 * rows.tl(i), rho = rows.rho(i);
      cn = fma(aln, cn, rows.m2(i) + kappa);
      aln = t * frcp(fma(t, fma(-rho, aln, 1.0 + rho), 1.0));
      al[i] = aln;
      c[i] = cn;
    }
    // c_{m-2} = 2 for m = 2; e_0, e_1 = 0, 1 plus kappa
    ic0 = frcp(fma(up ? aln : 2.0 * aln, cn, (up ? 1.0 : 0.0) + kappa));
  }
  // y: r_1 .. r_{NA-1} on entry, the solution on return
  __device__ __forceinline__ void solve(Rows<NA> rows, double* y, double g, bool up) const {
    double b = 0.0;
#pragma unroll
    for (int i = NA - 1; i >= 1; --i) {
      y[i] = fma(rows.rho(i), b, y[i]);
      b = al[i] * y[i];
      g = fma(-c[i], b, g);
    }
    y[0] = g * ic0;
    y[1] = al[1] * fma(up ? 1.0 : 2.0, y[0], y[1]);
#pragma unroll
    for (int i = 2; i < NA; ++i) y[i] = al[i] * (y[i - 1] + y[i]);
  }
};

// rows 1 .. NA - 1 of the two kinds of right-hand side (f(i): this lane's
// coefficient i); SET: out = , else out +=; NEG: minus
template <int NA, bool SET, bool NEG, typename F>
__device__ __forceinline__ void add_b2(Rows<NA> rows, const F& f, bool up, double* out) {
  const double f0 = f(0);
  double cur = f(1);
  double d = (up ? f0 : 2.0 * f0) - cur;
#pragma unroll
  for (int i = 1; i < NA; ++i) {
    const double next = i + 1 < NA ? f(i + 1 < NA ? i + 1 : i) : 0.0;
    const double dn = cur - next;
    const double v = NEG ? fma(rows.rho(i), dn, -d) : fma(-rows.rho(i), dn, d);
    out[i] = SET ? v : out[i] + v;
    cur = next;
    d = dn;
  }
}
template <int NA, bool SET, bool NEG, typename F>
__device__ __forceinline__ void add_b(Rows<NA> rows, const F& f, bool up, int addr,
                                      double* out) {
  using V = decltype(f(0));
  // row i needs the other parity's coefficients i - 1, i (even m) or i, i + 1
  V h[NA];
#pragma unroll
  for (int i = 1; i <= NA; ++i) {
    const V z = V(0);
    h[i - 1] = pass(up ? f(i - 1) : (i < NA ? f(i < NA ? i : 0) : z), addr);
  }
#pragma unroll
  for (int i = 1; i < NA; ++i) {
    const double d = (double)h[i - 1] - (double)h[i];
    out[i] = SET ? rows.m1(i) * d : fma(NEG ? -rows.m1(i) : rows.m1(i), d, out[i]);
  }
}
template <int NA>
__device__ __forceinline__ double own_sum(const double* y) {
  double a = y[0], b = y[1];
#pragma unroll
  for (int i = 2; i < NA; i += 2) {
    a += y[i];
    b += y[i + 1];
  }
  return a + b;
}
// sums over the series at the walls: top = sum a_n, bot = sum (-1)^n a_n
template <int NA>
__device__ __forceinline__ void wall_sums(const double* y, bool up, double& top,
                                          double& bot) {
  const double s = own_sum<NA>(y), o = across(s, s, up);
  top = s + o;
  bot = up ? o - s : s - o;
}
// z-derivative sums in units of 2/H: top = sum n^2 a_n, bot = sum (-1)^(n+1)
// n^2 a_n
template <int NA>
__device__ __forceinline__ void wall_dsums(Rows<NA> rows, const double* y, bool up,
                                           double& top, double& bot) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < NA; ++i) s = fma(rows.m2(i), y[i], s);
  const double o = across(s, s, up);
  top = s + o;
  bot = up ? s - o : o - s;
}
// k = 0: y'' = r; y holds the coefficients m >= 2 of the solution.  Bottom wall: y(0) - l_0 y'(0) = g0, y'(H) = 0; slit channel:
// y(0) - l_0 y'(0) = g0, y(H) + l_H y'(H) = gH (a = 2 l / H).
template <int NA, int GEOM>
__device__ __forceinline__ void zero_mode(Rows<NA> rows, double* y, bool up, double a0, double aH,
                                          double g0, double gH) {
  y[0] = 0.0;
  double sp, sm, sn2, sdm;
  wall_sums<NA>(y, up, sp, sm);
  wall_dsums<NA>(rows, y, up, sn2, sdm);
  if constexpr (GEOM == 0) {
    y[0] = up ? -sn2 : -sn2 - sm + g0 + a0 * (sdm - sn2);
  } else {
    const double y1 = frcp(2.0 + a0 + aH) * (gH - g0 + sm - sp - a0 * sdm - aH * sn2);
    y[0] = up ? y1 : gH - sp - aH * sn2 - (1.0 + aH) * y1;
  }
}
// out_m = s c_m sum over n > m of the other parity of n a_n, c_0 = 1/2 (the
// series of the derivative for s = 4 / H): own suffix sums, rounded to the
// transform's type and exchanged
template <int NA, typename D>
__device__ __forceinline__ void derivative(Rows<NA> rows, const double* y, bool up, int addr,
                                           double s, D* out) {
  double sum = 0.0;
  D after = D(0);
#pragma unroll
  for (int i = NA - 1; i >= 0; --i) {
    sum = fma(rows.n(i), y[i], sum);
    const D here = (D)(s * sum);
    // even outputs 2 i: odd terms from i on; odd outputs: even terms from i + 1
    const D v = pass(up ? here : after, addr);
    out[i] = i == 0 && !up ? D(0.5) * v : v;
    after = here;
  }
}

// For q > 0: E = e^{-q}, s = 1 - E^2 and ex = s - 2 q E = 2 E (sinh q - q), the
// last two without cancellation at small q.  Taylor coefficients f[j] = 1 / j!
// from LDS (as constants of the library function they would be kept in
// registers over the whole column loop).
__device__ __forceinline__ void wall_decay(LdsPtr f, double q, double& E, double& s,
                                           double& ex) {
  asm volatile("" : "+v"(f));
  // e^{-q} = 2^{-n} e^{-r}, |r| <= ln 2 / 2: 0.347^14 / 14! < 5e-18
  const double n = rint(q * 1.4426950408889634074);
  double r = fma(-n, 0x1.62e42fefa39efp-1, q);
  r = fma(-n, 0x1.abc9e3b39803fp-56, r);
  double p = f[13];
#pragma unroll
  for (int j = 12; j >= 0; --j) p = fma(-r, p, f[j]);
  E = ldexp(p, -(int)n);
  const double q2 = q * q;
  double t = f[19];                                 // (sinh q - q) / q^3
#pragma unroll
  for (int j = 8; j >= 1; --j) t = fma(q2, t, f[2 * j + 1]);
  t *= q2;
  const bool small = q < 1.0;
  s = small ? 2.0 * E * q * (1.0 + t) : fma(-E, E, 1.0);
  ex = small ? 2.0 * E * q * t : fma(-2.0 * q, E, s);
}

template <typename T, typename D, int NT, int NA, int GEOM, bool TIN, bool WOUT>
__global__ void __launch_bounds__(256, sizeof(D) == 4 ? 2 : 1)
k_columns_mfma(ColParams cp, int low_blocks, const int* __restrict__ band,
               const cplx_t<T>* in, cplx_t<T>* out, const double* __restrict__ zc,
               const double* __restrict__ Mf, const double* __restrict__ Pi) {
  using C = cplx_t<T>;
  using M = Mat<D>;
  using Acc = typename M::acc;
  constexpr int kHalf = NA / 2;                    // coefficients per lane group
  static_assert(4 * NT >= kHalf && NA % 2 == 0, "rows of the transform");
  constexpr int kNin = TIN ? 6 : 3;
  // the FP64 route of the low-wavenumber columns exists
  constexpr bool kLow = GEOM == 1 && sizeof(T) == 4 && NA <= 16;
  __shared__ D mf[NT * kHalf * 64];                // forward: [tile][step][lane]
  __shared__ D pi[NT * kHalf * 64];                // inverse: [tile][step][lane]
  __shared__ RowTab<NA> tabs;
  constexpr int kPark = sizeof(D) == 4 ? (TIN ? 2 : 1) * NA : 0;
  __shared__ D parked[kPark ? 4 * kPark * 64 : 1];
  __shared__ D zn[2 * NA];
  __shared__ double fact[GEOM == 1 ? 20 : 1];      // 1 / j!
  const DevParams& dp = cp.dp;
  const int lo = band[0], hi = band[1];
  if (lo > hi) return;
  const int N = dp.Nz;
  const double H = dp.H;
  // node tiles of 16 of the inverse transform, and whether the last one to four
  // nodes take the 4 x 4 products
  constexpr bool kTail = sizeof(D) == 4;
  const int P = hi - lo + 1;
  const bool tail = kTail && P % 16 >= 1 && P % 16 <= 4;
  const int tiles = tail ? P / 16 : (P + 15) / 16;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // --- tables ---------------------------------------------------------------
  for (int e = tid; e < NT * kHalf * 64; e += 256) {
    const int l = e & 63, s = (e >> 6) % kHalf, t = (e >> 6) / kHalf;
    const int row = l & 15, g4 = l >> 4;
    // forward: row -> coefficient j of group g; column -> node 4 s + g4
    {
      const int g = M::group(row), j = 4 * t + M::reg(row);
      const int n = 2 * ((g & 1) * kHalf + j) + (g >> 1), c = 4 * s + g4;
      mf[e] = (j < kHalf && n < N && c < N) ? (D)Mf[c * N + n] : D(0);
    }
    // inverse: row -> band node; column -> coefficient s of group g4 (the 4 x 4
    // tail takes its rows from lane % 4)
    {
      const int n = 2 * ((g4 & 1) * kHalf + s) + (g4 >> 1);
      const int c = lo + 16 * t + (kTail && tail && t == tiles ? l & 3 : row);
      pi[e] = (n < N && c <= hi) ? (D)Pi[c * N + n] : D(0);
    }
  }
  for (int e = tid; e < 2 * NA; e += 256) {
    const int p = e / NA, m = 2 * (e % NA) + p;
    const bool row = m >= 2 && m < N;
    double(*v)[NA] = tabs.v[p];
    v[0][e % NA] = row ? (m - 1.0) / (m + 1.0) : 0.0;
    v[1][e % NA] = row ? 0.25 * H * H / (4.0 * m * (m - 1.0)) : 0.0;
    v[2][e % NA] = m - 1.0;
    v[3][e % NA] = (double)m * m;
    v[4][e % NA] = m;
    zn[e] = e < N ? (D)zc[e] : D(0);
  }
  if (GEOM == 1 && tid < 20) {
    double f = 1.0;
    for (int j = 2; j <= tid; ++j) f *= j;
    fact[tid] = 1.0 / f;
  }
  __syncthreads();

  const int K = dp.Nkx * dp.Ny;
  const int G = (K + 15) / 16;                     // column groups
  const size_t PS = (size_t)K;
  const int col = lane & 15, g4 = lane >> 4;
  const bool up = lane >= 32;                      // odd parity
  const bool imag = (lane & 16) != 0;
  const int toff = up ? 5 * NA : 0;
  const double s2H = cp.s2H;
  const int xaddr = (lane ^ 32) * 4;               // for pass()
  const double l0 = dp.slip0, lH = GEOM == 1 ? dp.slipH : 0.0;
  const bool slip = l0 != 0.0 || lH != 0.0;        // uniform
  const int s_lo = lo / 4, s_hi = hi / 4;
  // a group's band values are loaded several steps ahead of their products; the
  // next group's during this one's inverse transform do not fit the registers
  // (80 spilled, 1.85 -> 2.60 ms at 2176^2)
  constexpr int kCh = 5;                           // steps in flight
  // (part L takes all but G_z, part T all but F_z)
  auto fetch = [&](C (&w)[kCh][kNin], int grp, int s0, bool part_l, bool part_t) {
    const int idc = min(grp * 16 + col, K - 1);
#pragma unroll
    for (int u = 0; u < kCh; ++u) {
      const int c = min(max(4 * (s0 + u) + g4, lo), hi);
      const C* src = in + (size_t)c * PS + idc;
#pragma unroll
      for (int ch = 0; ch < kNin; ++ch) w[u][ch].x = w[u][ch].y = T(0);
      if (s0 + u <= s_hi) {                        // uniform
#pragma unroll
        for (int ch = 0; ch < kNin; ++ch)
          if ((part_l || ch != 2) && (part_t || ch != 5)) w[u][ch] = src[(size_t)ch * N * PS];
      }
    }
  };
  // LOW: the column groups that hold columns of the low-wavenumber square
  // (their own workgroups and their own copy of the code, so that the FP64
  // route's registers do not weigh on the other groups)
  auto run = [&](auto low_tag) __attribute__((always_inline)) {
  constexpr bool LOW = decltype(low_tag)::value;
  const int ns = dp.lowk_ns;
  int grp, stride, last;
  if constexpr (LOW) {
    // wave w takes group w % per of the range of columns kx Ny - ns .. kx Ny +
    // ns, kx = w / per; a group met by the range before is left to it
    const int per = ns / 8 + 2, w = blockIdx.x * 4 + wave, q = w / per;
    if (q > ns + 1) return;
    const int first = max(q * dp.Ny - ns, 0) / 16;
    grp = first + w % per;
    stride = G;
    last = min((q * dp.Ny + ns) / 16, G - 1) + 1;
    if (q > 0 && grp <= ((q - 1) * dp.Ny + ns) / 16) return;
  } else {
    grp = (blockIdx.x - low_blocks) * 4 + wave;
    stride = (gridDim.x - low_blocks) * 4;
    last = G;
  }
  C w[kCh][kNin];
  for (; grp < last; grp += stride) {
    int ln = lane;                                 // (opaque, as in fresh())
    asm volatile("" : "+v"(ln));
    const int idx = grp * 16 + col;
    const bool valid = idx < K;
    const int idc = valid ? idx : K - 1;
    const int kxi = idc / dp.Ny, kyi = idc - kxi * dp.Ny;
    const int nyi = kyi <= dp.Ny / 2 ? kyi : kyi - dp.Ny;
    const bool nyq = kxi == dp.Nx / 2 || kyi == dp.Ny / 2;
    const double kx = cp.kxs * kxi, ky = cp.kys * nyi;
    const double k = sqrt(fma(kx, kx, ky * ky));
    const bool zero = k == 0.0;                    // the mean flow's column
    const bool zero_grp = grp == 0;                // (uniform)
    // Units: p times k^2 H/4, U and T times cU = eta k^2 H/4, W times cW = eta
    // (k^2 H/4)^2 make the derivative terms of every right-hand side enter with
    // factor one; the inverse goes into the output scale.  The mean flow takes
    // a k so small that the sweeps return its rows m >= 2 as they are.
    const double kp = zero ? 1e-9 * cp.s2H : k, ik = frcp(kp);
    const double cx = zero ? 1.0 : kx * ik, cy = ky * ik;
    const double k2 = kp * kp, kappa = zero ? 1.0 : 0.5 * kp * H;
    const double cWU = 0.25 * H * k2, cUW = 4.0 * cp.iH * ik * ik;   // cW / cU and inverse
    int lcol = -1;
    if constexpr (kLow) {
      lcol = nyq || !valid ? -1 : lowk_col(dp, kxi, nyi);
      if ((__any(lcol >= 0) != 0) != LOW) continue;
    }

    // --- forward transform of the band nodes ---------------------------------
    // vectors: i F_L, F_z, gamma / 2 (part L), F_T - (1/2) i k G_z, G_L / 2 (T)
    D aL[NA], aZ[NA], aG[TIN ? NA : 1], aT[NA], aH[TIN ? NA : 1];
    D* const park = &parked[(size_t)wave * kPark * 64 + lane];
    auto forward = [&](auto part_l, auto part_t) {
      constexpr bool PL = decltype(part_l)::value, PT = decltype(part_t)::value;
      constexpr int nL = PL ? (TIN ? 3 : 2) : 0, nT = PT ? (TIN ? 2 : 1) : 0;
      constexpr int nV = nL + nT;
      Acc acc[nV][2][NT];
#pragma unroll
      for (int v = 0; v < nV; ++v)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[v][0][t] = acc[v][1][t] = Acc{0, 0, 0, 0};
      const D dcx = (D)cx, dcy = (D)cy, hk = (D)(0.5 * k);
      const D hcx = (D)(0.5 * cx), hcy = (D)(0.5 * cy);
      for (int s0 = s_lo; s0 <= s_hi; s0 += kCh) {
        fetch(w, grp, s0, PL, PT);
#pragma unroll
        for (int u = 0; u < kCh; ++u) {
          if (s0 + u > s_hi) break;                 // uniform
          const int c = 4 * (s0 + u) + g4;
          const bool ok = c >= lo && c <= hi;
          D fr[kNin], fi[kNin];
#pragma unroll
          for (int ch = 0; ch < kNin; ++ch) {
            fr[ch] = ok ? (D)w[u][ch].x : D(0);
            fi[ch] = ok ? (D)w[u][ch].y : D(0);
          }
          D xr[nV], xi[nV];
          if constexpr (PL) {
            xr[0] = -fma(dcx, fi[0], dcy * fi[1]);
            xi[0] = fma(dcx, fr[0], dcy * fr[1]);
            xr[1] = fr[2];
            xi[1] = fi[2];
            if constexpr (TIN) {
              xr[2] = -fma(hcx, fi[4], -(hcy * fi[3]));
              xi[2] = fma(hcx, fr[4], -(hcy * fr[3]));
            }
          }
          if constexpr (PT) {
            xr[nL] = fma(dcx, fr[1], -(dcy * fr[0]));
            xi[nL] = fma(dcx, fi[1], -(dcy * fi[0]));
            if constexpr (TIN) {
              xr[nL] = fma(hk, fi[5], xr[nL]);
              xi[nL] = fma(-hk, fr[5], xi[nL]);
              xr[nL + 1] = fma(hcx, fr[3], hcy * fr[4]);
              xi[nL + 1] = fma(hcx, fi[3], hcy * fi[4]);
            }
          }
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const D a = mf[(t * kHalf + s0 + u) * 64 + ln];
#pragma unroll
            for (int v = 0; v < nV; ++v) {
              acc[v][0][t] = M::mma(a, xr[v], acc[v][0][t]);
              acc[v][1][t] = M::mma(a, xi[v], acc[v][1][t]);
            }
          }
        }
      }
      auto take = [&](int v, D* dst) {
#pragma unroll
        for (int j = 0; j < kHalf; ++j) {
          D x = acc[v][0][j / 4][j % 4], y = acc[v][1][j / 4][j % 4];
          swap16(x, y);
          dst[j] = x;
          dst[kHalf + j] = y;
        }
      };
      if constexpr (PL) {
        take(0, aL);
        take(1, aZ);
        if constexpr (TIN) take(2, aG);
      }
      if constexpr (PT) {
        take(nL, aT);
        if constexpr (TIN) take(nL + 1, aH);
      }
    };
    using Yes = std::integral_constant<bool, true>;
    using No = std::integral_constant<bool, false>;
    if constexpr (sizeof(D) == 4) {
      forward(Yes{}, Yes{});
      // the T vectors wait in LDS for their turn
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        park[i * 64] = aT[i];
        if constexpr (TIN) park[(NA + i) * 64] = aH[i];
      }
    } else {
      forward(Yes{}, No{});                        // fewer registers at once
    }

    // --- the BVPs ----------------------------------------------------------------
    HalfOp<NA> op;
    // wall velocities of the column (uniform ones in the mean flow only), as
    // this lane's part of i u_L and u_T at z = 0 and z = H
    double wU0 = 0.0, wT0 = 0.0, wUH = 0.0, wTH = 0.0;
    {
      auto wall = [&](int i, const double* w, double& wu, double& wt) {
        Z2 x = zmk(0, 0), y = zmk(0, 0);
        if (dp.wallspec) {
          const C* p = static_cast<const C*>(dp.wallspec) + i * PS + idc;
          x = zmk((double)p[0].x, (double)p[0].y);
          y = zmk((double)p[PS].x, (double)p[PS].y);
        }
        if (zero) {
          const double nxy = (double)dp.Nx * (double)dp.Ny;
          x = zmk(fma(nxy, w[0], x.x), 0);
          y = zmk(fma(nxy, w[1], y.x), 0);
        }
        const double c = dp.eta * cWU;              // cU
        x = c * x;
        y = c * y;
        wu = imag ? cx * x.x + cy * y.x : -(cx * x.y + cy * y.y);
        wt = imag ? cx * y.y - cy * x.y : cx * y.x - cy * x.x;
      };
      if (zero_grp || dp.wallspec) {
        wall(0, dp.wall0, wU0, wT0);
        if constexpr (GEOM == 1) wall(2, dp.wallH, wUH, wTH);
      }
    }
    // (the k = 0 column has its own first coefficients)
    auto solve = [&](double* y, double g, double g0, double gH) {
      op.solve(fresh(tabs, toff), y, g, up);
      if (zero_grp) {
        const double y0 = y[0];
        zero_mode<NA, GEOM>(fresh(tabs, toff), y, up, l0 * s2H, lH * s2H, g0, gH);
        y[0] = zero ? y[0] : y0;
      }
    };
    // F_z of the low-wavenumber square: FP64 coefficients from the apply's
    // FP64 route, or (stage entry point, no such route) from an FP64 transform
    // of the input's band values
    auto low_fz = [&](double* f) {
#pragma unroll
      for (int i = 0; i < NA; ++i) f[i] = (double)aZ[i];
      if (lcol >= 0) {
        if (dp.lowk_coef) {
          const double* e = reinterpret_cast<const double*>(dp.lowk_coef + (size_t)lcol * N);
#pragma unroll
          for (int i = 0; i < NA; ++i) {
            const int n = 2 * i + (up ? 1 : 0);
            f[i] = n < N ? e[2 * n + (imag ? 1 : 0)] : 0.0;
          }
        } else {
#pragma unroll
          for (int i = 0; i < NA; ++i) f[i] = 0.0;
          for (int c = lo; c <= hi; ++c) {
            const C t = in[((size_t)2 * N + c) * PS + idc];
            const double v = (double)(imag ? t.y : t.x);
#pragma unroll
            for (int i = 0; i < NA; ++i) {
              const int n = 2 * i + (up ? 1 : 0);
              if (n < N) f[i] = fma(cp.dctf[c * N + n], v, f[i]);
            }
          }
        }
      }
    };
    double U[NA], W[NA], Y[NA];                     // U holds p first
    {
      const double f = 0.25 * H * k;
      add_b2<NA, true, false>(fresh(tabs, toff), [&](int i) { return f * (double)aL[i]; }, up,
                              U);
    }
    if constexpr (LOW) {
      double f[NA];
      low_fz(f);
      add_b<NA, false, false>(fresh(tabs, toff), [&](int i) { return f[i]; }, up, xaddr, U);
    } else {
      add_b<NA, false, false>(fresh(tabs, toff), [&](int i) { return aZ[i]; }, up, xaddr, U);
    }
    op.prepare(fresh(tabs, toff), k2, kappa, up);
    solve(U, 0.0, 0.0, 0.0);
    const double pS = own_sum<NA>(U), pO = across(pS, pS, up);
    // W
    add_b<NA, true, false>(fresh(tabs, toff), [&](int i) { return U[i]; }, up, xaddr, W);
    {
      const double fz = 0.25 * kappa * kappa, fg = fz * k;
      auto force = [&](double z, int i) {
        if constexpr (TIN) return fma(fg, (double)aG[i], fz * z);
        else return fz * z;
      };
      if constexpr (LOW) {
        double f[NA];
        low_fz(f);
        add_b2<NA, false, true>(fresh(tabs, toff), [&](int i) { return force(f[i], i); }, up,
                                W);
      } else {
        add_b2<NA, false, true>(fresh(tabs, toff),
                                [&](int i) { return force((double)aZ[i], i); }, up, W);
      }
      solve(W, fz * pO, 0.0, 0.0);
    }
    if (zero_grp) {
#pragma unroll
      for (int i = 0; i < NA; ++i) W[i] = zero ? 0.0 : W[i];
    }
    // U, in place of p (each row after its last use)
    {
      const double fp = zero ? 0.0 : ik, fl = 0.25 * H;
      add_b2<NA, true, true>(
          fresh(tabs, toff), [&](int i) { return fma(fp, U[i], fl * (double)aL[i]); }, up, U);
      if constexpr (TIN)
        add_b<NA, false, false>(fresh(tabs, toff), [&](int i) { return aG[i]; }, up, xaddr, U);
      solve(U, fl * pS, wU0, wUH);
    }
    // T
    if constexpr (sizeof(D) == 8) {
      forward(No{}, Yes{});
    } else {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        aT[i] = park[i * 64];
        if constexpr (TIN) aH[i] = park[(NA + i) * 64];
      }
    }
    {
      const double ft = 0.25 * H;
      add_b2<NA, true, true>(fresh(tabs, toff), [&](int i) { return ft * (double)aT[i]; }, up,
                             Y);
      if constexpr (TIN)
        add_b<NA, false, true>(fresh(tabs, toff), [&](int i) { return aH[i]; }, up, xaddr, Y);
      solve(Y, 0.0, wT0, wTH);
    }

    // --- wall correction -------------------------------------------------------------
    // adds the node functions E = e^{kap (z - z0)} and Z = z E, transformed in
    // B's type: U += Z zU + E eU, W += Z zW + E eW, T += E eT.  They are real,
    // so both sets of the exchange are the same.
    auto basis = [&](auto type, double z0, double kap, double zU, double zW, double eU,
                     double eW, double eT) {
      using B = decltype(type);
      using MB = Mat<B>;
      typename MB::acc acc[2][NT];
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0][t][e] = acc[1][t][e] = B(0);
#pragma unroll
      for (int s = 0; s < kHalf; ++s) {
        if (4 * s >= N) break;                      // uniform
        __builtin_amdgcn_sched_barrier(0);
        const int c = 4 * s + (ln >> 4);
        B z, a[NT];
        if constexpr (sizeof(B) == sizeof(D)) {
          z = zn[c];                                // (zero rows past the nodes)
#pragma unroll
          for (int t = 0; t < NT; ++t) a[t] = mf[(t * kHalf + s) * 64 + ln];
        } else {
          z = c < N ? zc[c] : B(0);
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const int row = ln & 15, g = MB::group(row), j = 4 * t + MB::reg(row);
            const int n = 2 * ((g & 1) * kHalf + j) + (g >> 1);
            a[t] = (j < kHalf && n < N && c < N) ? cp.dctf[c * N + n] : B(0);
          }
        }
        const B f = exp((B)kap * (z - (B)z0)), zf = z * f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          acc[0][t] = MB::mma(a[t], f, acc[0][t]);
          acc[1][t] = MB::mma(a[t], zf, acc[1][t]);
        }
      }
#pragma unroll
      for (int j = 0; j < kHalf; ++j) {
        B e0 = acc[0][j / 4][j % 4], e1 = e0, q0 = acc[1][j / 4][j % 4], q1 = q0;
        swap16(e0, e1);
        swap16(q0, q1);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int i = j + h * kHalf;
          const double E = (double)(h ? e1 : e0), Z = (double)(h ? q1 : q0);
          U[i] = fma(E, eU, fma(Z, zU, U[i]));
          W[i] = fma(E, cWU * eW, fma(Z, cWU * zW, W[i]));
          Y[i] = fma(E, eT, Y[i]);
        }
      }
    };
    // boundary data u^W - u_DP at the walls, plus the slip terms (App. A)
    double tU, tW, tT, bU, bW, bT;
    wall_sums<NA>(U, up, tU, bU);
    wall_sums<NA>(W, up, tW, bW);
    wall_sums<NA>(Y, up, tT, bT);
    double U0 = wU0 - bU, T0 = wT0 - bT, UH = wUH - tU, TH = wTH - tT;
    const double w0 = -cUW * bW, wH = -cUW * tW;    // (in the units of U)
    if (slip) {
      double dt, db;
      wall_dsums<NA>(fresh(tabs, toff), U, up, dt, db);
      U0 += l0 * s2H * db;
      UH -= lH * s2H * dt;
      wall_dsums<NA>(fresh(tabs, toff), Y, up, dt, db);
      T0 += l0 * s2H * db;
      TH -= lH * s2H * dt;
    }
    const double p0 = kp * l0, pH = kp * lH;
    const double i0 = frcp(1.0 + 2.0 * p0);
    if constexpr (GEOM == 0) {
      // i u_L = B z e^{-kz} + C e^{-kz}, w = B z e^{-kz} + w_0 e^{-kz}, with
      // B = k ((1 + k l_0) w_0 - U_0) / (1 + 2 k l_0), C = (U_0 + l_0 B) /
      // (1 + k l_0); u_T = T_0 / (1 + k l_0) e^{-kz}
      double B = kp * i0 * fma(1.0 + p0, w0, -U0);
      const double i1 = frcp(1.0 + p0);
      double CU = i1 * (U0 + l0 * B), CT = i1 * T0, CW = w0;
      if (zero) B = CU = CT = CW = 0.0;
      basis(D(0), 0.0, -kp, B, B, CU, CW, CT);
    } else {
      // Unknowns g = C_0 / (2 eta k), h = D_0~ / (2 eta k) of the pressure
      // part and C_z, D_z~: continuity at the two walls gives i C_L = C_z - g,
      // i D_L~ = -D_z~ - h exactly, w(0) = w_0 gives C_z = w_0 - E D_z~, the
      // slip row at z = 0 gives g; what is left are two rows (w and i u_L at
      // z = H) for D_z~ and h.  Without slip their determinant is
      // 4 q^2 E^2 - s^2, taken without cancellation (q = kH, s = 1 - E^2).
      const double q = kp * H;
      double E, s, ex;
      wall_decay((LdsPtr)fact, q, E, s, ex);
      const double E2 = E * E;
      const double r0 = i0 * (1.0 - 2.0 * p0);
      const double gam = q * (1.0 - pH) - (1.0 - 2.0 * pH);
      const double G0 = i0 * fma(1.0 + p0, w0, -U0);
      const double a11 = fma(-2.0 * q * i0, E2, s), a12 = q * fma(-E2, r0, 1.0);
      const double a21 = -fma(2.0 * gam * i0, E2, 1.0 + E2 + pH * s);
      const double a22 = -fma(E2 * gam, r0, q * (1.0 + pH) + 1.0 + 2.0 * pH);
      const double b1 = fma(-q * E, G0, fma(-E, w0, wH));
      const double b2 = fma(-E * gam, G0, fma(-E * (1.0 - pH), w0, UH));
      const double det = slip ? fma(a11, a22, -(a12 * a21))
                              : -ex * fma(2.0 * q, E, s);
      const double id = frcp(det);
      double Dz = id * fma(b1, a22, -(b2 * a12)), h = id * fma(a11, b2, -(a21 * b1));
      double g = fma(-E * r0, h, fma(-2.0 * E * i0, Dz, G0));
      double Cz = fma(-E, Dz, w0);
      // across k: (1 + k l0) C_T + (1 - k l0) E D_T = T_0, E (1 - k lH) C_T +
      // (1 + k lH) D_T = T_H
      const double it = frcp((1.0 + p0) * (1.0 + pH) - (1.0 - p0) * (1.0 - pH) * E2);
      double CT = it * ((1.0 + pH) * T0 - (1.0 - p0) * E * TH);
      double DT = it * ((1.0 + p0) * TH - E * (1.0 - pH) * T0);
      if (zero) Dz = h = g = Cz = CT = DT = 0.0;
      const double CU = Cz - g, DU = -Dz - h, kg = kp * g, kh = kp * h;
      if constexpr (LOW) {
        // low-wavenumber square: node functions and transform in FP64 (their
        // combination cancels strongly as kH -> 0)
        basis(0.0, 0.0, -kp, kg, kg, CU, Cz, CT);
        basis(0.0, H, kp, -kh, kh, DU, Dz, DT);
      } else {
        basis(D(0), 0.0, -kp, kg, kg, CU, Cz, CT);
        basis(D(0), H, kp, -kh, kh, DU, Dz, DT);
      }
    }

    // --- inverse transform to the band nodes ---------------------------------------
    // vectors: U, W, T and, for the vorticity, (1/2)(k W + U') and -(1/2) T'.  With
    // FP32 transforms they leave their units and take the output's scale here, in
    // FP64: the factors go with the fourth power of a length and 1 / eta (1e36 H^2
    // / (Nx Ny eta) in the mean flow, whose k is a stand-in), beyond FP32 for legal
    // boxes.  With FP64 transforms the nodes take them: 64 nodes, one wall, 303 us
    // at 256^2 against 345 (more registers spilled).
    constexpr int kV = WOUT ? 5 : 3;
    constexpr bool kCoef = sizeof(D) == 4;
    const double su = cp.scale * cUW, sw = su * cUW;   // (scale holds 1 / eta)
    const double au = kCoef ? su : 1.0, aw = kCoef ? sw : 1.0;
    D cf[kV][NA];
    if constexpr (WOUT) {
      const double sd = s2H * au;                      // (1/2)(4/H)
      derivative<NA, D>(fresh(tabs, toff), U, up, xaddr, sd, cf[3]);
      derivative<NA, D>(fresh(tabs, toff), Y, up, xaddr, -sd, cf[4]);
      const double hw = 0.5 * k * (kCoef ? sw : cUW);
#pragma unroll
      for (int i = 0; i < NA; ++i) cf[3][i] += (D)(hw * W[i]);
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      cf[0][i] = (D)(au * U[i]);
      cf[1][i] = (D)(aw * W[i]);
      cf[2][i] = (D)(au * Y[i]);
    }
#pragma unroll
    for (int v = 0; v < kV; ++v)
#pragma unroll
      for (int j = 0; j < kHalf; ++j) swap16(cf[v][j], cf[v][kHalf + j]);
    const double nu = kCoef ? 1.0 : su;
    const D nw = kCoef ? D(1) : (D)sw;
    const D ox = (D)(nu * cx), oy = (D)(nu * cy), hk = (D)(0.5 * k * nu);
    auto store = [&](int c, const D (&re)[kV], const D (&im)[kV]) {
      if (c <= hi && valid) {
        C* dst = out + (size_t)c * PS + idx;
        auto put = [&](int ch, D r, D i) {
          C o;
          o.x = nyq ? T(0) : (T)r;
          o.y = nyq ? T(0) : (T)i;
          dst[(size_t)ch * N * PS] = o;
        };
        // u_L = -i U, omega_T = -i (i omega_T)
        const D lr = im[0], li = -re[0], tr = re[2], ti = im[2];
        put(0, fma(ox, lr, -(oy * tr)), fma(ox, li, -(oy * ti)));
        put(1, fma(oy, lr, ox * tr), fma(oy, li, ox * ti));
        put(2, nw * re[1], nw * im[1]);
        if constexpr (WOUT) {
          const D qr = im[3], qi = -re[3], pr = re[4], pim = im[4];
          put(3, fma(ox, pr, -(oy * qr)), fma(ox, pim, -(oy * qi)));
          put(4, fma(oy, pr, ox * qr), fma(oy, pim, ox * qi));
          put(5, -hk * ti, hk * tr);
        }
      }
    };
    for (int t = 0; t < tiles; ++t) {
      Acc acc[kV][2];
#pragma unroll
      for (int v = 0; v < kV; ++v) acc[v][0] = acc[v][1] = Acc{0, 0, 0, 0};
#pragma unroll
      for (int j = 0; j < kHalf; ++j) {
        const D a = pi[(t * kHalf + j) * 64 + ln];
#pragma unroll
        for (int v = 0; v < kV; ++v) {
          acc[v][0] = M::mma(a, cf[v][j], acc[v][0]);
          acc[v][1] = M::mma(a, cf[v][kHalf + j], acc[v][1]);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        D re[kV], im[kV];
#pragma unroll
        for (int v = 0; v < kV; ++v) {
          re[v] = acc[v][0][r];
          im[v] = acc[v][1][r];
        }
        store(lo + 16 * t + M::row(g4, r), re, im);
      }
    }
    if constexpr (kTail) {
      if (tail) {
        // the last one to four nodes: sixteen 4 x 4 products of one
        // coefficient each (a lane's block uses its own coefficients, a
        // quarter of the series), then the four lane groups' sums are added so
        // that group g keeps node g -- an eighth of the tile's matrix cycles
        f4v acc[kV][2];
#pragma unroll
        for (int v = 0; v < kV; ++v) acc[v][0] = acc[v][1] = f4v{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < kHalf; ++j) {
          const float a = pi[(tiles * kHalf + j) * 64 + ln];
#pragma unroll
          for (int v = 0; v < kV; ++v) {
            acc[v][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, cf[v][j], acc[v][0], 0, 0, 0);
            acc[v][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, cf[v][kHalf + j], acc[v][1],
                                                           0, 0, 0);
          }
        }
        auto gather = [&](const f4v& x) {
          float a = x[0], b = x[1], c = x[2], d = x[3];
          swap16(a, b);
          swap16(c, d);
          const float e = a + b, f = c + d;          // nodes 0, 1 and 2, 3
          const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(e),
                                                          __float_as_uint(f), false, false);
          return __uint_as_float(q[0]) + __uint_as_float(q[1]);
        };
        D re[kV], im[kV];
#pragma unroll
        for (int v = 0; v < kV; ++v) {
          re[v] = gather(acc[v][0]);
          im[v] = gather(acc[v][1]);
        }
        store(lo + 16 * tiles + g4, re, im);
      }
    }
  }
  };
  if (kLow && (int)blockIdx.x < low_blocks) {
    if constexpr (kLow) run(std::integral_constant<bool, true>{});
  } else {
    run(std::integral_constant<bool, false>{});
  }
}

template <typename T, typename D, int NT, int NA, int GEOM, bool TIN, bool WOUT>
static void launch_one(const fcmdp_solver* s, const ColParams& cp, const void* in,
                       void* out, hipStream_t st) {
  using C = cplx_t<T>;
  const int G = (s->dp.Nkx * s->dp.Ny + 15) / 16;
  // as many workgroups as stay resident (registers: two per CU with FP32
  // transforms, one with FP64), each looping over column groups
  const int most = std::max(1, s->num_cu) * (sizeof(D) == 4 ? 2 : 1);
  // one wavefront per group of the low-wavenumber columns: ns + 2 ranges of
  // 2 ns + 1 columns
  const int ns = s->dp.lowk_ns;
  const int low = ns < 0 ? 0 : ((ns + 2) * (ns / 8 + 2) + 3) / 4;
  hipLaunchKernelGGL((k_columns_mfma<T, D, NT, NA, GEOM, TIN, WOUT>),
                     dim3(std::min((G + 3) / 4, most) + low), dim3(256), 0, st, cp, low,
                     s->band, (const C*)in, (C*)out, s->zc, s->dct_f, s->dct_i);
}
template <typename T, typename D, int NT, int NA, int GEOM>
static void launch_channels(const fcmdp_solver* s, const ColParams& cp, const void* in,
                            void* out, hipStream_t st) {
  const bool tin = s->dp.nch_in == 6, wout = s->dp.nch_out == 6;
  if (tin && wout) launch_one<T, D, NT, NA, GEOM, true, true>(s, cp, in, out, st);
  else if (tin) launch_one<T, D, NT, NA, GEOM, true, false>(s, cp, in, out, st);
  else if (wout) launch_one<T, D, NT, NA, GEOM, false, true>(s, cp, in, out, st);
  else launch_one<T, D, NT, NA, GEOM, false, false>(s, cp, in, out, st);
}
template <typename T, typename D, int NT, int NA>
static void launch_geometry(const fcmdp_solver* s, const ColParams& cp, const void* in,
                            void* out, hipStream_t st) {
  if (s->dp.geometry == 1) launch_channels<T, D, NT, NA, 1>(s, cp, in, out, st);
  else launch_channels<T, D, NT, NA, 0>(s, cp, in, out, st);
}

hipError_t launch_columns_mfma(const fcmdp_solver* s, const void* spec_in,
                               void* spec_out, hipStream_t st) {
  ColParams cp;
  cp.dp = s->dp;
  cp.scale = 1.0 / ((double)s->dp.Nx * (double)s->dp.Ny * s->dp.eta);
  cp.kxs = 2.0 * M_PI / s->dp.Lx;
  cp.kys = 2.0 * M_PI / s->dp.Ly;
  cp.dctf = s->dct_f;
  cp.iH = 1.0 / s->dp.H;
  cp.s2H = 2.0 / s->dp.H;
  // the smallest half-length that holds ceil(Nz / 2) coefficients per parity:
  // 10 for the 19 nodes of a 2700^2 layer, FP32 data; 16 would sweep 60% more
  const int Nz = s->dp.Nz;
  if (s->mixed && Nz <= 32 && !s->force_vector_dct) {
    if (Nz <= 20) launch_geometry<float, float, 2, 10>(s, cp, spec_in, spec_out, st);
    else launch_geometry<float, float, 2, 16>(s, cp, spec_in, spec_out, st);
  } else if (s->mixed) {
    if (Nz <= 32) launch_geometry<float, double, 2, 16>(s, cp, spec_in, spec_out, st);
    else if (Nz <= 48) launch_geometry<float, double, 3, 24>(s, cp, spec_in, spec_out, st);
    else launch_geometry<float, double, 4, 32>(s, cp, spec_in, spec_out, st);
  } else {
    if (Nz <= 20) launch_geometry<double, double, 2, 10>(s, cp, spec_in, spec_out, st);
    else if (Nz <= 32) launch_geometry<double, double, 2, 16>(s, cp, spec_in, spec_out, st);
    else if (Nz <= 48) launch_geometry<double, double, 3, 24>(s, cp, spec_in, spec_out, st);
    else launch_geometry<double, double, 4, 32>(s, cp, spec_in, spec_out, st);
  }
  return hipGetLastError();
}

}  // namespace fcmdp

// Complex helpers, small DFTs held in registers and the split steps of the real
// transforms, shared by the FFT kernels.
#pragma once

#include "fcmdp_internal.h"

namespace fcmdp {

// offsets of the primes' cos / sin tables
struct DftOff { int off[32]; };

template <typename C> __device__ inline C cmul(C a, C b) {
  C r;
  r.x = a.x * b.x - a.y * b.y;
  r.y = a.x * b.y + a.y * b.x;
  return r;
}
template <typename C> __device__ inline C cadd(C a, C b) {
  C r; r.x = a.x + b.x; r.y = a.y + b.y; return r;
}
template <typename C> __device__ inline C csub(C a, C b) {
  C r; r.x = a.x - b.x; r.y = a.y - b.y; return r;
}
// multiply by (sign * i)
template <typename C, typename T> __device__ inline C cmul_si(C a, T sign) {
  C r; r.x = -sign * a.y; r.y = sign * a.x; return r;
}
template <typename C, typename T> __device__ inline C cscale(C a, T s) {
  C r; r.x = a.x * s; r.y = a.y * s; return r;
}

// ---- small DFTs: y_k = sum_q v_q e^{sign 2 pi i q k / R} --------------------
template <typename T, typename C>
__device__ inline void dft2(C* v) {
  const C a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}

template <typename T, typename C>
__device__ inline void dft4(C* v, T sign) {
  const C s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
  const C s13 = cadd(v[1], v[3]), d13 = cmul_si<C, T>(csub(v[1], v[3]), sign);
  v[0] = cadd(s02, s13);
  v[2] = csub(s02, s13);
  v[1] = cadd(d02, d13);
  v[3] = csub(d02, d13);
}

template <typename T, typename C>
__device__ inline void dft8(C* v, T sign) {
  C e[4] = {v[0], v[2], v[4], v[6]};
  C o[4] = {v[1], v[3], v[5], v[7]};
  dft4<T, C>(e, sign);
  dft4<T, C>(o, sign);
  const T r = T(0.70710678118654752440084436210484903928);
  C w1; w1.x = r; w1.y = sign * r;
  C w3; w3.x = -r; w3.y = sign * r;
  const C t0 = o[0];
  const C t1 = cmul(o[1], w1);
  const C t2 = cmul_si<C, T>(o[2], sign);
  const C t3 = cmul(o[3], w3);
  v[0] = cadd(e[0], t0); v[4] = csub(e[0], t0);
  v[1] = cadd(e[1], t1); v[5] = csub(e[1], t1);
  v[2] = cadd(e[2], t2); v[6] = csub(e[2], t2);
  v[3] = cadd(e[3], t3); v[7] = csub(e[3], t3);
}

// radix 16 as two radix-8 halves (even / odd inputs) and one twiddled
// radix-2 combination
template <typename T, typename C>
__device__ inline void dft16(C* v, T sign) {
  C e[8], o[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) { e[m] = v[2 * m]; o[m] = v[2 * m + 1]; }
  dft8<T, C>(e, sign);
  dft8<T, C>(o, sign);
  // cos and sin of pi k / 8, k = 0..7
  const T c[8] = {T(1), T(0.92387953251128675613), T(0.70710678118654752440),
                  T(0.38268343236508977173), T(0), T(-0.38268343236508977173),
                  T(-0.70710678118654752440), T(-0.92387953251128675613)};
  const T sn[8] = {T(0), T(0.38268343236508977173), T(0.70710678118654752440),
                   T(0.92387953251128675613), T(1), T(0.92387953251128675613),
                   T(0.70710678118654752440), T(0.38268343236508977173)};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    C w; w.x = c[k]; w.y = sign * sn[k];
    const C t = cmul(o[k], w);
    v[k] = cadd(e[k], t);
    v[k + 8] = csub(e[k], t);
  }
}

// odd prime P: pair terms j and P-j; cs[2m], cs[2m+1] = cos, sin(2 pi m/P)
template <typename T, typename C, int P>
__device__ inline void dft_prime(C* v, const T* cs, T sign) {
  constexpr int Hh = (P - 1) / 2;
  C a[Hh], b[Hh];
  C y0 = v[0];
#pragma unroll
  for (int j = 1; j <= Hh; ++j) {
    a[j - 1] = cadd(v[j], v[P - j]);
    b[j - 1] = csub(v[j], v[P - j]);
    y0 = cadd(y0, a[j - 1]);
  }
  C out[P];
  out[0] = y0;
#pragma unroll
  for (int k = 1; k <= Hh; ++k) {
    C A = v[0];
    C B; B.x = T(0); B.y = T(0);
#pragma unroll
    for (int j = 1; j <= Hh; ++j) {
      const int m = (j * k) % P;
      const T c = cs[2 * m], s = cs[2 * m + 1];
      A.x += a[j - 1].x * c; A.y += a[j - 1].y * c;
      B.x += b[j - 1].x * s; B.y += b[j - 1].y * s;
    }
    const C iB = cmul_si<C, T>(B, sign);
    out[k] = cadd(A, iB);
    out[P - k] = csub(A, iB);
  }
#pragma unroll
  for (int k = 0; k < P; ++k) v[k] = out[k];
}

// R1 R2 coprime points by the prime-factor map: input n = R2 n1 + R1 n2,
// output k with k = k1 mod R1, k = k2 mod R2; no twiddles.
template <typename T, typename C, int R1, int R2>
__device__ inline void dft_pfa(C* v, T sign);

// cos, sin (2 pi m / P) for the small odd factors
template <typename T, int P> struct OddTable;
template <typename T> struct OddTable<T, 3> {
  static constexpr T cs[6] = {T(1), T(0), T(-0.5), T(0.86602540378443864676),
                              T(-0.5), T(-0.86602540378443864676)};
};
template <typename T> struct OddTable<T, 5> {
  static constexpr T cs[10] = {
      T(1), T(0), T(0.30901699437494742410), T(0.95105651629515357212),
      T(-0.80901699437494742410), T(0.58778525229247312917),
      T(-0.80901699437494742410), T(-0.58778525229247312917),
      T(0.30901699437494742410), T(-0.95105651629515357212)};
};
template <typename T> struct OddTable<T, 7> {
  static constexpr T cs[14] = {
      T(1), T(0), T(0.62348980185873353053), T(0.78183148246802980871),
      T(-0.22252093395631440429), T(0.97492791218182360702),
      T(-0.90096886790241912624), T(0.43388373911755812048),
      T(-0.90096886790241912624), T(-0.43388373911755812048),
      T(-0.22252093395631440429), T(-0.97492791218182360702),
      T(0.62348980185873353053), T(-0.78183148246802980871)};
};

// R points; cs: run-time table of the primes 11, 13, 17
template <typename T, typename C, int R>
__device__ __forceinline__ void dft_any(C* v, const T* __restrict__ cs, T sign) {
  if constexpr (R == 2) dft2<T, C>(v);
  else if constexpr (R == 3 || R == 5 || R == 7) dft_prime<T, C, R>(v, OddTable<T, R>::cs, sign);
  else if constexpr (R == 4) dft4<T, C>(v, sign);
  else if constexpr (R == 8) dft8<T, C>(v, sign);
  else if constexpr (R == 16) dft16<T, C>(v, sign);
  else if constexpr (R == 6) dft_pfa<T, C, 2, 3>(v, sign);
  else if constexpr (R == 10) dft_pfa<T, C, 2, 5>(v, sign);
  else if constexpr (R == 12) dft_pfa<T, C, 4, 3>(v, sign);
  else if constexpr (R == 14) dft_pfa<T, C, 2, 7>(v, sign);
  else if constexpr (R == 15) dft_pfa<T, C, 3, 5>(v, sign);
  else if constexpr (R == 9) {
    // 3 x 3: columns n mod 3, twiddles e^{sign 2 pi i n k / 9}, rows
    constexpr T c1 = T(0.76604444311897803520), s1 = T(0.64278760968653932632);
    constexpr T c2 = T(0.17364817766693034885), s2 = T(0.98480775301220805937);
    constexpr T c4 = T(-0.93969262078590838405), s4 = T(0.34202014332566873304);
    C x[3][3];
#pragma unroll
    for (int n = 0; n < 3; ++n) {
#pragma unroll
      for (int m = 0; m < 3; ++m) x[n][m] = v[n + 3 * m];
      dft_prime<T, C, 3>(x[n], OddTable<T, 3>::cs, sign);
    }
    auto tw = [&](C& a, T c, T s) {
      C w; w.x = c; w.y = sign * s;
      a = cmul(a, w);
    };
    tw(x[1][1], c1, s1); tw(x[1][2], c2, s2);
    tw(x[2][1], c2, s2); tw(x[2][2], c4, s4);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      C y[3] = {x[0][k], x[1][k], x[2][k]};
      dft_prime<T, C, 3>(y, OddTable<T, 3>::cs, sign);
#pragma unroll
      for (int q = 0; q < 3; ++q) v[k + 3 * q] = y[q];
    }
  } else {
    dft_prime<T, C, R>(v, cs, sign);
  }
}

template <typename T, typename C, int R1, int R2>
__device__ inline void dft_pfa(C* v, T sign) {
  constexpr int R = R1 * R2;
  C x[R2][R1];
#pragma unroll
  for (int n2 = 0; n2 < R2; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) x[n2][n1] = v[(R2 * n1 + R1 * n2) % R];
    dft_any<T, C, R1>(x[n2], nullptr, sign);
  }
#pragma unroll
  for (int k1 = 0; k1 < R1; ++k1) {
    C y[R2];
#pragma unroll
    for (int n2 = 0; n2 < R2; ++n2) y[n2] = x[n2][k1];
    dft_any<T, C, R2>(y, nullptr, sign);
#pragma unroll
    for (int k = 0; k < R; ++k)
      if (k % R1 == k1) v[k] = y[k % R2];
  }
}

// split step of the real transform: X_k from Z_k and Z_{M-k} (w = e^{-2 pi i k/Nx})
template <typename C>
__device__ inline C r2c_post(C zk, C zm, C w) {
  using T = decltype(zk.x);
  zm.y = -zm.y;
  const C e = cscale(cadd(zk, zm), T(0.5));
  const C d = csub(zk, zm);
  C o; o.x = T(0.5) * d.y; o.y = T(-0.5) * d.x;      // -i d / 2
  return cadd(e, cmul(w, o));
}

// inverse split step: Z_k from X_k and X_{M-k} (w = e^{-2 pi i k/Nx})
template <typename C>
__device__ inline C c2r_pre(C xk, C xm, C w) {
  xm.y = -xm.y;                                   // conj(X_{M-k})
  const C A = cadd(xk, xm);
  const C B = csub(xk, xm);
  w.y = -w.y;                                     // e^{+2 pi i k/Nx}
  const C wb = cmul(w, B);
  C z; z.x = A.x - wb.y; z.y = A.y + wb.x;        // A + i w B
  return z;
}

}  // namespace fcmdp

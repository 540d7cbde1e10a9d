// Row transforms of any supported length, both precisions: the x- and y-passes
// of lengths without a fixed plan, and in FP64 all but small grids (fft.hip).
//
// A workgroup owns a batch of rows in LDS and steps through a run-time plan of
// few, large radices (at most 16 in FP32, 12 in FP64, and the primes 11, 13,
// 17; 360 = 9 8 5, 768 = 12 8 8): every stage costs a round trip through LDS
// and a barrier, so two or three stages of composite radices instead of four
// to six small ones are what shortens a batch.  A stage's butterflies are
// dealt to the threads across all rows of the batch (short rows keep whole
// wavefronts busy), read into registers, and written back in place, so that
// one buffer holds the batch and more workgroups fit on a CU than with two.
// Twiddles are stored per stage as [q][k], the order in which the lanes read
// them.  Bound by latency (LDS round trips and barriers), which the other
// workgroups of the CU hide; measured against the run-time plans with a
// gathered twiddle per butterfly input and one wavefront per row (FP32) or two
// buffers and radices up to 8 (FP64), forward x / y / inverse x in us: 360
// points FP32 80/61/86 -> 39/37/43, 756 x 442 172/138/171 -> 116/87/110, 1176
// 463/329/482 -> 310/261/255, 768 FP64 775/630/820 -> 439/324/436.  The fixed
// plans of fft.hip, one wavefront per row without barriers, stay for their
// lengths (forward, fixed against run-time, with the full batches that rows of
// 1280 to 2548 points in x now keep: 2176 points 2.34 / 4.4 ms, 768 0.28 / 0.48,
// 2700 1.50 / 2.61).
#include <algorithm>
#include <cmath>

#include "dft.h"
#include "fcmdp_internal.h"

namespace fcmdp {

// elements of a row batch that a thread may hold
constexpr int row_cap(bool fp32, int R) {
  return (fp32 ? 32 : 16) / R < 1 ? 1 : (fp32 ? 32 : 16) / R > 8 ? 8 : (fp32 ? 32 : 16) / R;
}

// idx / d for idx < 2^16, d < 2^15 by a multiplication (m = ceil(2^32 / d),
// 0 for d = 1)
__device__ __forceinline__ int quick_div(int idx, unsigned m) {
  return m ? (int)__umulhi((unsigned)idx, m) : idx;
}
static unsigned quick_mul(int d) { return d == 1 ? 0u : (unsigned)((0x100000000ull + d - 1) / d); }

template <typename T, int R>
__device__ __forceinline__ void row_stage(cplx_t<T>* lds, int S, int rows, const RowPlan& pl,
                                          int s, const cplx_t<T>* __restrict__ tws,
                                          const T* __restrict__ cs, T sign) {
  using C = cplx_t<T>;
  constexpr int NB = row_cap(sizeof(T) == 4, R);
  const int nb = pl.n / R, Ns = pl.ns[s], total = rows * nb;
  const unsigned mnb = pl.mnb[s], mns = pl.mns[s];
  const C* tw = tws + pl.tw[s];
  C v[NB][R];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int idx = threadIdx.x + i * blockDim.x;
    if (idx < total) {
      const int r = quick_div(idx, mnb);
      const C* src = lds + r * (S - nb) + idx;       // row r, butterfly idx - r nb
#pragma unroll
      for (int q = 0; q < R; ++q) v[i][q] = src[q * nb];
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int idx = threadIdx.x + i * blockDim.x;
    if (idx < total) {
      const int r = quick_div(idx, mnb), j = idx - r * nb;
      const int k = j - quick_div(j, mns) * Ns;
      if (s > 0) {
#pragma unroll
        for (int q = 1; q < R; ++q) {
          C w = tw[(q - 1) * Ns + k];
          w.y *= -sign;                              // the table is for sign = -1
          v[i][q] = cmul(v[i][q], w);
        }
      }
      dft_any<T, C, R>(v[i], cs, sign);
      C* dst = lds + r * S + (j - k) * R + k;
#pragma unroll
      for (int q = 0; q < R; ++q) dst[q * Ns] = v[i][q];
    }
  }
  __syncthreads();
}

// transforms `rows` rows of stride S; the caller has synchronised
template <typename T>
__device__ __forceinline__ void row_plan(cplx_t<T>* lds, int S, int rows, const RowPlan& pl,
                                         const cplx_t<T>* __restrict__ tws,
                                         const T* __restrict__ dftc, const DftOff& doff,
                                         T sign) {
  for (int s = 0; s < pl.nst; ++s) {
    const int R = pl.radix[s];
    const T* cs = dftc + doff.off[R];
    switch (R) {
#define FCMDP_STAGE(r) \
  case r: row_stage<T, r>(lds, S, rows, pl, s, tws, cs, sign); break;
      FCMDP_STAGE(2) FCMDP_STAGE(3) FCMDP_STAGE(4) FCMDP_STAGE(5) FCMDP_STAGE(6)
      FCMDP_STAGE(7) FCMDP_STAGE(8) FCMDP_STAGE(9) FCMDP_STAGE(10) FCMDP_STAGE(11)
      FCMDP_STAGE(12) FCMDP_STAGE(13) FCMDP_STAGE(17)
      default:
        if constexpr (sizeof(T) == 4) {
          switch (R) { FCMDP_STAGE(14) FCMDP_STAGE(15) FCMDP_STAGE(16) default: break; }
        }
        break;
#undef FCMDP_STAGE
    }
  }
}

// Row batch of workgroup b of n in an x-pass whose transposed runs are half a
// 128-byte line: workgroups b and b + 8, which run on the same XCD one after
// the other, take neighbouring batches, so that both halves of a line meet in
// that XCD's L2.
__device__ __forceinline__ int paired_batch(int b, int n) {
  const int q = b & ~15, r = b & 15;
  return q + 16 <= n ? q + 2 * (r & 7) + (r >> 3) : b;
}

struct RowArgs {
  int Nx, Ny, Nz, Nkx, rows;
  unsigned m_rows, m_len, m_half;   // quick divisors: rows (or row pairs), M, M / 2 + 1
};

// x-pass, real rows -> half spectrum, written transposed (`rows` consecutive y
// per kx)
template <typename T>
__global__ void __launch_bounds__(1024)
k_rows_x_r2c(RowArgs ra, RowPlan pl, const int* __restrict__ band, const T* __restrict__ grid,
             cplx_t<T>* __restrict__ spec, const cplx_t<T>* __restrict__ tws,
             const cplx_t<T>* __restrict__ rtw, const T* __restrict__ dftc, DftOff doff) {
  using C = cplx_t<T>;
  extern __shared__ unsigned char lds_raw[];
  C* lds = reinterpret_cast<C*>(lds_raw);
  const int p = blockIdx.y, c = p % ra.Nz;
  if (c < band[0] || c > band[1]) return;
  const int M = ra.Nx / 2, S = (M + 1) | 1, rows = ra.rows, nt = blockDim.x;
  const int yb = rows * (int)sizeof(C) == 64 ? paired_batch(blockIdx.x, gridDim.x) : blockIdx.x;
  const int y0 = yb * rows, nr = min(rows, ra.Ny - y0);
  const C* src = reinterpret_cast<const C*>(grid + ((size_t)p * ra.Ny + y0) * ra.Nx);
#pragma unroll 4
  for (int e = threadIdx.x; e < nr * M; e += nt) {
    const int r = quick_div(e, ra.m_len);
    lds[r * (S - M) + e] = src[e];
  }
  __syncthreads();
  row_plan<T>(lds, S, nr, pl, tws, dftc, doff, T(-1));
  const int half = M / 2 + 1;
  for (int e = threadIdx.x; e < nr * half; e += nt) {
    const int r = quick_div(e, ra.m_half), k = e - r * half;
    C* row = lds + r * S;
    const C zk = row[k];
    if (k == 0) {
      row[0] = r2c_post(zk, zk, rtw[0]);
      row[M] = r2c_post(zk, zk, rtw[M]);
    } else {
      const C zm = row[M - k];
      row[k] = r2c_post(zk, zm, rtw[k]);
      if (M - k != k) row[M - k] = r2c_post(zm, zk, rtw[M - k]);
    }
  }
  __syncthreads();
  C* dst = spec + (size_t)p * ra.Nkx * ra.Ny + y0;
  if (sizeof(T) == 4 && rows % 2 == 0) {
    // two consecutive rows per thread: one 16-byte store (y0 and Ny even)
    const int h = rows / 2;
    for (int e = threadIdx.x; e < (M + 1) * h; e += nt) {
      const int k = quick_div(e, ra.m_rows), r = 2 * (e - k * h);
      if (r < nr) {                                  // (nr is even)
        const C a = lds[r * S + k], b = lds[(r + 1) * S + k];
        *reinterpret_cast<float4*>(dst + (size_t)k * ra.Ny + r) =
            make_float4(a.x, a.y, b.x, b.y);
      }
    }
  } else {
    for (int e = threadIdx.x; e < (M + 1) * rows; e += nt) {
      const int k = quick_div(e, ra.m_rows), r = e - k * rows;
      if (r < nr) dst[(size_t)k * ra.Ny + r] = lds[r * S + k];
    }
  }
}

// x-pass, half spectrum -> real rows
template <typename T>
__global__ void __launch_bounds__(1024)
k_rows_x_c2r(RowArgs ra, RowPlan pl, const int* __restrict__ band,
             const cplx_t<T>* __restrict__ spec, T* __restrict__ grid,
             const cplx_t<T>* __restrict__ tws, const cplx_t<T>* __restrict__ rtw,
             const T* __restrict__ dftc, DftOff doff) {
  using C = cplx_t<T>;
  extern __shared__ unsigned char lds_raw[];
  C* lds = reinterpret_cast<C*>(lds_raw);
  const int p = blockIdx.y, c = p % ra.Nz;
  if (c < band[0] || c > band[1]) return;
  const int M = ra.Nx / 2, S = (M + 1) | 1, rows = ra.rows, nt = blockDim.x;
  const int yb = rows * (int)sizeof(C) == 64 ? paired_batch(blockIdx.x, gridDim.x) : blockIdx.x;
  const int y0 = yb * rows, nr = min(rows, ra.Ny - y0);
  const C* src = spec + (size_t)p * ra.Nkx * ra.Ny + y0;
  if (sizeof(T) == 4 && rows % 2 == 0) {
    const int h = rows / 2;
#pragma unroll 4
    for (int e = threadIdx.x; e < (M + 1) * h; e += nt) {
      const int k = quick_div(e, ra.m_rows), r = 2 * (e - k * h);
      if (r < nr) {
        const float4 v = *reinterpret_cast<const float4*>(src + (size_t)k * ra.Ny + r);
        C a, b;
        a.x = v.x; a.y = v.y; b.x = v.z; b.y = v.w;
        lds[r * S + k] = a;
        lds[(r + 1) * S + k] = b;
      }
    }
  } else {
#pragma unroll 4
    for (int e = threadIdx.x; e < (M + 1) * rows; e += nt) {
      const int k = quick_div(e, ra.m_rows), r = e - k * rows;
      if (r < nr) lds[r * S + k] = src[(size_t)k * ra.Ny + r];
    }
  }
  __syncthreads();
  const int half = M / 2 + 1;
  for (int e = threadIdx.x; e < nr * half; e += nt) {
    const int r = quick_div(e, ra.m_half), k = e - r * half;
    C* row = lds + r * S;
    if (k == 0) {
      C x0 = row[0], xm = row[M];
      x0.y = T(0);
      xm.y = T(0);
      row[0] = c2r_pre(x0, xm, rtw[0]);
    } else {
      const C xk = row[k], xm = row[M - k];
      row[k] = c2r_pre(xk, xm, rtw[k]);
      if (M - k != k) row[M - k] = c2r_pre(xm, xk, rtw[M - k]);
    }
  }
  __syncthreads();
  row_plan<T>(lds, S, nr, pl, tws, dftc, doff, T(1));
  C* dst = reinterpret_cast<C*>(grid + ((size_t)p * ra.Ny + y0) * ra.Nx);
  for (int e = threadIdx.x; e < nr * M; e += nt) {
    const int r = quick_div(e, ra.m_len);
    dst[e] = lds[r * (S - M) + e];
  }
}

// y-pass, in place on contiguous rows (`rows` consecutive kx)
template <typename T>
__global__ void __launch_bounds__(1024)
k_rows_y(RowArgs ra, RowPlan pl, const int* __restrict__ band, cplx_t<T>* __restrict__ spec,
         const cplx_t<T>* __restrict__ tws, const T* __restrict__ dftc, DftOff doff, T sign) {
  using C = cplx_t<T>;
  extern __shared__ unsigned char lds_raw[];
  C* lds = reinterpret_cast<C*>(lds_raw);
  const int p = blockIdx.y, c = p % ra.Nz;
  if (c < band[0] || c > band[1]) return;
  const int N = ra.Ny, k0 = blockIdx.x * ra.rows, nr = min(ra.rows, ra.Nkx - k0);
  C* g = spec + ((size_t)p * ra.Nkx + k0) * N;
#pragma unroll 4
  for (int e = threadIdx.x; e < nr * N; e += blockDim.x) lds[e] = g[e];
  __syncthreads();
  row_plan<T>(lds, N, nr, pl, tws, dftc, doff, sign);
#pragma unroll 4
  for (int e = threadIdx.x; e < nr * N; e += blockDim.x) g[e] = lds[e];
}

// ---- host side -----------------------------------------------------------------
// Fewest stages, then the smallest largest radix; odd radices first (their
// strided first writes meet no bank conflicts).
static void search(int m, int most, bool fp32, int* cur, int depth, int* best, int* nbest) {
  if (m == 1) {
    const int top = *std::max_element(cur, cur + depth);
    if (*nbest == 0 || depth < *nbest ||
        (depth == *nbest && top < *std::max_element(best, best + *nbest))) {
      std::copy(cur, cur + depth, best);
      *nbest = depth;
    }
    return;
  }
  if (depth == kRowStages || (*nbest && depth >= *nbest)) return;
  static const int all[] = {17, 16, 15, 14, 13, 12, 11, 10, 9, 8, 7, 6, 5, 4, 3, 2};
  for (int R : all) {
    if (R > most || m % R) continue;
    if (!fp32 && R >= 14 && R <= 16) continue;
    cur[depth] = R;
    search(m / R, R, fp32, cur, depth + 1, best, nbest);
  }
}

bool make_row_plan(int n, bool fp32, RowPlan* pl) {
  int cur[kRowStages], best[kRowStages], nst = 0;
  search(n, 17, fp32, cur, 0, best, &nst);
  if (n < 2 || nst == 0) return false;
  std::stable_sort(best, best + nst, [](int a, int b) {
    return (a & 1) != (b & 1) ? (a & 1) > (b & 1) : a > b;
  });
  pl->n = n;
  pl->nst = nst;
  int Ns = 1, tw = 0;
  for (int s = 0; s < nst; ++s) {
    const int R = best[s];
    pl->radix[s] = R;
    pl->ns[s] = Ns;
    pl->mns[s] = quick_mul(Ns);
    pl->mnb[s] = quick_mul(n / R);
    pl->tw[s] = tw;
    if (s > 0) tw += (R - 1) * Ns;
    Ns *= R;
  }
  pl->ntw = tw;
  return true;
}

// Threads for a batch of `rows` rows in lds bytes of LDS: every stage's
// butterflies must fit the registers; among those the fewest lane slots spent
// over all stages (idle lanes of last rounds included), weighed against the
// wavefronts that are resident on a CU (sixteen at most: 128 registers).  0:
// none fits.
static int row_threads(const RowPlan& pl, int rows, size_t lds, bool fp32) {
  const int per_cu = (int)(kLdsBudget / lds);
  int best = 0;
  double best_cost = 0;
  for (int t = 64; t <= 1024; t += 64) {
    double work = 0;
    bool ok = true;
    for (int s = 0; s < pl.nst; ++s) {
      const int R = pl.radix[s], total = rows * (pl.n / R), n = (total + t - 1) / t;
      if (n > row_cap(fp32, R)) ok = false;
      work += (double)n * t * (R + 2);
    }
    if (!ok || per_cu == 0) continue;
    const double waves = std::min(16.0, (double)(per_cu * t / 64));
    const double cost = work / std::pow(waves, 0.7);
    if (!best || cost < best_cost) {
      best = t;
      best_cost = cost;
    }
  }
  return best;
}

static RowArgs row_args(const fcmdp_solver* s, int rows, int pair) {
  const int M = s->dp.Nx / 2;
  return RowArgs{s->dp.Nx, s->dp.Ny, s->dp.Nz, s->dp.Nkx, rows,
                 quick_mul(pair ? rows / 2 : rows), quick_mul(M), quick_mul(M / 2 + 1)};
}

template <typename T>
static hipError_t rows_x(bool fwd, const fcmdp_solver* s, int nch, const void* in, void* out,
                         hipStream_t st) {
  using C = cplx_t<T>;
  const DevParams& dp = s->dp;
  const bool fp32 = sizeof(T) == 4;
  const RowPlan& pl = s->rplan_x;
  const int M = dp.Nx / 2;
  const size_t row = ((size_t)(M + 1) | 1) * sizeof(C);
  // Runs of a full 128-byte line on the transposed side, but half of one, in
  // paired batches, where a CU's LDS holds three full batches or fewer: more
  // workgroups to hide the barriers of each other.  Forward / inverse in us,
  // full against half: 1176 points FP32 578/495 -> 565/476, 756 FP32 246/191 ->
  // 219/173, 768 FP64 758/742 -> 738/677; with seven batches already there
  // (360 FP32) 109/81 -> 112/82.  In FP32 not where one full batch fits: the two
  // half ones are slower at 30 of 33 lengths from 1280 to 2548 (1280^2, 8 planes
  // 563/841 against 668/941, 2000^2 1376/2089 against 1546/2230; the others lose
  // 1 to 3% full: 1632, 2268, 2500).  In FP64 the two are even there (1500^2 15%
  // for full, 2160^2 8% for half).  Fewer rows also if LDS or threads run out.
  const int line = fp32 ? 16 : 8;
  const size_t full = line * row;
  const bool half = 4 * full > kLdsBudget && (!fp32 || 2 * full <= kLdsBudget);
  int rows = s->rows_x > 0 ? s->rows_x : half ? line / 2 : line, nt = 0;
  for (;; rows = rows == 12 ? 8 : rows / 2) {
    nt = rows * row <= kLdsBudget ? row_threads(pl, rows, rows * row, fp32) : 0;
    if (nt || rows == 1) break;
  }
  if (!nt) return hipErrorInvalidValue;
  DftOff doff;
  for (int i = 0; i < 32; ++i) doff.off[i] = s->dft_off[i];
  const RowArgs ra = row_args(s, rows, fp32 && rows % 2 == 0);
  const dim3 g((dp.Ny + rows - 1) / rows, nch * dp.Nz);
  if (fwd)
    hipLaunchKernelGGL(k_rows_x_r2c<T>, g, dim3(nt), rows * row, st, ra, pl, s->band,
                       (const T*)in, (C*)out, (const C*)s->tws_x, (const C*)s->tw_r,
                       (const T*)s->dftc_t, doff);
  else
    hipLaunchKernelGGL(k_rows_x_c2r<T>, g, dim3(nt), rows * row, st, ra, pl, s->band,
                       (const C*)in, (T*)out, (const C*)s->tws_x, (const C*)s->tw_r,
                       (const T*)s->dftc_t, doff);
  return hipGetLastError();
}

template <typename T>
static hipError_t rows_y(const fcmdp_solver* s, int nch, void* spec, int sign, hipStream_t st) {
  using C = cplx_t<T>;
  const DevParams& dp = s->dp;
  const bool fp32 = sizeof(T) == 4;
  const RowPlan& pl = s->rplan_y;
  const size_t row = (size_t)dp.Ny * sizeof(C);
  // about 2048 points per batch: several workgroups per CU, and few enough
  // butterflies that a stage is one or two rounds
  int rows = s->rows_y > 0 ? s->rows_y : std::max(1, std::min(16, 2048 / dp.Ny)), nt = 0;
  for (;; rows /= 2) {
    nt = rows * row <= kLdsBudget ? row_threads(pl, rows, rows * row, fp32) : 0;
    if (nt || rows == 1) break;
  }
  if (!nt) return hipErrorInvalidValue;
  DftOff doff;
  for (int i = 0; i < 32; ++i) doff.off[i] = s->dft_off[i];
  const RowArgs ra = row_args(s, rows, 0);
  const dim3 g((dp.Nkx + rows - 1) / rows, nch * dp.Nz);
  hipLaunchKernelGGL(k_rows_y<T>, g, dim3(nt), rows * row, st, ra, pl, s->band, (C*)spec,
                     (const C*)s->tws_y, (const T*)s->dftc_t, doff, T(sign));
  return hipGetLastError();
}

hipError_t launch_rows_x(bool fwd, const fcmdp_solver* s, int nch, const void* in, void* out,
                         hipStream_t st) {
  return s->mixed ? rows_x<float>(fwd, s, nch, in, out, st)
                  : rows_x<double>(fwd, s, nch, in, out, st);
}
hipError_t launch_rows_y(const fcmdp_solver* s, int nch, void* spec, int sign, hipStream_t st) {
  return s->mixed ? rows_y<float>(s, nch, spec, sign, st) : rows_y<double>(s, nch, spec, sign, st);
}

// whether every stage of the pass fits a workgroup, one row at a time
bool row_plan_fits(const RowPlan& pl, bool fp32) {
  const size_t row = ((size_t)(pl.n + 1) | 1) * (fp32 ? 8 : 16);
  return row <= kLdsBudget && row_threads(pl, 1, row, fp32) > 0;
}

}  // namespace fcmdp

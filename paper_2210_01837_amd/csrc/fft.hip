// xy Fourier transforms (step 2 and step 7 of Sec. 3.4, the periodic part of
// the paper's 3D FFT), hand-written mixed-radix Stockham FFTs in LDS.
//
//  forward: x-pass  real rows (Nx) -> half spectrum (Nx/2+1), written
//           transposed so that y becomes the contiguous axis:
//              grid[p][y][x]  ->  spec[p][kx][y]
//           y-pass  complex rows of length Ny, in place (contiguous).
//  inverse: y-pass (sign +) in place, then the complex-to-real x-pass that
//           reads the transposed layout back into real rows.
//
// The real transforms use the standard packing of a length-Nx real row into
// a length-Nx/2 complex sequence z_n = x_{2n} + i x_{2n+1}, one complex FFT,
// and a split step with the twiddles e^{-2 pi i k/Nx}.  Only planes inside the
// particle band [band[0], band[1]] are transformed.  All transforms are
// unnormalised; the 1/(Nx Ny) factor is applied by the column solve.
#include "dft.h"
#include "fcmdp_internal.h"

namespace fcmdp {

// One Stockham stage over nrows transforms of length N stored row-major.
template <typename T, int R>
__device__ inline void fft_stage(const cplx_t<T>* __restrict__ src,
                                 cplx_t<T>* __restrict__ dst, int N, int Ns,
                                 int nrows, const cplx_t<T>* __restrict__ tw,
                                 const double* __restrict__ cs_d, T sign) {
  using C = cplx_t<T>;
  const int nb = N / R;
  const int twstep = N / (Ns * R);
  T cs[2 * R];
  if constexpr (R != 2 && R != 4 && R != 8) {
#pragma unroll
    for (int m = 0; m < 2 * R; ++m) cs[m] = (T)cs_d[m];
  }
  const int total = nrows * nb;
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int r = idx / nb;
    const int j = idx - r * nb;
    const int base = r * N;
    C v[R];
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = src[base + j + q * nb];
    const int k = j % Ns;
    if (Ns > 1) {
#pragma unroll
      for (int q = 1; q < R; ++q) {
        C w = tw[q * k * twstep];
        w.y *= -sign;            // tw holds e^{-i...}; sign=-1 keeps it
        v[q] = cmul(v[q], w);
      }
    }
    if constexpr (R == 2) dft2<T, C>(v);
    else if constexpr (R == 4) dft4<T, C>(v, sign);
    else if constexpr (R == 8) dft8<T, C>(v, sign);
    else dft_prime<T, C, R>(v, cs, sign);
    const int out = (j - k) * R + k;
#pragma unroll
    for (int q = 0; q < R; ++q) dst[base + out + q * Ns] = v[q];
  }
}

// In-LDS FFT of nrows rows; returns the buffer holding the result.
template <typename T>
__device__ cplx_t<T>* fft_lds(cplx_t<T>* a, cplx_t<T>* b, int N,
                              const FFTPlan& plan, int nrows,
                              const cplx_t<T>* __restrict__ tw,
                              const double* __restrict__ dftc,
                              const int* __restrict__ dft_off, T sign) {
  cplx_t<T>* src = a;
  cplx_t<T>* dst = b;
  int Ns = 1;
  for (int s = 0; s < plan.nstages; ++s) {
    const int R = plan.radix[s];
    const double* cs = dftc + dft_off[R];
    switch (R) {
      case 2: fft_stage<T, 2>(src, dst, N, Ns, nrows, tw, cs, sign); break;
      case 3: fft_stage<T, 3>(src, dst, N, Ns, nrows, tw, cs, sign); break;
      case 4: fft_stage<T, 4>(src, dst, N, Ns, nrows, tw, cs, sign); break;
      case 5: fft_stage<T, 5>(src, dst, N, Ns, nrows, tw, cs, sign); break;
      case 7: fft_stage<T, 7>(src, dst, N, Ns, nrows, tw, cs, sign); break;
      case 8: fft_stage<T, 8>(src, dst, N, Ns, nrows, tw, cs, sign); break;
      case 11: fft_stage<T, 11>(src, dst, N, Ns, nrows, tw, cs, sign); break;
      case 13: fft_stage<T, 13>(src, dst, N, Ns, nrows, tw, cs, sign); break;
      case 17: fft_stage<T, 17>(src, dst, N, Ns, nrows, tw, cs, sign); break;
      default: break;
    }
    __syncthreads();
    cplx_t<T>* t = src; src = dst; dst = t;
    Ns *= R;
  }
  return src;
}

// ---- x-pass, real -> half spectrum, transposed write -------------------------
template <typename T>
__global__ void __launch_bounds__(256)
k_fft_x_r2c(DevParams dp, FFTPlan plan, const int* __restrict__ band,
            const T* __restrict__ grid, cplx_t<T>* __restrict__ spec,
            const cplx_t<T>* __restrict__ tw, const cplx_t<T>* __restrict__ rtw,
            const double* __restrict__ dftc, DftOff doff, int rows) {
  using C = cplx_t<T>;
  extern __shared__ unsigned char lds_raw[];
  C* bufA = reinterpret_cast<C*>(lds_raw);
  const int M = dp.Nx / 2;
  C* bufB = bufA + rows * M;
  const int p = blockIdx.y;
  const int c = p % dp.Nz;
  if (c < band[0] || c > band[1]) return;
  const int y0 = blockIdx.x * rows;
  const int nr = min(rows, dp.Ny - y0);
  const C* src = reinterpret_cast<const C*>(grid + ((size_t)p * dp.Ny + y0) * dp.Nx);
  for (int idx = threadIdx.x; idx < nr * M; idx += blockDim.x) bufA[idx] = src[idx];
  __syncthreads();
  C* Z = fft_lds<T>(bufA, bufB, M, plan, nr, tw, dftc, doff.off, T(-1));
  const size_t pbase = (size_t)p * dp.Nkx * dp.Ny;
  for (int idx = threadIdx.x; idx < nr * (M + 1); idx += blockDim.x) {
    const int k = idx / nr;
    const int r = idx - k * nr;
    const C zk = Z[r * M + (k == M ? 0 : k)];
    C zc = Z[r * M + (k == 0 ? 0 : M - k)];
    zc.y = -zc.y;
    const C e = cscale(cadd(zk, zc), T(0.5));
    const C d = csub(zk, zc);
    C o; o.x = T(0.5) * d.y; o.y = T(-0.5) * d.x;      // -i d / 2
    spec[pbase + (size_t)k * dp.Ny + y0 + r] = cadd(e, cmul(rtw[k], o));
  }
}

// ---- y-pass, in place, contiguous rows ------------------------------------
template <typename T>
__global__ void __launch_bounds__(256)
k_fft_y(DevParams dp, FFTPlan plan, const int* __restrict__ band,
        cplx_t<T>* __restrict__ spec, const cplx_t<T>* __restrict__ tw,
        const double* __restrict__ dftc, DftOff doff, int rows, T sign) {
  using C = cplx_t<T>;
  extern __shared__ unsigned char lds_raw[];
  C* bufA = reinterpret_cast<C*>(lds_raw);
  C* bufB = bufA + rows * dp.Ny;
  const int p = blockIdx.y;
  const int c = p % dp.Nz;
  if (c < band[0] || c > band[1]) return;
  const int k0 = blockIdx.x * rows;
  const int nr = min(rows, dp.Nkx - k0);
  C* row = spec + ((size_t)p * dp.Nkx + k0) * dp.Ny;
  for (int idx = threadIdx.x; idx < nr * dp.Ny; idx += blockDim.x) bufA[idx] = row[idx];
  __syncthreads();
  C* res = fft_lds<T>(bufA, bufB, dp.Ny, plan, nr, tw, dftc, doff.off, sign);
  for (int idx = threadIdx.x; idx < nr * dp.Ny; idx += blockDim.x) row[idx] = res[idx];
}

// ---- x-pass, half spectrum -> real, transposed read -----------------------
template <typename T>
__global__ void __launch_bounds__(256)
k_fft_x_c2r(DevParams dp, FFTPlan plan, const int* __restrict__ band,
            const cplx_t<T>* __restrict__ spec, T* __restrict__ grid,
            const cplx_t<T>* __restrict__ tw, const cplx_t<T>* __restrict__ rtw,
            const double* __restrict__ dftc, DftOff doff, int rows) {
  using C = cplx_t<T>;
  extern __shared__ unsigned char lds_raw[];
  const int M = dp.Nx / 2;
  C* bufA = reinterpret_cast<C*>(lds_raw);        // rows * M
  C* bufB = bufA + rows * M;                        // rows * (M + 1)
  const int p = blockIdx.y;
  const int c = p % dp.Nz;
  if (c < band[0] || c > band[1]) return;
  const int y0 = blockIdx.x * rows;
  const int nr = min(rows, dp.Ny - y0);
  const size_t pbase = (size_t)p * dp.Nkx * dp.Ny;
  for (int idx = threadIdx.x; idx < nr * (M + 1); idx += blockDim.x) {
    const int k = idx / nr;
    const int r = idx - k * nr;
    bufB[r * (M + 1) + k] = spec[pbase + (size_t)k * dp.Ny + y0 + r];
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < nr * M; idx += blockDim.x) {
    const int r = idx / M;
    const int k = idx - r * M;
    C xk = bufB[r * (M + 1) + k];
    C xm = bufB[r * (M + 1) + (M - k)];
    if (k == 0) { xk.y = T(0); xm.y = T(0); }
    xm.y = -xm.y;                                   // conj(X_{M-k})
    const C A = cadd(xk, xm);
    const C B = csub(xk, xm);
    C w = rtw[k];
    w.y = -w.y;                                     // e^{+2 pi i k/Nx}
    const C wb = cmul(w, B);
    C z; z.x = A.x - wb.y; z.y = A.y + wb.x;        // A + i w B
    bufA[r * M + k] = z;
  }
  __syncthreads();
  C* res = fft_lds<T>(bufA, bufB, M, plan, nr, tw, dftc, doff.off, T(1));
  C* dst = reinterpret_cast<C*>(grid + ((size_t)p * dp.Ny + y0) * dp.Nx);
  for (int idx = threadIdx.x; idx < nr * M; idx += blockDim.x) dst[idx] = res[idx];
}

// ---- row-owned in-place transforms ------------------------------------------
// One wavefront owns one row in LDS.  A Stockham stage first reads every
// butterfly input of the lane into registers and then writes the outputs back in
// place.  Butterfly j of a stage belongs to lane j mod 64, so the loop trip counts
// are uniform and there are no index divisions by the row count; the row is
// private to its wavefront, whose LDS accesses complete in issue order, and
// stages need no workgroup barrier.
constexpr int kLanes = 64;

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- fixed plans ("codelets") ----------------------------------------------
// The stage sequence is a template argument (stage code = 16 R + NB); stages
// are inlined one after another, so registers are allocated per stage and
// nothing goes through a call stack.
//
// Between stages s and s + 1 the row is stored in LDS with the layout
//   element i at i + (i / B) * pad          (B a power of two),
// chosen per boundary at compile time.  B divides both the read stride of
// stage s + 1 (N / R_{s+1}) and the write stride of stage s (or every
// radix-R_s block of stage s lies within one B-segment), so that every
// butterfly input and output sits at a constant offset from one address per
// butterfly; the pad spreads the strided writes of stage s (lanes R_s
// elements apart for the first stage) over the LDS banks.  Before the first
// and after the last stage the row is unpadded.
struct RowLay {
  int B, pad;
};

// bank conflicts of one access of 64 lanes to 8-byte elements at the given
// element indices: 64 four-byte banks, 32 lanes per cycle
constexpr int lds_conflicts(const int* idx) {
  int cost = 0;
  for (int g = 0; g < 2; ++g) {
    int cnt[64] = {};
    int worst = 0;
    for (int l = 32 * g; l < 32 * g + 32; ++l) {
      if (idx[l] < 0) continue;
      for (int h = 0; h < 2; ++h) {
        const int b = (2 * idx[l] + h) & 63;
        if (++cnt[b] > worst) worst = cnt[b];
      }
    }
    cost += worst;
  }
  return cost;
}

constexpr int lay_at(RowLay L, int i) { return i + (i / L.B) * L.pad; }

// layout after a stage of radix R with input stride Ns (next stage reads
// with stride nbn) in a row of length N
constexpr RowLay choose_lay(int N, int R, int Ns, int nbn) {
  RowLay best{N, 0};                                // unpadded
  int best_cost = 1 << 30;
  for (int B = 1; B < N; B *= 2) {
    const bool write_lin = Ns % B == 0 || B % (Ns * R) == 0;
    const bool read_lin = nbn % B == 0;
    if (!write_lin || !read_lin) continue;
    // at most one pad element per eight, so that rows grow by 12.5% at most
    const int max_pad = B >= 8 ? B / 8 : 1;
    for (int pad = 0; pad <= max_pad; ++pad) {
      const RowLay L{B, pad};
      int w[64] = {}, r[64] = {};
      for (int t = 0; t < 64; ++t) {
        const int k = t % Ns;
        const int out = (t - k) * R + k;            // stage output, q = 0
        w[t] = t < N / R ? lay_at(L, out) : -1;
        r[t] = t < nbn ? lay_at(L, t) : -1;         // next stage input, q = 0
      }
      // conflicts first, then the smallest row
      const int cost = (lds_conflicts(w) + lds_conflicts(r)) * (1 << 20) +
                       lay_at(L, N - 1);
      if (cost < best_cost) {
        best_cost = cost;
        best = L;
      }
    }
  }
  return best;
}

template <int... Codes>
struct CodeletLayout {
  static constexpr int kStages = sizeof...(Codes);
  static constexpr int kRad[kStages] = {(Codes >> 4)...};
  static constexpr int kN = (1 * ... * (Codes >> 4));
  struct Table {
    RowLay lay[kStages + 1];                        // lay[s]: input of stage s
    int span;
    constexpr Table() : lay(), span(kN) {
      lay[0] = RowLay{kN, 0};
      int Ns = 1;
      for (int s = 0; s < kStages; ++s) {
        if (s + 1 < kStages)
          lay[s + 1] = choose_lay(kN, kRad[s], Ns, kN / kRad[s + 1]);
        else
          lay[s + 1] = RowLay{kN, 0};
        const int e = lay_at(lay[s + 1], kN - 1) + 1;
        if (e > span) span = e;
        Ns *= kRad[s];
      }
    }
  };
  static constexpr Table kTable = Table();
};

// One stage of a fixed plan: every size is a compile-time constant, inputs
// in layout LI, outputs in layout LO.
template <typename T, int R, int NB, int N, int NS, int BI, int PI, int BO, int PO>
__device__ __forceinline__ void stage_fixed(cplx_t<T>* row, int t,
                                            const cplx_t<T>* __restrict__ tw,
                                            const T* __restrict__ cs, T sign) {
  using C = cplx_t<T>;
  constexpr RowLay LI{BI, PI}, LO{BO, PO};
  constexpr int nb = N / R;
  constexpr int twstep = N / (NS * R);
  static_assert(nb % BI == 0 || BI >= N, "stage input layout not linear");
  static_assert(NS % BO == 0 || BO % (NS * R) == 0 || BO >= N,
                "stage output layout not linear");
  constexpr int rstep = lay_at(LI, nb);             // offset of input q = 1
  constexpr int wstep = NS % BO == 0 ? lay_at(LO, NS) : NS;
  C v[NB][R];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int j = t + kLanes * i;
    if (j < nb) {
      const int base = (int)((unsigned)j / BI) * PI + j;
#pragma unroll
      for (int q = 0; q < R; ++q) v[i][q] = row[base + q * rstep];
    }
  }
  wave_sync();
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int j = t + kLanes * i;
    if (j < nb) {
      C* x = v[i];
      const int k = j % NS;
      if constexpr (NS > 1) {
#pragma unroll
        for (int q = 1; q < R; ++q) {
          C w = tw[q * k * twstep];
          w.y *= -sign;
          x[q] = cmul(x[q], w);
        }
      }
      dft_any<T, C, R>(x, cs, sign);
      const int out = (j - k) * R + k;
      const int base = (int)((unsigned)out / BO) * PO + out;
#pragma unroll
      for (int q = 0; q < R; ++q) row[base + q * wstep] = x[q];
    }
  }
  wave_sync();
}

template <typename T, typename Lay, int S, int NS, int Code, int... Rest>
__device__ __forceinline__ void run_codes(cplx_t<T>* row, int t,
                                          const cplx_t<T>* __restrict__ tw,
                                          const T* __restrict__ dftc,
                                          const DftOff& doff, T sign) {
  constexpr int R = Code >> 4, NB = Code & 15;
  constexpr RowLay LI = Lay::kTable.lay[S], LO = Lay::kTable.lay[S + 1];
  stage_fixed<T, R, NB, Lay::kN, NS, LI.B, LI.pad, LO.B, LO.pad>(row, t, tw, dftc + doff.off[R],
                                                                  sign);
  if constexpr (sizeof...(Rest) > 0)
    run_codes<T, Lay, S + 1, NS * R, Rest...>(row, t, tw, dftc, doff, sign);
}

template <int... Codes>
struct FixedRows {
  using Lay = CodeletLayout<Codes...>;
  static constexpr int kN = Lay::kN;                // transform length
  template <typename T>
  __device__ __forceinline__ static void run(cplx_t<T>* row, int t,
                             const cplx_t<T>* __restrict__ tw,
                             const T* __restrict__ dftc, const DftOff& doff,
                             T sign) {
    run_codes<T, Lay, 0, 1, Codes...>(row, t, tw, dftc, doff, sign);
  }
  __host__ __device__ static constexpr int span(int n) {
    return n > Lay::kTable.span ? n : Lay::kTable.span;
  }
};

// LDS row stride of the x passes (Nx/2 + 1 elements at least, odd so that the
// transposed accesses of 16 rows fall into different banks)
template <typename Run>
__host__ __device__ constexpr int x_stride(int M) {
  return Run::span(M + 1) | 1;
}

// x-pass, real rows -> half spectrum, ROWS rows per workgroup, written
// transposed as ROWS-long runs of consecutive y.
template <typename T, int ROWS, typename Run>
__global__ void __launch_bounds__(ROWS * kLanes)
k_fftw_x_r2c(DevParams dp, const int* __restrict__ band, const T* __restrict__ grid,
             cplx_t<T>* __restrict__ spec, const cplx_t<T>* __restrict__ tw,
             const cplx_t<T>* __restrict__ rtw, const T* __restrict__ dftc, DftOff doff) {
  using C = cplx_t<T>;
  extern __shared__ unsigned char lds_raw[];
  C* lds = reinterpret_cast<C*>(lds_raw);
  const int M = dp.Nx / 2;
  const int S = x_stride<Run>(M);                   // row stride in LDS
  const int p = blockIdx.y;
  const int c = p % dp.Nz;
  if (c < band[0] || c > band[1]) return;           // whole workgroup
  const int y0 = blockIdx.x * ROWS;
  const int nr = min(ROWS, dp.Ny - y0);
  const int wr = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int t = threadIdx.x % kLanes;
  C* row = lds + wr * S;
  // rows past the grid edge (tail workgroup) transform a copy of row y0
  const int y = wr < nr ? y0 + wr : y0;
  const C* src = reinterpret_cast<const C*>(grid + ((size_t)p * dp.Ny + y) * dp.Nx);
#pragma unroll 4
  for (int i = t; i < M; i += kLanes) row[i] = src[i];
  wave_sync();
  Run::template run<T>(row, t, tw, dftc, doff, T(-1));
  for (int k = t; k <= M / 2; k += kLanes) {
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
  const size_t pbase = (size_t)p * dp.Nkx * dp.Ny;
  if constexpr (ROWS % 2 == 0 && sizeof(T) == 4) {
    // two consecutive rows per thread: one 16-byte store (y0 and Ny even)
    for (int idx = threadIdx.x; idx < (M + 1) * (ROWS / 2); idx += ROWS * kLanes) {
      const int k = idx / (ROWS / 2);
      const int r = 2 * (idx % (ROWS / 2));
      C* dst = spec + pbase + (size_t)k * dp.Ny + y0 + r;
      const C a = lds[r * S + k], b = lds[(r + 1) * S + k];
      if (r + 1 < nr && (dp.Ny & 1) == 0) {
        *reinterpret_cast<float4*>(dst) = make_float4(a.x, a.y, b.x, b.y);
      } else {
        if (r < nr) dst[0] = a;
        if (r + 1 < nr) dst[1] = b;
      }
    }
  } else {
    for (int idx = threadIdx.x; idx < (M + 1) * ROWS; idx += ROWS * kLanes) {
      const int k = idx / ROWS;
      const int r = idx % ROWS;
      if (r < nr) spec[pbase + (size_t)k * dp.Ny + y0 + r] = lds[r * S + k];
    }
  }
}

// y-pass, in place on contiguous rows of length Ny.
template <typename T, int ROWS, typename Run>
__global__ void __launch_bounds__(ROWS * kLanes)
k_fftw_y(DevParams dp, const int* __restrict__ band, cplx_t<T>* __restrict__ spec,
         const cplx_t<T>* __restrict__ tw,
         const T* __restrict__ dftc, DftOff doff, T sign) {
  using C = cplx_t<T>;
  extern __shared__ unsigned char lds_raw[];
  const int p = blockIdx.y;
  const int c = p % dp.Nz;
  if (c < band[0] || c > band[1]) return;
  const int wr = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int t = threadIdx.x % kLanes;
  const int kx = blockIdx.x * ROWS + wr;
  if (kx >= dp.Nkx) return;                         // a whole wavefront
  const int N = dp.Ny;
  C* row = reinterpret_cast<C*>(lds_raw) + wr * Run::span(N);
  C* g = spec + ((size_t)p * dp.Nkx + kx) * N;
#pragma unroll 4
  for (int i = t; i < N; i += kLanes) row[i] = g[i];
  wave_sync();
  Run::template run<T>(row, t, tw, dftc, doff, sign);
#pragma unroll 4
  for (int i = t; i < N; i += kLanes) g[i] = row[i];
}

// y-pass as a persistent loop: workgroup g (one wavefront) transforms the
// band rows g, g + G, ... and loads the next row into registers while the
// current one is transformed in LDS, so that every wavefront keeps memory
// requests in flight through its arithmetic.  Fixed-length plans only.
template <typename T, typename Run>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 8)))
k_fftw_y_pipe(DevParams dp, const int* __restrict__ band, cplx_t<T>* __restrict__ spec,
              const cplx_t<T>* __restrict__ tw,
              const T* __restrict__ dftc, DftOff doff, T sign, int nch) {
  using C = cplx_t<T>;
  constexpr int N = Run::kN;                        // == dp.Ny
  constexpr int PER = (N + 63) / 64;
  extern __shared__ unsigned char lds_raw[];
  C* row = reinterpret_cast<C*>(lds_raw);
  const int lo = band[0], hi = band[1];
  if (lo > hi) return;
  const int P = hi - lo + 1;
  const int total = nch * P * dp.Nkx;               // band rows
  const int t = threadIdx.x;
  int r = blockIdx.x;
  if (r >= total) return;
  // row r: kx fastest, then band plane, then channel
  auto row_ptr = [&](int rr) {
    const int kx = rr % dp.Nkx, q = rr / dp.Nkx;
    const int ch = q / P, c = lo + q - ch * P;
    return spec + ((size_t)(ch * dp.Nz + c) * dp.Nkx + kx) * N;
  };
  C pre[PER];
  {
    const C* g = row_ptr(r);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (t + 64 * i < N) pre[i] = g[t + 64 * i];
  }
  for (; r < total; r += gridDim.x) {
    C* g = row_ptr(r);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (t + 64 * i < N) row[t + 64 * i] = pre[i];
    const int rn = r + gridDim.x;
    if (rn < total) {
      const C* gn = row_ptr(rn);
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (t + 64 * i < N) pre[i] = gn[t + 64 * i];
    }
    wave_sync();
    // the tables and the lane index are opaque to the optimiser inside the
    // loop, so that table loads and LDS addresses are not hoisted out of it
    // (which would hold every twiddle and address of the plan in registers)
    const C* twl = tw;
    const T* csl = dftc;
    int tl = t;
    asm volatile("" : "+s"(twl), "+s"(csl), "+v"(tl));
    Run::template run<T>(row, tl, twl, csl, doff, sign);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (t + 64 * i < N) g[t + 64 * i] = row[t + 64 * i];
    wave_sync();
  }
}

// x-pass, half spectrum -> real rows, reading ROWS-long runs of the
// transposed layout.
template <typename T, int ROWS, typename Run>
__global__ void __launch_bounds__(ROWS * kLanes)
k_fftw_x_c2r(DevParams dp, const int* __restrict__ band, const cplx_t<T>* __restrict__ spec,
             T* __restrict__ grid, const cplx_t<T>* __restrict__ tw,
             const cplx_t<T>* __restrict__ rtw, const T* __restrict__ dftc, DftOff doff) {
  using C = cplx_t<T>;
  extern __shared__ unsigned char lds_raw[];
  C* lds = reinterpret_cast<C*>(lds_raw);
  const int M = dp.Nx / 2;
  const int S = x_stride<Run>(M);                   // row stride in LDS
  const int p = blockIdx.y;
  const int c = p % dp.Nz;
  if (c < band[0] || c > band[1]) return;
  const int y0 = blockIdx.x * ROWS;
  const int nr = min(ROWS, dp.Ny - y0);
  const size_t pbase = (size_t)p * dp.Nkx * dp.Ny;
  if constexpr (ROWS % 2 == 0 && sizeof(T) == 4) {
    // two consecutive rows per thread: one 16-byte load (y0 and Ny even)
    const int total = (M + 1) * (ROWS / 2);
    if (nr == ROWS && (dp.Ny & 1) == 0) {
      // whole workgroup: a thread issues all of its loads (nine cover the
      // half spectrum of 2176-point rows) before the first LDS store
      constexpr int kB = 9;
      for (int base = threadIdx.x; base < total; base += kB * ROWS * kLanes) {
        float4 v[kB];
#pragma unroll
        for (int u = 0; u < kB; ++u) {
          const int idx = min(base + u * ROWS * kLanes, total - 1);   // in bounds
          const int k = idx / (ROWS / 2);
          const int r = 2 * (idx % (ROWS / 2));
          v[u] = *reinterpret_cast<const float4*>(spec + pbase + (size_t)k * dp.Ny + y0 + r);
        }
#pragma unroll
        for (int u = 0; u < kB; ++u) {
          const int idx = base + u * ROWS * kLanes;
          if (idx < total) {
            const int k = idx / (ROWS / 2);
            const int r = 2 * (idx % (ROWS / 2));
            lds[r * S + k] = make_float2(v[u].x, v[u].y);
            lds[(r + 1) * S + k] = make_float2(v[u].z, v[u].w);
          }
        }
      }
    } else {
      for (int idx = threadIdx.x; idx < total; idx += ROWS * kLanes) {
        const int k = idx / (ROWS / 2);
        const int r = 2 * (idx % (ROWS / 2));
        const C* src = spec + pbase + (size_t)k * dp.Ny + y0;
        C a, b;
        if (r + 1 < nr && (dp.Ny & 1) == 0) {
          const float4 v = *reinterpret_cast<const float4*>(src + r);
          a.x = v.x; a.y = v.y; b.x = v.z; b.y = v.w;
        } else {
          // rows past the grid edge transform a copy of row y0
          a = src[r < nr ? r : 0];
          b = src[r + 1 < nr ? r + 1 : 0];
        }
        lds[r * S + k] = a;
        lds[(r + 1) * S + k] = b;
      }
    }
  } else {
    for (int idx = threadIdx.x; idx < (M + 1) * ROWS; idx += ROWS * kLanes) {
      const int k = idx / ROWS;
      const int r = idx % ROWS;
      // rows past the grid edge transform a copy of row y0
      lds[r * S + k] = spec[pbase + (size_t)k * dp.Ny + y0 + (r < nr ? r : 0)];
    }
  }
  __syncthreads();
  const int wr = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
  const int t = threadIdx.x % kLanes;
  C* row = lds + wr * S;
  for (int k = t; k <= M / 2; k += kLanes) {
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
  wave_sync();
  Run::template run<T>(row, t, tw, dftc, doff, T(1));
  if (wr < nr) {
    C* dst = reinterpret_cast<C*>(grid + ((size_t)p * dp.Ny + y0 + wr) * dp.Nx);
#pragma unroll 4
    for (int i = t; i < M; i += kLanes) dst[i] = row[i];
  }
}

template <typename T, int ROWS, typename Run>
static void launch_wave_x(bool fwd, const fcmdp_solver* s, int nch, const void* in,
                          void* out, const DftOff& doff, hipStream_t st) {
  using C = cplx_t<T>;
  const DevParams& dp = s->dp;
  const int M = dp.Nx / 2;
  const size_t lds = (size_t)ROWS * x_stride<Run>(M) * sizeof(C);
  dim3 g((dp.Ny + ROWS - 1) / ROWS, nch * dp.Nz);
  const T* cs = (const T*)s->dftc_t;
  if (fwd)
    hipLaunchKernelGGL((k_fftw_x_r2c<T, ROWS, Run>), g, dim3(ROWS * kLanes),
                       lds, st, dp, s->band, (const T*)in, (C*)out,
                       (const C*)s->tw_x, (const C*)s->tw_r, cs, doff);
  else
    hipLaunchKernelGGL((k_fftw_x_c2r<T, ROWS, Run>), g, dim3(ROWS * kLanes),
                       lds, st, dp, s->band, (const C*)in, (T*)out,
                       (const C*)s->tw_x, (const C*)s->tw_r, cs, doff);
}

// rows per workgroup of the x passes: the most (up to 16) that fit in LDS, and
// twelve when sixteen do not fit but twelve do (1350-point rows): more
// wavefronts and longer transposed runs than eight
static int rows_fitting(size_t row_bytes, int maxrows) {
  int r = maxrows;
  while (r > 1 && (size_t)r * row_bytes > kLdsBudget) r /= 2;
  return r;
}
template <typename T, typename Run>
static void wave_x_rows(bool fwd, const fcmdp_solver* s, int nch, const void* in,
                        void* out, const DftOff& doff, hipStream_t st) {
  const size_t row = (size_t)x_stride<Run>(s->dp.Nx / 2) * sizeof(cplx_t<T>);
  int r = s->rows_x;
  if (r == 0) {
    r = rows_fitting(row, 16);
    if (r == 8 && 12 * row <= kLdsBudget) r = 12;
  }
  switch (r) {
    case 16: launch_wave_x<T, 16, Run>(fwd, s, nch, in, out, doff, st); break;
    case 12: launch_wave_x<T, 12, Run>(fwd, s, nch, in, out, doff, st); break;
    case 8: launch_wave_x<T, 8, Run>(fwd, s, nch, in, out, doff, st); break;
    case 4: launch_wave_x<T, 4, Run>(fwd, s, nch, in, out, doff, st); break;
    case 2: launch_wave_x<T, 2, Run>(fwd, s, nch, in, out, doff, st); break;
    default: launch_wave_x<T, 1, Run>(fwd, s, nch, in, out, doff, st); break;
  }
}

template <typename T, int ROWS, typename Run>
static void launch_wave_y(const fcmdp_solver* s, int nch, void* spec, const DftOff& doff,
                          T sign, hipStream_t st) {
  using C = cplx_t<T>;
  const DevParams& dp = s->dp;
  const size_t lds = (size_t)ROWS * Run::span(dp.Ny) * sizeof(C);
  dim3 g((dp.Nkx + ROWS - 1) / ROWS, nch * dp.Nz);
  hipLaunchKernelGGL((k_fftw_y<T, ROWS, Run>), g, dim3(ROWS * kLanes), lds, st,
                     dp, s->band, (C*)spec, (const C*)s->tw_y, (const T*)s->dftc_t, doff, sign);
}

template <typename T, typename Run>
static void wave_y_rows(const fcmdp_solver* s, int nch, void* spec, const DftOff& doff,
                        T sign, hipStream_t st) {
  // rows are independent; one per workgroup packs LDS best
  switch (s->rows_y) {
    case 8: launch_wave_y<T, 8, Run>(s, nch, spec, doff, sign, st); break;
    case 4: launch_wave_y<T, 4, Run>(s, nch, spec, doff, sign, st); break;
    case 2: launch_wave_y<T, 2, Run>(s, nch, spec, doff, sign, st); break;
    default: launch_wave_y<T, 1, Run>(s, nch, spec, doff, sign, st); break;
  }
}

// Persistent y-pass: as many one-wavefront workgroups as stay resident (LDS
// and registers allow eight per compute unit).
template <typename T, typename Run>
static void wave_y_pipe(const fcmdp_solver* s, int nch, void* spec, const DftOff& doff,
                        T sign, hipStream_t st) {
  using C = cplx_t<T>;
  const DevParams& dp = s->dp;
  const size_t lds = (size_t)Run::span(dp.Ny) * sizeof(C);
  const int per_cu = (int)std::min<size_t>(8, kLdsBudget / lds);
  const int g = std::max(1, s->num_cu) * std::max(1, per_cu);
  hipLaunchKernelGGL((k_fftw_y_pipe<T, Run>), dim3(g), dim3(64), lds, st, dp,
                     s->band, (C*)spec, (const C*)s->tw_y, (const T*)s->dftc_t, doff, sign,
                     nch);
}

// Codelets compiled for the transform lengths of the large workloads (single
// precision, 64 threads per row); Codelet<i> has length kCodeletLength[i].
// Few stages of large radices, the odd ones first: a stage is a round trip of the
// row through LDS, and composite radices cost little arithmetic.  Forward /
// inverse transforms, 2700 = 3 3 3 5 5 4 with 1350 = 3 3 3 5 5 2 against
// 15 15 12 and 15 9 10: 2.02/2.19 -> 1.53/1.60 ms (13 planes, three channels);
// 768 = 4 8 8 3 against 12 8 8: 293/294 -> 277/279 us (18 planes, six).
static const int kCodeletLength[] = {1088, 2176, 384, 768, 1350, 2700};
using Codelet0 = FixedRows<8 * 16 + 3, 8 * 16 + 3, 17 * 16 + 1>;
using Codelet1 = FixedRows<16 * 16 + 3, 8 * 16 + 5, 17 * 16 + 2>;
using Codelet2 = FixedRows<16 * 16 + 1, 8 * 16 + 1, 3 * 16 + 2>;
using Codelet3 = FixedRows<12 * 16 + 1, 8 * 16 + 2, 8 * 16 + 2>;
using Codelet4 = FixedRows<15 * 16 + 2, 9 * 16 + 3, 10 * 16 + 3>;
using Codelet5 = FixedRows<15 * 16 + 3, 15 * 16 + 3, 12 * 16 + 4>;

template <typename T>
static void wave_x(bool fwd, const fcmdp_solver* s, int nch, const void* in, void* out,
                   const DftOff& doff, hipStream_t st) {
  switch (s->codelet_x) {
    case 0: wave_x_rows<T, Codelet0>(fwd, s, nch, in, out, doff, st); return;
    case 1: wave_x_rows<T, Codelet1>(fwd, s, nch, in, out, doff, st); return;
    case 2: wave_x_rows<T, Codelet2>(fwd, s, nch, in, out, doff, st); return;
    case 3: wave_x_rows<T, Codelet3>(fwd, s, nch, in, out, doff, st); return;
    case 4: wave_x_rows<T, Codelet4>(fwd, s, nch, in, out, doff, st); return;
    case 5: wave_x_rows<T, Codelet5>(fwd, s, nch, in, out, doff, st); return;
    default: break;
  }
}

template <typename T>
static void wave_y(const fcmdp_solver* s, int nch, void* spec, const DftOff& doff,
                         T sign, hipStream_t st) {
  if (!s->force_no_pipeline) {
    switch (s->codelet_y) {
      case 0: wave_y_pipe<T, Codelet0>(s, nch, spec, doff, sign, st); return;
      case 1: wave_y_pipe<T, Codelet1>(s, nch, spec, doff, sign, st); return;
      case 2: wave_y_pipe<T, Codelet2>(s, nch, spec, doff, sign, st); return;
      case 3: wave_y_pipe<T, Codelet3>(s, nch, spec, doff, sign, st); return;
      case 4: wave_y_pipe<T, Codelet4>(s, nch, spec, doff, sign, st); return;
      case 5: wave_y_pipe<T, Codelet5>(s, nch, spec, doff, sign, st); return;
      default: break;
    }
  }
  switch (s->codelet_y) {
    case 0: wave_y_rows<T, Codelet0>(s, nch, spec, doff, sign, st); return;
    case 1: wave_y_rows<T, Codelet1>(s, nch, spec, doff, sign, st); return;
    case 2: wave_y_rows<T, Codelet2>(s, nch, spec, doff, sign, st); return;
    case 3: wave_y_rows<T, Codelet3>(s, nch, spec, doff, sign, st); return;
    case 4: wave_y_rows<T, Codelet4>(s, nch, spec, doff, sign, st); return;
    case 5: wave_y_rows<T, Codelet5>(s, nch, spec, doff, sign, st); return;
    default: break;
  }
}

int fft_lds_row(int codelet, int n, bool x) {
  switch (codelet) {
    case 0: return x ? x_stride<Codelet0>(n) : Codelet0::span(n);
    case 1: return x ? x_stride<Codelet1>(n) : Codelet1::span(n);
    case 2: return x ? x_stride<Codelet2>(n) : Codelet2::span(n);
    case 3: return x ? x_stride<Codelet3>(n) : Codelet3::span(n);
    case 4: return x ? x_stride<Codelet4>(n) : Codelet4::span(n);
    case 5: return x ? x_stride<Codelet5>(n) : Codelet5::span(n);
    default: return x ? (n + 1) | 1 : n;
  }
}

int fft_codelet(int n, bool fp32) {
  if (!fp32) return -1;
  for (int i = 0; i < (int)(sizeof(kCodeletLength) / sizeof(int)); ++i)
    if (kCodeletLength[i] == n) return i;
  return -1;
}

static int rows_for(int len, size_t elem, int bufs_extra, int maxrows) {
  // two ping-pong buffers of rows*len complex words within kLdsBudget
  size_t per = 2 * (size_t)len * elem + (size_t)bufs_extra * elem;
  int r = (int)(kLdsBudget / per);
  if (r < 1) r = 1;
  if (r > maxrows) r = maxrows;
  return r;
}

static DftOff dft_offsets(const fcmdp_solver* s) {
  DftOff doff;
  for (int i = 0; i < 32; ++i) doff.off[i] = s->dft_off[i];
  return doff;
}

// Passes with workgroup-owned rows, two buffers and radices up to 8: small FP64
// grids, and a cross-check (variant FCMDP_VARIANT_GENERIC_FFT).
template <typename T>
static void generic_x(bool fwd, const fcmdp_solver* s, int nch, const void* in, void* out,
                      const DftOff& doff, hipStream_t st) {
  using C = cplx_t<T>;
  const DevParams& dp = s->dp;
  const int M = dp.Nx / 2;
  const int planes = nch * dp.Nz;
  int rows = rows_for(M, sizeof(C), fwd ? 0 : 1, 16);
  if (rows > dp.Ny) rows = dp.Ny;
  const dim3 g((dp.Ny + rows - 1) / rows, planes);
  if (fwd)
    hipLaunchKernelGGL(k_fft_x_r2c<T>, g, dim3(256), 2 * (size_t)rows * M * sizeof(C), st,
                       dp, s->plan_x, s->band, (const T*)in, (C*)out, (const C*)s->tw_x,
                       (const C*)s->tw_r, s->dftc, doff, rows);
  else
    hipLaunchKernelGGL(k_fft_x_c2r<T>, g, dim3(256),
                       (size_t)rows * (2 * M + 1) * sizeof(C), st, dp, s->plan_x, s->band,
                       (const C*)in, (T*)out, (const C*)s->tw_x, (const C*)s->tw_r, s->dftc,
                       doff, rows);
}
template <typename T>
static void generic_y(const fcmdp_solver* s, int nch, void* spec, const DftOff& doff, T sign,
                      hipStream_t st) {
  using C = cplx_t<T>;
  const DevParams& dp = s->dp;
  int rows = rows_for(dp.Ny, sizeof(C), 0, 16);
  if (rows > dp.Nkx) rows = dp.Nkx;
  const int planes = nch * dp.Nz;
  hipLaunchKernelGGL(k_fft_y<T>, dim3((dp.Nkx + rows - 1) / rows, planes), dim3(256),
                     2 * (size_t)rows * dp.Ny * sizeof(C), st, dp, s->plan_y, s->band,
                     (C*)spec, (const C*)s->tw_y, s->dftc, doff, rows, sign);
}

// FP64 grids of at most 1600 KiB a channel with short rows take the two-buffer
// kernels: small code and 256 threads for few points, where a launch of
// fft_rows.hip is all latency.  Forward + inverse in us, fft_rows against these:
// 24^2 x 32 planes 29 / 25, 64^2 x 32 44 / 38, 128^2 x 8 49 / 44, 80^2 x 32 47 /
// 43 (at the line); beyond it 90^2 x 32 51 / 51 to 61 / 66, 32 x 180 x 32 47 / 56
// to 63 / 96, 400 x 64 x 8 51 / 55.  Not in FP32, where their smaller radices
// round more (an apply at 90^2: 6.6e-7 against 6.1e-7 from 64 bits).  Rows per
// workgroup that a caller asks for are those of fft_rows.
static bool small_grid(const fcmdp_solver* s) {
  const DevParams& dp = s->dp;
  const size_t channel = sizeof(double) * (size_t)dp.Nz * dp.Ny * dp.Nx;
  return !s->mixed && channel <= 1600 * 1024 && dp.Nx <= 320 && dp.Ny <= 128 &&
         s->rows_x == 0 && s->rows_y == 0;
}

// One pass: the fixed plan of the length where there is one, else the two-buffer
// kernels or the run-time plan of fft_rows.hip.
static hipError_t x_pass(bool fwd, const fcmdp_solver* s, int nch, const void* in, void* out,
                         hipStream_t st) {
  const DftOff doff = dft_offsets(s);
  if (s->force_generic_fft || small_grid(s)) {
    if (s->mixed) generic_x<float>(fwd, s, nch, in, out, doff, st);
    else generic_x<double>(fwd, s, nch, in, out, doff, st);
  } else if (s->codelet_x >= 0) {
    wave_x<float>(fwd, s, nch, in, out, doff, st);
  } else {
    return launch_rows_x(fwd, s, nch, in, out, st);
  }
  return hipGetLastError();
}
static hipError_t y_pass(const fcmdp_solver* s, int nch, void* spec, int sign, hipStream_t st) {
  const DftOff doff = dft_offsets(s);
  if (s->force_generic_fft || small_grid(s)) {
    if (s->mixed) generic_y<float>(s, nch, spec, doff, (float)sign, st);
    else generic_y<double>(s, nch, spec, doff, (double)sign, st);
  } else if (s->codelet_y >= 0) {
    wave_y<float>(s, nch, spec, doff, (float)sign, st);
  } else {
    return launch_rows_y(s, nch, spec, sign, st);
  }
  return hipGetLastError();
}

// Channels per group of an x- and a y-pass that run one after the other on it.
// A group whose planes stay in the 256 MB last-level cache between the two saves
// the second its reads from HBM; each further pair of launches costs its
// drained ends.  The band is known to the device only; the line is for bands of
// about half of the Nz planes.  Forward / inverse in us, all channels against
// groups: 768^2 FP64 (151 MB a channel) 745/682 -> 672/654 by two; 1176^2 FP32
// (177 MB) 562/476 -> 525/490 by one; 768^2 FP32 (76 MB) 310/301 -> 293/294 by
// three; but 756 x 442 (217 MB all channels) 223/174 -> 241/191 and 2176^2 (606 MB
// a channel) 2217/2394 -> 2584/2659 by one.  Six channels with 14, 24 and all of 32
// planes reached, time by groups over time by all, FP32 forward: 1344^2 (232 MB)
// 0.94 0.92 0.95, 1500^2 (288 MB) 0.95 0.94 0.99, 1560^2 (312 MB) 0.93 0.99 1.02,
// 1536^2 (302 MB, fixed x plan) 1.02 1.00 1.05; FP64 forward and inverse: 864^2
// (192 MB) 0.98 0.93 0.96, 1040^2 (277 MB) 0.94 0.96 1.01, 1080^2 (299 MB) 0.92
// 0.95 1.00.
static int fft_group(const fcmdp_solver* s, int nch) {
  const double mb = (s->mixed ? 8e-6 : 16e-6) * s->dp.Nz * s->dp.Nkx * s->dp.Ny;
  const double fits = 320;
  if (mb * nch <= fits || mb > fits) return nch;
  const int most = (int)(fits / mb), groups = (nch + most - 1) / most;
  return (nch + groups - 1) / groups;
}

hipError_t launch_fft_forward(const fcmdp_solver* s, const void* grid,
                              void* spec, hipStream_t st) {
  const DevParams& dp = s->dp;
  const size_t t = s->mixed ? 4 : 8;
  const size_t ch_grid = t * dp.Nz * dp.Ny * dp.Nx, ch_spec = 2 * t * dp.Nz * dp.Nkx * dp.Ny;
  const int group = fft_group(s, dp.nch_in);
  hipError_t e = hipSuccess;
  for (int c = 0; c < dp.nch_in && e == hipSuccess; c += group) {
    const int nch = std::min(group, dp.nch_in - c);
    void* q = (char*)spec + c * ch_spec;
    e = x_pass(true, s, nch, (const char*)grid + c * ch_grid, q, st);
    if (e == hipSuccess) e = y_pass(s, nch, q, -1, st);
  }
  return e;
}

hipError_t launch_fft_inverse(const fcmdp_solver* s, void* spec, void* grid,
                              hipStream_t st) {
  const DevParams& dp = s->dp;
  const size_t t = s->mixed ? 4 : 8;
  const size_t ch_grid = t * dp.Nz * dp.Ny * dp.Nx, ch_spec = 2 * t * dp.Nz * dp.Nkx * dp.Ny;
  // (in FP32 the inverse gains nothing from groups)
  const int group = s->mixed ? dp.nch_out : fft_group(s, dp.nch_out);
  hipError_t e = hipSuccess;
  for (int c = 0; c < dp.nch_out && e == hipSuccess; c += group) {
    const int nch = std::min(group, dp.nch_out - c);
    void* q = (char*)spec + c * ch_spec;
    e = y_pass(s, nch, q, 1, st);
    if (e == hipSuccess) e = x_pass(false, s, nch, q, (char*)grid + c * ch_grid, st);
  }
  return e;
}

}  // namespace fcmdp

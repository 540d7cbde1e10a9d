// Particle preparation: domain checks and cell keys, the z-band of touched
// Chebyshev planes, a stable LSD radix sort of particles by xy cell, cell
// start offsets, and per-particle ES weight records in sorted order.
//
// The sort makes every later reduction order a function of the input alone
// (particles of one cell keep their input order), so spreading is
// deterministic without atomics.
#include <utility>

#include "fcmdp_internal.h"
#include "es.h"

namespace fcmdp {

// ----------------------------------------------------------------------------
// prep: keys, band, domain errors
// ----------------------------------------------------------------------------
constexpr int kSortThreads = 256;
constexpr int kSortItems = 2048;                 // per workgroup and pass
constexpr int kSortChunks = kSortItems / 64;     // 32
// place of a digit's count of one workgroup: [workgroup][digit] or, for the
// scan over workgroups, [digit][workgroup]
struct HistAt {
  int digit, block;
  __device__ int operator()(int d, int b) const { return d * digit + b * block; }
};

// cell key of particle j (ncells if outside the domain) and its z window
// (cB < cA: none)
template <typename Tin>
__device__ __forceinline__ uint32_t cell_key(const DevParams& dp, const double* zc,
                                             const Tin* __restrict__ pos, int j, int* cA,
                                             int* cB) {
  const double x = (double)pos[3 * (size_t)j + 0];
  const double y = (double)pos[3 * (size_t)j + 1];
  const double z = (double)pos[3 * (size_t)j + 2];
  *cA = 0;
  *cB = -1;
  bool ok = isfinite(x) && isfinite(y) && isfinite(z) && z >= 0.0;
  if (ok) ok = dp.geometry == 0 ? (z + dp.alpha <= dp.H) : (z <= dp.H);
  if (!ok) return (uint32_t)dp.ncells;
  int ix, iy;
  double fx, fy;
  cell_of(wrap_coord(x, dp.Lx), dp.h, dp.Nx, &ix, &fx);
  cell_of(wrap_coord(y, dp.Ly), dp.h, dp.Ny, &iy, &fy);
  z_window(dp, zc, z, cA, cB);
  return (uint32_t)(iy * dp.Nx + ix);
}

// keys, band and domain errors of 2048 particles per workgroup, and their
// histogram of the first sort digit
template <typename Tin>
__global__ void __launch_bounds__(1024)
k_prep(DevParams dp, int n, const Tin* __restrict__ pos,
       const double* __restrict__ zc, uint32_t* __restrict__ keys,
       int* __restrict__ band, unsigned int* __restrict__ nbad, HistAt at,
       uint32_t* __restrict__ hist) {
  __shared__ int s_lo, s_hi, s_bad;
  __shared__ uint32_t h[256];
  if (threadIdx.x == 0) {
    s_lo = dp.Nz;
    s_hi = -1;
    s_bad = 0;
  }
  if (threadIdx.x < 256) h[threadIdx.x] = 0;
  __syncthreads();
  int lo = dp.Nz, hi = -1, bad = 0;
#pragma unroll
  for (int i = 0; i < kSortItems / 1024; ++i) {
    const int j = blockIdx.x * kSortItems + i * 1024 + threadIdx.x;
    if (j >= n) break;
    int cA, cB;
    const uint32_t key = cell_key(dp, zc, pos, j, &cA, &cB);
    keys[j] = key;
    atomicAdd(&h[key & 255u], 1u);
    if (key >= (uint32_t)dp.ncells) ++bad;
    if (cB >= cA) {
      lo = min(lo, cA);
      hi = max(hi, cB);
    }
  }
  if (hi >= 0) {
    atomicMin(&s_lo, lo);
    atomicMax(&s_hi, hi);
  }
  if (bad) atomicAdd(&s_bad, bad);
  __syncthreads();
  if (threadIdx.x < 256) hist[at(threadIdx.x, blockIdx.x)] = h[threadIdx.x];
  if (threadIdx.x == 0) {
    // the band only widens, so a workgroup whose planes are already inside
    // it skips the (contended) atomics
    if (s_hi >= 0) {
      const int glo = __atomic_load_n(&band[0], __ATOMIC_RELAXED);
      const int ghi = __atomic_load_n(&band[1], __ATOMIC_RELAXED);
      if (s_lo < glo) atomicMin(&band[0], s_lo);
      if (s_hi > ghi) atomicMax(&band[1], s_hi);
    }
    if (s_bad) atomicAdd(nbad, (unsigned)s_bad);
  }
}

__global__ void k_init_band(int* band, unsigned int* nbad, int lo, int hi,
                            int reset_bad) {
  band[0] = lo;
  band[1] = hi;
  if (reset_bad) *nbad = 0u;
}

hipError_t launch_set_band(const fcmdp_solver* s, int lo, int hi,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_init_band, dim3(1), dim3(1), 0, st, s->band, s->nbad,
                     lo, hi, 0);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// zero fill (a kernel rather than a memset so that it is safe inside
// captured graphs)
// ----------------------------------------------------------------------------
__global__ void k_fill_zero(uint4* p, size_t n16, unsigned char* tail,
                            size_t ntail) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

hipError_t launch_fill(void* ptr, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  const size_t n16 = bytes / 16;
  const size_t ntail = bytes - n16 * 16;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, st,
                     (uint4*)ptr, n16, (unsigned char*)ptr + n16 * 16, ntail);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// Stable LSD radix sort, 8-bit digits.  Stable ranks inside a 64-item chunk
// come from eight ballots (lanes with an equal digit), chunk counts are
// prefix-summed per digit in LDS.
//
// Up to kSmallSort particles one workgroup does everything (keys, band and all
// passes, with the items in LDS): the launches of the general path, about 4 us
// each, were most of a small call's particle stage.  Beyond that a pass is a
// histogram and a scatter of 2048 items per workgroup; a scatter workgroup
// derives its offsets from the histograms itself while there are few of them
// (kFewBlocks), otherwise a kernel scans each digit's counts first.  Figures at
// launch_sort.
// ----------------------------------------------------------------------------
constexpr int kSmallSort = 4096;
constexpr int kFewBlocks = 64;

__global__ void __launch_bounds__(kSortThreads)
k_radix_hist(int n, const uint32_t* __restrict__ keys, int shift, HistAt at,
             uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int base = blockIdx.x * kSortItems;
  for (int i = threadIdx.x; i < kSortItems; i += kSortThreads) {
    const int g = base + i;
    if (g < n) atomicAdd(&h[(keys[g] >> shift) & 255u], 1u);
  }
  __syncthreads();
  hist[at(threadIdx.x, blockIdx.x)] = h[threadIdx.x];
}

// exclusive prefix sum of one value per thread over the first 256 threads
// (four wavefronts); every thread of the workgroup calls it
__device__ __forceinline__ uint32_t scan256(uint32_t v, uint32_t* part) {
  const int t = threadIdx.x, lane = t & 63;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (t < 256 && lane == 63) part[t >> 6] = x;
  __syncthreads();
  uint32_t base = 0;
  for (int w = 0; w < (t >> 6) && w < 4; ++w) base += part[w];
  return base + x - v;
}

// lanes of this wavefront with the same digit (among the active ones)
__device__ __forceinline__ uint64_t same_digit(int d, bool active) {
  uint64_t mask = __ballot(active);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const uint64_t bal = __ballot(((d >> b) & 1) != 0);
    mask &= ((d >> b) & 1) ? bal : ~bal;
  }
  return mask;
}

// FEW: hist holds the workgroups' counts; else their exclusive sums per digit,
// with the digits' totals in tot
template <bool FEW>
__global__ void __launch_bounds__(kSortThreads)
k_radix_scatter(int n, const uint32_t* __restrict__ kin,
                const int* __restrict__ vin, uint32_t* __restrict__ kout,
                int* __restrict__ vout, int shift, int nblk,
                const uint32_t* __restrict__ hist, const uint32_t* __restrict__ tot,
                int first_pass) {
  __shared__ uint32_t cnt[kSortChunks][256];
  __shared__ uint32_t boff[256];
  __shared__ uint32_t part[4];
  const int t = threadIdx.x;
  for (int i = t; i < kSortChunks * 256; i += kSortThreads)
    (&cnt[0][0])[i] = 0u;
  {
    uint32_t before = 0, total = 0;
    if constexpr (FEW) {
#pragma unroll 8
      for (int b = 0; b < nblk; ++b) {
        const uint32_t c = hist[b * 256 + t];
        before += b < (int)blockIdx.x ? c : 0u;
        total += c;
      }
    } else {
      before = hist[(size_t)t * nblk + blockIdx.x];
      total = tot[t];
    }
    boff[t] = before + scan256(total, part);
  }
  __syncthreads();

  const int lane = t & 63;
  const int wave = t >> 6;
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint32_t key[8];
  int val[8];
  int dig[8];
  int rank[8];
  const int base = blockIdx.x * kSortItems;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int q = wave * 8 + r;
    const int g = base + q * 64 + lane;
    const bool active = g < n;
    uint32_t k = active ? kin[g] : 0u;
    int v = active ? (first_pass ? g : vin[g]) : 0;
    const int d = (int)((k >> shift) & 255u);
    const uint64_t mask = same_digit(d, active);
    key[r] = k;
    val[r] = v;
    dig[r] = active ? d : -1;
    rank[r] = __popcll(mask & lt_mask);
    if (active && (mask & lt_mask) == 0ull)   // lowest lane of this digit
      cnt[q][d] = (uint32_t)__popcll(mask);
  }
  __syncthreads();
  {  // per digit: exclusive prefix over chunks
    uint32_t run = 0;
    for (int q = 0; q < kSortChunks; ++q) {
      const uint32_t c = cnt[q][t];
      cnt[q][t] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    if (dig[r] < 0) continue;
    const int q = wave * 8 + r;
    const uint32_t dst = boff[dig[r]] + cnt[q][dig[r]] + (uint32_t)rank[r];
    kout[dst] = key[r];
    vout[dst] = val[r];
  }
}

// workgroup d: exclusive scan of digit d's counts over the workgroups, and
// their total
__global__ void __launch_bounds__(256)
k_scan_digit(uint32_t* __restrict__ hist, int nblk, uint32_t* __restrict__ tot) {
  __shared__ uint32_t part[4], sum;
  uint32_t* a = hist + (size_t)blockIdx.x * nblk;
  const int t = threadIdx.x;
  uint32_t carry = 0;
  for (int base = 0; base < nblk; base += 256) {
    const int i = base + t;
    const uint32_t v = i < nblk ? a[i] : 0u;
    const uint32_t x = scan256(v, part);
    if (i < nblk) a[i] = carry + x;
    if (t == 255) sum = x + v;
    __syncthreads();
    carry += sum;
    __syncthreads();
  }
  if (t == 0) tot[blockIdx.x] = carry;
}

// keys, band, domain errors and the whole sort of n <= kSmallSort particles
template <typename Tin>
__global__ void __launch_bounds__(1024)
k_small_sort(DevParams dp, int n, const Tin* __restrict__ pos, const double* __restrict__ zc,
             uint32_t* __restrict__ keys, int* __restrict__ vals, int* __restrict__ band,
             unsigned int* __restrict__ nbad, int passes) {
  constexpr int kPer = kSmallSort / 1024, kChunks = kSmallSort / 64;
  __shared__ uint32_t skey[kSmallSort];
  __shared__ uint16_t sval[kSmallSort];
  __shared__ uint16_t cnt[kChunks][256];
  __shared__ uint32_t boff[256], part[4];
  __shared__ int s_lo, s_hi, s_bad;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (t == 0) {
    s_lo = dp.Nz;
    s_hi = -1;
    s_bad = 0;
  }
  __syncthreads();
  // item q * 64 + lane of chunk q = 16 r + wave
  const int chunks = (n + 63) / 64;
  uint32_t key[kPer];
  int val[kPer], lo = dp.Nz, hi = -1, bad = 0;
#pragma unroll 1
  for (int r = 0; r < kPer; ++r) {
    const int g = (16 * r + wave) * 64 + lane;
    if (16 * r >= chunks) break;                     // uniform
    uint32_t k = 0xffffffffu;
    if (g < n) {
      int cA, cB;
      k = cell_key(dp, zc, pos, g, &cA, &cB);
      if (k >= (uint32_t)dp.ncells) ++bad;
      if (cB >= cA) {
        lo = min(lo, cA);
        hi = max(hi, cB);
      }
    }
    skey[g] = k;
    sval[g] = (uint16_t)g;
  }
  if (hi >= 0) {
    atomicMin(&s_lo, lo);
    atomicMax(&s_hi, hi);
  }
  if (bad) atomicAdd(&s_bad, bad);
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  for (int pass = 0; pass < passes; ++pass) {
    const int shift = 8 * pass;
    for (int i = t; i < chunks * 128; i += 1024)
      reinterpret_cast<uint32_t*>(&cnt[0][0])[i] = 0u;
    __syncthreads();
    int rank[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      if (16 * r >= chunks) break;                   // uniform
      const int q = 16 * r + wave, g = q * 64 + lane;
      const bool active = g < n;
      key[r] = skey[g];
      val[r] = sval[g];
      const int d = (int)((key[r] >> shift) & 255u);
      const uint64_t mask = same_digit(d, active);
      rank[r] = __popcll(mask & lt_mask);
      if (active && (mask & lt_mask) == 0ull) cnt[q][d] = (uint16_t)__popcll(mask);
    }
    __syncthreads();
    uint32_t run = 0;
    if (t < 256)
      for (int q = 0; q < chunks; ++q) {
        const uint32_t c = cnt[q][t];
        cnt[q][t] = (uint16_t)run;
        run += c;
      }
    const uint32_t off = scan256(run, part);
    if (t < 256) boff[t] = off;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      const int q = 16 * r + wave, g = q * 64 + lane;
      if (g < n) {
        const int d = (int)((key[r] >> shift) & 255u);
        const int dst = boff[d] + cnt[q][d] + rank[r];
        skey[dst] = key[r];
        sval[dst] = (uint16_t)val[r];
      }
    }
    __syncthreads();
  }
  for (int g = t; g < n; g += 1024) {
    keys[g] = skey[g];
    vals[g] = sval[g];
  }
  if (t == 0) {
    band[0] = s_lo;
    band[1] = s_hi;
    *nbad = (unsigned)s_bad;
  }
}

// cell_start[c] = first sorted position with key >= c, for c = 0..ncells.  A
// workgroup takes kCellBlock consecutive cells: half of its threads each find
// the position of the first and of the past-the-end cell by a 128-ary search
// over all keys (three rounds for two million; a binary search is a chain of
// twenty dependent loads), then the threads search the keys between the two,
// in LDS where they fit.  These workgroups come first in the launch of
// k_records, which reads only the sorted keys too: as a kernel of their own they
// took 4 us of a small call's 125 and 19 us at 1M particles.
constexpr int kCellBlock = 1024, kCellKeys = 2048;
template <typename Keys>
__device__ __forceinline__ int lower_bound(const Keys& keys, int lo, int hi, uint32_t c) {
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (keys[mid] < c) lo = mid + 1; else hi = mid;
  }
  return lo;
}
__device__ __forceinline__ void cell_starts(int block, int n, int ncells,
                                            const uint32_t* __restrict__ keys,
                                            int* __restrict__ cell_start) {
  __shared__ int cnt[2][2];
  __shared__ uint32_t sk[kCellKeys];
  const int c0 = block * kCellBlock;
  const int side = threadIdx.x >> 7, t = threadIdx.x & 127;
  const uint32_t c = (uint32_t)(c0 + side * kCellBlock);
  int lo = 0, hi = n;                              // the answer is in [lo, hi]
  while (true) {
    const int len = hi - lo, step = len / 128 + 1;
    // probes lo + step - 1, lo + 2 step - 1, ...: how many lie below c
    const int p = lo + (t + 1) * step - 1;
    const uint64_t below = __ballot(p < hi && keys[p < hi ? p : 0] < c);
    if ((t & 63) == 0) cnt[side][t >> 6] = __popcll(below);
    __syncthreads();
    const int k = cnt[side][0] + cnt[side][1];
    hi = min(hi, lo + (k + 1) * step - 1);
    lo += k * step;
    if (!__syncthreads_or(step > 1)) break;          // step 1: lo is the answer
  }
  if (t == 0) cnt[side][0] = lo;
  __syncthreads();
  lo = cnt[0][0];
  hi = cnt[1][0];
  const int m = hi - lo;
  if (m <= kCellKeys) {
    for (int i = threadIdx.x; i < m; i += 256) sk[i] = keys[lo + i];
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < kCellBlock / 256; ++i) {
    const int cell = c0 + i * 256 + threadIdx.x;
    if (cell <= ncells)
      cell_start[cell] = m <= kCellKeys ? lo + lower_bound(sk, 0, m, (uint32_t)cell)
                                        : lower_bound(keys, lo, hi, (uint32_t)cell);
  }
}

// Keys, band and domain errors of all particles, then the sort (keyA, valA).
template <typename Tin>
static void sort_impl(const fcmdp_solver* s, int n, const Tin* pos, hipStream_t st) {
  if (n > 0 && n <= kSmallSort && !s->force_large_call) {
    hipLaunchKernelGGL(k_small_sort<Tin>, dim3(1), dim3(1024), 0, st, s->dp, n, pos, s->zc,
                       s->keyA, s->valA, s->band, s->nbad, s->key_passes);
  } else {
    hipLaunchKernelGGL(k_init_band, dim3(1), dim3(1), 0, st, s->band, s->nbad, s->dp.Nz, -1,
                       1);
    if (n == 0) return;
    const int nblk = (n + kSortItems - 1) / kSortItems;
    uint32_t* tot = s->hist + 256 * (size_t)s->nblk_cap;
    // an odd number of passes starts in the second buffers, so that the
    // result lies in keyA / valA
    const bool odd = s->key_passes & 1;
    uint32_t* kin = odd ? s->keyB : s->keyA;
    uint32_t* kout = odd ? s->keyA : s->keyB;
    int* vin = odd ? s->valB : s->valA;
    int* vout = odd ? s->valA : s->valB;
    const bool few = nblk <= kFewBlocks;
    const HistAt at = few ? HistAt{1, 256} : HistAt{nblk, 1};
    hipLaunchKernelGGL(k_prep<Tin>, dim3(nblk), dim3(1024), 0, st, s->dp, n, pos, s->zc, kin,
                       s->band, s->nbad, at, s->hist);
    for (int pass = 0; pass < s->key_passes; ++pass) {
      const int shift = 8 * pass;
      if (pass > 0)
        hipLaunchKernelGGL(k_radix_hist, dim3(nblk), dim3(kSortThreads), 0, st, n, kin, shift,
                           at, s->hist);
      if (few) {
        hipLaunchKernelGGL(k_radix_scatter<true>, dim3(nblk), dim3(kSortThreads), 0, st, n,
                           kin, vin, kout, vout, shift, nblk, s->hist, tot, pass == 0);
      } else {
        hipLaunchKernelGGL(k_scan_digit, dim3(256), dim3(256), 0, st, s->hist, nblk, tot);
        hipLaunchKernelGGL(k_radix_scatter<false>, dim3(nblk), dim3(kSortThreads), 0, st, n,
                           kin, vin, kout, vout, shift, nblk, s->hist, tot, pass == 0);
      }
      std::swap(kin, kout);
      std::swap(vin, vout);
    }
  }
}

// Keys, sort and the cell starts, which were a kernel of their own then (now in
// the launch of k_records), against one histogram, scan and scatter kernel per
// pass with a serial scan of the workgroup totals and a final copy: 61 -> 23 us
// at 1031 particles, 110 -> 63 at 17k, 125 -> 74 at 131k, 245 -> 141 at 1M.  Bound
// by launches up to some 10^5 particles, then by the scattered writes.
hipError_t launch_sort(const fcmdp_solver* s, int n, const void* pos, hipStream_t st) {
  if (s->mixed) sort_impl<float>(s, n, (const float*)pos, st);
  else sort_impl<double>(s, n, (const double*)pos, st);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// per-particle records in sorted order
// ----------------------------------------------------------------------------
// Four lanes build the records of one sorted particle and write each as
// whole 16-byte vectors (no LDS staging, so occupancy is limited by registers
// only and the scattered reads of the unsorted inputs overlap across many
// wavefronts).  The folded z weights are stored densely over all Nz nodes
// (zero outside the particle's window), so readers index them by node
// without window arithmetic.
__device__ __forceinline__ void store4(float* p, float a, float b, float c, float d) {
  *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}
__device__ __forceinline__ void store4(double* p, double a, double b, double c,
                                       double d) {
  reinterpret_cast<double2*>(p)[0] = make_double2(a, b);
  reinterpret_cast<double2*>(p)[1] = make_double2(c, d);
}

template <typename Tin, typename T>
__global__ void __launch_bounds__(256)
k_records(DevParams dp, int n, const uint32_t* __restrict__ skeys,
          const int* __restrict__ perm, const Tin* __restrict__ pos,
          const Tin* __restrict__ F, const Tin* __restrict__ Tq,
          const double* __restrict__ zc, int4* __restrict__ pinfo,
          T* __restrict__ pw, T* __restrict__ pf, T* __restrict__ psi,
          double* __restrict__ psi64, T* __restrict__ pdw, T* __restrict__ dpsi,
          int cell_blocks, int* __restrict__ cell_start) {
  if ((int)blockIdx.x < cell_blocks) {               // whole workgroup
    cell_starts(blockIdx.x, n, dp.ncells, skeys, cell_start);
    return;
  }
  // four lanes per particle (its quad): lane q writes x/y weight part q,
  // the z weights of the node groups q, q + 4, ... (four nodes each) and
  // its share of the other records, so that the kernel evaluations of one
  // particle run in four independent chains
  const int gid = (blockIdx.x - cell_blocks) * blockDim.x + threadIdx.x;
  const int i = gid >> 2, q = gid & 3;
  if (i >= n) return;
  const int Nz = dp.Nz;
  // FP64 z weights: the monopole's, and with torques spread through the
  // kernel derivative also the dipole's (the spread's FP64 vertical force
  // then carries their torque part)
  const int rows64 = dp.dt_torque ? 2 : 1;
  T* w = pw + (size_t)i * 32;
  T* f = pf + (size_t)i * 8;
  T* ps = psi + (size_t)i * 2 * Nz;
  double* ps64 = psi64 ? psi64 + (size_t)i * rows64 * Nz : nullptr;
  T* dw = pdw ? pdw + (size_t)i * 16 : nullptr;
  T* dps = dpsi ? dpsi + (size_t)i * Nz : nullptr;
  if (skeys[i] >= (uint32_t)dp.ncells) {
    // outside the domain: zero records (never read by the grid kernels)
    for (int e = 8 * q; e < 8 * q + 8; e += 4) store4(w + e, T(0), T(0), T(0), T(0));
    if (q < 2) store4(f + 4 * q, T(0), T(0), T(0), T(0));
    for (int e = q; e < 2 * Nz; e += 4) ps[e] = T(0);
    if (ps64)
      for (int e = q; e < rows64 * Nz; e += 4) ps64[e] = 0.0;
    if (dw)
      for (int e = q; e < 16; e += 4) dw[e] = T(0);
    if (dps)
      for (int e = q; e < Nz; e += 4) dps[e] = T(0);
    return;
  }
  const int j = perm[i];
  const double x = wrap_coord((double)pos[3 * (size_t)j + 0], dp.Lx);
  const double y = wrap_coord((double)pos[3 * (size_t)j + 1], dp.Ly);
  const double z = (double)pos[3 * (size_t)j + 2];
  int ix, iy;
  double fx, fy;
  cell_of(x, dp.h, dp.Nx, &ix, &fx);
  cell_of(y, dp.h, dp.Ny, &iy, &fy);
  int cA, cB;
  z_window(dp, zc, z, &cA, &cB);
  if (q == 0) pinfo[i] = make_int4(ix, iy, cA, cB);
  if (q < 2) {
    // forces (q = 0) and torques (q = 1), padded to four
    const Tin* src = q == 0 ? F : Tq;
    T a = T(0), b = T(0), c = T(0);
    if (src) {
      a = (T)src[3 * (size_t)j + 0];
      b = (T)src[3 * (size_t)j + 1];
      c = (T)src[3 * (size_t)j + 2];
    }
    store4(f + 4 * q, a, b, c, T(0));
  }
  // x or y weights of the M or D kernel (part q), 7 (eighth slot zero)
  {
    const double off = q & 1 ? fy : fx;
    const double beta = q < 2 ? dp.beta_m : dp.beta_d;
    const double inv = q < 2 ? dp.inv_norm_m : dp.inv_norm_d;
    T v[8];
#pragma unroll
    for (int d = 0; d < kWin; ++d)
      v[d] = es_eval<T>(((double)(d - 3) - off) * dp.h, dp.alpha, beta, inv);
    v[7] = T(0);
    store4(w + 8 * q, v[0], v[1], v[2], v[3]);
    store4(w + 8 * q + 4, v[4], v[5], v[6], v[7]);
  }
  // derivative of the dipole kernel along x (q = 0) and y (q = 1), truncated
  if (dw && q < 2) {
    const double off = q ? fy : fx;
    T v[8];
#pragma unroll
    for (int d = 0; d < kWin; ++d)
      v[d] = es_deval<T>(((double)(d - 3) - off) * dp.h, dp.alpha, dp.beta_d,
                         dp.inv_norm_d, dp.tstar_d);
    v[7] = T(0);
    store4(dw + 8 * q, v[0], v[1], v[2], v[3]);
    store4(dw + 8 * q + 4, v[4], v[5], v[6], v[7]);
  }
  // folded z weights
  const double zim_top = 2.0 * dp.H - z;
  auto zw = [&](int c, T& pm, T& pd) {
    pm = T(0);
    pd = T(0);
    if (c < cA || c > cB) return;
    const double zcv = zc[c];
    pm = es_eval<T>(zcv - z, dp.alpha, dp.beta_m, dp.inv_norm_m) -
         es_eval<T>(zcv + z, dp.alpha, dp.beta_m, dp.inv_norm_m);
    pd = es_eval<T>(zcv - z, dp.alpha, dp.beta_d, dp.inv_norm_d) -
         es_eval<T>(zcv + z, dp.alpha, dp.beta_d, dp.inv_norm_d);
    if (dp.geometry == 1) {
      pm -= es_eval<T>(zcv - zim_top, dp.alpha, dp.beta_m, dp.inv_norm_m);
      pd -= es_eval<T>(zcv - zim_top, dp.alpha, dp.beta_d, dp.inv_norm_d);
    }
  };
  if (Nz % 4 == 0) {
    // node groups of four: groups q, q + 4, ... of this lane
    for (int c = 4 * q; c < Nz; c += 16) {
      T pm[4], pd[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) zw(c + e, pm[e], pd[e]);
      store4(ps + c, pm[0], pm[1], pm[2], pm[3]);
      store4(ps + Nz + c, pd[0], pd[1], pd[2], pd[3]);
    }
  } else {
    for (int c = q; c < Nz; c += 4) zw(c, ps[c], ps[Nz + c]);
  }
  // the monopole z weights once more in FP64 (the exact low-wavenumber
  // vertical force of the mixed slit channel)
  if (ps64) {
    for (int row = 0; row < rows64; ++row) {
      const double beta = row ? dp.beta_d : dp.beta_m;
      const double inv = row ? dp.inv_norm_d : dp.inv_norm_m;
      auto p64 = [&](int c) {
        if (c < cA || c > cB) return 0.0;
        const double zcv = zc[c];
        double pm = es_eval<double>(zcv - z, dp.alpha, beta, inv) -
                    es_eval<double>(zcv + z, dp.alpha, beta, inv);
        if (dp.geometry == 1) pm -= es_eval<double>(zcv - zim_top, dp.alpha, beta, inv);
        return pm;
      };
      double* dst = ps64 + (size_t)row * Nz;
      if (Nz % 2 == 0) {
        // 16-byte stores (an even Nz keeps every row 16-byte aligned); node
        // pairs q, q + 4, ... of this lane
        double2* r2 = reinterpret_cast<double2*>(dst);
        for (int c = 2 * q; c < Nz; c += 8) r2[c / 2] = make_double2(p64(c), p64(c + 1));
      } else {
        for (int c = q; c < Nz; c += 4) dst[c] = p64(c);
      }
    }
  }
  // z derivative of the folded dipole kernel: the direct term's derivative
  // and the mirror images' (phi'(z_c - z) - phi'(z_c + z), minus
  // phi'(z_c - (2H - z)) between two walls)
  if (dps) {
    for (int c = q; c < Nz; c += 4) {
      T d = T(0);
      if (c >= cA && c <= cB) {
        const double zcv = zc[c];
        d = es_deval<T>(zcv - z, dp.alpha, dp.beta_d, dp.inv_norm_d, dp.tstar_d) -
            es_deval<T>(zcv + z, dp.alpha, dp.beta_d, dp.inv_norm_d, dp.tstar_d);
        if (dp.geometry == 1)
          d -= es_deval<T>(zcv - zim_top, dp.alpha, dp.beta_d, dp.inv_norm_d,
                           dp.tstar_d);
      }
      dps[c] = d;
    }
  }
}

template <typename Tin, typename T>
static void records_impl(const fcmdp_solver* s, int n, const void* pos,
                         const void* F, const void* Tq, hipStream_t st) {
  const int cell_blocks = s->dp.ncells / kCellBlock + 1;
  hipLaunchKernelGGL((k_records<Tin, T>), dim3(cell_blocks + (4 * (size_t)n + 255) / 256),
                     dim3(256), 0, st, s->dp, n, s->keyA, s->valA, (const Tin*)pos,
                     (const Tin*)F, (const Tin*)Tq, s->zc, s->pinfo,
                     (T*)s->pw, (T*)s->pf, (T*)s->psi,
                     s->dp.lowk_ns >= 0 ? s->psi64 : nullptr,
                     (s->dp.dt_torque || s->dp.dt_omega) ? (T*)s->pdw : nullptr,
                     (s->dp.dt_torque || s->dp.dt_omega) ? (T*)s->dpsi : nullptr,
                     cell_blocks, s->cell_start);
}

// The forces of the records alone, for another apply on the same positions.
template <typename T>
__global__ void __launch_bounds__(256)
k_forces(int n, int ncells, const uint32_t* __restrict__ skeys, const int* __restrict__ perm,
         const T* __restrict__ F, T* __restrict__ pf) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || skeys[i] >= (uint32_t)ncells) return;
  const T* f = F + 3 * (size_t)perm[i];
  store4(pf + 8 * (size_t)i, f[0], f[1], f[2], T(0));
}

hipError_t launch_forces(const fcmdp_solver* s, int n, const void* F, hipStream_t st) {
  const dim3 g((n + 255) / 256);
  if (s->mixed)
    hipLaunchKernelGGL(k_forces<float>, g, dim3(256), 0, st, n, s->dp.ncells, s->keyA,
                       s->valA, (const float*)F, (float*)s->pf);
  else
    hipLaunchKernelGGL(k_forces<double>, g, dim3(256), 0, st, n, s->dp.ncells, s->keyA,
                       s->valA, (const double*)F, (double*)s->pf);
  return hipGetLastError();
}

hipError_t launch_records(const fcmdp_solver* s, int n, const void* pos,
                          const void* F, const void* T, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (s->mixed)
    records_impl<float, float>(s, n, pos, F, T, st);
  else
    records_impl<double, double>(s, n, pos, F, T, st);
  return hipGetLastError();
}

}  // namespace fcmdp

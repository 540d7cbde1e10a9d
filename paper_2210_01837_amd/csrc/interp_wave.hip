// Interpolation with one wavefront per particle (step 8 of Sec. 3.4), for calls
// with few particles.
//
// Lanes 0..48 are the nodes of the particle's 7 x 7 window; every lane sums its
// column of nodes with the z weights (scalars of the wavefront), then applies
// its x/y weight, and the lanes are added.  A particle reads its whole window
// itself (7 rows of 28 bytes per plane and channel, from the L2), about four
// times the grid per particle at monolayer densities, but nothing is staged and
// no workgroup waits for another plane: the aligned tiles of interp_part.hip
// are too few workgroups there (18 on a 90 x 90 grid), each a chain of one
// staged plane after the other.  Figures and the line between the two at
// launch_interp.
#include "fcmdp_internal.h"

namespace fcmdp {

namespace {

// NCH = 6: velocities and angular velocities; 3: velocities, or (DT) Omega =
// (1/2) sum u x grad Delta_D through the derivative of the dipole kernel.
template <typename T, int NCH, bool DT>
__global__ void __launch_bounds__(256)
k_interp_wave(DevParams dp, int n, const uint32_t* __restrict__ skeys,
              const int* __restrict__ perm, const int4* __restrict__ pinfo,
              const T* __restrict__ pw, const T* __restrict__ psi,
              const T* __restrict__ pdw, const T* __restrict__ dpsi,
              const T* __restrict__ quad, const T* __restrict__ grid, T* __restrict__ U,
              T* __restrict__ Om) {
  const int lane = threadIdx.x & 63;
  const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (i >= n) return;
  const size_t j = (size_t)perm[i];
  if (skeys[i] >= (uint32_t)dp.ncells) {             // outside the domain
    if (lane < 3) {
      U[3 * j + lane] = T(NAN);
      if (Om) Om[3 * j + lane] = T(NAN);
    }
    return;
  }
  const int Nx = dp.Nx, Ny = dp.Ny, Nz = dp.Nz;
  const int4 inf = pinfo[i];
  const bool on = lane < 49;
  const int dx = on ? lane % 7 : 0, dy = on ? lane / 7 : 0;
  int x = inf.x - 3 + dx, y = inf.y - 3 + dy;
  x = x < 0 ? x + Nx : x >= Nx ? x - Nx : x;
  y = y < 0 ? y + Ny : y >= Ny ? y - Ny : y;
  const size_t plane = (size_t)Nx * Ny;
  const T* g = grid + (size_t)y * Nx + x;
  const T* zm = psi + (size_t)i * 2 * Nz;
  // column sums: velocities with the monopole weights, and with the dipole
  // weights the vorticity or (DT) the velocities again, with psi_D and psi_D'
  T a[3] = {0, 0, 0}, b[3] = {0, 0, 0}, d[3] = {0, 0, 0};
#pragma unroll 4
  for (int c = inf.z; c <= inf.w; ++c) {
    const T q = quad[c], wm = q * zm[c];
    const T wd = NCH == 6 || DT ? q * zm[Nz + c] : T(0);
    const T wq = DT ? q * dpsi[(size_t)i * Nz + c] : T(0);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      const T u = g[((size_t)ch * Nz + c) * plane];
      a[ch] = fma(wm, u, a[ch]);
      if constexpr (NCH == 6) b[ch] = fma(wd, g[((size_t)(ch + 3) * Nz + c) * plane], b[ch]);
      if constexpr (DT) {
        b[ch] = fma(wd, u, b[ch]);
        d[ch] = fma(wq, u, d[ch]);
      }
    }
  }
  const T* w = pw + (size_t)i * 32;
  const T wM = on ? w[dx] * w[8 + dy] : T(0);
  T o[6];
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) o[ch] = wM * a[ch];
  if constexpr (NCH == 6) {
    const T wD = on ? w[16 + dx] * w[24 + dy] : T(0);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) o[3 + ch] = wD * b[ch];
  }
  if constexpr (DT) {
    const T* v = pdw + (size_t)i * 16;
    const T h = on ? T(0.5) : T(0);
    const T wx = h * v[dx] * w[24 + dy], wy = h * w[16 + dx] * v[8 + dy];
    const T wz = h * w[16 + dx] * w[24 + dy];
    o[3] = fma(wz, d[1], -(wy * b[2]));
    o[4] = fma(wx, b[2], -(wz * d[0]));
    o[5] = fma(wy, b[0], -(wx * b[1]));
  }
  constexpr int NOUT = NCH == 6 || DT ? 6 : 3;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1)
#pragma unroll
    for (int e = 0; e < NOUT; ++e) o[e] += __shfl_xor(o[e], m);
  if (lane == 0) {
#pragma unroll
    for (int e = 0; e < 3; ++e) U[3 * j + e] = o[e];
    if constexpr (NOUT == 6)
      if (Om)
#pragma unroll
        for (int e = 0; e < 3; ++e) Om[3 * j + e] = o[3 + e];
  }
}

template <typename T, int NCH, bool DT>
void wave_launch(const fcmdp_solver* s, int n, const T* grid, T* U, T* Om, hipStream_t st) {
  hipLaunchKernelGGL((k_interp_wave<T, NCH, DT>), dim3((n + 3) / 4), dim3(256), 0, st, s->dp,
                     n, s->keyA, s->valA, s->pinfo, (const T*)s->pw, (const T*)s->psi,
                     (const T*)s->pdw, (const T*)s->dpsi, (const T*)s->quad, grid, U, Om);
}

template <typename T>
hipError_t wave_impl(const fcmdp_solver* s, int n, const T* grid, T* U, T* Om,
                     hipStream_t st) {
  if (Om && s->dp.dt_omega) wave_launch<T, 3, true>(s, n, grid, U, Om, st);
  else if (Om && s->dp.nch_out == 6) wave_launch<T, 6, false>(s, n, grid, U, Om, st);
  else wave_launch<T, 3, false>(s, n, grid, U, nullptr, st);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_interp_wave(const fcmdp_solver* s, int n, const void* grid, void* U,
                              void* Omega, hipStream_t st) {
  return s->mixed
             ? wave_impl<float>(s, n, (const float*)grid, (float*)U, (float*)Omega, st)
             : wave_impl<double>(s, n, (const double*)grid, (double*)U, (double*)Omega, st);
}

}  // namespace fcmdp

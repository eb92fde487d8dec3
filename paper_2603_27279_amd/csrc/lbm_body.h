// Device code of the lattice Boltzmann solver shared with the rods' force launch: the
// velocity set, a cell's moments, and the immersed-boundary stencil.
#pragma once
#include "lbm_internal.h"

namespace lbmx {

// D3Q19 in the order of lbm.h (the loops over i are unrolled, so every lookup
// is a compile-time constant).
__device__ __forceinline__ constexpr int CX(int i) {
  constexpr int v[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
  return v[i];
}
__device__ __forceinline__ constexpr int CY(int i) {
  constexpr int v[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
  return v[i];
}
__device__ __forceinline__ constexpr int CZ(int i) {
  constexpr int v[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
  return v[i];
}
__device__ __forceinline__ constexpr int OPP(int i) {
  constexpr int v[19] = {0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17};
  return v[i];
}
// The direction with the z component reversed (specular reflection).
__device__ __forceinline__ constexpr int FLIPZ(int i) {
  constexpr int v[19] = {0, 1, 2, 3, 4, 6, 5, 7, 8, 9, 10, 13, 14, 11, 12, 17, 18, 15, 16};
  return v[i];
}

__device__ __forceinline__ double weight(int i) {
  return i == 0 ? 1.0 / 3.0 : (i < 7 ? 1.0 / 18.0 : 1.0 / 36.0);
}

// Density and velocity (shifted by half the uniform force) of cell c of populations f.
__device__ __forceinline__ void cell_moments(const Lattice& L, const double* __restrict__ f, long c,
                                             double& rho, double& ux, double& uy, double& uz) {
  double mx = 0.0, my = 0.0, mz = 0.0;
  rho = 0.0;
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    const double v = f[i * L.cells + c];
    rho += v;
    mx += CX(i) * v; my += CY(i) * v; mz += CZ(i) * v;
  }
  ux = (mx + 0.5 * L.gx) / rho;
  uy = (my + 0.5 * L.gy) / rho;
  uz = (mz + 0.5 * L.gz) / rho;
}

// Peskin's four-point delta along one axis.
__device__ __forceinline__ double peskin4(double r) {
  r = fabs(r);
  if (r <= 1.0) return (3.0 - 2.0 * r + sqrt(1.0 + 4.0 * r - 4.0 * r * r)) * 0.125;
  if (r <= 2.0) return (5.0 - 2.0 * r - sqrt(-7.0 + 12.0 * r - 4.0 * r * r)) * 0.125;
  return 0.0;
}

// One node of the 4 x 4 x 4 stencil of position (x, y, z) per lane: lane k of
// the particle's wave takes x offset k & 3, y offset (k >> 2) & 3, z offset
// k >> 4 from floor - 1, so the 64 lanes of a wave touch 64 distinct nodes.
// Returns the node's cell index (wrapped periodically) and its weight
// (phi_z phi_y) phi_x. With walls in z a node beyond them takes no part: its
// weight is 0 (and its index clamped into the lattice).
__device__ __forceinline__ long stencil_node(const Lattice& L, double x, double y, double z, int k,
                                             double& w) {
  const int ox = k & 3, oy = (k >> 2) & 3, oz = k >> 4;
  const int nx = (int)floor(x) - 1 + ox, ny = (int)floor(y) - 1 + oy, nz = (int)floor(z) - 1 + oz;
  w = peskin4((double)nz - z) * peskin4((double)ny - y) * peskin4((double)nx - x);
  const int ix = ((nx % L.nx) + L.nx) % L.nx, iy = ((ny % L.ny) + L.ny) % L.ny;
  int iz;
  if (L.walls) {
    if (nz < 0 || nz >= L.nz) w = 0.0;
    iz = nz < 0 ? 0 : (nz >= L.nz ? L.nz - 1 : nz);
  } else {
    iz = ((nz % L.nz) + L.nz) % L.nz;
  }
  return ((long)iz * L.ny + iy) * L.nx + ix;
}

// Spread -scale F_p of every particle onto the force field g [3][cells], workgroup blk
// of 256 threads: one wave per particle, each lane adding its node's share with a
// hardware FP64 atomic (device memory from hipMalloc is coarse-grained, where these
// are exact adds; the sums agree to rounding with any order).
__device__ __forceinline__ void ibm_spread(const Lattice& L, const double* __restrict__ X,
                                           const double* __restrict__ F, long n, double scale,
                                           double* g, long blk) {
  const long t = blk * 256 + threadIdx.x;
  const long p = t >> 6;
  if (p >= n) return;
  const int k = (int)(t & 63);
  double w;
  const long c = stencil_node(L, X[p], X[n + p], X[2 * n + p], k, w);
  if (w == 0.0) return;  // outside the support, or beyond a wall
  const double fx = -scale * F[p], fy = -scale * F[n + p], fz = -scale * F[2 * n + p];
  unsafeAtomicAdd(&g[c], fx * w);
  unsafeAtomicAdd(&g[L.cells + c], fy * w);
  unsafeAtomicAdd(&g[2 * L.cells + c], fz * w);
}

}  // namespace lbmx

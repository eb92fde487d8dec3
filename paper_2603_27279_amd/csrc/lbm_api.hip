// Lattice Boltzmann fluid solver (Methods, "Lattice Boltzmann method"): one
// fused kernel per step. Each thread owns a cell: it reads the cell's 19
// populations (coalesced, SoA by direction), forms density and velocity (the
// velocity shifted by half the body force), relaxes towards the second-order
// equilibrium (BGK), adds Guo's forcing term and pushes every post-collision
// population to the neighbouring cell along its direction: for each direction
// consecutive threads write consecutive addresses, so the writes stay as
// coalesced as the reads. At a bounce-back wall the population comes back
// reversed at its own cell (less the moving lid's momentum term), at a
// free-slip wall with its z component reversed. 304 bytes move per cell update,
// 19 doubles in and 19 out; the kernel is bound by HBM bandwidth.
#include "rod.h"
#include "lbm.h"
#include "lbm_internal.h"
#include "lbm_body.h"

#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <string>

namespace lbmx {

__global__ __launch_bounds__(256) void k_lbm(Lattice L, const double* __restrict__ src,
                                             double* __restrict__ dst) {
  const long c = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= L.cells) return;
  const int x = (int)(c % L.nx);
  const long r = c / L.nx;
  const int y = (int)(r % L.ny), z = (int)(r / L.ny);
  double f[19];
#pragma unroll
  for (int i = 0; i < 19; ++i) f[i] = src[i * L.cells + c];
  double rho = 0.0, mx = 0.0, my = 0.0, mz = 0.0;
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    rho += f[i];
    mx += CX(i) * f[i]; my += CY(i) * f[i]; mz += CZ(i) * f[i];
  }
  double gx = L.gx, gy = L.gy, gz = L.gz;  // uniform force plus the spread field
  if (L.gfield) {
    gx += L.gfield[c]; gy += L.gfield[L.cells + c]; gz += L.gfield[2 * L.cells + c];
  }
  const double ux = (mx + 0.5 * gx) / rho, uy = (my + 0.5 * gy) / rho, uz = (mz + 0.5 * gz) / rho;
  const double uu = ux * ux + uy * uy + uz * uz, ug = ux * gx + uy * gy + uz * gz;
  const double omega = 1.0 / L.tau, pre = 1.0 - 0.5 / L.tau;
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    const double cu = CX(i) * ux + CY(i) * uy + CZ(i) * uz;
    const double cg = CX(i) * gx + CY(i) * gy + CZ(i) * gz;
    const double w = weight(i);
    const double feq = w * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu);
    const double fs = f[i] - omega * (f[i] - feq) + pre * w * (3.0 * (cg - ug) + 9.0 * cu * cg);
    int zd = z + CZ(i);
    if (L.walls && (zd < 0 || zd >= L.nz)) {
      if (zd >= L.nz && L.walls == 2) {  // free-slip top: z reversed, at this cell
        dst[FLIPZ(i) * L.cells + c] = fs;
      } else {  // halfway bounce-back, less 6 w rho (c . lid) at a moving top wall
        const double mv = zd >= L.nz ? 6.0 * w * rho * (CX(i) * L.lidx + CY(i) * L.lidy) : 0.0;
        dst[OPP(i) * L.cells + c] = fs - mv;
      }
      continue;
    }
    zd = (zd + L.nz) % L.nz;
    const int xd = (x + CX(i) + L.nx) % L.nx, yd = (y + CY(i) + L.ny) % L.ny;
    dst[i * L.cells + ((long)zd * L.ny + yd) * L.nx + xd] = fs;
  }
}

__global__ __launch_bounds__(256) void k_lbm_moments(Lattice L, const double* __restrict__ f,
                                                     double* rho_o, double* u_o) {
  const long c = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= L.cells) return;
  double rho, ux, uy, uz;
  cell_moments(L, f, c, rho, ux, uy, uz);
  rho_o[c] = rho;
  u_o[c] = ux;
  u_o[L.cells + c] = uy;
  u_o[2 * L.cells + c] = uz;
}

// ---------------------------------------------------------------- immersed boundary
// Fluid velocity at each particle: U(X) = sum over the 64 stencil nodes of
// u(x) delta(x - X). One wave per particle, the node terms summed across the wave;
// a lane forms its node's velocity from the 19 populations. The alternative, a pass that
// first takes the velocity of every cell (u set), moves 184 B per cell, near a particle
// or not, but forms a node's velocity once, where close particles share it. 10,314
// particles, pass and read against direct: 73 and 30 us at 152 cells per particle, 31
// and 29 at 64, 22 and 26 at 32, 19 and 21 at 16, 17 and 18 at 8 (and the pass is one
// launch more).
template <bool PASS>
__global__ __launch_bounds__(256) void k_ibm_interp(Lattice L, const double* __restrict__ f,
                                                   const double* __restrict__ u,
                                                   const double* __restrict__ X, long n,
                                                   double* U) {
  const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long p = t >> 6;
  if (p >= n) return;  // whole waves: 64 divides the block size
  const int k = (int)(t & 63);
  double w;
  const long c = stencil_node(L, X[p], X[n + p], X[2 * n + p], k, w);
  double ux, uy, uz;
  if constexpr (PASS) {
    ux = u[c]; uy = u[L.cells + c]; uz = u[2 * L.cells + c];
  } else {
    double rho;
    cell_moments(L, f, c, rho, ux, uy, uz);
  }
  double ax = ux * w, ay = uy * w, az = uz * w;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    ax += __shfl_xor(ax, o);
    ay += __shfl_xor(ay, o);
    az += __shfl_xor(az, o);
  }
  if (k == 0) {
    U[p] = ax; U[n + p] = ay; U[2 * n + p] = az;
  }
}

__global__ __launch_bounds__(256) void k_ibm_spread(Lattice L, const double* __restrict__ X,
                                                   const double* __restrict__ F, long n,
                                                   double scale, double* g) {
  ibm_spread(L, X, F, n, scale, g, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_fill0(double* a, long n) {
  const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) a[k] = 0.0;
}

}  // namespace lbmx

using namespace lbmx;

namespace lbmx {
static unsigned blocks_of(long n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_lbm_step(lbm_ctx* c, const double* gfield, hipStream_t s) {
  Lattice L = c->L;
  L.gfield = gfield;
  hipLaunchKernelGGL(k_lbm, dim3(blocks_of(L.cells)), dim3(256), 0, s, L,
                     (const double*)c->f[c->cur], c->f[1 - c->cur]);
  c->cur = 1 - c->cur;
  return hipGetLastError();
}
hipError_t launch_lbm_moments(const lbm_ctx* c, double* rho, double* u, hipStream_t s) {
  hipLaunchKernelGGL(k_lbm_moments, dim3(blocks_of(c->L.cells)), dim3(256), 0, s, c->L,
                     (const double*)c->f[c->cur], rho, u);
  return hipGetLastError();
}
hipError_t launch_ibm_interp(const lbm_ctx* c, double* rho, double* u, const double* X, long n,
                             double* U, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const double* f = c->f[c->cur];
  if (32 * n <= c->L.cells) {  // (measured at k_ibm_interp)
    hipLaunchKernelGGL(k_ibm_interp<false>, dim3(blocks_of(64 * n)), dim3(256), 0, s, c->L, f,
                       (const double*)nullptr, X, n, U);
    return hipGetLastError();
  }
  hipError_t e = launch_lbm_moments(c, rho, u, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_ibm_interp<true>, dim3(blocks_of(64 * n)), dim3(256), 0, s, c->L, f,
                     (const double*)u, X, n, U);
  return hipGetLastError();
}
hipError_t launch_ibm_spread(const lbm_ctx* c, const double* X, const double* F, long n,
                             double scale, double* g, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_ibm_spread, dim3(blocks_of(64 * n)), dim3(256), 0, s, c->L, X, F, n, scale, g);
  return hipGetLastError();
}
hipError_t launch_fill0(double* a, long n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill0, dim3(blocks_of(n)), dim3(256), 0, s, a, n);
  return hipGetLastError();
}
}  // namespace lbmx


static thread_local std::string g_lbm_err;

static int lfail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_lbm_err = buf;
  return code;
}

#define LHIP(x)                                                                     \
  do {                                                                              \
    hipError_t e_ = (x);                                                            \
    if (e_ != hipSuccess) return lfail(ROD_E_HIP, "%s: %s", #x, hipGetErrorString(e_)); \
  } while (0)

static unsigned lblocks(long cells) { return (unsigned)((cells + 255) / 256); }

extern "C" {

const char* lbm_last_error(void) { return g_lbm_err.c_str(); }

int lbm_init(lbm_ctx** out, const lbm_desc* d, const double* f0, void* hip_stream) {
  if (!out || !d || !f0) return lfail(ROD_E_INVALID, "NULL argument");
  *out = nullptr;
  if (d->nx < 1 || d->ny < 1 || d->nz < 1) return lfail(ROD_E_INVALID, "nx, ny, nz must be >= 1");
  const long cells = (long)d->nx * d->ny * d->nz;
  if (cells > 2147483647L) return lfail(ROD_E_INVALID, "more than 2^31 - 1 cells");
  if (!(d->tau > 0.5) || !std::isfinite(d->tau)) return lfail(ROD_E_INVALID, "tau must be > 1/2");
  for (int k = 0; k < 3; ++k)
    if (!std::isfinite(d->force[k])) return lfail(ROD_E_INVALID, "force must be finite");
  if (d->walls_z < 0 || d->walls_z > 2) return lfail(ROD_E_INVALID, "walls_z must be 0, 1 or 2");
  if (!std::isfinite(d->lid_velocity[0]) || !std::isfinite(d->lid_velocity[1]))
    return lfail(ROD_E_INVALID, "lid_velocity must be finite");
  if ((d->lid_velocity[0] != 0.0 || d->lid_velocity[1] != 0.0) && d->walls_z != 1)
    return lfail(ROD_E_INVALID, "a lid velocity needs walls_z = 1 (a no-slip top wall)");
  lbm_ctx* c = new lbm_ctx();
  c->L = Lattice{d->nx, d->ny, d->nz, d->walls_z, cells, d->tau, d->force[0], d->force[1],
                 d->force[2], nullptr, d->lid_velocity[0], d->lid_velocity[1]};
  c->s = (hipStream_t)hip_stream;
  const size_t bytes = 19 * sizeof(double) * (size_t)cells;
  hipError_t e = hipMalloc(&c->f[0], bytes);
  if (e == hipSuccess) e = hipMalloc(&c->f[1], bytes);
  if (e == hipSuccess) e = hipMemcpyAsync(c->f[0], f0, bytes, hipMemcpyDeviceToDevice, c->s);
  if (e != hipSuccess) {
    if (c->f[0]) (void)hipFree(c->f[0]);
    if (c->f[1]) (void)hipFree(c->f[1]);
    delete c;
    return lfail(ROD_E_HIP, "allocation or copy failed: %s", hipGetErrorString(e));
  }
  *out = c;
  return ROD_OK;
}

int lbm_step(lbm_ctx* c, int64_t n) {
  if (!c) return lfail(ROD_E_INVALID, "context is NULL");
  if (n < 0) return lfail(ROD_E_INVALID, "n must be >= 0");
  for (int64_t k = 0; k < n; ++k) {
    hipLaunchKernelGGL(k_lbm, dim3(lblocks(c->L.cells)), dim3(256), 0, c->s, c->L,
                       (const double*)c->f[c->cur], c->f[1 - c->cur]);
    LHIP(hipGetLastError());
    c->cur = 1 - c->cur;
  }
  return ROD_OK;
}

int lbm_populations(lbm_ctx* c, double* f) {
  if (!c || !f) return lfail(ROD_E_INVALID, "NULL argument");
  LHIP(hipMemcpyAsync(f, c->f[c->cur], 19 * sizeof(double) * (size_t)c->L.cells,
                      hipMemcpyDeviceToDevice, c->s));
  return ROD_OK;
}

int lbm_moments(lbm_ctx* c, double* rho, double* u) {
  if (!c || !rho || !u) return lfail(ROD_E_INVALID, "NULL argument");
  hipLaunchKernelGGL(k_lbm_moments, dim3(lblocks(c->L.cells)), dim3(256), 0, c->s, c->L,
                     (const double*)c->f[c->cur], rho, u);
  LHIP(hipGetLastError());
  return ROD_OK;
}

int lbm_free(lbm_ctx* c) {
  if (!c) return ROD_OK;
  (void)hipStreamSynchronize(c->s);
  (void)hipDeviceSynchronize();  // a coupled cycle may have used it on another stream
  (void)hipFree(c->f[0]);
  (void)hipFree(c->f[1]);
  if (c->work) (void)hipFree(c->work);
  delete c;
  return ROD_OK;
}

}  // extern "C"

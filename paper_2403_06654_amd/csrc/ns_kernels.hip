// Pointwise kernels of the fractional-step driver (gfx950, FP64): linear
// combinations, a norm and the manufactured Taylor-Green fields.
// These are memory-bound elementwise passes; each thread handles one point
// (grid-stride loops), reads are coalesced along x.
#include <hip/hip_runtime.h>

#include <cmath>

#include "ns.hpp"
#include "vd_common.hpp"

namespace vd {

namespace {

constexpr int kT = 256;

inline unsigned grid_of(size_t n) {
  size_t b = (n + kT - 1) / kT;
  return (unsigned)(b < 65536 ? b : 65536);
}

__global__ __launch_bounds__(kT) void k_lincomb(LinArgs a) {
  for (size_t e = blockIdx.x * (size_t)kT + threadIdx.x; e < a.n; e += (size_t)gridDim.x * kT) {
    double s = 0.0;
    for (int t = 0; t < a.nt; ++t) s += a.c[t] * a.in[t][e];
    a.out[e] = s;
  }
}

__global__ __launch_bounds__(kT) void k_recip(const double* __restrict__ x, double* __restrict__ out, size_t n) {
  for (size_t e = blockIdx.x * (size_t)kT + threadIdx.x; e < n; e += (size_t)gridDim.x * kT) out[e] = 1.0 / x[e];
}

__global__ __launch_bounds__(kT) void k_tg(int n, double t, double s, double* __restrict__ u, double* __restrict__ p,
                                           double* __restrict__ rho, double* __restrict__ du,
                                           double* __restrict__ drho) {
  const size_t N = (size_t)n * n * n;
  const double h = 2.0 * M_PI / n;
  const double ct = cos(t), st = sin(t);
  for (size_t e = blockIdx.x * (size_t)kT + threadIdx.x; e < N; e += (size_t)gridDim.x * kT) {
    const int ix = (int)(e % n), iy = (int)((e / n) % n), iz = (int)(e / ((size_t)n * n));
    const double x = ix * h, y = iy * h, z = iz * h;
    const double sx = sin(x), cx = cos(x), sy = sin(y), cy = cos(y), sz = sin(z), cz = cos(z);
    u[e] = ct * sx * cy * cz;
    u[N + e] = ct * cx * sy * cz;
    u[2 * N + e] = -2.0 * ct * cx * cy * sz;
    p[e] = st * sin(2.0 * x) * sin(2.0 * y) * sin(2.0 * z);
    rho[e] = 1.0 + 0.5 * (s - 1.0) * (1.0 + st * sx * sy * sz);
    if (du) {
      du[e] = -st * sx * cy * cz;
      du[N + e] = -st * cx * sy * cz;
      du[2 * N + e] = 2.0 * st * cx * cy * sz;
    }
    if (drho) drho[e] = 0.5 * (s - 1.0) * ct * sx * sy * sz;
  }
}

// Each block reduces its contiguous share of the entries in a fixed order
// (strided per thread, then the block tree).
__global__ __launch_bounds__(kT) void k_square(const double* __restrict__ x, size_t n, double* __restrict__ part) {
  __shared__ double sh[kT];
  const int b = blockIdx.x, nb = gridDim.x;
  const size_t chunk = (n + nb - 1) / nb;
  const size_t lo = (size_t)b * chunk, hi = lo + chunk < n ? lo + chunk : n;
  double acc = 0.0;
  for (size_t e = lo + threadIdx.x; e < hi; e += kT) acc += x[e] * x[e];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int o = kT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[b] = sh[0];
}

}  // namespace

void ns_lincomb(const LinArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_lincomb, dim3(grid_of(a.n)), dim3(kT), 0, st, a);
}

void ns_recip(const double* x, double* out, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_recip, dim3(grid_of(n)), dim3(kT), 0, st, x, out, n);
}

void ns_tg_fields(int n, double t, double s, double* u, double* p, double* rho, double* du, double* drho,
                  hipStream_t st) {
  const size_t N = (size_t)n * n * n;
  hipLaunchKernelGGL(k_tg, dim3(grid_of(N)), dim3(kT), 0, st, n, t, s, u, p, rho, du, drho);
}

int ns_dot_blocks(size_t n) {
  size_t b = (n + 8 * kT - 1) / (8 * kT);
  return (int)(b < 1024 ? (b > 0 ? b : 1) : 1024);
}

void ns_square(const double* x, size_t n, double* part, int nb, hipStream_t st) {
  hipLaunchKernelGGL(k_square, dim3(nb), dim3(kT), 0, st, x, n, part);
}

}  // namespace vd

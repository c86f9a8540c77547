// Kernels of the fractional-step driver (ns.cpp): fused FP64 spectral passes
// (ns_passes.hip) and pointwise kernels, reductions and the manufactured
// Taylor-Green fields (eq. VDINSE.solexact; ns_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

#include "../../include/vdsolve.h"
#include "passes.hpp"

namespace vd {

// Transforms and geometry of a grid made by vd_grid_create (vdsolve.cpp).
const Geom& grid_geom(const vd_grid* G);
const void* grid_twiddles(const vd_grid* G);

// vd_solve_pressure (direct form, Fourier grid) from and to packed spectra on
// the grid's stream; x0hat: the initial guess if opts->use_x0.
vd_status grid_solve_pressure_spec(vd_grid* G, const void* fhat, const void* x0hat, void* phat,
                                   const vd_solve_opts* opts, vd_solve_info* info);

// A stack is nf fields one after another, `stride` slots (one packed field)
// apart.  Grids are n^3, n a power of two in [16, 512].  gate (optional): a
// nonzero device flag makes the launch do nothing.

// z pass of a stack: t0 = Fz^-1 v, t1 = Fz^-1 (i k'_z v), t2 = Fz^-1 (-k_z^2 v)
// (hess: -k'_z^2), v = in * *in_scale, with precond also (I - nu Lap)^-1;
// outputs separate from in.
struct NsZArgs {
  const void* in;
  void *t0, *t1, *t2;
  size_t stride;
  Geom g;
  double nu = 0;
  int precond = 0;
  const double* in_scale = nullptr;
  const int* gate = nullptr;
};
void ns_z_pass(const NsZArgs& a, int nf, bool hess, const void* tw, hipStream_t st);

// y pass on its output, in place: t0 -> Fy^-1 t0, t1 -> Fy^-1 t1,
// y1 = Fy^-1 (i k'_y t0) and t2 -> Fy^-1 (t2 - k_y^2 t0); hess: t2 -> Fy^-1 t2,
// y2 = Fy^-1 (-k'_y^2 t0), y3 = Fy^-1 (i k'_y t1).
struct NsYArgs {
  void *t0, *t1, *t2, *y1, *y2 = nullptr, *y3 = nullptr;
  size_t stride;
  Geom g;
  const int* gate = nullptr;
};
void ns_y_pass(const NsYArgs& a, int nf, bool hess, const void* tw, hipStream_t st);

// x pass of zeta (eq. VDINSE.zeta) on three components' rows (y0, yy, yz, yl:
// stacks t0, y1, t1, t2 of the y pass):
//   out_i = a u_i + b W (Lap u_i + (sum_j u_j h_ij + sum_j gr_j d_j u_i) inv_sc),
// W = ir = 1 / rho, or 1 with unit (b takes 1 / Re); with rhs also
//   + ca n_i + cp nprev_i + cg d_i p / rho + ce ext_i,  n_i = (u . grad) u_i,
// p0, py, pz the rows of p's gradient (grad_rows), n_i written to nout; nprev,
// ext and nout are optional.  gr, h, ir, nprev, ext, nout: physical.  out: rows
// transformed along x, or physical.
struct NsZetaArgs {
  const void *y0, *yy, *yz, *yl;
  size_t stride;  // slots per field
  size_t n;       // grid points
  const double *gr, *h, *ir;
  double a, b, inv_sc, norm, sx;
  bool unit = false;
  const void *p0 = nullptr, *py = nullptr, *pz = nullptr;
  const double *nprev = nullptr, *ext = nullptr;
  double ca = 0, cp = 0, cg = 0, ce = 0;
  double* nout = nullptr;
  void* out;
  const int* gate = nullptr;
};
void ns_zeta_pass(const Geom& g, const NsZetaArgs& a, bool rhs, bool phys, const void* tw, hipStream_t st);

// x pass of a density's coefficients from the hess passes' rows: rho,
// ir = 1 / rho, gradient gr (3) and Hessian h (00 01 02 11 12 22).
struct NsCoefArgs {
  const void *y0, *t1, *t2, *y1, *y2, *y3;
  double *rho, *ir, *gr, *h;
  size_t n;
  double norm, sx;
};
void ns_coef_pass(const Geom& g, const NsCoefArgs& a, const void* tw, hipStream_t st);

// x pass of (u . grad) q: y0 the stack of u's rows; q0, qy, qz the rows of q's
// gradient; out: rows transformed along x.
struct NsAdvArgs {
  const void* y0;
  size_t stride;
  const void *q0, *qy, *qz;
  double norm, sx;
  void* out;
};
void ns_advect_pass(const Geom& g, const NsAdvArgs& a, const void* tw, hipStream_t st);

// x pass of grad(q) / rho (ir = 1 / rho), a stack of three; rows
// transformed along x, or physical.
struct NsGradArgs {
  const void *q0, *qy, *qz;
  const double* ir;
  double norm, sx;
  size_t stride;
  void* out;
};
void ns_grad_pass(const Geom& g, const NsGradArgs& a, bool phys, const void* tw, hipStream_t st);

// Spectral pointwise steps.  Crank-Nicolson density (c = dt / (2 Re Sc)):
// rho1 = ((1 - c k^2) rho + s S + sa na + sb nb) / (1 + c k^2) (S, nb
// optional), rhm = (rho + rho1) / 2.
struct NsDensArgs {
  const void *rho, *S, *na, *nb;
  double c, s, sa, sb;
  void *rho1, *rhm;
  Geom g;
  size_t n;  // slots
};
void ns_density(const NsDensArgs& a, hipStream_t st);
// out = c i k' . v of a stack of three
void ns_div(const Geom& g, const void* v, size_t stride, double c, void* out, hipStream_t st);
// p += phi - (div grad)^-1 div v
void ns_pressure(const Geom& g, const void* v, size_t stride, const void* phi, void* p, hipStream_t st);

// out = sum_t c_t in_t (up to 3 terms); out may alias an input.
struct LinArgs {
  int nt = 0;
  const double* in[3] = {};
  double c[3] = {};
  double* out = nullptr;
  size_t n = 0;
};
void ns_lincomb(const LinArgs& a, hipStream_t st);

// out = 1 / x
void ns_recip(const double* x, double* out, size_t n, hipStream_t st);

// eq. VDINSE.solexact on the n^3 grid of [0, 2 pi)^3 at time t: u (3 fields
// one after another), p, rho, and when non-null the time derivatives du (3
// fields) and drho.
void ns_tg_fields(int n, double t, double s, double* u, double* p, double* rho, double* du, double* drho,
                  hipStream_t st);

// part[b] = sum over block b's share of x . x, in a fixed order within a block.
int ns_dot_blocks(size_t n);
void ns_square(const double* x, size_t n, double* part, int nb, hipStream_t st);

}  // namespace vd

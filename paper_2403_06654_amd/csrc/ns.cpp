// Host driver of the fractional-step scheme for the variable-density
// incompressible Navier-Stokes equations on [0, 2 pi)^3 (Sec. 2):
//   1. advection terms at n+1/2 by Adams-Bashforth (Euler on the first step);
//   2. Crank-Nicolson density (eq. VDINSE.num.mass.proj), a diagonal solve in
//      Fourier space;
//   3. rho^(n+1/2) = (rho^(n+1) + rho^n) / 2;
//   4. intermediate velocity (eq. VDINSE.num.momentum.proj): the implicit
//      viscous system u* - dt/2 zeta(rho^(n+1/2), u*) = rhs, by right-
//      preconditioned GMRES with (I - dt/(2 Re) Lap)^-1 (eq. VDINSE.V) from u^n;
//   5. L_rho phi = div(u*) / dt (eq. VDINSE.Lrho.num) by the pressure solver
//      of this library, warm-started from the previous phi;
//   6. u^(n+1) = u* - dt grad(phi) / rho^(n+1/2) (eq. VDINSE.num.proj);
//   7. p^(n+1/2) = p^(n-1/2) + phi - (div grad)^-1 div(dt/2 rho zeta(rho,
//      grad(phi) / rho)) (eq. VDINSE.num.p.update, scalar form).
// zeta is eq. VDINSE.zeta.  Derivatives are spectral (first derivatives with
// the Nyquist mode zeroed, the Laplacian with it kept).
//
// Between steps the state is kept as packed spectra: linear steps (the density,
// the divergence, the projection and the pressure update) act on them directly,
// and a product is formed by the fused passes of ns_passes.hip, which take each
// factor and all its derivatives to physical space in one sweep per axis.  The
// physical fields of the state are brought up to date at the end of a call.
// The viscous system's Krylov vectors are stacks of three spectra in the
// Gram-Schmidt, stopping-test and mailbox machinery of the other solvers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <initializer_list>
#include <new>
#include <utility>
#include <vector>

#include "../../include/vdsolve.h"
#include "mail.hpp"
#include "ns.hpp"

using namespace vd;

struct vd_ns {
  int n = 0;
  size_t N = 0, ns = 0;  // grid points; slots of a packed field (N / 2)
  vd_ns_params prm{};
  hipStream_t st = nullptr;
  vd_grid* grid = nullptr;
  Geom g{}, g3{};  // g3: a stack of three fields as one vector of the Krylov kernels
  const void* tw = nullptr;
  std::vector<void*> allocs;
  // state u^n (3 fields), rho^n, p^(n-1/2): physical, and as spectra (uh, rhoh,
  // ph) with the last phi (phih) and the previous advection terms (the velocity's
  // physical, nu; the density's spectral, nrh; [0] the newest)
  double *u = nullptr, *rho = nullptr, *p = nullptr;
  double *uh = nullptr, *rhoh = nullptr, *ph = nullptr, *phih = nullptr;
  double* nu[2] = {};
  double* nrh[2] = {};
  bool have_prev = false, have_state = false;
  bool spec = false;  // the spectra hold the state (else they are built from the physical fields)
  double t = 0;
  int steps = 0;
  // coefficients of a density: its values, gradient (3), Hessian (00 01 02 11 12 22), 1 / rho
  double *rh = nullptr, *cg = nullptr, *ch = nullptr, *cir = nullptr;
  // scratch: spectra of rho^(n+1) and rho^(n+1/2); rows of three components
  // (stacks T, Tz, Tl, Ty) and of a scalar's gradient (3); stacks of three
  double *rho1h = nullptr, *rhh = nullptr;
  double *T = nullptr, *Tz = nullptr, *Tl = nullptr, *Ty = nullptr, *pr = nullptr;
  double *bh = nullptr, *q3 = nullptr, *x3h = nullptr, *z3 = nullptr;
  double *f = nullptr, *Sf = nullptr, *Sh = nullptr;  // body force (physical), mass source (physical, spectrum)
  double* V = nullptr;  // GMRES basis, (restart + 1) stacks of three spectra
  double* part = nullptr;
  DevState* dst = nullptr;
  Mail* mail = nullptr;
  unsigned long long posts = 0;
  int nb = 0;
  std::vector<double> hpart;
  vd_ns_info last{};
  // optional HIP-event timing by class: 0 FFT transform passes, 1 pressure
  // solves, 2 viscous Krylov inner products and updates
  struct Pend {
    int cls;
    double bytes;
    hipEvent_t a, b;
  };
  bool prof = false;
  std::vector<Pend> pend;
  std::vector<hipEvent_t> spare;
  double pms[3] = {0, 0, 0}, pbytes[3] = {0, 0, 0};
  long long pcnt[3] = {0, 0, 0};
};

namespace {

struct Err {
  vd_status s;
};

inline void ck(hipError_t e) {
  if (e != hipSuccess) throw Err{VD_EDEVICE};
}

double* dalloc(vd_ns* h, size_t count) {
  void* p = nullptr;
  if (hipMalloc(&p, count * sizeof(double)) != hipSuccess) {
    hipGetLastError();
    throw Err{VD_ENOMEM};
  }
  h->allocs.push_back(p);
  return (double*)p;
}

void release(vd_ns* h) {
  for (auto& p : h->pend) {
    hipEventDestroy(p.a);
    hipEventDestroy(p.b);
  }
  for (hipEvent_t e : h->spare) hipEventDestroy(e);
  for (void* p : h->allocs) hipFree(p);
  if (h->mail) hipHostFree(h->mail);
  if (h->grid) vd_grid_destroy(h->grid);
  delete h;
}

hipEvent_t ev(vd_ns* h) {
  if (!h->spare.empty()) {
    hipEvent_t e = h->spare.back();
    h->spare.pop_back();
    return e;
  }
  hipEvent_t e;
  ck(hipEventCreate(&e));
  return e;
}

// Bracket the work launched by fn with events when profiling.
template <class F>
void timed(vd_ns* h, int cls, double bytes, F fn) {
  if (!h->prof) {
    fn();
    return;
  }
  vd_ns::Pend p{cls, bytes, ev(h), ev(h)};
  ck(hipEventRecord(p.a, h->st));
  fn();
  ck(hipEventRecord(p.b, h->st));
  h->pend.push_back(p);
}

void prof_flush(vd_ns* h) {
  for (auto& p : h->pend) {
    float ms = 0.f;
    ck(hipEventElapsedTime(&ms, p.a, p.b));
    h->pms[p.cls] += ms;
    h->pbytes[p.cls] += p.bytes;
    h->pcnt[p.cls] += 1;
    h->spare.push_back(p.a);
    h->spare.push_back(p.b);
  }
  h->pend.clear();
}
// Forget the records after the first n: launches that exited at their gate.
void prof_drop(vd_ns* h, size_t n) {
  for (size_t i = n; i < h->pend.size(); ++i) {
    h->spare.push_back(h->pend[i].a);
    h->spare.push_back(h->pend[i].b);
  }
  if (h->pend.size() > n) h->pend.resize(n, vd_ns::Pend{0, 0.0, nullptr, nullptr});
}

// Algorithmic bytes of a group of passes that reads and writes `fields` fields.
double fields_bytes(const vd_ns* h, double fields) { return 8.0 * (double)h->N * fields; }
// One whole transform: three passes, each reading and writing the field.
constexpr double kTransform = 6.0;

void fwd(vd_ns* h, const double* phys, void* spec) {
  timed(h, 0, fields_bytes(h, kTransform), [&] { fwd_transform(h->g, phys, spec, nullptr, h->tw, h->st); });
}
void inv(vd_ns* h, const void* spec, double* phys) {
  timed(h, 0, fields_bytes(h, kTransform), [&] { inv_transform(h->g, spec, phys, h->T, h->tw, h->st); });
}
// stacks of three fields
void fwd3(vd_ns* h, const double* phys, double* spec) {
  const double* in[3] = {phys, phys + h->N, phys + 2 * h->N};
  void* o[3] = {spec, spec + h->N, spec + 2 * h->N};
  timed(h, 0, fields_bytes(h, 3 * kTransform), [&] { fwd_transform_n(h->g, in, o, 3, h->tw, h->st); });
}
void inv3(vd_ns* h, const double* spec, double* phys) {
  const void* in[3] = {spec, spec + h->N, spec + 2 * h->N};
  void* wk[3] = {h->T, h->T + h->N, h->T + 2 * h->N};
  double* o[3] = {phys, phys + h->N, phys + 2 * h->N};
  timed(h, 0, fields_bytes(h, 3 * kTransform), [&] { inv_transform_n(h->g, in, o, wk, 3, h->tw, h->st); });
}
// y and z transforms of nf fields already transformed along x
void fwd_columns(vd_ns* h, double* spec, int nf, const int* gate = nullptr) {
  void* o[3] = {spec, spec + h->N, spec + 2 * h->N};
  timed(h, 0, fields_bytes(h, 4.0 * nf), [&] { fwd_columns_n(h->g, o, nf, h->tw, h->st, gate); });
}

void lin(vd_ns* h, double* out, size_t n, std::initializer_list<std::pair<double, const double*>> terms) {
  LinArgs a;
  for (auto& t : terms) {
    a.c[a.nt] = t.first;
    a.in[a.nt++] = t.second;
  }
  a.out = out;
  a.n = n;
  ns_lincomb(a, h->st);
}

// rows of the gradient of a scalar spectrum into pr
void scalar_rows(vd_ns* h, const double* spec) {
  timed(h, 0, fields_bytes(h, 8.0),
        [&] { grad_rows(h->g, spec, h->pr, h->pr + h->N, h->pr + 2 * h->N, h->tw, h->st); });
}

// rows of a stack of three components, their y and z derivatives and the y and
// z part of their Laplacians into T, Ty, Tz, Tl; `precond`: of
// (I - dt/(2 Re) Lap)^-1 of it, times *scale
void vector_rows(vd_ns* h, const double* spec, bool precond = false, const double* scale = nullptr,
                 const int* gate = nullptr) {
  NsZArgs z{};
  z.in = spec;
  z.t0 = h->T;
  z.t1 = h->Tz;
  z.t2 = h->Tl;
  z.stride = h->ns;
  z.g = h->g;
  z.nu = 0.5 * h->prm.dt / h->prm.re;
  z.precond = precond ? 1 : 0;
  z.in_scale = scale;
  z.gate = gate;
  timed(h, 0, fields_bytes(h, 12.0), [&] { ns_z_pass(z, 3, false, h->tw, h->st); });
  NsYArgs y{};
  y.t0 = h->T;
  y.t1 = h->Tz;
  y.t2 = h->Tl;
  y.y1 = h->Ty;
  y.stride = h->ns;
  y.g = h->g;
  y.gate = gate;
  timed(h, 0, fields_bytes(h, 21.0), [&] { ns_y_pass(y, 3, false, h->tw, h->st); });
}

// x pass of a u + b zeta(rho, u).  1 / Re goes into b, not into the field 1 / rho,
// which the pressure gradient takes too: at a Re that overflows times rho (flows
// without viscosity) only the viscous term may vanish.
NsZetaArgs zeta_args(const vd_ns* h, double a, double b, double* out) {
  NsZetaArgs z{};
  z.y0 = h->T;
  z.yy = h->Ty;
  z.yz = h->Tz;
  z.yl = h->Tl;
  z.stride = h->ns;
  z.n = h->N;
  z.gr = h->cg;
  z.h = h->ch;
  z.ir = h->cir;
  z.a = a;
  z.b = b / h->prm.re;
  z.inv_sc = 1.0 / h->prm.sc;
  z.norm = h->g.ntot_inv;
  z.sx = h->g.sx;
  z.out = out;
  return z;
}
void zeta(vd_ns* h, const NsZetaArgs& z, bool rhs, bool phys) {
  timed(h, 0, fields_bytes(h, rhs ? 34.0 : 25.0), [&] { ns_zeta_pass(h->g, z, rhs, phys, h->tw, h->st); });
}

// out = A x (spectra): x - dt/2 zeta(rho^(n+1/2), x), of M^-1 x * *scale if precond
void viscous_apply(vd_ns* h, const double* x, double* out, bool precond, const double* scale, const int* gate) {
  vector_rows(h, x, precond, scale, gate);
  NsZetaArgs z = zeta_args(h, 1.0, -0.5 * h->prm.dt, out);
  z.gate = gate;
  zeta(h, z, false, false);
  fwd_columns(h, out, 3, gate);
}

// density values, gradient, Hessian and 1 / rho of a density spectrum
void coefficients(vd_ns* h, const double* spec) {
  const size_t N = h->N;
  NsZArgs z{};
  z.in = spec;
  z.t0 = h->pr;
  z.t1 = h->pr + N;
  z.t2 = h->pr + 2 * N;
  z.stride = h->ns;
  z.g = h->g;
  timed(h, 0, fields_bytes(h, 4.0), [&] { ns_z_pass(z, 1, true, h->tw, h->st); });
  NsYArgs y{};
  y.t0 = h->pr;
  y.t1 = h->pr + N;
  y.t2 = h->pr + 2 * N;
  y.y1 = h->q3;
  y.y2 = h->q3 + N;
  y.y3 = h->q3 + 2 * N;
  y.stride = h->ns;
  y.g = h->g;
  timed(h, 0, fields_bytes(h, 9.0), [&] { ns_y_pass(y, 1, true, h->tw, h->st); });
  NsCoefArgs c{};
  c.y0 = y.t0;
  c.t1 = y.t1;
  c.t2 = y.t2;
  c.y1 = y.y1;
  c.y2 = y.y2;
  c.y3 = y.y3;
  c.rho = h->rh;
  c.ir = h->cir;
  c.gr = h->cg;
  c.h = h->ch;
  c.n = N;
  c.norm = h->g.ntot_inv;
  c.sx = h->g.sx;
  timed(h, 0, fields_bytes(h, 17.0), [&] { ns_coef_pass(h->g, c, h->tw, h->st); });
}

// spectrum of (u . grad) q: u's rows are in T, q's gradient rows in pr
void advect_scalar(vd_ns* h, double* out) {
  NsAdvArgs a{};
  a.y0 = h->T;
  a.stride = h->ns;
  a.q0 = h->pr;
  a.qy = h->pr + h->N;
  a.qz = h->pr + 2 * h->N;
  a.norm = h->g.ntot_inv;
  a.sx = h->g.sx;
  a.out = out;
  timed(h, 0, fields_bytes(h, 7.0), [&] { ns_advect_pass(h->g, a, h->tw, h->st); });
  fwd_columns(h, out, 1);
}

// grad(q) / rho from q's gradient rows (pr) and cir: a stack of three, spectra
// or (phys) physical
void grad_over_rho(vd_ns* h, double* out, bool phys) {
  NsGradArgs a{};
  a.q0 = h->pr;
  a.qy = h->pr + h->N;
  a.qz = h->pr + 2 * h->N;
  a.ir = h->cir;
  a.norm = h->g.ntot_inv;
  a.sx = h->g.sx;
  a.stride = h->ns;
  a.out = out;
  timed(h, 0, fields_bytes(h, 7.0), [&] { ns_grad_pass(h->g, a, phys, h->tw, h->st); });
  if (!phys) fwd_columns(h, out, 3);
}

// Euclidean norm of a physical field
double norm(vd_ns* h, const double* x, size_t n) {
  ns_square(x, n, h->part, h->nb, h->st);
  h->hpart.resize(h->nb);
  ck(hipMemcpyAsync(h->hpart.data(), h->part, h->nb * sizeof(double), hipMemcpyDeviceToHost, h->st));
  ck(hipStreamSynchronize(h->st));
  double s = 0.0;
  for (int b = 0; b < h->nb; ++b) s += h->hpart[b];
  return std::sqrt(s);
}

double post_value(vd_ns* h, unsigned long long seq) {
  if (!wait_mail(h->mail + MAIL_VALUE, seq, h->st)) throw Err{VD_EDEVICE};
  const double s = h->mail[MAIL_VALUE].v[0];
  return s < 0.0 ? 0.0 : std::sqrt(s);  // a NaN stays NaN
}
// Euclidean norm of the physical values of a spectral vector of geometry g
double norm_spec(vd_ns* h, const Geom& g, const double* x) {
  const unsigned long long seq = ++h->posts;
  mdot<double>(g, x, VecPtrs{}, 0, true, h->part, &h->dst->nrm2, h->st, nullptr, nullptr,
               Post{POST_MAIL, h->dst, seq});
  return post_value(h, seq);
}
// r = b - A x and its norm
double viscous_residual(vd_ns* h, const double* b, const double* x, double* r) {
  viscous_apply(h, x, h->q3, false, nullptr, nullptr);
  const unsigned long long seq = ++h->posts;
  sub_norm<double>(h->g3, b, h->q3, r, h->part, &h->dst->nrm2, h->st, Post{POST_MAIL, h->dst, seq});
  return post_value(h, seq);
}

// Right-preconditioned GMRES(m) on A x = x - dt/2 zeta(rho^(n+1/2), x) = b
// (stacks of three spectra) from the initial guess x0, which is kept.  The steps
// are queued one ahead of the host, as in vdsolve.cpp, and take the second
// Gram-Schmidt pass where the check asks for it (a cosine above 1e-8, orth_tol), not
// always: the stopping test is on the true residual, and over 32^3 to 128^3, Re = 1
// to 500, restart 10 and 30 and up to 44 steps a solve, solves with two passes
// always took the same steps to the same residuals (three digits) and to fields
// within 3e-13.
void solve_viscous(vd_ns* h, const double* b, const double* x0, double* x, int& iters, int& status, double& relres) {
  const size_t n3 = 3 * h->N;
  const int m = h->prm.restart;
  const double rtol = h->prm.visc_rtol;
  const double vb = 8.0 * (double)n3;
  iters = 0;
  status = VD_OK;
  relres = 0.0;
  const double bn = norm_spec(h, h->g3, b);
  if (bn == 0.0) {
    ck(hipMemsetAsync(x, 0, n3 * sizeof(double), h->st));
    return;
  }
  auto vec = [&](int j) { return h->V + (size_t)j * n3; };
  OpParams op{};
  op.kind = OP_HELMHOLTZ;
  op.rho0 = 1.0;
  op.nu = 0.5 * h->prm.dt / h->prm.re;
  op.precond = 1;
  const int* gate = &h->dst->halt;
  auto step = [&](int j) {
    viscous_apply(h, vec(j), vec(j + 1), true, &h->dst->vs[j], gate);
    VecPtrs P{};
    for (int i = 0; i <= j; ++i) P.p[i] = vec(i);
    timed(h, 2, vb * (2.0 * j + 5.0),
          [&] { gs_orthogonalize<double>(h->g3, vec(j + 1), P, j + 1, h->dst, h->part, h->st); });
  };
  const double* cur = x0;  // the iterate: x from the first cycle's end on
  double beta = viscous_residual(h, b, cur, vec(0));
  while (true) {
    relres = beta / bn;
    const bool ok = relres <= rtol;
    if (!(beta == beta)) status = VD_EBREAKDOWN;
    else if (!ok && iters >= h->prm.max_iter) status = VD_NOT_CONVERGED;
    if (ok || status != VD_OK) {
      if (cur != x) ck(hipMemcpyAsync(x, cur, n3 * sizeof(double), hipMemcpyDeviceToDevice, h->st));
      return;
    }
    const int jlast = std::min(m, h->prm.max_iter - iters) - 1;
    const unsigned long long run = h->posts;
    h->posts += (unsigned long long)jlast + 1;
    gmres_init(h->dst, beta, m, bn, rtol, jlast, run, h->st);
    StepState t;
    int k = 0;
    step(0);
    size_t mark = h->pend.size();
    for (int j = 0; j <= jlast; ++j) {
      if (j < jlast) step(j + 1);
      if (!wait_step(h->mail, j, run, h->st, &t)) throw Err{VD_EDEVICE};
      k = j + 1;
      if (t.bad || t.halt) break;
      mark = h->pend.size();
    }
    prof_drop(h, mark);
    iters += k;
    gmres_backsolve(h->dst, k, h->st);
    VecPtrs P{};
    for (int i = 0; i < k; ++i) P.p[i] = vec(i);
    lincomb<double>(h->g3, h->z3, P, k, h->dst->coef, h->st);
    for (int c = 0; c < 3; ++c)
      precond_axpy<double>(h->g, op, x + c * h->N, h->z3 + c * h->N, nullptr, 1.0, h->st, cur + c * h->N);
    cur = x;
    beta = viscous_residual(h, b, cur, vec(0));
  }
}

// body force f (physical) and mass source S (spectrum Sh) of eq.
// VDINSE.solexact at time t (uses the coefficients and the row scratch)
void manufactured(vd_ns* h, double t) {
  const size_t N = h->N;
  double *ue = h->q3, *pe = h->pr, *re = h->pr + N;
  ns_tg_fields(h->n, t, h->prm.s, ue, pe, re, h->f, h->Sf, h->st);  // f = du/dt, Sf = drho/dt
  fwd3(h, ue, h->bh);
  double *peh = h->x3h, *reh = h->x3h + N, *lap = h->x3h + 2 * N;
  fwd(h, pe, peh);
  fwd(h, re, reh);
  fwd(h, h->Sf, h->Sh);
  coefficients(h, reh);
  vector_rows(h, h->bh);
  scalar_rows(h, peh);
  // f = du/dt + (u . grad) u + grad p / rho - zeta(rho, u)
  NsZetaArgs z = zeta_args(h, 0.0, -1.0, h->f);
  z.p0 = h->pr;
  z.py = h->pr + N;
  z.pz = h->pr + 2 * N;
  z.ext = h->f;
  z.ca = z.cg = z.ce = 1.0;
  zeta(h, z, true, true);
  // S = drho/dt + u . grad rho - Lap rho / (Re Sc)
  scalar_rows(h, reh);
  advect_scalar(h, h->z3);
  lap_packed(h->g, reh, lap, h->st);
  lin(h, h->Sh, N, {{1.0, h->Sh}, {1.0, h->z3}, {-1.0 / (h->prm.re * h->prm.sc), lap}});
}

// phi (a spectrum) from the spectrum of div(u*) / dt, with the last step's as the
// initial guess
vd_status solve_pressure(vd_ns* h, const double* div, double* phih, vd_solve_info* pi) {
  vd_solve_opts o;
  vd_default_opts(&o);
  o.solver = h->prm.pres_solver;
  o.formulation = h->prm.pres_form;
  o.restart = h->prm.restart;
  o.rtol = h->prm.pres_rtol;
  o.max_iter = h->prm.max_iter;
  o.use_x0 = 1;
  vd_status ps = VD_OK;
  if (h->prm.pres_form == VD_FORM_L) {
    timed(h, 1, 0.0, [&] { ps = grid_solve_pressure_spec(h->grid, div, h->phih, phih, &o, pi); });
    return ps;
  }
  // the modified form changes the unknown in physical space
  double *f = h->q3, *phi = h->q3 + h->N;
  inv(h, div, f);
  inv(h, h->phih, phi);
  timed(h, 1, 0.0, [&] { ps = vd_solve_pressure(h->grid, f, phi, &o, pi); });
  if (ps >= 0) fwd(h, phi, phih);
  return ps;
}

// One step.  Everything that can refuse it (a mid-step density that is not
// positive, a breakdown of the pressure solve) works in scratch: the state, the
// advection terms, the last phi and the time change together at the end, so a
// step that throws leaves the state of the last completed one, and is the same
// step when it is tried again.
void step_once(vd_ns* h) {
  const size_t N = h->N;
  const double dt = h->prm.dt, re = h->prm.re, sc = h->prm.sc;
  const bool forced = h->prm.s > 0.0;
  if (!h->spec) {  // a state was set
    fwd3(h, h->u, h->uh);
    fwd(h, h->rho, h->rhoh);
    fwd(h, h->p, h->ph);
    ck(hipMemsetAsync(h->phih, 0, N * sizeof(double), h->st));
    h->spec = true;
  }
  if (forced) manufactured(h, h->t + 0.5 * dt);
  // Adams-Bashforth weights of the new and the previous advection terms (N^(-1) = N^n on the first step)
  const double w0 = h->have_prev ? 1.5 : 1.0, w1 = h->have_prev ? -0.5 : 0.0;
  vector_rows(h, h->uh);
  // 1., 2. the density's advection and Crank-Nicolson step; 3. the mid-step density
  scalar_rows(h, h->rhoh);
  advect_scalar(h, h->nrh[0]);
  NsDensArgs d{};
  d.rho = h->rhoh;
  d.S = forced ? h->Sh : nullptr;
  d.na = h->nrh[0];
  d.nb = h->have_prev ? h->nrh[1] : nullptr;
  d.c = 0.5 * dt / (re * sc);
  d.s = dt;
  d.sa = -dt * w0;
  d.sb = -dt * w1;
  d.rho1 = h->rho1h;
  d.rhm = h->rhh;
  d.g = h->g;
  d.n = h->ns;
  ns_density(d, h->st);
  // 4. intermediate velocity
  coefficients(h, h->rhh);
  scalar_rows(h, h->ph);
  NsZetaArgs z = zeta_args(h, 1.0, 0.5 * dt, h->bh);
  z.p0 = h->pr;
  z.py = h->pr + N;
  z.pz = h->pr + 2 * N;
  z.nprev = h->have_prev ? h->nu[1] : nullptr;
  z.ext = forced ? h->f : nullptr;
  z.ca = -dt * w0;
  z.cp = -dt * w1;
  z.cg = -dt;
  z.ce = dt;
  z.nout = h->nu[0];
  zeta(h, z, true, false);
  fwd_columns(h, h->bh, 3);
  double* us = h->x3h;
  int vit = 0, vst = 0;
  double vres = 0;
  solve_viscous(h, h->bh, h->uh, us, vit, vst, vres);
  // 5. pressure equation
  ns_div(h->g, us, h->ns, 1.0 / dt, h->z3, h->st);
  if (vd_set_density(h->grid, h->rh) != VD_OK) throw Err{VD_EDOMAIN};
  vd_solve_info pi{};
  double* phi = h->Sh;  // the mass source has been used
  const vd_status ps = solve_pressure(h, h->z3, phi, &pi);
  if (ps < 0 && ps != VD_NOT_CONVERGED) throw Err{ps};
  // 6. projection (from here on the step cannot be refused)
  scalar_rows(h, phi);
  grad_over_rho(h, h->z3, false);
  lin(h, h->uh, 3 * N, {{1.0, us}, {-dt, h->z3}});
  // 7. pressure update: p += phi - (div grad)^-1 div(dt/2 rho zeta(rho, grad(phi) / rho))
  vector_rows(h, h->z3);
  z = zeta_args(h, 0.0, 0.5 * dt, h->q3);
  z.unit = true;  // rho times 1 / rho
  zeta(h, z, false, false);
  fwd_columns(h, h->q3, 3);
  ns_pressure(h->g, h->q3, h->ns, phi, h->ph, h->st);
  std::swap(h->phih, h->Sh);
  // rho^(n+1) becomes the state, the current advection terms the previous ones
  std::swap(h->rhoh, h->rho1h);
  std::swap(h->nu[0], h->nu[1]);
  std::swap(h->nrh[0], h->nrh[1]);
  h->have_prev = true;
  h->t += dt;
  ++h->steps;
  h->last.t = h->t;
  h->last.steps = h->steps;
  h->last.visc_iters = vit;
  h->last.visc_status = vst;
  h->last.visc_rel_residual = vres;
  h->last.pres_iters = pi.iterations;
  h->last.pres_status = ps;
  h->last.pres_rel_residual = pi.rel_residual;
  h->last.pres_seconds = pi.seconds;
}

// the physical fields of the state from its spectra
void state_to_physical(vd_ns* h) {
  inv3(h, h->uh, h->u);
  inv(h, h->rhoh, h->rho);
  inv(h, h->ph, h->p);
}

}  // namespace

extern "C" {

void vd_ns_default_params(vd_ns_params* p) {
  if (!p) return;
  p->re = 1.0;
  p->sc = 1.0;
  p->dt = 0.01;
  p->s = 0.0;
  p->visc_rtol = 1e-12;
  p->pres_rtol = 1e-12;
  p->restart = 30;
  p->max_iter = 2000;
  p->pres_solver = VD_GMRES;
  p->pres_form = VD_FORM_L;
}

vd_status vd_ns_create(vd_ns** out, int n, const vd_ns_params* prm, hipStream_t stream) {
  if (!out) return VD_EINVAL;
  *out = nullptr;
  vd_ns_params p;
  if (prm) p = *prm;
  else vd_ns_default_params(&p);
  if (n < 16 || n > 512 || (n & (n - 1))) return VD_EINVAL;
  if (!(p.re > 0) || !(p.sc > 0) || !(p.dt > 0) || !(p.s >= 0) || !std::isfinite(p.re + p.sc + p.dt + p.s))
    return VD_EINVAL;
  if (!(p.visc_rtol > 0) || !(p.pres_rtol > 0) || p.restart < 1 || p.restart > 30 || p.max_iter < 1)
    return VD_EINVAL;
  if ((p.pres_solver != VD_GMRES && p.pres_solver != VD_CG && p.pres_solver != VD_RMR) ||
      (p.pres_form != VD_FORM_L && p.pres_form != VD_FORM_K))
    return VD_EINVAL;
  vd_ns* h = new (std::nothrow) vd_ns();
  if (!h) return VD_ENOMEM;
  h->n = n;
  h->N = (size_t)n * n * n;
  h->prm = p;
  h->st = stream;
  try {
    vd_grid_desc d{};
    d.ndim = 3;
    for (int i = 0; i < 3; ++i) {
      d.n[i] = n;
      d.basis[i] = VD_FOURIER;
      d.length[i] = 2.0 * M_PI;
    }
    const vd_status gs = vd_grid_create(&h->grid, &d, stream);
    if (gs != VD_OK) throw Err{gs};
    h->g = grid_geom(h->grid);
    h->tw = grid_twiddles(h->grid);
    h->ns = (size_t)h->g.nz * h->g.ny * h->g.M;
    h->g3 = h->g;
    h->g3.nz = 3 * h->g.nz;
    const size_t N = h->N;  // doubles of a field, physical or packed
    h->u = dalloc(h, 3 * N);
    h->rho = dalloc(h, N);
    h->p = dalloc(h, N);
    h->uh = dalloc(h, 3 * N);
    h->rhoh = dalloc(h, N);
    h->ph = dalloc(h, N);
    h->phih = dalloc(h, N);
    for (int i = 0; i < 2; ++i) {
      h->nu[i] = dalloc(h, 3 * N);
      h->nrh[i] = dalloc(h, N);
    }
    h->rh = dalloc(h, N);
    h->cg = dalloc(h, 3 * N);
    h->ch = dalloc(h, 6 * N);
    h->cir = dalloc(h, N);
    h->rho1h = dalloc(h, N);
    h->rhh = dalloc(h, N);
    h->T = dalloc(h, 3 * N);
    h->Tz = dalloc(h, 3 * N);
    h->Tl = dalloc(h, 3 * N);
    h->Ty = dalloc(h, 3 * N);
    h->pr = dalloc(h, 3 * N);
    h->bh = dalloc(h, 3 * N);
    h->q3 = dalloc(h, 3 * N);
    h->x3h = dalloc(h, 3 * N);
    h->z3 = dalloc(h, 3 * N);
    h->f = dalloc(h, 3 * N);
    h->Sf = dalloc(h, N);
    h->Sh = dalloc(h, N);
    h->V = dalloc(h, (size_t)(p.restart + 1) * 3 * N);
    h->nb = ns_dot_blocks(3 * N);
    h->part = dalloc(h, nred_partial());
    h->dst = (DevState*)dalloc(h, sizeof(DevState) / sizeof(double) + 1);
    ck(hipMemsetAsync(h->dst, 0, sizeof(DevState), stream));
    ck(make_mail(&h->mail, h->dst, stream));
  } catch (const Err& e) {
    release(h);
    return e.s;
  } catch (const std::bad_alloc&) {
    release(h);
    return VD_ENOMEM;
  }
  *out = h;
  return VD_OK;
}

vd_status vd_ns_destroy(vd_ns* h) {
  if (!h) return VD_EINVAL;
  if (h->st) hipStreamSynchronize(h->st);
  else hipDeviceSynchronize();
  release(h);
  return VD_OK;
}

vd_status vd_ns_set_state(vd_ns* h, const double* u, const double* rho, const double* p, double t) {
  if (!h || !u || !rho || !p || !std::isfinite(t)) return VD_EINVAL;
  const size_t N = h->N;
  if (hipMemcpyAsync(h->u, u, 3 * N * sizeof(double), hipMemcpyDeviceToDevice, h->st) != hipSuccess ||
      hipMemcpyAsync(h->rho, rho, N * sizeof(double), hipMemcpyDeviceToDevice, h->st) != hipSuccess ||
      hipMemcpyAsync(h->p, p, N * sizeof(double), hipMemcpyDeviceToDevice, h->st) != hipSuccess ||
      hipStreamSynchronize(h->st) != hipSuccess)
    return VD_EDEVICE;
  h->spec = false;
  h->t = t;
  h->steps = 0;
  h->have_prev = false;
  h->have_state = true;
  return VD_OK;
}

vd_status vd_ns_init_taylor_green(vd_ns* h) {
  if (!h || !(h->prm.s > 0.0)) return VD_EINVAL;
  ns_tg_fields(h->n, 0.0, h->prm.s, h->u, h->pr, h->rho, nullptr, nullptr, h->st);
  ns_tg_fields(h->n, -0.5 * h->prm.dt, h->prm.s, h->q3, h->p, h->pr, nullptr, nullptr, h->st);
  if (hipStreamSynchronize(h->st) != hipSuccess || hipGetLastError() != hipSuccess) return VD_EDEVICE;
  h->spec = false;
  h->t = 0.0;
  h->steps = 0;
  h->have_prev = false;
  h->have_state = true;
  return VD_OK;
}

vd_status vd_ns_step(vd_ns* h, int nsteps, vd_ns_info* info) {
  if (!h || nsteps < 0) return VD_EINVAL;
  if (!h->have_state) return VD_EINVAL;
  int done = 0;
  try {
    while (done < nsteps) {
      step_once(h);
      ++done;
      if (h->prof) {
        ck(hipStreamSynchronize(h->st));
        prof_flush(h);
      }
    }
    if (nsteps > 0) state_to_physical(h);
    ck(hipStreamSynchronize(h->st));
    ck(hipGetLastError());
    if (h->prof) prof_flush(h);
  } catch (const Err& e) {
    hipGetLastError();
    if (done > 0) {  // the state is that of the last completed step
      try {
        state_to_physical(h);
        ck(hipStreamSynchronize(h->st));
      } catch (const Err&) {
        hipGetLastError();
      }
    }
    return e.s;
  }
  if (info) *info = h->last;
  if (h->last.visc_status < 0) return (vd_status)h->last.visc_status;
  if (h->last.pres_status < 0) return (vd_status)h->last.pres_status;
  if (h->last.visc_status == VD_NOT_CONVERGED || h->last.pres_status == VD_NOT_CONVERGED) return VD_NOT_CONVERGED;
  return VD_OK;
}

vd_status vd_ns_get_state(vd_ns* h, double* u, double* rho, double* p, double* t) {
  if (!h) return VD_EINVAL;
  const size_t N = h->N;
  if ((u && hipMemcpyAsync(u, h->u, 3 * N * sizeof(double), hipMemcpyDeviceToDevice, h->st) != hipSuccess) ||
      (rho && hipMemcpyAsync(rho, h->rho, N * sizeof(double), hipMemcpyDeviceToDevice, h->st) != hipSuccess) ||
      (p && hipMemcpyAsync(p, h->p, N * sizeof(double), hipMemcpyDeviceToDevice, h->st) != hipSuccess) ||
      hipStreamSynchronize(h->st) != hipSuccess)
    return VD_EDEVICE;
  if (t) *t = h->t;
  return VD_OK;
}

vd_status vd_ns_errors(vd_ns* h, double* err) {
  if (!h || !err || !(h->prm.s > 0.0)) return VD_EINVAL;
  const size_t N = h->N;
  const double rn = std::sqrt((double)N);
  double *ue = h->q3, *pe = h->pr, *re = h->pr + N;
  try {
    // exact fields at t (u, rho) and at t - dt/2 (p)
    ns_tg_fields(h->n, h->t, h->prm.s, ue, pe, re, nullptr, nullptr, h->st);
    lin(h, ue, 3 * N, {{1.0, h->u}, {-1.0, ue}});
    lin(h, re, N, {{1.0, h->rho}, {-1.0, re}});
    err[0] = norm(h, ue, 3 * N) / rn;
    err[2] = norm(h, re, N) / rn;
    ns_tg_fields(h->n, h->t - 0.5 * h->prm.dt, h->prm.s, ue, pe, re, nullptr, nullptr, h->st);
    lin(h, pe, N, {{1.0, h->p}, {-1.0, pe}});
    err[1] = norm(h, pe, N) / rn;
    fwd3(h, h->u, h->x3h);
    ns_div(h->g, h->x3h, h->ns, 1.0, h->z3, h->st);
    err[3] = norm_spec(h, h->g, h->z3) / rn;
  } catch (const Err& e) {
    hipGetLastError();
    return e.s;
  }
  return VD_OK;
}

vd_status vd_ns_project(vd_ns* h, const double* rho, const double* u, double* out, vd_solve_info* info) {
  if (!h || !rho || !u || !out) return VD_EINVAL;
  const size_t N = h->N;
  vd_status ps = VD_OK;
  try {
    fwd3(h, u, h->x3h);
    ns_div(h->g, h->x3h, h->ns, 1.0, h->z3, h->st);
    if (vd_set_density(h->grid, rho) != VD_OK) return VD_EDOMAIN;
    vd_solve_opts o;
    vd_default_opts(&o);
    o.solver = VD_GMRES;
    o.restart = h->prm.restart;
    o.rtol = h->prm.pres_rtol;
    o.max_iter = h->prm.max_iter;
    double* phi = h->z3 + N;
    ps = grid_solve_pressure_spec(h->grid, h->z3, nullptr, phi, &o, info);
    if (ps < 0 && ps != VD_NOT_CONVERGED) return ps;
    ns_recip(rho, h->cir, N, h->st);
    scalar_rows(h, phi);
    grad_over_rho(h, h->q3, true);
    lin(h, out, 3 * N, {{1.0, u}, {-1.0, h->q3}});
    ck(hipStreamSynchronize(h->st));
    ck(hipGetLastError());
  } catch (const Err& e) {
    hipGetLastError();
    return e.s;
  }
  return ps;
}

vd_status vd_ns_profile_enable(vd_ns* h, int on) {
  if (!h) return VD_EINVAL;
  h->prof = on != 0;
  for (int c = 0; c < 3; ++c) {
    h->pms[c] = 0;
    h->pbytes[c] = 0;
    h->pcnt[c] = 0;
  }
  return VD_OK;
}

vd_status vd_ns_profile_read(vd_ns* h, double* ms, long long* count, double* bytes, int nclass) {
  if (!h || nclass < 0) return VD_EINVAL;
  for (int c = 0; c < nclass && c < 3; ++c) {
    if (ms) ms[c] = h->pms[c];
    if (count) count[c] = h->pcnt[c];
    if (bytes) bytes[c] = h->pbytes[c];
  }
  return VD_OK;
}

}  // extern "C"

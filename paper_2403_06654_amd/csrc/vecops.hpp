// Krylov vector algebra on packed spectral fields (host interface).
//
// Inner products are the Euclidean products of the physical grid values,
// evaluated from the packed half-spectrum by Parseval's identity: weight 1
// on the kx = 0 slot (which holds kx = 0 and kx = nx/2), 2 elsewhere,
// overall 1 / N.  Every reduction is two-stage with a fixed block count and
// a fixed summation order, so results are bitwise reproducible and do not
// depend on what else runs on the device.
#pragma once

#include <hip/hip_runtime.h>
#include <cstddef>
#include "passes.hpp"

namespace vd {

constexpr int kRedBlocks = 1024;  // partial sums per reduction (4 blocks per CU)

// What a kernel tells the waiting host, written straight into pinned host memory.
// The host polls seq for the number it expects (each is used once per mailbox)
// and takes the values when check fits all of them: the words may arrive in any
// order, so a step's kernel neither waits between its stores nor writes back its
// L2 for the host.  A step whose state went to the host as a copy of its own,
// with an event to wait for, cost about 10 us of the stream per Krylov step.
struct alignas(64) Mail {
  double v[2];
  unsigned long long flags;  // bit 0: bad, bit 1: halt, above: second passes of this cycle
  unsigned long long seq;
  unsigned long long check;  // mail_check of the four
};
__host__ __device__ inline unsigned long long mail_check(unsigned long long a, unsigned long long b,
                                                         unsigned long long flags, unsigned long long seq) {
  unsigned long long h = 0x9e3779b97f4a7c15ull;
  const unsigned long long w[4] = {a, b, flags, seq};
  for (int i = 0; i < 4; ++i) {
    h = (h ^ w[i]) * 0xff51afd7ed558ccdull;
    h ^= h >> 32;
  }
  return h;
}
// mailboxes of a solver state: two for the Krylov steps in turn, one for
// single reduced values
enum { MAIL_STEP = 0, MAIL_VALUE = 2, kMails = 3 };

// Solver scalars kept on the device (FP64 regardless of vector precision).
constexpr int kMaxRestart = 32;
struct DevState {
  double H[(kMaxRestart + 1) * kMaxRestart];  // column-major, ld = kMaxRestart + 1
  double cs[kMaxRestart], sn[kMaxRestart], g[kMaxRestart + 1], y[kMaxRestart];
  double red[kMaxVec + 2];   // outputs of the last reduction
  double red2[kMaxVec];      // the first-pass dots of the last Gram-Schmidt step
  Mail* mail;                // pinned host mailboxes (device address)
  unsigned long long run;    // step j of the current cycle or run posts run + j + 1
  double vs[kMaxRestart + 1];     // scale of each stored (unnormalised) basis vector
  double hcol[kMaxVec], ccol[kMaxVec], coef[kMaxVec];  // Gram-Schmidt coefficients
  double hn;                 // norm of the newest orthogonalised vector
  int reorth;                // second Gram-Schmidt pass ran for this step
  int nreorth;               // second passes of the current cycle
  double alpha, beta;
  double rz[2];              // CG: (r, M^-1 r); carried steps alternate between the two
  // Krylov stopping test, evaluated on the device after each step (GMRES:
  // resid / stop_bnorm <= stop_rtol on the Givens estimate; CG and RMR: on
  // the recursive residual), a non-finite scalar, or step jlast of the cycle
  // or run (restart length or iteration budget) sets halt
  double stop_bnorm, stop_rtol;
  int jlast;
  int step;                  // CG / RMR: steps completed in the current run
  // posted to the host after each step
  double resid;              // estimated (GMRES) or recursive residual norm
  double nrm2;               // last computed squared norm
  int bad;                   // non-finite scalar seen
  int halt;                  // the cycle or run has ended; gated kernels return at once
};

// A scalar step of CG or RMR that the final reduction of a vector kernel
// takes in its own launch once the reduced value is written (st: the
// solver's device state): beta = red[0] / rz and rz = red[0] (CG), alpha = red[0] / red[1] (RMR), or the stopping test on
// nrm2 (CG and RMR), that test on red[0] followed by CG's beta from red[1], or
// the reduced value posted to the host as number seq.
enum PostOp { POST_NONE = 0, POST_CG_BETA, POST_RMR_ALPHA, POST_REC_CHECK, POST_CG_STEP, POST_MAIL };
struct Post {
  int op = POST_NONE;
  DevState* st = nullptr;
  unsigned long long seq = 0;
};

// partial[b][i] = sum_e w_e Re(conj(V_i[e]) x[e]) (i < nv), plus |x|^2 at
// index nv when want_norm.  Then reduce into st->red (times 1/N).
template <typename R>
void mdot(const Geom& g, const void* x, const VecPtrs& V, int nv, bool want_norm, double* partial,
          double* out, hipStream_t s, Prof* prof = nullptr, const int* gate = nullptr, const Post& post = Post{});

// GMRES step: orthogonalise w against the stored basis V_0..V_{nv-1}
// (v_i = vs[i] V_i) in place; classical Gram-Schmidt with a measured
// orthogonality check and a conditional second pass.  Leaves the
// Hessenberg column in st->hcol (+ st->ccol), ||w|| in st->hn and
// vs[nv] = 1 / ||w||, and applies the Givens rotations to column nv - 1
// (st->resid = new residual estimate).
// On small fields a caller may take parts of it elsewhere: with dot_blocks, that
// many blocks have already written the dots' partials; without finish, the
// check, the second pass and the rotations are left to the next operator pass.
struct GsParts {
  int dot_blocks = 0;
  bool finish = true;
};
template <typename R>
void gs_orthogonalize(const Geom& g, void* w, const VecPtrs& V, int nv, DevState* st, double* partial,
                      hipStream_t s, Prof* prof = nullptr, const GsParts& parts = GsParts{});
int gs_update_blocks(const Geom& g);  // block partials of the check dots (small fields)

// The same step for nsys <= kMaxBatch independent systems together (one
// launch per pass for all of them; system k: w[k], V[k], st[k], partial[k];
// a system whose halt flag is set is skipped).  The kernels and reduction
// orders are those of one system, so each system's result is the same as
// when it is orthogonalised alone.
template <typename R>
void gs_orthogonalize_batch(const Geom& g, void* const* w, const VecPtrs* V, int nv, DevState* const* st,
                            double* const* partial, int nsys, hipStream_t s, Prof* prof = nullptr,
                            const GsParts& parts = GsParts{});

// Device states and reduction partials of a set of systems (single-block
// scalar kernels index them by blockIdx.y).
struct DevStates {
  DevState* st[kMaxBatch];
  double* partial[kMaxBatch];
};

// z = sum_i c_i V_i
template <typename R>
void lincomb(const Geom& g, void* z, const VecPtrs& V, int nv, const double* coef, hipStream_t s);

// v *= (*s_dev) * s_host
template <typename R>
void scale(const Geom& g, void* v, const double* s_dev, double s_host, hipStream_t s);

// r = b - q, and |r|^2 reduced into out[0]
template <typename R>
void sub_norm(const Geom& g, const void* b, const void* q, void* r, double* partial, double* out,
              hipStream_t s, const Post& post = Post{});

// Gates: the kernels below that take OpParams honour p.gate; the others take
// an explicit gate.  A nonzero *gate makes the launch do nothing.
// x += a M^-1 z   (a = (*a_dev) * a_host; M^-1 diagonal, Helmholtz kx = 0 mirrored), or
// x = x_from + a M^-1 z
template <typename R>
void precond_axpy(const Geom& g, const OpParams& p, void* x, const void* z, const double* a_dev,
                  double a_host, hipStream_t s, const void* x_from = nullptr);

// (r, M^-1 r) reduced into out[0]
template <typename R>
void dot_rMr(const Geom& g, const OpParams& p, const void* r, double* partial, double* out,
             hipStream_t s, const Post& post = Post{});

// The block partials of mdot, not reduced: rec_step reduces them itself.
template <typename R>
void dot_partials(const Geom& g, const void* x, const void* v, bool want_norm, double* partial, hipStream_t s,
                  const int* gate);
// Second half of a CG or RMR step (rmr = false / true) after dot_partials of
// (p, q) or of (r, w) and |w|^2:
//   alpha = rz / (p, q)          or (r, w) / |w|^2
//   x += alpha p                 or alpha M^-1 r
//   rnew = r - alpha q           (q: w for RMR; rnew must be another buffer)
// with the new |r|^2 (red[0]), for CG also (r, M^-1 r) (red[1]), the stopping
// test and CG's beta.  Gated by st->halt.
// Where the operator's passes carry parts of the step (RecCarry): dot_blocks left
// the dots' partials, slot holds rz, and without finish the test and beta are
// left to the next step's first pass.
struct RecParts {
  int dot_blocks = 0;
  int slot = 0;
  bool finish = true;
};
template <typename R>
void rec_step(const Geom& g, const OpParams& op, bool rmr, void* x, const void* r, void* rnew, const void* p,
              const void* q, DevState* st, double* partial, hipStream_t s, const RecParts& parts = RecParts{});
int rec_step_blocks(const Geom& g);  // block partials that rec_step leaves
// CG on a Chebyshev grid with its dense preconditioner V D V^T, in the basis V
// (rt = V^T r, p = V pt, x accumulated as V xt; qq: q and V^T q, one after the
// other; lam, scale, sx: D as in the contraction's epilogue): after
// dot_partials of (pt, V^T q),  xt += alpha pt, r -= alpha q,
// rt -= alpha V^T q, then as rec_step.
struct EigDiag {
  const double* lam;
  double scale, sx;
};
template <typename R>
void eig_step(const Geom& g, const EigDiag& d, void* xt, void* r, void* rt, const void* pt, const void* qq,
              DevState* st, double* partial, hipStream_t s);
// pt = D rt + beta pt (first: pt = D rt, and (rt, D rt) reduced into rz)
template <typename R>
void eig_p(const Geom& g, const EigDiag& d, void* pt, const void* rt, bool first, DevState* st, double* partial,
           hipStream_t s);
// CG: p = M^-1 r + beta p   (beta = st->beta)
template <typename R>
void cg_p(const Geom& g, const OpParams& op, void* p, const void* r, const DevState* st, hipStream_t s);
// RMR: r -= alpha w; |r|^2 -> out[0]
template <typename R>
void axpy_norm(const Geom& g, void* r, const void* w, const double* a_dev, double sign, double* partial,
               double* out, hipStream_t s, const int* gate = nullptr, const Post& post = Post{});

// precision casts between spectral vectors: dst(float) = src(double) * s
void cast_d2f(const Geom& g, const void* src, void* dst, double s, hipStream_t st);
// dst(double) += src(float) * s
void axpy_f2d(const Geom& g, const void* src, void* dst, double s, hipStream_t st);
void cast_f2d(const Geom& g, const void* src, void* dst, hipStream_t st);

// Zero the 2^D nullspace slots of a packed pressure spectrum; write the
// removed Euclidean norm (physical units) to *removed.
void project_range(const Geom& g, void* spec, double* removed, hipStream_t st);
// Zero the mean (DC) of a packed FP64 spectrum; removed Euclidean norm to *removed.
void zero_mean(const Geom& g, void* spec, double* removed, hipStream_t st);

// Scalar kernels of the Krylov methods.
// Gives a new state its mailboxes (device address of kMails of them).
void set_mail(DevState* st, Mail* mail, hipStream_t s);
// Starts a GMRES cycle: H, g, the basis scales and the stopping test
// (bnorm, rtol, last step jlast of this cycle; halt and the second-pass count
// cleared); step j posts run + j + 1.
void gmres_init(DevState* st, double beta, int m, double bnorm, double rtol, int jlast, unsigned long long run,
                hipStream_t s);
void gmres_backsolve(DevState* st, int k, hipStream_t s);  // y, and coef = y * vs
// Starts a CG or RMR run: its stopping test (bnorm, rtol, last step jlast),
// step = 0, halt and bad cleared; step j posts run + j + 1.
void rec_init(DevState* st, double bnorm, double rtol, int jlast, unsigned long long run, hipStream_t s);

// Density set-up: a = 1/rho and copies, min/max/sum reductions.
void density_setup(const double* rho, size_t n, double* a64, float* a32, float* rho32, double* partial,
                   double* out /* [sum, min, max, nonfinite_or_nonpositive] */, hipStream_t s);

// Modified pressure form (eq. VDINSE.Krho), physical FP64 grid values:
// out = sign * in * sqrt(rho), or sign * in / sqrt(rho) if `inverse`
// (in == nullptr: in = 1).
void rho_sqrt_mul(const double* rho, const double* in, double* out, bool inverse, double sign, size_t n,
                  hipStream_t s);
// kc = Lap(rho^-1/2) sqrt(rho) = -c (FP64 and FP32 copies).
void kcoef_finish(const double* rho, const double* lap_psi, double* kc64, float* kc32, size_t n, hipStream_t s);

size_t nred_partial();  // doubles needed for `partial`

}  // namespace vd

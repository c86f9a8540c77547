// Device side of a Gram-Schmidt step shared by the vector kernels and by the
// operator passes of small fields, which carry parts of it.
#pragma once

#include <cmath>

#include "vd_common.hpp"
#include "vecops.hpp"

namespace vd {

// Small fields: one pass's block partials (at most kFoldBlocks per value) are
// reduced by every block of the next pass.  The dots and the check dots take
// the two halves of each partial row.
constexpr size_t kFoldElems = 131072;
constexpr int kFoldBlocks = 256;
constexpr int kFoldHalf = kRedBlocks / 2;

// Choice of tol: the Arnoldi relation A V_j = V_{j+1} H_j holds to rounding
// whatever the orthogonality, so the computed least-squares residual
// |beta e1 - H y| differs from the true one |V_{j+1}(beta e1 - H y)| only by
// the factor |V_{j+1}| <= sqrt(1 + (j+1) delta), delta the largest cosine
// between basis vectors.  Orthogonality must therefore stay far from 1
// (else the basis degenerates and convergence stalls), not below the solve
// tolerance.  tol = 1e-8 (FP64) keeps that factor within 2e-7 of 1 for 32
// vectors; 1e-4 (FP32 inner solves, target 1e-5) within 0.2%.  A tighter
// tol only makes the second pass fire whenever the operator is close to the
// identity (velocity solves), where |w'| << |w| magnifies the rounding of the
// first-pass dots.
template <typename R>
constexpr double orth_tol() { return sizeof(R) == 8 ? 1e-8 : 1e-4; }

// v plus the value that the DPP pattern CTRL brings to this lane (0 where it
// brings none, and in the rows that ROWS leaves out)
template <int CTRL, int ROWS>
__device__ __forceinline__ double add_dpp(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, true);
  return v + __hiloint2double(hi, lo);
}
// Sum over the wavefront (all 64 lanes active), returned in every lane: row
// shifts by 1, 2, 4, 8 leave each 16-lane row's sum in its last lane, two row
// broadcasts carry them to lane 63.  A fixed tree on the vector ALU: the same
// tree through LDS permutes costs two LDS round trips per step, which the
// latency-bound reductions of small fields feel.
__device__ __forceinline__ double wave_sum(double v) {
  v = add_dpp<0x111, 0xf>(v);  // row_shr:1
  v = add_dpp<0x112, 0xf>(v);  // row_shr:2
  v = add_dpp<0x114, 0xf>(v);  // row_shr:4
  v = add_dpp<0x118, 0xf>(v);  // row_shr:8
  v = add_dpp<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v = add_dpp<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                          __builtin_amdgcn_readlane(__double2loint(v), 63));
}

// Sum of one value's nblk <= kRedBlocks block partials by one wavefront, in a
// fixed order: lanes stride over them, then the wavefront's tree.  Every lane
// issues all its loads before the first addition.  A loop that added each
// partial as it arrived paid up to sixteen dependent load latencies: on 1024
// partials of 9-16 values k_gs_prep took 6.8 us (4.5 now) and k_gs_check 9.4 us
// (5.2 now).
__device__ __forceinline__ double sum_partials(const double* __restrict__ p, int nblk) {
  constexpr int Q = kRedBlocks / 64;
  const int lane = threadIdx.x & 63;
  double v[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) v[q] = lane + 64 * q < nblk ? p[lane + 64 * q] : 0.0;
  double s = v[0];
#pragma unroll
  for (int q = 1; q < Q; ++q) s += v[q];
  return wave_sum(s);
}

// The halt flag where a block of the same launch may set it: one thread of a block
// reads it, and the whole block goes by what it saw (through LDS, at a barrier).
// Wavefronts that each read it could part: some would return, and the others would
// go on past a barrier without what the first were to write for them.
__device__ __forceinline__ int halt_now(const int* flag) {
  return flag ? __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
}
__device__ __forceinline__ void set_halt(DevState* st) {
  __hip_atomic_store(&st->halt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Values to the host (one thread).
__device__ __forceinline__ void post_mail(Mail* m, double a, double b, unsigned long long flags,
                                          unsigned long long seq) {
  const unsigned long long c = mail_check((unsigned long long)__double_as_longlong(a),
                                          (unsigned long long)__double_as_longlong(b), flags, seq);
  __hip_atomic_store(&m->v[0], a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(&m->v[1], b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(&m->flags, flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(&m->check, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(&m->seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// The state after step j of a cycle or run (bad and halt as just decided); mail
// and run: the state's.
__device__ __forceinline__ void post_step(Mail* mail, unsigned long long run, int j, double resid, double nrm2,
                                          bool bad, bool halt, int nreorth) {
  post_mail(mail + MAIL_STEP + (j & 1), resid, nrm2,
            (bad ? 1ull : 0ull) | (halt ? 2ull : 0ull) | ((unsigned long long)nreorth << 2), run + j + 1);
}

// Scalar steps of CG and RMR, taken by one thread on the reduced values
// (passed in: see k_reduce) and on the state as it was loaded ahead of them.
struct RecState {
  double rz, stop_bnorm, stop_rtol;  // rz: of the step that ends
  int step, bad, jlast;
  Mail* mail;
  unsigned long long run;
};
__device__ __forceinline__ RecState rec_state(const DevState* st, int slot = 0) {
  return RecState{st->rz[slot], st->stop_bnorm, st->stop_rtol, st->step, st->bad, st->jlast, st->mail, st->run};
}
__device__ __forceinline__ double cg_beta(double rz, double rzn) { return rz != 0.0 ? rzn / rz : 0.0; }
__device__ __forceinline__ void cg_beta_step(DevState* st, const RecState& s, double rzn, int slot = 0) {
  // beta = (r, M r)_new / (r, M r)
  const double beta = cg_beta(s.rz, rzn);
  st->beta = beta;
  st->rz[slot] = rzn;
  if (!isfinite(beta)) st->bad = 1;
}
__device__ __forceinline__ void rmr_alpha_step(DevState* st, double rw, double ww) {  // alpha = (r, w) / (w, w)
  st->alpha = ww > 0.0 ? rw / ww : 0.0;
  if (!isfinite(st->alpha)) st->bad = 1;
}
// Stopping test of a CG or RMR step on its recursive residual (n2 = its
// square, also in st->nrm2), the host loop's test taken on the device: a
// non-finite scalar, the tolerance, or the last step of the run sets halt.
// step counts the steps.
__device__ __forceinline__ bool rec_check_step(DevState* st, const RecState& s, double n2) {
  const int j = s.step;
  st->step = j + 1;
  const double rn = n2 < 0.0 ? 0.0 : sqrt(n2);
  const bool bad = s.bad != 0;
  const bool halt = bad || !(n2 == n2) || rn / s.stop_bnorm <= s.stop_rtol || j >= s.jlast;
  if (halt) set_halt(st);
  post_step(s.mail, s.run, j, rn, n2, bad, halt, 0);
  return halt;
}

// leading dimension of the column-major Hessenberg matrix
__device__ __forceinline__ int ldh() { return kMaxRestart + 1; }

// The larger of v and the value that the DPP pattern CTRL brings to this lane (v
// itself where it brings none, and in the rows that ROWS leaves out)
template <int CTRL, int ROWS>
__device__ __forceinline__ double max_dpp(double v) {
  const int vl = __double2loint(v), vh = __double2hiint(v);
  const int lo = __builtin_amdgcn_update_dpp(vl, vl, CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(vh, vh, CTRL, ROWS, 0xf, false);
  return fmax(v, __hiloint2double(hi, lo));
}
__device__ __forceinline__ double lane_value(double v, int lane) {  // lane: the same in the whole wavefront
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// Largest of the wavefront's values (all 64 lanes active); a NaN is dropped.
__device__ __forceinline__ double wave_max(double v) {
  v = max_dpp<0x111, 0xf>(v);
  v = max_dpp<0x112, 0xf>(v);
  v = max_dpp<0x114, 0xf>(v);
  v = max_dpp<0x118, 0xf>(v);
  v = max_dpp<0x142, 0xa>(v);
  v = max_dpp<0x143, 0xc>(v);
  return lane_value(v, 63);
}

// Orthogonality check of the first pass, taken by one wavefront with lane i on
// basis vector i (val: the reduced dots (V_i, w') and, at nv, ||w'||^2).
struct GsCheck {
  double h, v;   // this lane's first-pass coefficient and vector scale
  double csel;   // its second-pass coefficient (0: the vector passed the test)
  double hn;     // norm of the orthogonalised vector
  bool orth;     // no second pass needed
  bool finite;
};
// What the check and the rotations read from the state (lane i: vector i).
// Loaded ahead of the reduction that they wait for, so that its latency hides
// theirs (1 to 2 us of a step on small fields).
struct GsState {
  double v = 0, h = 0, cs = 0, sn = 0;
  double g = 0, stop_bnorm = 0, stop_rtol = 0;
  int nreorth = 0, bad = 0, jlast = 0;
  Mail* mail = nullptr;
  unsigned long long run = 0;
};
__device__ __forceinline__ GsState gs_state(const DevState* st, int nv, bool rotations) {
  const int lane = threadIdx.x & 63;
  GsState s;
  if (lane < nv) {
    s.v = st->vs[lane];
    s.h = st->hcol[lane];
  }
  if (rotations) {
    if (lane < nv - 1) {
      s.cs = st->cs[lane];
      s.sn = st->sn[lane];
    }
    s.g = st->g[nv - 1];
    s.stop_bnorm = st->stop_bnorm;
    s.stop_rtol = st->stop_rtol;
    s.nreorth = st->nreorth;
    s.bad = st->bad;
    s.jlast = st->jlast;
    s.mail = st->mail;
    s.run = st->run;
  }
  return s;
}
__device__ __forceinline__ GsCheck gs_check(const GsState& s, const double* val, int nv, double tol) {
  const int lane = threadIdx.x & 63;
  GsCheck k;
  k.h = s.h;
  k.v = s.v;
  const double c = lane < nv ? k.v * val[lane] : 0.0;
  const double n2 = val[nv];
  const double thr = tol * sqrt(n2);
  k.orth = n2 > 0.0 && wave_max(fabs(c)) <= thr;
  // The second pass subtracts only the components that fail the test: the
  // others already meet the tolerance accepted when no second pass runs.
  // (n2 <= 0 selects every nonzero component.)
  k.csel = (!k.orth && lane < nv && !(fabs(c) <= thr)) ? c : 0.0;
  const double h2 = n2 - wave_sum(k.csel * k.csel);
  // wave_max drops NaN, and a NaN norm would read as a lucky breakdown
  k.finite = isfinite(n2) && isfinite(wave_sum(c * c));
  k.hn = k.orth ? sqrt(n2) : (h2 > 0.0 ? sqrt(h2) : 0.0);
  return k;
}

// The Givens rotations of GMRES on the new Hessenberg column j = nv - 1 (the
// second pass, if any, changes only w, not H) and the stopping test of the
// host loop, taken here so that the next step, when already queued, exits at
// its gates.  One full wavefront, lane i on row i: the rotations are a serial
// chain, and their operands come from the lanes' registers.
__device__ __forceinline__ void gs_givens(DevState* st, const GsState& s, const GsCheck& k, int nv) {
  const int lane = threadIdx.x & 63, j = nv - 1;
  const double hc = k.h + k.csel;  // Hessenberg column before rotation
  const double hn = k.hn;
  double* H = st->H + j * ldh();
  double a = lane_value(hc, 0), row = 0.0;
  for (int i = 0; i < j; ++i) {  // previous rotations, in order, then the new one
    const double b = lane_value(hc, i + 1), c = lane_value(s.cs, i), sn = lane_value(s.sn, i);
    const double t = c * a + sn * b;
    if (lane == i) row = t;
    a = -sn * a + c * b;
  }
  const double rr = hypot(a, hn);
  // the three quotients a / rr, hn / rr and 1 / hn, a lane each
  const double num = lane == 0 ? a : lane == 1 ? hn : 1.0, den = lane == 2 ? hn : rr;
  const double q = den > 0.0 ? num / den : (lane == 0 ? 1.0 : 0.0);
  const double cr = lane_value(q, 0), sr = lane_value(q, 1), inv = lane_value(q, 2);
  if (lane == j) row = rr;
  if (lane <= nv) H[lane] = row;  // row nv: 0
  if (lane != 0) return;
  const int nreorth = s.nreorth + (k.orth ? 0 : 1);
  st->reorth = k.orth ? 0 : 1;
  st->nreorth = nreorth;
  st->hn = hn;
  st->vs[nv] = inv;
  st->cs[j] = cr;
  st->sn[j] = sr;
  st->g[j + 1] = -sr * s.g;
  st->g[j] = cr * s.g;
  const double resid = fabs(sr * s.g);
  st->resid = resid;
  const bool bad = s.bad || !k.finite || !isfinite(rr) || !isfinite(sr * s.g);
  const bool halt = bad || resid / s.stop_bnorm <= s.stop_rtol || j >= s.jlast;
  if (bad) st->bad = 1;
  if (halt) set_halt(st);
  post_step(s.mail, s.run, j, resid, 0.0, bad, halt, nreorth);
}

// End of the orthogonality check, by one full wavefront: the reduced values and
// second-pass coefficients to the state, then the rotations.
__device__ __forceinline__ void gs_end(DevState* st, const GsState& s, const GsCheck& k, const double* val, int nv) {
  const int lane = threadIdx.x & 63;
  if (lane <= nv) st->red[lane] = val[lane];
  if (lane < nv) {
    st->ccol[lane] = k.csel;
    st->coef[lane] = k.csel * k.v;
  }
  gs_givens(st, s, k, nv);
}

}  // namespace vd

// Fused pseudo-spectral passes of the variable-density operators (gfx950).
//
// Pressure operator (the paper's L_rho = div(rho^-1 grad), eq. VDINSE.Lrho,
// discretised as eq. VDINSE.Lrho.num), applied as A = -L_rho to a packed
// half-spectrum v, optionally preceded by the constant-density
// pseudo-inverse (Sec. 3, Sec. 4.2) -- right preconditioning:
//
//   P1 (z, inverse)  u = M^-1 v;  T1 = Fz^-1 u,  T1z = Fz^-1 (i k'_z u)
//   P2 (y, inverse)  U = Fy^-1 T1, Gy = Fy^-1 (i k'_y T1), Gz = Fy^-1 T1z
//   P3 (x, rows)     Q_d = Fx (a/N Fx^-1 G_d), with G_x = i k'_x U and the
//                    x-derivative of the divergence applied on the way out
//   P4 (y, forward)  S = Fy Qx' + i k'_y Fy Qy,  Qz2 = Fy Qz
//   P5 (z, forward)  y = -(Fz S + i k'_z Fz Qz2)
//
// 23 field transfers in 3D.  k' is the wavenumber with the Nyquist index
// zeroed (odd derivative).  2D grids skip P2/P4, 1D grids do everything in
// P3.  The Helmholtz-type operator rho u - nu Lap u (implicit viscous step)
// uses the same skeleton with one field: Fz^-1, Fy^-1, x: Fx(rho Fx^-1), Fy,
// Fz, plus nu |k|^2 (M^-1 v) added in P5 (Nyquist kept in |k|^2).
//
// Column passes (P1, P2, P4, P5) tile TC adjacent columns x the whole line:
// lanes map to adjacent columns, so every global access is a contiguous run
// of TC complex values.  The row pass loads whole rows.  All passes are
// in-place safe except those that gather a mirror element (Helmholtz, kx = 0).
#include <cstddef>
#include <cstdio>
#include <initializer_list>

#include "fft_core.hpp"
#include "gs_device.hpp"

#include "passes.hpp"
#include "spectral.hpp"

namespace vd {

// ------------------------------------------------------------ config

// Points per thread of a column line.  Measured on MI355X at 256^3 and 512^3
// (FP64 passes, us per launch, E = 16 -> 8):
//   L = 256: Helmholtz z-first 78 -> 62, z-last 99 -> 81, plain FFT 47 -> 44,
//            pressure y-inverse 127 -> 122; but pressure z-last 76 -> 86 and
//            y-forward 134 -> 135 (two transforms per thread, one more LDS
//            exchange each);
//   L = 512: every pass 40-70% slower (a 256-thread tile is then only 4
//            columns wide, 64 B per row access).
// E = 16 in FP64 needs ~256 VGPRs in the two-field modes and a 64 KB tile
// (one or two waves per SIMD); E = 8 halves both.
enum ColMode {
  COL_FFT_FWD = 0,  // NF fields, forward
  COL_FFT_INV,      // NF fields, inverse
  COL_P_FIRST,      // v -> Fz^-1(M v), Fz^-1(i k'_z M v)
  COL_P_MIDINV,     // T1, T1z -> Fy^-1 T1, Fy^-1(i k'_y T1), Fy^-1 T1z
  COL_P_MIDFWD,     // Qx', Qy, Qz -> Fy Qx' + i k'_y Fy Qy, Fy Qz
  COL_P_LAST,       // S, Qz2 -> -(Fz S + i k'_z Fz Qz2)
  COL_H_FIRST,      // v -> Fz^-1(M v)
  COL_H_LAST,       // Q2, v -> Fz Q2 + nu |k|^2 M v
};

// Lines of 512 points: points per thread E and threads per block NT, per
// pass (the tile is NT / (512 / E) columns wide and holds that many lines in
// LDS; 16 columns take 136 KiB in FP64, one block per CU).  Measured at
// 512^3, microseconds per pass for (E, NT) = (16, 256) / (16, 512) /
// (8, 1024):
//   FP64 pressure z-first 737 / 775 / 792, y-inverse 1086 / 1083 / 1241,
//        y-forward 1105 / 1075 / 1121, z-last 819 / 745 / 739;
//   FP64 Helmholtz z-first 525 / 562 / 511, z-last 1084 / 926 / 797, y
//        transforms 426 / 419 / 410 and 407 / 404 / 395;
//   FP32 pressure z-first 442 / 320 / 377, y-inverse 764 / 589 / 582,
//        y-forward 770 / 598 / 571, z-last 470 / 411 / 405.
// The wider tiles write longer contiguous runs of each line segment; the
// FP64 pressure z-first pass (one field in, two out) keeps two blocks per CU.
template <typename R, int MODE>
struct Col512 {
  static constexpr bool DBL = sizeof(R) == 8;
  static constexpr bool WIDE = DBL ? (MODE == COL_H_FIRST || MODE == COL_H_LAST || MODE == COL_FFT_FWD ||
                                      MODE == COL_FFT_INV)
                                   : (MODE == COL_P_MIDINV || MODE == COL_P_MIDFWD || MODE == COL_P_LAST);
  static constexpr int E = WIDE ? 8 : 16;
  static constexpr int NT = WIDE ? 1024 : (DBL && MODE == COL_P_FIRST ? 256 : 512);
};

// Small fields (SM).  Up to kSmallField slots a pass is not bound by memory but
// by how long one wavefront takes: its dependent loads (halt flag, twiddles,
// data) and its instructions, four cycles each with nothing else to run on the
// SIMD (32^3 FP64: 4 to 32 blocks, 5.2-7.9 us a pass against 1.5 us for a
// launch that returns at its gate).  So the small configuration
//   - issues the data and twiddle loads before it waits for the halt flag,
//   - gives a thread 8 points of a column line (4 of a row) and a block few
//     columns (TC: at least 64 B runs),
//   - runs the two or three transforms of a pressure pass side by side, one
//     group of wavefronts each (NG), instead of one after another.
// 32^3 FP64, before -> now: z-first 5.2 -> 4.4 us, y-inverse 6.3 -> 3.6,
// x 6.2 -> 4.2, y-forward 7.9 -> 3.8, z-last 6.4 -> 4.0; x pass of a 257 x 512
// wall grid 7.6 -> 5.5.  Larger fields keep the shapes below, which are chosen
// for bandwidth: with the limit at 2^20 slots a 64 x 128 x 256 FP32+refine
// solve took 3481 us instead of 3417.  (128^3 FP64 K took 1888 instead of 1953: the
// best limit depends on the type and lies between, where it is not measured.)
constexpr size_t kSmallField = kFoldElems;

constexpr int col_groups(int mode) {
  return mode == COL_P_FIRST || mode == COL_P_LAST ? 2 : mode == COL_P_MIDINV || mode == COL_P_MIDFWD ? 3 : 1;
}

template <int L>
struct ColSmall {
  static constexpr int E = 8, T = L / E;
  static constexpr int TC = L <= 64 ? 64 / T : (L == 128 ? 8 : 4);
  static constexpr int NTG = T * TC;  // threads per group, a multiple of 64
};
// lengths that the small configuration is built for
constexpr bool col_has_small(int L, int mode) { return L <= 256 || (col_groups(mode) <= 2 && L <= 1024); }

template <int L, typename R, int MODE, bool SM = false, bool GS = false>
struct ColCfg {
  // (GS: a Helmholtz pass gets a second group for the dots)
  static constexpr int NG = SM ? (GS && MODE == COL_H_LAST ? 2 : col_groups(MODE)) : 1;
  static constexpr bool E8 = sizeof(R) == 8 && L < 512 && MODE != COL_P_LAST && MODE != COL_P_MIDFWD;
  static constexpr int E = SM ? ColSmall<L>::E
                              : L == 512 ? Col512<R, MODE>::E : E8 ? (L >= 8 ? 8 : L) : (L >= 16 ? 16 : L);
  static constexpr int T = L / E;
  static constexpr int NTG = SM ? ColSmall<L>::NTG : L == 512 ? Col512<R, MODE>::NT : 256;
  static constexpr int NT = NG * NTG;                    // threads per block
  static constexpr int TC = NTG / T;                     // columns per tile
};

template <int L, typename R, bool SM = false>
struct RowCfg {
  // 8 points per thread: the x pass keeps a field's inverse and forward
  // transforms plus the half-length pre/post-processing live at once, and
  // 16 points per thread would cap FP64 occupancy at one wave/SIMD or spill.
  // FP32 rows too: at 256^3 (128-point rows) 16 points per thread took the
  // pressure x pass 126 us and the Helmholtz x pass 48 us, 8 points 113 and
  // 40 us.
  // Small fields: 4 points per thread where the row still fits a wavefront.
  static constexpr int E = SM && L >= 16 && L <= 256 ? 4 : L >= 16 ? 8 : L;
  static constexpr int T = L / E;
  static_assert(T <= 64, "a row must fit one wavefront");
  // A row's T threads are adjacent lanes of one wavefront and each row owns
  // its LDS slice, so the LDS exchanges need only wavefront-level ordering
  // (no block barrier).  Blocks are a few wavefronts (the CU overlaps the
  // load, transform and store phases of several blocks); the block shares
  // the twiddle tables, staged once in LDS.
  static constexpr int RW = 64 / T;  // rows per wavefront
  static constexpr int LP = row_pitch<L>();
  static constexpr bool WAVE = true;
};

// ------------------------------------------------------ column kernels


// One system's arguments in a batched launch: blockIdx.y selects system k
// of nb, which has its own fields, coefficient rows, preconditioner
// constant, input scale and gate (several independent systems solved
// together: the components of a velocity solve, or pressure solves on grids
// of one shape).
struct SysArgs {
  const void* in[3];
  void* out[3];
  const void* coef;  // row passes: the system's coefficient rows
  double rho0;
  const double* in_scale;
  const int* gate;
};

struct ColArgs {
  const void* in[3];
  void* out[3];
  int nf;            // fields for the plain FFT modes
  int outer, inner;  // data [outer][L][inner]
  int ntile;
  Geom g;
  double rho0, nu;
  int precond;
  const double* in_scale;
  const int* gate;  // nonzero *gate: the launch does nothing
  // The launch's systems: system blockIdx.y < nb reads its fields, scale,
  // preconditioner constant and gate from sys[blockIdx.y] (a launch of one
  // system has nb = 1, filled from in/out/rho0/in_scale/gate by the
  // launcher; the plain FFT modes take fields 1..nf-1 from in/out).
  int nb;
  SysArgs sys[kMaxBatch];
};

template <int L, int E, int RPAT, typename R>
__device__ __forceinline__ void col_load(C2<R>* reg, const C2<R>* p, size_t base, int inner,
                                         int t, bool ok) {
#pragma unroll
  for (int s = 0; s < E; ++s) {
    int idx = pat_index<L, E, RPAT>(t, s);
    reg[s] = ok ? ldg(p + base + (size_t)idx * inner) : C2<R>{R(0), R(0)};
  }
}
template <int L, int E, int RPAT, typename R>
__device__ __forceinline__ void col_store(const C2<R>* reg, C2<R>* p, size_t base, int inner,
                                          int t, bool ok) {
  if (!ok) return;
#pragma unroll
  for (int s = 0; s < E; ++s) {
    int idx = pat_index<L, E, RPAT>(t, s);
    stg(p + base + (size_t)idx * inner, reg[s]);
  }
}

// The block's system, sys[blockIdx.y] of the kernel's first argument (of
// type Args, at the start of the kernel-argument segment), read in place:
// constant memory at a uniform address, so scalar loads.  Indexing the
// by-value argument itself with a run-time index would make the compiler
// copy the whole argument block to scratch memory first.
typedef __attribute__((address_space(4))) const SysArgs KSys;
template <typename Args>
__device__ __forceinline__ KSys* block_sys() {
  typedef __attribute__((address_space(4))) const char KChar;
  KChar* seg = (KChar*)__builtin_amdgcn_kernarg_segment_ptr();
  return (KSys*)(seg + offsetof(Args, sys)) + blockIdx.y;
}

// Gram-Schmidt work of a small field's first or last pass (GsCarry): a step
// then is the operator's passes and one update kernel.  On their own, the dots
// and the check each were a launch of 4 to 7 us that mostly waited for its first
// loads; here
//   - the last pass forms the dots with its result while it still holds it: its
//     groups of wavefronts share the vectors, and the first few each are
//     loaded before the transform;
//   - every block of the first pass reduces the check dots for itself while its
//     column is on the way, and one more block takes the rotations, so that
//     their serial chain runs beside the transforms.
// 32^3 FP64, us a launch, on their own -> here: dots 4.1 + z-last 3.8 -> 6.0, check
// 7.0 + z-first 4.3 -> 6.3; solve 897 -> 677 us, 24 served 2D requests 11.7 -> 11.2 ms.
struct ColGs {
  int nv;      // last pass: vectors of the dots; first pass: vectors of the step to finish
  int nb;      // first pass: blocks that left the check dots
  double tol, scale;
  struct Sys {
    DevState* st;
    double* partial;
    const void* V[kMaxVec];
  } sys[kMaxBatch];
};
// CG and RMR work of the first or last pass (RecCarry), for fields of any size:
// the direction's update, a pass of its own over three fields, takes one field
// more in the first pass, which reads the direction anyway; the dots of the last
// pass' result, two fields, take at most one; and the reduction with the stopping
// test runs beside the first pass in one more block.  128^3 FP64, us a step: k_cg_p
// 10.6 + z-first 8.6 -> 15.3, z-last 10.8 + dots 6.7 -> 11.7, reduction 4.0 -> 0; K
// form by CG 1780 -> 1676 us a solve.
struct ColRec {
  int cg, precond;
  int nb, slot;
  double scale;
  DevState* st;
  double* partial;
  const void* r;
  void* p;
};
// What a launch carries beside the transforms.
enum Carry { CARRY_NONE = 0, CARRY_GS, CARRY_REC };
template <typename T>
struct ColCarryKernArgs {  // the kernel-argument segment of k_col_gs and k_col_rec
  ColArgs a;
  const void* tw;
  T carry;
};
typedef __attribute__((address_space(4))) const ColGs KGs;
template <typename T>
__device__ __forceinline__ auto* kern_carry() {
  typedef __attribute__((address_space(4))) const char KChar;
  typedef __attribute__((address_space(4))) const T KT;
  return (KT*)((KChar*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(ColCarryKernArgs<T>, carry));
}

// val[0..K) = the sums of nb <= kFoldBlocks block partials, by all NW wavefronts
// of the block.  Four lanes sum a value, with up to 16 loads each in flight: with
// one or two wavefronts a tree over all lanes for every value, one value after
// another, took longer than the loads.
template <int NW>
__device__ __forceinline__ void fold_sums(const double* partial, int nb, int K, double scale, double* val) {
  constexpr int Q = 16;
  const int q = threadIdx.x & 3;
  for (int i = threadIdx.x >> 2; i < K; i += 16 * NW) {
    const double* src = partial + (size_t)i * kRedBlocks;
    double s = 0.0;
    for (int b0 = q; b0 < nb; b0 += 4 * Q) {
      double t[Q];
#pragma unroll
      for (int m = 0; m < Q; ++m) t[m] = b0 + 4 * m < nb ? src[b0 + 4 * m] : 0.0;
#pragma unroll
      for (int h = Q / 2; h > 0; h >>= 1) {
#pragma unroll
        for (int m = 0; m < h; ++m) t[m] += t[m + h];
      }
      s += t[0];
    }
    s = add_dpp<0xb1, 0xf>(s);  // lanes q ^ 1
    s = add_dpp<0x4e, 0xf>(s);  // lanes q ^ 2
    if (q == 0) val[i] = s * scale;
  }
}

// M^-1 r at kz = pat_index(t, s) of a thread's column, all E points: r and, where
// the Helmholtz inverse needs it, r at the mirror have been loaded.
template <int L, int E, int RPAT, bool HELM, typename R>
__device__ __forceinline__ C2<R> precond_point(int s, C2<R> r, C2<R> rm, int kx, int ky, int t, const ColArgs& a,
                                               double rho0) {
  const int kz = pat_index<L, E, RPAT>(t, s);
  if constexpr (HELM) {
    const HelmMult<R> h = mult_helm<R>(kx, ky, kz, a.g, rho0, a.nu, false);
    return kx ? cscale(r, h.g0) : diag_packed(r, rm, h.g0, h.gN);
  } else {
    return cscale(r, mult_press<R>(kx, ky, kz, a.g, rho0));
  }
}

template <int L, typename R, int MODE, bool SM, int CARRY>
__device__ __forceinline__ void col_pass(const ColArgs& a, const C2<R>* __restrict__ twtab) {
  constexpr bool GS = CARRY == CARRY_GS, REC = CARRY == CARRY_REC;
  constexpr bool ENDS = REC && (MODE == COL_P_FIRST || MODE == COL_H_FIRST);
  constexpr bool DOT = REC && (MODE == COL_P_LAST || MODE == COL_H_LAST);
  static_assert(!REC || ENDS || DOT, "CG and RMR work of first and last passes");
  using Cf = ColCfg<L, R, MODE, SM, GS>;
  constexpr bool CHECK = GS && MODE == COL_P_FIRST, DOTS = GS && (MODE == COL_P_LAST || MODE == COL_H_LAST);
  static_assert(!GS || (SM && (CHECK || DOTS)), "Gram-Schmidt work of small fields' first and last passes");
  constexpr int E = Cf::E, T = Cf::T, TC = Cf::TC, NTG = Cf::NTG, NG = Cf::NG, NT = Cf::NT;
  using S = Sched<L, E>;
  constexpr int R0 = S::template first_radix<false>();
  constexpr int R1 = S::template last_radix<false>();
  constexpr int LDSN = S::npass > 1 ? NG * TC * L : 1;
  // this block's system, read from the kernel-argument segment (one code
  // path for a launch of one system and a batch)
  KSys* sy = block_sys<ColArgs>();
  const int* gate = sy->gate;
  // CHECK, ENDS: this launch's own extra block may set the flag (halt_now); in the
  // others it was written before the launch
  constexpr bool OWN = CHECK || ENDS;
  if (!SM && !OWN && gate && *gate) return;
  const void* in0 = sy->in[0];
  const void* in1 = sy->in[1];
  const void* in2 = sy->in[2];
  void* out0 = sy->out[0];
  void* out1 = sy->out[1];
  void* out2 = sy->out[2];
  const double* iscale = sy->in_scale;
  const double rho0 = sy->rho0;
  __shared__ C2<R> lds_raw[LDSN];
  // twiddle table staged in LDS (see k_row)
  __shared__ C2<R> tw_lds[L];

  const int grp = NG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NTG) : 0;
  const int tid = NG > 1 ? threadIdx.x - grp * NTG : threadIdx.x;
  const int c = tid % TC, t = tid / TC;
  // CHECK: the block past the tiles takes the rotations
  // (ENDS: the stopping test)
  const bool rotations = (CHECK || ENDS) && (int)blockIdx.x == a.ntile;
  const int ob = CHECK || ENDS ? 0 : blockIdx.x / a.ntile, tile = CHECK || ENDS ? blockIdx.x : blockIdx.x % a.ntile;
  const int col = tile * TC + c;
  const bool ok = col < a.inner && !rotations;
  // A block that sees the flag leaves its tile as it is: what follows a halted step
  // reads neither the direction and the vector that this pass would complete nor
  // its results.
  __shared__ int halted;
  int seen = 0;  // thread 0's reading, on its way until the block's first barrier
  if (OWN && threadIdx.x == 0) seen = halt_now(gate);
  const size_t base = (size_t)ob * L * a.inner + col;
  LdsCol<R> lds{lds_raw + (NG > 1 ? grp * TC * L : 0), c, TC};
  C2<R> reg[E];

  // DOTS: this group's vectors, i = grp + NG q for q < nq, VB at a time (four
  // spill where 512 threads share the registers with M v)
  constexpr int VB = MODE == COL_H_LAST && L == 512 && sizeof(R) == 8 ? 2 : 4;
  __shared__ double dsum[DOTS ? NT / 64 : 1][DOTS ? kMaxVec / 2 : 1];
  C2<R> vb[DOTS ? VB : 1][E];
  KGs* gs = GS ? kern_carry<ColGs>() : nullptr;
  const int nv = GS ? gs->nv : 0, nq = DOTS ? (nv - grp + NG - 1) / NG : 0;
  auto load_vectors = [&](int q0) {
#pragma unroll
    for (int b = 0; b < VB; ++b)
      if (q0 + b < nq)
        col_load<L, E, R1>(vb[DOTS ? b : 0], (const C2<R>*)gs->sys[blockIdx.y].V[grp + NG * (q0 + b)], base, a.inner, t,
                           ok);
  };
  auto dots = [&]() {  // reg: this thread's part of the result, in every group
    const double w = (col & (a.g.M - 1)) == 0 ? 1.0 : 2.0;  // as spec_w
    const int wave = threadIdx.x >> 6;
    for (int q0 = 0; q0 < nq; q0 += VB) {
      if (q0) load_vectors(q0);
#pragma unroll
      for (int b = 0; b < VB; ++b) {
        if (q0 + b >= nq) continue;
        double d = 0.0;
#pragma unroll
        for (int s = 0; s < E; ++s)
          d += (double)vb[DOTS ? b : 0][s].x * (double)reg[s].x + (double)vb[DOTS ? b : 0][s].y * (double)reg[s].y;
        d = wave_sum(w * d);
        if ((threadIdx.x & 63) == 0) dsum[DOTS ? wave : 0][DOTS ? q0 + b : 0] = d;
      }
    }
    __syncthreads();
    const int i = threadIdx.x;
    if (i < nv) {
      constexpr int WG = NTG / 64 > 0 ? NTG / 64 : 1;  // wavefronts per group
      double d = 0.0;
#pragma unroll
      for (int q = 0; q < WG; ++q) d += dsum[DOTS ? (i % NG) * WG + q : 0][DOTS ? i / NG : 0];
      gs->sys[blockIdx.y].partial[(size_t)i * kRedBlocks + blockIdx.x] = d;
    }
  };
  if constexpr (DOTS) load_vectors(0);
  // ENDS: the end of the step before.  The first wavefront sums the partials of
  // (r, M^-1 r) for beta, in the last block also those of |r|^2 for the test; rz
  // alternates between two entries, because blocks still read the old one.
  auto* rec = kern_carry<ColRec>();  // used with REC only
  __shared__ double cbeta;
  const bool upd = ENDS && rec->cg;
  auto end_step = [&]() {
    if (threadIdx.x >= 64 || !(rec->cg || rotations)) return;
    DevState* st = rec->st;
    const double* part = rec->partial + 2 * kRedBlocks;
    RecState s{};
    double old = 0.0;
    if (rotations) s = rec_state(st, rec->slot);
    if (rec->cg) old = st->rz[rec->slot];
    const double rzn = rec->cg ? sum_partials(part + kRedBlocks, rec->nb) * rec->scale : 0.0;
    if (rotations) {
      const double n2 = sum_partials(part, rec->nb) * rec->scale;
      if (threadIdx.x == 0 && !seen) {
        st->red[0] = n2;
        st->red[1] = rzn;
        if (!rec_check_step(st, s, n2) && rec->cg) cg_beta_step(st, s, rzn, rec->slot ^ 1);
      }
    } else if (threadIdx.x == 0) {
      cbeta = cg_beta(old, rzn);
    }
  };
  // p = M^-1 r + beta p on this thread's points (x: p), with r loaded before
  constexpr bool HELM = MODE == COL_H_FIRST;
  C2<R> rr[ENDS ? E : 1], rm[ENDS && HELM ? E : 1];
  auto load_r = [&]() {
    if (!upd) return;
    const C2<R>* r = (const C2<R>*)rec->r;
    col_load<L, E, R0>(rr, r, base, a.inner, t, ok);
    if constexpr (ENDS && HELM) {
      const int ky = col / a.g.M;
      if (col % a.g.M == 0 && rec->precond && ok) {
#pragma unroll
        for (int s = 0; s < E; ++s)
          rm[s] = ldg(r + (size_t)((a.g.ny - ky) % a.g.ny) * a.g.M + (size_t)((L - pat_index<L, E, R0>(t, s)) % L) * a.inner);
      }
    }
  };
  auto new_p = [&](C2<R>* x) {
    const double b = cbeta;
    const int ky = col / a.g.M, kx = col % a.g.M;
#pragma unroll
    for (int s = 0; s < E; ++s) {
      C2<R> z = rr[ENDS ? s : 0];
      if (rec->precond)
        z = precond_point<L, E, R0, HELM>(s, z, rm[ENDS && HELM ? s : 0], kx, ky, t, a, rho0);
      x[s] = ok ? C2<R>{R(z.x + b * x[s].x), R(z.y + b * x[s].y)} : C2<R>{R(0), R(0)};
    }
  };
  // DOT: (y, p), and for RMR |y|^2, of the result y that group 0 holds; p's points
  // in the same pattern
  __shared__ double rsum[DOT ? NT / 64 : 1][2];
  C2<R> pv[DOT ? E : 1];
  auto load_p = [&]() {
    if (grp == 0) col_load<L, E, R1>(pv, (const C2<R>*)rec->p, base, a.inner, t, ok);
  };
  auto rec_dots = [&](const C2<R>* y) {
    double d = 0.0, n = 0.0;
    if (grp == 0) {
      const double w = (col & (a.g.M - 1)) == 0 ? 1.0 : 2.0;  // as spec_w
#pragma unroll
      for (int s = 0; s < E; ++s) {
        d += w * ((double)pv[DOT ? s : 0].x * (double)y[s].x + (double)pv[DOT ? s : 0].y * (double)y[s].y);
        n += w * ((double)y[s].x * (double)y[s].x + (double)y[s].y * (double)y[s].y);
      }
      d = wave_sum(d);
      n = wave_sum(n);
      if ((threadIdx.x & 63) == 0) {
        rsum[DOT ? threadIdx.x >> 6 : 0][0] = d;
        rsum[DOT ? threadIdx.x >> 6 : 0][1] = n;
      }
    }
    __syncthreads();
    if (threadIdx.x < (rec->cg ? 1 : 2)) {
      constexpr int WG = NTG / 64;
      double v = rsum[0][threadIdx.x];
#pragma unroll
      for (int q = 1; q < WG; ++q) v += rsum[DOT ? q : 0][threadIdx.x];
      rec->partial[(size_t)threadIdx.x * kRedBlocks + blockIdx.x] = v;
    }
  };
  if constexpr (SM && ENDS) load_r();
  if constexpr (SM && DOT) load_p();
  // CHECK: coefficients of the second pass, the scale of the result
  __shared__ double cval[CHECK ? kMaxVec + 2 : 1], ccl[CHECK ? kMaxVec : 1], cinv;
  __shared__ int again;
  double vscale = 1.0;
  R mult[SM && MODE == COL_P_FIRST ? E : 1];

  if constexpr (SM) {
    // every load that does not depend on another one, then the halt flag
    constexpr int NTW = (L + NT - 1) / NT;
    C2<R> twr[NTW];
#pragma unroll
    for (int i = 0; i < NTW; ++i)
      if (i * NT + (int)threadIdx.x < L) twr[i] = ldg(twtab + L + i * NT + threadIdx.x);
    const void* src = NG == 3 ? (MODE == COL_P_MIDINV ? (grp == 2 ? in1 : in0) : (grp == 0 ? in0 : grp == 1 ? in1 : in2))
                      : MODE == COL_P_LAST && grp == 1 ? in1 : in0;
    col_load<L, E, R0>(reg, (const C2<R>*)src, base, a.inner, t, ok);
    if constexpr (MODE == COL_P_FIRST) {  // divisions, while the loads are on their way
      const int ky = col / a.g.M, kx = col % a.g.M;
#pragma unroll
      for (int s = 0; s < E; ++s)
        mult[s] = a.precond ? mult_press<R>(kx, ky, pat_index<L, E, R0>(t, s), a.g, rho0) : R(1);
    }
    GsState state{};
    DevState* st = CHECK ? gs->sys[blockIdx.y].st : nullptr;
    if (CHECK && threadIdx.x < 64) state = gs_state(st, nv, rotations);
    if (!OWN && gate && *gate) return;
#pragma unroll
    for (int i = 0; i < NTW; ++i)
      if (i * NT + (int)threadIdx.x < L) tw_lds[i * NT + threadIdx.x] = twr[i];
    if constexpr (CHECK) {
      fold_sums<NT / 64>(gs->sys[blockIdx.y].partial + kFoldHalf, gs->nb, nv + 1, gs->scale, cval);
      if (threadIdx.x == 0) halted = seen;
      __syncthreads();
      if (halted) return;
      if (threadIdx.x < 64) {
        const GsCheck k = gs_check(state, cval, nv, gs->tol);
        if (rotations) {
          gs_end(st, state, k, cval, nv);
        } else {
          if ((int)threadIdx.x < nv) ccl[threadIdx.x] = k.csel * k.v;
          if (threadIdx.x == 0) {
            again = !k.orth;
            cinv = k.hn > 0.0 ? 1.0 / k.hn : 0.0;
          }
        }
      }
      if (rotations) return;
    }
  } else {
    for (int i = threadIdx.x; i < L; i += blockDim.x) tw_lds[i] = twtab[L + i];
  }
  if constexpr (ENDS) {
    end_step();
    if (rotations) return;
    if (threadIdx.x == 0) halted = seen;
  }
  __syncthreads();
  if (ENDS && halted) return;
  const C2<R>* tw = tw_lds;
  // CHECK: the second pass on this tile.  Both groups hold the column and form
  // the same values; group 0 writes them back after its transform, when both
  // have consumed their loads.
  C2<R> kept[CHECK || (SM && ENDS) ? E : 1];
  if constexpr (SM && ENDS) {
    if (upd) {
      new_p(reg);
#pragma unroll
      for (int s = 0; s < E; ++s) kept[s] = reg[s];
    }
  }
  if constexpr (CHECK) {
    static_assert(S::npass > 1, "a barrier between the loads and the stores");
    vscale = cinv;
    if (again) {
      double xr[E], xi[E];
#pragma unroll
      for (int s = 0; s < E; ++s) {
        xr[s] = reg[s].x;
        xi[s] = reg[s].y;
      }
      for (int i = 0; i < nv; ++i) {
        const double ci = ccl[i];
        if (ci == 0.0) continue;
        C2<R> v[E];
        col_load<L, E, R0>(v, (const C2<R>*)gs->sys[blockIdx.y].V[i], base, a.inner, t, ok);
#pragma unroll
        for (int s = 0; s < E; ++s) {
          xr[s] -= ci * (double)v[s].x;
          xi[s] -= ci * (double)v[s].y;
        }
      }
#pragma unroll
      for (int s = 0; s < E; ++s) kept[s] = reg[s] = C2<R>{R(xr[s]), R(xi[s])};
    }
  }

  if constexpr (SM && NG > 1 && MODE != COL_H_LAST) {
    // one transform per group; every group meets the same barriers
    if constexpr (MODE == COL_P_FIRST) {
      const R sc = CHECK ? R(vscale) : in_scale_of<R>(iscale);
#pragma unroll
      for (int s = 0; s < E; ++s) {
        reg[s] = cscale(reg[s], mult[s] * sc);
        if (grp == 1) reg[s] = cik(reg[s], kprime_of<R>(pat_index<L, E, R0>(t, s), L, R(a.g.sz)));
      }
      fft_line<L, E, +1, false>(reg, lds, tw, t);
      col_store<L, E, R1>(reg, (C2<R>*)(grp ? out1 : out0), base, a.inner, t, ok);
      if constexpr (CHECK) {
        if (again && grp == 0) col_store<L, E, R0>(kept, (C2<R>*)in0, base, a.inner, t, ok);
      }
      if constexpr (ENDS) {
        if (upd && grp == 0) col_store<L, E, R0>(kept, (C2<R>*)rec->p, base, a.inner, t, ok);
      }
    } else if constexpr (MODE == COL_P_MIDINV) {
      // in place (out0 = in0, out2 = in1): both readers of in0 have consumed
      // their loads before the first exchange's barrier
      static_assert(S::npass > 1, "a barrier between the loads and the stores");
      if (grp == 1) {
#pragma unroll
        for (int s = 0; s < E; ++s) reg[s] = cik(reg[s], kprime_of<R>(pat_index<L, E, R0>(t, s), L, R(a.g.sy)));
      }
      fft_line<L, E, +1, false>(reg, lds, tw, t);
      col_store<L, E, R1>(reg, (C2<R>*)(grp == 0 ? out0 : grp == 1 ? out1 : out2), base, a.inner, t, ok);
    } else {
      constexpr bool LAST = MODE == COL_P_LAST;
      const R sk = LAST ? R(a.g.sz) : R(a.g.sy);
      fft_line<L, E, -1, false>(reg, lds, tw, t);
      __syncthreads();  // group 1's tile has been read
      if (grp == 1) {
#pragma unroll
        for (int s = 0; s < E; ++s) {
          const int idx = pat_index<L, E, R1>(t, s);
          lds.st(idx, cik(reg[s], kprime_of<R>(idx, L, sk)));
        }
      }
      __syncthreads();
      if (grp == 0) {
        const LdsCol<R> other{lds_raw + TC * L, c, TC};
#pragma unroll
        for (int s = 0; s < E; ++s) {
          const C2<R> d = other.ld(pat_index<L, E, R1>(t, s));
          reg[s] = LAST ? C2<R>{-(reg[s].x + d.x), -(reg[s].y + d.y)} : reg[s] + d;
        }
        col_store<L, E, R1>(reg, (C2<R>*)out0, base, a.inner, t, ok);
      } else if (!LAST && grp == 2) {
        col_store<L, E, R1>(reg, (C2<R>*)out1, base, a.inner, t, ok);
      }
      if constexpr (DOT) rec_dots(reg);
      if constexpr (DOTS) {  // the result to the other group through group 0's tile
        const LdsCol<R> mine{lds_raw, c, TC};
        if (grp == 0) {
#pragma unroll
          for (int s = 0; s < E; ++s) mine.st(pat_index<L, E, R1>(t, s), reg[s]);
        }
        __syncthreads();
        if (grp != 0) {
#pragma unroll
          for (int s = 0; s < E; ++s) reg[s] = mine.ld(pat_index<L, E, R1>(t, s));
        }
        dots();
      }
    }
    return;
  }

  if constexpr (MODE == COL_FFT_FWD || MODE == COL_FFT_INV) {
    constexpr int DIR = MODE == COL_FFT_FWD ? -1 : +1;
    const int nf = a.nf;
    for (int f = 0; f < nf; ++f) {
      if (!SM || f) col_load<L, E, R0>(reg, (const C2<R>*)(f ? a.in[f] : in0), base, a.inner, t, ok);
      fft_line<L, E, DIR, false>(reg, lds, tw, t);
      col_store<L, E, R1>(reg, (C2<R>*)(f ? a.out[f] : out0), base, a.inner, t, ok);
    }
  } else if constexpr (MODE == COL_P_FIRST) {
    // z pass: line index = kz; column = ky * M + kx
    const int ky = col / a.g.M, kx = col % a.g.M;
    const R sc = in_scale_of<R>(iscale);
    col_load<L, E, R0>(reg, (const C2<R>*)in0, base, a.inner, t, ok);
    if constexpr (ENDS) {
      if (upd) {
        load_r();
        new_p(reg);
        col_store<L, E, R0>(reg, (C2<R>*)rec->p, base, a.inner, t, ok);
      }
    }
    C2<R> r2[E];
#pragma unroll
    for (int s = 0; s < E; ++s) {
      int kz = pat_index<L, E, R0>(t, s);
      R m = a.precond ? mult_press<R>(kx, ky, kz, a.g, rho0) : R(1);
      reg[s] = cscale(reg[s], m * sc);
      r2[s] = cik(reg[s], kprime_of<R>(kz, L, R(a.g.sz)));
    }
    fft_line<L, E, +1, false>(reg, lds, tw, t);
    col_store<L, E, R1>(reg, (C2<R>*)out0, base, a.inner, t, ok);
    fft_line<L, E, +1, false>(r2, lds, tw, t);
    col_store<L, E, R1>(r2, (C2<R>*)out1, base, a.inner, t, ok);
  } else if constexpr (MODE == COL_P_MIDINV) {
    // y pass over z-physical data: line index = ky
    col_load<L, E, R0>(reg, (const C2<R>*)in0, base, a.inner, t, ok);
    C2<R> r2[E];
#pragma unroll
    for (int s = 0; s < E; ++s) r2[s] = cik(reg[s], kprime_of<R>(pat_index<L, E, R0>(t, s), L, R(a.g.sy)));
    fft_line<L, E, +1, false>(reg, lds, tw, t);
    col_store<L, E, R1>(reg, (C2<R>*)out0, base, a.inner, t, ok);
    fft_line<L, E, +1, false>(r2, lds, tw, t);
    col_store<L, E, R1>(r2, (C2<R>*)out1, base, a.inner, t, ok);
    col_load<L, E, R0>(reg, (const C2<R>*)in1, base, a.inner, t, ok);
    fft_line<L, E, +1, false>(reg, lds, tw, t);
    col_store<L, E, R1>(reg, (C2<R>*)out2, base, a.inner, t, ok);
  } else if constexpr (MODE == COL_P_MIDFWD || MODE == COL_P_LAST) {
    // forward y (MIDFWD) or z (LAST) with the divergence term of this axis
    constexpr bool LAST = MODE == COL_P_LAST;
    const R sk = LAST ? R(a.g.sz) : R(a.g.sy);
    C2<R> acc[E];
    col_load<L, E, R0>(acc, (const C2<R>*)in0, base, a.inner, t, ok);
    fft_line<L, E, -1, false>(acc, lds, tw, t);
    col_load<L, E, R0>(reg, (const C2<R>*)in1, base, a.inner, t, ok);
    fft_line<L, E, -1, false>(reg, lds, tw, t);
#pragma unroll
    for (int s = 0; s < E; ++s) {
      C2<R> d = cik(reg[s], kprime_of<R>(pat_index<L, E, R1>(t, s), L, sk));
      acc[s] = LAST ? C2<R>{-(acc[s].x + d.x), -(acc[s].y + d.y)} : acc[s] + d;
    }
    col_store<L, E, R1>(acc, (C2<R>*)out0, base, a.inner, t, ok);
    if constexpr (DOT) {
      load_p();
      rec_dots(acc);
    }
    if constexpr (!LAST) {
      col_load<L, E, R0>(reg, (const C2<R>*)in2, base, a.inner, t, ok);
      fft_line<L, E, -1, false>(reg, lds, tw, t);
      col_store<L, E, R1>(reg, (C2<R>*)out1, base, a.inner, t, ok);
    }
  } else if constexpr (MODE == COL_H_FIRST || MODE == COL_H_LAST) {
    if constexpr (DOTS) {
      if (grp != 0) {  // the second group meets the transform's barriers and takes its part of the dots
#pragma unroll
        for (int i = 0; i < 2 * (S::npass - 1); ++i) __syncthreads();
        __syncthreads();
        __syncthreads();
        const LdsCol<R> res{lds_raw, c, TC};
#pragma unroll
        for (int s = 0; s < E; ++s) reg[s] = res.ld(pat_index<L, E, R1>(t, s));
        dots();
        return;
      }
    }
    constexpr bool FIRST = MODE == COL_H_FIRST;
    constexpr int RP = FIRST ? R0 : R1;  // pattern in which v is needed
    const int ky = col / a.g.M, kx = col % a.g.M;
    const R sc = in_scale_of<R>(iscale);
    const C2<R>* v = (const C2<R>*)(FIRST ? in0 : in1);
    C2<R> mv[E];
    if constexpr (SM && FIRST) {
#pragma unroll
      for (int s = 0; s < E; ++s) mv[s] = reg[s];
      if constexpr (ENDS) {
        if (upd) col_store<L, E, R0>(kept, (C2<R>*)rec->p, base, a.inner, t, ok);
      }
    } else {
      col_load<L, E, RP>(mv, v, base, a.inner, t, ok);
      if constexpr (ENDS) {
        if (upd) {
          load_r();
          new_p(mv);
          col_store<L, E, R0>(mv, (C2<R>*)rec->p, base, a.inner, t, ok);
        }
      }
    }
    const bool need_mirror = (kx == 0) && (a.precond || !FIRST);
    const int kym = (a.g.ny - ky) % a.g.ny;
    const size_t basem = (size_t)ob * L * a.inner + (size_t)kym * a.g.M;
#pragma unroll
    for (int s = 0; s < E; ++s) {
      int kz = pat_index<L, E, RP>(t, s);
      if (!a.precond && FIRST) {
        mv[s] = cscale(mv[s], sc);
      } else {
        HelmMult<R> h = a.precond ? mult_helm<R>(kx, ky, kz, a.g, rho0, a.nu, !FIRST)
                                  : HelmMult<R>{R(0), R(0)};
        if (!a.precond) {  // last pass without preconditioner: nu |k|^2 v
          R kyz = ksq_yz<R>(ky, kz, a.g);
          R kx2 = R(kx) * R(a.g.sx);
          R kn = R(a.g.M) * R(a.g.sx);
          h.g0 = R(a.nu) * (kyz + kx2 * kx2);
          h.gN = R(a.nu) * (kyz + kn * kn);
        }
        if (need_mirror && ok) {
          int kzm = (L - kz) % L;
          C2<R> pm = ldg(v + basem + (size_t)kzm * a.inner);
          mv[s] = cscale(diag_packed(mv[s], pm, h.g0, h.gN), sc);
        } else {
          mv[s] = cscale(mv[s], h.g0 * sc);
        }
      }
    }
    if constexpr (FIRST) {
      fft_line<L, E, +1, false>(mv, lds, tw, t);
      col_store<L, E, R1>(mv, (C2<R>*)out0, base, a.inner, t, ok);
    } else {
      if (!SM) col_load<L, E, R0>(reg, (const C2<R>*)in0, base, a.inner, t, ok);
      fft_line<L, E, -1, false>(reg, lds, tw, t);
#pragma unroll
      for (int s = 0; s < E; ++s) reg[s] = reg[s] + mv[s];
      col_store<L, E, R1>(reg, (C2<R>*)out0, base, a.inner, t, ok);
      if constexpr (DOT) {
        if constexpr (!SM) load_p();
        rec_dots(reg);
      }
      if constexpr (DOTS) {
        __syncthreads();  // the tile's last exchange has been read
#pragma unroll
        for (int s = 0; s < E; ++s) lds.st(pat_index<L, E, R1>(t, s), reg[s]);
        __syncthreads();
        dots();
      }
    }
  }
}

template <int L, typename R, int MODE, bool SM>
__global__ __launch_bounds__((ColCfg<L, R, MODE, SM>::NT)) void k_col(ColArgs a, const C2<R>* __restrict__ twtab) {
  col_pass<L, R, MODE, SM, CARRY_NONE>(a, twtab);
}
template <int L, typename R, int MODE>
__global__ __launch_bounds__((ColCfg<L, R, MODE, true, true>::NT)) void k_col_gs(ColArgs a,
                                                                               const C2<R>* __restrict__ twtab,
                                                                               ColGs) {
  col_pass<L, R, MODE, true, CARRY_GS>(a, twtab);
}
template <int L, typename R, int MODE, bool SM>
__global__ __launch_bounds__((ColCfg<L, R, MODE, SM>::NT)) void k_col_rec(ColArgs a, const C2<R>* __restrict__ twtab,
                                                                         ColRec) {
  col_pass<L, R, MODE, SM, CARRY_REC>(a, twtab);
}

// --------------------------------------------------------- row kernels

enum RowMode {
  ROW_R2C = 0,  // real rows -> packed spectrum (forward)
  ROW_C2R,      // packed spectrum -> real rows, times cscale
  ROW_P,        // pressure x pass, nf fields: field 0 gets i k'_x in and out
  ROW_P1,       // 1D pressure: y = -i k'_x F(a F^-1(i k'_x M v))
  ROW_H,        // Helmholtz x pass (rho times), one field
  ROW_H1,       // 1D Helmholtz: y = F(rho F^-1(M v)) + nu k^2 M v
};

struct RowArgs {
  const void* in[3];
  void* out[3];
  int nf;
  int nrows;
  const void* coef;  // real rows (R), nullptr for transforms
  double cscale;
  Geom g;
  double rho0, nu;
  int precond;
  const double* in_scale;
  const int* gate;  // nonzero *gate: the launch does nothing
  // The operator x passes (ROW_P, ROW_H): system blockIdx.y < nb reads its
  // fields, coefficient rows, scale, preconditioner constant and gate from
  // sys[blockIdx.y] (nb = 1 for one system, filled by the launcher); the
  // other modes use in/out/coef/... directly.
  int nb;
  SysArgs sys[kMaxBatch];
};

// Wavefronts per block: the pressure x pass runs its (up to three) fields as
// one wavefront each over the same rows; the other modes run four
// wavefronts over consecutive row groups.
template <int MODE>
constexpr bool row_field_waves() { return MODE == ROW_P; }
template <int MODE>
constexpr int row_waves() { return row_field_waves<MODE>() ? 3 : 4; }

// Row passes that loop over row groups in a grid capped at kRowGridCap
// blocks.  In the loop the compiler keeps each thread's twiddle factors
// (they depend only on its lane) in registers across rows instead of reading
// them from LDS for every row, at the price of 40-60 more VGPRs.  Measured per
// kernel against one row group per block: the FP64 pressure x pass on
// 256-point rows (512^3 grid) 1733 -> 1628 us at two waves per SIMD instead
// of three, the Helmholtz x pass on 128-point rows 72.0 -> 69.4 us (FP64) and
// 40.0 -> 38.8 us (FP32).  Elsewhere the lost occupancy costs more (the FP64
// pressure x pass on 128-point rows 205 -> 249 us).  Blocks that loop
// without keeping the twiddles are slower still: many short blocks overlap
// their load, transform and store phases better than a few long ones.
template <int L, typename R, int MODE>
constexpr bool row_loop() {
  return (MODE == ROW_P && L == 256 && sizeof(R) == 8) || (MODE == ROW_H && L == 128);
}

template <int L, typename R, int MODE, bool SM>
__global__ __launch_bounds__(64 * row_waves<MODE>()) void k_row(RowArgs a, const C2<R>* __restrict__ twtab) {
  using Cf = RowCfg<L, R, SM>;
  constexpr int E = Cf::E, T = Cf::T, RW = Cf::RW, LP = Cf::LP;
  constexpr bool WV = Cf::WAVE;
  using S = Sched<L, E>;
  constexpr int RI1 = S::template last_radix<false>();   // inverse output pattern
  constexpr int RF0 = S::template first_radix<true>();   // forward input pattern (== RI1)
  static_assert(RI1 == RF0, "pattern mismatch");
  constexpr int NW = row_waves<MODE>();
  constexpr bool FW = row_field_waves<MODE>();
  constexpr int RB = FW ? RW : NW * RW;  // rows per block
  // the operator x passes: the block's system (one code path for a launch
  // of one system and a batch); the other modes: the launch's arguments
  constexpr bool SYS = MODE == ROW_P || MODE == ROW_H;
  KSys* sy = SYS ? block_sys<RowArgs>() : nullptr;
  const int* gate = SYS ? sy->gate : a.gate;
  if (!SM && gate && *gate) return;
  auto IN = [&](int f) -> const void* {
    if constexpr (SYS) return sy->in[f];
    else return a.in[f];
  };
  auto OUT = [&](int f) -> void* {
    if constexpr (SYS) return sy->out[f];
    else return a.out[f];
  };
  const void* coefp = SYS ? sy->coef : a.coef;
  const double* iscale = SYS ? sy->in_scale : a.in_scale;
  const double rho0 = SYS ? sy->rho0 : a.rho0;
  __shared__ C2<R> lds_all[NW * RW * LP];
  // twiddle tables in LDS: a load in every butterfly pass from global memory
  // (even an L1 hit) costs latency inside the transform and address registers
  __shared__ C2<R> tw_lds[2 * L];
  // ROW_P: wavefront w handles field w of the block's rows, so the fields
  // share each coefficient row through the CU's L1 instead of re-reading it
  // from HBM, and each thread keeps only one field's transforms live.
  // readfirstlane tells the compiler the wave index is wave-uniform, so the
  // field's pointers stay in scalar registers.
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int lane = threadIdx.x % 64;
  const int fsel = FW ? wave : 0;
  const int t = lane % T;
  const int rr = (FW ? 0 : wave * RW) + lane / T;  // row within the block
  // The x passes sweep the rows last group first: the pass before them (a
  // y pass, ascending z) leaves its most recent output in the 256 MB
  // Infinity Cache, and the y pass after them (ascending z again) starts on
  // what this pass wrote last.  At 256^3 FP64 the three pressure fields
  // (384 MiB) exceed that cache; the reversed sweep takes the x pass from
  // 218 to 199 us and the following y pass from 130 to 114 us.
  const int ngroups = (a.nrows + RB - 1) / RB;
  int row = 0;
  bool ok = false;
  LdsRow<R> lds{lds_all + (FW ? fsel * RW + rr : rr) * LP};
  const R sx = R(a.g.sx);
  C2<R> reg[E];
  constexpr bool LOOP = !SM && row_loop<L, R, MODE>();
  auto place = [&](int grp) {
    const int bx = (MODE == ROW_P || MODE == ROW_H) ? ngroups - 1 - grp : grp;
    row = bx * RB + rr;
    ok = row < a.nrows;
  };

  // small fields: the block's row (spectral or real pairs, in natural order
  // t + s T) and the twiddles are on their way before the halt flag is read
  C2<R> first[SM ? E : 1];
  if constexpr (SM) {
    constexpr int NT = 64 * NW, NTW = (2 * L + 127) / 128;  // ROW_P may run two wavefronts
    static_assert(NT >= 128, "at least two wavefronts");
    place(blockIdx.x);
    const C2<R>* src = (const C2<R>*)IN(fsel);
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const int k = MODE == ROW_R2C ? pat_index<L, E, RF0>(t, s) : t + s * T;
      first[s] = ok ? ldg(src + (size_t)row * L + k) : C2<R>{R(0), R(0)};
    }
    C2<R> twr[NTW];
    const int nt = blockDim.x;
#pragma unroll
    for (int i = 0; i < NTW; ++i)
      if (i * nt + (int)threadIdx.x < 2 * L) twr[i] = ldg(twtab + L + i * nt + threadIdx.x);
    if (gate && *gate) return;
#pragma unroll
    for (int i = 0; i < NTW; ++i)
      if (i * nt + (int)threadIdx.x < 2 * L) tw_lds[i * nt + threadIdx.x] = twr[i];
  } else {
    for (int i = threadIdx.x; i < 2 * L; i += blockDim.x) tw_lds[i] = twtab[L + i];
  }
  __syncthreads();
  const C2<R>* tw = tw_lds;       // length-L table
  const C2<R>* twN = tw_lds + L;  // length-2L table, first L entries used

  auto pre_mult = [&](int f, int k, C2<R> X) -> C2<R> {
    if constexpr (MODE == ROW_P) {
      if (f == 0) return cik(X, R(k) * sx);  // slot 0: k'_x = 0 for both halves
      return X;
    } else if constexpr (MODE == ROW_P1) {
      R m = a.precond ? mult_press<R>(k, 0, 0, a.g, rho0) : R(1);
      return cik(X, R(k) * sx * m * in_scale_of<R>(iscale));
    } else if constexpr (MODE == ROW_H1) {
      R sc = in_scale_of<R>(iscale);
      if (!a.precond) return cscale(X, sc);
      HelmMult<R> h = mult_helm<R>(k, 0, 0, a.g, rho0, a.nu, false);
      if (k == 0) return C2<R>{X.x * h.g0 * sc, X.y * h.gN * sc};
      return cscale(X, h.g0 * sc);
    } else {
      return X;
    }
  };

  auto inverse_row = [&](const C2<R>* __restrict__ src, int f) {
    // stage the packed row, build Z_k = E_k + i O_k for the half-length FFT
    lds_sync<WV>();
#pragma unroll
    for (int s = 0; s < E; ++s) {
      int k = t + s * T;
      C2<R> X = SM ? first[SM ? s : 0] : ok ? ldg(src + (size_t)row * L + k) : C2<R>{R(0), R(0)};
      lds.st(k, pre_mult(f, k, X));
    }
    lds_sync<WV>();
    constexpr int RI0 = S::template first_radix<false>();
#pragma unroll
    for (int s = 0; s < E; ++s) {
      int k = pat_index<L, E, RI0>(t, s);
      C2<R> Z;
      if (k == 0) {
        C2<R> P0 = lds.ld(0);
        Z = C2<R>{P0.x + P0.y, P0.x - P0.y};
      } else {
        C2<R> Xk = lds.ld(k), Xm = cconj(lds.ld(L - k));
        C2<R> e = Xk + Xm;
        C2<R> o = cmulc(Xk - Xm, ldg(twN + k));  // times exp(+2 pi i k / N)
        Z = C2<R>{e.x - o.y, e.y + o.x};
      }
      reg[s] = Z;
    }
    fft_line<L, E, +1, false, WV>(reg, lds, tw, t);
  };

  auto forward_post = [&](int f, C2<R>* __restrict__ dst, const C2<R>* __restrict__ vsrc) {
    // reg holds Z_k for k = t + s T (forward output, radix E last)
    lds_sync<WV>();
#pragma unroll
    for (int s = 0; s < E; ++s) lds.st(t + s * T, reg[s]);
    lds_sync<WV>();
#pragma unroll
    for (int s = 0; s < E; ++s) {
      int k = t + s * T;
      C2<R> Zk = reg[s], X;
      if (k == 0) {
        X = C2<R>{Zk.x + Zk.y, Zk.x - Zk.y};
      } else {
        C2<R> Zm = cconj(lds.ld(L - k));
        C2<R> e = Zk + Zm;
        C2<R> wd = cmul(ldg(twN + k), Zk - Zm);
        X = C2<R>{R(0.5) * (e.x + wd.y), R(0.5) * (e.y - wd.x)};
      }
      if constexpr (MODE == ROW_P) {
        if (f == 0) X = cik(X, R(k) * sx);
      } else if constexpr (MODE == ROW_P1) {
        X = cik(X, -R(k) * sx);
      } else if constexpr (MODE == ROW_H1) {
        // + nu |k|^2 M v (slot 0: halves kx = 0 and kx = nx/2)
        C2<R> V = ok ? ldg(vsrc + (size_t)row * L + k) : C2<R>{R(0), R(0)};
        R sc = in_scale_of<R>(iscale);
        R k2 = R(k) * sx;
        k2 *= k2;
        R kn = R(a.g.M) * sx;
        if (a.precond) {
          HelmMult<R> h = mult_helm<R>(k, 0, 0, a.g, rho0, a.nu, true);
          if (k == 0) X = X + C2<R>{R(0), V.y * h.gN * sc};
          else X = X + cscale(V, h.g0 * sc);
        } else {
          if (k == 0) X = X + C2<R>{R(0), V.y * R(a.nu) * kn * kn * sc};
          else X = X + cscale(V, R(a.nu) * k2 * sc);
        }
      }
      if (ok) stg(dst + (size_t)row * L + k, X);
    }
  };

  // row groups: one per block, or a loop over them (row_loop)
  for (int grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
    place(grp);
    if constexpr (MODE == ROW_R2C) {
      const C2<R>* src = (const C2<R>*)IN(0);  // real row viewed as complex pairs
#pragma unroll
      for (int s = 0; s < E; ++s) {
        int m = pat_index<L, E, RF0>(t, s);
        reg[s] = SM ? first[SM ? s : 0] : ok ? ldg(src + (size_t)row * L + m) : C2<R>{R(0), R(0)};
      }
      fft_line<L, E, -1, true, WV>(reg, lds, tw, t);
      forward_post(0, (C2<R>*)OUT(0), nullptr);
    } else if constexpr (MODE == ROW_C2R) {
      inverse_row((const C2<R>*)IN(0), 0);
      const R cs = R(a.cscale);
      C2<R>* dst = (C2<R>*)OUT(0);
      if (ok) {
#pragma unroll
        for (int s = 0; s < E; ++s) {
          int m = pat_index<L, E, RI1>(t, s);
          stg(dst + (size_t)row * L + m, cscale(reg[s], cs));
        }
      }
    } else {
      const C2<R>* coef = (const C2<R>*)coefp;
      const R cs = R(a.cscale);
      const int f = fsel;
      // pressure x pass: issue the coefficient row's loads before the inverse
      // transform so that their latency hides behind it (measured: 215 -> 204
      // us at 256^3 FP64; the single-field Helmholtz pass is faster without)
      constexpr bool PREFETCH = MODE == ROW_P || SM;
      C2<R> qv[PREFETCH ? E : 1];
      if constexpr (PREFETCH) {
#pragma unroll
        for (int s = 0; s < E; ++s) {
          int m = pat_index<L, E, RI1>(t, s);
          qv[s] = ok ? ldg(coef + (size_t)row * L + m) : C2<R>{R(0), R(0)};
        }
      }
      inverse_row((const C2<R>*)IN(f), f);
#pragma unroll
      for (int s = 0; s < E; ++s) {
        C2<R> q;
        if constexpr (PREFETCH) {
          q = qv[s];
        } else {
          int m = pat_index<L, E, RI1>(t, s);
          q = ok ? ldg(coef + (size_t)row * L + m) : C2<R>{R(0), R(0)};
        }
        reg[s] = C2<R>{reg[s].x * (q.x * cs), reg[s].y * (q.y * cs)};
      }
      fft_line<L, E, -1, true, WV>(reg, lds, tw, t);
      forward_post(f, (C2<R>*)OUT(f), (const C2<R>*)IN(0));
    }
    if constexpr (!LOOP) break;  // no back edge: nothing is hoisted
  }
}

// -------------------------------------------------- precond kernel

template <typename R>
__global__ __launch_bounds__(256) void k_precond(const C2<R>* __restrict__ r, C2<R>* __restrict__ z, Geom g,
                                                 int kind, double rho0, double nu, size_t n) {
  size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const unsigned ue = (unsigned)e, q = ue / (unsigned)g.M;  // at most 2^29 slots
  const int kx = (int)(ue - q * (unsigned)g.M);
  const int ky = (int)(q % (unsigned)g.ny), kz = (int)(q / (unsigned)g.ny);
  C2<R> v = ldg(r + e);
  if (kind == OP_PRESSURE) {
    stg(z + e, cscale(v, mult_press<R>(kx, ky, kz, g, rho0)));
  } else {
    HelmMult<R> h = mult_helm<R>(kx, ky, kz, g, rho0, nu, false);
    if (kx == 0) {
      int kym = (g.ny - ky) % g.ny, kzm = (g.nz - kz) % g.nz;
      C2<R> pm = ldg(r + ((size_t)kzm * g.ny + kym) * g.M);
      stg(z + e, diag_packed(v, pm, h.g0, h.gN));
    } else {
      stg(z + e, cscale(v, h.g0));
    }
  }
}

// ------------------------------------------------- spectral Laplacian

// y = Lap x on a packed spectrum (symbol -|k|^2, Nyquist kept; the kx = 0
// slot mixes with its mirror because its two halves differ).  Out of place.
__global__ __launch_bounds__(256) void k_lap_packed(const C2<double>* __restrict__ x, C2<double>* __restrict__ y,
                                                    Geom g, size_t n) {
  size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const unsigned ue = (unsigned)e, q = ue / (unsigned)g.M;  // at most 2^29 slots
  const int kx = (int)(ue - q * (unsigned)g.M);
  const int ky = (int)(q % (unsigned)g.ny), kz = (int)(q / (unsigned)g.ny);
  const double kyz = ksq_yz<double>(ky, kz, g);
  const double kxp = (double)kx * g.sx, kn = (double)g.M * g.sx;
  const C2<double> v = ldg(x + e);
  if (kx == 0) {
    const int kym = (g.ny - ky) % g.ny, kzm = (g.nz - kz) % g.nz;
    const C2<double> pm = ldg(x + ((size_t)kzm * g.ny + kym) * g.M);
    stg(y + e, diag_packed(v, pm, -kyz, -(kyz + kn * kn)));
  } else {
    stg(y + e, cscale(v, -(kyz + kxp * kxp)));
  }
}

void lap_packed(const Geom& g, const void* x, void* y, hipStream_t st) {
  const size_t n = (size_t)g.nz * g.ny * g.M;
  hipLaunchKernelGGL(k_lap_packed, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const C2<double>*)x,
                     (C2<double>*)y, g, n);
}

// ------------------------------------------------------------ launchers

// A launch of one system carries it as sys[0] (the kernels read every
// system's arguments from sys[blockIdx.y]).
template <typename Args>
static void as_systems(Args& a) {
  if (a.nb > 0) return;
  a.nb = 1;
  SysArgs& y = a.sys[0];
  for (int i = 0; i < 3; ++i) {
    y.in[i] = a.in[i];
    y.out[i] = a.out[i];
  }
  y.rho0 = a.rho0;
  y.in_scale = a.in_scale;
  y.gate = a.gate;
}

static bool small_field(const Geom& g) { return (size_t)g.nz * g.ny * g.M <= kSmallField; }

template <typename R, int MODE, int L, bool SM>
static void launch_col_S(const ColArgs& a0, const void* tw, hipStream_t st) {
  using Cf = ColCfg<L, R, MODE, SM>;
  ColArgs a = a0;
  as_systems(a);
  a.ntile = (a.inner + Cf::TC - 1) / Cf::TC;
  dim3 grid(a.outer * a.ntile, a.nb);
  hipLaunchKernelGGL((k_col<L, R, MODE, SM>), grid, dim3(Cf::NT), 0, st, a, (const C2<R>*)tw);
}
template <typename R, int MODE, int L>
static void launch_col_L(const ColArgs& a, const void* tw, hipStream_t st) {
  if constexpr (col_has_small(L, MODE)) {
    if (small_field(a.g)) {
      launch_col_S<R, MODE, L, true>(a, tw, st);
      return;
    }
  }
  launch_col_S<R, MODE, L, false>(a, tw, st);
}

// Lengths whose first and last pass carry Gram-Schmidt work (a 1024-point tile
// already fills a block's registers).
constexpr int kGsLength = 512;
bool op_carries_gs(const Geom& g) {
  return small_field(g) && !g.cheb && g.nz > 1 && g.nz <= kGsLength;
}
// the Helmholtz passes read mirror elements of their input, which another block's second pass may be writing
bool op_carries_check(const Geom& g, int kind) { return kind == OP_PRESSURE && op_carries_gs(g); }

template <typename F>
static void for_gs_length(int L, F&& f) {
  switch (L) {
    case 16: f(std::integral_constant<int, 16>{}); break;
    case 32: f(std::integral_constant<int, 32>{}); break;
    case 64: f(std::integral_constant<int, 64>{}); break;
    case 128: f(std::integral_constant<int, 128>{}); break;
    case 256: f(std::integral_constant<int, 256>{}); break;
    case 512: f(std::integral_constant<int, 512>{}); break;
    default: fprintf(stderr, "vdsolve: unsupported column length %d\n", L);
  }
}
int op_dot_blocks(const Geom& g) {
  int n = 0;
  for_gs_length(g.nz, [&](auto len) {
    constexpr int TC = ColSmall<decltype(len)::value>::TC;
    n = (g.ny * g.M + TC - 1) / TC;
  });
  return n;
}

// A first (CHECK) or last pass with the Gram-Schmidt work of c.
template <typename R, int MODE>
static void launch_col_gs(int len, const ColArgs& a0, const GsCarry& c, const void* tw, hipStream_t st) {
  constexpr bool CHECK = MODE == COL_P_FIRST;
  ColArgs a = a0;
  as_systems(a);
  ColGs gs{};
  gs.nv = CHECK ? c.nv - 1 : c.nv;
  gs.nb = c.check_blocks;
  gs.tol = orth_tol<R>();
  gs.scale = a.g.ntot_inv;
  for (int k = 0; k < a.nb; ++k) {
    gs.sys[k].st = c.st[k];
    gs.sys[k].partial = c.partial[k];
    for (int i = 0; i < gs.nv; ++i) gs.sys[k].V[i] = c.V[k].p[i];
  }
  for_gs_length(len, [&](auto l) {
    constexpr int L = decltype(l)::value;
    using Cf = ColCfg<L, R, MODE, true, true>;
    a.ntile = (a.inner + Cf::TC - 1) / Cf::TC;
    hipLaunchKernelGGL((k_col_gs<L, R, MODE>), dim3(a.ntile + (CHECK ? 1 : 0), a.nb), dim3(Cf::NT), 0, st, a,
                       (const C2<R>*)tw, gs);
  });
}

bool op_carries_rec(const Geom& g) { return !g.cheb && g.nz > 1 && g.nz <= kGsLength; }
template <typename R>
int op_rec_blocks(const Geom& g, int kind) {
  int n = 0;
  for_gs_length(g.nz, [&](auto len) {
    constexpr int L = decltype(len)::value;
    const int tc = small_field(g) ? ColSmall<L>::TC
                   : kind == OP_PRESSURE ? ColCfg<L, R, COL_P_LAST>::TC : ColCfg<L, R, COL_H_LAST>::TC;
    n = (g.ny * g.M + tc - 1) / tc;
  });
  return n <= kRedBlocks ? n : 0;
}
template int op_rec_blocks<double>(const Geom&, int);
template int op_rec_blocks<float>(const Geom&, int);

// A first or last pass with the CG or RMR work of c.
template <typename R, int MODE>
static void launch_col_rec(int len, const ColArgs& a0, const RecCarry& c, const void* tw, hipStream_t st) {
  constexpr bool FIRST = MODE == COL_P_FIRST || MODE == COL_H_FIRST;
  ColArgs a = a0;
  as_systems(a);
  const ColRec rec{c.cg ? 1 : 0, c.precond ? 1 : 0, c.nb, c.slot, a.g.ntot_inv, c.st, c.partial, c.r, c.p};
  for_gs_length(len, [&](auto l) {
    constexpr int L = decltype(l)::value;
    auto go = [&](auto sm) {
      constexpr bool SM = decltype(sm)::value;
      using Cf = ColCfg<L, R, MODE, SM>;
      a.ntile = (a.inner + Cf::TC - 1) / Cf::TC;
      hipLaunchKernelGGL((k_col_rec<L, R, MODE, SM>), dim3(a.ntile + (FIRST ? 1 : 0), a.nb), dim3(Cf::NT), 0, st, a,
                         (const C2<R>*)tw, rec);
    };
    if (small_field(a.g)) go(std::true_type{});
    else go(std::false_type{});
  });
}

template <typename R, int MODE>
static void launch_col(int L, const ColArgs& a, const void* tw, hipStream_t st) {
  switch (L) {
    case 16: launch_col_L<R, MODE, 16>(a, tw, st); break;
    case 32: launch_col_L<R, MODE, 32>(a, tw, st); break;
    case 64: launch_col_L<R, MODE, 64>(a, tw, st); break;
    case 128: launch_col_L<R, MODE, 128>(a, tw, st); break;
    case 256: launch_col_L<R, MODE, 256>(a, tw, st); break;
    case 512: launch_col_L<R, MODE, 512>(a, tw, st); break;
    case 1024: launch_col_L<R, MODE, 1024>(a, tw, st); break;
    default: fprintf(stderr, "vdsolve: unsupported column length %d\n", L);
  }
}

template <typename R, int MODE>
static void first_pass(const Geom& g, const OpParams& p, const ColArgs& a, const void* tw, hipStream_t st) {
  if constexpr (MODE == COL_P_FIRST) {
    if (p.gs && p.gs->check) {
      launch_col_gs<R, MODE>(g.nz, a, *p.gs, tw, st);
      return;
    }
  }
  if (p.rec && p.rec->ends) launch_col_rec<R, MODE>(g.nz, a, *p.rec, tw, st);
  else launch_col<R, MODE>(g.nz, a, tw, st);
}
template <typename R, int MODE>
static void last_pass(const Geom& g, const OpParams& p, const ColArgs& a, const void* tw, hipStream_t st) {
  if (p.gs) launch_col_gs<R, MODE>(g.nz, a, *p.gs, tw, st);
  else if (p.rec && p.rec->dots) launch_col_rec<R, MODE>(g.nz, a, *p.rec, tw, st);
  else launch_col<R, MODE>(g.nz, a, tw, st);
}

// Blocks of a looping row pass (eight per CU on 256 CUs), per system.
constexpr int kRowGridCap = 2048;

template <typename R, int MODE, int L, bool SM>
static void launch_row_S(const RowArgs& a0, const void* tw, hipStream_t st) {
  constexpr int RW = RowCfg<L, R, SM>::RW;
  RowArgs a = a0;
  int ny = 1;
  if constexpr (MODE == ROW_P || MODE == ROW_H) {
    if (a.nb == 0) a.sys[0].coef = a.coef;
    as_systems(a);
    ny = a.nb;
  }
  const int rb = row_field_waves<MODE>() ? RW : row_waves<MODE>() * RW;
  const int ngroups = (a.nrows + rb - 1) / rb;
  dim3 grid(!SM && row_loop<L, R, MODE>() && ngroups > kRowGridCap ? kRowGridCap : ngroups, ny);
  // ROW_P: one wavefront per field (<= 3)
  const int waves = row_field_waves<MODE>() ? a.nf : row_waves<MODE>();
  hipLaunchKernelGGL((k_row<L, R, MODE, SM>), grid, dim3(64 * waves), 0, st, a, (const C2<R>*)tw);
}
template <typename R, int MODE, int L>
static void launch_row_L(const RowArgs& a, const void* tw, hipStream_t st) {
  if constexpr (MODE != ROW_P1 && MODE != ROW_H1 && L >= 16) {
    if (small_field(a.g)) {
      launch_row_S<R, MODE, L, true>(a, tw, st);
      return;
    }
  }
  launch_row_S<R, MODE, L, false>(a, tw, st);
}

template <typename R, int MODE>
static void launch_row(int L, const RowArgs& a, const void* tw, hipStream_t st) {
  switch (L) {
    case 8: launch_row_L<R, MODE, 8>(a, tw, st); break;
    case 16: launch_row_L<R, MODE, 16>(a, tw, st); break;
    case 32: launch_row_L<R, MODE, 32>(a, tw, st); break;
    case 64: launch_row_L<R, MODE, 64>(a, tw, st); break;
    case 128: launch_row_L<R, MODE, 128>(a, tw, st); break;
    case 256: launch_row_L<R, MODE, 256>(a, tw, st); break;
    case 512: launch_row_L<R, MODE, 512>(a, tw, st); break;
    default: fprintf(stderr, "vdsolve: unsupported row length %d\n", L);
  }
}

static ColArgs col_args(const Geom& g, const OpParams* p) {
  ColArgs a{};
  a.g = g;
  if (p) {
    a.rho0 = p->rho0;
    a.nu = p->nu;
    a.precond = p->precond;
    a.in_scale = p->in_scale;
    a.gate = p->gate;
  }
  return a;
}
// a plain transform pass of an operator application: no operator
// parameters, but the application's gate
static ColArgs col_args_fft(const Geom& g, const OpParams& p) {
  ColArgs a = col_args(g, nullptr);
  a.gate = p.gate;
  return a;
}
static RowArgs row_args(const Geom& g, const OpParams* p) {
  RowArgs a{};
  a.g = g;
  a.nrows = g.ny * g.nz;
  if (p) {
    a.rho0 = p->rho0;
    a.nu = p->nu;
    a.precond = p->precond;
    a.in_scale = p->in_scale;
    a.gate = p->gate;
  }
  return a;
}

// Fields each pass reads plus writes (3D): pressure P1..P5, Helmholtz P1..P5.
constexpr double kPassFields[10] = {3, 5, 7, 5, 3, 2, 2, 3, 2, 3};
// and those that a first or last pass adds for the Krylov step that it carries
// (the second pass of Gram-Schmidt, which few steps take, left out)
static double first_carry_fields(const OpParams& p) { return p.rec && p.rec->ends && p.rec->cg ? 2 : 0; }
static double last_carry_fields(const OpParams& p) {
  return p.gs ? p.gs->nv : p.rec && p.rec->dots ? 1 : 0;
}

template <typename R>
void op_apply(const Geom& g, const OpParams& p, const void* v, void* y, const OpWork& w, const void* coef,
              const void* twtab, hipStream_t st, Prof* prof) {
  const bool pr = prof && prof->on;
  const double fb = (double)g.nz * g.ny * g.M * sizeof(C2<R>);  // one field
#define VD_TC(c, carry) \
  if (pr) prof->begin(c, st, (kPassFields[c] + (carry)) * fb);
#define VD_T0(c) VD_TC(c, 0)
#define VD_T1() \
  if (pr) prof->end(st);
  const size_t zin = (size_t)g.ny * g.M;  // inner size of the z pass
  if (p.kind == OP_PRESSURE) {
    if (g.nz == 1) {  // 1D
      RowArgs r = row_args(g, &p);
      r.in[0] = v;
      r.out[0] = y;
      r.coef = coef;
      r.cscale = g.ntot_inv;
      VD_T0(2) launch_row<R, ROW_P1>(g.M, r, twtab, st); VD_T1()
      return;
    }
    void *t0 = w.t[0], *t1 = w.t[1], *t2 = w.t[2];
    ColArgs a = col_args(g, &p);
    a.outer = 1;
    a.inner = (int)zin;
    a.in[0] = v;
    a.out[0] = t0;
    a.out[1] = t1;
    VD_TC(0, first_carry_fields(p)) first_pass<R, COL_P_FIRST>(g, p, a, twtab, st); VD_T1()
    RowArgs r = row_args(g, &p);
    r.coef = coef;
    r.cscale = g.ntot_inv;
    if (g.ny > 1) {
      ColArgs b = col_args(g, &p);
      b.outer = g.nz;
      b.inner = g.M;
      b.in[0] = t0;
      b.in[1] = t1;
      b.out[0] = t0;
      b.out[1] = t2;
      b.out[2] = t1;
      VD_T0(1) launch_col<R, COL_P_MIDINV>(g.ny, b, twtab, st); VD_T1()
      r.nf = 3;
      r.in[0] = t0; r.in[1] = t2; r.in[2] = t1;
      r.out[0] = t0; r.out[1] = t2; r.out[2] = t1;
      VD_T0(2) launch_row<R, ROW_P>(g.M, r, twtab, st); VD_T1()
      ColArgs c = col_args(g, &p);
      c.outer = g.nz;
      c.inner = g.M;
      c.in[0] = t0; c.in[1] = t2; c.in[2] = t1;
      c.out[0] = t0; c.out[1] = t1;
      VD_T0(3) launch_col<R, COL_P_MIDFWD>(g.ny, c, twtab, st); VD_T1()
    } else {
      r.nf = 2;
      r.in[0] = t0; r.in[1] = t1;
      r.out[0] = t0; r.out[1] = t1;
      VD_T0(2) launch_row<R, ROW_P>(g.M, r, twtab, st); VD_T1()
    }
    ColArgs d = col_args(g, &p);
    d.outer = 1;
    d.inner = (int)zin;
    d.in[0] = t0;
    d.in[1] = t1;
    d.out[0] = y;
    VD_TC(4, last_carry_fields(p)) last_pass<R, COL_P_LAST>(g, p, d, twtab, st); VD_T1()
  } else {
    if (g.nz == 1) {
      RowArgs r = row_args(g, &p);
      r.in[0] = v;
      r.out[0] = y;
      r.coef = coef;
      r.cscale = g.ntot_inv;
      VD_T0(7) launch_row<R, ROW_H1>(g.M, r, twtab, st); VD_T1()
      return;
    }
    void* t0 = w.t[0];
    ColArgs a = col_args(g, &p);
    a.outer = 1;
    a.inner = (int)zin;
    a.in[0] = v;
    a.out[0] = t0;
    VD_TC(5, first_carry_fields(p)) first_pass<R, COL_H_FIRST>(g, p, a, twtab, st); VD_T1()
    if (g.ny > 1) {
      ColArgs b = col_args_fft(g, p);
      b.outer = g.nz;
      b.inner = g.M;
      b.nf = 1;
      b.in[0] = t0;
      b.out[0] = t0;
      VD_T0(6) launch_col<R, COL_FFT_INV>(g.ny, b, twtab, st); VD_T1()
    }
    RowArgs r = row_args(g, &p);
    r.in[0] = t0;
    r.out[0] = t0;
    r.coef = coef;
    r.cscale = g.ntot_inv;
    VD_T0(7) launch_row<R, ROW_H>(g.M, r, twtab, st); VD_T1()
    if (g.ny > 1) {
      ColArgs b = col_args_fft(g, p);
      b.outer = g.nz;
      b.inner = g.M;
      b.nf = 1;
      b.in[0] = t0;
      b.out[0] = t0;
      VD_T0(8) launch_col<R, COL_FFT_FWD>(g.ny, b, twtab, st); VD_T1()
    }
    ColArgs d = col_args(g, &p);
    d.outer = 1;
    d.inner = (int)zin;
    d.in[0] = t0;
    d.in[1] = v;
    d.out[0] = y;
    VD_TC(9, last_carry_fields(p)) last_pass<R, COL_H_LAST>(g, p, d, twtab, st); VD_T1()
  }
#undef VD_T0
#undef VD_TC
#undef VD_T1
}

template <typename R>
void op_apply_batch(const Geom& g, const OpParams& p, const OpBatch& b, const void* coef, const void* twtab,
                    hipStream_t st, Prof* prof) {
  const int nb = b.nb;
  const bool pr = prof && prof->on;
  const double fb = (double)g.nz * g.ny * g.M * sizeof(C2<R>);  // one field
  const size_t zin = (size_t)g.ny * g.M;
  const bool helm = p.kind == OP_HELMHOLTZ;
  // system k's fields in[]/out[] of a launch, with its own scale (first
  // pass only), preconditioner constant, coefficient rows and gate
  auto sys_of = [&](int k, std::initializer_list<const void*> in, std::initializer_list<void*> out, bool scaled) {
    SysArgs y{};
    int i = 0;
    for (const void* q : in) y.in[i++] = q;
    i = 0;
    for (void* q : out) y.out[i++] = q;
    y.coef = b.coef[k] ? b.coef[k] : coef;
    y.rho0 = helm ? p.rho0 : b.rho0[k];
    y.in_scale = scaled ? b.in_scale[k] : nullptr;
    y.gate = b.gate[k];
    return y;
  };
  auto col = [&](bool fft) {
    ColArgs a = fft ? col_args_fft(g, p) : col_args(g, &p);
    a.gate = nullptr;
    a.in_scale = nullptr;
    a.nb = nb;
    return a;
  };
  auto timed = [&](int cls, double fields, auto&& launch) {
    if (pr) prof->begin(cls, st, fields * fb);
    launch();
    if (pr) prof->end(st);
  };
  if (helm) {
    // one work field per system
    ColArgs a = col(false);
    a.outer = 1;
    a.inner = (int)zin;
    for (int k = 0; k < nb; ++k) a.sys[k] = sys_of(k, {b.v[k]}, {b.t[k][0]}, true);
    timed(5, 2.0 * nb, [&] { first_pass<R, COL_H_FIRST>(g, p, a, twtab, st); });
    ColArgs c = col(true);
    c.outer = g.nz;
    c.inner = g.M;
    c.nf = 1;
    for (int k = 0; k < nb; ++k) c.sys[k] = sys_of(k, {b.t[k][0]}, {b.t[k][0]}, false);
    if (g.ny > 1) timed(6, 2.0 * nb, [&] { launch_col<R, COL_FFT_INV>(g.ny, c, twtab, st); });
    RowArgs r = row_args(g, &p);
    r.gate = nullptr;
    r.in_scale = nullptr;
    r.coef = nullptr;
    r.cscale = g.ntot_inv;
    r.nb = nb;
    for (int k = 0; k < nb; ++k) r.sys[k] = sys_of(k, {b.t[k][0]}, {b.t[k][0]}, false);
    timed(7, 3.0 * nb, [&] { launch_row<R, ROW_H>(g.M, r, twtab, st); });
    if (g.ny > 1) timed(8, 2.0 * nb, [&] { launch_col<R, COL_FFT_FWD>(g.ny, c, twtab, st); });
    ColArgs d = col(false);
    d.outer = 1;
    d.inner = (int)zin;
    for (int k = 0; k < nb; ++k) d.sys[k] = sys_of(k, {b.t[k][0], b.v[k]}, {b.y[k]}, true);
    timed(9, (3.0 + last_carry_fields(p)) * nb, [&] { last_pass<R, COL_H_LAST>(g, p, d, twtab, st); });
    return;
  }
  // pressure (2D and 3D grids): the passes of op_apply, system k on
  // blockIdx.y with its own coefficient rows and preconditioner constant
  ColArgs a = col(false);
  a.outer = 1;
  a.inner = (int)zin;
  for (int k = 0; k < nb; ++k) a.sys[k] = sys_of(k, {b.v[k]}, {b.t[k][0], b.t[k][1]}, true);
  timed(0, 3.0 * nb, [&] { first_pass<R, COL_P_FIRST>(g, p, a, twtab, st); });
  RowArgs r = row_args(g, &p);
  r.gate = nullptr;
  r.in_scale = nullptr;
  r.coef = nullptr;
  r.cscale = g.ntot_inv;
  r.nb = nb;
  if (g.ny > 1) {
    ColArgs c = col(false);
    c.outer = g.nz;
    c.inner = g.M;
    for (int k = 0; k < nb; ++k)
      c.sys[k] = sys_of(k, {b.t[k][0], b.t[k][1]}, {b.t[k][0], b.t[k][2], b.t[k][1]}, false);
    timed(1, 5.0 * nb, [&] { launch_col<R, COL_P_MIDINV>(g.ny, c, twtab, st); });
    r.nf = 3;
    for (int k = 0; k < nb; ++k)
      r.sys[k] = sys_of(k, {b.t[k][0], b.t[k][2], b.t[k][1]}, {b.t[k][0], b.t[k][2], b.t[k][1]}, false);
    timed(2, 7.0 * nb, [&] { launch_row<R, ROW_P>(g.M, r, twtab, st); });
    ColArgs c2 = col(false);
    c2.outer = g.nz;
    c2.inner = g.M;
    for (int k = 0; k < nb; ++k)
      c2.sys[k] = sys_of(k, {b.t[k][0], b.t[k][2], b.t[k][1]}, {b.t[k][0], b.t[k][1]}, false);
    timed(3, 5.0 * nb, [&] { launch_col<R, COL_P_MIDFWD>(g.ny, c2, twtab, st); });
  } else {
    r.nf = 2;
    for (int k = 0; k < nb; ++k) r.sys[k] = sys_of(k, {b.t[k][0], b.t[k][1]}, {b.t[k][0], b.t[k][1]}, false);
    timed(2, 5.0 * nb, [&] { launch_row<R, ROW_P>(g.M, r, twtab, st); });
  }
  ColArgs d = col(false);
  d.outer = 1;
  d.inner = (int)zin;
  for (int k = 0; k < nb; ++k) d.sys[k] = sys_of(k, {b.t[k][0], b.t[k][1]}, {b.y[k]}, false);
  timed(4, (3.0 + last_carry_fields(p)) * nb, [&] { last_pass<R, COL_P_LAST>(g, p, d, twtab, st); });
}

template <typename R>
void precond_apply(const Geom& g, const OpParams& p, const void* r, void* z, hipStream_t st) {
  size_t n = (size_t)g.nz * g.ny * g.M;
  hipLaunchKernelGGL((k_precond<R>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const C2<R>*)r,
                     (C2<R>*)z, g, p.kind, p.rho0, p.nu, n);
}

void fwd_transform(const Geom& g, const double* phys, void* spec, void* work, const void* twtab,
                   hipStream_t st) {
  (void)work;
  RowArgs r = row_args(g, nullptr);
  r.in[0] = phys;
  r.out[0] = spec;
  launch_row<double, ROW_R2C>(g.M, r, twtab, st);
  if (g.cheb) return;  // z is physical (Chebyshev nodes): x transform only
  if (g.ny > 1) {
    ColArgs b = col_args(g, nullptr);
    b.outer = g.nz;
    b.inner = g.M;
    b.nf = 1;
    b.in[0] = spec;
    b.out[0] = spec;
    launch_col<double, COL_FFT_FWD>(g.ny, b, twtab, st);
  }
  if (g.nz > 1) {
    ColArgs b = col_args(g, nullptr);
    b.outer = 1;
    b.inner = g.ny * g.M;
    b.nf = 1;
    b.in[0] = spec;
    b.out[0] = spec;
    launch_col<double, COL_FFT_FWD>(g.nz, b, twtab, st);
  }
}

void inv_transform(const Geom& g, const void* spec, double* phys, void* work, const void* twtab,
                   hipStream_t st) {
  const void* cur = spec;
  if (g.nz > 1 && !g.cheb) {
    ColArgs b = col_args(g, nullptr);
    b.outer = 1;
    b.inner = g.ny * g.M;
    b.nf = 1;
    b.in[0] = cur;
    b.out[0] = work;
    launch_col<double, COL_FFT_INV>(g.nz, b, twtab, st);
    cur = work;
  }
  if (g.ny > 1) {
    ColArgs b = col_args(g, nullptr);
    b.outer = g.nz;
    b.inner = g.M;
    b.nf = 1;
    b.in[0] = cur;
    b.out[0] = work;
    launch_col<double, COL_FFT_INV>(g.ny, b, twtab, st);
    cur = work;
  }
  RowArgs r = row_args(g, nullptr);
  r.in[0] = cur;
  r.out[0] = phys;
  r.cscale = g.ntot_inv;
  launch_row<double, ROW_C2R>(g.M, r, twtab, st);
}

void fwd_columns_n(const Geom& g, void* const* spec, int nf, const void* twtab, hipStream_t st, const int* gate) {
  ColArgs b = col_args(g, nullptr);
  b.gate = gate;
  b.nf = nf;
  for (int f = 0; f < nf; ++f) b.in[f] = b.out[f] = spec[f];
  if (g.ny > 1) {
    b.outer = g.nz;
    b.inner = g.M;
    launch_col<double, COL_FFT_FWD>(g.ny, b, twtab, st);
  }
  if (g.nz > 1) {
    b.outer = 1;
    b.inner = g.ny * g.M;
    launch_col<double, COL_FFT_FWD>(g.nz, b, twtab, st);
  }
}

void grad_rows(const Geom& g, const void* v, void* q0, void* qy, void* qz, const void* twtab, hipStream_t st) {
  ColArgs a = col_args(g, nullptr);
  a.outer = 1;
  a.inner = g.ny * g.M;
  a.in[0] = v;
  a.out[0] = q0;
  a.out[1] = qz;
  launch_col<double, COL_P_FIRST>(g.nz, a, twtab, st);
  ColArgs b = col_args(g, nullptr);
  b.outer = g.nz;
  b.inner = g.M;
  b.in[0] = q0;
  b.in[1] = qz;
  b.out[0] = q0;
  b.out[1] = qy;
  b.out[2] = qz;
  launch_col<double, COL_P_MIDINV>(g.ny, b, twtab, st);
}

// nf <= 3 fields at once: the column passes take every field in one launch
// (each block transforms its column of each field in turn), the x pass runs
// per field.  work[f] are distinct spectral buffers (the inverse's scratch).
void fwd_transform_n(const Geom& g, const double* const* phys, void* const* spec, int nf, const void* twtab,
                     hipStream_t st) {
  for (int f = 0; f < nf; ++f) {
    RowArgs r = row_args(g, nullptr);
    r.in[0] = phys[f];
    r.out[0] = spec[f];
    launch_row<double, ROW_R2C>(g.M, r, twtab, st);
  }
  if (!g.cheb) fwd_columns_n(g, spec, nf, twtab, st);
}

void inv_transform_n(const Geom& g, const void* const* spec, double* const* phys, void* const* work, int nf,
                     const void* twtab, hipStream_t st) {
  const void* cur[3] = {spec[0], nf > 1 ? spec[1] : nullptr, nf > 2 ? spec[2] : nullptr};
  if (g.nz > 1 && !g.cheb) {
    ColArgs b = col_args(g, nullptr);
    b.outer = 1;
    b.inner = g.ny * g.M;
    b.nf = nf;
    for (int f = 0; f < nf; ++f) {
      b.in[f] = cur[f];
      b.out[f] = work[f];
      cur[f] = work[f];
    }
    launch_col<double, COL_FFT_INV>(g.nz, b, twtab, st);
  }
  if (g.ny > 1) {
    ColArgs b = col_args(g, nullptr);
    b.outer = g.nz;
    b.inner = g.M;
    b.nf = nf;
    for (int f = 0; f < nf; ++f) {
      b.in[f] = cur[f];
      b.out[f] = work[f];
      cur[f] = work[f];
    }
    launch_col<double, COL_FFT_INV>(g.ny, b, twtab, st);
  }
  for (int f = 0; f < nf; ++f) {
    RowArgs r = row_args(g, nullptr);
    r.in[0] = cur[f];
    r.out[0] = phys[f];
    r.cscale = g.ntot_inv;
    launch_row<double, ROW_C2R>(g.M, r, twtab, st);
  }
}

template <typename R>
void row_pass_p2(const Geom& g, void* f0, void* f1, const void* coef, const void* twtab, hipStream_t st, Prof* prof,
                 const int* gate) {
  RowArgs r = row_args(g, nullptr);
  r.gate = gate;
  r.nf = 2;
  r.in[0] = f0;
  r.in[1] = f1;
  r.out[0] = f0;
  r.out[1] = f1;
  r.coef = coef;
  r.cscale = g.ntot_inv;
  const bool pr = prof && prof->on;
  if (pr) prof->begin(2, st, 5.0 * g.nz * g.ny * g.M * sizeof(C2<R>));
  launch_row<R, ROW_P>(g.M, r, twtab, st);
  if (pr) prof->end(st);
}
template void row_pass_p2<double>(const Geom&, void*, void*, const void*, const void*, hipStream_t, Prof*,
                                  const int*);
template void row_pass_p2<float>(const Geom&, void*, void*, const void*, const void*, hipStream_t, Prof*,
                                 const int*);

template void op_apply<double>(const Geom&, const OpParams&, const void*, void*, const OpWork&, const void*,
                               const void*, hipStream_t, Prof*);
template void op_apply<float>(const Geom&, const OpParams&, const void*, void*, const OpWork&, const void*,
                              const void*, hipStream_t, Prof*);
template void op_apply_batch<double>(const Geom&, const OpParams&, const OpBatch&, const void*, const void*,
                                     hipStream_t, Prof*);
template void op_apply_batch<float>(const Geom&, const OpParams&, const OpBatch&, const void*, const void*,
                                    hipStream_t, Prof*);
template void precond_apply<double>(const Geom&, const OpParams&, const void*, void*, hipStream_t);
template void precond_apply<float>(const Geom&, const OpParams&, const void*, void*, hipStream_t);

}  // namespace vd

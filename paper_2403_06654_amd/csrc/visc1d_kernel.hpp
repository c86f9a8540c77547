// Batched one-dimensional implicit viscous solver (gfx950): the kernel.
//
// Sec. 3.1, eq. VDINSE.Vrho: V_rho u = u - (a / rho)(D2 u + rho'' u + rho' D1 u)
// = b, right-preconditioned by V^-1 = (I - a D2)^-1 (eq. VDINSE.V), solved by
// GMRES(m) (classical Gram-Schmidt with a measured check, and a second pass where
// it fails), CG or the Richardson minimal-residual iteration.
//
// Every system of a batch shares the differentiation matrices and V^-1, so a
// matrix-vector product over a group of 16 systems is a dense product
// (unknowns x unknowns) x (unknowns x 16): one workgroup runs a group in
// lockstep and forms those products with v_mfma_f64_16x16x4_f64, each of its
// NW wavefronts owning TPW row tiles.  The 16 columns are independent
// through every step (products, per-system reductions in a fixed order,
// per-system scalars), so a system gives the same bits alone or in any batch;
// a system that has converged, failed or was never present keeps computing
// masked columns until its whole group is done.  Vectors live in registers in
// the accumulator layout; the right-hand operand of a product goes through
// one LDS buffer; the Krylov basis, the Hessenberg matrices and the density
// coefficients sit in a per-group workspace, each element read back only by
// the lane that wrote it.
//
// Unknowns: all n points (Fourier) or the n - 2 interior points (Chebyshev,
// u(+-1) = 0); rho' = D1 rho and rho'' = D2 rho use every point.
//
// The same kernel runs the pressure operators of the one-dimensional
// Chebyshev-collocation study of Sec. 3.2 (template parameter OP): on the
// interior values, with the wall values eliminated by the Neumann condition
// (D1 P, D2 P: the extension P folded into the matrices),
//   L_rho z = (1/rho) D2 P z - (rho'/rho^2) D1 P z      (eq. VDINSE.Lrho)
//   K_rho z = D2 P z + c z,  c = -D2 P psi / psi, psi = rho^-1/2
//                                                      (eq. VDINSE.Krho)
// preconditioned by the pseudo-inverse of D2 P; solutions and preconditioned
// vectors get their wall values from the same extension.
//
// What bounds it: the products.  Three n x n x 16 products an iteration are
// n^2 / 3200 us of FP64 MFMA on one CU (20.5 us at 256 rows, 46 at 384), and a
// workgroup has to overlap the stream of the matrices from L2, the barriers and
// the pointwise work with them.  Microseconds per RMR iteration, one group alone
// on a CU, at 128 / 255 / 384 / 512 unknowns: 9.1 / 28.8 / 56.8 / 100.5 (10.2 /
// 31.8 / 82.1 / 152.6 with operands copied between registers from tile to tile
// and, above 256 unknowns, four wavefronts whose accumulators moved between the
// two register files); 8192 systems at 255 unknowns take 56.9 us (60.0).
// GMRES adds three reads of the basis per step, which at 4096 systems and 384
// unknowns run at 6 TB/s: there it stays bound by them (187 us, 211 before);
// with 500 systems a step takes 103.6 us (141.7).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "visc1d.hpp"

namespace vd {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kG = kVisc1dGroup;   // systems per workgroup
constexpr int kRed = 16;           // Gram-Schmidt coefficients reduced together
constexpr int kAhead = 8;          // loads of the serial per-system recurrences in flight together
// GMRES: components of the new vector along the basis above this fraction of
// its norm are removed by a second Gram-Schmidt pass (the 3D solver's FP64
// tolerance; the residual estimate then differs from the true one by at most
// sqrt(1 + (m+1) tol) - 1)
constexpr double kVisc1dOrthTol = 1e-8;

enum Kind { K_APPLY = 0, K_RMR = 1, K_GMRES = 2, K_CG = 3 };

// NW wavefronts of TPW row tiles (16 unknowns each)
template <int TPW, int NW>
struct Lay {
  static constexpr int NP = 16 * TPW * NW;   // padded unknowns
  static constexpr int KT = NP / 16;         // k tiles of the square matrices
  static constexpr int V = NP * kG;          // doubles of one tiled vector
  static constexpr int NB = (NP + 16) * kG;  // operand buffer (one more row tile for the full-width products)
};

template <int TPW>
struct Vec {
  v4d t[TPW];
};

struct Ln {
  int lane, wv, sl, lq;  // lane, wavefront, system of the lane, row quad
};

// v4d index of this lane's tile t in a tiled vector
template <int TPW>
__device__ __forceinline__ int vi4(const Ln& l, int t) {
  return (l.wv * TPW + t) * 64 + l.lane;
}

// unknown held by component r of this lane's tile t
template <int TPW>
__device__ __forceinline__ int vrow(const Ln& l, int t, int r) {
  return 16 * (l.wv * TPW + t) + l.lq + 4 * r;
}

// tiled index of (row i, system s)
__device__ __forceinline__ int tidx(int i, int s) {
  return (i >> 4) * 256 + (((i & 3) * 16 + s) << 2) + ((i >> 2) & 3);
}

template <int TPW>
__device__ __forceinline__ void vld(Vec<TPW>& v, const double* p, const Ln& l) {
  const v4d* q = reinterpret_cast<const v4d*>(p);
#pragma unroll
  for (int t = 0; t < TPW; ++t) v.t[t] = q[vi4<TPW>(l, t)];
}

template <int TPW>
__device__ __forceinline__ void vst(const Vec<TPW>& v, double* p, const Ln& l) {
  v4d* q = reinterpret_cast<v4d*>(p);
#pragma unroll
  for (int t = 0; t < TPW; ++t) q[vi4<TPW>(l, t)] = v.t[t];
}

template <int TPW>
__device__ __forceinline__ void vzero(Vec<TPW>& v) {
#pragma unroll
  for (int t = 0; t < TPW; ++t) v.t[t] = v4d{0.0, 0.0, 0.0, 0.0};
}

template <int TPW>
__device__ __forceinline__ double pdot(const Vec<TPW>& u, const Vec<TPW>& v) {
  double s = 0.0;
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) s += u.t[t][r] * v.t[t][r];
  return s;
}

// acc[m] = M_m B for NM matrices of kt k tiles (MFMA operand order, row tiles
// stored rs k tiles apart) and the operand B in the LDS buffer (tiled, 16
// columns).  Component q of a lane's v4d of k tile T is the operand of k step
// 4 T + q for both A and B.  The operands of a k tile go to one of RING register
// sets, RING - 1 tiles before its products: a tile of one matrix is TPW * NM * 256
// MFMA cycles, an L2 latency is 500 to 800.  The loop is unrolled over the sets,
// so no register is copied, and the barriers to the scheduler keep the loads
// ahead of the products.  Tiles past the last are the last again, and unused.
template <int TPW, int NW, int NM>
__device__ __forceinline__ void mv(const double* const (&M)[NM], int rs, int kt, const double* buf, const Ln& l,
                                   Vec<TPW> (&acc)[NM]) {
  constexpr int RING = TPW * NM >= 3 || NW > 4 ? 2 : 4;
  const int wv = __builtin_amdgcn_readfirstlane(l.wv);
  const v4d* bq = reinterpret_cast<const v4d*>(buf) + l.lane;
  const v4d* ap[NM];
  v4d av[RING][NM][TPW], bv[RING];
  auto load = [&](int r, int T) {
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int t = 0; t < TPW; ++t) av[r][m][t] = (ap[m] + (size_t)(t * rs + T) * 64)[l.lane];
    bv[r] = bq[T * 64];
  };
  auto mul = [&](int r) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int t = 0; t < TPW; ++t)
          acc[m].t[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[r][m][t][q], bv[r][q], acc[m].t[t], 0, 0, 0);
  };
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    ap[m] = reinterpret_cast<const v4d*>(M[m]) + (size_t)wv * TPW * rs * 64;
    vzero(acc[m]);
  }
#pragma unroll
  for (int r = 0; r < RING - 1; ++r) load(r, min(r, kt - 1));
  int T = 0;
#pragma unroll 1
  for (; T + RING <= kt; T += RING) {
#pragma unroll
    for (int r = 0; r < RING; ++r) {
      load((r + RING - 1) % RING, min(T + r + RING - 1, kt - 1));
      __builtin_amdgcn_sched_barrier(0);
      mul(r);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int r = 0; r < RING - 1; ++r)
    if (T + r < kt) mul(r);
}

// Rows of 16 lanes exchanged between two registers without LDS: the sum of
// the pair (a, b) over neighbouring rows (swap16) or over the two halves of the
// wavefront (swap32); rows of even index (lower half) return a's sum, the others b's.
__device__ __forceinline__ double swap16_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double swap32_add(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// Sums over the unknowns of each system of per-lane partial values, in a fixed
// order: the four lanes of a wavefront that hold the system by two exchanges,
// then the NW wavefronts in order.
template <int NW>
__device__ __forceinline__ double wave_total(const double* p) {
  double s = p[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) s += p[w * kG];
  return s;
}
// Every lane gets the sums of its own system, at one barrier: successive sums
// use the two halves of the scratch in turn, and the sum before the last was
// read by every wavefront before it came to the last one's barrier.
struct Red {
  double* p;  // [2][2][NW][kG]
  int ph;
};
template <int NV, int NW>
__device__ __forceinline__ void gsum(double (&v)[NV], Red& rd, const Ln& l) {
  static_assert(NV <= 2, "scratch of two values");
  double* red = rd.p + rd.ph * 2 * NW * kG;
  rd.ph ^= 1;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const double h = swap16_add(v[k], v[k]);
    v[k] = swap32_add(h, h);
  }
  if (l.lq == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) red[(k * NW + l.wv) * kG + l.sl] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = wave_total<NW>(red + k * NW * kG + l.sl);
}
// The first nv of kRed sums go to out[k][system], one thread each; begins its
// writes to out after a barrier and ends with one.  The exchanges are shared by
// two values each, so that quad q is left with values q, q + 4, q + 8, ...
template <int NW>
__device__ __forceinline__ void gsum_to(const double (&v)[kRed], int nv, double* red, double* out, const Ln& l) {
#pragma unroll
  for (int d = 0; d < kRed / 4; ++d) {
    const double s = swap32_add(swap16_add(v[4 * d], v[4 * d + 1]), swap16_add(v[4 * d + 2], v[4 * d + 3]));
    red[((4 * d + l.lq) * NW + l.wv) * kG + l.sl] = s;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < nv * kG; e += 64 * NW)
    out[e] = wave_total<NW>(red + (e / kG) * NW * kG + (e % kG));
  __syncthreads();
}

// w = A z with z in the operand buffer (A = V_rho, L_rho or K_rho).  D1 z
// and D2 z are two passes over the buffer (one matrix each, fewer live
// registers than both at once); z itself is read back from the buffer for
// the pointwise terms.  Coefficients (tiled): viscous ca = a/rho, rp = rho',
// rpp = rho''; L_rho ca = 1/rho, rp = -rho'/rho^2; K_rho rpp = c.
template <int TPW, int NW, int OP>
__device__ __forceinline__ void op_buf(const Visc1dArgs& a, const double* buf, Vec<TPW>& w, const double* wca,
                                       const double* wrp, const double* wrpp, const Ln& l) {
  const v4d* zq = reinterpret_cast<const v4d*>(buf);
  const v4d* caq = reinterpret_cast<const v4d*>(wca);
  const v4d* rpq = reinterpret_cast<const v4d*>(wrp);
  const v4d* rppq = reinterpret_cast<const v4d*>(wrpp);
  if constexpr (OP == OP1D_PRES_K) {
    Vec<TPW> d2[1];
    const double* const M2[1] = {a.D2I};
    mv<TPW, NW, 1>(M2, Lay<TPW, NW>::KT, (a.ni + 15) >> 4, buf, l, d2);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const int i = vi4<TPW>(l, t);
      const v4d z = zq[i], c = rppq[i];
#pragma unroll
      for (int r = 0; r < 4; ++r) w.t[t][r] = d2[0].t[t][r] + c[r] * z[r];
    }
  } else {
    Vec<TPW> d1[1], d2[1];
    const double* const M1[1] = {a.D1I};
    const double* const M2[1] = {a.D2I};
    mv<TPW, NW, 1>(M1, Lay<TPW, NW>::KT, (a.ni + 15) >> 4, buf, l, d1);
    mv<TPW, NW, 1>(M2, Lay<TPW, NW>::KT, (a.ni + 15) >> 4, buf, l, d2);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const int i = vi4<TPW>(l, t);
      if constexpr (OP == OP1D_VISC) {
        const v4d z = zq[i], ca = caq[i], rp = rpq[i], rpp = rppq[i];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          w.t[t][r] = z[r] - ca[r] * (d2[0].t[t][r] + rpp[r] * z[r] + rp[r] * d1[0].t[t][r]);
      } else {
        const v4d ca = caq[i], rp = rpq[i];
#pragma unroll
        for (int r = 0; r < 4; ++r) w.t[t][r] = ca[r] * d2[0].t[t][r] + rp[r] * d1[0].t[t][r];
      }
    }
  }
}

// Wavefronts per SIMD that the registers have to leave room for: two groups on a
// CU up to 256 unknowns (RMR, CG), one beyond that and with GMRES.
template <int TPW, int NW, int KIND>
constexpr int kVisc1dWaves = ((NW + 3) / 4) * (KIND == K_GMRES || TPW * NW > 16 ? 1 : 2);

}  // namespace

template <int TPW, int NW, int KIND, int OP>
__global__ __launch_bounds__(64 * NW, (kVisc1dWaves<TPW, NW, KIND>)) void k_visc1d(Visc1dArgs a) {
  constexpr int kT = 64 * NW;  // threads per workgroup
  using L = Lay<TPW, NW>;
  extern __shared__ __attribute__((aligned(32))) double lds[];
  const int m = KIND == K_GMRES ? a.restart : 0;
  double* buf = lds;                  // [NB] right-hand operand of the products
  double* red = buf + L::NB;          // GMRES: [kRed][NW][kG] wavefront partial sums
  Red rd{red + (m ? kRed : 0) * NW * kG, 0};  // scratch of the small sums
  double* hco = rd.p + 4 * NW * kG;   // [m + 1][kG] Hessenberg column being built
  double* cco = hco + (m + 1) * kG;   // [m + 1][kG] coefficients of the current pass, then y
  int* bad_s = reinterpret_cast<int*>(cco + (m + 1) * kG);  // [kG] density rejected
  int* stop_s = bad_s + kG;                                  // [kG] Arnoldi stop flags
  int* need = stop_s + kG;                                   // [m + 1] basis vectors of the second pass
  const Ln l{(int)threadIdx.x & 63, (int)threadIdx.x >> 6, (int)threadIdx.x & 15, ((int)threadIdx.x >> 4) & 3};
  const int g0 = blockIdx.x * kG;
  const int nsys = min(kG, a.batch - g0);
  const bool live = l.sl < nsys;
  const int ni = a.ni, np = a.np, off = a.off;
  double* W = a.work + (size_t)blockIdx.x * a.work_stride;
  double* wca = W;              // a / rho on the unknowns (tiled)
  double* wrp = W + L::V;       // rho'
  double* wrpp = W + 2 * L::V;  // rho''
  double* wb = W + 3 * L::V;    // right-hand side
  double* wx = W + 4 * L::V;    // solution (GMRES)

  // densities of the group, row i = grid point i; absent systems get rho = 1
  if (threadIdx.x < kG) bad_s[threadIdx.x] = 0;
  for (int e = threadIdx.x; e < L::NB; e += kT) buf[e] = 0.0;
  __syncthreads();
  for (int e = threadIdx.x; e < kG * np; e += kT) {
    const int s = e / np, i = e - s * np;
    double v = 1.0;
    if (s < nsys) {
      v = a.rho[(size_t)(g0 + s) * np + i];
      if (!(v > 0.0) || !isfinite(v)) bad_s[s] = 1;
    }
    if constexpr (OP == OP1D_PRES_K) {  // psi = rho^-1/2 on the unknowns, the operand of D2 P
      const int k = i - off;
      if (k >= 0 && k < ni) buf[tidx(k, s)] = 1.0 / sqrt(v);
    } else {
      buf[tidx(i, s)] = v;
    }
  }
  __syncthreads();
  const bool bad = bad_s[l.sl] != 0;
  if constexpr (OP == OP1D_PRES_K) {
    // c = -(D2 P psi) / psi
    Vec<TPW> acc[1], c, zero;
    const double* const M[1] = {a.D2I};
    mv<TPW, NW, 1>(M, Lay<TPW, NW>::KT, (a.ni + 15) >> 4, buf, l, acc);
    vzero(zero);
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = vrow<TPW>(l, t, r);
        const bool ok = live && !bad && i < ni;
        c.t[t][r] = ok ? -acc[0].t[t][r] / buf[tidx(i, l.sl)] : 0.0;
      }
    vst(zero, wca, l);
    vst(zero, wrp, l);
    vst(c, wrpp, l);
  } else {
    Vec<TPW> acc[2], ca;
    const double* const M[2] = {a.D1F, a.D2F};
    mv<TPW, NW, 2>(M, a.kt_full, a.kt_full, buf, l, acc);
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = vrow<TPW>(l, t, r);
        const bool ok = live && !bad && i < ni;
        const double rho_i = ok ? buf[tidx(i + off, l.sl)] : 1.0;
        if constexpr (OP == OP1D_VISC) {
          ca.t[t][r] = ok ? a.a / rho_i : 0.0;
        } else {  // L_rho: 1/rho and -rho'/rho^2
          ca.t[t][r] = ok ? 1.0 / rho_i : 0.0;
          acc[0].t[t][r] = ok ? -acc[0].t[t][r] / (rho_i * rho_i) : 0.0;
          acc[1].t[t][r] = 0.0;
        }
        if (!ok) {
          acc[0].t[t][r] = 0.0;
          acc[1].t[t][r] = 0.0;
        }
      }
    vst(ca, wca, l);
    vst(acc[0], wrp, l);
    vst(acc[1], wrpp, l);
  }
  __syncthreads();

  // a [batch][np] array of the group into registers (zero off the unknowns)
  auto gather = [&](const double* src, Vec<TPW>& v) {
    for (int e = threadIdx.x; e < L::V; e += kT) {
      const int T = e >> 8, ln = (e >> 2) & 63, r = e & 3;
      const int s = ln & 15, i = 16 * T + (ln >> 4) + 4 * r;
      buf[e] = (i < ni && s < nsys && !bad_s[s]) ? src[(size_t)(g0 + s) * np + off + i] : 0.0;
    }
    __syncthreads();
    vld(v, buf, l);
    __syncthreads();
  };
  // write a group vector to a.x; `field`: a pressure field (solution or
  // preconditioned vector), whose wall values follow from the Neumann
  // extension, else zero walls (viscous fields, pressure equation rows)
  auto scatter = [&](const Vec<TPW>& v, bool field) {
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = vrow<TPW>(l, t, r);
        if (live && i < ni) a.x[(size_t)(g0 + l.sl) * np + off + i] = bad ? 0.0 : v.t[t][r];
      }
    if constexpr (OP != OP1D_VISC) {
      if (field) {
        double wsum[2] = {0.0, 0.0};
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = vrow<TPW>(l, t, r);
            if (i < ni) {
              wsum[0] += a.E0[i] * v.t[t][r];
              wsum[1] += a.EM[i] * v.t[t][r];
            }
          }
        gsum<2, NW>(wsum, rd, l);
        if (l.wv == 0 && l.lq == 0 && live) {
          a.x[(size_t)(g0 + l.sl) * np] = bad ? 0.0 : wsum[0];
          a.x[(size_t)(g0 + l.sl) * np + np - 1] = bad ? 0.0 : wsum[1];
        }
        return;
      }
    }
    const int nw = np - ni;  // points outside the unknowns: the two walls
    for (int e = threadIdx.x; e < nsys * nw; e += kT) {
      const int s = e / nw, k = e - s * nw;
      a.x[(size_t)(g0 + s) * np + (k < off ? k : ni + k)] = 0.0;
    }
  };
  // residual history entry k of this lane's system (one writer per system)
  double* hrow = a.hist ? a.hist + (size_t)(g0 + l.sl) * a.hist_cap : nullptr;
  auto record = [&](int k, double v) {
    if (hrow && live && l.wv == 0 && l.lq == 0 && k < a.hist_cap) hrow[k] = v;
  };
  auto finish = [&](int it, double rel, int status) {
    if (l.wv == 0 && l.lq == 0 && live) {
      a.iters[g0 + l.sl] = bad ? 0 : it;
      a.relres[g0 + l.sl] = bad ? 0.0 : rel;
      a.status[g0 + l.sl] = bad ? -3 : status;
    }
  };
  // Z = M^-1 R (Z = R without preconditioner)
  auto prec = [&](const Vec<TPW>& R, Vec<TPW>& Z) {
    if (a.precond) {
      vst(R, buf, l);
      __syncthreads();
      Vec<TPW> acc[1];
      const double* const M[1] = {a.VI};
      mv<TPW, NW, 1>(M, L::KT, (a.ni + 15) >> 4, buf, l, acc);
      __syncthreads();
      Z = acc[0];
    } else {
      Z = R;
    }
  };
  // Wv = V_rho Z; Z stays in the operand buffer until the next product.  A sum
  // over the unknowns, with its barrier, has to come before that.
  auto apply = [&](const Vec<TPW>& Z, Vec<TPW>& Wv) {
    vst(Z, buf, l);
    __syncthreads();
    op_buf<TPW, NW, OP>(a, buf, Wv, wca, wrp, wrpp, l);
  };
  // R = b - V_rho X; returns ||R|| of this lane's system
  auto residual = [&](const Vec<TPW>& X, Vec<TPW>& R) -> double {
    Vec<TPW> w, bv;
    apply(X, w);
    vld(bv, wb, l);
#pragma unroll
    for (int t = 0; t < TPW; ++t) R.t[t] = bv.t[t] - w.t[t];
    double s[1] = {pdot(R, R)};
    gsum<1, NW>(s, rd, l);
    return sqrt(s[0]);
  };

  Vec<TPW> B;
  gather(a.b, B);
  if constexpr (KIND == K_APPLY) {
    Vec<TPW> Y;
    const bool pre = a.mode == VISC1D_APPLY_PREC;
    if (pre) {
      prec(B, Y);
    } else {
      apply(B, Y);
    }
    scatter(Y, pre);
    finish(0, 0.0, 0);
    return;
  } else {
    vst(B, wb, l);
    double bn;
    {
      double s[1] = {pdot(B, B)};
      gsum<1, NW>(s, rd, l);
      bn = sqrt(s[0]);
    }
    Vec<TPW> X;
    if (a.use_x0) gather(a.x, X);
    else vzero(X);
    if (bn == 0.0) vzero(X);
    bool done = !live || bad || bn == 0.0;
    int it = 0, status = 0;
    double rel = 0.0;
    Vec<TPW> R;

    if constexpr (KIND == K_RMR) {
      // z = M^-1 r; w = A z; alpha = (r, w) / (w, w); x += alpha z; r -= alpha w.
      // x lives in the workspace (read and written once per iteration) so that
      // the registers hold two groups per CU.
      double rn = residual(X, R);
      vst(X, wx, l);
      if (!done) record(0, rn / bn);
      else if (bn == 0.0) record(0, 0.0);
      while (true) {
        if (!done) {
          rel = rn / bn;
          if (!(rn == rn)) {
            status = -4;
            done = true;
          } else if (rel <= a.rtol) {
            done = true;
          } else if (it >= a.max_iter) {
            status = 1;
            done = true;
          }
        }
        if (!__any(!done)) break;
        Vec<TPW> Z, Wv;
        prec(R, Z);
        apply(Z, Wv);
        double s2[2] = {pdot(R, Wv), pdot(Wv, Wv)};
        gsum<2, NW>(s2, rd, l);
        const double alpha = s2[1] > 0.0 ? s2[0] / s2[1] : 0.0;
        if (!done) {
          // z is still in the operand buffer
          v4d* xq = reinterpret_cast<v4d*>(wx);
          const v4d* zq = reinterpret_cast<const v4d*>(buf);
#pragma unroll
          for (int t = 0; t < TPW; ++t) {
            xq[vi4<TPW>(l, t)] += alpha * zq[vi4<TPW>(l, t)];
            R.t[t] -= alpha * Wv.t[t];
          }
          ++it;
        }
        double s1[1] = {pdot(R, R)};
        gsum<1, NW>(s1, rd, l);
        if (!done) {
          rn = sqrt(s1[0]);
          record(it, rn / bn);
        }
        // the true residual now and then, against drift of the recurrence
        const bool need = !done && (rn / bn <= a.rtol || it % 50 == 0);
        if (__any(need)) {
          Vec<TPW> R2, Xc;
          vld(Xc, wx, l);
          const double rn2 = residual(Xc, R2);
          if (need) {
            R = R2;
            rn = rn2;
          }
        }
      }
      vld(X, wx, l);
      scatter(X, true);
    } else if constexpr (KIND == K_CG) {
      // Preconditioned conjugate gradient (Sec. 3.1 solver list): z = M^-1 r;
      // p = z (first step and restarts) or z + beta p with
      // beta = (r, z) / (r, z)_previous; q = A p; alpha = (r, z) / (p, q);
      // x += alpha p; r -= alpha q.  x and p live in the workspace.  When the
      // recursive residual meets the tolerance the true residual replaces
      // it, and if that does not, the iteration restarts from it.  CG is not
      // meant for the non-symmetric collocation operators; the paper runs it
      // on them anyway and reports how it fails (Secs. 3.1 and 3.2).
      double* wp = W + 5 * L::V;
      double rn = residual(X, R);
      vst(X, wx, l);
      if (!done) record(0, rn / bn);
      else if (bn == 0.0) record(0, 0.0);
      double rz = 0.0;
      bool fresh = true;
      while (true) {
        if (!done) {
          rel = rn / bn;
          if (!(rn == rn)) {
            status = -4;
            done = true;
          } else if (rel <= a.rtol) {
            done = true;
          } else if (it >= a.max_iter) {
            status = 1;
            done = true;
          }
        }
        if (!__any(!done)) break;
        {
          Vec<TPW> Z, P;
          prec(R, Z);
          double s1[1] = {pdot(R, Z)};
          gsum<1, NW>(s1, rd, l);
          if (fresh) {
            P = Z;
          } else {
            vld(P, wp, l);
            const double beta = rz != 0.0 ? s1[0] / rz : 0.0;
#pragma unroll
            for (int t = 0; t < TPW; ++t) P.t[t] = Z.t[t] + beta * P.t[t];
          }
          rz = s1[0];
          fresh = false;
          vst(P, wp, l);
        }
        // q = A p with p in the operand buffer; p is read back from there
        // (each lane its own entries) rather than kept in registers
        {
          Vec<TPW> P;
          vld(P, wp, l);
          vst(P, buf, l);
        }
        __syncthreads();
        Vec<TPW> Q;
        op_buf<TPW, NW, OP>(a, buf, Q, wca, wrp, wrpp, l);
        const v4d* pq = reinterpret_cast<const v4d*>(buf);
        double s2[1] = {0.0};
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
          const v4d pv = pq[vi4<TPW>(l, t)];
#pragma unroll
          for (int r = 0; r < 4; ++r) s2[0] += pv[r] * Q.t[t][r];
        }
        gsum<1, NW>(s2, rd, l);
        const double alpha = s2[0] != 0.0 ? rz / s2[0] : 0.0;
        if (!done) {
          v4d* xq = reinterpret_cast<v4d*>(wx);
#pragma unroll
          for (int t = 0; t < TPW; ++t) {
            xq[vi4<TPW>(l, t)] += alpha * pq[vi4<TPW>(l, t)];
            R.t[t] -= alpha * Q.t[t];
          }
          ++it;
        }
        double s1[1] = {pdot(R, R)};
        gsum<1, NW>(s1, rd, l);
        if (!done) {
          rn = sqrt(s1[0]);
          record(it, rn / bn);
        }
        const bool need = !done && rn / bn <= a.rtol;
        if (__any(need)) {
          Vec<TPW> R2, Xc;
          vld(Xc, wx, l);
          const double rn2 = residual(Xc, R2);
          if (need) {
            R = R2;
            rn = rn2;
            fresh = true;
          }
        }
      }
      vld(X, wx, l);
      scatter(X, true);
    } else {
      // right-preconditioned GMRES(m), classical Gram-Schmidt with a measured check
      double* wbas = W + 5 * L::V;                 // [m + 1] tiled basis vectors
      double* wH = wbas + (size_t)(m + 1) * L::V;  // [m][m + 1][kG]: column j, row i
      double* wcs = wH + (size_t)(m + 1) * m * kG; // [m][kG]
      double* wsn = wcs + (size_t)m * kG;          // [m][kG]
      double* wg = wsn + (size_t)m * kG;           // [m + 1][kG]
      const bool owner = l.wv == 0 && l.lq == 0;   // lanes 0..15 of wavefront 0 keep the per-system scalars
      double beta = residual(X, R);
      vst(X, wx, l);
      if (!done) record(0, beta / bn);
      else if (bn == 0.0) record(0, 0.0);
      while (true) {
        if (!done) {
          rel = beta / bn;
          if (!(beta == beta)) {
            status = -4;
            done = true;
          } else if (rel <= a.rtol) {
            done = true;
          } else if (it >= a.max_iter) {
            status = 1;
            done = true;
          }
        }
        const bool cyc = !done;
        if (!__any(cyc)) break;
        Vec<TPW> Vj;
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) Vj.t[t][r] = cyc ? R.t[t][r] / beta : 0.0;
        vst(Vj, wbas, l);
        if (owner) {
          wg[l.sl] = beta;
          for (int i = 1; i <= m; ++i) wg[i * kG + l.sl] = 0.0;
        }
        bool park = !cyc;
        int k = 0, jend = 0;
        for (int j = 0; j < m; ++j) {
          Vec<TPW> Z, Wv;
          prec(Vj, Z);
          apply(Z, Wv);
          if (!park) ++it;
          // Classical Gram-Schmidt with a measured check, as in the 3D solver:
          // h = V^T w, w' = w - V h, then c = V^T w'.  A second pass subtracts
          // only the components with |c_i| > tol ||w'|| of some system of the
          // group and reads only those basis vectors (CGS2 read the basis four
          // times per step, this reads it three times plus the few
          // selected).  (w', w') is summed along with c, and is the new vector's
          // norm when nothing is selected.
          // kFly vectors' loads are in flight at a time (past the last vector, the
          // last again): one at a time, each waited out an L2 latency.
          constexpr int kFly = TPW > 2 ? 2 : 4;
          // cco[i][s] = (v_i, w) for i <= j, and (w, w) at i = j + 1
          auto basis_dots = [&](bool norm) {
            const int nd = j + 1 + (norm ? 1 : 0);
            const double ww = norm ? pdot(Wv, Wv) : 0.0;
            for (int i0 = 0; i0 < nd; i0 += kRed) {
              double p[kRed];
#pragma unroll
              for (int c0 = 0; c0 < kRed; c0 += kFly) {
                if (i0 + c0 <= j) {
                  Vec<TPW> vi[kFly];
#pragma unroll
                  for (int c = 0; c < kFly; ++c) vld(vi[c], wbas + (size_t)min(i0 + c0 + c, j) * L::V, l);
#pragma unroll
                  for (int c = 0; c < kFly; ++c) p[c0 + c] = pdot(vi[c], Wv);
                }
#pragma unroll
                for (int c = 0; c < kFly; ++c)
                  if (i0 + c0 + c > j) p[c0 + c] = ww;
              }
              gsum_to<NW>(p, min(kRed, nd - i0), red, cco + (size_t)i0 * kG, l);
            }
          };
          // w -= sum_i cco[i] v_i over i <= j, or over the vectors flagged in need
          auto basis_update = [&](bool flagged) {
            for (int i0 = 0; i0 <= j; i0 += kFly) {
              if (flagged) {
                for (int i = i0; i <= min(i0 + kFly - 1, j); ++i) {
                  if (!need[i]) continue;  // uniform across the block
                  const double c = cco[i * kG + l.sl];
                  Vec<TPW> vi;
                  vld(vi, wbas + (size_t)i * L::V, l);
#pragma unroll
                  for (int t = 0; t < TPW; ++t) Wv.t[t] -= c * vi.t[t];
                }
                continue;
              }
              Vec<TPW> vi[kFly];
#pragma unroll
              for (int c = 0; c < kFly; ++c) vld(vi[c], wbas + (size_t)min(i0 + c, j) * L::V, l);
#pragma unroll
              for (int c = 0; c < kFly; ++c) {
                if (i0 + c > j) break;
                const double y = cco[(i0 + c) * kG + l.sl];
#pragma unroll
                for (int t = 0; t < TPW; ++t) Wv.t[t] -= y * vi[c].t[t];
              }
            }
          };
          basis_dots(false);
          for (int e = threadIdx.x; e < (j + 1) * kG; e += kT) hco[e] = cco[e];
          basis_update(false);
          basis_dots(true);
          double s[1] = {cco[(j + 1) * kG + l.sl]};
          // keep c_i[s] only where it fails the test (NaN fails); vector i is
          // read when any system keeps it
          bool second = false;
          for (int e0 = 0; e0 < (j + 1) * kG; e0 += kT) {
            const int e = e0 + (int)threadIdx.x;
            bool keep = false;
            if (e < (j + 1) * kG) {
              keep = !(fabs(cco[e]) <= kVisc1dOrthTol * sqrt(s[0]));
              if (!keep) cco[e] = 0.0;
            }
            const unsigned long long kept = __ballot(keep);
            if (l.sl == 0 && e < (j + 1) * kG) need[e / kG] = (kept >> (l.lq * kG)) & 0xffffull ? 1 : 0;
            second |= kept != 0;
          }
          if (__syncthreads_or(second)) {
            basis_update(true);
            for (int e = threadIdx.x; e < (j + 1) * kG; e += kT) hco[e] += cco[e];
            s[0] = pdot(Wv, Wv);
            gsum<1, NW>(s, rd, l);
          }
          const double hn = sqrt(s[0]);
#pragma unroll
          for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) Vj.t[t][r] = hn > 0.0 ? Wv.t[t][r] / hn : 0.0;
          vst(Vj, wbas + (size_t)(j + 1) * L::V, l);
          if (owner && !park) {
            // previous rotations on the new column, then the new rotation
            double hj = hco[l.sl];
            for (int i0 = 0; i0 < j; i0 += kAhead) {  // kAhead rotations loaded at a time
              double cv[kAhead], sv[kAhead];
#pragma unroll
              for (int q = 0; q < kAhead; ++q) {
                const int i = min(i0 + q, j - 1);
                cv[q] = wcs[i * kG + l.sl];
                sv[q] = wsn[i * kG + l.sl];
              }
#pragma unroll
              for (int q = 0; q < kAhead; ++q) {
                const int i = i0 + q;
                if (i >= j) break;
                const double hb = hco[(i + 1) * kG + l.sl];
                wH[((size_t)j * (m + 1) + i) * kG + l.sl] = cv[q] * hj + sv[q] * hb;
                hj = -sv[q] * hj + cv[q] * hb;
              }
            }
            const double rr = hypot(hj, hn);
            const double c = rr > 0.0 ? hj / rr : 1.0, sg = rr > 0.0 ? hn / rr : 0.0;
            wcs[j * kG + l.sl] = c;
            wsn[j * kG + l.sl] = sg;
            wH[((size_t)j * (m + 1) + j) * kG + l.sl] = rr;
            const double gj = wg[j * kG + l.sl];
            const double gn = -sg * gj;
            wg[(j + 1) * kG + l.sl] = gn;
            wg[j * kG + l.sl] = c * gj;
            record(it, fabs(gn) / bn);
            stop_s[l.sl] = (fabs(gn) / bn <= a.rtol || hn == 0.0 || it >= a.max_iter || !(rr == rr)) ? 1 : 0;
          }
          __syncthreads();
          if (!park) {
            k = j + 1;
            park = stop_s[l.sl] != 0;
          }
          jend = j + 1;
          if (!__any(!park)) break;
        }
        // back-solve H y = g (y into cco), then x += M^-1 (V y)
        if (owner) {
          for (int i = jend - 1; i >= 0; --i) {
            double yi = 0.0;
            if (i < k) {
              double t = wg[i * kG + l.sl];
              for (int q0 = i + 1; q0 < k; q0 += kAhead) {
                double hv[kAhead];
#pragma unroll
                for (int q = 0; q < kAhead; ++q)
                  hv[q] = wH[((size_t)min(q0 + q, k - 1) * (m + 1) + i) * kG + l.sl];
#pragma unroll
                for (int q = 0; q < kAhead; ++q)
                  if (q0 + q < k) t -= hv[q] * cco[(q0 + q) * kG + l.sl];
              }
              const double d = wH[((size_t)i * (m + 1) + i) * kG + l.sl];
              yi = d != 0.0 ? t / d : 0.0;
            }
            cco[i * kG + l.sl] = yi;
          }
        }
        __syncthreads();
        Vec<TPW> C, Z;
        vzero(C);
        for (int i = 0; i < jend; ++i) {
          const double y = cco[i * kG + l.sl];
          Vec<TPW> vi;
          vld(vi, wbas + (size_t)i * L::V, l);
          if (i < k) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) C.t[t] += y * vi.t[t];
          }
        }
        __syncthreads();  // cco is rewritten by the next cycle
        prec(C, Z);
        vld(X, wx, l);
        if (cyc) {
#pragma unroll
          for (int t = 0; t < TPW; ++t) X.t[t] += Z.t[t];
        }
        vst(X, wx, l);
        beta = residual(X, R);
      }
      vld(X, wx, l);
      scatter(X, true);
    }
    finish(it, rel, status);
  }
}

namespace {

template <int TPW, int NW, int OP>
hipError_t launch_tpw(const Visc1dArgs& a, hipStream_t st) {
  using L = Lay<TPW, NW>;
  constexpr int kT = 64 * NW;
  const int kind = a.mode != VISC1D_SOLVE    ? K_APPLY
                   : a.solver == VISC1D_RMR ? K_RMR
                   : a.solver == VISC1D_CG  ? K_CG
                                            : K_GMRES;
  const int m = kind == K_GMRES ? a.restart : 0;
  const size_t lds = (size_t)(L::NB + ((m ? kRed : 0) + 4) * NW * kG + 2 * (m + 1) * kG) * sizeof(double) +
                     (2 * kG + m + 1) * sizeof(int);
  const void* fn = kind == K_APPLY ? reinterpret_cast<const void*>(&k_visc1d<TPW, NW, K_APPLY, OP>)
                   : kind == K_RMR ? reinterpret_cast<const void*>(&k_visc1d<TPW, NW, K_RMR, OP>)
                   : kind == K_CG  ? reinterpret_cast<const void*>(&k_visc1d<TPW, NW, K_CG, OP>)
                                   : reinterpret_cast<const void*>(&k_visc1d<TPW, NW, K_GMRES, OP>);
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((a.batch + kG - 1) / kG);
  if (kind == K_APPLY) hipLaunchKernelGGL((k_visc1d<TPW, NW, K_APPLY, OP>), grid, dim3(kT), lds, st, a);
  else if (kind == K_RMR) hipLaunchKernelGGL((k_visc1d<TPW, NW, K_RMR, OP>), grid, dim3(kT), lds, st, a);
  else if (kind == K_CG) hipLaunchKernelGGL((k_visc1d<TPW, NW, K_CG, OP>), grid, dim3(kT), lds, st, a);
  else hipLaunchKernelGGL((k_visc1d<TPW, NW, K_GMRES, OP>), grid, dim3(kT), lds, st, a);
  return hipGetLastError();
}

}  // namespace

}  // namespace vd

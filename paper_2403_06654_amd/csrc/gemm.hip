// Dense contractions of the Chebyshev direction on MFMA (gfx950), and the
// wall-bounded pressure operator built from them.
//
// C[M][N] = epilogue(alpha * A[M][K] * B[K][N]): A a small dense matrix of the
// z direction, B a field whose rows are z levels and whose columns are the
// packed x spectrum viewed as reals (the z matrices are real, so complex
// columns contract as pairs of real columns).  A block computes a 16 x 16
// or 16 x 32 tile with v_mfma_f64_16x16x4_f64 (FP32: v_mfma_f32_16x16x4_f32), stepping
// K by 4; operands are read straight from global memory (the A matrix and
// the field each fit in L2).  Lane l feeds
// A[l % 16][l / 16] and B[l / 16][l % 16]; accumulator r of lane l holds
// D[4 (l / 16) + r][l % 16] for the FP32 instruction and D[l / 16 + 4 r][l % 16]
// for the FP64 one (both checked by a one-hot probe of each lane).
#include <cstdio>

#include "../../include/vdsolve.h"
#include "cheb_ops.hpp"
#include "spectral.hpp"

namespace vd {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <typename R>
struct Mfma;
template <>
struct Mfma<double> {
  using V = v4d;
  static __device__ __forceinline__ int row(int lk, int r) { return lk + 4 * r; }
  static __device__ __forceinline__ V mac(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<float> {
  using V = v4f;
  static __device__ __forceinline__ int row(int lk, int r) { return 4 * lk + r; }
  static __device__ __forceinline__ V mac(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// Epilogue of the first contraction of the preconditioner: row j (the j-th
// generalised eigenvector), real column c of the packed spectrum (kx = c/2;
// kx = 0 holds kx = 0 and nx/2, both with k' = 0) is scaled by
// s / (k'^2 + lambda_j), and the constant mode (kx slot 0, j = 0) is zeroed.
struct EpiArgs {
  int kind;                // 0 plain, 1 preconditioner diagonal
  const double* alpha_dev; // optional device scalar multiplying the product
  double alpha;
  const double* lam;       // eigenvalues (device, FP64)
  double scale;            // rho0 / h_x
  double sx;               // 2 pi / L_x
  const int* gate;         // nonzero *gate: the launch does nothing
};

// One 512-thread block per 16 x 16 TN tile of C; the 8 waves split K (wave w
// takes the k-steps w, w+8, w+16, ...), and the eight partial tiles are summed
// through LDS before the epilogue.  The Chebyshev contractions are small
// (M = 257 or 514 rows, N = 512 real columns, K = 257 or 514): a launch is bound
// by its loads, their latency and their number, not by MFMA or HBM (at
// M = K = 514 the loads alone take 11.5 of 13.3 us).  So the first batch of loads
// is issued before the halt flag is read, batches are short (KU k-steps), and
// where there are enough 16 x 16 tiles (kGemmTiles) a
// wave computes two column tiles from one 16 B load of B per k-step and lane:
// lane li then holds columns 2 li and 2 li + 1.  4 and 16 waves, 32 x 32 tiles per
// wave and tiles staged in LDS (22-26 us at M = K = 514) are slower.
// Whatever the tile, an element is the same sum: a wave's k-steps go to two chains
// in turn, and the chains of all waves are added in FP64.  (FP32 products, relative
// error at K = 257 / 514 / 1026: 7.8e-8 / 1.06e-7 / 1.47e-7; with one chain per
// column tile 1.06e-7 / 1.47e-7 / 2.05e-7, for 2 to 3% of the TN = 2 launch.)
// AT: A is stored transposed ([K][M]), so a load of 16 consecutive rows is
// one contiguous run.
constexpr int kGemmWaves = 8, kGemmKU = 3;
// Two column tiles above three 16 x 16 tiles per CU.  A block of two takes 1.5 times
// as long as a block of one: at 513 to 768 tiles that is two rounds of the CUs
// against three, which gains nothing, and beyond it does gain.  Measured, us per
// launch (TN = 1 / TN = 2, N = 512): M = 257, K = 257 (544 tiles) 5.4 / 5.6 in FP64,
// 4.2 / 4.5 in FP32; M = 257, K = 514 8.6 / 8.9 and 6.4 / 7.0; M = 385, K = 385 (800
// tiles) 8.2 / 7.3 and 6.3 / 5.8; M = K = 514 (1056 tiles) 12.7 / 12.0 and 9.7 / 9.7;
// M = K = 770 23.8 / 20.4 and 16.4 / 16.3.  (257 to 512 tiles, one round against two,
// gains 3% in FP64 (-9 to 11%) and nothing in FP32; they keep the single tile.)
constexpr int kGemmTiles = 768;

template <typename R, bool AT, int TN>
__global__ __launch_bounds__(64 * kGemmWaves) void k_gemm(const R* __restrict__ A, int lda, const R* __restrict__ B,
                                                          int ldb, R* __restrict__ C, int ldc, int M, int N, int K,
                                                          EpiArgs e) {
  using MF = Mfma<R>;
  constexpr int W = kGemmWaves, KU = kGemmKU, TS = 16 * TN, LD = TS + 1;
  __shared__ double part[W][16 * LD];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = blockIdx.y * 16, c0 = blockIdx.x * TS;
  const int li = lane & 15, lk = lane >> 4;
  const int ra = r0 + li, cb = c0 + TN * li;
  const bool rin = ra < M, cin = cb < N;  // TN = 2: N is even
  // two chains per column tile, alternate k-steps of this wave, added in FP64
  typename MF::V acc[TN][2] = {};
  R a[KU], b[KU][TN];
  auto load = [&](int s0) {
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int k = 4 * (s0 + W * u) + lk;
      const bool kin = k < K;
      a[u] = (kin && rin) ? (AT ? A[(size_t)k * lda + ra] : A[(size_t)ra * lda + k]) : R(0);
      if constexpr (TN == 2) {
        const C2<R> v = (kin && cin) ? ldg((const C2<R>*)(B + (size_t)k * ldb + cb)) : C2<R>{R(0), R(0)};
        b[u][0] = v.x;
        b[u][1] = v.y;
      } else {
        b[u][0] = (kin && cin) ? B[(size_t)k * ldb + cb] : R(0);
      }
    }
  };
  load(w);
  if (e.gate && *e.gate) return;
  static_assert(KU % 2 == 1, "the chains change places from batch to batch");
  int s0 = w;
  bool more = true;
  while (more) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int u = 0; u < KU; ++u) {
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[j][(h + u) & 1] = MF::mac(a[u], b[u][j], acc[j][(h + u) & 1]);
      }
      s0 += W * KU;
      more = 4 * s0 < K;
      if (!more) break;
      load(s0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double* o = part[w] + MF::row(lk, r) * LD + TN * li;
#pragma unroll
    for (int j = 0; j < TN; ++j) o[j] = (double)acc[j][0][r] + (double)acc[j][1][r];
  }
  __syncthreads();
  if (threadIdx.x >= 16 * TS) return;
  const double al = (e.alpha_dev ? *e.alpha_dev : 1.0) * e.alpha;
  const int tr = threadIdx.x / TS, tc = threadIdx.x % TS;
  const int row = r0 + tr, col = c0 + tc;
  if (row >= M || col >= N) return;
  const int o = tr * LD + tc;
  double v = 0.0;
#pragma unroll
  for (int q = 0; q < W; ++q) v += part[q][o];
  v *= al;
  if (e.kind == 1) {
    const int kx = col >> 1;
    const double kp = kx * e.sx;  // slot 0: k' = 0 for both halves
    if (kx == 0 && row == 0) v = 0.0;
    else v *= e.scale / (kp * kp + e.lam[row]);
  }
  C[(size_t)row * ldc + col] = R(v);
}

template <typename R, bool AT = true>
static void gemm(const R* A, int lda, const R* B, int ldb, R* C, int ldc, int M, int N, int K, const EpiArgs& e,
                 hipStream_t s) {
  const dim3 grid((N + 15) / 16, (M + 15) / 16), bl(64 * kGemmWaves);
  // pairs of columns: an even row length and pairs that sit aligned
  const bool pairs = N % 2 == 0 && ldb % 2 == 0 && (size_t)B % (2 * sizeof(R)) == 0;
  if (pairs && (long long)grid.x * grid.y > kGemmTiles)
    hipLaunchKernelGGL((k_gemm<R, AT, 2>), dim3((N + 31) / 32, grid.y), bl, 0, s, A, lda, B, ldb, C, ldc, M, N, K, e);
  else
    hipLaunchKernelGGL((k_gemm<R, AT, 1>), grid, bl, 0, s, A, lda, B, ldb, C, ldc, M, N, K, e);
}

static EpiArgs plain(double alpha = 1.0, const double* alpha_dev = nullptr) {
  EpiArgs e{};
  e.kind = 0;
  e.alpha = alpha;
  e.alpha_dev = alpha_dev;
  return e;
}

template <typename R>
void gemm_plain(const void* A, const void* B, void* C, int M, int N, int K, hipStream_t s) {
  gemm<R, false>((const R*)A, K, (const R*)B, N, (R*)C, N, M, N, K, plain(), s);
}

// ------------------------------------------------------------ C2 operator

template <typename R>
const R* mat(const ChebDev& cd, int which);

template <>
const double* mat<double>(const ChebDev& cd, int which) {
  return cd.m64[which];
}
template <>
const float* mat<float>(const ChebDev& cd, int which) {
  return cd.m32[which];
}

template <typename R>
void c2_apply(const Geom& g, const ChebDev& cd, const OpParams& p, const void* v, void* y, void* wY, void* wT,
              const void* coef, const void* twtab, hipStream_t st, Prof* prof) {
  const int nz = g.nz, n = 2 * g.M;  // real columns
  const size_t fs = (size_t)nz * n;  // reals per field
  R* T = (R*)wT;                     // [2 nz][n]
  auto gated = [&](EpiArgs e) {
    e.gate = p.gate;
    return e;
  };
  if (p.precond) {
    EpiArgs e{};
    e.kind = 1;
    e.alpha = 1.0;
    e.alpha_dev = p.in_scale;
    e.lam = cd.lam;
    e.scale = p.rho0 / cd.hx;
    e.sx = g.sx;
    gemm<R>(mat<R>(cd, CH_VT), nz, (const R*)v, n, (R*)wY, n, nz, n, nz, gated(e), st);              // diag * V^T v
    gemm<R>(mat<R>(cd, CH_PRE_V), 2 * nz, (const R*)wY, n, T, n, 2 * nz, n, nz, gated(plain()), st);  // [I V; G V]
  } else {
    gemm<R>(mat<R>(cd, CH_PRE), 2 * nz, (const R*)v, n, T, n, 2 * nz, n, nz, gated(plain(1.0, p.in_scale)),
            st);  // [I; G]
  }
  // x pass over the 2 nz rows: field 0 (I u) gets i k'_x in and out, field 1 (G u) plain
  row_pass_p2<R>(g, T, T + fs, coef, twtab, st, prof, p.gate);
  gemm<R>(mat<R>(cd, CH_POST), 2 * nz, T, n, (R*)y, n, nz, n, 2 * nz, gated(plain()), st);  // [-I^T | G^T]
}

template <typename R>
void c2_precond(const Geom& g, const ChebDev& cd, double rho0, const void* r, void* z, void* wY, hipStream_t st,
                const int* gate) {
  const int nz = g.nz, n = 2 * g.M;
  EpiArgs e{};
  e.kind = 1;
  e.alpha = 1.0;
  e.lam = cd.lam;
  e.scale = rho0 / cd.hx;
  e.sx = g.sx;
  e.gate = gate;
  EpiArgs e2 = plain();
  e2.gate = gate;
  gemm<R>(mat<R>(cd, CH_VT), nz, (const R*)r, n, (R*)wY, n, nz, n, nz, e, st);
  gemm<R>(mat<R>(cd, CH_V), nz, (const R*)wY, n, (R*)z, n, nz, n, nz, e2, st);
}

template <typename R>
void c2_to_eigen(const Geom& g, const ChebDev& cd, const void* r, void* rt, hipStream_t st) {
  const int nz = g.nz, n = 2 * g.M;
  gemm<R>(mat<R>(cd, CH_VT), nz, (const R*)r, n, (R*)rt, n, nz, n, nz, plain(), st);
}
template <typename R>
void c2_from_eigen(const Geom& g, const ChebDev& cd, const void* xt, void* x, hipStream_t st) {
  const int nz = g.nz, n = 2 * g.M;
  gemm<R>(mat<R>(cd, CH_V), nz, (const R*)xt, n, (R*)x, n, nz, n, nz, plain(), st);
}
template <typename R>
void c2_apply_eigen(const Geom& g, const ChebDev& cd, const void* pt, void* qq, void* wT, const void* coef,
                    const void* twtab, hipStream_t st, Prof* prof, const int* gate) {
  const int nz = g.nz, n = 2 * g.M;
  R* T = (R*)wT;  // [2 nz][n]
  EpiArgs e = plain();
  e.gate = gate;
  gemm<R>(mat<R>(cd, CH_PRE_V), 2 * nz, (const R*)pt, n, T, n, 2 * nz, n, nz, e, st);  // [I V; G V]
  row_pass_p2<R>(g, T, T + (size_t)nz * n, coef, twtab, st, prof, gate);
  gemm<R>(mat<R>(cd, CH_POST), 2 * nz, T, n, (R*)qq, n, 2 * nz, n, 2 * nz, e, st);  // [Q; V^T Q]
}

void c2_rhs(const Geom& g, const ChebDev& cd, const void* fhat, void* b, hipStream_t st) {
  const int nz = g.nz, n = 2 * g.M;
  gemm<double>(cd.m64[CH_RHS], nz, (const double*)fhat, n, (double*)b, n, nz, n, nz, plain(), st);
}

// rho_L = I rho, coef = h_x w_LGL / rho_L (FP64 and FP32), bad-count
__global__ void k_c2_coef(const double* __restrict__ rhoL, const double* __restrict__ wl, double hx, int nz, int n,
                          double* __restrict__ c64, float* __restrict__ c32, int* bad) {
  size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)nz * n) return;
  const int j = (int)(e / n);
  const double r = rhoL[e];
  if (!(r > 0.0) || !isfinite(r)) atomicAdd(bad, 1);
  const double c = hx * wl[j] / r;
  c64[e] = c;
  c32[e] = (float)c;
}

void c2_density(const Geom& g, const ChebDev& cd, const double* rho, double* rhoL, double* c64, float* c32, int* bad,
                hipStream_t st) {
  const int nz = g.nz, n = 2 * g.M;
  gemm<double>(cd.m64[CH_I], nz, rho, n, rhoL, n, nz, n, nz, plain(), st);
  const size_t tot = (size_t)nz * n;
  hipLaunchKernelGGL(k_c2_coef, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, rhoL, cd.wl, cd.hx, nz, n,
                     c64, c32, bad);
}

// Remove the z-mean of the real and imaginary parts of the kx = 0 slot
// (the constant and the alternating-in-x modes, constant in z); removed
// physical norm to *removed.
__global__ void k_c2_project(C2<double>* __restrict__ s, int nz, int M, double inv_nx, double* removed) {
  __shared__ double sr[256], si[256];
  double a = 0, b = 0;
  for (int j = threadIdx.x; j < nz; j += 256) {
    C2<double> v = s[(size_t)j * M];
    a += v.x;
    b += v.y;
  }
  sr[threadIdx.x] = a;
  si[threadIdx.x] = b;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      sr[threadIdx.x] += sr[threadIdx.x + o];
      si[threadIdx.x] += si[threadIdx.x + o];
    }
    __syncthreads();
  }
  const double mr = sr[0] / nz, mi = si[0] / nz;
  for (int j = threadIdx.x; j < nz; j += 256) {
    C2<double> v = s[(size_t)j * M];
    s[(size_t)j * M] = C2<double>{v.x - mr, v.y - mi};
  }
  if (threadIdx.x == 0 && removed) *removed = sqrt((double)nz * (mr * mr + mi * mi) * inv_nx);
}

void c2_project(const Geom& g, void* spec, double* removed, hipStream_t st) {
  hipLaunchKernelGGL(k_c2_project, dim3(1), dim3(256), 0, st, (C2<double>*)spec, g.nz, g.M, g.ntot_inv, removed);
}

extern "C" vd_status vd_dense_matmul(int precision, const void* A, const void* B, void* C, int M, int N, int K,
                                     hipStream_t stream) {
  if (!A || !B || !C || M < 1 || N < 1 || K < 1) return VD_EINVAL;
  if (precision == VD_FP64) gemm_plain<double>(A, B, C, M, N, K, stream);
  else if (precision == VD_FP32_REFINE) gemm_plain<float>(A, B, C, M, N, K, stream);
  else return VD_EINVAL;
  if (hipStreamSynchronize(stream) != hipSuccess) return VD_EDEVICE;
  return hipGetLastError() == hipSuccess ? VD_OK : VD_EDEVICE;
}

template void gemm_plain<double>(const void*, const void*, void*, int, int, int, hipStream_t);
template void gemm_plain<float>(const void*, const void*, void*, int, int, int, hipStream_t);
template void c2_apply<double>(const Geom&, const ChebDev&, const OpParams&, const void*, void*, void*, void*,
                               const void*, const void*, hipStream_t, Prof*);
template void c2_apply<float>(const Geom&, const ChebDev&, const OpParams&, const void*, void*, void*, void*,
                              const void*, const void*, hipStream_t, Prof*);
#define VD_EIGEN(R)                                                                                      \
  template void c2_to_eigen<R>(const Geom&, const ChebDev&, const void*, void*, hipStream_t);            \
  template void c2_from_eigen<R>(const Geom&, const ChebDev&, const void*, void*, hipStream_t);          \
  template void c2_apply_eigen<R>(const Geom&, const ChebDev&, const void*, void*, void*, const void*,   \
                                  const void*, hipStream_t, Prof*, const int*);
VD_EIGEN(double)
VD_EIGEN(float)
template void c2_precond<double>(const Geom&, const ChebDev&, double, const void*, void*, void*, hipStream_t,
                                 const int*);
template void c2_precond<float>(const Geom&, const ChebDev&, double, const void*, void*, void*, hipStream_t,
                                const int*);

}  // namespace vd

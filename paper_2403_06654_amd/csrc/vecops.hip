// Krylov vector algebra and scalar recurrences (gfx950).
//
// Vector kernels stream packed spectral fields with grid-stride loops over a
// fixed number of blocks; reductions accumulate in FP64 whatever the vector
// precision, reduce within the block in a fixed tree (wave shuffles, then
// LDS across the four waves) and finish in a single-block kernel that adds
// the per-block partials in block order.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include "gs_device.hpp"
#include "spectral.hpp"
#include "vecops.hpp"

namespace vd {

constexpr int kRedStride = kMaxVec + 2;

size_t nred_partial() { return (size_t)kRedBlocks * kRedStride; }

// Blocks of the streaming and reduction kernels: 4 per CU for large fields,
// fewer for small ones (at least 1024 elements per block) so that small
// problems do not pay for empty blocks and long partial reductions.  A pure
// function of the field size: results stay bitwise reproducible.
static int nblk(size_t n) {
  size_t b = (n + 1023) / 1024;
  return (int)(b < 1 ? 1 : (b > (size_t)kRedBlocks ? kRedBlocks : b));
}

// Reduce acc[0..K) across a 256-thread block; value i of block b goes to
// partial[i * kRedBlocks + b] (callers pass partial + b), so that the final
// reduction reads each value's block partials contiguously.
template <int K>
__device__ __forceinline__ void block_store(const double* acc, int k_used, double* partial) {
  __shared__ double sh[4][K > 0 ? K : 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < K; ++i) {
    if (i < k_used) {
      double v = wave_sum(acc[i]);
      if (lane == 0) sh[w][i] = v;
    }
  }
  __syncthreads();
  if (threadIdx.x < k_used) {
    int i = threadIdx.x;
    partial[(size_t)i * kRedBlocks] = ((sh[0][i] + sh[1][i]) + sh[2][i]) + sh[3][i];
  }
}

// M (half the x length) is a power of two for every grid (Fourier axes are
// powers of two), so the kx = 0 test is a mask, not a 64-bit division
__device__ __forceinline__ double spec_w(size_t e, int M) { return (e & (size_t)(M - 1)) == 0 ? 1.0 : 2.0; }

// One wave per output value (a 1024-thread block).  No block-wide barrier.
__device__ __forceinline__ void reduce_values(const double* __restrict__ partial, int nblk, int K, double scale,
                                              double* __restrict__ out) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int i = w; i < K; i += 16) {
    const double v = sum_partials(partial + (size_t)i * kRedBlocks, nblk);
    if (lane == 0) out[i] = v * scale;
  }
}

// The final reduction, optionally followed (same launch, after a block
// barrier) by the scalar step that consumes its result: one launch less per
// step than a separate one-thread kernel.  The step takes the reduced values
// from LDS, not from out: out is written by other lanes (other waves for the
// second value) in this launch, and a load of it through st is not ordered
// after those stores (the compiler may serve it from the scalar cache).
__global__ __launch_bounds__(1024) void k_reduce(const double* __restrict__ partial, int nblk, int K, double scale,
                                                 double* __restrict__ out, const int* __restrict__ gate, int post,
                                                 DevState* st, unsigned long long seq) {
  if (gate && *gate) return;
  __shared__ double val[2];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  RecState rs{};
  if (post != POST_NONE) rs = rec_state(st);
  for (int i = w; i < K; i += 16) {
    const double v = sum_partials(partial + (size_t)i * kRedBlocks, nblk) * scale;
    if (lane == 0) {
      out[i] = v;
      if (i < 2) val[i] = v;
    }
  }
  if (post == POST_NONE) return;
  __syncthreads();
  if (threadIdx.x) return;
  if (post == POST_CG_BETA) cg_beta_step(st, rs, val[0]);
  else if (post == POST_RMR_ALPHA) rmr_alpha_step(st, val[0], val[1]);
  else if (post == POST_REC_CHECK) rec_check_step(st, rs, val[0]);
  else if (post == POST_CG_STEP) {
    if (!rec_check_step(st, rs, val[0])) cg_beta_step(st, rs, val[1]);
  }
  else if (post == POST_MAIL) post_mail(rs.mail + MAIL_VALUE, val[0], 0.0, 0, seq);
}

// gate (here and below): optional device flag; when nonzero the launch does
// nothing (a Krylov step queued past the end of its run)
static void reduce(const double* partial, int nb, int K, double scale, double* out, hipStream_t s,
                   const int* gate = nullptr, const Post& post = Post{}) {
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(1024), 0, s, partial, nb, K, scale, out, gate, post.op, post.st,
                     post.seq);
}

static size_t nspec(const Geom& g) { return (size_t)g.nz * g.ny * g.M; }

// ------------------------------------------------------------ multi-dot

// The Gram-Schmidt kernels (and the dot pass) serve several independent
// systems in one launch (the components of a velocity solve): blockIdx.y
// selects system k of the set, with its own vector, basis, device state,
// partials and gate; one system is a set of one.
template <typename R>
struct SysSet {
  C2<R>* x[kMaxBatch];
  VecPtrs V[kMaxBatch];
  DevState* st[kMaxBatch];
  double* partial[kMaxBatch];
  const int* gate[kMaxBatch];
};

template <typename R, int NV>
__global__ __launch_bounds__(256) void k_mdot(SysSet<R> S, int nv, int want_norm, size_t n, int M) {
  const int sy = blockIdx.y;
  const int* gate = S.gate[sy];
  if (gate && *gate) return;
  const C2<R>* __restrict__ x = S.x[sy];
  const VecPtrs& V = S.V[sy];
  double* __restrict__ partial = S.partial[sy];
  double acc[NV + 1];
#pragma unroll
  for (int i = 0; i <= NV; ++i) acc[i] = 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    // Each vector's load is consumed at once (the compiler then waits for it
    // before the next), which keeps the kernel near 55 VGPRs and 7 waves per
    // SIMD.  Measured on MI355X at 256^3 FP64: loading all vectors first
    // (112 VGPRs, 4 waves) ran 4% slower, and splitting the vectors over the
    // block's wavefronts 1.5% slower.
    C2<R> xv = ldg(x + e);
    const double w = spec_w(e, M);
    const double xr = xv.x, xi = xv.y;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (i < nv) {
        C2<R> v = ldg((const C2<R>*)V.p[i] + e);
        acc[i] += w * ((double)v.x * xr + (double)v.y * xi);
      }
    }
    if (want_norm) acc[NV] += w * (xr * xr + xi * xi);
  }
  double out[NV + 1];
#pragma unroll
  for (int i = 0; i <= NV; ++i) out[i] = acc[i];
  // move the norm next to the used dots
#pragma unroll
  for (int i = 0; i < NV; ++i)
    if (i == nv) out[i] = acc[NV];
  block_store<NV + 1>(out, nv + (want_norm ? 1 : 0), partial + blockIdx.x);
}

template <typename R>
static SysSet<R> one_system(const void* x, const VecPtrs& V, DevState* st, double* partial, const int* gate) {
  SysSet<R> S{};
  S.x[0] = (C2<R>*)x;
  S.V[0] = V;
  S.st[0] = st;
  S.partial[0] = partial;
  S.gate[0] = gate;
  return S;
}

// Block partials only (the caller reduces them), for nsys systems.
template <typename R>
static void mdot_partials_set(const Geom& g, const SysSet<R>& S, int nsys, int nv, bool want_norm, hipStream_t s) {
  size_t n = nspec(g);
  dim3 gr(nblk(n), nsys), bl(256);
  const int wn = want_norm ? 1 : 0;
  if (nv <= 1) hipLaunchKernelGGL((k_mdot<R, 1>), gr, bl, 0, s, S, nv, wn, n, g.M);
  else if (nv <= 2) hipLaunchKernelGGL((k_mdot<R, 2>), gr, bl, 0, s, S, nv, wn, n, g.M);
  else if (nv <= 4) hipLaunchKernelGGL((k_mdot<R, 4>), gr, bl, 0, s, S, nv, wn, n, g.M);
  else if (nv <= 8) hipLaunchKernelGGL((k_mdot<R, 8>), gr, bl, 0, s, S, nv, wn, n, g.M);
  else if (nv <= 16) hipLaunchKernelGGL((k_mdot<R, 16>), gr, bl, 0, s, S, nv, wn, n, g.M);
  else if (nv <= 24) hipLaunchKernelGGL((k_mdot<R, 24>), gr, bl, 0, s, S, nv, wn, n, g.M);
  else hipLaunchKernelGGL((k_mdot<R, kMaxVec>), gr, bl, 0, s, S, nv, wn, n, g.M);
}

template <typename R>
static void mdot_partials(const Geom& g, const void* x, const VecPtrs& V, int nv, bool want_norm, double* partial,
                          hipStream_t s, const int* gate = nullptr) {
  mdot_partials_set<R>(g, one_system<R>(x, V, nullptr, partial, gate), 1, nv, want_norm, s);
}


template <typename R>
void mdot(const Geom& g, const void* x, const VecPtrs& V, int nv, bool want_norm, double* partial, double* out,
          hipStream_t s, Prof* prof, const int* gate, const Post& post) {
  mdot_partials<R>(g, x, V, nv, want_norm, partial, s, gate);
  if (prof) prof->end(s);
  reduce(partial, nblk(nspec(g)), nv + (want_norm ? 1 : 0), g.ntot_inv, out, s, gate, post);
}

// ------------------------------------------------ Gram-Schmidt (GMRES)
//
// Basis vectors are stored unnormalised with a scale vs[i] (v_i = vs[i] *
// V_i); every consumer folds the scale into its coefficients, and the
// operator takes it as an input scale, so no pass is spent on normalising.
// One Arnoldi step (w = A M^-1 v_j, nv = j + 1):
//   pass 1  k_mdot:      raw_i = (V_i, w)                         h_i = vs_i raw_i
//   pass 2  k_gs_update: w' = w - sum_i h_i v_i, and in the same pass the
//                        dots c_i = (v_i, w') and ||w'||^2
//   check   c measures the orthogonality actually lost by classical
//           Gram-Schmidt; if max|c_i| <= tol ||w'|| the step is done
//           (H[:, j] = h, H[j+1, j] = ||w'||), else
//   pass 3  w'' = w' - sum_{i in S} c_i v_i over the set S of components
//           with |c_i| > tol ||w'|| (the others already meet the test),
//           H[:, j] = h + c_S, ||w''||^2 = ||w'||^2 - |c_S|^2, accurate
//           because |c| << ||w'||.  It reads only the vectors in S.
// Pass 3 exits at once when not needed, so the common step costs two
// passes over the basis.

// The scalar steps below run in the block that finishes the cross-block
// reduction of the pass before them (one launch instead of two).  Reduced
// values stay in LDS; per-vector work runs one lane per basis vector
// (nv <= kMaxVec < 64), so no thread walks the device state serially.
// blockIdx.y: the system (st[k], partial[k]) of a set
__global__ __launch_bounds__(1024) void k_gs_prep(DevStates S, int nv, int nb, double scale) {
  DevState* st = S.st[blockIdx.y];
  const double* __restrict__ partial = S.partial[blockIdx.y];
  if (st->halt) return;
  __shared__ double val[kMaxVec + 2];
  reduce_values(partial, nb, nv, scale, val);
  __syncthreads();
  const int i = threadIdx.x;
  if (i < nv) {
    const double v = st->vs[i], h = v * val[i];
    st->red2[i] = val[i];
    st->hcol[i] = h;
    st->coef[i] = h * v;
  }
}

__global__ __launch_bounds__(1024) void k_gs_check(DevStates S, int nv, double tol, int nb, double scale) {
  DevState* st = S.st[blockIdx.y];
  const double* __restrict__ partial = S.partial[blockIdx.y];
  __shared__ double val[kMaxVec + 2];
  if (st->halt) {  // a step queued past the end of the cycle: no second pass either
    if (threadIdx.x == 0) st->reorth = 0;
    return;
  }
  const GsState gs = gs_state(st, nv, true);
  reduce_values(partial, nb, nv + 1, scale, val);
  __syncthreads();
  if (threadIdx.x >= 64) return;  // one wavefront from here on
  gs_end(st, gs, gs_check(gs, val, nv, tol), val, nv);
}

template <typename R, int NV>
__global__ __launch_bounds__(256) void k_gs_update(SysSet<R> S, int nv, size_t n, int M) {
  // systems in reverse order and each swept last row first, so that the
  // pass starts on what the dot pass read last (ascending systems and rows),
  // still in the Infinity Cache
  const int sy = (int)(gridDim.y - 1 - blockIdx.y);
  const DevState* __restrict__ st = S.st[sy];
  if (st->halt) return;
  C2<R>* __restrict__ x = S.x[sy];
  const VecPtrs& V = S.V[sy];
  double* __restrict__ partial = S.partial[sy];
  double c[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) c[i] = i < nv ? st->coef[i] : 0.0;
  double acc[NV + 1];
#pragma unroll
  for (int i = 0; i <= NV; ++i) acc[i] = 0.0;
  // Same elements per thread as the dot pass, visited in the opposite order:
  // the dot pass ends on the top of every vector, which is then still in the
  // Infinity Cache (measured 299 -> 294 us at 256^3 FP64, 13 streams).
  const size_t stride = (size_t)gridDim.x * 256, e0 = (size_t)blockIdx.x * 256 + threadIdx.x;
  for (size_t k = (n + stride - 1) / stride; k-- > 0;) {
    const size_t e = k * stride + e0;
    if (e >= n) continue;
    C2<R> vv[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (i < nv) vv[i] = ldg((const C2<R>*)V.p[i] + e);
    C2<R> xv = ldg(x + e);
    double xr = xv.x, xi = xv.y;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (i < nv) {
        xr -= c[i] * (double)vv[i].x;
        xi -= c[i] * (double)vv[i].y;
      }
    }
    C2<R> nx{R(xr), R(xi)};
    stg(x + e, nx);
    const double w = spec_w(e, M);
    const double yr = nx.x, yi = nx.y;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (i < nv) acc[i] += w * ((double)vv[i].x * yr + (double)vv[i].y * yi);
    acc[NV] += w * (yr * yr + yi * yi);
  }
  double out[NV + 1];
#pragma unroll
  for (int i = 0; i <= NV; ++i) out[i] = acc[i];
#pragma unroll
  for (int i = 0; i <= NV; ++i)
    if (i == nv) out[i] = acc[NV];
  block_store<NV + 1>(out, nv + 1, partial + blockIdx.x);
}

// The second pass is its own kernel symbol so that profiles separate it.
template <typename R, int NV>
__global__ __launch_bounds__(256) void k_gs_reorth(SysSet<R> S, int nv, size_t n) {
  const int sy = blockIdx.y;
  const DevState* __restrict__ st = S.st[sy];
  if (!st->reorth) return;
  C2<R>* __restrict__ x = S.x[sy];
  const VecPtrs& V = S.V[sy];
  double c[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) c[i] = i < nv ? st->coef[i] : 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    C2<R> xv = ldg(x + e);
    double xr = xv.x, xi = xv.y;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (i < nv && c[i] != 0.0) {  // uniform: vectors that passed the check are not read
        C2<R> v = ldg((const C2<R>*)V.p[i] + e);
        xr -= c[i] * (double)v.x;
        xi -= c[i] * (double)v.y;
      }
    }
    stg(x + e, C2<R>{R(xr), R(xi)});
  }
}

// ---- The same step on small fields: three launches instead of five.
//
// Up to kFoldElems elements (64^3, 512^2) a step moves a few MB that sit in
// the caches, and its time is launches and dependent load latencies.  So a
// block takes 256 elements, its wavefronts split the vectors between them (H
// groups of four wavefronts, NVH vectors each) and every thread has all its
// loads in flight at once.  The blocks are few enough (kFoldBlocks) that each
// block of the update and of the second pass reduces all the block partials
// of the pass before it by itself, some KB from L2, instead of waiting for a
// launch that does so: k_gs_prep runs inside k_gs_update_s, and k_gs_check
// with the second pass inside k_gs_finish (block 0 writes the state).  Larger
// fields keep the kernels above: they are bound by the basis stream, and their
// up to 1024 partials per value are too many to reduce in every block.
// Of an FP64 or FP32 pressure step on a Fourier grid only the update is left here:
// the operator's last pass forms the dots and the next step's first pass takes
// the check (op_carries_gs).  The dots and the check dots alternate between two
// halves of each partial row, because blocks of one launch read the first while others write the second.
// Measured per launch, before -> now (rocprofv3, median over a solve):
//   32^3 FP64, 9-16 vectors: dots 14.6 -> 4.3 us, update with k_gs_prep 12.2 +
//     3.8 -> 5.7 us, check with second pass 4.6 + 1.7 -> 6.1 us;
//   101 x 64 slots FP32, 5-8 vectors: 9.1 -> 3.8, 7.6 + 1.8 -> 5.0 and
//     3.9 + 1.8 -> 4.6 us.
static bool folds(size_t n) { return n <= kFoldElems; }
static int fold_blocks(size_t n) { return (int)std::min<size_t>((n + 255) / 256, kFoldBlocks); }

// val[0..K) = the sums of the block partials (nb <= kFoldBlocks each), by all
// NW wavefronts of the block; ends with a block barrier.
template <int KMAX, int NW>
__device__ __forceinline__ void fold_reduce(const double* __restrict__ partial, int nb, int K, double scale,
                                            double* val) {
  constexpr int PW = (KMAX + NW - 1) / NW, Q = kFoldBlocks / 64;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double v[PW];
#pragma unroll
  for (int p = 0; p < PW; ++p) {
    v[p] = 0.0;
    const int i = w + NW * p;
    if (i < K) {
      const double* src = partial + (size_t)i * kRedBlocks;
      double t[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) t[q] = lane + 64 * q < nb ? src[lane + 64 * q] : 0.0;
#pragma unroll
      for (int q = 0; q < Q; ++q) v[p] += t[q];
    }
  }
#pragma unroll
  for (int p = 0; p < PW; ++p) {
    const double t = wave_sum(v[p]);
    if (lane == 0 && w + NW * p < K) val[w + NW * p] = t * scale;
  }
  __syncthreads();
}

// Dots of split h's vectors (acc), and with NORM split 0's acc[NVH], to the
// block partials of this block (value nv: the norm).
template <int NVH, int H, bool NORM>
__device__ __forceinline__ void fold_store(const double* acc, int nv, double* partial) {
  constexpr int K = NVH + (NORM ? 1 : 0);
  __shared__ double sh[4 * H][K];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < K; ++q) {
    const double t = wave_sum(acc[q]);
    if (lane == 0) sh[w][q] = t;
  }
  __syncthreads();
  const int i = threadIdx.x;
  if (i < nv + (NORM ? 1 : 0)) {
    const int h = i == nv ? 0 : i / NVH, q = i == nv ? NVH : i - h * NVH;
    const double(*p)[K] = sh + 4 * h;
    partial[(size_t)i * kRedBlocks + blockIdx.x] = ((p[0][q] + p[1][q]) + p[2][q]) + p[3][q];
  }
}

template <typename R, int NVH, int H>
__global__ __launch_bounds__(256 * H) void k_mdot_s(SysSet<R> S, int nv, size_t n, int M) {
  const int sy = blockIdx.y;
  const int* gate = S.gate[sy];
  if (gate && *gate) return;
  const C2<R>* __restrict__ x = S.x[sy];
  const int i0 = NVH * __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);  // the split's first vector
  const void* const* V = S.V[sy].p + i0;
  const int nvh = nv - i0;
  double acc[NVH];
#pragma unroll
  for (int i = 0; i < NVH; ++i) acc[i] = 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + (threadIdx.x & 255); e < n; e += (size_t)gridDim.x * 256) {
    C2<R> vv[NVH];
    const C2<R> xv = ldg(x + e);
#pragma unroll
    for (int i = 0; i < NVH; ++i)
      if (i < nvh) vv[i] = ldg((const C2<R>*)V[i] + e);
    const double w = spec_w(e, M);
    const double xr = xv.x, xi = xv.y;
#pragma unroll
    for (int i = 0; i < NVH; ++i)
      if (i < nvh) acc[i] += w * ((double)vv[i].x * xr + (double)vv[i].y * xi);
  }
  fold_store<NVH, H, false>(acc, nv, S.partial[sy]);
}

// w' = w - sum_i h_i v_i with its check dots; the dots of k_mdot_s are reduced
// here.  Every split forms its part of the sum; they meet in LDS.
template <typename R, int NVH, int H>
__global__ __launch_bounds__(256 * H) void k_gs_update_s(SysSet<R> S, int nv, size_t n, int M, double scale, int nbd) {
  const int sy = blockIdx.y;
  DevState* st = S.st[sy];
  if (st->halt) return;
  C2<R>* __restrict__ x = S.x[sy];
  double* partial = S.partial[sy];
  __shared__ double val[NVH * H], cl[NVH * H];
  __shared__ C2<double> part[H > 1 ? H : 1][H > 1 ? 256 : 1];
  const int h = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), i0 = NVH * h, te = threadIdx.x & 255;
  const void* const* V = S.V[sy].p + i0;
  const int nvh = nv - i0;
  const size_t stride = (size_t)gridDim.x * 256, b0 = (size_t)blockIdx.x * 256;
  C2<R> vv[NVH], xv;
  auto load = [&](size_t e) {
    xv = C2<R>{R(0), R(0)};
#pragma unroll
    for (int i = 0; i < NVH; ++i) vv[i] = C2<R>{R(0), R(0)};
    if (e >= n) return;
    xv = ldg(x + e);
#pragma unroll
    for (int i = 0; i < NVH; ++i)
      if (i < nvh) vv[i] = ldg((const C2<R>*)V[i] + e);
  };
  load(b0 + te);  // the first elements' loads overlap the reduction
  fold_reduce<NVH * H, 4 * H>(partial, nbd, nv, scale, val);  // nbd blocks formed the dots
  if ((int)threadIdx.x < NVH * H) {
    const int i = threadIdx.x;
    double c = 0.0;
    if (i < nv) {
      const double v = st->vs[i], hh = v * val[i];
      c = hh * v;
      if (blockIdx.x == 0) {
        st->red2[i] = val[i];
        st->hcol[i] = hh;
      }
    }
    cl[i] = c;
  }
  __syncthreads();
  double acc[NVH + 1];
#pragma unroll
  for (int i = 0; i <= NVH; ++i) acc[i] = 0.0;
  for (size_t b = b0; b < n; b += stride) {  // the same trips for every thread of the block
    const size_t e = b + te;
    if (b != b0) load(e);
    double sr = 0.0, si = 0.0;
#pragma unroll
    for (int i = 0; i < NVH; ++i) {
      const double c = cl[i0 + i];
      sr += c * (double)vv[i].x;
      si += c * (double)vv[i].y;
    }
    if constexpr (H > 1) {
      if (b != b0) __syncthreads();  // the last trip's sums have been read
      part[h][te] = C2<double>{sr, si};
      __syncthreads();
      sr = si = 0.0;
#pragma unroll
      for (int q = 0; q < H; ++q) {
        sr += part[q][te].x;
        si += part[q][te].y;
      }
    }
    const C2<R> nx{R((double)xv.x - sr), R((double)xv.y - si)};
    // every split has loaded this x before the barrier above
    if (h == 0 && e < n) stg(x + e, nx);
    const double w = spec_w(e, M);
    const double yr = nx.x, yi = nx.y;
#pragma unroll
    for (int i = 0; i < NVH; ++i) acc[i] += w * ((double)vv[i].x * yr + (double)vv[i].y * yi);
    acc[NVH] += w * (yr * yr + yi * yi);  // 0 past the end
  }
  fold_store<NVH, H, true>(acc, nv, partial + kFoldHalf);
}

// The orthogonality check in every block, the second pass over the vectors
// that failed it, and in block 0 the Givens rotations and the stopping test.
// (A block that sees the halt flag of block 0 skips its part of the second
// pass: the vector that ends a cycle is never read.)
template <typename R, int NV>
__global__ __launch_bounds__(256) void k_gs_finish(SysSet<R> S, int nv, size_t n, double tol, double scale) {
  const int sy = blockIdx.y;
  DevState* st = S.st[sy];
  __shared__ double val[NV + 1], cl[NV];
  __shared__ int again, halted;
  GsState gs{};
  if (threadIdx.x < 64) gs = gs_state(st, nv, blockIdx.x == 0);
  if (threadIdx.x == 0) halted = halt_now(&st->halt);
  fold_reduce<NV + 1, 4>(S.partial[sy] + kFoldHalf, gridDim.x, nv + 1, scale, val);  // ends with a barrier
  if (halted) return;
  GsCheck k{};
  if (threadIdx.x < 64) {
    k = gs_check(gs, val, nv, tol);
    if ((int)threadIdx.x < nv) cl[threadIdx.x] = k.csel * k.v;
    if (threadIdx.x == 0) again = !k.orth;
  }
  __syncthreads();
  if (again) {
    C2<R>* __restrict__ x = S.x[sy];
    const VecPtrs& V = S.V[sy];
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
      const C2<R> xv = ldg(x + e);
      double xr = xv.x, xi = xv.y;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        if (i < nv && cl[i] != 0.0) {
          const C2<R> v = ldg((const C2<R>*)V.p[i] + e);
          xr -= cl[i] * (double)v.x;
          xi -= cl[i] * (double)v.y;
        }
      }
      stg(x + e, C2<R>{R(xr), R(xi)});
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < 64) gs_end(st, gs, k, val, nv);
}

template <typename R, int NVH, int H>
static void launch_gs_small(const Geom& g, const SysSet<R>& S, int nsys, int nv, const GsParts& parts, hipStream_t s,
                            Prof* prof) {
  const size_t n = nspec(g);
  const dim3 gr(fold_blocks(n), nsys);
  const bool pr = prof && prof->on;
  const double fb = (double)n * sizeof(C2<R>) * nsys;
  if (parts.dot_blocks == 0) {
    if (pr) prof->begin(10, s, (nv + 1) * fb);
    hipLaunchKernelGGL((k_mdot_s<R, NVH, H>), gr, dim3(256 * H), 0, s, S, nv, n, g.M);
    if (pr) prof->end(s);
  } else if (pr) {
    prof->tally(10);
  }
  if (pr) prof->begin(11, s, (nv + 2) * fb);
  hipLaunchKernelGGL((k_gs_update_s<R, NVH, H>), gr, dim3(256 * H), 0, s, S, nv, n, g.M, g.ntot_inv,
                     parts.dot_blocks ? parts.dot_blocks : (int)gr.x);
  if (pr) prof->end(s);
  if (parts.finish)
    hipLaunchKernelGGL((k_gs_finish<R, NVH * H < kMaxVec ? NVH * H : kMaxVec>), gr, dim3(256), 0, s, S, nv, n,
                       orth_tol<R>(), g.ntot_inv);
}
int gs_update_blocks(const Geom& g) { return fold_blocks(nspec(g)); }

template <typename R, int NV>
static void launch_gs(const Geom& g, const SysSet<R>& S, int nsys, int nv, int second, hipStream_t s) {
  const dim3 gr(nblk(nspec(g)), nsys);
  if (second) hipLaunchKernelGGL((k_gs_reorth<R, NV>), gr, dim3(256), 0, s, S, nv, nspec(g));
  else hipLaunchKernelGGL((k_gs_update<R, NV>), gr, dim3(256), 0, s, S, nv, nspec(g), g.M);
}

// One Arnoldi orthogonalisation for nsys independent systems at the same
// step (nv basis vectors each); each system's kernels return at once once
// its own halt flag is set.
template <typename R>
static void gs_orthogonalize_set(const Geom& g, const SysSet<R>& S, int nsys, int nv, const GsParts& parts,
                                 hipStream_t s, Prof* prof) {
  if (folds(nspec(g))) {
    if (nv <= 4) launch_gs_small<R, 4, 1>(g, S, nsys, nv, parts, s, prof);
    else if (nv <= 8) launch_gs_small<R, 8, 1>(g, S, nsys, nv, parts, s, prof);
    else if (nv <= 16) launch_gs_small<R, 8, 2>(g, S, nsys, nv, parts, s, prof);
    else if (nv <= 24) launch_gs_small<R, 8, 3>(g, S, nsys, nv, parts, s, prof);
    else launch_gs_small<R, 9, 4>(g, S, nsys, nv, parts, s, prof);
    return;
  }
  const bool pr = prof && prof->on;
  const double fb = (double)nspec(g) * sizeof(C2<R>) * nsys;
  if (pr) prof->begin(10, s, (nv + 1) * fb);
  const int nb = nblk(nspec(g));
  mdot_partials_set<R>(g, S, nsys, nv, false, s);
  if (pr) prof->end(s);
  DevStates D{};
  for (int k = 0; k < nsys; ++k) {
    D.st[k] = S.st[k];
    D.partial[k] = S.partial[k];
  }
  hipLaunchKernelGGL(k_gs_prep, dim3(1, nsys), dim3(1024), 0, s, D, nv, nb, g.ntot_inv);
  for (int second = 0; second < 2; ++second) {
    if (pr && !second) prof->begin(11, s, (nv + 2) * fb);
    if (nv <= 4) launch_gs<R, 4>(g, S, nsys, nv, second, s);
    else if (nv <= 8) launch_gs<R, 8>(g, S, nsys, nv, second, s);
    else if (nv <= 16) launch_gs<R, 16>(g, S, nsys, nv, second, s);
    else if (nv <= 24) launch_gs<R, 24>(g, S, nsys, nv, second, s);
    else launch_gs<R, kMaxVec>(g, S, nsys, nv, second, s);
    if (pr && !second) prof->end(s);
    if (!second) hipLaunchKernelGGL(k_gs_check, dim3(1, nsys), dim3(1024), 0, s, D, nv, orth_tol<R>(), nb, g.ntot_inv);
  }
}

template <typename R>
void gs_orthogonalize(const Geom& g, void* w, const VecPtrs& V, int nv, DevState* st, double* partial,
                      hipStream_t s, Prof* prof, const GsParts& parts) {
  // the dot pass is gated by the system's halt flag like the other kernels
  gs_orthogonalize_set<R>(g, one_system<R>(w, V, st, partial, &st->halt), 1, nv, parts, s, prof);
}

template <typename R>
void gs_orthogonalize_batch(const Geom& g, void* const* w, const VecPtrs* V, int nv, DevState* const* st,
                            double* const* partial, int nsys, hipStream_t s, Prof* prof, const GsParts& parts) {
  SysSet<R> S{};
  for (int k = 0; k < nsys; ++k) {
    S.x[k] = (C2<R>*)w[k];
    S.V[k] = V[k];
    S.st[k] = st[k];
    S.partial[k] = partial[k];
    S.gate[k] = &st[k]->halt;
  }
  gs_orthogonalize_set<R>(g, S, nsys, nv, parts, s, prof);
}

// ------------------------------------------------------------- lincomb

// ALL: every vector's load in flight at once (small fields, latency-bound:
// 14.8 -> 6.3 us at 32^3 FP64, 18 vectors); otherwise each load is consumed at
// once (more wavefronts, for fields that stream from HBM).
template <typename R, int NV, bool ALL>
__global__ __launch_bounds__(256) void k_lincomb(C2<R>* __restrict__ z, VecPtrs V, int nv,
                                                 const double* __restrict__ coef, size_t n) {
  double c[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) c[i] = i < nv ? coef[i] : 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    double zr = 0.0, zi = 0.0;
    C2<R> vv[ALL ? NV : 1];
    if constexpr (ALL) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
        if (i < nv) vv[i] = ldg((const C2<R>*)V.p[i] + e);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (i < nv) {
        const C2<R> v = ALL ? vv[i] : ldg((const C2<R>*)V.p[i] + e);
        zr += c[i] * (double)v.x;
        zi += c[i] * (double)v.y;
      }
    }
    stg(z + e, C2<R>{R(zr), R(zi)});
  }
}

template <typename R, bool ALL>
static void launch_lincomb(const Geom& g, void* z, const VecPtrs& V, int nv, const double* coef, hipStream_t s) {
  const size_t n = nspec(g);
  const dim3 gr(ALL ? (unsigned)((n + 255) / 256) : (unsigned)nblk(n)), bl(256);
  if (nv <= 4) hipLaunchKernelGGL((k_lincomb<R, 4, ALL>), gr, bl, 0, s, (C2<R>*)z, V, nv, coef, n);
  else if (nv <= 16) hipLaunchKernelGGL((k_lincomb<R, 16, ALL>), gr, bl, 0, s, (C2<R>*)z, V, nv, coef, n);
  else hipLaunchKernelGGL((k_lincomb<R, kMaxVec, ALL>), gr, bl, 0, s, (C2<R>*)z, V, nv, coef, n);
}
template <typename R>
void lincomb(const Geom& g, void* z, const VecPtrs& V, int nv, const double* coef, hipStream_t s) {
  if (folds(nspec(g))) launch_lincomb<R, true>(g, z, V, nv, coef, s);
  else launch_lincomb<R, false>(g, z, V, nv, coef, s);
}

// ---------------------------------------------------------- elementwise

template <typename R>
__global__ __launch_bounds__(256) void k_scale(C2<R>* __restrict__ v, const double* __restrict__ sd, double sh,
                                               size_t n) {
  const R s = R((sd ? *sd : 1.0) * sh);
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256)
    stg(v + e, cscale(ldg(v + e), s));
}
template <typename R>
void scale(const Geom& g, void* v, const double* s_dev, double s_host, hipStream_t s) {
  hipLaunchKernelGGL((k_scale<R>), dim3(nblk(nspec(g))), dim3(256), 0, s, (C2<R>*)v, s_dev, s_host, nspec(g));
}

template <typename R>
__global__ __launch_bounds__(256) void k_sub_norm(const C2<R>* __restrict__ b, const C2<R>* __restrict__ q,
                                                  C2<R>* __restrict__ r, size_t n, int M,
                                                  double* __restrict__ partial) {
  double acc = 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    C2<R> bv = ldg(b + e), qv = ldg(q + e);
    C2<R> rv = bv - qv;
    stg(r + e, rv);
    acc += spec_w(e, M) * ((double)rv.x * rv.x + (double)rv.y * rv.y);
  }
  block_store<1>(&acc, 1, partial + blockIdx.x);
}
template <typename R>
void sub_norm(const Geom& g, const void* b, const void* q, void* r, double* partial, double* out, hipStream_t s,
              const Post& post) {
  hipLaunchKernelGGL((k_sub_norm<R>), dim3(nblk(nspec(g))), dim3(256), 0, s, (const C2<R>*)b, (const C2<R>*)q,
                     (C2<R>*)r, nspec(g), g.M, partial);
  reduce(partial, nblk(nspec(g)), 1, g.ntot_inv, out, s, nullptr, post);
}

template <typename R>
__global__ __launch_bounds__(256) void k_precond_axpy(C2<R>* x, const C2<R>* x_from, const C2<R>* __restrict__ z,
                                                      Geom g, int kind, double rho0, double nu, const double* ad, double ah,
                                                      size_t n, const int* __restrict__ gate) {
  if (gate && *gate) return;
  const double a = (ad ? *ad : 1.0) * ah;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    C2<R> mz = precond_at<R>(z, e, g, kind, rho0, nu);
    C2<R> xv = ldg(x_from + e);
    stg(x + e, C2<R>{R(xv.x + a * mz.x), R(xv.y + a * mz.y)});
  }
}
template <typename R>
void precond_axpy(const Geom& g, const OpParams& p, void* x, const void* z, const double* a_dev, double a_host,
                  hipStream_t s, const void* x_from) {
  hipLaunchKernelGGL((k_precond_axpy<R>), dim3(nblk(nspec(g))), dim3(256), 0, s, (C2<R>*)x,
                     (const C2<R>*)(x_from ? x_from : x), (const C2<R>*)z, g, p.precond ? p.kind : -1, p.rho0, p.nu, a_dev, a_host, nspec(g), p.gate);
}

template <typename R>
__global__ __launch_bounds__(256) void k_dot_rMr(const C2<R>* __restrict__ r, Geom g, int kind, double rho0,
                                                 double nu, size_t n, double* __restrict__ partial,
                                                 const int* __restrict__ gate) {
  if (gate && *gate) return;
  double acc = 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    C2<R> rv = ldg(r + e), mz = precond_at<R>(r, e, g, kind, rho0, nu);
    acc += spec_w(e, g.M) * ((double)rv.x * mz.x + (double)rv.y * mz.y);
  }
  block_store<1>(&acc, 1, partial + blockIdx.x);
}
template <typename R>
void dot_rMr(const Geom& g, const OpParams& p, const void* r, double* partial, double* out, hipStream_t s,
             const Post& post) {
  hipLaunchKernelGGL((k_dot_rMr<R>), dim3(nblk(nspec(g))), dim3(256), 0, s, (const C2<R>*)r, g,
                     p.precond ? p.kind : -1, p.rho0, p.nu, nspec(g), partial, p.gate);
  reduce(partial, nblk(nspec(g)), 1, g.ntot_inv, out, s, p.gate, post);
}

template <typename R>
void dot_partials(const Geom& g, const void* x, const void* v, bool want_norm, double* partial, hipStream_t s,
                  const int* gate) {
  VecPtrs P{};
  P.p[0] = v;
  mdot_partials<R>(g, x, P, 1, want_norm, partial, s, gate);
}

// alpha of a CG or RMR step from the block partials of its dots, by every block
// for itself (a few KB from L2; one launch less than reducing them first).
// Thread 0 of block 0 keeps the state.  Ends with a block barrier.
template <bool RMR>
__device__ __forceinline__ double step_alpha(DevState* st, const double* __restrict__ partial, int nb,
                                             double scale, int slot) {
  __shared__ double sh[2];
  const int w = threadIdx.x >> 6;
  if (w < (RMR ? 2 : 1)) {
    const double v = sum_partials(partial + (size_t)w * kRedBlocks, nb) * scale;
    if ((threadIdx.x & 63) == 0) sh[w] = v;
  }
  __syncthreads();
  double a;
  bool bad;
  if constexpr (RMR) {  // (r, w) / (w, w)
    a = sh[1] > 0.0 ? sh[0] / sh[1] : 0.0;
    bad = !isfinite(a);
  } else {  // rz / (p, A p)
    a = sh[0] != 0.0 ? st->rz[slot] / sh[0] : 0.0;
    bad = !isfinite(a) || sh[0] <= 0.0;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->alpha = a;
    if (bad) st->bad = 1;
  }
  return a;
}

// The new residual goes to another buffer: with the Helmholtz multipliers
// (r, M^-1 r) and M^-1 r need the mirror element of kx = 0 slots, which its own
// thread may already have updated in place.
// In place of k_cg_xr, k_dot_rMr and two reductions of their own (128^3 FP64:
// 15.6 + 8.4 + 2 x 4 us a step) this takes 18.6 us.
template <typename R, bool RMR>
__global__ __launch_bounds__(256) void k_rec_step(C2<R>* __restrict__ x, const C2<R>* __restrict__ r,
                                                  C2<R>* __restrict__ rnew, const C2<R>* __restrict__ p,
                                                  const C2<R>* __restrict__ q, DevState* st, Geom g, int kind,
                                                  double rho0, double nu, size_t n, double* partial, int nb,
                                                  double scale, int slot) {
  if (st->halt) return;
  const double a = step_alpha<RMR>(st, partial, nb, scale, slot);
  double acc[2] = {0.0, 0.0};
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    const C2<R> xv = ldg(x + e), rv = ldg(r + e), qv = ldg(q + e);
    const C2<R> d = RMR ? precond_at<R>(r, e, g, kind, rho0, nu) : ldg(p + e);
    stg(x + e, C2<R>{R(xv.x + a * d.x), R(xv.y + a * d.y)});
    const C2<R> nr{R(rv.x - a * qv.x), R(rv.y - a * qv.y)};
    stg(rnew + e, nr);
    const double w = spec_w(e, g.M);
    acc[0] += w * ((double)nr.x * nr.x + (double)nr.y * nr.y);
    if constexpr (!RMR) {
      C2<R> z = nr;
      if (kind >= 0) {
        const unsigned ue = (unsigned)e, u = ue / (unsigned)g.M;
        const int kx = (int)(ue - u * (unsigned)g.M);
        const int ky = (int)(u % (unsigned)g.ny), kz = (int)(u / (unsigned)g.ny);
        if (kind == OP_PRESSURE) {
          z = cscale(nr, mult_press<R>(kx, ky, kz, g, rho0));
        } else {
          const HelmMult<R> h = mult_helm<R>(kx, ky, kz, g, rho0, nu, false);
          if (kx != 0) {
            z = cscale(nr, h.g0);
          } else {
            const size_t em = ((size_t)((g.nz - kz) % g.nz) * g.ny + (g.ny - ky) % g.ny) * g.M;
            const C2<R> rm = ldg(r + em), qm = ldg(q + em);
            z = diag_packed(nr, C2<R>{R(rm.x - a * qm.x), R(rm.y - a * qm.y)}, h.g0, h.gN);
          }
        }
      }
      acc[1] += w * ((double)nr.x * z.x + (double)nr.y * z.y);
    }
  }
  block_store<2>(acc, RMR ? 1 : 2, partial + 2 * kRedBlocks + blockIdx.x);
}
int rec_step_blocks(const Geom& g) { return nblk(nspec(g)); }
template <typename R>
void rec_step(const Geom& g, const OpParams& op, bool rmr, void* x, const void* r, void* rnew, const void* p,
              const void* q, DevState* st, double* partial, hipStream_t s, const RecParts& parts) {
  const size_t n = nspec(g);
  const int nb = nblk(n), kind = op.precond ? op.kind : -1, nbd = parts.dot_blocks ? parts.dot_blocks : nb;
  if (rmr)
    hipLaunchKernelGGL((k_rec_step<R, true>), dim3(nb), dim3(256), 0, s, (C2<R>*)x, (const C2<R>*)r, (C2<R>*)rnew,
                       (const C2<R>*)p, (const C2<R>*)q, st, g, kind, op.rho0, op.nu, n, partial, nbd, g.ntot_inv,
                       parts.slot);
  else
    hipLaunchKernelGGL((k_rec_step<R, false>), dim3(nb), dim3(256), 0, s, (C2<R>*)x, (const C2<R>*)r, (C2<R>*)rnew,
                       (const C2<R>*)p, (const C2<R>*)q, st, g, kind, op.rho0, op.nu, n, partial, nbd, g.ntot_inv,
                       parts.slot);
  if (!parts.finish) return;
  reduce(partial + 2 * kRedBlocks, nb, rmr ? 1 : 2, g.ntot_inv, st->red, s, &st->halt,
         Post{rmr ? POST_REC_CHECK : POST_CG_STEP, st});
}

// D rt at row (eigenvector) `row`, packed wavenumber slot kx
template <typename R>
__device__ __forceinline__ double eig_mult(const EigDiag& d, int row, int kx) {
  const double kp = kx * d.sx;  // slot 0: k' = 0 for both halves
  return kx == 0 && row == 0 ? 0.0 : d.scale / (kp * kp + d.lam[row]);
}
template <typename R>
__global__ __launch_bounds__(256) void k_eig_step(C2<R>* __restrict__ xt, C2<R>* __restrict__ r,
                                                  C2<R>* __restrict__ rt, const C2<R>* __restrict__ pt,
                                                  const C2<R>* __restrict__ qq, DevState* st, EigDiag d, size_t n,
                                                  int M, double* partial, int nb, double scale) {
  if (st->halt) return;
  const double a = step_alpha<false>(st, partial, nb, scale, 0);
  double acc[2] = {0.0, 0.0};
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    const C2<R> xv = ldg(xt + e), pv = ldg(pt + e), rv = ldg(r + e), tv = ldg(rt + e), qv = ldg(qq + e),
                qt = ldg(qq + n + e);
    stg(xt + e, C2<R>{R(xv.x + a * pv.x), R(xv.y + a * pv.y)});
    const C2<R> nr{R(rv.x - a * qv.x), R(rv.y - a * qv.y)}, nt{R(tv.x - a * qt.x), R(tv.y - a * qt.y)};
    stg(r + e, nr);
    stg(rt + e, nt);
    const double w = spec_w(e, M), m = eig_mult<R>(d, (int)((unsigned)e / (unsigned)M), (int)(e & (size_t)(M - 1)));
    acc[0] += w * ((double)nr.x * nr.x + (double)nr.y * nr.y);
    acc[1] += w * m * ((double)nt.x * nt.x + (double)nt.y * nt.y);
  }
  block_store<2>(acc, 2, partial + 2 * kRedBlocks + blockIdx.x);
}
// Blocks of the Chebyshev CG kernels: one element per thread while the
// partials stay within what one reduction takes.
static int eig_blocks(size_t n) { return (int)std::min<size_t>((n + 255) / 256, kRedBlocks); }
template <typename R>
void eig_step(const Geom& g, const EigDiag& d, void* xt, void* r, void* rt, const void* pt, const void* qq,
              DevState* st, double* partial, hipStream_t s) {
  const size_t n = nspec(g);
  const int nb = eig_blocks(n);
  hipLaunchKernelGGL((k_eig_step<R>), dim3(nb), dim3(256), 0, s, (C2<R>*)xt, (C2<R>*)r, (C2<R>*)rt, (const C2<R>*)pt,
                     (const C2<R>*)qq, st, d, n, g.M, partial, nblk(n), g.ntot_inv);
  reduce(partial + 2 * kRedBlocks, nb, 2, g.ntot_inv, st->red, s, &st->halt, Post{POST_CG_STEP, st});
}
template <typename R>
__global__ __launch_bounds__(256) void k_eig_p(C2<R>* __restrict__ pt, const C2<R>* __restrict__ rt, EigDiag d,
                                               int first, const DevState* __restrict__ st, size_t n, int M,
                                               double* __restrict__ partial) {
  if (!first && st->halt) return;
  const double b = first ? 0.0 : st->beta;
  double acc = 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    const C2<R> tv = ldg(rt + e);
    const double m = eig_mult<R>(d, (int)((unsigned)e / (unsigned)M), (int)(e & (size_t)(M - 1)));
    C2<R> z{R(m * tv.x), R(m * tv.y)};
    if (first) {
      acc += spec_w(e, M) * ((double)tv.x * z.x + (double)tv.y * z.y);
    } else {
      const C2<R> pv = ldg(pt + e);
      z = C2<R>{R(z.x + b * pv.x), R(z.y + b * pv.y)};
    }
    stg(pt + e, z);
  }
  if (first) block_store<1>(&acc, 1, partial + blockIdx.x);
}
template <typename R>
void eig_p(const Geom& g, const EigDiag& d, void* pt, const void* rt, bool first, DevState* st, double* partial,
           hipStream_t s) {
  const size_t n = nspec(g);
  const int nb = eig_blocks(n);
  hipLaunchKernelGGL((k_eig_p<R>), dim3(nb), dim3(256), 0, s, (C2<R>*)pt, (const C2<R>*)rt, d, first ? 1 : 0, st, n,
                     g.M, partial);
  if (first) reduce(partial, nb, 1, g.ntot_inv, st->red, s, nullptr, Post{POST_CG_BETA, st});
}

template <typename R>
__global__ __launch_bounds__(256) void k_cg_p(C2<R>* __restrict__ p, const C2<R>* __restrict__ r, Geom g, int kind,
                                              double rho0, double nu, const DevState* __restrict__ st, size_t n,
                                              const int* __restrict__ gate) {
  if (gate && *gate) return;
  const double b = st->beta;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    C2<R> mz = precond_at<R>(r, e, g, kind, rho0, nu);
    C2<R> pv = ldg(p + e);
    stg(p + e, C2<R>{R(mz.x + b * pv.x), R(mz.y + b * pv.y)});
  }
}
template <typename R>
void cg_p(const Geom& g, const OpParams& op, void* p, const void* r, const DevState* st, hipStream_t s) {
  hipLaunchKernelGGL((k_cg_p<R>), dim3(nblk(nspec(g))), dim3(256), 0, s, (C2<R>*)p, (const C2<R>*)r, g,
                     op.precond ? op.kind : -1, op.rho0, op.nu, st, nspec(g), op.gate);
}

template <typename R>
__global__ __launch_bounds__(256) void k_axpy_norm(C2<R>* __restrict__ r, const C2<R>* __restrict__ w,
                                                   const double* __restrict__ ad, double sign, size_t n, int M,
                                                   double* __restrict__ partial, const int* __restrict__ gate) {
  if (gate && *gate) return;
  const double a = *ad * sign;
  double acc = 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    C2<R> rv = ldg(r + e), wv = ldg(w + e);
    C2<R> nr{R(rv.x + a * wv.x), R(rv.y + a * wv.y)};
    stg(r + e, nr);
    acc += spec_w(e, M) * ((double)nr.x * nr.x + (double)nr.y * nr.y);
  }
  block_store<1>(&acc, 1, partial + blockIdx.x);
}
template <typename R>
void axpy_norm(const Geom& g, void* r, const void* w, const double* a_dev, double sign, double* partial, double* out,
               hipStream_t s, const int* gate, const Post& post) {
  hipLaunchKernelGGL((k_axpy_norm<R>), dim3(nblk(nspec(g))), dim3(256), 0, s, (C2<R>*)r, (const C2<R>*)w, a_dev, sign,
                     nspec(g), g.M, partial, gate);
  reduce(partial, nblk(nspec(g)), 1, g.ntot_inv, out, s, gate, post);
}

// ---------------------------------------------------------------- casts

__global__ __launch_bounds__(256) void k_cast_d2f(const C2<double>* __restrict__ a, C2<float>* __restrict__ b,
                                                  double s, size_t n) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    C2<double> v = ldg(a + e);
    stg(b + e, C2<float>{float(v.x * s), float(v.y * s)});
  }
}
__global__ __launch_bounds__(256) void k_axpy_f2d(const C2<float>* __restrict__ a, C2<double>* __restrict__ b,
                                                  double s, size_t n) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    C2<float> v = ldg(a + e);
    C2<double> w = ldg(b + e);
    stg(b + e, C2<double>{w.x + s * (double)v.x, w.y + s * (double)v.y});
  }
}
__global__ __launch_bounds__(256) void k_cast_f2d(const C2<float>* __restrict__ a, C2<double>* __restrict__ b,
                                                  size_t n) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    C2<float> v = ldg(a + e);
    stg(b + e, C2<double>{(double)v.x, (double)v.y});
  }
}
void cast_d2f(const Geom& g, const void* src, void* dst, double s, hipStream_t st) {
  hipLaunchKernelGGL(k_cast_d2f, dim3(nblk(nspec(g))), dim3(256), 0, st, (const C2<double>*)src, (C2<float>*)dst, s,
                     nspec(g));
}
void axpy_f2d(const Geom& g, const void* src, void* dst, double s, hipStream_t st) {
  hipLaunchKernelGGL(k_axpy_f2d, dim3(nblk(nspec(g))), dim3(256), 0, st, (const C2<float>*)src, (C2<double>*)dst, s,
                     nspec(g));
}
void cast_f2d(const Geom& g, const void* src, void* dst, hipStream_t st) {
  hipLaunchKernelGGL(k_cast_f2d, dim3(nblk(nspec(g))), dim3(256), 0, st, (const C2<float>*)src, (C2<double>*)dst,
                     nspec(g));
}

// ---------------------------------------------------------- range projection

__global__ void k_project(C2<double>* __restrict__ s, Geom g, double* removed) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double acc = 0.0;
  const int nkz = g.nz > 1 ? 2 : 1, nky = g.ny > 1 ? 2 : 1;
  for (int a = 0; a < nkz; ++a)
    for (int b = 0; b < nky; ++b) {
      size_t kz = a ? g.nz / 2 : 0, ky = b ? g.ny / 2 : 0;
      size_t e = (kz * g.ny + ky) * g.M;
      C2<double> v = s[e];
      acc += v.x * v.x + v.y * v.y;
      s[e] = C2<double>{0.0, 0.0};
    }
  *removed = sqrt(acc * g.ntot_inv);
}
// Zero the mean (the real part of the DC slot) of a packed FP64 spectrum.
__global__ void k_zero_mean(C2<double>* s, Geom g, double* removed) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double dc = s[0].x;  // sum of the grid values (unnormalised transform)
  s[0].x = 0.0;
  if (removed) *removed = fabs(dc) * sqrt(g.ntot_inv);
}
void zero_mean(const Geom& g, void* spec, double* removed, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_mean, dim3(1), dim3(64), 0, st, (C2<double>*)spec, g, removed);
}

void project_range(const Geom& g, void* spec, double* removed, hipStream_t st) {
  hipLaunchKernelGGL(k_project, dim3(1), dim3(64), 0, st, (C2<double>*)spec, g, removed);
}

// ------------------------------------------------------- scalar kernels

// One wavefront (one thread clearing the 1056 entries of H took 6.8 us; 1.7 now).
__global__ __launch_bounds__(64) void k_gmres_init(DevState* st, double beta, int m, double bnorm, double rtol,
                                                   int jlast, unsigned long long run) {
  const int t = threadIdx.x;
  for (int i = t; i < (kMaxRestart + 1) * kMaxRestart; i += 64) st->H[i] = 0.0;
  if (t <= m && t <= kMaxRestart) st->g[t] = t == 0 ? beta : 0.0;
  if (t <= kMaxRestart) st->vs[t] = t == 0 ? 1.0 / beta : 0.0;
  if (t != 0) return;
  st->stop_bnorm = bnorm;
  st->stop_rtol = rtol;
  st->jlast = jlast;
  st->halt = 0;
  st->resid = beta;
  st->bad = 0;
  st->reorth = 0;
  st->nreorth = 0;
  st->run = run;
}

// Column j of the Hessenberg matrix: the Gram-Schmidt coefficients h (plus
// the second-pass corrections c when that pass ran); subdiagonal ||w||.
// One wavefront, lane i on row i: the triangle goes to LDS with all loads in
// flight, then column by column (18.8 us with one thread walking it in memory, 6.0 now,
// at 18 columns).
__global__ __launch_bounds__(64) void k_gmres_backsolve(DevState* st, int k) {
  static_assert(kMaxRestart < 64, "one lane per row");
  __shared__ double H[(kMaxRestart + 1) * kMaxRestart];
  const int t = threadIdx.x, ld = ldh();
#pragma unroll 17
  for (int i = t; i < (kMaxRestart + 1) * kMaxRestart; i += 64)
    if (i < k * ld) H[i] = st->H[i];
  double s = t < k ? st->g[t] : 0.0;
  const double v = t < k ? st->vs[t] : 0.0;
  __syncthreads();
  double y = 0.0;
  for (int l = k - 1; l >= 0; --l) {
    const double d = H[l + l * ld];
    const double q = d != 0.0 ? s / d : 0.0;   // meaningful in lane l
    const double yl = __shfl(q, l, 64);
    if (t == l) y = yl;
    if (t < l) s -= H[t + l * ld] * yl;
  }
  if (t < k) {
    st->y[t] = y;
    st->coef[t] = y * v;  // stored basis is unnormalised
  }
}

void gmres_init(DevState* st, double beta, int m, double bnorm, double rtol, int jlast, unsigned long long run,
                hipStream_t s) {
  hipLaunchKernelGGL(k_gmres_init, dim3(1), dim3(64), 0, s, st, beta, m, bnorm, rtol, jlast, run);
}
void gmres_backsolve(DevState* st, int k, hipStream_t s) {
  hipLaunchKernelGGL(k_gmres_backsolve, dim3(1), dim3(64), 0, s, st, k);
}

__global__ void k_rec_init(DevState* st, double bnorm, double rtol, int jlast, unsigned long long run) {
  if (threadIdx.x) return;
  st->stop_bnorm = bnorm;
  st->stop_rtol = rtol;
  st->jlast = jlast;
  st->step = 0;
  st->halt = 0;
  st->bad = 0;
  st->run = run;
}
void rec_init(DevState* st, double bnorm, double rtol, int jlast, unsigned long long run, hipStream_t s) {
  hipLaunchKernelGGL(k_rec_init, dim3(1), dim3(64), 0, s, st, bnorm, rtol, jlast, run);
}

__global__ void k_set_mail(DevState* st, Mail* mail) {
  if (threadIdx.x == 0) st->mail = mail;
}
void set_mail(DevState* st, Mail* mail, hipStream_t s) {
  hipLaunchKernelGGL(k_set_mail, dim3(1), dim3(64), 0, s, st, mail);
}

// --------------------------------------------------------- density set-up

__global__ __launch_bounds__(256) void k_density(const double* __restrict__ rho, size_t n, double* __restrict__ a64,
                                                 float* __restrict__ a32, float* __restrict__ r32,
                                                 double* __restrict__ partial) {
  double sum = 0.0, mn = INFINITY, mx = -INFINITY, bad = 0.0;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    double r = rho[e];
    if (!(r > 0.0) || !isfinite(r)) bad += 1.0;
    sum += r;
    mn = fmin(mn, r);
    mx = fmax(mx, r);
    double a = 1.0 / r;
    a64[e] = a;
    a32[e] = (float)a;
    r32[e] = (float)r;
  }
  __shared__ double sh[4][4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int o = 32; o > 0; o >>= 1) {
    sum += __shfl_xor(sum, o, 64);
    mn = fmin(mn, __shfl_xor(mn, o, 64));
    mx = fmax(mx, __shfl_xor(mx, o, 64));
    bad += __shfl_xor(bad, o, 64);
  }
  if (lane == 0) {
    sh[w][0] = sum;
    sh[w][1] = mn;
    sh[w][2] = mx;
    sh[w][3] = bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double* p = partial + (size_t)blockIdx.x * kRedStride;
    p[0] = ((sh[0][0] + sh[1][0]) + sh[2][0]) + sh[3][0];
    p[1] = fmin(fmin(sh[0][1], sh[1][1]), fmin(sh[2][1], sh[3][1]));
    p[2] = fmax(fmax(sh[0][2], sh[1][2]), fmax(sh[2][2], sh[3][2]));
    p[3] = ((sh[0][3] + sh[1][3]) + sh[2][3]) + sh[3][3];
  }
}
// One thread per block partial, then fixed shuffle and LDS trees (a single
// thread walking the 1024 partials took 233 us, one dependent load after
// another).
__global__ __launch_bounds__(1024) void k_density_fin(const double* __restrict__ partial, int nblk, double* out) {
  __shared__ double sh[4][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double sum = 0.0, mn = INFINITY, mx = -INFINITY, bad = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 1024) {
    const double* p = partial + (size_t)b * kRedStride;
    sum += p[0];
    mn = fmin(mn, p[1]);
    mx = fmax(mx, p[2]);
    bad += p[3];
  }
  sum = wave_sum(sum);
  bad = wave_sum(bad);
  mn = -wave_max(-mn);
  mx = wave_max(mx);
  if (lane == 0) {
    sh[0][w] = sum;
    sh[1][w] = mn;
    sh[2][w] = mx;
    sh[3][w] = bad;
  }
  __syncthreads();
  if (threadIdx.x) return;
  for (int i = 1; i < 16; ++i) {
    sh[0][0] += sh[0][i];
    sh[1][0] = fmin(sh[1][0], sh[1][i]);
    sh[2][0] = fmax(sh[2][0], sh[2][i]);
    sh[3][0] += sh[3][i];
  }
  out[0] = sh[0][0];
  out[1] = sh[1][0];
  out[2] = sh[2][0];
  out[3] = sh[3][0];
}
void density_setup(const double* rho, size_t n, double* a64, float* a32, float* rho32, double* partial, double* out,
                   hipStream_t s) {
  hipLaunchKernelGGL(k_density, dim3(nblk(n)), dim3(256), 0, s, rho, n, a64, a32, rho32, partial);
  hipLaunchKernelGGL(k_density_fin, dim3(1), dim3(1024), 0, s, partial, nblk(n), out);
}

// ----------------------------------------------- modified pressure form

// out = sign * rho^(+-1/2) * in on physical grid values (the change of
// unknown phi = sqrt(rho) Phi and the right-hand side sqrt(rho) f); in ==
// nullptr stands for in = 1.
__global__ __launch_bounds__(256) void k_rho_sqrt_mul(const double* __restrict__ rho, const double* __restrict__ in,
                                                      double* __restrict__ out, int inverse, double sign, size_t n) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    const double r = sqrt(rho[e]), v = in ? in[e] : 1.0;
    out[e] = sign * (inverse ? v / r : v * r);
  }
}
void rho_sqrt_mul(const double* rho, const double* in, double* out, bool inverse, double sign, size_t n,
                  hipStream_t s) {
  hipLaunchKernelGGL(k_rho_sqrt_mul, dim3(nblk(n)), dim3(256), 0, s, rho, in, out, inverse ? 1 : 0, sign, n);
}

// kc = Lap(psi) / psi = -c with psi = rho^-1/2 (so Lap(psi) / psi =
// Lap(psi) sqrt(rho)), in FP64 and FP32.
__global__ __launch_bounds__(256) void k_kcoef(const double* __restrict__ rho, const double* __restrict__ lap_psi,
                                               double* __restrict__ kc64, float* __restrict__ kc32, size_t n) {
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
    const double v = lap_psi[e] * sqrt(rho[e]);
    kc64[e] = v;
    kc32[e] = (float)v;
  }
}
void kcoef_finish(const double* rho, const double* lap_psi, double* kc64, float* kc32, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_kcoef, dim3(nblk(n)), dim3(256), 0, s, rho, lap_psi, kc64, kc32, n);
}

// ------------------------------------------------------- instantiations

#define VD_INST(R)                                                                                             \
  template void mdot<R>(const Geom&, const void*, const VecPtrs&, int, bool, double*, double*, hipStream_t,    \
                        Prof*, const int*, const Post&);                                                       \
  template void lincomb<R>(const Geom&, void*, const VecPtrs&, int, const double*, hipStream_t);               \
  template void scale<R>(const Geom&, void*, const double*, double, hipStream_t);                              \
  template void gs_orthogonalize<R>(const Geom&, void*, const VecPtrs&, int, DevState*, double*, hipStream_t,  \
                                    Prof*, const GsParts&);                                                                    \
  template void gs_orthogonalize_batch<R>(const Geom&, void* const*, const VecPtrs*, int, DevState* const*,   \
                                          double* const*, int, hipStream_t, Prof*, const GsParts&);                          \
  template void sub_norm<R>(const Geom&, const void*, const void*, void*, double*, double*, hipStream_t,       \
                            const Post&);                                                                      \
  template void precond_axpy<R>(const Geom&, const OpParams&, void*, const void*, const double*, double,       \
                                hipStream_t, const void*);                                                     \
  template void dot_rMr<R>(const Geom&, const OpParams&, const void*, double*, double*, hipStream_t,           \
                           const Post&);                                                                       \
  template void dot_partials<R>(const Geom&, const void*, const void*, bool, double*, hipStream_t, const int*); \
  template void rec_step<R>(const Geom&, const OpParams&, bool, void*, const void*, void*, const void*,        \
                            const void*, DevState*, double*, hipStream_t, const RecParts&);                                     \
  template void eig_step<R>(const Geom&, const EigDiag&, void*, void*, void*, const void*, const void*,        \
                            DevState*, double*, hipStream_t);                                                  \
  template void eig_p<R>(const Geom&, const EigDiag&, void*, const void*, bool, DevState*, double*,            \
                         hipStream_t);                                                                         \
  template void cg_p<R>(const Geom&, const OpParams&, void*, const void*, const DevState*, hipStream_t);       \
  template void axpy_norm<R>(const Geom&, void*, const void*, const double*, double, double*, double*,         \
                             hipStream_t, const int*, const Post&);

VD_INST(double)
VD_INST(float)

}  // namespace vd

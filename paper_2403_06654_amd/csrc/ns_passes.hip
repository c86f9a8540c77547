// Fused spectral passes of the fractional-step driver (gfx950, FP64).
//
// The driver keeps its fields as packed spectra and evaluates products in
// physical space.  Everything that a product needs of a field -- the field, its
// three derivatives, its Laplacian or its second derivatives -- is formed on
// the way to physical space:
//   z pass   reads a spectrum once and writes Fz^-1 of it, of i k'_z times it
//            and of its z second derivative;
//   y pass   adds the y derivatives the same way (in place, one or three
//            more fields);
//   x pass   takes the rows to physical space, forms the x derivatives and the
//            pointwise products there, and writes the product's rows, already
//            transformed along x.
// Forward y and z transforms (passes.hip) finish the spectrum.  Applying the
// viscous operator to a preconditioned vector this way moves 70 fields in 5
// launches; with a derivative kernel and a whole transform per derivative it
// moved 201 in about 60 launches.  128^3: a step 14.5 -> 8.3 ms (of the rest
// two thirds are the pressure solve); z pass of three fields 35.6 us (12 fields,
// 5.7 TB/s), y pass 53.5 us (21 fields, 6.6 TB/s), zeta's x pass 85 us (25
// fields, 4.9 TB/s).
//
// Bound: memory (FP64 transforms and products at ~2.5 flop/B).  Tiles are 8
// points per thread as in passes.hip, 128 B runs or more in the column passes;
// in the x passes wavefront c takes component (or derivative) c of the same
// rows, so the coefficient rows that the components share are read through one
// CU's cache.
#include <cstddef>
#include <cstdio>

#include "fft_core.hpp"
#include "ns.hpp"
#include "spectral.hpp"

namespace vd {

namespace {

using Cd = C2<double>;

// Element at a byte offset from a wave-uniform base.  A field has at most 1 GB,
// so the offset is 32 bits wide and every array of a kernel shares it (scalar
// base + vector offset addressing); 64-bit addresses per array and element took
// over a hundred registers in the x passes.
__device__ __forceinline__ Cd ldb(const void* base, unsigned off, int c = 0) {
  return ldg((const Cd*)((const char*)base + off) + c);
}
__device__ __forceinline__ void stb(void* base, unsigned off, int c, Cd v) {
  stg((Cd*)((char*)base + off) + c, v);
}

// The value is computed here.
__device__ __forceinline__ void pin(Cd& v) { asm volatile("" : "+v"(v.x), "+v"(v.y)); }

// ------------------------------------------------------------ column passes

template <int L>
struct NsCol {
  static constexpr int E = 8, T = L / E;
  static constexpr int TC = L <= 64 ? 64 / T : (L == 128 ? 16 : 8);
  static constexpr int NT = T * TC;
};

// Loads that depend on nothing go first, then the halt flag and the barrier
// that publishes the twiddle table.
template <int L, int NT>
struct TwRegs {
  static constexpr int N = (L + NT - 1) / NT;
  Cd r[N];
  __device__ __forceinline__ void load(const Cd* __restrict__ tab) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (i * NT + (int)threadIdx.x < L) r[i] = ldg(tab + i * NT + threadIdx.x);
  }
  __device__ __forceinline__ void store(Cd* lds) const {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (i * NT + (int)threadIdx.x < L) lds[i * NT + threadIdx.x] = r[i];
  }
};

// off: byte offset of the line's element 0; ld: bytes between elements
template <int L, int E, int RPAT>
__device__ __forceinline__ void line_load(Cd* reg, const void* p, unsigned off, unsigned ld, int t) {
#pragma unroll
  for (int s = 0; s < E; ++s) reg[s] = ldb(p, off + (unsigned)pat_index<L, E, RPAT>(t, s) * ld);
}
template <int L, int E, int RPAT>
__device__ __forceinline__ void line_store(const Cd* reg, void* p, unsigned off, unsigned ld, int t) {
#pragma unroll
  for (int s = 0; s < E; ++s) stb(p, off + (unsigned)pat_index<L, E, RPAT>(t, s) * ld, 0, reg[s]);
}

// z pass of field blockIdx.y of a stack: t0 = Fz^-1 v, t1 = Fz^-1 (i k'_z v) and
// t2 = Fz^-1 (-k_z^2 v) (HESS: -k'_z^2, two first derivatives), where v is the
// input times in_scale and, with `precond`, (I - nu Lap)^-1.
template <int L, bool HESS>
__global__ __launch_bounds__(NsCol<L>::NT) void k_ns_z(NsZArgs a, const Cd* __restrict__ twtab) {
  using Cf = NsCol<L>;
  constexpr int E = Cf::E, TC = Cf::TC, NT = Cf::NT;
  using S = Sched<L, E>;
  constexpr int R0 = S::template first_radix<false>(), R1 = S::template last_radix<false>();
  __shared__ Cd lds_raw[TC * L];
  __shared__ Cd tw[L];
  const int inner = a.g.ny * a.g.M;
  const int c = threadIdx.x % TC, t = threadIdx.x / TC;
  const int col = blockIdx.x * TC + c;  // the tiles divide the columns exactly (powers of two)
  const size_t f = (size_t)blockIdx.y * a.stride;
  const Cd* v = (const Cd*)a.in + f;
  const unsigned off = (unsigned)col * 16u, ld = (unsigned)inner * 16u;
  Cd x[E], w[E];
  TwRegs<L, NT> twr;
  twr.load(twtab + L);
  line_load<L, E, R0>(x, v, off, ld, t);
  const double sc = a.in_scale ? *a.in_scale : 1.0;
  if (a.gate && *a.gate) return;
  twr.store(tw);
  __syncthreads();
  LdsCol<double> lds{lds_raw, c, TC};
  const int ky = col / a.g.M, kx = col % a.g.M;
  const int kym = (a.g.ny - ky) % a.g.ny;
#pragma unroll
  for (int s = 0; s < E; ++s) {
    if (!a.precond) {
      x[s] = cscale(x[s], sc);
      continue;
    }
    const int kz = pat_index<L, E, R0>(t, s);
    const HelmMult<double> h = mult_helm<double>(kx, ky, kz, a.g, 1.0, a.nu, false);
    if (kx == 0) {
      const Cd pm = ldb(v, (unsigned)((L - kz) % L) * ld + (unsigned)(kym * a.g.M) * 16u);
      x[s] = cscale(diag_packed(x[s], pm, h.g0, h.gN), sc);
    } else {
      x[s] = cscale(x[s], h.g0 * sc);
    }
  }
#pragma unroll
  for (int s = 0; s < E; ++s) w[s] = x[s];
  fft_line<L, E, +1, false>(w, lds, tw, t);
  line_store<L, E, R1>(w, (Cd*)a.t0 + f, off, ld, t);
#pragma unroll
  for (int s = 0; s < E; ++s) w[s] = cik(x[s], kprime_of<double>(pat_index<L, E, R0>(t, s), L, a.g.sz));
  fft_line<L, E, +1, false>(w, lds, tw, t);
  line_store<L, E, R1>(w, (Cd*)a.t1 + f, off, ld, t);
#pragma unroll
  for (int s = 0; s < E; ++s) {
    const int kz = pat_index<L, E, R0>(t, s);
    const double k1 = kprime_of<double>(kz, L, a.g.sz);
    w[s] = cscale(x[s], HESS ? -k1 * k1 : -ksq_of<double>(kz, L, a.g.sz));
  }
  fft_line<L, E, +1, false>(w, lds, tw, t);
  line_store<L, E, R1>(w, (Cd*)a.t2 + f, off, ld, t);
}

// y pass of field blockIdx.y of a stack, on the z pass's output, in place:
// t0 -> Fy^-1 t0, t1 -> Fy^-1 t1, y1 = Fy^-1 (i k'_y t0), and
//   t2 -> Fy^-1 (t2 - k_y^2 t0)      (the y and z part of the Laplacian), or
//   HESS: t2 -> Fy^-1 t2, y2 = Fy^-1 (-k'_y^2 t0), y3 = Fy^-1 (i k'_y t1).
template <int L, bool HESS>
__global__ __launch_bounds__(NsCol<L>::NT) void k_ns_y(NsYArgs a, const Cd* __restrict__ twtab) {
  using Cf = NsCol<L>;
  constexpr int E = Cf::E, TC = Cf::TC, NT = Cf::NT;
  using S = Sched<L, E>;
  constexpr int R0 = S::template first_radix<false>(), R1 = S::template last_radix<false>();
  __shared__ Cd lds_raw[TC * L];
  __shared__ Cd tw[L];
  const int inner = a.g.M, tiles = (inner + TC - 1) / TC;
  const int c = threadIdx.x % TC, t = threadIdx.x / TC;
  const int col = (blockIdx.x % tiles) * TC + c;
  const bool ok = col < inner;  // 16 points: 8 columns of a 32-column tile
  const unsigned ld = (unsigned)inner * 16u;
  const unsigned off = (blockIdx.x / tiles) * (unsigned)L * ld + (ok ? (unsigned)col * 16u : 0u);
  const size_t f = (size_t)blockIdx.y * a.stride;
  Cd *t0 = (Cd*)a.t0 + f, *t1 = (Cd*)a.t1 + f, *t2 = (Cd*)a.t2 + f;
  Cd x[E], w[E];
  TwRegs<L, NT> twr;
  twr.load(twtab + L);
  line_load<L, E, R0>(x, t0, off, ld, t);
  if (a.gate && *a.gate) return;
  twr.store(tw);
  __syncthreads();
  LdsCol<double> lds{lds_raw, c, TC};
  auto out = [&](Cd* p) {
    fft_line<L, E, +1, false>(w, lds, tw, t);
    if (ok) line_store<L, E, R1>(w, p, off, ld, t);
  };
  if constexpr (HESS) {
    line_load<L, E, R0>(w, t2, off, ld, t);
  } else {
    line_load<L, E, R0>(w, t2, off, ld, t);
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const double k2 = ksq_of<double>(pat_index<L, E, R0>(t, s), L, a.g.sy);
      w[s] = C2<double>{w[s].x - k2 * x[s].x, w[s].y - k2 * x[s].y};
    }
  }
  out(t2);
#pragma unroll
  for (int s = 0; s < E; ++s) w[s] = cik(x[s], kprime_of<double>(pat_index<L, E, R0>(t, s), L, a.g.sy));
  out((Cd*)a.y1 + f);
  if constexpr (HESS) {
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const double k1 = kprime_of<double>(pat_index<L, E, R0>(t, s), L, a.g.sy);
      w[s] = cscale(x[s], -k1 * k1);
    }
    out((Cd*)a.y2 + f);
  }
#pragma unroll
  for (int s = 0; s < E; ++s) w[s] = x[s];
  out(t0);  // every thread of the line has loaded its t0 before the first exchange
  line_load<L, E, R0>(x, t1, off, ld, t);
  if constexpr (HESS) {
#pragma unroll
    for (int s = 0; s < E; ++s) w[s] = cik(x[s], kprime_of<double>(pat_index<L, E, R0>(t, s), L, a.g.sy));
    out((Cd*)a.y3 + f);
  }
#pragma unroll
  for (int s = 0; s < E; ++s) w[s] = x[s];
  out(t1);
}

// ------------------------------------------------------------- row passes

// 4 points per thread: the zeta pass holds a row's spectrum, its field, two
// sums and the transform in flight (at 8 points it spilled).
template <int L>
struct NsRow {
  static constexpr int E = 4, T = L / E, RW = 64 / T, LP = row_pitch<L>();
};

// One wavefront's rows: packed spectrum values X (register s holds k = t + s T)
// to real pairs (register s holds pair t + pair(s)), unnormalised,
// and back.
template <int L>
struct RowFft {
  static constexpr int E = NsRow<L>::E, T = NsRow<L>::T;
  using S = Sched<L, E>;
  static constexpr int RI0 = S::template first_radix<false>();
  static constexpr int RI = S::template last_radix<false>();
  static_assert(RI == S::template first_radix<true>(), "inverse output pattern = forward input pattern");
  LdsRow<double> lds;
  const Cd* tw;   // length L
  const Cd* twN;  // length 2L
  int lane;       // the thread's place in its row

  // register s holds pair lane + pair(s)
  static __device__ __forceinline__ constexpr int pair(int s) { return T * (s / RI) + (s % RI) * (L / RI); }

  // An opaque copy of the lane's index per transform: otherwise the compiler
  // keeps every twiddle factor of the lane in registers from one transform of
  // a kernel to the next (300 registers in the zeta pass).
  __device__ __forceinline__ int fresh() const {
    int v = lane;
    asm volatile("" : "+v"(v));
    return v;
  }

  __device__ __forceinline__ void to_real(const Cd* X, Cd* reg) const {
    const int t = fresh();
    lds_sync<true>();
#pragma unroll
    for (int s = 0; s < E; ++s) lds.st(t + s * T, X[s]);
    lds_sync<true>();
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const int k = pat_index<L, E, RI0>(t, s);
      const Cd Xk = lds.ld(k), Xm = cconj(lds.ld((L - k) % L));
      if (k == 0) {
        reg[s] = Cd{Xk.x + Xk.y, Xk.x - Xk.y};
      } else {
        const Cd e = Xk + Xm, o = cmulc(Xk - Xm, twN[k]);
        reg[s] = Cd{e.x - o.y, e.y + o.x};
      }
    }
    fft_line<L, E, +1, false, true>(reg, lds, tw, t);
  }

  __device__ __forceinline__ void to_spec(Cd* reg, Cd* X) const {
    const int t = fresh();
    fft_line<L, E, -1, true, true>(reg, lds, tw, t);
    lds_sync<true>();
#pragma unroll
    for (int s = 0; s < E; ++s) lds.st(t + s * T, reg[s]);
    lds_sync<true>();
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const int k = t + s * T;
      const Cd Zk = reg[s];
      if (k == 0) {
        X[s] = Cd{Zk.x + Zk.y, Zk.x - Zk.y};
      } else {
        const Cd Zm = cconj(lds.ld(L - k));
        const Cd e = Zk + Zm, d = cmul(twN[k], Zk - Zm);
        X[s] = Cd{0.5 * (e.x + d.y), 0.5 * (e.y - d.x)};
      }
    }
  }
};

// The common frame of the row kernels: three wavefronts over the same rows,
// twiddle tables and the wavefront's own exchange rows in LDS.  Row groups
// divide the n^2 rows exactly (powers of two, RW <= 32 <= n^2).
#define VD_NS_ROWS(GATE)                                                     \
  using Cf = NsRow<L>;                                                       \
  constexpr int E = Cf::E, T = Cf::T, RW = Cf::RW, LP = Cf::LP;              \
  __shared__ Cd rows_lds[3 * RW * LP];                                       \
  __shared__ Cd tw[2 * L];                                                   \
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);           \
  const int lane = threadIdx.x % 64, t = lane % T, rr = lane / T;            \
  /* byte offset of this lane's element 0 of its row in every field */       \
  const unsigned off = ((blockIdx.x * RW + rr) * L + t) * 16u;               \
  TwRegs<2 * L, 192> twr;                                                    \
  twr.load(twtab + L);                                                       \
  if ((GATE) && *(GATE)) return;                                             \
  twr.store(tw);                                                             \
  __syncthreads();                                                           \
  const RowFft<L> F{LdsRow<double>{rows_lds + (wv * RW + rr) * LP}, tw, tw + L, t};

template <int E, int T>
__device__ __forceinline__ void row_load(Cd* X, const void* p, unsigned off) {
#pragma unroll
  for (int s = 0; s < E; ++s) X[s] = ldb(p, off, s * T);
}
template <int E, int T>
__device__ __forceinline__ void row_store(const Cd* X, void* p, unsigned off) {
#pragma unroll
  for (int s = 0; s < E; ++s) stb(p, off, s * T, X[s]);
}

// x pass of zeta (eq. VDINSE.zeta), wavefront i on component i:
//   out_i = a u_i + b W (Lap u_i + (sum_j u_j h_ij + sum_j g_j d_j u_i) / Sc)
// with W = 1 / rho (ir), or 1 (unit; b holds 1 / Re); and, for the
// right-hand side of a step (RHS), n_i = (u . grad) u_i written to nout and
//   out_i += ca n_i + cp nprev_i + cg d_i p / rho + ce ext_i.
// The rows of out are transformed along x, or (PHYS) physical.
template <int L, bool RHS, bool PHYS>
__global__ __launch_bounds__(192) void k_ns_zeta_x(NsZetaArgs a, const Cd* __restrict__ twtab) {
  VD_NS_ROWS(a.gate)
  __shared__ Cd ush[3 * E * 64];
  const size_t fo = (size_t)wv * a.stride;  // this component (a field is as large physical as packed)
  Cd y0[E], X[E], reg[E], acc[E], u[E], adv[RHS ? E : 1];
  row_load<E, T>(y0, (const Cd*)a.y0 + fo, off);
  F.to_real(y0, u);
#pragma unroll
  for (int s = 0; s < E; ++s) {
    u[s] = cscale(u[s], a.norm);
    ush[(wv * E + s) * 64 + lane] = u[s];
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < E; ++s) acc[s] = Cd{0.0, 0.0};
  if constexpr (RHS) {
#pragma unroll
    for (int s = 0; s < E; ++s) adv[s] = Cd{0.0, 0.0};
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    if (j == 0) {
#pragma unroll
      for (int s = 0; s < E; ++s) X[s] = cik(y0[s], (double)(t + s * T) * a.sx);
    } else {
      row_load<E, T>(X, (const Cd*)(j == 1 ? a.yy : a.yz) + fo, off);
    }
    F.to_real(X, reg);
    const double* gr = a.gr + (size_t)j * a.n;
    // Hessian entry (wv, j) of 00 01 02 11 12 22
    const double* hh = a.h + (size_t)(wv + j + (wv > 0 && j > 0 ? 1 : 0)) * a.n;
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const Cd q = ldb(gr, off, F.pair(s)), h = ldb(hh, off, F.pair(s)), uj = ush[(j * E + s) * 64 + lane];
      const Cd d = cscale(reg[s], a.norm);
      acc[s].x += q.x * d.x + uj.x * h.x;
      acc[s].y += q.y * d.y + uj.y * h.y;
      if constexpr (RHS) {
        adv[s].x += uj.x * d.x;
        adv[s].y += uj.y * d.y;
      }
    }
    // The sums are wanted at the end only, and the compiler would move their
    // additions there, with every direction's operands held in registers (290
    // of them) until then.
#pragma unroll
    for (int s = 0; s < E; ++s) {
      pin(acc[s]);
      if constexpr (RHS) pin(adv[s]);
    }
  }
  // Laplacian: the x part here (slot 0 holds kx = 0 and kx = nx/2)
  row_load<E, T>(X, (const Cd*)a.yl + fo, off);
  const double kn = (double)L * a.sx;
#pragma unroll
  for (int s = 0; s < E; ++s) {
    const int k = t + s * T;
    const double kx = (double)k * a.sx, k0 = kx * kx, k1 = k == 0 ? kn * kn : k0;
    X[s] = Cd{X[s].x - k0 * y0[s].x, X[s].y - k1 * y0[s].y};
  }
  F.to_real(X, reg);
#pragma unroll
  for (int s = 0; s < E; ++s) {
    const Cd q = ldb(a.ir, off, F.pair(s));
    const double wx = a.unit ? 1.0 : q.x, wy = a.unit ? 1.0 : q.y;
    reg[s] = Cd{a.a * u[s].x + a.b * wx * (reg[s].x * a.norm + a.inv_sc * acc[s].x),
                a.a * u[s].y + a.b * wy * (reg[s].y * a.norm + a.inv_sc * acc[s].y)};
  }
  if constexpr (RHS) {
    Cd gp[E];
    row_load<E, T>(X, wv == 0 ? a.p0 : wv == 1 ? a.py : a.pz, off);
    if (wv == 0) {
#pragma unroll
      for (int s = 0; s < E; ++s) X[s] = cik(X[s], (double)(t + s * T) * a.sx);
    }
    F.to_real(X, gp);
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const int m = F.pair(s);
      const Cd q = ldb(a.ir, off, m);
      const double c = a.cg * a.norm;
      reg[s].x += a.ca * adv[s].x + c * q.x * gp[s].x;
      reg[s].y += a.ca * adv[s].y + c * q.y * gp[s].y;
      if (a.nprev) {
        const Cd np = ldb((const Cd*)a.nprev + fo, off, m);
        reg[s].x += a.cp * np.x;
        reg[s].y += a.cp * np.y;
      }
      if (a.ext) {
        const Cd ex = ldb((const Cd*)a.ext + fo, off, m);
        reg[s].x += a.ce * ex.x;
        reg[s].y += a.ce * ex.y;
      }
      if (a.nout) stb((Cd*)a.nout + fo, off, m, adv[s]);
    }
  }
  if constexpr (PHYS) {
#pragma unroll
    for (int s = 0; s < E; ++s) stb((Cd*)a.out + fo, off, F.pair(s), reg[s]);
  } else {
    F.to_spec(reg, X);
    row_store<E, T>(X, (Cd*)a.out + fo, off);
  }
}

// x pass of a density's coefficients: rho, 1 / rho, its gradient and its
// Hessian (00 01 02 11 12 22), physical; the derivatives by wavefront: along x
// (and xx), along y (and xy, yy, yz), along z (and xz, zz).
template <int L>
__global__ __launch_bounds__(192) void k_ns_coef_x(NsCoefArgs a, const Cd* __restrict__ twtab) {
  VD_NS_ROWS((const int*)nullptr)
  Cd x[E], X[E], reg[E];
  auto emit = [&](double* out) {
    F.to_real(X, reg);
#pragma unroll
    for (int s = 0; s < E; ++s) stb(out, off, F.pair(s), cscale(reg[s], a.norm));
  };
  auto dx = [&](int times) {  // X = (i k'_x)^times x
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const double k = (double)(t + s * T) * a.sx;
      X[s] = times == 1 ? cik(x[s], k) : cscale(x[s], -k * k);
    }
    // slot 0 holds kx = 0 and kx = nx/2: k'_x = 0 for both, and so is k above
  };
  const size_t n = a.n;
  if (wv == 0) {
    row_load<E, T>(x, a.y0, off);
#pragma unroll
    for (int s = 0; s < E; ++s) X[s] = x[s];
    F.to_real(X, reg);
#pragma unroll
    for (int s = 0; s < E; ++s) {
      const Cd r = cscale(reg[s], a.norm);
      stb(a.rho, off, F.pair(s), r);
      stb(a.ir, off, F.pair(s), Cd{1.0 / r.x, 1.0 / r.y});
    }
    dx(1);
    emit(a.gr);
    dx(2);
    emit(a.h);
  } else if (wv == 1) {
    row_load<E, T>(x, a.y1, off);
#pragma unroll
    for (int s = 0; s < E; ++s) X[s] = x[s];
    emit(a.gr + n);
    dx(1);
    emit(a.h + n);
    row_load<E, T>(X, a.y2, off);
    emit(a.h + 3 * n);
    row_load<E, T>(X, a.y3, off);
    emit(a.h + 4 * n);
  } else {
    row_load<E, T>(x, a.t1, off);
#pragma unroll
    for (int s = 0; s < E; ++s) X[s] = x[s];
    emit(a.gr + 2 * n);
    dx(1);
    emit(a.h + 2 * n);
    row_load<E, T>(X, a.t2, off);
    emit(a.h + 5 * n);
  }
}

// x pass of (u . grad) q for a scalar q: wavefront d forms u_d d_d q from the
// rows of u (y0) and of q (q0, qy, qz); wavefront 0 adds the three and writes
// the rows, transformed along x.
template <int L>
__global__ __launch_bounds__(192) void k_ns_advect_x(NsAdvArgs a, const Cd* __restrict__ twtab) {
  VD_NS_ROWS((const int*)nullptr)
  __shared__ Cd psh[3 * E * 64];
  Cd X[E], u[E], reg[E];
  row_load<E, T>(X, (const Cd*)a.y0 + (size_t)wv * a.stride, off);
  F.to_real(X, u);
  row_load<E, T>(X, wv == 0 ? a.q0 : wv == 1 ? a.qy : a.qz, off);
  if (wv == 0) {
#pragma unroll
    for (int s = 0; s < E; ++s) X[s] = cik(X[s], (double)(t + s * T) * a.sx);
  }
  F.to_real(X, reg);
  const double c = a.norm * a.norm;
#pragma unroll
  for (int s = 0; s < E; ++s) {
    reg[s] = Cd{c * u[s].x * reg[s].x, c * u[s].y * reg[s].y};
    psh[(wv * E + s) * 64 + lane] = reg[s];
  }
  __syncthreads();
  if (wv != 0) return;
#pragma unroll
  for (int s = 0; s < E; ++s) {
    const Cd p1 = psh[(E + s) * 64 + lane], p2 = psh[(2 * E + s) * 64 + lane];
    reg[s] = (reg[s] + p1) + p2;
  }
  F.to_spec(reg, X);
  row_store<E, T>(X, a.out, off);
}

// x pass of grad(q) / rho: wavefront d writes component d, its rows transformed
// along x or (PHYS) physical (ir = 1 / rho).
template <int L, bool PHYS>
__global__ __launch_bounds__(192) void k_ns_gradq_x(NsGradArgs a, const Cd* __restrict__ twtab) {
  VD_NS_ROWS((const int*)nullptr)
  Cd X[E], reg[E];
  row_load<E, T>(X, wv == 0 ? a.q0 : wv == 1 ? a.qy : a.qz, off);
  if (wv == 0) {
#pragma unroll
    for (int s = 0; s < E; ++s) X[s] = cik(X[s], (double)(t + s * T) * a.sx);
  }
  F.to_real(X, reg);
#pragma unroll
  for (int s = 0; s < E; ++s) {
    const Cd q = ldb(a.ir, off, F.pair(s));
    reg[s] = Cd{a.norm * q.x * reg[s].x, a.norm * q.y * reg[s].y};
  }
  Cd* out = (Cd*)a.out + (size_t)wv * a.stride;  // a field is as large physical as packed
  if constexpr (PHYS) {
#pragma unroll
    for (int s = 0; s < E; ++s) stb(out, off, F.pair(s), reg[s]);
  } else {
    F.to_spec(reg, X);
    row_store<E, T>(X, out, off);
  }
}

// ------------------------------------------------------- spectral pointwise

__device__ __forceinline__ void slot_of(size_t e, const Geom& g, int& kx, int& ky, int& kz) {
  const unsigned ue = (unsigned)e, q = ue / (unsigned)g.M;
  kx = (int)(ue - q * (unsigned)g.M);
  ky = (int)(q % (unsigned)g.ny);
  kz = (int)(q / (unsigned)g.ny);
}

// Crank-Nicolson density: with k = c |k|^2 (Nyquist kept),
//   rho1 = ((1 - k) rho + d) / (1 + k),  d = s S + sa Na + sb Nb,
// and the mid-step density rhm = (rho + rho1) / 2.  The kx = 0 slot packs two
// modes with different symbols: they are separated through the mirror slot.
__global__ __launch_bounds__(256) void k_ns_density(NsDensArgs a) {
  const Cd *rho = (const Cd*)a.rho, *S = (const Cd*)a.S, *na = (const Cd*)a.na, *nb = (const Cd*)a.nb;
  auto rhs = [&](size_t e) {
    const Cd x = ldg(na + e);
    Cd d{a.sa * x.x, a.sa * x.y};
    if (nb) {
      const Cd y = ldg(nb + e);
      d.x += a.sb * y.x;
      d.y += a.sb * y.y;
    }
    if (S) {
      const Cd z = ldg(S + e);
      d.x += a.s * z.x;
      d.y += a.s * z.y;
    }
    return d;
  };
  for (size_t e = blockIdx.x * (size_t)256 + threadIdx.x; e < a.n; e += (size_t)gridDim.x * 256) {
    int kx, ky, kz;
    slot_of(e, a.g, kx, ky, kz);
    const double kyz = ksq_yz<double>(ky, kz, a.g);
    const double kxx = (double)kx * a.g.sx, kn = (double)a.g.M * a.g.sx;
    const double c0 = a.c * (kyz + kxx * kxx);
    const Cd r = ldg(rho + e), d = rhs(e);
    Cd r1;
    if (kx == 0) {
      const double cN = a.c * (kyz + kn * kn);
      const int kym = (a.g.ny - ky) % a.g.ny, kzm = (a.g.nz - kz) % a.g.nz;
      const size_t em = ((size_t)kzm * a.g.ny + kym) * a.g.M;
      r1 = diag_packed(r, ldg(rho + em), (1.0 - c0) / (1.0 + c0), (1.0 - cN) / (1.0 + cN)) +
           diag_packed(d, rhs(em), 1.0 / (1.0 + c0), 1.0 / (1.0 + cN));
    } else {
      const double q = 1.0 / (1.0 + c0);
      r1 = Cd{((1.0 - c0) * r.x + d.x) * q, ((1.0 - c0) * r.y + d.y) * q};
    }
    stg((Cd*)a.rho1 + e, r1);
    stg((Cd*)a.rhm + e, Cd{0.5 * (r.x + r1.x), 0.5 * (r.y + r1.y)});
  }
}

// i k' . v of a stack of three spectra at slot e
__device__ __forceinline__ Cd div_at(const Cd* v, size_t stride, size_t e, int kx, int ky, int kz, const Geom& g) {
  const Cd a = cik(ldg(v + e), (double)kx * g.sx);  // slot 0: k'_x = 0 for both halves
  const Cd b = cik(ldg(v + stride + e), kprime_of<double>(ky, g.ny, g.sy));
  const Cd c = cik(ldg(v + 2 * stride + e), kprime_of<double>(kz, g.nz, g.sz));
  return (a + b) + c;
}
__global__ __launch_bounds__(256) void k_ns_div(Geom g, const Cd* __restrict__ v, size_t stride, double c,
                                                Cd* __restrict__ out) {
  for (size_t e = blockIdx.x * (size_t)256 + threadIdx.x; e < stride; e += (size_t)gridDim.x * 256) {
    int kx, ky, kz;
    slot_of(e, g, kx, ky, kz);
    stg(out + e, cscale(div_at(v, stride, e, kx, ky, kz, g), c));
  }
}

// p += phi - (div grad)^-1 div v (symbol -1 / |k'|^2, zero on its nullspace)
__global__ __launch_bounds__(256) void k_ns_pressure(Geom g, const Cd* __restrict__ v, size_t stride,
                                                     const Cd* __restrict__ phi, Cd* __restrict__ p) {
  for (size_t e = blockIdx.x * (size_t)256 + threadIdx.x; e < stride; e += (size_t)gridDim.x * 256) {
    int kx, ky, kz;
    slot_of(e, g, kx, ky, kz);
    const Cd d = cscale(div_at(v, stride, e, kx, ky, kz, g), mult_press<double>(kx, ky, kz, g, 1.0));
    const Cd f = ldg(phi + e), q = ldg(p + e);
    stg(p + e, Cd{q.x + f.x + d.x, q.y + f.y + d.y});
  }
}

unsigned slots_grid(size_t n) {
  const size_t b = (n + 255) / 256;
  return (unsigned)(b < 8192 ? b : 8192);
}

template <int L, bool HESS>
void launch_z(const NsZArgs& a, int nf, const void* tw, hipStream_t st) {
  const int inner = a.g.ny * a.g.M;
  hipLaunchKernelGGL((k_ns_z<L, HESS>), dim3(inner / NsCol<L>::TC, nf), dim3(NsCol<L>::NT), 0, st, a, (const Cd*)tw);
}
template <int L, bool HESS>
void launch_y(const NsYArgs& a, int nf, const void* tw, hipStream_t st) {
  const int tiles = (a.g.M + NsCol<L>::TC - 1) / NsCol<L>::TC;
  hipLaunchKernelGGL((k_ns_y<L, HESS>), dim3(a.g.nz * tiles, nf), dim3(NsCol<L>::NT), 0, st, a, (const Cd*)tw);
}

// one case per line length of the driver's cubic grids (columns n, rows n / 2)
#define VD_NS_CASES(N, CALL)                                                  \
  switch (N) {                                                                \
    case 16: CALL(16, 8); break;                                              \
    case 32: CALL(32, 16); break;                                             \
    case 64: CALL(64, 32); break;                                             \
    case 128: CALL(128, 64); break;                                           \
    case 256: CALL(256, 128); break;                                          \
    case 512: CALL(512, 256); break;                                          \
    default: fprintf(stderr, "vdsolve: unsupported grid size %d\n", (int)(N)); \
  }

template <int L>
dim3 row_blocks(const Geom& g) { return dim3((unsigned)((size_t)g.ny * g.nz / NsRow<L>::RW)); }

}  // namespace

void ns_z_pass(const NsZArgs& a, int nf, bool hess, const void* tw, hipStream_t st) {
#define CALL(N, H) (hess ? launch_z<N, true>(a, nf, tw, st) : launch_z<N, false>(a, nf, tw, st))
  VD_NS_CASES(a.g.nz, CALL)
#undef CALL
}
void ns_y_pass(const NsYArgs& a, int nf, bool hess, const void* tw, hipStream_t st) {
#define CALL(N, H) (hess ? launch_y<N, true>(a, nf, tw, st) : launch_y<N, false>(a, nf, tw, st))
  VD_NS_CASES(a.g.ny, CALL)
#undef CALL
}
void ns_zeta_pass(const Geom& g, const NsZetaArgs& a, bool rhs, bool phys, const void* tw, hipStream_t st) {
#define CALL(N, H)                                                                                           \
  if (!rhs) hipLaunchKernelGGL((k_ns_zeta_x<H, false, false>), row_blocks<H>(g), dim3(192), 0, st, a, (const Cd*)tw); \
  else if (phys) hipLaunchKernelGGL((k_ns_zeta_x<H, true, true>), row_blocks<H>(g), dim3(192), 0, st, a, (const Cd*)tw); \
  else hipLaunchKernelGGL((k_ns_zeta_x<H, true, false>), row_blocks<H>(g), dim3(192), 0, st, a, (const Cd*)tw)
  VD_NS_CASES(g.nx, CALL)
#undef CALL
}
void ns_coef_pass(const Geom& g, const NsCoefArgs& a, const void* tw, hipStream_t st) {
#define CALL(N, H) hipLaunchKernelGGL((k_ns_coef_x<H>), row_blocks<H>(g), dim3(192), 0, st, a, (const Cd*)tw)
  VD_NS_CASES(g.nx, CALL)
#undef CALL
}
void ns_advect_pass(const Geom& g, const NsAdvArgs& a, const void* tw, hipStream_t st) {
#define CALL(N, H) hipLaunchKernelGGL((k_ns_advect_x<H>), row_blocks<H>(g), dim3(192), 0, st, a, (const Cd*)tw)
  VD_NS_CASES(g.nx, CALL)
#undef CALL
}
void ns_grad_pass(const Geom& g, const NsGradArgs& a, bool phys, const void* tw, hipStream_t st) {
#define CALL(N, H)                                                                                              \
  if (phys) hipLaunchKernelGGL((k_ns_gradq_x<H, true>), row_blocks<H>(g), dim3(192), 0, st, a, (const Cd*)tw); \
  else hipLaunchKernelGGL((k_ns_gradq_x<H, false>), row_blocks<H>(g), dim3(192), 0, st, a, (const Cd*)tw)
  VD_NS_CASES(g.nx, CALL)
#undef CALL
}

void ns_density(const NsDensArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(k_ns_density, dim3(slots_grid(a.n)), dim3(256), 0, st, a);
}
void ns_div(const Geom& g, const void* v, size_t stride, double c, void* out, hipStream_t st) {
  hipLaunchKernelGGL(k_ns_div, dim3(slots_grid(stride)), dim3(256), 0, st, g, (const Cd*)v, stride, c, (Cd*)out);
}
void ns_pressure(const Geom& g, const void* v, size_t stride, const void* phi, void* p, hipStream_t st) {
  hipLaunchKernelGGL(k_ns_pressure, dim3(slots_grid(stride)), dim3(256), 0, st, g, (const Cd*)v, stride,
                     (const Cd*)phi, (Cd*)p);
}

}  // namespace vd

// Device kernels of the local-relaxation message-passing step for gfx950 (CDNA4).
//
// One pass over a bucket of clusters of dimension De computes, per cluster e
// (paper Sec. 4.2: theta_e, Q_C, Q_{C,beta} and their (sub)gradients):
//   a1  eta = (1 - theta) nu + theta zeta           (Algorithm 2 extrapolation, fused in the loads)
//   a2  theta_e = h_e - sum_children 1 (x) eta_{e->f} + sum_parents eta_{g->e}
//   a3  cyclic Jacobi eigen-decomposition theta_e = U diag(l) U^H
//   a4  Gibbs state rho = U softmax(-beta l) U^H and F_beta (stable shifted form), or the
//       normalised ground projector P0/g and lambda_min
//   a5  partial traces T_{e->f} = Tr_{e\f} rho for every child f, and rho itself when e
//       has parents (consumed by the message update)
//   a8  in certify mode: FP64 lambda_min and the backward-error margin 8 De eps ||theta||_F
// The message kernel applies a6 (gradient and update) per message.
//
// Two cluster kernels:
//   * k_cluster_reg: one lane per cluster, the whole De x De problem in registers with
//     compile-time indexing (De <= 4: sites and edges of 2-local problems).  No LDS, no
//     cross-lane traffic; a wave advances 64 independent clusters.
//   * k_cluster_lds: one wavefront per cluster for 8 <= De <= 64; the matrix lives in LDS and
//     the De/2 disjoint rotations of each round-robin step are applied in parallel.
#pragma once

#include "lrh_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <type_traits>
#include <utility>

namespace lrh {

// ------------------------------------------------------------------------------------------
// small helpers
// ------------------------------------------------------------------------------------------

// FP32 iterations use the single hardware instructions (v_sqrt_f32, v_rsq_f32, v_rcp_f32,
// v_exp_f32, v_log_f32; about 1 ulp), far inside the FP32 tolerances and much shorter than the
// correctly rounded sequences on the serial chain of a one-lane-per-cluster kernel.  FP64 keeps
// IEEE division, square root and the libm exponential and logarithm.
template <typename T> __device__ __forceinline__ T dsqrt(T x);
template <> __device__ __forceinline__ float dsqrt<float>(float x) { return __builtin_amdgcn_sqrtf(x); }
template <> __device__ __forceinline__ double dsqrt<double>(double x) { return sqrt(x); }
template <typename T> __device__ __forceinline__ T drsq(T x);   // 1 / sqrt(x)
template <> __device__ __forceinline__ float drsq<float>(float x) { return __builtin_amdgcn_rsqf(x); }
template <> __device__ __forceinline__ double drsq<double>(double x) { return 1.0 / sqrt(x); }
template <typename T> __device__ __forceinline__ T ddiv(T a, T b);   // a / b
template <> __device__ __forceinline__ float ddiv<float>(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
template <> __device__ __forceinline__ double ddiv<double>(double a, double b) { return a / b; }
template <typename T> __device__ __forceinline__ T dexp(T x);
template <> __device__ __forceinline__ float dexp<float>(float x) {
  return __builtin_amdgcn_exp2f(x * 1.44269504088896341f);
}
template <> __device__ __forceinline__ double dexp<double>(double x) { return exp(x); }
template <typename T> __device__ __forceinline__ T dlog(T x);
template <> __device__ __forceinline__ float dlog<float>(float x) {
  return __builtin_amdgcn_logf(x) * 0.693147180559945309f;
}
template <> __device__ __forceinline__ double dlog<double>(double x) { return log(x); }
template <typename T> __device__ __forceinline__ T dfma(T a, T b, T c);
template <> __device__ __forceinline__ float dfma<float>(float a, float b, float c) { return fmaf(a, b, c); }
template <> __device__ __forceinline__ double dfma<double>(double a, double b, double c) { return fma(a, b, c); }

// Cluster handled by workgroup i of a launch with one workgroup per cluster (n of them).  The
// dispatcher hands consecutive workgroups to the 8 XCDs in turn, and each XCD has its own L2;
// consecutive clusters read neighbouring messages (one cache line holds the same component of
// many consecutive messages), so every XCD takes one contiguous run of clusters instead.
__device__ __forceinline__ int64_t xcd_cluster(int64_t i, int64_t n) {
  constexpr int64_t kXcd = 8;
  const int64_t q = n / kXcd, r = n % kXcd;
  const int64_t x = i % kXcd, j = i / kXcd;
  return x * q + (x < r ? x : r) + j;
}

// Algorithm 2 extrapolation / averaging (1 - th) x + th y, with one explicit rounding
// pattern so that every kernel computing it from the same inputs gets the same bits.
template <typename T>
__device__ __forceinline__ T extrap(T x, T y, T th) {
  return dfma<T>(T(1) - th, x, th * y);
}

// Jacobi rotation parameters for a pair with (real-ified) off-diagonal magnitude r > 0:
// tau = (a_qq - a_pp) / (2 r), t = sign(tau) / (|tau| + sqrt(tau^2 + 1)), c = 1/sqrt(1+t^2).
template <typename T>
__device__ __forceinline__ void rot_params(T app, T aqq, T r, T& t, T& c, T& s) {
  T tau = ddiv<T>(aqq - app, T(2) * r);
  T at = fabs(tau);
  t = ddiv<T>(tau >= T(0) ? T(1) : T(-1), at + dsqrt<T>(dfma<T>(tau, tau, T(1))));
  c = drsq<T>(dfma<T>(t, t, T(1)));
  s = t * c;
}

__host__ __device__ constexpr int pdep_bits(int a, int x, int mask, int nbits) {
  int out = 0, ia = 0, ix = 0;
  for (int b = 0; b < nbits; ++b) {
    if ((mask >> b) & 1) { out |= ((a >> ia) & 1) << b; ++ia; }
    else { out |= ((x >> ix) & 1) << b; ++ix; }
  }
  return out;
}
__host__ __device__ constexpr int pext_bits(int i, int mask, int nbits) {
  int out = 0, k = 0;
  for (int b = 0; b < nbits; ++b)
    if ((mask >> b) & 1) { out |= ((i >> b) & 1) << k; ++k; }
  return out;
}
__host__ __device__ constexpr int log2i(int D) { return D <= 1 ? 0 : 1 + log2i(D / 2); }

// ------------------------------------------------------------------------------------------
// register-resident cluster kernel (one lane per cluster, D_e <= 8)
// ------------------------------------------------------------------------------------------

// Hermitian D x D matrix kept as its packed upper triangle (real parts and imaginary parts);
// every index is a compile-time constant after unrolling, so the storage lives in registers
// and each independent entry is carried once across the sweep loop.
template <typename T, bool CPLX, int D>
struct HMat {
  static constexpr int NT = D * (D + 1) / 2;
  T r[NT];
  T i[CPLX ? NT : 1];
  __device__ __forceinline__ T re(int a, int b) const {
    return a <= b ? r[tri_index(a, b, D)] : r[tri_index(b, a, D)];
  }
  __device__ __forceinline__ T im(int a, int b) const {
    if constexpr (!CPLX) return T(0);
    else return a < b ? i[tri_index(a, b, D)] : (a > b ? -i[tri_index(b, a, D)] : T(0));
  }
  __device__ __forceinline__ void set(int a, int b, T vr, T vi) {
    if (a <= b) {
      r[tri_index(a, b, D)] = vr;
      if constexpr (CPLX) i[tri_index(a, b, D)] = (a == b) ? T(0) : vi;
    } else {
      r[tri_index(b, a, D)] = vr;
      if constexpr (CPLX) i[tri_index(b, a, D)] = -vi;
    }
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      r[k] = T(0);
      if constexpr (CPLX) i[k] = T(0);
    }
  }
};

// packed message / term components <-> HMat (layout: real upper triangle row-major, then the
// imaginary strict upper triangle)
template <typename T, bool CPLX, int D, typename Get>
__device__ __forceinline__ void unpack(Get get, HMat<T, CPLX, D>& M) {
#pragma unroll
  for (int a = 0; a < D; ++a)
#pragma unroll
    for (int b = a; b < D; ++b) M.r[tri_index(a, b, D)] = get(tri_index(a, b, D));
  if constexpr (CPLX) {
#pragma unroll
    for (int a = 0; a < D; ++a) {
      M.i[tri_index(a, a, D)] = T(0);
#pragma unroll
      for (int b = a + 1; b < D; ++b) M.i[tri_index(a, b, D)] = get(D * (D + 1) / 2 + stri_index(a, b, D));
    }
  }
}

template <typename T, bool CPLX, int D, typename Get>
__device__ __forceinline__ void unpack_add(Get get, HMat<T, CPLX, D>& M) {
#pragma unroll
  for (int a = 0; a < D; ++a)
#pragma unroll
    for (int b = a; b < D; ++b) M.r[tri_index(a, b, D)] += get(tri_index(a, b, D));
  if constexpr (CPLX) {
#pragma unroll
    for (int a = 0; a < D; ++a)
#pragma unroll
      for (int b = a + 1; b < D; ++b) M.i[tri_index(a, b, D)] += get(D * (D + 1) / 2 + stri_index(a, b, D));
  }
}

template <typename T, bool CPLX, int D, typename Put>
__device__ __forceinline__ void pack(Put put, const HMat<T, CPLX, D>& M) {
#pragma unroll
  for (int a = 0; a < D; ++a)
#pragma unroll
    for (int b = a; b < D; ++b) put(tri_index(a, b, D), M.r[tri_index(a, b, D)]);
  if constexpr (CPLX) {
#pragma unroll
    for (int a = 0; a < D; ++a)
#pragma unroll
      for (int b = a + 1; b < D; ++b) put(D * (D + 1) / 2 + stri_index(a, b, D), M.i[tri_index(a, b, D)]);
  }
}

// Calls f(integral_constant<int, M>) for the compile-time mask M == mask among the masks that
// select log2(DC) of the log2(DE) site bits (the positions a child can occupy in its parent).
// A flat fold over the candidate masks (no recursion), so everything inlines into the caller.
template <int DE, int DC, int M, typename F>
__device__ __forceinline__ void mask_case(int mask, F& f) {
  if constexpr (__builtin_popcount(M) == log2i(DC)) {
    if (mask == M) {
      f(std::integral_constant<int, M>{});
      // An empty statement that differs per case: without it the compiler merges the cases into
      // one path that indexes the register matrices with a runtime offset, which moves them to
      // scratch memory (12-24 bytes per lane in every register kernel with children).
      __asm__ volatile("; mask case %0" :: "n"(M));
    }
  }
}
template <int DE, int DC, typename F, int... I>
__device__ __forceinline__ void mask_dispatch_seq(int mask, F& f, std::integer_sequence<int, I...>) {
  (mask_case<DE, DC, I + 1>(mask, f), ...);
}
template <int DE, int DC, typename F>
__device__ __forceinline__ void mask_dispatch(int mask, F&& f) {
  mask_dispatch_seq<DE, DC>(mask, f, std::make_integer_sequence<int, DE - 1>{});
}

// theta_e -= 1_{e\f} (x) X for a child whose sites occupy bit mask MASK of e's index.
template <typename T, bool CPLX, int DE, int DC, int MASK>
__device__ __forceinline__ void lift_sub(HMat<T, CPLX, DE>& A, const HMat<T, CPLX, DC>& X) {
  constexpr int NB = log2i(DE);
#pragma unroll
  for (int a = 0; a < DE; ++a)
#pragma unroll
    for (int b = a; b < DE; ++b) {
      if (((a ^ b) & ~MASK & (DE - 1)) == 0) {
        const int x = pext_bits(a, MASK, NB), y = pext_bits(b, MASK, NB);
        A.r[tri_index(a, b, DE)] -= X.re(x, y);
        if constexpr (CPLX) A.i[tri_index(a, b, DE)] -= X.im(x, y);
      }
    }
}

// T = Tr_{e\f} rho for a child at mask MASK.
template <typename T, bool CPLX, int DE, int DC, int MASK>
__device__ __forceinline__ void ptrace_reg(const HMat<T, CPLX, DE>& Rh, HMat<T, CPLX, DC>& Tm) {
  constexpr int NB = log2i(DE);
  constexpr int NR = DE / DC;
#pragma unroll
  for (int a = 0; a < DC; ++a)
#pragma unroll
    for (int b = a; b < DC; ++b) {
      T sr = T(0), si = T(0);
#pragma unroll
      for (int x = 0; x < NR; ++x) {
        sr += Rh.re(pdep_bits(a, x, MASK, NB), pdep_bits(b, x, MASK, NB));
        if constexpr (CPLX) si += Rh.im(pdep_bits(a, x, MASK, NB), pdep_bits(b, x, MASK, NB));
      }
      Tm.set(a, b, sr, si);
    }
}

// 1 / x and 1 / sqrt(x) of a positive normal number: the hardware estimate and two Newton steps
// (within about one unit in the last place), a third of the dependent instructions of the exact
// division and root.
__device__ __forceinline__ double rcp_nr(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double rsq_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// The Jacobi solvers (but the one-lane ones in float and at D = 8) work on the matrix over 2^e,
// e = norm_exponent(||A||_F^2): its norm is then near one, and the elements whose squares underflow, which
// are left as they are or rotated with a phase that is not quite of modulus one, are far under the
// tolerance.  The scaling is exact.  (Unscaled, complex matrices of norm 1e-130, in float 1e-14, never met
// it.)  0 where the squared norm is zero or not finite.
template <typename T>
__device__ __forceinline__ int norm_exponent(T nrm2) {
  int e = 0;
  if (nrm2 > T(0) && isfinite(nrm2)) (void)frexp(nrm2, &e);
  return (e + 1) >> 1;
}

// A rotation that annihilates a_pq = r e^{i phi}: t, c and g = s e^{-i phi} (real: gi unused), from
// the diagonal and a_pq, by Newton reciprocals.  An element below 1e-290 (or, complex, whose square
// is) is left as it is: nz false, t = 0, c = 1, g = 0.
template <bool CPLX>
__device__ __forceinline__ void rot_nr(double app, double aqq, double xr, double xi, bool on, bool& nz, double& rr, double& t,
                                       double& c, double& gr, double& gi) {
  double ir;   // 1 / r
  if constexpr (CPLX) {
    const double r2 = fma(xr, xr, xi * xi);
    nz = !(r2 < 1e-290) && on;
    ir = rsq_nr(nz ? r2 : 1.0);
    rr = r2 * ir;
  } else {
    rr = fabs(xr);
    nz = !(rr < 1e-290) && on;
    ir = rcp_nr(nz ? rr : 1.0);
  }
  const double tau = 0.5 * (aqq - app) * ir;
  double at = fabs(tau);
  at = at > 1e150 ? 1e150 : at;   // its square must not overflow (a NaN stays)
  const double v = fma(at, at, 1.0);
  t = rcp_nr(fma(v, rsq_nr(v), at));
  t = tau >= 0.0 ? t : -t;
  t = nz ? t : 0.0;
  c = nz ? rsq_nr(fma(t, t, 1.0)) : 1.0;
  const double s = t * c;
  if constexpr (CPLX) {
    gr = s * xr * ir;
    gi = -(s * xi * ir);
  } else {
    gr = xr < 0.0 ? -s : s;
    gi = 0.0;
  }
}

// A sweep of the register solver in double for D = 2, 4: rounds r = 1 .. D - 1 of the disjoint pairs
// (p, p ^ r), whose rotations are computed together before they are applied, so that their chains of dependent
// instructions overlap.  (Row by row with exact divisions and roots, a wave of 4 x 4 complex
// clusters took 15 us whatever its size: latency.)  G = [[c, conj(g)], [-g, c]].
template <bool CPLX, int D, bool VEC>
__device__ __forceinline__ void jacobi_sweep_rounds(HMat<double, CPLX, D>& A, double (&ur)[D][D], double (&ui)[D][D]) {
#pragma unroll
  for (int r = 1; r < D; ++r) {
    bool nz[D / 2];
    double rr[D / 2], t[D / 2], c[D / 2], gr[D / 2], gi[D / 2];
    int n = 0;
#pragma unroll
    for (int p = 0; p < D; ++p) {
      const int q = p ^ r;
      if (q < p) continue;
      rot_nr<CPLX>(A.re(p, p), A.re(q, q), A.re(p, q), A.im(p, q), true, nz[n], rr[n], t[n], c[n], gr[n], gi[n]);
      ++n;
    }
    n = 0;
#pragma unroll
    for (int p = 0; p < D; ++p) {
      const int q = p ^ r;
      if (q < p) continue;
      const double cc = c[n], g_r = gr[n], g_i = gi[n];
      const double app = A.re(p, p), aqq = A.re(q, q), xr = A.re(p, q), xi = A.im(p, q);
#pragma unroll
      for (int k = 0; k < D; ++k) {
        if (k == p || k == q) continue;
        // column update (A G); rows follow by Hermitian symmetry
        const double pr = A.re(k, p), pi = A.im(k, p), qr = A.re(k, q), qi = A.im(k, q);
        if constexpr (CPLX) {
          A.set(k, p, fma(g_i, qi, fma(-g_r, qr, cc * pr)), fma(-g_i, qr, fma(-g_r, qi, cc * pi)));
          A.set(k, q, fma(g_i, pi, fma(g_r, pr, cc * qr)), fma(-g_i, pr, fma(g_r, pi, cc * qi)));
        } else {
          A.set(k, p, fma(-g_r, qr, cc * pr), 0.0);
          A.set(k, q, fma(g_r, pr, cc * qr), 0.0);
        }
      }
      A.set(p, p, app - t[n] * rr[n], 0.0);
      A.set(q, q, aqq + t[n] * rr[n], 0.0);
      A.set(p, q, nz[n] ? 0.0 : xr, nz[n] ? 0.0 : xi);
      if constexpr (VEC) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
          const double pr = ur[k][p], qr = ur[k][q];
          if constexpr (CPLX) {
            const double pi = ui[k][p], qi = ui[k][q];
            ur[k][p] = fma(g_i, qi, fma(-g_r, qr, cc * pr));
            ui[k][p] = fma(-g_i, qr, fma(-g_r, qi, cc * pi));
            ur[k][q] = fma(g_i, pi, fma(g_r, pr, cc * qr));
            ui[k][q] = fma(-g_i, pr, fma(g_r, pi, cc * qi));
          } else {
            ur[k][p] = fma(-g_r, qr, cc * pr);
            ur[k][q] = fma(g_r, pr, cc * qr);
          }
        }
      }
      ++n;
    }
  }
}

// One cyclic sweep of two-sided Jacobi rotations over all pairs (p < q), row by row: in float, and at D = 8
// in double (where the registers are full).  Branch-free: a pair with a_pq == 0 gets the identity
// rotation (t = 0, c = 1, s = 0), so the unrolled sweep is straight-line code.  (The dual values of
// float evaluations carry this order's rounding, so it stays.)
template <typename T, bool CPLX, int D, bool VEC>
__device__ __forceinline__ void jacobi_sweep_reg(HMat<T, CPLX, D>& A, T (&ur)[D][D], T (&ui)[D][D]) {
#pragma unroll
  for (int p = 0; p < D - 1; ++p)
#pragma unroll
    for (int q = p + 1; q < D; ++q) {
      const T xr = A.re(p, q);
      const T xi = A.im(p, q);
      const T r = CPLX ? dsqrt<T>(dfma<T>(xr, xr, xi * xi)) : fabs(xr);
      const bool nz = (r != T(0));
      const T rs = nz ? r : T(1);
      // e^{-i phi} with a_pq = r e^{i phi}; real case: sign(a_pq)
      T er, ei;
      if constexpr (CPLX) {
        er = nz ? ddiv<T>(xr, rs) : T(1);
        ei = nz ? ddiv<T>(-xi, rs) : T(0);
      } else {
        er = nz ? copysign(T(1), xr) : T(1);
        ei = T(0);
      }
      const T app = A.re(p, p), aqq = A.re(q, q);
      T t, c, s;
      rot_params<T>(app, aqq, rs, t, c, s);
      t = nz ? t : T(0);
      c = nz ? c : T(1);
      s = nz ? s : T(0);
#pragma unroll
      for (int k = 0; k < D; ++k) {
        if (k == p || k == q) continue;
        // column update (A G): w = a_kq e^{-i phi}; rows follow by Hermitian symmetry
        const T pr = A.re(k, p), pi = A.im(k, p);
        const T qr = A.re(k, q), qi = A.im(k, q);
        const T wr = CPLX ? (qr * er - qi * ei) : qr * er;
        const T wi = CPLX ? (qr * ei + qi * er) : T(0);
        A.set(k, p, c * pr - s * wr, c * pi - s * wi);
        A.set(k, q, s * pr + c * wr, s * pi + c * wi);
      }
      A.set(p, p, app - t * r, T(0));
      A.set(q, q, aqq + t * r, T(0));
      A.set(p, q, nz ? T(0) : xr, nz ? T(0) : xi);
      if constexpr (VEC) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
          const T pr = ur[k][p], pi = CPLX ? ui[k][p] : T(0);
          const T qr = ur[k][q], qi = CPLX ? ui[k][q] : T(0);
          const T wr = CPLX ? (qr * er - qi * ei) : qr * er;
          const T wi = CPLX ? (qr * ei + qi * er) : T(0);
          ur[k][p] = c * pr - s * wr;
          ur[k][q] = s * pr + c * wr;
          if constexpr (CPLX) {
            ui[k][p] = c * pi - s * wi;
            ui[k][q] = s * pi + c * wi;
          }
        }
      }
    }
}

// Squared off-diagonal Frobenius norm, accumulated in FP64 whatever T: the convergence test of
// the FP32 iterations is taken in FP64, so near-degenerate clusters (large rotation angles on
// tiny off-diagonals) are judged on the FP32 matrix without a second rounding of the test.
template <typename T, bool CPLX, int D>
__device__ __forceinline__ double offdiag2(const HMat<T, CPLX, D>& A) {
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a)
#pragma unroll
    for (int b = a + 1; b < D; ++b) {
      const double x = (double)A.r[tri_index(a, b, D)];
      s = fma(x, x, s);
      if constexpr (CPLX) {
        const double y = (double)A.i[tri_index(a, b, D)];
        s = fma(y, y, s);
      }
    }
  return 2.0 * s;
}

template <typename T>
struct FusedCoef { T thp, ithp, thc; };

// Read in place of an absent coefficient row or term block, so that those loads need no branch.
// 64 doubles hold a packed complex 8 x 8 block, the largest a register kernel takes.
static __device__ FusedParams kZeroRow;
static __device__ double kZeroTerms[64];

template <typename T, bool CPLX, int DE, int DC, int MODE>
__device__ void cluster_reg_body(const ClusterArgs<T>& A, int64_t c) {
  constexpr bool VEC = (MODE != MODE_CERTIFY);
  HMat<T, CPLX, DE> H;
  const bool fused = (A.fp != nullptr);
  // iteration coefficients: the fused row, else the stage table row, else the launch's own
  // theta and beta (fused launches are replayed from a graph across stages)
  const bool from_row = fused || A.tab != nullptr;
  const FusedParams* fq = fused ? A.fp : (A.tab ? A.tab : &kZeroRow);
  const FusedCoef<T> fc{(T)fq->theta_prev, (T)fq->inv_thL_prev, (T)fq->theta_cur};
  const T th = from_row ? fc.thc : (T)A.theta;
  const T beta = from_row ? (T)fq->beta : (T)A.beta;
  // Loads are issued in two waves before any arithmetic or store: first every index (h offset,
  // child and parent message ids, masks, marginal slots), then every value, branch-free with a
  // valid index for an empty slot.  One cluster per lane and a cold L2 make each dependent round
  // trip a full memory latency.  This applies to single-site children (at most log2(D_e) of
  // them) and to the first kHoistPar parents of a 2 x 2 cluster; larger cases keep the plain
  // per-slot loops.  The arithmetic and its order are unchanged.
  constexpr bool HOIST_CH = (DC == 2);
  constexpr bool HOIST_PAR = (DE == 2);
  constexpr int MAXCH = HOIST_CH ? log2i(DE) : 1;
  constexpr int NCC = HOIST_CH ? (CPLX ? 4 : 3) : 1;
  constexpr int NCP = HOIST_PAR ? (CPLX ? 4 : 3) : 1;
  constexpr int kHoistPar = 4;
  // Source pointers are chosen per launch so that every hoisted load below is unconditional: an
  // absent array is replaced by one that is present and the value read from it is never used,
  // and an empty slot reads message 0 (a child or parent bucket that exists holds at least one).
  const bool need_g = fused && !A.fused_first;  // the fused form's gradient step
  // ---- index loads ----
  const int64_t ho = A.hoff[c];
  const int32_t gid = A.gid[c];
  const int32_t rs_read = (A.rslot ? A.rslot : A.gid)[c];  // gid: a stand-in of n entries
  const int64_t rs_self = A.rslot ? rs_read : -1;
  int cm[MAXCH], cmask[MAXCH], crs[MAXCH];
  if constexpr (HOIST_CH) {
    const int32_t* rsp = fused ? A.ch_rslot : A.ch;  // the launcher requires ch_rslot when fused
#pragma unroll
    for (int s = 0; s < MAXCH; ++s) {
      const int64_t so = (int64_t)(s < A.maxch ? s : 0) * A.n + c;
      const int m = A.ch[so];
      cm[s] = s < A.maxch ? m : -1;
      cmask[s] = A.chmask[so];
      crs[s] = rsp[so];
    }
  }
  int pm[kHoistPar];
  if constexpr (HOIST_PAR) {
    if (A.maxpar > 0) {
#pragma unroll
      for (int s = 0; s < kHoistPar; ++s) {
        const int m = A.par[(int64_t)(s < A.maxpar ? s : 0) * A.n + c];
        pm[s] = s < A.maxpar ? m : -1;
      }
    } else {
#pragma unroll
      for (int s = 0; s < kHoistPar; ++s) pm[s] = -1;
    }
  }
  // ---- value loads ----
  static_assert((CPLX ? DE * DE : DE * (DE + 1) / 2) <= 64, "term block beyond kZeroTerms");
  const double* hb = ho >= 0 ? A.h + ho : kZeroTerms;
  unpack<T, CPLX, DE>([&](int k) { return (T)hb[k]; }, H);
  T cn[MAXCH][NCC], cz[MAXCH][NCC], cg[MAXCH][NCC];
  if constexpr (HOIST_CH) {
    const T* sN = fused ? A.nu_c_prev : A.nu_c;
    const T* sZ = fused ? A.ze_c_prev : (A.ze_c ? A.ze_c : A.nu_c);
    const T* sR = need_g ? A.Rprev_c : sN;
    const T* sT = need_g ? A.Tprev_c : sN;
#pragma unroll
    for (int s = 0; s < MAXCH; ++s) {
      const int64_t m = cm[s] >= 0 ? cm[s] : 0;
      const int64_t rs = crs[s] >= 0 ? crs[s] : 0;
#pragma unroll
      for (int k = 0; k < NCC; ++k) {
        const int64_t o = (int64_t)k * A.Mc + m;
        cn[s][k] = sN[o];
        cz[s][k] = sZ[o];
        cg[s][k] = sR[need_g ? (int64_t)k * A.Sc + rs : o] - sT[o];
      }
    }
  }
  T pn[kHoistPar][NCP], pz[kHoistPar][NCP], pg[kHoistPar][NCP];
  if constexpr (HOIST_PAR) {
    if (A.maxpar > 0) {
      const T* sN = fused ? A.nu_p_prev : A.nu_p;
      const T* sZ = fused ? A.ze_p_prev : (A.ze_p ? A.ze_p : A.nu_p);
      const T* sR = need_g ? A.Rprev_p : sN;
      const T* sT = need_g ? A.Tprev_p : sN;
      const int64_t rs = rs_self >= 0 ? rs_self : 0;
      T r[NCP];
#pragma unroll
      for (int k = 0; k < NCP; ++k) r[k] = sR[need_g ? (int64_t)k * A.S + rs : (int64_t)k * A.Mp];
#pragma unroll
      for (int s = 0; s < kHoistPar; ++s) {
        const int64_t m = pm[s] >= 0 ? pm[s] : 0;
#pragma unroll
        for (int k = 0; k < NCP; ++k) {
          const int64_t o = (int64_t)k * A.Mp + m;
          pn[s][k] = sN[o];
          pz[s][k] = sZ[o];
          pg[s][k] = r[k] - sT[o];
        }
      }
    }
  }
  // ---- children: subtract lifted messages ----
  if constexpr (HOIST_CH) {
#pragma unroll
    for (int s = 0; s < MAXCH; ++s) {
      if (cm[s] < 0) continue;
      HMat<T, CPLX, DC> X;
      if (fused) {
        unpack<T, CPLX, DC>([&](int k) {
          T nu0 = cn[s][k], ze0 = cz[s][k];
          if (!A.fused_first) {
            ze0 = dfma<T>(cg[s][k], fc.ithp, ze0);
            nu0 = extrap<T>(nu0, ze0, fc.thp);
            const int64_t o = (int64_t)k * A.Mc + cm[s];
            A.nu_c_new[o] = nu0;
            A.ze_c_new[o] = ze0;
          }
          return extrap<T>(nu0, ze0, th);
        }, X);
      } else if (A.ze_c) {
        unpack<T, CPLX, DC>([&](int k) { return extrap<T>(cn[s][k], cz[s][k], th); }, X);
      } else {
        unpack<T, CPLX, DC>([&](int k) { return cn[s][k]; }, X);
      }
      mask_dispatch<DE, DC>(cmask[s], [&](auto mc) __attribute__((always_inline)) {
        lift_sub<T, CPLX, DE, DC, decltype(mc)::value>(H, X);
      });
    }
  } else if constexpr (DC > 0) {
    for (int s = 0; s < A.maxch; ++s) {
      const int m = A.ch[(int64_t)s * A.n + c];
      if (m < 0) continue;
      const int mask = A.chmask[(int64_t)s * A.n + c];
      HMat<T, CPLX, DC> X;
      if (fused) {
        // by (slot, cluster) when available: the same level of dependent loads as ch itself
        const int64_t rs = A.ch_rslot ? A.ch_rslot[(int64_t)s * A.n + c] : A.rslot_of_msg_c[m];
        unpack<T, CPLX, DC>([&](int k) {
          const int64_t o = (int64_t)k * A.Mc + m;
          T nu0 = A.nu_c_prev[o], ze0 = A.ze_c_prev[o];
          if (!A.fused_first) {
            T g = A.Rprev_c[(int64_t)k * A.Sc + rs] - A.Tprev_c[o];
            ze0 = dfma<T>(g, fc.ithp, ze0);
            nu0 = extrap<T>(nu0, ze0, fc.thp);
            A.nu_c_new[o] = nu0;
            A.ze_c_new[o] = ze0;
          }
          return extrap<T>(nu0, ze0, th);
        }, X);
      } else if (A.ze_c) {
        unpack<T, CPLX, DC>([&](int k) {
          const int64_t o = (int64_t)k * A.Mc + m;
          return extrap<T>(A.nu_c[o], A.ze_c[o], th);
        }, X);
      } else {
        unpack<T, CPLX, DC>([&](int k) { return A.nu_c[(int64_t)k * A.Mc + m]; }, X);
      }
      mask_dispatch<DE, DC>(mask, [&](auto mc) __attribute__((always_inline)) {
        lift_sub<T, CPLX, DE, DC, decltype(mc)::value>(H, X);
      });
    }
  }
  // ---- parents: add messages received ----
  int s_par0 = 0;
  if constexpr (HOIST_PAR) {
#pragma unroll
    for (int s = 0; s < kHoistPar; ++s) {
      if (pm[s] < 0) continue;
      if (fused) {
        unpack_add<T, CPLX, DE>([&](int k) {
          T nu0 = pn[s][k], ze0 = pz[s][k];
          if (!A.fused_first) {
            ze0 = dfma<T>(pg[s][k], fc.ithp, ze0);
            nu0 = extrap<T>(nu0, ze0, fc.thp);
          }
          return extrap<T>(nu0, ze0, th);
        }, H);
      } else if (A.ze_p) {
        unpack_add<T, CPLX, DE>([&](int k) { return extrap<T>(pn[s][k], pz[s][k], th); }, H);
      } else {
        unpack_add<T, CPLX, DE>([&](int k) { return pn[s][k]; }, H);
      }
    }
    s_par0 = kHoistPar;
  }
  for (int s = s_par0; s < A.maxpar; ++s) {
    const int m = A.par[(int64_t)s * A.n + c];
    if (m < 0) continue;
    if (fused) {
      unpack_add<T, CPLX, DE>([&](int k) {
        const int64_t o = (int64_t)k * A.Mp + m;
        T nu0 = A.nu_p_prev[o], ze0 = A.ze_p_prev[o];
        if (!A.fused_first) {
          T g = A.Rprev_p[(int64_t)k * A.S + rs_self] - A.Tprev_p[o];
          ze0 = dfma<T>(g, fc.ithp, ze0);
          nu0 = extrap<T>(nu0, ze0, fc.thp);
        }
        return extrap<T>(nu0, ze0, th);
      }, H);
    } else if (A.ze_p) {
      unpack_add<T, CPLX, DE>([&](int k) {
        const int64_t o = (int64_t)k * A.Mp + m;
        return extrap<T>(A.nu_p[o], A.ze_p[o], th);
      }, H);
    } else {
      unpack_add<T, CPLX, DE>([&](int k) { return A.nu_p[(int64_t)k * A.Mp + m]; }, H);
    }
  }
  // ---- a3: cyclic Jacobi (norms and the convergence test in FP64) ----
  double dg = 0.0;
#pragma unroll
  for (int k = 0; k < DE; ++k) {
    const double x = (double)H.r[tri_index(k, k, DE)];
    dg = fma(x, x, dg);
  }
  const double nrm2 = dg + offdiag2<T, CPLX, DE>(H);
  T ur[DE][DE], ui[DE][DE];  // eigenvectors (unused, and removed, without VEC / CPLX)
  if constexpr (VEC) {
#pragma unroll
    for (int i = 0; i < DE; ++i)
#pragma unroll
      for (int j = 0; j < DE; ++j) {
        ur[i][j] = (i == j) ? T(1) : T(0);
        if constexpr (CPLX) ui[i][j] = T(0);
      }
  }
  constexpr bool ROUNDS = std::is_same<T, double>::value && DE <= 4;
  const int ex = ROUNDS ? norm_exponent(nrm2) : 0;
  if constexpr (ROUNDS) {
#pragma unroll
    for (int i = 0; i < DE; ++i)
#pragma unroll
      for (int j = i; j < DE; ++j) H.set(i, j, ldexp(H.re(i, j), -ex), ldexp(H.im(i, j), -ex));
  }
  const double tol2 = A.tol * A.tol * (ROUNDS ? ldexp(nrm2, -2 * ex) : nrm2);
  bool conv = false;
  for (int sweep = 0; sweep <= A.max_sweeps; ++sweep) {
    if (offdiag2<T, CPLX, DE>(H) <= tol2) { conv = true; break; }
    if (sweep == A.max_sweeps) break;
    if constexpr (ROUNDS) {
      jacobi_sweep_rounds<CPLX, DE, VEC>(H, ur, ui);
    } else {
      jacobi_sweep_reg<T, CPLX, DE, VEC>(H, ur, ui);
    }
  }
  if (!conv && A.noconv) atomicAdd(A.noconv, 1ull);
  T lam[DE];
#pragma unroll
  for (int k = 0; k < DE; ++k) {
    lam[k] = H.r[tri_index(k, k, DE)];
    if constexpr (ROUNDS) lam[k] = ldexp(lam[k], ex);
  }
  T lmin = lam[0];
#pragma unroll
  for (int k = 0; k < DE; ++k) lmin = fmin(lmin, lam[k]);
  if (!isfinite((double)lmin) && A.nonfinite) atomicAdd(A.nonfinite, 1ull);
  if constexpr (MODE == MODE_CERTIFY) {
    // The rotated matrix differs from a diagonal one by its remaining off-diagonal part, so
    // lambda_min >= min diag - ||off||_2 >= min diag - ||off||_F (Weyl): the bound holds whether or
    // not the sweeps reached the tolerance.  The first term is the backward error of the rotations.
    A.scal[gid] = (double)lmin;
    A.scal2[gid] = 8.0 * DE * DBL_EPSILON * sqrt((double)nrm2) + ldexp(sqrt(offdiag2<T, CPLX, DE>(H)), ex);
    return;
  } else {
    // ---- a4: marginal weights ----
    T p[DE];
    if constexpr (MODE == MODE_GIBBS) {
      const T b = beta;
      T Z = T(0);
#pragma unroll
      for (int k = 0; k < DE; ++k) { p[k] = dexp<T>(-b * (lam[k] - lmin)); Z += p[k]; }
      const T iZ = ddiv<T>(T(1), Z);
#pragma unroll
      for (int k = 0; k < DE; ++k) p[k] *= iZ;
      if (A.scal) A.scal[gid] = (double)(lmin - ddiv<T>(dlog<T>(Z), b));
    } else {
      const T tau = (T)A.tau_rel * fmax(T(1), dsqrt<T>(nrm2));
      T g = T(0);
#pragma unroll
      for (int k = 0; k < DE; ++k) { p[k] = (lam[k] <= lmin + tau) ? T(1) : T(0); g += p[k]; }
      const T ig = ddiv<T>(T(1), g);
#pragma unroll
      for (int k = 0; k < DE; ++k) p[k] *= ig;
      if (A.scal) A.scal[gid] = (double)lmin;
    }
    // rho = U diag(p) U^H  (reuse H)
#pragma unroll
    for (int i = 0; i < DE; ++i)
#pragma unroll
      for (int j = i; j < DE; ++j) {
        T sr = T(0), si = T(0);
#pragma unroll
        for (int k = 0; k < DE; ++k) {
          const T a_r = ur[i][k] * p[k], a_i = CPLX ? ui[i][k] * p[k] : T(0);
          // (a_r + i a_i) * conj(u_jk)
          sr = dfma<T>(a_r, ur[j][k], sr);
          if constexpr (CPLX) {
            sr = dfma<T>(a_i, ui[j][k], sr);
            si = dfma<T>(a_i, ur[j][k], si);
            si = dfma<T>(-a_r, ui[j][k], si);
          }
        }
        H.set(i, j, sr, si);
      }
    // ---- outputs: own marginal ----
    if (rs_self >= 0 && A.R) {
      pack<T, CPLX, DE>([&](int k, T v) { A.R[(int64_t)k * A.S + rs_self] = v; }, H);
    }
    if (A.marg) {
      T* mo = A.marg + A.marg_off[gid];
      pack<T, CPLX, DE>([&](int k, T v) { mo[k] = v; }, H);
    }
    // ---- a5: partial traces onto the children ----
    if constexpr (DC > 0) {
      if (A.Tout) {
        // (unrolled, so that the hoisted slot arrays are indexed by constants and stay in registers)
#pragma unroll
        for (int s = 0; s < (HOIST_CH ? MAXCH : A.maxch); ++s) {
          int m, mask;
          if constexpr (HOIST_CH) {
            m = cm[s];
            mask = cmask[s];
          } else {
            m = A.ch[(int64_t)s * A.n + c];
            mask = m >= 0 ? A.chmask[(int64_t)s * A.n + c] : 0;
          }
          if (m < 0) continue;
          HMat<T, CPLX, DC> Tm;
          mask_dispatch<DE, DC>(mask, [&](auto mc) __attribute__((always_inline)) {
            ptrace_reg<T, CPLX, DE, DC, decltype(mc)::value>(H, Tm);
          });
          pack<T, CPLX, DC>([&](int k, T v) { A.Tout[(int64_t)k * A.Mc + m] = v; }, Tm);
        }
      }
    }
  }
}

template <typename T, bool CPLX, int DE, int DC, int MODE>
__global__ __launch_bounds__(256) void k_cluster_reg(ClusterArgs<T> A) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c < A.n) cluster_reg_body<T, CPLX, DE, DC, MODE>(A, c);
}

// ------------------------------------------------------------------------------------------
// wave-per-cluster LDS kernel (8 <= De <= 64)
// ------------------------------------------------------------------------------------------

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// Reductions over the 64 lanes of a wave built from DPP row operations (xor 1, xor 2, mirror
// within 8 lanes, mirror within 16 lanes: every lane of a row of 16 ends with the same sum) and
// four readlanes, instead of six LDS-crossbar shuffles.  Every lane of the wave must be active;
// the result is wave-uniform.
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double readlane_d(double v, int lane) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double row_sum16(double v) {
  v += dpp_mov<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp_mov<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp_mov<0x141>(v);   // row_half_mirror
  v += dpp_mov<0x140>(v);   // row_mirror
  return v;
}
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v = row_sum16(v);
  return (readlane_d(v, 0) + readlane_d(v, 16)) + (readlane_d(v, 32) + readlane_d(v, 48));
}
__device__ __forceinline__ double wave_min_dpp(double v) {
  v = fmin(v, dpp_mov<0xB1>(v));
  v = fmin(v, dpp_mov<0x4E>(v));
  v = fmin(v, dpp_mov<0x141>(v));
  v = fmin(v, dpp_mov<0x140>(v));
  return fmin(fmin(readlane_d(v, 0), readlane_d(v, 16)), fmin(readlane_d(v, 32), readlane_d(v, 48)));
}
__device__ __forceinline__ double wave_max_rows(double v) {   // v already uniform within each row
  return fmax(fmax(readlane_d(v, 0), readlane_d(v, 16)), fmax(readlane_d(v, 32), readlane_d(v, 48)));
}

template <typename T>
__device__ __forceinline__ T wave_min(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ __forceinline__ int pdep_rt(int a, int x, int mask, int nbits) {
  int out = 0, ia = 0, ix = 0;
  for (int b = 0; b < nbits; ++b) {
    if ((mask >> b) & 1) { out |= ((a >> ia) & 1) << b; ++ia; }
    else { out |= ((x >> ix) & 1) << b; ++ix; }
  }
  return out;
}
__device__ __forceinline__ int pext_rt(int i, int mask, int nbits) {
  int out = 0, k = 0;
  for (int b = 0; b < nbits; ++b)
    if ((mask >> b) & 1) { out |= ((i >> b) & 1) << k; ++k; }
  return out;
}

// round-robin tournament: round r (0..D-2), pair k (0..D/2-1) -> (p < q); every pair once.
__device__ __forceinline__ void rr_pair(int r, int k, int D, int& p, int& q) {
  if (k == 0) { p = r; q = D - 1; }
  else { p = (r + k) % (D - 1); q = (r - k + (D - 1)) % (D - 1); }
  if (p > q) { int t = p; p = q; q = t; }
}

// element (a, b) of a packed Hermitian stored at stride `st` (component k at base[k*st])
template <typename T, typename Get>
__device__ __forceinline__ void herm_elem(Get get, int a, int b, int D, bool cplx, T& vr, T& vi) {
  if (a <= b) {
    vr = get(tri_index(a, b, D));
    vi = (cplx && a < b) ? get(D * (D + 1) / 2 + stri_index(a, b, D)) : T(0);
  } else {
    vr = get(tri_index(b, a, D));
    vi = cplx ? -get(D * (D + 1) / 2 + stri_index(b, a, D)) : T(0);
  }
}

// Element (a, b) of a packed Hermitian without branches: both addresses are always valid, the
// imaginary part is selected (conjugated below the diagonal, zero on it).
template <typename T, bool CPLX, typename Get>
__device__ __forceinline__ void herm_elem_bf(Get get, int a, int b, int D, T& vr, T& vi) {
  const int lo = min(a, b), hi = max(a, b);
  vr = get(tri_index(lo, hi, D));
  if constexpr (CPLX) {
    const T v = get(D * (D + 1) / 2 + (lo < hi ? stri_index(lo, hi, D) : 0));
    vi = a < b ? v : (a > b ? -v : T(0));
  } else {
    vi = T(0);
  }
}

// ---- shared pieces of the LDS kernels ----
//
// A 64-lane wave holds G = 64/W clusters, W lanes each (W is a power of two, 8..64); lane `lt`
// of a cluster strides over that cluster's entries by W.  Every loop whose trip count depends
// on the data is made wave-uniform (per-cluster `done` flags, exit on __all), so barriers and
// cross-lane shuffles always see the whole wave.

template <int W, typename T>
__device__ __forceinline__ T seg_sum(T v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
template <int W, typename T>
__device__ __forceinline__ T seg_max(T v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
template <int W, typename T>
__device__ __forceinline__ T seg_min(T v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}

// theta_e = [h_e] - sum_children 1 (x) x_{e->f} + sum_parents x_{g->e}, written to (dr, di) with
// leading dimension DE+1; x = extrap(nu, zeta, th) when zeta is given.  Off-diagonal message
// elements are scaled by `offs` (packed-coordinate cotangents use 1/2).  Returns this lane's
// share of the squared Frobenius norm.
template <typename T, bool CPLX, int DE, int W>
__device__ T lds_assemble(const ClusterArgs<T>& A, int64_t c, int lt, const T* xc, const T* zc, const T* xp,
                          const T* zp, T th, bool with_h, T offs, T* dr, T* di) {
  constexpr int LD = DE + 1;
  constexpr int NB = log2i(DE);
  // A lane's elements in groups of up to 8 whose loads are issued together: every candidate element
  // is loaded from a valid address and then selected, and the index of a child or parent message is
  // read once per group (element by element, with a branch per child, the assembly was a chain of
  // dependent loads: half of the 45 us the adjoint of 8192 8 x 8 clusters took).
  constexpr int NE = DE * DE > W ? DE * DE / W : 1;
  constexpr int CH = NE < 8 ? NE : 8;
  static_assert(NE % CH == 0, "whole groups");
  if (W > DE * DE && lt >= DE * DE) return T(0);
  const int64_t ho = with_h ? A.hoff[c] : -1;
  const int Dc = A.Dc;
  T my_n2 = T(0);
  for (int base = 0; base < NE; base += CH) {
    T vr[CH], vi[CH];
#pragma unroll
    for (int e = 0; e < CH; ++e) vr[e] = vi[e] = T(0);
    if (ho >= 0) {
      const double* h = A.h + ho;
#pragma unroll
      for (int e = 0; e < CH; ++e) {
        const int idx = lt + (base + e) * W;
        herm_elem_bf<T, CPLX>([&](int k) { return (T)h[k]; }, idx / DE, idx % DE, DE, vr[e], vi[e]);
      }
    }
    for (int s = 0; s < A.maxch; ++s) {
      const int m = A.ch[(int64_t)s * A.n + c];
      const int mask = A.chmask[(int64_t)s * A.n + c];
      if (m < 0) continue;
      T er[CH], ei[CH];
#pragma unroll
      for (int e = 0; e < CH; ++e) {
        const int idx = lt + (base + e) * W;
        const int a = pext_rt(idx / DE, mask, NB), b = pext_rt(idx % DE, mask, NB);
        if (zc)
          herm_elem_bf<T, CPLX>([&](int k) { const int64_t o = (int64_t)k * A.Mc + m;
                                             return extrap<T>(xc[o], zc[o], th); }, a, b, Dc, er[e], ei[e]);
        else
          herm_elem_bf<T, CPLX>([&](int k) { return xc[(int64_t)k * A.Mc + m]; }, a, b, Dc, er[e], ei[e]);
      }
#pragma unroll
      for (int e = 0; e < CH; ++e) {
        const int idx = lt + (base + e) * W, i = idx / DE, j = idx % DE;
        const bool ok = ((i ^ j) & ~mask & (DE - 1)) == 0;
        const T sc = i == j ? T(1) : offs;   // a lifted element is diagonal where the child's is
        vr[e] -= ok ? sc * er[e] : T(0);
        if constexpr (CPLX) vi[e] -= ok ? sc * ei[e] : T(0);
      }
    }
    for (int s = 0; s < A.maxpar; ++s) {
      const int m = A.par[(int64_t)s * A.n + c];
      if (m < 0) continue;
      T er[CH], ei[CH];
#pragma unroll
      for (int e = 0; e < CH; ++e) {
        const int idx = lt + (base + e) * W;
        if (zp)
          herm_elem_bf<T, CPLX>([&](int k) { const int64_t o = (int64_t)k * A.Mp + m;
                                             return extrap<T>(xp[o], zp[o], th); }, idx / DE, idx % DE, DE, er[e], ei[e]);
        else
          herm_elem_bf<T, CPLX>([&](int k) { return xp[(int64_t)k * A.Mp + m]; }, idx / DE, idx % DE, DE, er[e], ei[e]);
      }
#pragma unroll
      for (int e = 0; e < CH; ++e) {
        const int idx = lt + (base + e) * W;
        const T sc = idx / DE == idx % DE ? T(1) : offs;
        vr[e] += sc * er[e];
        if constexpr (CPLX) vi[e] += sc * ei[e];
      }
    }
#pragma unroll
    for (int e = 0; e < CH; ++e) {
      const int idx = lt + (base + e) * W, i = idx / DE, j = idx % DE;
      dr[i * LD + j] = vr[e];
      if constexpr (CPLX) di[i * LD + j] = vi[e];
      my_n2 = dfma<T>(vr[e], vr[e], my_n2);
      if constexpr (CPLX) my_n2 = dfma<T>(vi[e], vi[e], my_n2);
    }
  }
  return my_n2;
}

// Rotation scratch of the round-robin parallel Jacobi (one per cluster).
template <typename T, int NP>
struct JacobiScratch {
  T c[NP], s[NP], er[NP], ei[NP], app[NP], aqq[NP];
  int p[NP], q[NP];
};

// Cyclic two-sided Jacobi on the LDS matrix (sar, sai) with eigenvectors accumulated in
// (sur, sui) when VEC.  Each round applies the DE/2 disjoint rotations of a round-robin
// tournament in parallel: columns (A G, U G), then rows (G^H A), then the exact 2x2 blocks.
// `done` clusters (converged, capped, or absent) skip the work but keep the wave together.
// Returns true when the off-diagonal norm fell below tol2 within max_sweeps sweeps.
template <typename T, bool CPLX, int DE, bool VEC, int W>
__device__ bool lds_jacobi(T* sar, T* sai, T* sur, T* sui, JacobiScratch<T, DE / 2>& J, double tol2, int max_sweeps,
                           int lt, bool active) {
  constexpr int LD = DE + 1;
  constexpr int NP = DE / 2;
  bool done = !active, conv = false;
  for (int sweep = 0;; ++sweep) {
    double off = 0.0;   // the convergence test in FP64 whatever T
    if (!done) {
      for (int idx = lt; idx < DE * DE; idx += W) {
        const int i = idx / DE, j = idx % DE;
        if (i != j) {
          const double x = (double)sar[i * LD + j];
          off = fma(x, x, off);
          if constexpr (CPLX) {
            const double y = (double)sai[i * LD + j];
            off = fma(y, y, off);
          }
        }
      }
    }
    off = seg_sum<W>(off);
    if (!done) {
      if (off <= tol2) { done = true; conv = true; }
      else if (sweep >= max_sweeps) { done = true; }
    }
    if (__all(done ? 1 : 0)) break;
    for (int r = 0; r < DE - 1; ++r) {
      if (!done) {
        for (int k = lt; k < NP; k += W) {
          int p, q;
          rr_pair(r, k, DE, p, q);
          const T xr = sar[p * LD + q];
          const T xi = CPLX ? sai[p * LD + q] : T(0);
          const T rr = CPLX ? dsqrt<T>(dfma<T>(xr, xr, xi * xi)) : fabs(xr);
          T t = T(0), cc = T(1), ss = T(0), er = T(1), ei = T(0);
          const T app = sar[p * LD + p], aqq = sar[q * LD + q];
          if (rr != T(0)) {
            rot_params<T>(app, aqq, rr, t, cc, ss);
            er = CPLX ? ddiv<T>(xr, rr) : copysign(T(1), xr);
            ei = CPLX ? ddiv<T>(-xi, rr) : T(0);
          }
          J.p[k] = p; J.q[k] = q;
          J.c[k] = cc; J.s[k] = ss; J.er[k] = er; J.ei[k] = ei;
          J.app[k] = app - t * rr;
          J.aqq[k] = aqq + t * rr;
        }
      }
      __syncthreads();
      if (!done) {
        // columns: A <- A G, U <- U G  (w = x_q e^{-i phi})
        for (int idx = lt; idx < DE * NP; idx += W) {
          const int i = idx % DE, k = idx / DE;
          const int p = J.p[k], q = J.q[k];
          const T cc = J.c[k], ss = J.s[k], er = J.er[k], ei = J.ei[k];
          {
            T pr = sar[i * LD + p], qr = sar[i * LD + q];
            T pi = CPLX ? sai[i * LD + p] : T(0), qi = CPLX ? sai[i * LD + q] : T(0);
            T wr = CPLX ? qr * er - qi * ei : qr * er;
            T wi = CPLX ? qr * ei + qi * er : T(0);
            sar[i * LD + p] = cc * pr - ss * wr;
            sar[i * LD + q] = ss * pr + cc * wr;
            if constexpr (CPLX) {
              sai[i * LD + p] = cc * pi - ss * wi;
              sai[i * LD + q] = ss * pi + cc * wi;
            }
          }
          if constexpr (VEC) {
            T pr = sur[i * LD + p], qr = sur[i * LD + q];
            T pi = CPLX ? sui[i * LD + p] : T(0), qi = CPLX ? sui[i * LD + q] : T(0);
            T wr = CPLX ? qr * er - qi * ei : qr * er;
            T wi = CPLX ? qr * ei + qi * er : T(0);
            sur[i * LD + p] = cc * pr - ss * wr;
            sur[i * LD + q] = ss * pr + cc * wr;
            if constexpr (CPLX) {
              sui[i * LD + p] = cc * pi - ss * wi;
              sui[i * LD + q] = ss * pi + cc * wi;
            }
          }
        }
      }
      __syncthreads();
      if (!done) {
        // rows: A <- G^H A  (w = x_q e^{+i phi})
        for (int idx = lt; idx < DE * NP; idx += W) {
          const int j = idx % DE, k = idx / DE;
          const int p = J.p[k], q = J.q[k];
          const T cc = J.c[k], ss = J.s[k], er = J.er[k], ei = -J.ei[k];
          T pr = sar[p * LD + j], qr = sar[q * LD + j];
          T pi = CPLX ? sai[p * LD + j] : T(0), qi = CPLX ? sai[q * LD + j] : T(0);
          T wr = CPLX ? qr * er - qi * ei : qr * er;
          T wi = CPLX ? qr * ei + qi * er : T(0);
          sar[p * LD + j] = cc * pr - ss * wr;
          sar[q * LD + j] = ss * pr + cc * wr;
          if constexpr (CPLX) {
            sai[p * LD + j] = cc * pi - ss * wi;
            sai[q * LD + j] = ss * pi + cc * wi;
          }
        }
      }
      __syncthreads();
      if (!done) {
        for (int k = lt; k < NP; k += W) {
          const int p = J.p[k], q = J.q[k];
          sar[p * LD + p] = J.app[k];
          sar[q * LD + q] = J.aqq[k];
          sar[p * LD + q] = T(0);
          sar[q * LD + p] = T(0);
          if constexpr (CPLX) {
            sai[p * LD + p] = T(0); sai[q * LD + q] = T(0);
            sai[p * LD + q] = T(0); sai[q * LD + p] = T(0);
          }
        }
      }
      __syncthreads();
    }
  }
  return conv;
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <typename F, int... I>
__device__ __forceinline__ void static_for_seq(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// v of lane l ^ M, M < 16, by DPP moves: quad_perm (M = 1, 2, 3), row_half_mirror (7) and row_mirror
// (15) within the 16-lane rows, and their products.
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_any(T v) {
  if constexpr (sizeof(T) == 8) {
    return dpp_mov<CTRL>(v);
  } else {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
  }
}
template <int M, typename T>
__device__ __forceinline__ T xor_lane(T v) {
  static_assert(M >= 0 && M < 16, "within a row of 16 lanes");
  if constexpr (M == 0) return v;
  else if constexpr (M == 1) return dpp_any<0xB1>(v);
  else if constexpr (M == 2) return dpp_any<0x4E>(v);
  else if constexpr (M == 3) return dpp_any<0x1B>(v);
  else if constexpr (M < 8) return dpp_any<0x141>(xor_lane<7 ^ M>(v));
  else return dpp_any<0x140>(xor_lane<15 ^ M>(v));
}

// Cyclic two-sided Jacobi of a DE x DE matrix (DE = 2, 4, 8, 16) on DE lanes, in registers.  Lane j
// holds column j of A and of U, register k the element of row j ^ k, so that with the pairs
// (j, j ^ r), r = 1 .. DE - 1, of a sweep the diagonal is register 0, the element to annihilate
// register r, the partner's element of the same row its register k ^ r, and the row rotations act on
// registers k and k ^ r: every index is a constant and every exchange an xor of the lane.  (In
// LDS with four barriers per round the 8 x 8 problem was bound by their latency: 8192 of them
// with vectors and the adjoint's products took 83 us.)  Rotations, exact 2 x 2 blocks and the FP64
// convergence test are those of the register kernel; G = [[c, conj(g)], [-g, c]], g = s e^{-i phi}.
// The matrix is read from LDS (sar, sai) and written back with U; lanes lt >= DE of a cluster's
// group and inactive clusters take part with a zero matrix.  Returns true (lanes lt < DE) when the
// off-diagonal norm fell below tol times the matrix's, nrm2 its square, within max_sweeps sweeps.
template <typename T, bool CPLX, int DE, bool VEC>
__device__ bool xor_jacobi(T* sar, T* sai, T* sur, T* sui, double tol, T nrm2, int max_sweeps, int lt, bool active) {
  constexpr int LD = DE + 1;
  const int ex = norm_exponent(nrm2);
  const double tol2 = tol * tol * ldexp((double)nrm2, -2 * ex);
  const bool mine = active && lt < DE;
  const int j = lt & (DE - 1);
  T ar[DE], ai[CPLX ? DE : 1], ur[VEC ? DE : 1], ui[VEC && CPLX ? DE : 1];
#pragma unroll
  for (int k = 0; k < DE; ++k) {
    const int o = (j ^ k) * LD + j;
    ar[k] = mine ? ldexp(sar[o], -ex) : T(0);
    if constexpr (CPLX) ai[k] = mine ? ldexp(sai[o], -ex) : T(0);
    if constexpr (VEC) ur[k] = k == 0 ? T(1) : T(0);
    if constexpr (VEC && CPLX) ui[k] = T(0);
  }
  bool done = !mine, conv = false;
  for (int sweep = 0;; ++sweep) {
    double off = 0.0;   // the convergence test in FP64 whatever T
#pragma unroll
    for (int k = 1; k < DE; ++k) {
      off = fma((double)ar[k], (double)ar[k], off);
      if constexpr (CPLX) off = fma((double)ai[k], (double)ai[k], off);
    }
    static_for<log2i(DE)>([&](auto b) { off += xor_lane<(1 << decltype(b)::value)>(off); });
    if (!done) {
      if (off <= tol2) { done = true; conv = true; }
      else if (sweep >= max_sweeps) { done = true; }
    }
    if (__all(done ? 1 : 0)) break;
    static_for<DE - 1>([&](auto rc) {
      constexpr int r = decltype(rc)::value + 1;
      constexpr int HB = 1 << log2i(r);                // j < j ^ r where this bit of j is clear
      const bool isp = (j & HB) == 0;
      const T dx = xor_lane<r>(ar[0]), ox = xor_lane<r>(ar[r]);
      const T app = isp ? ar[0] : dx, aqq = isp ? dx : ar[0];
      const T xr = isp ? ar[r] : ox;                   // a_qp, as lane p holds it, for both lanes
      T xi = T(0);
      if constexpr (CPLX) {
        const T oi = xor_lane<r>(ai[r]);
        xi = -(isp ? ai[r] : oi);                      // Im a_pq
      }
      // r = |a_pq| (an element below `tiny`, or whose square underflows, is left as it is), then
      // rot_params with the reciprocals that the whole wave waits for done by Newton steps
      constexpr bool dbl = sizeof(T) == 8;
      const T tiny = dbl ? T(1e-290) : T(FLT_MIN);
      T rr, ir, t, c;   // r, 1 / r
      bool nz;
      if constexpr (CPLX) {
        const T r2 = dfma<T>(xr, xr, xi * xi);
        nz = !(r2 < tiny) && !done;
        if constexpr (dbl) ir = rsq_nr(nz ? r2 : T(1));
        else ir = drsq<T>(nz ? r2 : T(1));
        rr = r2 * ir;
      } else {
        rr = fabs(xr);
        nz = !(rr < tiny) && !done;
        if constexpr (dbl) ir = rcp_nr(nz ? rr : T(1));
        else ir = ddiv<T>(T(1), nz ? rr : T(1));
      }
      {
        const T tau = T(0.5) * (aqq - app) * ir;
        T at = fabs(tau);
        if constexpr (dbl) {
          at = at > 1e150 ? 1e150 : at;   // its square must not overflow (a NaN stays)
          const T v = fma(at, at, 1.0);
          t = rcp_nr(fma(v, rsq_nr(v), at));
        } else {
          t = ddiv<T>(T(1), at + dsqrt<T>(dfma<T>(tau, tau, T(1))));
        }
        t = tau >= T(0) ? t : -t;
        t = nz ? t : T(0);
        if constexpr (dbl) c = rsq_nr(fma(t, t, 1.0));
        else c = drsq<T>(dfma<T>(t, t, T(1)));
        c = nz ? c : T(1);
      }
      const T s = t * c;
      // own column: c own + gam other, gam = -g (lane p) or conj(g) (lane q)
      T gr, gi = T(0);
      if constexpr (CPLX) {
        gr = s * xr * ir;
        gi = s * xi * ir;
        gr = isp ? -gr : gr;
      } else {
        gr = ((xr < T(0)) == isp) ? s : -s;
      }
      const auto cols = [&](auto& vr, auto& vi) {
#pragma unroll
        for (int k = 0; k < DE; ++k) {
          if (k > (k ^ r)) continue;
          const T xk = xor_lane<r>(vr[k ^ r]), xq = xor_lane<r>(vr[k]);
          if constexpr (CPLX) {
            const T yk = xor_lane<r>(vi[k ^ r]), yq = xor_lane<r>(vi[k]);
            const T nk = dfma<T>(-gi, yk, dfma<T>(gr, xk, c * vr[k])), mk = dfma<T>(gi, xk, dfma<T>(gr, yk, c * vi[k]));
            const T nq = dfma<T>(-gi, yq, dfma<T>(gr, xq, c * vr[k ^ r])),
                    mq = dfma<T>(gi, xq, dfma<T>(gr, yq, c * vi[k ^ r]));
            vr[k] = nk;
            vi[k] = mk;
            vr[k ^ r] = nq;
            vi[k ^ r] = mq;
          } else {
            const T nk = dfma<T>(gr, xk, c * vr[k]);
            vr[k ^ r] = dfma<T>(gr, xq, c * vr[k ^ r]);
            vr[k] = nk;
          }
        }
      };
      cols(ar, ai);
      if constexpr (VEC) cols(ur, ui);
      // rows i = j ^ k and i ^ r, with lane i's c and gam
      static_for<DE>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr (k < (k ^ r)) {
          const T ck = xor_lane<k>(c), hr = xor_lane<k>(gr);
          const T x = ar[k], y = ar[k ^ r];
          if constexpr (CPLX) {
            const T hi = xor_lane<k>(gi);
            const T xi2 = ai[k], yi2 = ai[k ^ r];
            ar[k] = dfma<T>(hi, yi2, dfma<T>(hr, y, ck * x));
            ai[k] = dfma<T>(-hi, y, dfma<T>(hr, yi2, ck * xi2));
            ar[k ^ r] = dfma<T>(hi, xi2, dfma<T>(-hr, x, ck * y));
            ai[k ^ r] = dfma<T>(-hi, x, dfma<T>(-hr, xi2, ck * yi2));
          } else {
            ar[k] = dfma<T>(hr, y, ck * x);
            ar[k ^ r] = dfma<T>(-hr, x, ck * y);
          }
        }
      });
      ar[0] = isp ? app - t * rr : aqq + t * rr;
      ar[r] = nz ? T(0) : ar[r];
      if constexpr (CPLX) {
        ai[0] = T(0);
        ai[r] = nz ? T(0) : ai[r];
      }
    });
  }
  if (mine) {
#pragma unroll
    for (int k = 0; k < DE; ++k) {
      const int o = (j ^ k) * LD + j;
      sar[o] = ldexp(ar[k], ex);
      if constexpr (CPLX) sai[o] = ldexp(ai[k], ex);
      if constexpr (VEC) sur[o] = ur[k];
      if constexpr (VEC && CPLX) sui[o] = ui[k];
    }
  }
  __syncthreads();
  return conv;
}

// Rotation scratch of a kernel: none where the matrix is solved in registers.
template <typename T, int DE, bool REG>
using ScratchFor = JacobiScratch<T, (REG && DE <= 16 ? 1 : DE / 2)>;

// The identity into (sur, sui) where the solve is in LDS, before the barrier that precedes it.
template <typename T, bool CPLX, int DE, bool VEC, int W, bool REG>
__device__ __forceinline__ void init_vectors(T* sur, T* sui, int lt, bool active) {
  if constexpr (VEC && !(REG && DE <= 16)) {
    if (active)
      for (int idx = lt; idx < DE * DE; idx += W) {
        const int i = idx / DE, j = idx % DE;
        sur[i * (DE + 1) + j] = (i == j) ? T(1) : T(0);
        if constexpr (CPLX) sui[i * (DE + 1) + j] = T(0);
      }
  }
}

// Eigenvalues onto the diagonal of (sar, sai), eigenvectors into (sur, sui) when VEC (see init_vectors),
// W >= min(DE, 64) lanes per cluster: in registers up to DE = 16 where the caller says so (REG), else in LDS.
// In LDS stay float ground projectors and spin-1 clusters, for the rounding that their order of rotations
// puts into the values they return, and complex or 16-dimensional clusters with a whole wave.
template <typename T, bool CPLX, int DE, bool VEC, int W, bool REG>
__device__ __forceinline__ bool cluster_jacobi(T* sar, T* sai, T* sur, T* sui, ScratchFor<T, DE, REG>& J, double tol,
                                               T nrm2, int max_sweeps, int lt, bool active) {
  if constexpr (REG && DE <= 16) {
    static_assert(W >= DE, "one lane per column");
    return xor_jacobi<T, CPLX, DE, VEC>(sar, sai, sur, sui, tol, nrm2, max_sweeps, lt, active);
  } else {
    const int ex = norm_exponent(nrm2);
    const auto scale = [&](int e) {
      if (active)
        for (int idx = lt; idx < DE * DE; idx += W) {
          const int o = idx / DE * (DE + 1) + idx % DE;
          sar[o] = ldexp(sar[o], e);
          if constexpr (CPLX) sai[o] = ldexp(sai[o], e);
        }
      __syncthreads();
    };
    scale(-ex);
    const bool conv = lds_jacobi<T, CPLX, DE, VEC, W>(sar, sai, sur, sui, J, tol * tol * ldexp((double)nrm2, -2 * ex),
                                                      max_sweeps, lt, active);
    scale(ex);
    return conv;
  }
}

// component k of a packed D x D Hermitian -> (i, j, imaginary?)
__device__ __forceinline__ void decode_comp(int k, int D, int& i, int& j, bool& im) {
  im = false;
  i = 0;
  if (k >= D * (D + 1) / 2) { im = true; k -= D * (D + 1) / 2; }
  const int rowlen0 = im ? D - 1 : D;
  while (k >= rowlen0 - i) { k -= rowlen0 - i; ++i; }
  j = i + k + (im ? 1 : 0);
}

// Write a cluster matrix Y (LDS) to its consumers: own marginal slot (if it has parents),
// the per-cluster output buffer, and the partial traces onto every child.
template <typename T, bool CPLX, int DE, int W>
__device__ void lds_outputs(const ClusterArgs<T>& A, int64_t c, int lt, int32_t gid, const T* yr, const T* yi) {
  constexpr int LD = DE + 1;
  constexpr int NB = log2i(DE);
  const int64_t rs_self = A.rslot ? A.rslot[c] : -1;
  constexpr int NCE = n_comps(DE, CPLX);
  for (int k = lt; k < NCE; k += W) {
    int i, j;
    bool im;
    decode_comp(k, DE, i, j, im);
    const T v = im ? yi[i * LD + j] : yr[i * LD + j];
    if (rs_self >= 0 && A.R) A.R[(int64_t)k * A.S + rs_self] = v;
    if (A.marg) A.marg[A.marg_off[gid] + k] = v;
  }
  const int Dc = A.Dc;
  if (A.Tout && Dc > 0) {
    const int NR = DE / Dc;
    const int NCC = CPLX ? Dc * Dc : Dc * (Dc + 1) / 2;
    for (int s = 0; s < A.maxch; ++s) {
      const int m = A.ch[(int64_t)s * A.n + c];
      if (m < 0) continue;
      const int mask = A.chmask[(int64_t)s * A.n + c];
      for (int k = lt; k < NCC; k += W) {
        int a, b;
        bool im;
        decode_comp(k, Dc, a, b, im);
        T sum = T(0);
        for (int x = 0; x < NR; ++x) {
          const int i = pdep_rt(a, x, mask, NB), j = pdep_rt(b, x, mask, NB);
          sum += im ? yi[i * LD + j] : yr[i * LD + j];
        }
        A.Tout[(int64_t)k * A.Mc + m] = sum;
      }
    }
  }
}

// Marginal weights from the eigenvalues on the diagonal of sar: Gibbs p (returns F_beta) or the
// normalised ground-space indicator (returns lambda_min).  Weights go to sp[].
template <typename T, int DE, int MODE, int W>
__device__ T lds_weights(const T* sar, T* sp, T lmin, T beta, T tau, int lt, bool active) {
  constexpr int LD = DE + 1;
  T w = T(0);
  if (active) {
    if constexpr (MODE == MODE_GIBBS) {
      for (int k = lt; k < DE; k += W) { T v = dexp<T>(-beta * (sar[k * LD + k] - lmin)); sp[k] = v; w += v; }
    } else {
      for (int k = lt; k < DE; k += W) { T v = (sar[k * LD + k] <= lmin + tau) ? T(1) : T(0); sp[k] = v; w += v; }
    }
  }
  const T Z = seg_sum<W>(w);
  __syncthreads();
  if (active)
    for (int k = lt; k < DE; k += W) sp[k] = ddiv<T>(sp[k], Z);
  __syncthreads();
  if constexpr (MODE == MODE_GIBBS) return lmin - ddiv<T>(dlog<T>(Z), beta);
  else return lmin;
}

// (yr, yi) = U diag(sp) U^H
template <typename T, bool CPLX, int DE, int W>
__device__ void lds_rebuild(const T* sur, const T* sui, const T* sp, T* yr, T* yi, int lt) {
  constexpr int LD = DE + 1;
  for (int idx = lt; idx < DE * DE; idx += W) {
    const int i = idx / DE, j = idx % DE;
    T sr = T(0), si = T(0);
    for (int k = 0; k < DE; ++k) {
      const T a_r = sur[i * LD + k] * sp[k];
      const T a_i = CPLX ? sui[i * LD + k] * sp[k] : T(0);
      sr = dfma<T>(a_r, sur[j * LD + k], sr);
      if constexpr (CPLX) {
        sr = dfma<T>(a_i, sui[j * LD + k], sr);
        si = dfma<T>(a_i, sur[j * LD + k], si);
        si = dfma<T>(-a_r, sui[j * LD + k], si);
      }
    }
    yr[i * LD + j] = sr;
    if constexpr (CPLX) yi[i * LD + j] = (i == j) ? T(0) : si;
  }
}

// W lanes per cluster, 64/W clusters per single-wave block.
template <typename T, bool CPLX, int DE, int MODE, int W>
__device__ __forceinline__ void cluster_lds_body(const ClusterArgs<T>& A, int block) {
  constexpr int LD = DE + 1;
  constexpr int G = 64 / W;
  constexpr int SZ = DE * LD;
  constexpr bool VEC = (MODE != MODE_CERTIFY);
  __shared__ T sar_[G * SZ];
  __shared__ T sai_[CPLX ? G * SZ : 1];
  __shared__ T sur_[VEC ? G * SZ : 1];
  __shared__ T sui_[(VEC && CPLX) ? G * SZ : 1];
  // (float ground values keep the order of rotations of the solver in LDS; a complex or 16-dimensional cluster
  // with a whole wave is solved there too, on all its lanes: 16 x 16 clusters in double, us, registers /
  // LDS: 2000 complex 440 / 297, 123 000 real 8000 / 5800)
  constexpr bool REG = (sizeof(T) == 8 || MODE == MODE_GIBBS) && !(W == 64 && (CPLX || DE == 16));
  __shared__ ScratchFor<T, DE, REG> J_[G];
  __shared__ T sp_[G * DE];
  const int g = threadIdx.x / W, lt = threadIdx.x % W;
  const int64_t c = (int64_t)block * G + g;
  const bool active = c < A.n;
  T* sar = sar_ + g * SZ;
  T* sai = CPLX ? sai_ + g * SZ : sai_;
  T* sur = VEC ? sur_ + g * SZ : sur_;
  T* sui = (VEC && CPLX) ? sui_ + g * SZ : sui_;
  T* sp = sp_ + g * DE;
  const T th = A.tab ? (T)A.tab->theta_cur : (T)A.theta;
  const T beta = A.tab ? (T)A.tab->beta : (T)A.beta;
  // ---- a1/a2: assemble theta_e at eta ----
  T n2 = T(0);
  if (active) n2 = lds_assemble<T, CPLX, DE, W>(A, c, lt, A.nu_c, A.ze_c, A.nu_p, A.ze_p, th, true, T(1), sar, sai);
  const T nrm2 = seg_sum<W>(n2);
  init_vectors<T, CPLX, DE, VEC, W, REG>(sur, sui, lt, active);
  __syncthreads();
  // ---- a3: parallel cyclic Jacobi ----
  const bool conv = cluster_jacobi<T, CPLX, DE, VEC, W, REG>(sar, sai, sur, sui, J_[g], A.tol, nrm2,
                                                        A.max_sweeps, lt, active);
  if (active && !conv && lt == 0 && A.noconv) atomicAdd(A.noconv, 1ull);
  T lmin = T(INFINITY);
  if (active)
    for (int k = lt; k < DE; k += W) lmin = fmin(lmin, sar[k * LD + k]);
  lmin = seg_min<W>(lmin);
  if (active && lt == 0 && !isfinite((double)lmin) && A.nonfinite) atomicAdd(A.nonfinite, 1ull);
  const int32_t gid = active ? A.gid[c] : 0;
  if constexpr (MODE == MODE_CERTIFY) {
    // remaining off-diagonal mass (Weyl, as in the register kernel)
    double off2 = 0.0;
    if (active)
      for (int idx = lt; idx < DE * DE; idx += W) {
        const int i = idx / DE, j = idx % DE;
        if (i == j) continue;
        const double xr = (double)sar[i * LD + j];
        off2 = fma(xr, xr, off2);
        if constexpr (CPLX) {
          const double xi = (double)sai[i * LD + j];
          off2 = fma(xi, xi, off2);
        }
      }
    off2 = seg_sum<W>(off2);
    if (active && lt == 0) {
      A.scal[gid] = (double)lmin;
      A.scal2[gid] = 8.0 * DE * DBL_EPSILON * sqrt((double)nrm2) + sqrt(off2);
    }
  } else {
    // ---- a4: weights and the marginal U diag(p) U^H (over A) ----
    const T val = lds_weights<T, DE, MODE, W>(sar, sp, lmin, beta, (T)A.tau_rel * fmax(T(1), dsqrt<T>(nrm2)), lt,
                                              active);
    if (active && lt == 0 && A.scal) A.scal[gid] = (double)val;
    if (active) lds_rebuild<T, CPLX, DE, W>(sur, sui, sp, sar, sai, lt);
    __syncthreads();
    // ---- a5: outputs ----
    if (active) lds_outputs<T, CPLX, DE, W>(A, c, lt, gid, sar, sai);
  }
}
template <typename T, bool CPLX, int DE, int MODE, int W>
__global__ __launch_bounds__(64) void k_cluster_lds(ClusterArgs<T> A) {
  cluster_lds_body<T, CPLX, DE, MODE, W>(A, blockIdx.x);
}

// 8 x 8 clusters (W lanes each), bonds and sites in one launch, in n8, nbe and nbs blocks of one wave.
// All three are chains of rotations that leave the chip idle, and the first needs the most registers.
template <typename T, bool CPLX, int MODE, int W>
__global__ __launch_bounds__(64) void k_cluster_lds8_pair(ClusterArgs<T> A, ClusterArgs<T> E, ClusterArgs<T> S, int n8,
                                                          int nbe) {
  const int b = blockIdx.x;
  if (b < n8) {
    cluster_lds_body<T, CPLX, 8, MODE, W>(A, b);
  } else if (b < n8 + nbe) {
    const int64_t c = (int64_t)(b - n8) * 64 + threadIdx.x;
    if (c < E.n) cluster_reg_body<T, CPLX, 4, 2, MODE>(E, c);
  } else {
    const int64_t c = (int64_t)(b - n8 - nbe) * 64 + threadIdx.x;
    if (c < S.n) cluster_reg_body<T, CPLX, 2, 0, MODE>(S, c);
  }
}

// ------------------------------------------------------------------------------------------
// clusters holding a spin-1 site (De = 3, 9, 27, 6, ... <= 64): the LDS Jacobi kernel driven by
// index tables instead of site bit masks, the De x De problem embedded in DEP x DEP (DEP the next
// power of two) with decoupled padding
// ------------------------------------------------------------------------------------------
//
// The padding indices De..DEP-1 carry a diagonal above every eigenvalue of theta_e and zero
// off-diagonal entries.  A Jacobi rotation of a pair with a zero off-diagonal is the identity
// (c = 1, s = 0) and a rotation of two other indices keeps zeros zero, so the padding indices stay
// eigenvectors e_k with their own diagonal: they are left out of lambda_min, the weights, the norms
// and the outputs by index.

template <typename T, bool CPLX, int DEP, int W>
__device__ T gen_assemble(const ClusterArgs<T>& A, int64_t c, int lt, T th, T* dr, T* di) {
  constexpr int LD = DEP + 1;
  const int De = A.De, Dc = A.Dc;
  const int64_t ho = A.hoff[c];
  T my_n2 = T(0);
  for (int idx = lt; idx < DEP * DEP; idx += W) {
    const int i = idx / DEP, j = idx % DEP;
    T vr = T(0), vi = T(0);
    if (i < De && j < De) {
      if (ho >= 0) herm_elem<T>([&](int k) { return (T)A.h[ho + k]; }, i, j, De, CPLX, vr, vi);
      for (int s = 0; s < A.maxch; ++s) {
        const int m = A.ch[(int64_t)s * A.n + c];
        if (m < 0) continue;
        const int32_t* g = A.gtab + ((int64_t)s * A.n + c) * De;
        const int ei = g[i], ej = g[j];
        if (((ei >> 8) & 0xff) != ((ej >> 8) & 0xff)) continue;   // different remaining index
        const int a = ei & 0xff, b = ej & 0xff;
        T er, eim;
        if (A.ze_c)
          herm_elem<T>([&](int k) { const int64_t o = (int64_t)k * A.Mc + m;
                                    return extrap<T>(A.nu_c[o], A.ze_c[o], th); }, a, b, Dc, CPLX, er, eim);
        else
          herm_elem<T>([&](int k) { return A.nu_c[(int64_t)k * A.Mc + m]; }, a, b, Dc, CPLX, er, eim);
        vr -= er;
        vi -= eim;
      }
      for (int s = 0; s < A.maxpar; ++s) {
        const int m = A.par[(int64_t)s * A.n + c];
        if (m < 0) continue;
        T er, eim;
        if (A.ze_p)
          herm_elem<T>([&](int k) { const int64_t o = (int64_t)k * A.Mp + m;
                                    return extrap<T>(A.nu_p[o], A.ze_p[o], th); }, i, j, De, CPLX, er, eim);
        else
          herm_elem<T>([&](int k) { return A.nu_p[(int64_t)k * A.Mp + m]; }, i, j, De, CPLX, er, eim);
        vr += er;
        vi += eim;
      }
      my_n2 = dfma<T>(vr, vr, my_n2);
      if constexpr (CPLX) my_n2 = dfma<T>(vi, vi, my_n2);
    }
    dr[i * LD + j] = vr;
    if constexpr (CPLX) di[i * LD + j] = vi;
  }
  return my_n2;
}

template <typename T, bool CPLX, int DEP, int W>
__device__ void gen_outputs(const ClusterArgs<T>& A, int64_t c, int lt, int32_t gid, const T* yr, const T* yi) {
  constexpr int LD = DEP + 1;
  const int De = A.De, Dc = A.Dc;
  const int64_t rs_self = A.rslot ? A.rslot[c] : -1;
  const int NCE = CPLX ? De * De : De * (De + 1) / 2;
  for (int k = lt; k < NCE; k += W) {
    int i, j;
    bool im;
    decode_comp(k, De, i, j, im);
    const T v = im ? yi[i * LD + j] : yr[i * LD + j];
    if (rs_self >= 0 && A.R) A.R[(int64_t)k * A.S + rs_self] = v;
    if (A.marg) A.marg[A.marg_off[gid] + k] = v;
  }
  if (A.Tout && Dc > 0) {
    const int NR = De / Dc;
    const int NCC = CPLX ? Dc * Dc : Dc * (Dc + 1) / 2;
    for (int s = 0; s < A.maxch; ++s) {
      const int m = A.ch[(int64_t)s * A.n + c];
      if (m < 0) continue;
      const int32_t* g = A.gtab + ((int64_t)s * A.n + c) * De;
      for (int k = lt; k < NCC; k += W) {
        int a, b;
        bool im;
        decode_comp(k, Dc, a, b, im);
        T sum = T(0);
        for (int x = 0; x < NR; ++x) {
          const int i = g[a * NR + x] >> 16, j = g[b * NR + x] >> 16;
          sum += im ? yi[i * LD + j] : yr[i * LD + j];
        }
        A.Tout[(int64_t)k * A.Mc + m] = sum;
      }
    }
  }
}

template <typename T, bool CPLX, int DEP, int MODE, int W>
__global__ __launch_bounds__(64) void k_cluster_gen(ClusterArgs<T> A) {
  constexpr int LD = DEP + 1;
  constexpr int G = 64 / W;
  constexpr int SZ = DEP * LD;
  constexpr bool VEC = (MODE != MODE_CERTIFY);
  __shared__ T sar_[G * SZ];
  __shared__ T sai_[CPLX ? G * SZ : 1];
  __shared__ T sur_[VEC ? G * SZ : 1];
  __shared__ T sui_[(VEC && CPLX) ? G * SZ : 1];
  constexpr bool REG = sizeof(T) == 8;
  __shared__ ScratchFor<T, DEP, REG> J_[G];
  __shared__ T sp_[G * DEP];
  const int g = threadIdx.x / W, lt = threadIdx.x % W;
  const int64_t c = (int64_t)blockIdx.x * G + g;
  const bool active = c < A.n;
  const int De = A.De;
  T* sar = sar_ + g * SZ;
  T* sai = CPLX ? sai_ + g * SZ : sai_;
  T* sur = VEC ? sur_ + g * SZ : sur_;
  T* sui = (VEC && CPLX) ? sui_ + g * SZ : sui_;
  T* sp = sp_ + g * DEP;
  const T th = A.tab ? (T)A.tab->theta_cur : (T)A.theta;
  const T beta = A.tab ? (T)A.tab->beta : (T)A.beta;
  // ---- a1/a2: assemble theta_e at eta, then the padding diagonal ----
  T n2 = T(0);
  if (active) n2 = gen_assemble<T, CPLX, DEP, W>(A, c, lt, th, sar, sai);
  const T nrm2 = seg_sum<W>(n2);
  __syncthreads();
  if (active)
    for (int k = De + lt; k < DEP; k += W) sar[k * LD + k] = T(2) * dsqrt<T>(nrm2) + T(1);   // > every eigenvalue
  init_vectors<T, CPLX, DEP, VEC, W, REG>(sur, sui, lt, active);
  __syncthreads();
  // ---- a3: parallel cyclic Jacobi over DEP (the padding stays decoupled) ----
  const bool conv = cluster_jacobi<T, CPLX, DEP, VEC, W, REG>(sar, sai, sur, sui, J_[g], A.tol, nrm2,
                                                         A.max_sweeps, lt, active);
  if (active && !conv && lt == 0 && A.noconv) atomicAdd(A.noconv, 1ull);
  T lmin = T(INFINITY);
  if (active)
    for (int k = lt; k < De; k += W) lmin = fmin(lmin, sar[k * LD + k]);
  lmin = seg_min<W>(lmin);
  if (active && lt == 0 && !isfinite((double)lmin) && A.nonfinite) atomicAdd(A.nonfinite, 1ull);
  const int32_t gid = active ? A.gid[c] : 0;
  if constexpr (MODE == MODE_CERTIFY) {
    double off2 = 0.0;   // off-diagonal mass left by the sweeps (Weyl)
    if (active)
      for (int idx = lt; idx < DEP * DEP; idx += W) {
        const int i = idx / DEP, j = idx % DEP;
        if (i == j) continue;
        const double xr = (double)sar[i * LD + j];
        off2 = fma(xr, xr, off2);
        if constexpr (CPLX) {
          const double xi = (double)sai[i * LD + j];
          off2 = fma(xi, xi, off2);
        }
      }
    off2 = seg_sum<W>(off2);
    if (active && lt == 0) {
      A.scal[gid] = (double)lmin;
      A.scal2[gid] = 8.0 * De * DBL_EPSILON * sqrt((double)nrm2) + sqrt(off2);
    }
  } else {
    // ---- a4: weights (padding indices excluded) and the marginal U diag(p) U^H ----
    T w = T(0);
    if (active) {
      const T tau = (T)A.tau_rel * fmax(T(1), dsqrt<T>(nrm2));
      for (int k = lt; k < DEP; k += W) {
        T v = T(0);
        if (k < De) {
          if constexpr (MODE == MODE_GIBBS) v = dexp<T>(-beta * (sar[k * LD + k] - lmin));
          else v = (sar[k * LD + k] <= lmin + tau) ? T(1) : T(0);
        }
        sp[k] = v;
        w += v;
      }
    }
    const T Z = seg_sum<W>(w);
    __syncthreads();
    if (active)
      for (int k = lt; k < DEP; k += W) sp[k] = ddiv<T>(sp[k], Z);
    __syncthreads();
    const T val = (MODE == MODE_GIBBS) ? lmin - ddiv<T>(dlog<T>(Z), beta) : lmin;
    if (active && lt == 0 && A.scal) A.scal[gid] = (double)val;
    if (active) lds_rebuild<T, CPLX, DEP, W>(sur, sui, sp, sar, sai, lt);
    __syncthreads();
    // ---- a5: outputs ----
    if (active) gen_outputs<T, CPLX, DEP, W>(A, c, lt, gid, sar, sai);
  }
}

// ------------------------------------------------------------------------------------------
// large clusters (De = 128, 256): one 1024-thread workgroup per cluster
// ------------------------------------------------------------------------------------------
//
// A De x De complex matrix and its eigenvectors do not fit one CU's LDS, so theta_e, U and
// rho live in a per-workgroup scratch slab in HBM (the workgroup walks clusters with a grid
// stride); the round-robin parallel Jacobi applies De/2 disjoint rotations per round with all
// 1024 threads.  The reconstruction rho = W W^H with W = U diag(sqrt p) is a dense contraction
// and runs on the matrix cores: v_mfma_f32_32x32x2_f32 (FP32) / v_mfma_f64_16x16x4_f64 (FP64),
// four real products per complex tile.

typedef float mfma_f32x16 __attribute__((ext_vector_type(16)));
typedef double mfma_f64x4 __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ T block_sum(T v, T* red) {
  v = wave_sum(v);
  const int w = threadIdx.x / 64, l = threadIdx.x % 64;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  T s = T(0);
  const int nw = blockDim.x / 64;
  for (int i = 0; i < nw; ++i) s += red[i];
  __syncthreads();
  return s;
}
template <typename T>
__device__ __forceinline__ T block_max(T v, T* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  const int w = threadIdx.x / 64, l = threadIdx.x % 64;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  T s = red[0];
  const int nw = blockDim.x / 64;
  for (int i = 1; i < nw; ++i) s = fmax(s, red[i]);
  __syncthreads();
  return s;
}
template <typename T>
__device__ __forceinline__ T block_min(T v, T* red) {
  v = wave_min(v);
  const int w = threadIdx.x / 64, l = threadIdx.x % 64;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  T s = red[0];
  const int nw = blockDim.x / 64;
  for (int i = 1; i < nw; ++i) s = fmin(s, red[i]);
  __syncthreads();
  return s;
}

// rho tile accumulation on the matrix cores; (wr, wi) = W rows, rho written to (orr, ori)
template <typename T, bool CPLX>
__device__ void mfma_rebuild(const T* ur, const T* ui, const T* sq, T* orr, T* ori, int D) {
  const int wave = threadIdx.x / 64, l = threadIdx.x % 64, nw = blockDim.x / 64;
  if constexpr (std::is_same<T, float>::value) {
    const int nt = D / 32;
    for (int tile = wave; tile < nt * nt; tile += nw) {
      const int I = tile / nt, J = tile % nt;
      mfma_f32x16 cr = {0}, ci = {0};
      const int i = I * 32 + (l % 32), j = J * 32 + (l % 32);
      for (int k0 = 0; k0 < D; k0 += 2) {
        const int k = k0 + l / 32;
        const float s = sq[k];
        const float ar = ur[(int64_t)i * D + k] * s, br = ur[(int64_t)j * D + k] * s;
        cr = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, br, cr, 0, 0, 0);
        if constexpr (CPLX) {
          const float ai = ui[(int64_t)i * D + k] * s, bi = ui[(int64_t)j * D + k] * s;
          cr = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, bi, cr, 0, 0, 0);
          ci = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, br, ci, 0, 0, 0);
          ci = __builtin_amdgcn_mfma_f32_32x32x2f32(-ar, bi, ci, 0, 0, 0);
        }
      }
      for (int r = 0; r < 16; ++r) {
        const int row = I * 32 + 8 * (r / 4) + 4 * (l / 32) + (r % 4), col = J * 32 + (l % 32);
        orr[(int64_t)row * D + col] = cr[r];
        if constexpr (CPLX) ori[(int64_t)row * D + col] = (row == col) ? 0.f : ci[r];
      }
    }
  } else {
    const int nt = D / 16;
    for (int tile = wave; tile < nt * nt; tile += nw) {
      const int I = tile / nt, J = tile % nt;
      mfma_f64x4 cr = {0}, ci = {0};
      const int i = I * 16 + (l % 16), j = J * 16 + (l % 16);
      for (int k0 = 0; k0 < D; k0 += 4) {
        const int k = k0 + l / 16;
        const double s = sq[k];
        const double ar = ur[(int64_t)i * D + k] * s, br = ur[(int64_t)j * D + k] * s;
        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, cr, 0, 0, 0);
        if constexpr (CPLX) {
          const double ai = ui[(int64_t)i * D + k] * s, bi = ui[(int64_t)j * D + k] * s;
          cr = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, bi, cr, 0, 0, 0);
          ci = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, ci, 0, 0, 0);
          ci = __builtin_amdgcn_mfma_f64_16x16x4f64(-ar, bi, ci, 0, 0, 0);
        }
      }
      for (int r = 0; r < 4; ++r) {
        const int row = I * 16 + 4 * r + (l / 16), col = J * 16 + (l % 16);
        orr[(int64_t)row * D + col] = cr[r];
        if constexpr (CPLX) ori[(int64_t)row * D + col] = (row == col) ? 0.0 : ci[r];
      }
    }
  }
}

// theta_e of cluster c assembled element by element into a row-major D x D slab (ar, ai) of
// element type S; with VEC the slab (ur, ui) is set to the identity.  Returns this thread's
// share of ||theta||_F^2.
// Element (i, j) of theta_e for cluster c: h_e, minus the lifted child messages, plus the parent
// messages (extrapolated with weight th when the zeta pointers are set).
template <typename T, bool CPLX>
__device__ __forceinline__ void theta_elem(const ClusterArgs<T>& A, int64_t c, int D, int NB, int64_t ho, int i, int j,
                                           T th, T& vr, T& vi) {
  const int Dc = A.Dc;
  vr = T(0);
  vi = T(0);
  if (ho >= 0) herm_elem<T>([&](int k) { return (T)A.h[ho + k]; }, i, j, D, CPLX, vr, vi);
  for (int s = 0; s < A.maxch; ++s) {
    const int m = A.ch[(int64_t)s * A.n + c];
    if (m < 0) continue;
    const int mask = A.chmask[(int64_t)s * A.n + c];
    if (((i ^ j) & ~mask & (D - 1)) != 0) continue;
    const int a = pext_rt(i, mask, NB), b = pext_rt(j, mask, NB);
    T er, ei;
    if (A.ze_c)
      herm_elem<T>([&](int k) { const int64_t o = (int64_t)k * A.Mc + m;
                                return extrap<T>(A.nu_c[o], A.ze_c[o], th); }, a, b, Dc, CPLX, er, ei);
    else
      herm_elem<T>([&](int k) { return A.nu_c[(int64_t)k * A.Mc + m]; }, a, b, Dc, CPLX, er, ei);
    vr -= er;
    vi -= ei;
  }
  for (int s = 0; s < A.maxpar; ++s) {
    const int m = A.par[(int64_t)s * A.n + c];
    if (m < 0) continue;
    T er, ei;
    if (A.ze_p)
      herm_elem<T>([&](int k) { const int64_t o = (int64_t)k * A.Mp + m;
                                return extrap<T>(A.nu_p[o], A.ze_p[o], th); }, i, j, D, CPLX, er, ei);
    else
      herm_elem<T>([&](int k) { return A.nu_p[(int64_t)k * A.Mp + m]; }, i, j, D, CPLX, er, ei);
    vr += er;
    vi += ei;
  }
}

template <typename T, typename S, bool CPLX, bool VEC>
__device__ T big_assemble(const ClusterArgs<T>& A, int64_t c, int D, S* ar, S* ai, S* ur, S* ui, T th, int tid,
                          int nth) {
  const int NB = log2i(D);
  const int64_t DD = (int64_t)D * D;
  const int64_t ho = A.hoff[c];
  T my_n2 = T(0);
  for (int64_t idx = tid; idx < DD; idx += nth) {
    const int i = (int)(idx / D), j = (int)(idx % D);
    T vr, vi;
    theta_elem<T, CPLX>(A, c, D, NB, ho, i, j, th, vr, vi);
    ar[idx] = (S)vr;
    if constexpr (CPLX) ai[idx] = (S)vi;
    if constexpr (VEC) {
      ur[idx] = (i == j) ? S(1) : S(0);
      if constexpr (CPLX) ui[idx] = S(0);
    }
    my_n2 = dfma<T>(vr, vr, my_n2);
    if constexpr (CPLX) my_n2 = dfma<T>(vi, vi, my_n2);
  }
  return my_n2;
}

// Outputs of a cluster whose marginal scale * (rr, ri) sits in a row-major slab: own marginal
// slot, per-cluster marginal, partial traces onto every child.
template <typename T, typename S, bool CPLX>
__device__ void big_outputs(const ClusterArgs<T>& A, int64_t c, int D, int32_t gid, const S* rr_, const S* ri_,
                            S scale, int tid, int nth) {
  const int NB = log2i(D);
  const int Dc = A.Dc;
  const int64_t rs_self = A.rslot ? A.rslot[c] : -1;
  const int NCE = CPLX ? D * D : D * (D + 1) / 2;
  for (int k = tid; k < NCE; k += nth) {
    int i, j;
    bool im;
    decode_comp(k, D, i, j, im);
    const T v = (T)(scale * (im ? ri_[(int64_t)i * D + j] : rr_[(int64_t)i * D + j]));
    if (rs_self >= 0 && A.R) A.R[(int64_t)k * A.S + rs_self] = v;
    if (A.marg) A.marg[A.marg_off[gid] + k] = v;
  }
  if (A.Tout && Dc > 0) {
    const int NR = D / Dc;
    const int NCC = CPLX ? Dc * Dc : Dc * (Dc + 1) / 2;
    for (int s = 0; s < A.maxch; ++s) {
      const int m = A.ch[(int64_t)s * A.n + c];
      if (m < 0) continue;
      const int mask = A.chmask[(int64_t)s * A.n + c];
      for (int k = tid; k < NCC; k += nth) {
        int a, b;
        bool im;
        decode_comp(k, Dc, a, b, im);
        S sum = S(0);
        for (int x = 0; x < NR; ++x) {
          const int i = pdep_rt(a, x, mask, NB), j = pdep_rt(b, x, mask, NB);
          sum += im ? ri_[(int64_t)i * D + j] : rr_[(int64_t)i * D + j];
        }
        A.Tout[(int64_t)k * A.Mc + m] = (T)(scale * sum);
      }
    }
  }
}

template <typename T, bool CPLX, int MODE>
__global__ __launch_bounds__(1024) void k_cluster_big(ClusterArgs<T> A, T* scratch, int64_t slab) {
  constexpr bool VEC = (MODE != MODE_CERTIFY);
  __shared__ T cs_c[128], cs_s[128], cs_er[128], cs_ei[128], cs_app[128], cs_aqq[128];
  __shared__ int cs_p[128], cs_q[128];
  __shared__ T red[16];
  __shared__ double redd[16];
  __shared__ T sp[256];
  const int D = A.De;
  const int NB = log2i(D);
  const int NP = D / 2;
  const int64_t DD = (int64_t)D * D;
  T* ar = scratch + (int64_t)blockIdx.x * slab;
  T* ai = ar + DD;   // unused for real problems
  T* ur = ar + (CPLX ? 2 : 1) * DD;
  T* ui = ur + DD;
  T* rr_ = ar + (CPLX ? 4 : 2) * DD;
  T* ri_ = rr_ + DD;
  const int tid = threadIdx.x, nth = blockDim.x;
  const T th = A.tab ? (T)A.tab->theta_cur : (T)A.theta;
  const T beta = A.tab ? (T)A.tab->beta : (T)A.beta;
  for (int64_t c = blockIdx.x; c < A.n; c += gridDim.x) {
    // ---- a2: assemble theta_e ----
    const int Dc = A.Dc;
    const T my_n2 = big_assemble<T, T, CPLX, VEC>(A, c, D, ar, ai, ur, ui, th, tid, nth);
    const T nrm2 = block_sum(my_n2, red);
    // ---- a3: parallel cyclic Jacobi over the slab ----
    const double tol2 = A.tol * A.tol * (double)nrm2;
    bool conv = false;
    for (int sweep = 0; sweep <= A.max_sweeps; ++sweep) {
      double off = 0.0;   // the convergence test in FP64 whatever T
      for (int64_t idx = tid; idx < DD; idx += nth) {
        if (idx / D != idx % D) {
          const double x = (double)ar[idx];
          off = fma(x, x, off);
          if constexpr (CPLX) {
            const double y = (double)ai[idx];
            off = fma(y, y, off);
          }
        }
      }
      off = block_sum(off, redd);
      if (off <= tol2) { conv = true; break; }
      if (sweep == A.max_sweeps) break;
      for (int r = 0; r < D - 1; ++r) {
        if (tid < NP) {
          int p, q;
          rr_pair(r, tid, D, p, q);
          const T xr = ar[(int64_t)p * D + q];
          const T xi = CPLX ? ai[(int64_t)p * D + q] : T(0);
          const T rr = CPLX ? dsqrt<T>(dfma<T>(xr, xr, xi * xi)) : fabs(xr);
          T t = T(0), cc = T(1), ss = T(0), er = T(1), ei = T(0);
          const T app = ar[(int64_t)p * D + p], aqq = ar[(int64_t)q * D + q];
          if (rr != T(0)) {
            rot_params<T>(app, aqq, rr, t, cc, ss);
            er = CPLX ? ddiv<T>(xr, rr) : copysign(T(1), xr);
            ei = CPLX ? ddiv<T>(-xi, rr) : T(0);
          }
          cs_p[tid] = p; cs_q[tid] = q;
          cs_c[tid] = cc; cs_s[tid] = ss; cs_er[tid] = er; cs_ei[tid] = ei;
          cs_app[tid] = app - t * rr;
          cs_aqq[tid] = aqq + t * rr;
        }
        __syncthreads();
        for (int idx = tid; idx < D * NP; idx += nth) {
          const int i = idx % D, k = idx / D;
          const int p = cs_p[k], q = cs_q[k];
          const T cc = cs_c[k], ss = cs_s[k], er = cs_er[k], ei = cs_ei[k];
          {
            const int64_t op = (int64_t)i * D + p, oq = (int64_t)i * D + q;
            T pr = ar[op], qr = ar[oq];
            T pi = CPLX ? ai[op] : T(0), qi = CPLX ? ai[oq] : T(0);
            T wr = CPLX ? qr * er - qi * ei : qr * er;
            T wi = CPLX ? qr * ei + qi * er : T(0);
            ar[op] = cc * pr - ss * wr;
            ar[oq] = ss * pr + cc * wr;
            if constexpr (CPLX) { ai[op] = cc * pi - ss * wi; ai[oq] = ss * pi + cc * wi; }
          }
          if constexpr (VEC) {
            const int64_t op = (int64_t)i * D + p, oq = (int64_t)i * D + q;
            T pr = ur[op], qr = ur[oq];
            T pi = CPLX ? ui[op] : T(0), qi = CPLX ? ui[oq] : T(0);
            T wr = CPLX ? qr * er - qi * ei : qr * er;
            T wi = CPLX ? qr * ei + qi * er : T(0);
            ur[op] = cc * pr - ss * wr;
            ur[oq] = ss * pr + cc * wr;
            if constexpr (CPLX) { ui[op] = cc * pi - ss * wi; ui[oq] = ss * pi + cc * wi; }
          }
        }
        __syncthreads();
        for (int idx = tid; idx < D * NP; idx += nth) {
          const int j = idx % D, k = idx / D;
          const int p = cs_p[k], q = cs_q[k];
          const T cc = cs_c[k], ss = cs_s[k], er = cs_er[k], ei = -cs_ei[k];
          const int64_t op = (int64_t)p * D + j, oq = (int64_t)q * D + j;
          T pr = ar[op], qr = ar[oq];
          T pi = CPLX ? ai[op] : T(0), qi = CPLX ? ai[oq] : T(0);
          T wr = CPLX ? qr * er - qi * ei : qr * er;
          T wi = CPLX ? qr * ei + qi * er : T(0);
          ar[op] = cc * pr - ss * wr;
          ar[oq] = ss * pr + cc * wr;
          if constexpr (CPLX) { ai[op] = cc * pi - ss * wi; ai[oq] = ss * pi + cc * wi; }
        }
        __syncthreads();
        if (tid < NP) {
          const int p = cs_p[tid], q = cs_q[tid];
          ar[(int64_t)p * D + p] = cs_app[tid];
          ar[(int64_t)q * D + q] = cs_aqq[tid];
          ar[(int64_t)p * D + q] = T(0);
          ar[(int64_t)q * D + p] = T(0);
          if constexpr (CPLX) {
            ai[(int64_t)p * D + p] = T(0); ai[(int64_t)q * D + q] = T(0);
            ai[(int64_t)p * D + q] = T(0); ai[(int64_t)q * D + p] = T(0);
          }
        }
        __syncthreads();
      }
    }
    if (!conv && tid == 0 && A.noconv) atomicAdd(A.noconv, 1ull);
    T lmin = T(INFINITY);
    for (int k = tid; k < D; k += nth) lmin = fmin(lmin, ar[(int64_t)k * D + k]);
    lmin = block_min(lmin, red);
    if (tid == 0 && !isfinite((double)lmin) && A.nonfinite) atomicAdd(A.nonfinite, 1ull);
    const int32_t gid = A.gid[c];
    if constexpr (MODE == MODE_CERTIFY) {
      if (tid == 0) {
        A.scal[gid] = (double)lmin;
        A.scal2[gid] = 8.0 * D * DBL_EPSILON * sqrt((double)nrm2);
      }
    } else {
      // ---- a4: weights (sqrt stored for the W W^H product) ----
      T w = T(0);
      for (int k = tid; k < D; k += nth) {
        const T lk = ar[(int64_t)k * D + k];
        T v;
        if constexpr (MODE == MODE_GIBBS) v = dexp<T>(-beta * (lk - lmin));
        else v = (lk <= lmin + (T)A.tau_rel * fmax(T(1), dsqrt<T>(nrm2))) ? T(1) : T(0);
        sp[k] = v;
        w += v;
      }
      const T Z = block_sum(w, red);
      for (int k = tid; k < D; k += nth) sp[k] = dsqrt<T>(sp[k] / Z);
      if (tid == 0 && A.scal) A.scal[gid] = (MODE == MODE_GIBBS) ? (double)(lmin - dlog<T>(Z) / beta) : (double)lmin;
      __syncthreads();
      mfma_rebuild<T, CPLX>(ur, ui, sp, rr_, ri_, D);
      __syncthreads();
      // ---- a5: outputs ----
      big_outputs<T, T, CPLX>(A, c, D, gid, rr_, ri_, T(1), tid, nth);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------
// Gibbs state by scaling and squaring on the matrix cores (accelerated iteration, De = 16, 32)
// ------------------------------------------------------------------------------------------
//
// The smoothed dual needs rho_e = exp(-beta theta_e) / Z and F_beta = -(1/beta) log Z only
// (Sec. 4.1.2); the eigenvectors are not needed for that.  With mu = Tr(theta)/D and
// X = beta (theta - mu), the scaling s is the least s >= 0 with r <= kMax 2^s, where r = sqrt(||X^2||_1)
// bounds the spectral radius of X (X^2 is a matrix the polynomial needs anyway, and its 1-norm is
// nearer to the radius than that of X), and
//     E0 = p(-X / 2^s)                  (ExpPoly: degree 12, four products)
//     Y0 = E0 / tau_0,  Y_j = Y_{j-1}^2 / tau_j    (j = 1..s)
//     rho = Y_s / Tr Y_s,  log Z = 2^s log tau_0 + sum_j 2^(s-j) log tau_j + log Tr Y_s
// for any positive rescalings tau_j (the one-wave kernel uses exact powers of two; the
// workgroup kernel tau_0 = Tr E0, tau_j = (Tr Y_{j-1})^2).
// A relative error e of p acts like e 2^s on X, at most 2 e r / kMax: 4e-15 r with double messages,
// under the float rounding of the messages with float ones.  Rounding in the squarings adds a
// relative error of order D u (spectral spread / gap) to rho: the part along the dominant eigenvector is
// removed by the final trace normalisation, the rest is damped once the spectrum separates.  With double
// messages everything runs in FP64.  With float messages the polynomial and the first squarings do
// (two in the one-wave kernel; in the workgroup kernel all but the last n32 <= log2(||X|| / 4)), the
// rest in FP32.
//
// One wavefront per cluster.  A matrix is NB x NB blocks of 16 x 16 held in the MFMA result
// layout: lane l, register r of block (I, J) is element (16 I + 4 r + l/16, 16 J + l%16).
// Every matrix here is Hermitian (a polynomial in X), so the A operand of block (I, K) at
// k-step kk, element (16 I + l%16, 16 K + 4 kk + l/16), is the conjugate of register kk of
// block (K, I): both operands come straight from the registers, with no data movement.
constexpr int kExpmLut = 8;   // children handled through the LDS index tables (more: generic path)
constexpr int kF64Squarings = 2;   // float-message path: squarings kept in FP64 before the FP32 ones

// The degree-12 polynomial p of the scaled exponential, p(x) ~ e^x on |x| <= kMax (every matrix here
// is Hermitian, so only its real spectrum counts): the least largest relative error |p e^-x - 1|
// under p(0) = p'(0) = 1, so that the error vanishes with x like x^2.  With y = kappa x it takes
// four products,
//     a6 = (y3 + b2 y2 + b1 y)^2 + r3 y3 + r2 y2 + r1 y,   p = (a6 + s3 y3 + s2 y2 + s1 y + s0) a6
//          + t2 y2 + t1 y + 1,    y2 = y y, y3 = y y2,
// kappa chosen to make the leading coefficient one.  (The form B1 + (B2 + A6) A6, A6 = B3 + B4^2, is that of
// Bader, Blanes and Casas, Computing the matrix exponential with an optimized Taylor polynomial
// approximation, 2019; there for Taylor coefficients.)  Double messages: error 1.4e-15 on
// |x| <= 0.75 with the coefficients rounded to doubles, 1.2e-15 before (a degree-12 Taylor polynomial,
// error 2e-14 on |x| <= 1/2, took five products by powers of X^3); float messages: 3.5e-10 on |x| <= 2
// (degree-8 Taylor: four products, 5.4e-9 on |x| <= 1/2).
template <typename T>
struct ExpPoly;
template <>
struct ExpPoly<double> {
  static constexpr double kMax = 0.75, kappa = 0.18890286463643001186, b2 = 0.57937322089049180036,
                          b1 = 0.68740475750695858833, r3 = -0.0226260036235939413, r2 = 1.9368132151596933149,
                          r1 = 1.0421080289587672922, s3 = 3.4844151622963205626, s2 = 1.7202447934751227396,
                          s1 = 4.8466204810446821081, s0 = 8.0545185343475532364, t2 = -11.530985678296578198,
                          t1 = -3.0999524658049970433;
};
template <>
struct ExpPoly<float> {
  static constexpr double kMax = 2.0, kappa = 0.18794616950573157704, b2 = 0.65021617857486515946,
                          b1 = 0.63003546334208741425, r3 = -0.041946904752406594485, r2 = 1.9627374771981224214,
                          r1 = 1.275754058867548299, s3 = 3.4605728791216365827, s2 = 1.8490087327993450794,
                          s1 = 4.4199263533945864807, s0 = 8.0978796474404292981, t2 = -12.219931968853453924,
                          t1 = -5.0102304112831659341;
};

// The number of squarings for a matrix of spectral radius at most nrm: the least s >= 0 with
// nrm <= kMax 2^s, at most 200 (0 for a NaN norm), from the binary exponent of nrm / kMax.
template <typename T>
__device__ __forceinline__ int expm_squarings(double nrm) {
  const double x = nrm * (1.0 / ExpPoly<T>::kMax);
  if (!(x > 1.0)) return 0;
  if (!(x <= 0x1p199)) return 200;
  int e;
  const double m = frexp(x, &e);   // x = m 2^e, 0.5 <= m < 1
  return m == 0.5 ? e - 1 : e;
}

// pext and pdep over the site bits of a one-wave cluster (at most 5 sites), for every site mask,
// built at compile time: pext[mask][i] packs the bits of i at the mask positions;
// pdepN[mask][(a << lnr) | x] places the bits of a at the mask positions and those of x at the
// other N - popcount(mask) = lnr positions.
struct SiteBitTables {
  unsigned char pext[32][32];
  unsigned char pdep4[16][16];
  unsigned char pdep5[32][32];
};
constexpr SiteBitTables make_site_bit_tables() {
  SiteBitTables t{};
  for (int m = 0; m < 32; ++m)
    for (int i = 0; i < 32; ++i) t.pext[m][i] = (unsigned char)pext_bits(i, m, 5);
  for (int m = 0; m < 16; ++m) {
    const int lnr = 4 - __builtin_popcount(m);
    for (int p = 0; p < 16; ++p) t.pdep4[m][p] = (unsigned char)pdep_bits(p >> lnr, p & ((1 << lnr) - 1), m, 4);
  }
  for (int m = 0; m < 32; ++m) {
    const int lnr = 5 - __builtin_popcount(m);
    for (int p = 0; p < 32; ++p) t.pdep5[m][p] = (unsigned char)pdep_bits(p >> lnr, p & ((1 << lnr) - 1), m, 5);
  }
  return t;
}
static __constant__ SiteBitTables kSiteBits = make_site_bit_tables();

template <int NB, bool CPLX>
struct XMat {
  double re[NB][NB][4];
  double im[CPLX ? NB : 1][CPLX ? NB : 1][4];
};

// C (+)= X Y for Hermitian X; C accumulates onto its contents, column block by column block,
// so C may alias Y (never X).
template <int NB, bool CPLX>
__device__ __forceinline__ void xmm(const XMat<NB, CPLX>& X, const XMat<NB, CPLX>& Y, XMat<NB, CPLX>& C) {
#pragma unroll
  for (int J = 0; J < NB; ++J) {
    mfma_f64x4 cr[NB], ci[NB];
#pragma unroll
    for (int I = 0; I < NB; ++I) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        cr[I][r] = C.re[I][J][r];
        if constexpr (CPLX) ci[I][r] = C.im[I][J][r];
      }
#pragma unroll
      for (int K = 0; K < NB; ++K)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          cr[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(X.re[K][I][kk], Y.re[K][J][kk], cr[I], 0, 0, 0);
          if constexpr (CPLX) {
            cr[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(X.im[K][I][kk], Y.im[K][J][kk], cr[I], 0, 0, 0);
            ci[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(X.re[K][I][kk], Y.im[K][J][kk], ci[I], 0, 0, 0);
            ci[I] = __builtin_amdgcn_mfma_f64_16x16x4f64(-X.im[K][I][kk], Y.re[K][J][kk], ci[I], 0, 0, 0);
          }
        }
    }
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        C.re[I][J][r] = cr[I][r];
        if constexpr (CPLX) C.im[I][J][r] = ci[I][r];
      }
  }
}

// lane-local diagonal test for register r of a diagonal block
__device__ __forceinline__ bool xdiag(int r, int l) { return 4 * r + (l >> 4) == (l & 15); }

// FP32 matrices for the last squarings of the float-message path, in the v_mfma_f32_16x16x4_f32
// result layout: lane l, register r of block (I, J) is element (16 I + 4 (l/16) + r, 16 J + l%16).
// Lane group g = l/16 supplies the k index 4 g + kk at k-step kk, so for Hermitian X the A operand
// of block (I, K) is the conjugate of register kk of block (K, I), as in the FP64 layout.
template <int NB, bool CPLX>
struct XMat32 {
  float re[NB][NB][4];
  float im[CPLX ? NB : 1][CPLX ? NB : 1][4];
};
typedef float mfma_f32x4 __attribute__((ext_vector_type(4)));

template <int NB, bool CPLX>
__device__ __forceinline__ void xmm32(const XMat32<NB, CPLX>& X, const XMat32<NB, CPLX>& Y, XMat32<NB, CPLX>& C) {
#pragma unroll
  for (int J = 0; J < NB; ++J) {
    mfma_f32x4 cr[NB], ci[NB];
#pragma unroll
    for (int I = 0; I < NB; ++I) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        cr[I][r] = C.re[I][J][r];
        if constexpr (CPLX) ci[I][r] = C.im[I][J][r];
      }
#pragma unroll
      for (int K = 0; K < NB; ++K)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          cr[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(X.re[K][I][kk], Y.re[K][J][kk], cr[I], 0, 0, 0);
          if constexpr (CPLX) {
            cr[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(X.im[K][I][kk], Y.im[K][J][kk], cr[I], 0, 0, 0);
            ci[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(X.re[K][I][kk], Y.im[K][J][kk], ci[I], 0, 0, 0);
            ci[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(-X.im[K][I][kk], Y.re[K][J][kk], ci[I], 0, 0, 0);
          }
        }
    }
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        C.re[I][J][r] = cr[I][r];
        if constexpr (CPLX) C.im[I][J][r] = ci[I][r];
      }
  }
}

// Trace of an FP32-layout matrix: the diagonal sits in lanes whose 4-lane group (l % 16) / 4
// equals l / 16 (lanes 0-3, 20-23, 40-43, 60-63), register l % 4; two quad-permute DPP steps
// and four readlanes sum it.  Used only for the binary exponent of the rescaling steps.
template <int CTRL>
__device__ __forceinline__ float dpp_movf(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int NB, bool CPLX>
__device__ __forceinline__ float xtrace32(const XMat32<NB, CPLX>& M, int l) {
  float v = 0.f;
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * (l >> 4) + r == (l & 15)) v += M.re[I][I][r];
  v += dpp_movf<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_movf<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  const auto rl = [&](int lane) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane)); };
  return (rl(0) + rl(20)) + (rl(40) + rl(60));
}

template <int NB, bool CPLX>
__device__ __forceinline__ void xzero(XMat<NB, CPLX>& M) {
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J < NB; ++J)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        M.re[I][J][r] = 0.0;
        if constexpr (CPLX) M.im[I][J][r] = 0.0;
      }
}

// Trace of an FP64-layout matrix: the diagonal sits in lanes with l % 4 == l / 16, register
// (l % 16) / 4 of every diagonal block, four lanes 4 apart in each row of 16.  Two row-shift
// DPP steps leave each row's sum in its lane 12 + l / 16; four readlanes add the rows.
template <int NB, bool CPLX>
__device__ __forceinline__ double xtrace(const XMat<NB, CPLX>& M, int l) {
  double v = 0.0;
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (xdiag(r, l)) v += M.re[I][I][r];
  v += dpp_mov<0x114>(v);   // row_shr:4
  v += dpp_mov<0x118>(v);   // row_shr:8
  return (readlane_d(v, 12) + readlane_d(v, 29)) + (readlane_d(v, 46) + readlane_d(v, 63));
}

// The same sum for a matrix in the FP32 layout (see XMat32), in double.
template <int NB, bool CPLX>
__device__ __forceinline__ double xtrace_f32(const XMat<NB, CPLX>& M, int l) {
  double v = 0.0;
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * (l >> 4) + r == (l & 15)) v += M.re[I][I][r];
  v += dpp_mov<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_mov<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  return (readlane_d(v, 0) + readlane_d(v, 20)) + (readlane_d(v, 40) + readlane_d(v, 60));
}

// FP32 estimate of the trace of an FP64-layout matrix, for the binary exponent of a rescaling
// (the value only picks an exact power of two): the diagonal lanes as in xtrace, the sum in FP32.
template <int NB, bool CPLX>
__device__ __forceinline__ float xtrace_est(const XMat<NB, CPLX>& M, int l) {
  double t = 0.0;
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (xdiag(r, l)) t += M.re[I][I][r];
  float v = (float)t;
  v += dpp_movf<0x114>(v);   // row_shr:4
  v += dpp_movf<0x118>(v);   // row_shr:8
  const auto rl = [&](int lane) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane)); };
  return (rl(12) + rl(29)) + (rl(46) + rl(63));
}

// log x = k log 2 + log m for a positive double x: k (returned in kk, an integer-valued double)
// and log m, m = x 2^-k in [1/sqrt 2, sqrt 2), from log m = 2 atanh(z), z = (m - 1) / (m + 1),
// |z| <= 0.1716, with the odd series of atanh summed to z^19 (the first omitted term is below
// 1e-17).  m - 1 is exact, so log m is accurate to a few units in the last place.  A NaN or
// infinite x gives a NaN.
__device__ __forceinline__ double log_split(double x, double& kk) {
  int k = __builtin_amdgcn_frexp_exp(x);          // x = m 2^k, m in [0.5, 1)
  double m = __builtin_amdgcn_frexp_mant(x);
  if (m < 0.70710678118654752440) {
    m *= 2.0;
    --k;
  }
  kk = (double)k;
  const double z = (m - 1.0) / (m + 1.0), z2 = z * z;
  double p = 1.0 / 19;
  p = fma(p, z2, 1.0 / 17);
  p = fma(p, z2, 1.0 / 15);
  p = fma(p, z2, 1.0 / 13);
  p = fma(p, z2, 1.0 / 11);
  p = fma(p, z2, 1.0 / 9);
  p = fma(p, z2, 1.0 / 7);
  p = fma(p, z2, 1.0 / 5);
  p = fma(p, z2, 1.0 / 3);
  p = fma(p, z2, 1.0);
  return 2.0 * z * p;
}

// Diagonal updates v + a of a diagonal block: for the real 16 x 16 case (registers to spare at
// full occupancy) as fma(a, dg[r], v) with a per-lane 0.0 / 1.0 indicator, one instruction; in
// the other cases as a lane select, which keeps the indicator out of the registers.
template <int NB, bool CPLX>
struct XDiag {
  static constexpr bool kFma = NB == 1 && !CPLX;
  double dg[kFma ? 4 : 1];
  int l;
  __device__ __forceinline__ explicit XDiag(int lane) : l(lane) {
    if constexpr (kFma) {
#pragma unroll
      for (int r = 0; r < 4; ++r) dg[r] = xdiag(r, lane) ? 1.0 : 0.0;
    }
  }
  __device__ __forceinline__ double add(int r, double a, double v) const {
    if constexpr (kFma) return fma(a, dg[r], v);   // exactly v off the diagonal
    else return xdiag(r, l) ? v + a : v;
  }
};

// D = a I + b A + c A2 (+ d A3) (+ D)
template <int NB, bool CPLX, bool WITH3, bool DIAG, bool ADD>
__device__ __forceinline__ void xpoly(XMat<NB, CPLX>& D, double a, double b, double c, double d,
                                      const XMat<NB, CPLX>& A1, const XMat<NB, CPLX>& A2,
                                      const XMat<NB, CPLX>& A3, const XDiag<NB, CPLX>& dg) {
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J < NB; ++J)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double v = ADD ? fma(b, A1.re[I][J][r], D.re[I][J][r]) : b * A1.re[I][J][r];
        v = fma(c, A2.re[I][J][r], v);
        if constexpr (WITH3) v = fma(d, A3.re[I][J][r], v);
        if (DIAG && I == J) v = dg.add(r, a, v);
        D.re[I][J][r] = v;
        if constexpr (CPLX) {
          double w = ADD ? fma(b, A1.im[I][J][r], D.im[I][J][r]) : b * A1.im[I][J][r];
          w = fma(c, A2.im[I][J][r], w);
          if constexpr (WITH3) w = fma(d, A3.im[I][J][r], w);
          D.im[I][J][r] = w;
        }
      }
}

template <typename T, bool CPLX, int DE>
__device__ __forceinline__ void cluster_expm_body(const ClusterArgs<T>& A, int64_t block) {
  constexpr int LD = DE + 1;
  constexpr int NB = DE / 16;
  __shared__ T sar[DE * LD];
  __shared__ T sai[CPLX ? DE * LD : 1];
  const int64_t c = xcd_cluster(block, A.n);
  const int l = threadIdx.x;
  const T th = A.tab ? (T)A.tab->theta_cur : (T)A.theta;
  const double beta = A.tab ? A.tab->beta : A.beta;
  constexpr int NBITS = log2i(DE);
  static_assert(NBITS == 4 || NBITS == 5, "the one-wave kernel covers D = 16 and 32");
  const int Dc = A.Dc;
  const int nch = A.maxch;
  const bool lut = nch <= kExpmLut;   // cluster-uniform
  // per child: pext of every cluster index onto the child's sites, and pdep of (child index a,
  // complement index x) back to the cluster index, as LDS tables
  __shared__ unsigned char pextL[kExpmLut][DE], depL[kExpmLut][DE];
  __shared__ T stc_r[kExpmLut][DE * DE / 4];
  __shared__ T stc_i[CPLX ? kExpmLut : 1][CPLX ? DE * DE / 4 : 1];
  XMat<NB, CPLX> X, P2, P3, M;
  // ---- a1/a2: assemble theta_e at eta ----
  // D_c and D_e / D_c are powers of two: shifts and masks instead of integer division
  const int ldc = Dc > 0 ? __builtin_ctz(Dc) : 0;
  const int lnr = NBITS - ldc;
  if (lut) {
    for (int s = 0; s < nch; ++s) {
      const int mask = A.chmask[(int64_t)s * A.n + c] & (DE - 1);
      if (l < DE) {
        pextL[s][l] = kSiteBits.pext[mask][l];
        if constexpr (NBITS == 4) depL[s][l] = kSiteBits.pdep4[mask][l];
        else depL[s][l] = kSiteBits.pdep5[mask][l];
      }
    }
    __syncthreads();
    // branch-free element assembly: every candidate element is loaded from a valid address and
    // then selected, so the lanes of the wave never diverge
    // (h_e, then the children in slot order, then the parents: the order of the generic path)
    const int64_t ho = A.hoff[c];
    T acr[NB][NB][4], aci[NB][NB][4];
    // h_e from its packed upper triangle (real plane, then the strict upper imaginary plane);
    // the cluster-uniform test sits outside the loop so that a lane's loads issue together.  The
    // packed index of (lo, hi), lo <= hi, is lo (2D + 1 - lo) / 2 + hi - lo, and the strict one
    // lo (2D - 1 - lo) / 2 + hi - lo - 1; both products are even.
    if (ho >= 0) {
      const double* hp = A.h + ho;
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J < NB; ++J)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = 16 * I + 4 * r + (l >> 4), j = 16 * J + (l & 15);
            const unsigned lo = (unsigned)min(i, j), hi = (unsigned)max(i, j);
            acr[I][J][r] = (T)hp[((lo * (2u * DE + 1u - lo)) >> 1) + hi - lo];
            if constexpr (CPLX) {
              const double v = hp[DE * (DE + 1) / 2 + (lo < hi ? ((lo * (2u * DE - 1u - lo)) >> 1) + hi - lo - 1u : 0u)];
              aci[I][J][r] = (T)(i < j ? v : (i > j ? -v : 0.0));
            } else {
              aci[I][J][r] = T(0);
            }
          }
    } else {
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J < NB; ++J)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            acr[I][J][r] = T(0);
            aci[I][J][r] = T(0);
          }
    }
    // the (extrapolated) child messages, dense D_c x D_c in LDS, one pass over all children
    for (int idx = l; idx < nch << (2 * ldc); idx += 64) {
      const int s = idx >> (2 * ldc), ab = idx & ((1 << (2 * ldc)) - 1);
      const int m = A.ch[(int64_t)s * A.n + c];
      if (m < 0) continue;
      const int a = ab >> ldc, b = ab & (Dc - 1);
      T er, ei;
      if (A.ze_c)
        herm_elem_bf<T, CPLX>([&](int k) { const int64_t o = (int64_t)k * A.Mc + m;
                                           return extrap<T>(A.nu_c[o], A.ze_c[o], th); }, a, b, Dc, er, ei);
      else
        herm_elem_bf<T, CPLX>([&](int k) { return A.nu_c[(int64_t)k * A.Mc + m]; }, a, b, Dc, er, ei);
      stc_r[s][ab] = er;
      if constexpr (CPLX) stc_i[s][ab] = ei;
    }
    __syncthreads();
    for (int s = 0; s < nch; ++s) {
      const int m = A.ch[(int64_t)s * A.n + c];
      if (m < 0) continue;   // cluster-uniform
      const int mask = A.chmask[(int64_t)s * A.n + c];
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J < NB; ++J)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = 16 * I + 4 * r + (l >> 4), j = 16 * J + (l & 15);
            const bool ok = ((i ^ j) & ~mask & (DE - 1)) == 0;
            const int ab = (pextL[s][i] << ldc) | pextL[s][j];
            acr[I][J][r] -= ok ? stc_r[s][ab] : T(0);
            if constexpr (CPLX) aci[I][J][r] -= ok ? stc_i[s][ab] : T(0);
          }
    }
    for (int s = 0; s < A.maxpar; ++s) {
      const int m = A.par[(int64_t)s * A.n + c];
      if (m < 0) continue;   // cluster-uniform
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J < NB; ++J)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = 16 * I + 4 * r + (l >> 4), j = 16 * J + (l & 15);
            T er, ei;
            if (A.ze_p)
              herm_elem_bf<T, CPLX>([&](int k) { const int64_t o = (int64_t)k * A.Mp + m;
                                                 return extrap<T>(A.nu_p[o], A.ze_p[o], th); }, i, j, DE, er, ei);
            else
              herm_elem_bf<T, CPLX>([&](int k) { return A.nu_p[(int64_t)k * A.Mp + m]; }, i, j, DE, er, ei);
            acr[I][J][r] += er;
            aci[I][J][r] += ei;
          }
    }
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J < NB; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          X.re[I][J][r] = (double)acr[I][J][r];
          if constexpr (CPLX) X.im[I][J][r] = (double)aci[I][J][r];
        }
  } else {
    lds_assemble<T, CPLX, DE, 64>(A, c, l, A.nu_c, A.ze_c, A.nu_p, A.ze_p, th, true, T(1), sar, sai);
    __syncthreads();
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J < NB; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int o = (16 * I + 4 * r + (l >> 4)) * LD + 16 * J + (l & 15);
          X.re[I][J][r] = (double)sar[o];
          if constexpr (CPLX) X.im[I][J][r] = (double)sai[o];
        }
  }
  // ---- shift, scale ----
  const double mu = xtrace(X, l) / DE;
  const XDiag<NB, CPLX> dg(l);
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int r = 0; r < 4; ++r) X.re[I][I][r] = dg.add(r, -mu, X.re[I][I][r]);
  using EP = ExpPoly<T>;
  const double sc = -EP::kappa * beta;
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J < NB; ++J)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        X.re[I][J][r] *= sc;
        if constexpr (CPLX) X.im[I][J][r] *= sc;
      }
  // The scale: the square root of the induced 1-norm of X^2, an upper bound of the spectral radius
  // of X that is never above X's own 1-norm (||X^2||_1 <= ||X||_1^2) and costs nothing more, as the
  // polynomial needs X^2 anyway; X and X^2 are then scaled by exact powers of two.  The 1-norm is the
  // largest column sum (X^2 is Hermitian).  Column 16 J + l%16 of block column J is spread over the
  // registers of the lanes l%16 + 16 g; two xor-shuffles complete it in every lane, a DPP row
  // maximum then leaves the largest column sum in every lane.  (Moduli of complex entries and the
  // root are the hardware square root's: the norm only chooses s.)
  xzero(P2);
  xmm(X, X, P2);
  double rmax = 0.0;
#pragma unroll
  for (int J = 0; J < NB; ++J) {
    double a = 0.0;
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (CPLX) a += __builtin_amdgcn_sqrt(fma(P2.re[I][J][r], P2.re[I][J][r], P2.im[I][J][r] * P2.im[I][J][r]));
        else a += fabs(P2.re[I][J][r]);
      }
    a += __shfl_xor(a, 16, 64);
    a += __shfl_xor(a, 32, 64);
    rmax = fmax(rmax, a);
  }
  rmax = fmax(rmax, dpp_mov<0xB1>(rmax));    // quad_perm [1, 0, 3, 2]
  rmax = fmax(rmax, dpp_mov<0x4E>(rmax));    // quad_perm [2, 3, 0, 1]
  rmax = fmax(rmax, dpp_mov<0x141>(rmax));   // row_half_mirror
  rmax = fmax(rmax, dpp_mov<0x140>(rmax));   // row_mirror
  // every lane holds the same value; make s scalar
  const int s = __builtin_amdgcn_readfirstlane(expm_squarings<T>(__builtin_amdgcn_sqrt(rmax) * (1.0 / EP::kappa)));
  {
    const double f1 = ldexp(1.0, -s), f2 = ldexp(1.0, -2 * s);
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J < NB; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          X.re[I][J][r] *= f1;
          P2.re[I][J][r] *= f2;
          if constexpr (CPLX) {
            X.im[I][J][r] *= f1;
            P2.im[I][J][r] *= f2;
          }
        }
  }
  // ---- E0 = p(X / kappa) (see ExpPoly) ----
  xzero(P3);
  xmm(X, P2, P3);
  M = P3;
  xpoly<NB, CPLX, false, false, true>(M, 0.0, EP::b1, EP::b2, 0.0, X, P2, P3, dg);
  {
    XMat<NB, CPLX> B;
    xpoly<NB, CPLX, true, false, false>(B, 0.0, EP::r1, EP::r2, EP::r3, X, P2, P3, dg);
    xmm(M, M, B);   // a6
    M = B;
    xpoly<NB, CPLX, true, true, true>(M, EP::s0, EP::s1, EP::s2, EP::s3, X, P2, P3, dg);
    xpoly<NB, CPLX, false, true, false>(X, 1.0, EP::t1, EP::t2, 0.0, X, P2, P3, dg);
    xmm(M, B, X);
    M = X;
  }
  // ---- normalise and square s times ----
  // Every rescaling is by an exact power of two 2^-e_j, e_j the binary exponent of the trace
  // (frexp's exponent minus one; a non-finite trace leaves the result non-finite, which is flagged):
  // first E0 itself (e_0, so Y_0 has trace in [1, 2)), then the squares j = 3, 7, 11, ...  For a
  // PSD Y with trace at least 1 the largest eigenvalue is at least 1/D, so four unscaled
  // squarings keep the trace within [D^-16, 2^16], far inside the FP32 and FP64 ranges, and up to
  // three more after the last rescaling keep it above D^-8.  The exponents are accumulated as an
  // integer, E <- 2E + e_j (starting from E = e_0), so no logarithm or division sits in the loop:
  //     log Z = E log 2 + log Tr Y_s,   rho = Y_s / Tr Y_s.
  // X and M alternate as product buffers (the loop is unrolled by two).
  // E holds the accumulated exponent as of squaring jr (jr = -1: before the first); the value
  // after squaring j is E 2^(j - jr), so only the rescaling points touch it (ldexp is exact here).
  double E;
  int jr = -1;
  {
    const int e0 = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_frexp_expf(xtrace_est(M, l)) - 1);
    E = (double)e0;
    const double sc0 = ldexp(1.0, -e0);
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J < NB; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          M.re[I][J][r] *= sc0;
          if constexpr (CPLX) M.im[I][J][r] *= sc0;
        }
  }
  // Float messages: the squarings after the first kF64Squarings run on the FP32 matrix cores.  A
  // relative rounding error e in Y_j acts on rho like an error of about 2^(s-j) e in
  // X = beta (theta - mu).  2^s is below r = sqrt(||X^2||_1), the bound that set it, so after two squarings
  // the float ones perturb X by at most about r u_32 / 4 times the product's error growth.  r is at
  // most D^(1/4) times ||X|| (2 at D = 16, 2.4 at 32; 1.6 seen at 32), so this is the order of what the float
  // rounding of the messages themselves puts on X (beta ||nu|| u_32).  The polynomial and the first
  // squarings, where the error would be amplified most, stay in FP64.
  int n64 = s;
  if constexpr (std::is_same<T, float>::value) n64 = s < kF64Squarings ? s : kF64Squarings;
  auto post = [&](XMat<NB, CPLX>& Y, int j) {
    if ((j & 3) == 3) {
      const int e = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_frexp_expf(xtrace_est(Y, l)) - 1);
      E = ldexp(E, j - jr) + (double)e;
      jr = j;
      const double sc2 = ldexp(1.0, -e);
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J < NB; ++J)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            Y.re[I][J][r] *= sc2;
            if constexpr (CPLX) Y.im[I][J][r] *= sc2;
          }
    }
  };
  for (int j = 0; j < n64; j += 2) {
    xzero(X);
    xmm(M, M, X);
    post(X, j);
    if (j + 1 < n64) {
      xzero(M);
      xmm(X, X, M);
      post(M, j + 1);
    } else {
      M = X;
    }
  }
  if (n64 < s) {
    // Squarings n64 .. s-1.  The first takes its operands straight from the FP64 registers: there
    // lane group g, register kk holds row 4 kk + g, which serves as well as row 4 g + kk as the k
    // index of a step, since both operands use the same one; its result is in the FP32 layout.
    XMat32<NB, CPLX> Ya, Yb;
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J < NB; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          Ya.re[I][J][r] = (float)M.re[I][J][r];
          if constexpr (CPLX) Ya.im[I][J][r] = (float)M.im[I][J][r];
        }
    auto post32 = [&](XMat32<NB, CPLX>& Y, int j) {
      if ((j & 3) == 3) {
        const int e = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_frexp_expf(xtrace32(Y, l)) - 1);
        E = ldexp(E, j - jr) + (double)e;
        jr = j;
        const float sc2 = ldexpf(1.f, -e);
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
          for (int J = 0; J < NB; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              Y.re[I][J][r] *= sc2;
              if constexpr (CPLX) Y.im[I][J][r] *= sc2;
            }
      }
    };
    for (int j = n64; j < s; j += 2) {
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = 0; J < NB; ++J)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            Yb.re[I][J][r] = 0.f;
            if constexpr (CPLX) Yb.im[I][J][r] = 0.f;
          }
      xmm32(Ya, Ya, Yb);
      post32(Yb, j);
      if (j + 1 < s) {
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
          for (int J = 0; J < NB; ++J)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              Ya.re[I][J][r] = 0.f;
              if constexpr (CPLX) Ya.im[I][J][r] = 0.f;
            }
        xmm32(Yb, Yb, Ya);
        post32(Ya, j + 1);
      } else {
        Ya = Yb;
      }
    }
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J < NB; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          M.re[I][J][r] = (double)Ya.re[I][J][r];
          if constexpr (CPLX) M.im[I][J][r] = (double)Ya.im[I][J][r];
        }
  }
  // row of register r of a diagonal block: the FP64 layout, or the FP32 one after float squarings
  const bool tail32 = n64 < s;
  const auto row = [&](int r) { return tail32 ? 4 * (l >> 4) + r : 4 * r + (l >> 4); };
  double L;
  {
    E = ldexp(E, s - 1 - jr);   // the exponent after the last squaring
    const double tf = tail32 ? xtrace_f32(M, l) : xtrace(M, l);
    double kf;
    const double lm = log_split(tf, kf);
    L = fma(E + kf, 0.69314718055994530942, lm);   // E + kf is exact
    // 1 / tf from the hardware reciprocal and two Newton steps (tf is a positive normal number)
    double it = __builtin_amdgcn_rcp(tf);
    it = fma(fma(-tf, it, 1.0), it, it);
    it = fma(fma(-tf, it, 1.0), it, it);
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J < NB; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          M.re[I][J][r] *= it;
          if constexpr (CPLX) M.im[I][J][r] *= it;
        }
  }
  const double F = mu - L / beta;
  const int32_t gid = A.gid[c];
  if (l == 0) {
    if (A.scal) A.scal[gid] = F;
    if (!isfinite(F) && A.nonfinite) atomicAdd(A.nonfinite, 1ull);
  }
  // ---- a5: rho back to LDS, then the outputs ----
  __syncthreads();
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = 0; J < NB; ++J)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = (16 * I + row(r)) * LD + 16 * J + (l & 15);
        sar[o] = (T)M.re[I][J][r];
        if constexpr (CPLX) sai[o] = (T)M.im[I][J][r];
      }
  __syncthreads();
  if (!lut) {
    lds_outputs<T, CPLX, DE, 64>(A, c, l, gid, sar, sai);
    return;
  }
  // own marginal slot and per-cluster marginal, straight from the registers (upper triangle)
  const int64_t rs_self = A.rslot ? A.rslot[c] : -1;
  if ((rs_self >= 0 && A.R) || A.marg) {
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = 0; J < NB; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * I + row(r), j = 16 * J + (l & 15);
          if (i > j) continue;
          const int kr = tri_index(i, j, DE);
          const T vr = (T)M.re[I][J][r];
          if (rs_self >= 0 && A.R) A.R[(int64_t)kr * A.S + rs_self] = vr;
          if (A.marg) A.marg[A.marg_off[gid] + kr] = vr;
          if constexpr (CPLX) {
            if (i < j) {
              const int ki = DE * (DE + 1) / 2 + stri_index(i, j, DE);
              const T vi = (T)M.im[I][J][r];
              if (rs_self >= 0 && A.R) A.R[(int64_t)ki * A.S + rs_self] = vi;
              if (A.marg) A.marg[A.marg_off[gid] + ki] = vi;
            }
          }
        }
  }
  // partial traces onto every child, all (child, component) pairs across the lanes
  if (A.Tout && Dc > 0) {
    const int NR = 1 << lnr;
    const int NCC = CPLX ? Dc * Dc : Dc * (Dc + 1) / 2;
    for (int idx = l; idx < nch * NCC; idx += 64) {
      int s = 0, k = idx;
      while (k >= NCC) {   // (child, component) without an integer division; at most nch steps
        k -= NCC;
        ++s;
      }
      const int m = A.ch[(int64_t)s * A.n + c];
      if (m < 0) continue;
      int a, b;
      bool im;
      decode_comp(k, Dc, a, b, im);
      const T* y = im ? sai : sar;
      T sum = T(0);
      for (int x = 0; x < NR; ++x) sum += y[depL[s][(a << lnr) + x] * LD + depL[s][(b << lnr) + x]];
      A.Tout[(int64_t)k * A.Mc + m] = sum;
    }
  }
}

template <typename T, bool CPLX, int DE>
__global__ __launch_bounds__(64) void k_cluster_expm(ClusterArgs<T> A) {
  cluster_expm_body<T, CPLX, DE>(A, blockIdx.x);
}

// The 16-dimensional clusters with the bonds and sites below them in one launch (float): the first
// nbe + nbs workgroups are those of the pair kernel, whose waves wait on memory and on one
// another's rotations most of the time (26 000 plaquettes: 14 + 5 us as launches of their own), the
// rest one wave per 16-dimensional cluster.  The buckets do not depend on one another.
template <typename T, bool CPLX>
__global__ __launch_bounds__(64) void k_cluster_expm16_pair(ClusterArgs<T> A, ClusterArgs<T> E, ClusterArgs<T> S, int nbe,
                                                            int nbs) {
  const int b = blockIdx.x;
  if (b < nbe) {
    const int64_t c = (int64_t)b * 64 + threadIdx.x;
    if (c < E.n) cluster_reg_body<T, CPLX, 4, 2, MODE_GIBBS>(E, c);
  } else if (b < nbe + nbs) {
    const int64_t c = (int64_t)(b - nbe) * 64 + threadIdx.x;
    if (c < S.n) cluster_reg_body<T, CPLX, 2, 0, MODE_GIBBS>(S, c);
  } else {
    cluster_expm_body<T, CPLX, 16>(A, b - nbe - nbs);
  }
}

// Workgroup variant for De = 32, 64, 128, 256: five matrices in a per-workgroup slab, row-major.  A
// complex Hermitian matrix R + i N (R symmetric, N antisymmetric) is kept as the one real matrix
// Z = R + N (so Z^T = R - N), half the memory of two planes.  For commuting Hermitian factors
//     Z' = Z1 Z2 - 2 N1 N2,   Z'^T = Z1^T Z2^T - 2 N1 N2,
// so the two off-diagonal blocks (I, J) and (J, I) of a product take three real block products (four
// with separate planes) and the second comes out transposed, as the lanes need it.  Only the 16 x 16
// blocks on and above the diagonal are computed.  For both, the operands of a k-step are rows and
// columns k of the matrix: KS whole rows, and for complex matrices KS whole columns, go to LDS at a
// time (LDS-direct loads, two buffers, one barrier per step), where every wave reads the fragments of
// its blocks.  The kernel is bound by the memory traffic of the products: reading fragments from the
// slab (32 x 32 tiles per wave, no LDS, two planes) moved 10 MB per 256 x 256 product at 5 TB/s.
//
// Blocks of a product and the waves that compute them: `passes` sweeps over the rows, in each of
// which a wave holds the accumulators of `nblk` blocks (ab[b], bb[b] index its A and B fragments).
template <int DE>
struct WgPlan;
template <>
struct WgPlan<256> {   // 36 tiles of 2 x 2 blocks: three per wave, three waves per SIMD
  static constexpr int waves = 12, passes = 3, na = 2, nb = 2, nblk = 4, ks = 16;
  static constexpr int ab[4] = {0, 0, 1, 1}, bb[4] = {0, 1, 0, 1};
};
template <>
struct WgPlan<128> {   // 36 blocks, three per wave: rows in runs of three, the rest as two and one
  static constexpr int waves = 12, passes = 1, na = 2, nb = 3, nblk = 3, ks = 32;
  static constexpr int ab[3] = {0, 0, 1}, bb[3] = {0, 1, 2};
};
template <>
struct WgPlan<64> {    // 10 blocks, two per wave
  static constexpr int waves = 5, passes = 1, na = 2, nb = 2, nblk = 2, ks = 16;
  static constexpr int ab[2] = {0, 1}, bb[2] = {0, 1};
};
template <>
struct WgPlan<32> {    // 3 blocks, one per wave
  static constexpr int waves = 3, passes = 1, na = 1, nb = 1, nblk = 1, ks = 8;
  static constexpr int ab[1] = {0}, bb[1] = {0};
};
// A rows then B columns (in blocks) of every (pass, wave)
struct WgBlocks {
  unsigned char t256[36][4], t128[12][5], t64[5][4], t32[3][2];
};
constexpr WgBlocks make_wg_blocks() {
  WgBlocks w{};
  int t = 0;
  for (int i = 0; i < 8; ++i)
    for (int j = i; j < 8; ++j, ++t) {
      w.t256[t][0] = (unsigned char)(2 * i);
      w.t256[t][1] = (unsigned char)(2 * i + 1);
      w.t256[t][2] = (unsigned char)(2 * j);
      w.t256[t][3] = (unsigned char)(2 * j + 1);
    }
  constexpr unsigned char g128[12][5] = {{0, 0, 0, 1, 2}, {0, 0, 3, 4, 5}, {1, 1, 1, 2, 3}, {1, 1, 4, 5, 6},
                                         {2, 2, 2, 3, 4}, {2, 2, 5, 6, 7}, {3, 3, 3, 4, 5}, {4, 4, 4, 5, 6},
                                         {5, 5, 5, 6, 7}, {0, 1, 6, 7, 7}, {3, 4, 6, 7, 7}, {6, 7, 6, 7, 7}};
  constexpr unsigned char g64[5][4] = {{0, 0, 0, 1}, {0, 0, 2, 3}, {1, 1, 1, 2}, {1, 3, 3, 3}, {2, 2, 2, 3}};
  constexpr unsigned char g32[3][2] = {{0, 0}, {0, 1}, {1, 1}};
  for (int i = 0; i < 12; ++i)
    for (int k = 0; k < 5; ++k) w.t128[i][k] = g128[i][k];
  for (int i = 0; i < 5; ++i)
    for (int k = 0; k < 4; ++k) w.t64[i][k] = g64[i][k];
  for (int i = 0; i < 3; ++i)
    for (int k = 0; k < 2; ++k) w.t32[i][k] = g32[i][k];
  return w;
}
static __constant__ WgBlocks kWgBlocks = make_wg_blocks();
template <int DE>
__device__ __forceinline__ int wg_block(int t, int k) {
  if constexpr (DE == 256) return kWgBlocks.t256[t][k];
  else if constexpr (DE == 128) return kWgBlocks.t128[t][k];
  else if constexpr (DE == 64) return kWgBlocks.t64[t][k];
  else return kWgBlocks.t32[t][k];
}
template <bool CPLX, int DE>
constexpr int wg_stage_bytes() { return WgPlan<DE>::ks * DE * (CPLX ? 2 : 1) * (int)sizeof(double); }

__device__ __forceinline__ mfma_f64x4 wg_mma(double a, double b, mfma_f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int wg_row(int l, int r) { return 4 * r + (l >> 4); }   // row of result register r
// Bank swizzles of a stage.  Row k: the four rows that one fragment read touches would start on the
// same bank, so its blocks of 16 elements are permuted by block ^ wg_swizzle(k), which depends on the
// low bits of k only (those of l / 16 for a reading lane).  Columns are staged as DE pieces of CC
// 16-byte chunks (element (i, k0 + .)); piece i has its chunks permuted by chunk ^ wg_csw(i), which
// spreads the 16 pieces of a fragment over the banks.
template <typename S, int DE>
__device__ __forceinline__ int wg_swizzle(int k) {
  return sizeof(S) == 8 ? (k & 1) : (DE >= 64 ? (k & 3) : ((k >> 1) & 1));
}
template <int CC>
__device__ __forceinline__ int wg_csw(int i) {
  static_assert(CC == 2 || CC == 4 || CC == 8 || CC == 16, "chunks per piece");
  return CC == 16 ? (i & 15) : CC == 8 ? ((i >> 1) & 7) : CC == 4 ? ((i >> 2) & 3) : ((i >> 3) & 1);
}

// Sizes of a stage: KS rows (complex: and columns) of X (and of Y unless SAME; then half as many).
template <bool CPLX, int DE, bool SAME>
struct WgStage {
  using P = WgPlan<DE>;
  static constexpr int NPL = CPLX ? 2 : 1;
  static constexpr int KS0 = P::ks / (SAME ? 1 : 2);
  static constexpr int KS = KS0 < DE ? KS0 : DE;
  static constexpr int NK = DE / KS;
  static constexpr int PB = KS * DE * (int)sizeof(double);   // bytes of a panel (rows or columns)
  static constexpr int NINS = PB / 1024;                 // wave loads per panel
  static constexpr int CPR = DE / 2;   // 16-byte chunks per row
  static constexpr int CC = KS / 2;    // and per column piece
  static constexpr int NPAN = NPL * (SAME ? 1 : 2);
  static_assert(NINS * 1024 == PB && KS % 4 == 0 && NK * KS == DE, "whole wave loads and stages");
  static_assert(NPAN * PB <= wg_stage_bytes<CPLX, DE>(), "stage fits its buffer");
};

// Rows (and columns) k0 .. k0 + KS - 1 to the buffer, by LDS-direct loads spread over the waves:
// panels X rows, X columns, Y rows, Y columns.
template <bool CPLX, int DE, bool SAME>
__device__ __forceinline__ void wg_fill(const double* X, const double* Y, int k0, unsigned char* buf, int wave, int l) {
  using G = WgStage<CPLX, DE, SAME>;
  constexpr int EPC = 2;   // elements per chunk
#pragma unroll
  for (int pan = 0; pan < G::NPAN; ++pan) {
    const double* Z = pan < G::NPL ? X : Y;
#pragma unroll 2
    for (int q = wave; q < G::NINS; q += G::P::waves) {
      const int ch = q * 64 + l;
      int64_t o;
      if (pan % G::NPL == 0) {
        const int k = ch / G::CPR, cp = ch % G::CPR;
        o = (int64_t)(k0 + k) * DE + (cp ^ (wg_swizzle<double, DE>(k) * 8)) * EPC;   // 8 chunks per block
      } else {
        const int i = ch / G::CC, cp = ch % G::CC;
        o = (int64_t)i * DE + k0 + (cp ^ wg_csw<G::CC>(i)) * EPC;
      }
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(Z + o),
                                       (__attribute__((address_space(3))) void*)(buf + pan * G::PB + q * 1024), 16, 0, 0);
    }
  }
}

// Accumulators of a wave's blocks: real: s1 the block; complex: s1 of Z1 Z2, s4 of (Z1^T Z2^T), p2 of
// -(2 N1)(2 N2)
template <bool CPLX, int DE>
struct WgAcc {
  static constexpr int N = WgPlan<DE>::nblk;
  mfma_f64x4 s1[N], s4[CPLX ? N : 1], p2[CPLX ? N : 1];
};

// One stage: the next one's loads are issued into `nxt` (k0 >= 0), then the products of the rows in
// `st` are accumulated.  The two are different buffers: `restrict` tells the compiler so, which
// would otherwise wait for the loads before the first read.  oz, ow: byte offsets of a lane's row and
// column elements at kk = 0 (A blocks, then B blocks).
template <bool CPLX, int DE, bool SAME>
__device__ __forceinline__ void wg_step(const unsigned char* __restrict__ st, unsigned char* __restrict__ nxt, const double* X,
                                        const double* Y, int k0, int wave, int l,
                                        const int (&oz)[WgPlan<DE>::na + WgPlan<DE>::nb],
                                        const int (&ow)[WgPlan<DE>::na + WgPlan<DE>::nb], WgAcc<CPLX, DE>& acc) {
  using P = WgPlan<DE>;
  using G = WgStage<CPLX, DE, SAME>;
  constexpr int NF = P::na + P::nb;
  if (k0 >= 0) wg_fill<CPLX, DE, SAME>(X, Y, k0, nxt, wave, l);
#pragma unroll 4
  for (int kk = 0; kk < G::KS / 4; ++kk) {
    double z[NF], w[NF];
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      z[q] = *reinterpret_cast<const double*>(st + oz[q] + kk * 4 * DE * (int)sizeof(double));
      // chunk (4 kk + l / 16) / EPC of the piece, permuted: kk only toggles bits of the offset
      if constexpr (CPLX) w[q] = *reinterpret_cast<const double*>(st + (ow[q] ^ (kk * 4 * (int)sizeof(double))));
    }
#pragma unroll
    for (int b = 0; b < P::nblk; ++b) {
      const int ia = P::ab[b], ib = P::na + P::bb[b];
      if constexpr (CPLX) {
        // A operands are transposes of what the lanes hold
        acc.s1[b] = wg_mma(w[ia], z[ib], acc.s1[b]);
        acc.s4[b] = wg_mma(z[ia], w[ib], acc.s4[b]);
        acc.p2[b] = wg_mma(z[ia] - w[ia], z[ib] - w[ib], acc.p2[b]);
      } else {
        acc.s1[b] = wg_mma(z[ia], z[ib], acc.s1[b]);
      }
    }
  }
}

// epi(I, J, v, u): the block (I, J) of X Y (SAME: Y is X), v[r] element (i, j) of the result's Z, u[r]
// element (j, i), for every block I <= J.  X, Y: slab matrices.  s0, s1: buffers of
// wg_stage_bytes().  All waves call it, after a barrier that follows the writes of X and Y; it ends
// with one itself.
template <bool CPLX, int DE, bool SAME, typename Epi>
__device__ __forceinline__ void wg_product(const double* X, const double* Y, unsigned char* s0, unsigned char* s1, int tid,
                                           Epi&& epi) {
  using P = WgPlan<DE>;
  using G = WgStage<CPLX, DE, SAME>;
  static_assert(G::NK % 2 == 0, "stages alternate between the buffers");
  constexpr int NF = P::na + P::nb;
  constexpr int ES = (int)sizeof(double);
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64;
  const int lr = l >> 4, lc = l & 15;
  wg_fill<CPLX, DE, SAME>(X, Y, 0, s0, wave, l);
#pragma unroll 1
  for (int pass = 0; pass < P::passes; ++pass) {
    const int t = pass * P::waves + wave;
    int blk[NF], oz[NF], ow[NF];
#pragma unroll
    for (int q = 0; q < NF; ++q) {
      blk[q] = wg_block<DE>(t, q);
      const int pan = q < P::na || SAME ? 0 : G::NPL * G::PB;   // X's panels, or Y's
      oz[q] = pan + (lr * DE + 16 * (blk[q] ^ wg_swizzle<double, DE>(lr)) + lc) * ES;
      ow[q] = pan + G::PB + (16 * blk[q] + lc) * G::CC * 16 + (((lr * ES / 16) ^ wg_csw<G::CC>(lc)) * 16 | (lr * ES & 15));
    }
    WgAcc<CPLX, DE> acc;
#pragma unroll
    for (int b = 0; b < P::nblk; ++b) {
      acc.s1[b] = mfma_f64x4{0, 0, 0, 0};
      if constexpr (CPLX) acc.s4[b] = acc.p2[b] = mfma_f64x4{0, 0, 0, 0};
    }
#pragma unroll 1
    for (int K = 0; K < G::NK; K += 2) {
      __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's loads of the stage have landed
      __syncthreads();                      // and every wave's; the other buffer is no longer read
      wg_step<CPLX, DE, SAME>(s0, s1, X, Y, (K + 1) * G::KS, wave, l, oz, ow, acc);
      __builtin_amdgcn_s_waitcnt(0x0f70);
      __syncthreads();
      const int k0 = K + 2 < G::NK ? (K + 2) * G::KS : (pass + 1 < P::passes ? 0 : -1);
      wg_step<CPLX, DE, SAME>(s1, s0, X, Y, k0, wave, l, oz, ow, acc);
    }
#pragma unroll
    for (int b = 0; b < P::nblk; ++b) {
      const int I = blk[P::ab[b]], J = blk[P::na + P::bb[b]];
      if (I > J) continue;   // a 2 x 2 tile on the diagonal also covers its block below it
      if constexpr (CPLX) {
        const mfma_f64x4 p = 0.5 * acc.p2[b];
        epi(I, J, acc.s1[b] + p, acc.s4[b] + p);
      } else {
        epi(I, J, acc.s1[b], acc.s1[b]);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);   // the epilogues' stores, before anyone stages them
  __syncthreads();
}

// Plan of a float squaring: all tiles of 32 x 32 in one pass at D = 256 (half the accumulators of a
// double product), else as WgPlan.
template <int DE>
struct WgPlan32 : WgPlan<DE> {};
template <>
struct WgPlan32<256> {
  static constexpr int waves = 12, passes = 1, na = 6, nb = 6, nblk = 12, ks = 16;
  static constexpr int ab[12] = {0, 0, 1, 1, 2, 2, 3, 3, 4, 4, 5, 5}, bb[12] = {0, 1, 0, 1, 2, 3, 2, 3, 4, 5, 4, 5};
};
// block index of A fragment q (q < na), or B fragment q - na
template <int DE>
__device__ __forceinline__ int wg_block32(int wave, int q) {
  if constexpr (DE == 256) {
    const int a = q < 6 ? q : q - 6;
    return wg_block<256>(wave + 12 * (a >> 1), (q < 6 ? 0 : 2) + (a & 1));
  } else {
    return wg_block<DE>(wave, q);
  }
}

// One step of wg_square32: when the stage in `st` has landed, the next one's loads into `nxt`, then the
// products (`restrict`: see wg_step).
template <typename Fill, typename Prod>
__device__ __forceinline__ void wg_square32_step(const unsigned char* __restrict__ st, unsigned char* __restrict__ nxt,
                                                 Fill&& fill, Prod&& products) {
  __builtin_amdgcn_s_waitcnt(0x0f70);
  __syncthreads();
  fill(nxt);
  products(reinterpret_cast<const float*>(st));
}

// epi(I, J, re, im): block (I, J) of Y Y for a Hermitian float matrix in two planes (real: one), on the
// FP32 matrix cores, four real products per complex one.  A 2 x 2 tile on the diagonal also gives
// its block below it.  Buffers and barriers as wg_product.
template <bool CPLX, int DE, typename Epi>
__device__ __forceinline__ void wg_square32(const float* Y, unsigned char* s0, unsigned char* s1, int tid, Epi&& epi) {
  using P = WgPlan32<DE>;
  constexpr int NPL = CPLX ? 2 : 1;
  constexpr int KS = 2 * P::ks < DE / 2 ? 2 * P::ks : DE / 2;
  constexpr int NK = DE / KS, CPR = DE / 4, NINS = KS * CPR / 64, PB = KS * DE * 4, NF = P::na + P::nb;
  static_assert(NINS * 64 == KS * CPR && NK % 2 == 0 && KS % 4 == 0 && NPL * PB <= wg_stage_bytes<CPLX, DE>(), "stages");
  constexpr int64_t DD = (int64_t)DE * DE;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64;
  const int lr = l >> 4, lc = l & 15;
  const auto fill = [&](int k0, unsigned char* buf) {
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl)
#pragma unroll 2
      for (int q = wave; q < NINS; q += P::waves) {
        const int ch = q * 64 + l, k = ch / CPR, cp = ch % CPR;
        const float* src = Y + pl * DD + (int64_t)(k0 + k) * DE + (cp ^ (wg_swizzle<float, DE>(k) * 4)) * 4;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)(buf + pl * PB + q * 1024), 16, 0, 0);
      }
  };
  int blk[NF], off[NF];
#pragma unroll
  for (int q = 0; q < NF; ++q) {
    blk[q] = wg_block32<DE>(wave, q);
    off[q] = lr * DE + 16 * (blk[q] ^ wg_swizzle<float, DE>(lr)) + lc;
  }
  mfma_f32x4 cr[P::nblk], ci[CPLX ? P::nblk : 1];
#pragma unroll
  for (int b = 0; b < P::nblk; ++b) {
    cr[b] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (CPLX) ci[b] = mfma_f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const auto products = [&](const float* __restrict__ st) {
#pragma unroll 2
    for (int kk = 0; kk < KS / 4; ++kk) {
      float r[NF], n[NF];
#pragma unroll
      for (int q = 0; q < NF; ++q) {
        r[q] = st[off[q] + kk * 4 * DE];
        if constexpr (CPLX) n[q] = st[off[q] + kk * 4 * DE + KS * DE];
      }
#pragma unroll
      for (int b = 0; b < P::nblk; ++b) {
        const int ia = P::ab[b], ib = P::na + P::bb[b];
        cr[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(r[ia], r[ib], cr[b], 0, 0, 0);
        if constexpr (CPLX) {
          cr[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(n[ia], n[ib], cr[b], 0, 0, 0);
          ci[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(r[ia], n[ib], ci[b], 0, 0, 0);
          ci[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(-n[ia], r[ib], ci[b], 0, 0, 0);
        }
      }
    }
  };
  fill(0, s0);
#pragma unroll 1
  for (int K = 0; K < NK; K += 2) {
    wg_square32_step(s0, s1, [&](unsigned char* nxt) { fill((K + 1) * KS, nxt); }, products);
    wg_square32_step(s1, s0, [&](unsigned char* nxt) { if (K + 2 < NK) fill((K + 2) * KS, nxt); }, products);
  }
#pragma unroll
  for (int b = 0; b < P::nblk; ++b) epi(blk[P::ab[b]], blk[P::na + P::bb[b]], cr[b], CPLX ? ci[b] : cr[b]);
  __builtin_amdgcn_s_waitcnt(0x0f70);   // the epilogues' stores, before anyone stages them
  __syncthreads();
}

// Elements (i, j) of block (I, J), I <= J, to the slab matrix C: v, and u to (j, i).
template <int DE>
__device__ __forceinline__ void wg_store(double* C, int I, int J, int l, const double (&v)[4], const double (&u)[4]) {
  const int j = 16 * J + (l & 15);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 16 * I + wg_row(l, r);
    C[i * DE + j] = v[r];
    if (I != J) C[j * DE + i] = u[r];
  }
}
// The result instead as planes R and N: of its upper triangle, as the outputs read it, or (FULL) whole.
template <bool CPLX, typename D, int DE, bool FULL = false>
__device__ __forceinline__ void wg_store_planes(D* C, int I, int J, int l, const double (&v)[4], const double (&u)[4]) {
  constexpr int64_t DD = (int64_t)DE * DE;
  const int j = 16 * J + (l & 15);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 16 * I + wg_row(l, r);
    const D re = CPLX ? (D)(0.5 * (v[r] + u[r])) : (D)v[r];
    C[i * DE + j] = re;
    if (FULL && I != J) C[j * DE + i] = re;
    if constexpr (CPLX) {
      const D im = (D)(0.5 * (v[r] - u[r]));
      C[DD + i * DE + j] = im;
      if (FULL && I != J) C[DD + j * DE + i] = -im;
    }
  }
}

// Trace of theta_e (this thread's share).
template <typename T, bool CPLX, int DE>
__device__ double wg_trace(const ClusterArgs<T>& A, int64_t c, T th, int tid, int nth) {
  double tr = 0.0;
  for (int i = tid; i < DE; i += nth) {
    T vr, vi;
    theta_elem<T, CPLX>(A, c, DE, log2i(DE), A.hoff[c], i, i, th, vr, vi);
    tr += (double)vr;
  }
  return tr;
}

// X = sc (theta_e - mu) into the slab (Z form): one row per wave at a time, a lane on fixed columns,
// only j >= i (the rest by symmetry).  With NORMS returns min(||X||_1, ||X||_F), each sum in a fixed
// order; part: (nth / 64 + 1) DE doubles of LDS.
template <typename T, bool CPLX, int DE, bool NORMS>
__device__ double wg_assemble(const ClusterArgs<T>& A, int64_t c, double* X, T th, double sc, double mu, double* part,
                              double* red, int tid, int nth) {
  constexpr int NC = DE > 64 ? DE / 64 : 1;   // columns per lane
  const int64_t ho = A.hoff[c];
  const int wave = tid / 64, l = tid % 64, nw = nth / 64;
  double col[NC], n2 = 0.0;
#pragma unroll
  for (int t = 0; t < NC; ++t) col[t] = 0.0;
  for (int i = wave; i < DE; i += nw) {
    double row = 0.0;
#pragma unroll
    for (int t = 0; t < NC; ++t) {
      const int j = 64 * t + l;
      if (j < i || j >= DE) continue;
      T vr, vi;
      theta_elem<T, CPLX>(A, c, DE, log2i(DE), ho, i, j, th, vr, vi);
      const double xr = sc * ((double)vr - (i == j ? mu : 0.0));
      const double xi = CPLX && i != j ? sc * (double)vi : 0.0;
      X[i * DE + j] = xr + xi;
      if (i != j) X[j * DE + i] = xr - xi;
      if constexpr (NORMS) {
        const double m2 = fma(xr, xr, xi * xi), m = __builtin_amdgcn_sqrt(m2);
        row += m;
        col[t] += i != j ? m : 0.0;
        n2 += i != j ? 2.0 * m2 : m2;
      }
    }
    if constexpr (NORMS) {
      row = wave_sum(row);
      if (l == 0) part[nw * DE + i] = row;
    }
  }
  if constexpr (!NORMS) return 0.0;
#pragma unroll
  for (int t = 0; t < NC; ++t)
    if (64 * t + l < DE) part[wave * DE + 64 * t + l] = col[t];
  __syncthreads();
  double rmax = 0.0;
  for (int i = tid; i < DE; i += nth) {
    double a = part[nw * DE + i];
    for (int w = 0; w < nw; ++w) a += part[w * DE + i];
    rmax = fmax(rmax, a);
  }
  return fmin(sqrt(block_sum(n2, red)), block_max(rmax, red));
}

// Outputs of a cluster whose marginal scale * Y sits in the slab (planes of the upper triangle): own
// marginal slot, per-cluster marginal, partial traces onto every child.  One row of the packed upper triangle per wave at a
// time, the lanes along it.
template <typename T, typename S, bool CPLX, int DE>
__device__ void wg_outputs(const ClusterArgs<T>& A, int64_t c, int32_t gid, const S* Y, double scale, int tid, int nth) {
  constexpr int64_t DD = (int64_t)DE * DE;
  constexpr int NB = log2i(DE);
  const int wave = tid / 64, l = tid % 64, nw = nth / 64;
  const int Dc = A.Dc;
  const int64_t rs_self = A.rslot ? A.rslot[c] : -1;
  if ((rs_self >= 0 && A.R) || A.marg) {
    T* mg = A.marg ? A.marg + A.marg_off[gid] : nullptr;
    for (int i = wave; i < DE; i += nw)
      for (int j = i + l; j < DE; j += 64) {
        const int kr = tri_index(i, j, DE);
        const T vr = (T)(scale * (double)Y[i * DE + j]);
        if (rs_self >= 0 && A.R) A.R[(int64_t)kr * A.S + rs_self] = vr;
        if (mg) mg[kr] = vr;
        if constexpr (CPLX) {
          if (i < j) {
            const int ki = DE * (DE + 1) / 2 + stri_index(i, j, DE);
            const T vi = (T)(scale * (double)Y[DD + i * DE + j]);
            if (rs_self >= 0 && A.R) A.R[(int64_t)ki * A.S + rs_self] = vi;
            if (mg) mg[ki] = vi;
          }
        }
      }
  }
  if (!A.Tout || Dc <= 0) return;
  const int NR = DE / Dc;
  for (int s = 0; s < A.maxch; ++s) {
    const int m = A.ch[(int64_t)s * A.n + c];
    if (m < 0) continue;
    const int mask = A.chmask[(int64_t)s * A.n + c];
    for (int a = wave; a < Dc; a += nw)
      for (int b = a + l; b < Dc; b += 64) {
        const int i0 = pdep_rt(a, 0, mask, NB), j0 = pdep_rt(b, 0, mask, NB);
        double sr = 0.0, si = 0.0;
        for (int x = 0; x < NR; ++x) {
          const int y = pdep_rt(0, x, mask, NB);
          const int o = (i0 | y) * DE + (j0 | y);
          sr += (double)Y[o];
          if constexpr (CPLX) si += (double)Y[DD + o];
        }
        A.Tout[(int64_t)tri_index(a, b, Dc) * A.Mc + m] = (T)(scale * sr);
        if constexpr (CPLX) {
          if (a < b) A.Tout[(int64_t)(Dc * (Dc + 1) / 2 + stri_index(a, b, Dc)) * A.Mc + m] = (T)(scale * si);
        }
      }
  }
}

template <typename T, bool CPLX, int DE>
__global__ __launch_bounds__(WgPlan<DE>::waves * 64) void k_cluster_expm_wg(ClusterArgs<T> A, double* scratch, int64_t slab) {
  constexpr int64_t DD = (int64_t)DE * DE;
  constexpr int NPL = CPLX ? 2 : 1;
  constexpr int NB16 = DE / 16;
  __shared__ __attribute__((aligned(1024))) unsigned char stage0[wg_stage_bytes<CPLX, DE>()], stage1[wg_stage_bytes<CPLX, DE>()];
  __shared__ double red[16];
  using EP = ExpPoly<T>;
  const int tid = threadIdx.x, nth = blockDim.x, l = tid % 64;
  double* base = scratch + (int64_t)blockIdx.x * slab;
  double *X = base, *P2 = base + NPL * DD, *P3 = base + 2 * NPL * DD;
  const T th = A.tab ? (T)A.tab->theta_cur : (T)A.theta;
  const double beta = A.tab ? A.tab->beta : A.beta;
  // neighbouring clusters (whose messages share cache lines) to the same XCD
  for (int64_t c0 = 0; c0 < A.n; c0 += gridDim.x) {
    const int64_t nc = A.n - c0 < (int64_t)gridDim.x ? A.n - c0 : (int64_t)gridDim.x;
    if ((int64_t)blockIdx.x >= nc) break;   // block-uniform
    const int64_t c = c0 + xcd_cluster(blockIdx.x, nc);
    double *M = base + 3 * NPL * DD, *Q = base + 4 * NPL * DD;
    // ---- a1/a2: X = -kappa beta (theta_e - mu) at eta ----
    constexpr bool kF32 = std::is_same<T, float>::value;
    const double mu = block_sum(wg_trace<T, CPLX, DE>(A, c, th, tid, nth), red) / DE;
    const double xn = wg_assemble<T, CPLX, DE, kF32>(A, c, X, th, -EP::kappa * beta, mu,
                                                     reinterpret_cast<double*>(stage0), red, tid, nth);
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    // ---- X^2, its column sums (per block row, in the still unused Q) and the scale; see k_cluster_expm ----
    wg_product<CPLX, DE, true>(X, X, stage0, stage1, tid, [&](int I, int J, mfma_f64x4 av, mfma_f64x4 au) {
      double v[4], u[4], m[4], cs = 0.0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v[r] = av[r];
        u[r] = au[r];
        // modulus: R^2 + N^2 = (v^2 + u^2) / 2
        m[r] = CPLX ? __builtin_amdgcn_sqrt(0.5 * fma(v[r], v[r], u[r] * u[r])) : fabs(v[r]);
        cs += m[r];
      }
      cs += __shfl_xor(cs, 16, 64);
      cs += __shfl_xor(cs, 32, 64);
      if (l < 16) Q[I * DE + 16 * J + l] = cs;
      if (I != J) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          m[r] = row_sum16(m[r]);
          if ((l & 15) == 0) Q[J * DE + 16 * I + 4 * r + (l >> 4)] = m[r];
        }
      }
      wg_store<DE>(P2, I, J, l, v, u);
    });
    double rmax = 0.0;
    for (int i = tid; i < DE; i += nth) {
      double a = 0.0;
      for (int b = 0; b < NB16; ++b) a += Q[b * DE + i];
      rmax = fmax(rmax, a);
    }
    int n32 = 0;   // squarings in FP32, see below
    if constexpr (kF32) {
      int e;
      const double x = xn * (1.0 / EP::kappa), m = frexp(x, &e);   // x = m 2^e, 0.5 <= m < 1
      if (m == 0.5) --e;                                           // the least e with x <= 2^e
      n32 = x > 8.0 && x <= 0x1p199 ? e - 3 : 0;                   // (a NaN norm: none)
    }
    n32 = __builtin_amdgcn_readfirstlane(n32);
    // (at least one double squaring before the float ones)
    const int s = max(__builtin_amdgcn_readfirstlane(expm_squarings<T>(sqrt(block_max(rmax, red)) * (1.0 / EP::kappa))),
                      n32 > 0 ? n32 + 1 : 0);
    const int n64 = s - n32;
    float* fa = reinterpret_cast<float*>(P2);
    float* fb = reinterpret_cast<float*>(P3);
    const double f1 = ldexp(1.0, -s), f2 = ldexp(1.0, -2 * s);
    // ---- E0 = p(X / kappa) (see ExpPoly): P3 = X P2, M = b(X) ----
    // (offsets of register r: o of (i, j), ot of (j, i))
    const auto off = [&](int I, int J, int r) { return (16 * I + 4 * r + (l >> 4)) * DE + 16 * J + (l & 15); };
    const auto offt = [&](int I, int J, int r) { return (16 * J + (l & 15)) * DE + 16 * I + 4 * r + (l >> 4); };
    wg_product<CPLX, DE, false>(X, P2, stage0, stage1, tid, [&](int I, int J, mfma_f64x4 av, mfma_f64x4 au) {
      double v[4], u[4], wv[4], wu[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = off(I, J, r);
        v[r] = f1 * f2 * av[r];
        wv[r] = fma(EP::b2 * f2, P2[o], fma(EP::b1 * f1, X[o], v[r]));
        u[r] = v[r];
        wu[r] = wv[r];
        if constexpr (CPLX) {
          const int ot = offt(I, J, r);
          u[r] = f1 * f2 * au[r];
          wu[r] = fma(EP::b2 * f2, P2[ot], fma(EP::b1 * f1, X[ot], u[r]));
        }
      }
      wg_store<DE>(P3, I, J, l, v, u);
      wg_store<DE>(M, I, J, l, wv, wu);
    });
    // Q = a6, and a6 + s3 y3 + s2 y2 + s1 y + s0 over P3 (off the diagonal blocks each element is read
    // only by the thread that replaces it; within a diagonal block the whole wave reads first)
    wg_product<CPLX, DE, true>(M, M, stage0, stage1, tid, [&](int I, int J, mfma_f64x4 av, mfma_f64x4 au) {
      double v[4], u[4], wv[4], wu[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = off(I, J, r);
        const double x1 = f1 * X[o], x2 = f2 * P2[o], x3 = P3[o];
        v[r] = fma(EP::r3, x3, fma(EP::r2, x2, fma(EP::r1, x1, av[r])));
        wv[r] = fma(EP::s3, x3, fma(EP::s2, x2, fma(EP::s1, x1, v[r])));
        u[r] = v[r];
        wu[r] = wv[r];
        if constexpr (CPLX) {
          if (I != J) {
            const int ot = offt(I, J, r);
            const double y1 = f1 * X[ot], y2 = f2 * P2[ot], y3 = P3[ot];
            u[r] = fma(EP::r3, y3, fma(EP::r2, y2, fma(EP::r1, y1, au[r])));
            wu[r] = fma(EP::s3, y3, fma(EP::s2, y2, fma(EP::s1, y1, u[r])));
          }
        }
        if (I == J && 4 * r + (l >> 4) == (l & 15)) wv[r] += EP::s0;
      }
      wg_store<DE>(Q, I, J, l, v, u);
      wg_store<DE>(P3, I, J, l, wv, wu);
    });
    // Float messages: the last n32 squarings in FP32, a relative rounding error e in the first of them
    // acting on X = beta (theta - mu) like 2^n32 e: 2^n32 stays below ||X|| / 4, ||X|| the smaller of X's
    // 1- and Frobenius norms, so that this stays near what the float rounding of the messages already
    // puts on X.  They work on two float planes in the slabs of X^2 and X^3, which the polynomial no
    // longer needs by then; the double squaring before them writes these.  The last product of all
    // writes planes too.
    double trp = 0.0;   // this thread's share of the trace
    wg_product<CPLX, DE, false>(P3, Q, stage0, stage1, tid, [&](int I, int J, mfma_f64x4 av, mfma_f64x4 au) {
      double v[4], u[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = off(I, J, r);
        v[r] = fma(EP::t2 * f2, P2[o], fma(EP::t1 * f1, X[o], av[r]));
        u[r] = v[r];
        if constexpr (CPLX) {
          const int ot = offt(I, J, r);
          u[r] = fma(EP::t2 * f2, P2[ot], fma(EP::t1 * f1, X[ot], au[r]));
        }
        if (I == J && 4 * r + (l >> 4) == (l & 15)) {
          v[r] += 1.0;
          u[r] += 1.0;
          trp += v[r];
        }
      }
      if (s == 0) wg_store_planes<CPLX, double, DE>(M, I, J, l, v, u);
      else wg_store<DE>(M, I, J, l, v, u);
    });
    // ---- normalise and square: Z_{j+1} = Z_j^2 / (Tr Z_j)^2 ----
    double t = block_sum(trp, red);
    double L = log(t);
    for (int j = 0; j < n64; ++j) {
      const double scale = 1.0 / (t * t);
      const bool last32 = kF32 && j + 1 == n64 && n64 < s;
      trp = 0.0;
      wg_product<CPLX, DE, true>(M, M, stage0, stage1, tid, [&](int I, int J, mfma_f64x4 av, mfma_f64x4 au) {
        double v[4], u[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = scale * av[r];
          u[r] = scale * au[r];
          if (I == J && 4 * r + (l >> 4) == (l & 15)) trp += v[r];
        }
        if (last32) wg_store_planes<CPLX, float, DE, true>(fa, I, J, l, v, u);
        else if (j + 1 == s) wg_store_planes<CPLX, double, DE>(Q, I, J, l, v, u);
        else wg_store<DE>(Q, I, J, l, v, u);
      });
      double* tp = M;
      M = Q;
      Q = tp;
      t = block_sum(trp, red);
      L = fma(2.0, L, log(t));
    }
    if constexpr (kF32) {
      for (int j = n64; j < s; ++j) {
        const float scale = (float)(1.0 / (t * t));
        trp = 0.0;
        wg_square32<CPLX, DE>(fa, stage0, stage1, tid, [&](int I, int J, mfma_f32x4 ar, mfma_f32x4 ai) {
          // (the blocks of a 2 x 2 tile on the diagonal stand as computed, the others are mirrored)
          const bool mirror = I < J && !(DE == 256 && I / 2 == J / 2);
          const int jj = 16 * J + (l & 15);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = 16 * I + 4 * (l >> 4) + r;
            const float vr = scale * ar[r];
            if (i == jj) trp += (double)vr;
            fb[i * DE + jj] = vr;
            if (mirror) fb[jj * DE + i] = vr;
            if constexpr (CPLX) {
              const float vi = i == jj ? 0.f : scale * ai[r];
              fb[DD + i * DE + jj] = vi;
              if (mirror) fb[DD + jj * DE + i] = -vi;
            }
          }
        });
        float* tp = fa;
        fa = fb;
        fb = tp;
        t = block_sum(trp, red);
        L = fma(2.0, L, log(t));
      }
    }
    const double F = mu - L / beta;
    const int32_t gid = A.gid[c];
    if (tid == 0) {
      if (A.scal) A.scal[gid] = F;
      if (!isfinite(F) && A.nonfinite) atomicAdd(A.nonfinite, 1ull);
    }
    // ---- a5: outputs of rho = Z_s / Tr Z_s ----
    if (kF32 && n64 < s) wg_outputs<T, float, CPLX, DE>(A, c, gid, fa, 1.0 / t, tid, nth);
    else wg_outputs<T, double, CPLX, DE>(A, c, gid, M, 1.0 / t, tid, nth);
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------
// certified lambda_min for De >= 64 without eigenvectors (a8)
// ------------------------------------------------------------------------------------------
//
// theta_e (FP64, in a per-workgroup slab) is reduced to a Hermitian tridiagonal matrix by De - 2
// Householder reflections H = I - tau v v^H acting on the trailing block (A <- H A H with the
// rank-2 form A - v w^H - w v^H, w = p - (tau/2)(v^H p) v, p = tau A v).  A diagonal unitary
// makes the off-diagonal real and non-negative, so the eigenvalues are those of the real
// symmetric tridiagonal (d, |e|).  lambda_min is then bracketed by multisection on Sturm counts
// (number of eigenvalues below x from the signs of the LDL^T pivots), 256 points per round;
// the lower end of the final bracket, below which no eigenvalue lies, is returned.
//
// Every tridiagonalisation here works on theta_e / 2^e, e the binary exponent of its largest component
// (unit_exponent), and takes the bracket and the margin back by 2^e: powers of two are exact, no
// square of an entry overflows, and a square that underflows belongs to an entry below 1e-140, where the
// margin 8 De eps ||theta_e||_F is above 1e-14.

// e with 2^(e-1) <= amax < 2^e; 0 for a matrix that is zero or holds an infinity (NaN entries are not
// in the maximum: they show in the norm)
__device__ __forceinline__ int unit_exponent(double amax) {
  int e = 0;
  if (amax > 0.0 && amax <= DBL_MAX) (void)frexp(amax, &e);
  return e;
}

// Norm xn of a column x, |x_0| and tau = 2 / ||v||^2, v = x + (x_0 / |x_0|) ||x|| e_1, of a matrix scaled as
// above.  A square below 1e-280 may have lost its digits (x_0 |x_0|^-1 would have another modulus than 1,
// and the reflection not be one): such an x_0 counts as zero.  A column of norm below 1e-120 is not
// reflected (tau = 0).  Either changes theta_e by less than 1e-118 of its largest entry.  (tau = 0
// too where a NaN or infinity reached the column.)
__device__ __forceinline__ void householder_scalars(double xn2, double x0r, double x0i, double& xn, double& a0,
                                                    double& tau) {
  const double a2 = fma(x0r, x0r, x0i * x0i);
  xn = sqrt(xn2);
  a0 = a2 > 1e-280 ? sqrt(a2) : 0.0;
  const double vn2 = 2.0 * (xn2 + a0 * xn);
  tau = xn2 > 1e-240 ? 2.0 / vn2 : 0.0;
}

// Value and margin of a cluster from the scaled bracket's lower end and the scaled squared norm.  Scaled
// finite entries keep every quantity of the reduction finite, so the norm tells whether all were.
__device__ __forceinline__ void store_tridiag_bound(const ClusterArgs<double>& A, int32_t gid, int De, double lo,
                                                    double nrm2, int e) {
  const double v = isfinite(nrm2) ? ldexp(lo, e) : nrm2 - nrm2;   // NaN: a bracket of some rows is no bound
  A.scal[gid] = v;
  A.scal2[gid] = ldexp(8.0 * De * DBL_EPSILON * sqrt(nrm2), e);
  if (!isfinite(v) && A.nonfinite) atomicAdd(A.nonfinite, 1ull);
}

// theta_e is in the slab, each element written by the thread that scales it here.
template <bool CPLX, int DE>
__device__ void tridiag_lambda_min(const ClusterArgs<double>& A, int64_t c, double* ar, double* ai) {
  __shared__ double vr[DE], vi[DE], pr[DE], pi[DE];
  __shared__ double qvr[DE], qvi[DE], qwr[DE], qwi[DE];
  __shared__ double dg[DE], e2[DE];
  __shared__ double red[16];
  const int tid = threadIdx.x, nth = blockDim.x;
  double amax = 0.0, n2 = 0.0;
  for (int idx = tid; idx < DE * DE; idx += nth) {
    amax = fmax(amax, fabs(ar[idx]));
    if constexpr (CPLX) amax = fmax(amax, fabs(ai[idx]));
  }
  const int ex = unit_exponent(block_max(amax, red));
  for (int idx = tid; idx < DE * DE; idx += nth) {
    const double xr = ldexp(ar[idx], -ex);
    ar[idx] = xr;
    n2 = fma(xr, xr, n2);
    if constexpr (CPLX) {
      const double xi = ldexp(ai[idx], -ex);
      ai[idx] = xi;
      n2 = fma(xi, xi, n2);
    }
  }
  const double nrm2 = block_sum(n2, red);
  {
    // The rank-2 update of each reflection is applied during the next reflection's sweep over
    // the trailing matrix (pending vectors qv, qw): every trailing element is read and written
    // once per reflection instead of read twice and written once.  Row k and the final 2 x 2
    // block are corrected on the fly.
    for (int i = tid; i < DE; i += nth) {
      qvr[i] = 0.0;
      qvi[i] = 0.0;
      qwr[i] = 0.0;
      qwi[i] = 0.0;
    }
    __syncthreads();
    // pending correction of element (r, cc): v_r conj(w_cc) + w_r conj(v_cc)
    auto pend = [&](int r, int cc, double& ur, double& ui) {
      ur = fma(qvr[r], qwr[cc], fma(qvi[r], qwi[cc], fma(qwr[r], qvr[cc], qwi[r] * qvi[cc])));
      ui = fma(qvi[r], qwr[cc], fma(-qvr[r], qwi[cc], fma(qwi[r], qvr[cc], -qwr[r] * qvi[cc])));
    };
    for (int k = 0; k < DE - 2; ++k) {
      const int m = DE - k - 1;
      const int64_t rk = (int64_t)k * DE + k + 1;   // x_i = A[k+1+i][k] = conj(A[k][k+1+i])
      double xs = 0.0;
      for (int i = tid; i < m; i += nth) {
        double ur, ui;
        pend(k, k + 1 + i, ur, ui);
        const double xr = ar[rk + i] - ur;
        const double xim = CPLX ? ai[rk + i] - ui : 0.0;
        vr[i] = xr;     // x, turned into v below
        vi[i] = -xim;
        xs = fma(xr, xr, xs);
        if constexpr (CPLX) xs = fma(xim, xim, xs);
      }
      const double xn2 = block_sum(xs, red);
      const double x0r = vr[0], x0i = vi[0];
      double xn, a0, tau;
      householder_scalars(xn2, x0r, x0i, xn, a0, tau);
      if (tid == 0) {
        double ur, ui;
        pend(k, k, ur, ui);
        dg[k] = ar[(int64_t)k * DE + k] - ur;
        e2[k] = xn2;
      }
      // an already reduced column (block-uniform) reflects nothing (v = 0) but still flushes the
      // pending update into the trailing matrix
      const bool act = tau > 0.0;
      const double ur0 = a0 > 0.0 ? x0r / a0 : 1.0, ui0 = a0 > 0.0 ? x0i / a0 : 0.0;
      __syncthreads();
      if (act) {
        if (tid == 0) {   // v = x - alpha e1, alpha = -(x0/|x0|) ||x||
          vr[0] = fma(ur0, xn, x0r);
          vi[0] = fma(ui0, xn, x0i);
        }
      } else {
        for (int i = tid; i < m; i += nth) {
          vr[i] = 0.0;
          vi[i] = 0.0;
        }
      }
      __syncthreads();
      // p = tau A22 v on the updated A22, written back as it is read; A22 is Hermitian, so row i
      // of A22 v reads column i (coalesced across i)
      for (int i = tid; i < m; i += nth) {
        const int cc = k + 1 + i;
        const double wcr = qwr[cc], wci = qwi[cc], vcr = qvr[cc], vci = qvi[cc];
        double* col_r = ar + (int64_t)(k + 1) * DE + cc;
        double* col_i = CPLX ? ai + (int64_t)(k + 1) * DE + cc : nullptr;
        double sr = 0.0, si = 0.0;
#pragma unroll 4
        for (int j = 0; j < m; ++j) {
          const int r = k + 1 + j;
          const double a_r = col_r[(int64_t)j * DE] -
                             fma(qvr[r], wcr, fma(qvi[r], wci, fma(qwr[r], vcr, qwi[r] * vci)));
          col_r[(int64_t)j * DE] = a_r;
          sr = fma(a_r, vr[j], sr);
          if constexpr (CPLX) {
            const double b_i = col_i[(int64_t)j * DE] -
                               fma(qvi[r], wcr, fma(-qvr[r], wci, fma(qwi[r], vcr, -qwr[r] * vci)));
            col_i[(int64_t)j * DE] = b_i;
            const double a_i = -b_i;   // Im A[cc][r]
            sr = fma(-a_i, vi[j], sr);
            si = fma(a_r, vi[j], fma(a_i, vr[j], si));
          }
        }
        pr[i] = tau * sr;
        pi[i] = tau * si;
      }
      __syncthreads();
      double ks = 0.0;
      for (int i = tid; i < m; i += nth) ks = fma(vr[i], pr[i], fma(vi[i], pi[i], ks));
      const double K = 0.5 * tau * block_sum(ks, red);
      // the update of this reflection, A22 -= v w^H + w v^H with w = p - K v, becomes pending
      for (int i = tid; i < m; i += nth) {
        qvr[k + 1 + i] = vr[i];
        qvi[k + 1 + i] = vi[i];
        qwr[k + 1 + i] = fma(-K, vr[i], pr[i]);
        qwi[k + 1 + i] = fma(-K, vi[i], pi[i]);
      }
      __syncthreads();
    }
    if (tid == 0) {
      double ur, ui;
      pend(DE - 2, DE - 2, ur, ui);
      dg[DE - 2] = ar[(int64_t)(DE - 2) * DE + DE - 2] - ur;
      pend(DE - 1, DE - 1, ur, ui);
      dg[DE - 1] = ar[(int64_t)(DE - 1) * DE + DE - 1] - ur;
      pend(DE - 2, DE - 1, ur, ui);
      const double xr = ar[(int64_t)(DE - 2) * DE + DE - 1] - ur;
      const double xi = CPLX ? ai[(int64_t)(DE - 2) * DE + DE - 1] - ui : 0.0;
      e2[DE - 2] = fma(xr, xr, xi * xi);
      e2[DE - 1] = 0.0;
    }
    __syncthreads();
    // Gershgorin bracket (every thread, same order: identical values)
    double lo = INFINITY, hi = -INFINITY, emax = 0.0;
    for (int i = 0; i < DE; ++i) {
      const double r = (i > 0 ? sqrt(e2[i - 1]) : 0.0) + sqrt(e2[i]);
      lo = fmin(lo, dg[i] - r);
      hi = fmax(hi, dg[i] + r);
      emax = fmax(emax, e2[i]);
    }
    const double pivmin = DBL_MIN * fmax(1.0, emax);
    const double span0 = fmax(hi - lo, DBL_MIN);
    lo -= 2.0 * DBL_EPSILON * fabs(lo) + span0 * DBL_EPSILON;
    hi += 2.0 * DBL_EPSILON * fabs(hi) + span0 * DBL_EPSILON;
    for (int round = 0; round < 12; ++round) {
      if (hi - lo <= 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi))) break;   // a few ulps of lambda_min
      const double x = lo + (hi - lo) * (double)(tid + 1) / (double)(nth + 1);
      int cnt = 0;
      double q = dg[0] - x;
      if (fabs(q) < pivmin) q = -pivmin;
      cnt += q < 0.0;
      for (int i = 1; i < DE; ++i) {
        q = (dg[i] - x) - e2[i - 1] / q;
        if (fabs(q) < pivmin) q = -pivmin;
        cnt += q < 0.0;
      }
      const double first = block_min(cnt > 0 ? (double)tid : (double)nth, red);
      const int t = (int)first;
      const double nlo = t == 0 ? lo : lo + (hi - lo) * (double)t / (double)(nth + 1);
      const double nhi = t == nth ? hi : lo + (hi - lo) * (double)(t + 1) / (double)(nth + 1);
      if (!(nhi - nlo < hi - lo)) break;
      lo = nlo;
      hi = nhi;
    }
    if (tid == 0) store_tridiag_bound(A, A.gid[c], DE, lo, nrm2, ex);
    __syncthreads();
  }
}

template <bool CPLX, int DE>
__global__ __launch_bounds__(256) void k_cluster_tridiag(ClusterArgs<double> A, double* scratch, int64_t slab) {
  constexpr int64_t DD = (int64_t)DE * DE;
  const int tid = threadIdx.x, nth = blockDim.x;
  double* ar = scratch + (int64_t)blockIdx.x * slab;
  double* ai = CPLX ? ar + DD : nullptr;
  for (int64_t c = blockIdx.x; c < A.n; c += gridDim.x) {
    big_assemble<double, double, CPLX, false>(A, c, DE, ar, ai, (double*)nullptr, (double*)nullptr, 0.0, tid, nth);
    tridiag_lambda_min<CPLX, DE>(A, c, ar, ai);
  }
}

// Certification at De = 64, 128 with the matrix in registers: DE / 16 waves, wave g holding rows
// j = G e + g (e = 0 .. 15, G = DE / 16), lane l of it columns l + 64 q, so every wave keeps work as the
// trailing block shrinks and the elements of a vector at a row are one LDS broadcast per wave.  The
// reflections of tridiag_lambda_min with the rank-2 update applied at once; three barriers each: the
// row to LDS, the partial products of A v (every wave forms the norm by itself), then w = p - K v by
// the first wave.  Its bracketing too, 4 DE points a round.
// In the slab, one column per thread read and written per reflection, the 1018 128 x 128 clusters of a
// 1024-site chain took 5.0 ms, bound by the latency of its memory traffic, the 64 x 64 ones 1.0 ms; here
// 2.4 and 0.41 ms, three fifths of it the reflections (3 us each at 128, the chain between the barriers).
template <bool CPLX, int DE>
__global__ __launch_bounds__(DE * 4) void k_certify_tridiag(ClusterArgs<double> A) {
  constexpr int G = DE / 16, NE = 16, NC = DE / 64, NI = CPLX ? NE : 1;
  static_assert(DE % 64 == 0, "columns l + 64 q");
  __shared__ double2 sx[2][DE], sw[DE], part[G][DE];
  __shared__ double dg[DE], e2[DE];
  __shared__ double red[16];
  const int tid = threadIdx.x, l = tid % 64;
  const int g = __builtin_amdgcn_readfirstlane(tid / 64);
  const int64_t c = xcd_cluster(blockIdx.x, A.n);
  const int64_t ho = A.hoff[c];
  double ar[NC][NE], ai[NC][NI], amax = 0.0, my = 0.0;
#pragma unroll 4   // in full it is 8000 instructions
  for (int e = 0; e < NE; ++e)
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      double vr, vi;
      theta_elem<double, CPLX>(A, c, DE, log2i(DE), ho, G * e + g, l + 64 * q, 0.0, vr, vi);
      amax = fmax(amax, fabs(vr));
      if constexpr (CPLX) amax = fmax(amax, fabs(vi));
#pragma unroll
      for (int f = 0; f < NE; ++f)
        if (f == e) {
          ar[q][f] = vr;
          if constexpr (CPLX) ai[q][f] = vi;
        }
    }
  const int ex = __builtin_amdgcn_readfirstlane(unit_exponent(block_max(amax, red)));
#pragma unroll
  for (int e = 0; e < NE; ++e)
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      ar[q][e] = ldexp(ar[q][e], -ex);
      my = fma(ar[q][e], ar[q][e], my);
      if constexpr (CPLX) {
        ai[q][e] = ldexp(ai[q][e], -ex);
        my = fma(ai[q][e], ai[q][e], my);
      }
    }
  const double nrm2 = block_sum(my, red);
  for (int k = 0; k < DE - 2; ++k) {
    double2* x = sx[k & 1];
    // x_j = A[j][k] = conj(A[k][j]), j > k
    if (k % G == g) {
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const int i = l + 64 * q;
        double rr = 0.0, ri = 0.0;
#pragma unroll
        for (int e = 0; e < NE; ++e)
          if (e == k / G) {
            rr = ar[q][e];
            if constexpr (CPLX) ri = ai[q][e];
          }
        x[i] = i > k ? double2{rr, -ri} : double2{0.0, 0.0};
        if (i == k) dg[k] = rr;
      }
    }
    __syncthreads();
    double2 xi[NC];
    double xs = 0.0;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      xi[q] = x[l + 64 * q];
      xs = fma(xi[q].x, xi[q].x, fma(xi[q].y, xi[q].y, xs));
    }
    const double xn2 = wave_sum_dpp(xs);
    const double2 x0 = x[k + 1];
    double xn, a0, tau;
    householder_scalars(xn2, x0.x, x0.y, xn, a0, tau);
    // v = x - alpha e1, alpha = -(x0/|x0|) ||x||; x = 0: nothing to reflect
    const double ia = a0 > 0.0 ? xn / a0 : 0.0;
    const double2 v0 = a0 > 0.0 ? double2{fma(x0.x, ia, x0.x), fma(x0.y, ia, x0.y)} : double2{xn, 0.0};
    if (tid == 0) e2[k] = xn2;
    // (A v)_i = sum_j conj(A[j][i]) v_j over this wave's rows
    double sr[NC], si[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) sr[q] = si[q] = 0.0;
#pragma unroll
    for (int e0 = 0; e0 < NE; e0 += 4) {   // four LDS reads in flight to a branch
      if (G * (e0 + 4) - 1 <= k) continue;   // rows done with (their v_j is zero)
      double2 v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = x[G * (e0 + e) + g];
        if (G * (e0 + e) + g == k + 1) v[e] = v0;
      }
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        if (64 * q + 63 <= k) continue;   // columns done with
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double b = ar[q][e0 + e];
          sr[q] = fma(b, v[e].x, sr[q]);
          if constexpr (CPLX) {
            const double d = ai[q][e0 + e];
            sr[q] = fma(d, v[e].y, sr[q]);
            si[q] = fma(b, v[e].y, fma(-d, v[e].x, si[q]));
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      part[g][l + 64 * q] = double2{sr[q], si[q]};
      if (l + 64 * q == k + 1) xi[q] = v0;   // the lane's elements of v
    }
    __syncthreads();
    if (g == 0) {
      double2 pp[NC];
      double ks = 0.0;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        double pr = 0.0, pi = 0.0;
#pragma unroll
        for (int h = 0; h < G; ++h) {
          const double2 t = part[h][l + 64 * q];
          pr += t.x;
          pi += t.y;
        }
        pp[q] = l + 64 * q > k ? double2{tau * pr, tau * pi} : double2{0.0, 0.0};
        ks = fma(xi[q].x, pp[q].x, fma(xi[q].y, pp[q].y, ks));
      }
      const double K = 0.5 * tau * wave_sum_dpp(ks);
#pragma unroll
      for (int q = 0; q < NC; ++q) sw[l + 64 * q] = double2{fma(-K, xi[q].x, pp[q].x), fma(-K, xi[q].y, pp[q].y)};
      if (l == 0) x[k + 1] = v0;
    }
    __syncthreads();
    // A22 -= v w^H + w v^H
    double2 wi[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) wi[q] = sw[l + 64 * q];
#pragma unroll
    for (int e0 = 0; e0 < NE; e0 += 4) {
      if (G * (e0 + 4) - 1 <= k) continue;
      double2 v[4], w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = x[G * (e0 + e) + g];
        w[e] = sw[G * (e0 + e) + g];
      }
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        if (64 * q + 63 <= k) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (CPLX) {
            ar[q][e0 + e] -=
                fma(v[e].x, wi[q].x, fma(v[e].y, wi[q].y, fma(w[e].x, xi[q].x, w[e].y * xi[q].y)));
            ai[q][e0 + e] -=
                fma(v[e].y, wi[q].x, fma(-v[e].x, wi[q].y, fma(w[e].y, xi[q].x, -w[e].x * xi[q].y)));
          } else {
            ar[q][e0 + e] -= fma(v[e].x, wi[q].x, w[e].x * xi[q].x);
          }
        }
      }
    }
  }
  {   // the last 2 x 2 block: rows DE - 2 and DE - 1 are the last register of waves G - 2 and G - 1
    const double zr = ar[NC - 1][NE - 1], zi = CPLX ? ai[NC - 1][NI - 1] : 0.0;
    if (g == G - 2 && l == 62) dg[DE - 2] = zr;
    if (g == G - 2 && l == 63) e2[DE - 2] = fma(zr, zr, zi * zi);
    if (g == G - 1 && l == 63) {
      dg[DE - 1] = zr;
      e2[DE - 1] = 0.0;
    }
  }
  __syncthreads();
  // Gershgorin bracket
  double lo = INFINITY, hi = -INFINITY, emax = 0.0;
  if (tid < DE) {
    const double b = (tid > 0 ? sqrt(e2[tid - 1]) : 0.0) + sqrt(e2[tid]);
    lo = dg[tid] - b;
    hi = dg[tid] + b;
    emax = e2[tid];
  }
  lo = block_min(lo, red);
  hi = block_max(hi, red);
  emax = block_max(emax, red);
  const double pivmin = DBL_MIN * fmax(1.0, emax);
  const double span0 = fmax(hi - lo, DBL_MIN);
  lo -= 2.0 * DBL_EPSILON * fabs(lo) + span0 * DBL_EPSILON;
  hi += 2.0 * DBL_EPSILON * fabs(hi) + span0 * DBL_EPSILON;
  constexpr int NP = DE * 4;
  for (int round = 0; round < 12; ++round) {
    if (hi - lo <= 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi))) break;   // a few ulps of lambda_min
    const double y = lo + (hi - lo) * (double)(tid + 1) / (double)(NP + 1);
    int cnt = 0;
    double q = dg[0] - y;
    if (fabs(q) < pivmin) q = -pivmin;
    cnt += q < 0.0;
#pragma unroll 4
    for (int r = 1; r < DE; ++r) {
      // the reciprocal to an ulp or two: a relative change of e2, as a rounding of the quotient is
      q = fmin(fmax(fma(-e2[r - 1], rcp_nr(q), dg[r] - y), -1e300), 1e300);
      if (fabs(q) < pivmin) q = -pivmin;
      cnt += q < 0.0;
    }
    const int t = (int)block_min(cnt > 0 ? (double)tid : (double)NP, red);
    const double nlo = t == 0 ? lo : lo + (hi - lo) * (double)t / (double)(NP + 1);
    const double nhi = t == NP ? hi : lo + (hi - lo) * (double)(t + 1) / (double)(NP + 1);
    if (!(nhi - nlo < hi - lo)) break;
    lo = nlo;
    hi = nhi;
  }
  if (tid == 0) store_tridiag_bound(A, A.gid[c], DE, lo, nrm2, ex);
}

// ------------------------------------------------------------------------------------------
// lambda_min-only certification, De = 64, 128, 256 (one workgroup of 256 threads per cluster)
// ------------------------------------------------------------------------------------------
//
// Q_C needs lambda_min of every theta_e and nothing else (Sec. 4.2).  Lanczos from a seeded
// start vector builds the tridiagonal T_k of theta_e on the Krylov space; its smallest
// eigenvalue rho is, by interlacing, at least lambda_min and converges to it, typically long
// before k = De.  rho is certified from below by one Cholesky factorisation of
// S = theta_e - sigma I at sigma = rho - eta.  If the factorisation runs to completion in
// floating point, the computed factor R satisfies R^H R = S + dS with |dS| <= g |R^H| |R|
// (backward error of Cholesky: g = gamma_{De+1} for real and sqrt(2) gamma_{2De+4} for complex
// arithmetic), so R^H R is positive semidefinite and
//     lambda_min(theta_e) >= sigma - g || |R| ||_2^2 - u max_i |theta_ii - sigma|
//                         >= sigma - g || |R| ||_1 || |R| ||_inf - u max_i |theta_ii - sigma|,
// the last term for the rounding of the shift.  The bound returned is that right-hand side less
// a term for the rounding of the assembly of theta_e; it is handed over as lambda = rho and
// margin = rho - bound.  If a pivot is not positive (rho not yet converged, or the start vector
// blind to the lowest eigenvector), the cluster is certified by the tridiagonalisation path
// instead (counted in the fallback counter).
//
// Memory: theta_e (full, row-major) in the workgroup's slab; Lanczos vectors, T_k and one
// column-major panel of NB columns of the factor in LDS.  A matrix-vector product reads the
// slab once (column t of the Hermitian theta_e gives row t of theta_e q, coalesced across t);
// the right-looking blocked factorisation reads and writes the trailing lower triangle once per
// panel.
// At 256 dimensions (the 1017 clusters of a 1024-site chain, 56 to 72 Lanczos steps) the time goes to the
// products, bound by what the caches deliver (13.5 us each, 4 MiB of L2 serving 32 matrices), then the
// factorisation, and the barriers of both: 12.5 ms with every row in the slab, three barriers to a
// panel column and to a sum, and divisions on 1024 points in ritz_min; 10.0 ms with rows in LDS, one
// barrier each, and reciprocals on 256 points; 9.1 ms with the trailing update on the matrix cores.

// Smallest eigenvalue of the symmetric tridiagonal (al[0..k-1], off-diagonal be[0..k-2]) by
// multisection on Sturm counts from the bracket [Gershgorin lower end, min_i al_i]; the midpoint of
// the final bracket.  One wave per SIMD counts: the chain of reciprocals is latency, and with 1024
// points a round the instructions of four waves, divisions then, came one after another (67 us a call
// at about 50 steps).
__device__ double ritz_min(const double* al, const double* be, int k, double* red) {
  const int tid = threadIdx.x;
  constexpr int nth = 256;   // counting threads, of at least as many in the workgroup
  double lo = INFINITY, hi = INFINITY, emax = 0.0;
  for (int i = 0; i < k; ++i) {   // every thread, same order: identical values
    const double bl = i > 0 ? be[i - 1] : 0.0, br = i + 1 < k ? be[i] : 0.0;
    lo = fmin(lo, al[i] - fabs(bl) - fabs(br));
    hi = fmin(hi, al[i]);
    emax = fmax(emax, br * br);
  }
  const double pivmin = DBL_MIN * fmax(1.0, emax);
  for (int round = 0; round < 12; ++round) {
    if (hi - lo <= 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi))) break;
    int cnt = 0;
    if (tid < nth) {
      const double x = lo + (hi - lo) * (double)(tid + 1) / (double)(nth + 1);
      double q = al[0] - x;
      if (fabs(q) < pivmin) q = -pivmin;
      cnt += q < 0.0;
#pragma unroll 4
      for (int i = 1; i < k; ++i) {
        q = fmin(fmax(fma(-be[i - 1] * be[i - 1], rcp_nr(q), al[i] - x), -1e300), 1e300);
        if (fabs(q) < pivmin) q = -pivmin;
        cnt += q < 0.0;
      }
    }
    const int t = (int)block_min(cnt > 0 ? (double)tid : (double)nth, red);
    const double nlo = t == 0 ? lo : lo + (hi - lo) * (double)t / (double)(nth + 1);
    const double nhi = t == nth ? hi : lo + (hi - lo) * (double)(t + 1) / (double)(nth + 1);
    if (!(nhi - nlo < hi - lo)) break;
    lo = nlo;
    hi = nhi;
  }
  return 0.5 * (lo + hi);
}

__device__ __forceinline__ uint32_t mix32(uint32_t x) {   // a 32-bit integer finaliser
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

template <bool CPLX, int DE>
__global__ __launch_bounds__(1024) void k_certify_lanczos(ClusterArgs<double> A, double* scratch, int64_t slab) {
  constexpr int64_t DD = (int64_t)DE * DE;
  constexpr int NT = 1024;
  constexpr int NW = NT / 64;
  constexpr int H = DE / 2;                  // shift-diagonals 0 .. H of the half storage
  constexpr int G = NT / DE;                 // threads per row in the matrix-vector product
  constexpr int KMAX = DE < 192 ? DE : 192;  // Lanczos steps at most
  constexpr int NB = 16;                     // Cholesky panel width (one wave per panel column)
  __shared__ double qr[DE], qi[CPLX ? DE : 1];
  __shared__ double yr[G][DE], yi[CPLX ? G : 1][CPLX ? DE : 1];
  __shared__ double al[KMAX], be[KMAX];
  // rows sh < NL of the half storage live in LDS, under the panel that is used after them: 28 of the
  // 129 complex rows.  (As many again in registers spill more than they save; so do more than four
  // slab loads in flight to a thread.)
  constexpr int NC = CPLX ? 2 : 1;
  constexpr int NL = DE == 256 ? 56 / NC : 0;
  static_assert(NL % G == 0 && NL <= H, "whole groups of rows, the last one in the slab");
  __shared__ double lds[(NL > NB ? NL : NB) * DE * NC];
  double(*Pr)[DE] = (double(*)[DE])lds, (*Pi)[DE] = (double(*)[DE])(lds + (NC - 1) * NB * DE);
  __shared__ double rsum[DE];
  __shared__ double csum[NB];
  __shared__ double red[NW], rsa[NW], rsb[NW];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const int t = tid % DE, g = tid / DE;
  const double u = 0.5 * DBL_EPSILON;
  const int NBITS = log2i(DE);
  double* ar = scratch + (int64_t)blockIdx.x * slab;
  double* ai = CPLX ? ar + DD : nullptr;
  // half storage for the Lanczos products: B[s][t] = theta[(t + s) mod De][t], s = 0 .. De/2
  double* br = ar;
  double* bi = CPLX ? ar + (int64_t)(H + 1) * DE : nullptr;
  for (int64_t c = blockIdx.x; c < A.n; c += gridDim.x) {
    const int32_t gid = A.gid[c];
    const int64_t ho = A.hoff[c];
    double my = 0.0;
    for (int idx = tid; idx < (H + 1) * DE; idx += NT) {
      const int sh = idx / DE, tt = idx % DE;
      double vr_, vi_;
      theta_elem<double, CPLX>(A, c, DE, NBITS, ho, (tt + sh) & (DE - 1), tt, 0.0, vr_, vi_);
      if (sh < NL) {
        lds[sh * NC * DE + tt] = vr_;
        if constexpr (CPLX) lds[(sh * NC + 1) * DE + tt] = vi_;
      } else {
        br[idx] = vr_;
        if constexpr (CPLX) bi[idx] = vi_;
      }
      // every off-diagonal pair once, except on the last shift-diagonal (twice there)
      const double w = (sh == 0 || sh == H) ? 1.0 : 2.0;
      my = fma(w * vr_, vr_, my);
      if constexpr (CPLX) my = fma(w * vi_, vi_, my);
    }
    const double nf = sqrt(block_sum(my, red));
    // ---- Lanczos ----
    my = 0.0;
    if (tid < DE) {
      const uint32_t h0 = mix32((uint32_t)gid * 0x9e3779b9u ^ mix32(2u * (uint32_t)tid + 1u));
      qr[tid] = (double)h0 * 0x1p-32 - 0.5;
      my = qr[tid] * qr[tid];
      if constexpr (CPLX) {
        qi[tid] = (double)mix32(h0 + 0x632be5abu) * 0x1p-32 - 0.5;
        my = fma(qi[tid], qi[tid], my);
      }
    }
    const double q0 = 1.0 / sqrt(block_sum(my, red));
    if (tid < DE) {
      qr[tid] *= q0;
      if constexpr (CPLX) qi[tid] *= q0;
    }
    double ppr = 0.0, ppi = 0.0, bprev = 0.0;   // q_{k-1} (thread tid < De) and beta_{k-1}
    double rho = INFINITY, rho_old = INFINITY, dlast = INFINITY;
    __syncthreads();
    for (int k = 0; k < KMAX; ++k) {
      {
        // (theta q)_t = sum_s conj(B[s][t]) q_{t+s} + sum_{0<s<H} B[s][t-s] q_{t-s}; both reads of
        // shift-diagonal s are coalesced across t (the second is the first rotated by s).
        // Thread (g, t) takes the shift-diagonals s = g mod G.
        double sr = 0.0, si = 0.0;
        int t1 = t;
        asm volatile("" : "+v"(t1));   // else the addresses of all rows are kept over the steps, and spill
        auto add = [&](int sh, double b_r, double b_i, double c_r, double c_i) {
          const int up = (t1 + sh) & (DE - 1), dn = (t1 - sh) & (DE - 1);
          const double xr = qr[up], yr_ = qr[dn];
          sr = fma(b_r, xr, sr);
          sr = fma(c_r, yr_, sr);
          if constexpr (CPLX) {
            const double xi = qi[up], yi_ = qi[dn];
            sr = fma(b_i, xi, sr);
            sr = fma(-c_i, yi_, sr);
            si = fma(b_r, xi, fma(-b_i, xr, si));
            si = fma(c_r, yi_, fma(c_i, yr_, si));
          }
        };
#pragma unroll 2
        for (int sh = g; sh < NL; sh += G) {
          const double* rr = lds + sh * NC * DE;
          const int dn = (t1 - sh) & (DE - 1);
          const double z = sh > 0 ? 1.0 : 0.0;   // the diagonal once
          add(sh, rr[t1], CPLX ? rr[DE + t1] : 0.0, z * rr[dn], CPLX ? z * rr[DE + dn] : 0.0);
        }
#pragma unroll 2
        for (int sh = NL + g; sh <= H; sh += G) {
          const double* rr = br + (int64_t)sh * DE;
          const int dn = (t1 - sh) & (DE - 1);
          const bool two = sh > 0 && sh < H;
          const double b_r = rr[t1];
          const double c_r = two ? rr[dn] : 0.0;
          double b_i = 0.0, c_i = 0.0;
          if constexpr (CPLX) {
            const double* ri = bi + (int64_t)sh * DE;
            b_i = ri[t1];
            c_i = two ? ri[dn] : 0.0;
          }
          add(sh, b_r, b_i, c_r, c_i);
        }
        yr[g][t] = sr;
        if constexpr (CPLX) yi[g][t] = si;
      }
      __syncthreads();
      double wr = 0.0, wi = 0.0, ma = 0.0;
      if (tid < DE) {
#pragma unroll
        for (int h = 0; h < G; ++h) {
          wr += yr[h][tid];
          if constexpr (CPLX) wi += yi[h][tid];
        }
        wr = fma(-bprev, ppr, wr);
        ma = qr[tid] * wr;
        if constexpr (CPLX) {
          wi = fma(-bprev, ppi, wi);
          ma = fma(qi[tid], wi, ma);
        }
      }
      // sums over the waves that hold the vector, one barrier each (a buffer of its own: it is read
      // again only after the barrier of the next sum)
      auto vec_sum = [&](double v, double* buf) {
        if (tid < DE) {
          v = wave_sum_dpp(v);
          if (lane == 0) buf[wave] = v;
        }
        __syncthreads();
        double z = 0.0;
#pragma unroll
        for (int h = 0; h < DE / 64; ++h) z += buf[h];
        return z;
      };
      const double alpha = vec_sum(ma, rsa);
      double mb = 0.0;
      if (tid < DE) {
        wr = fma(-alpha, qr[tid], wr);
        mb = wr * wr;
        if constexpr (CPLX) {
          wi = fma(-alpha, qi[tid], wi);
          mb = fma(wi, wi, mb);
        }
      }
      const double beta = sqrt(vec_sum(mb, rsb));
      const bool invariant = !(beta > 64.0 * u * nf);   // Krylov space invariant (or no progress)
      if (tid == 0) {
        al[k] = alpha;
        be[k] = beta;
      }
      if (tid < DE) {
        ppr = qr[tid];
        if constexpr (CPLX) ppi = qi[tid];
        if (!invariant) {
          const double ib = 1.0 / beta;
          qr[tid] = wr * ib;
          if constexpr (CPLX) qi[tid] = wi * ib;
        }
      }
      bprev = beta;
      __syncthreads();
      const int kk = k + 1;
      if (invariant || kk == KMAX || (kk >= 16 && (kk & 7) == 0)) {
        rho = ritz_min(al, be, kk, red);
        dlast = invariant ? 0.0 : fabs(rho_old - rho);
        rho_old = rho;
        if (dlast <= 64.0 * u * nf) break;
      }
    }
    // the full matrix for the factorisation, over the half storage
    big_assemble<double, double, CPLX, false>(A, c, DE, ar, ai, (double*)nullptr, (double*)nullptr, 0.0, tid, NT);
    __syncthreads();
    // ---- Cholesky of theta - sigma I, sigma = rho - eta ----
    const double eta = 2.0 * dlast + 16.0 * DE * u * nf;
    const double sigma = A.cert_method == 2 ? rho + 1.0 + nf : rho - eta;
    bool ok = isfinite(sigma) && dlast <= 1e-10 * nf;   // unconverged Ritz value: fall back
    double dmax = 0.0, cmax = 0.0;
    for (int i = tid; i < DE; i += NT) rsum[i] = 0.0;
    for (int p = 0; p < DE && ok; p += NB) {
      const int m = DE - p;   // rows p .. De-1 of the panel
      for (int idx = tid; idx < m * NB; idx += NT) {
        const int r = idx / NB, q = idx % NB;
        const int64_t o = (int64_t)(p + r) * DE + p + q;
        double vr_ = ar[o], vi_ = CPLX ? ai[o] : 0.0;
        if (r == q) {
          vr_ -= sigma;
          vi_ = 0.0;
          dmax = fmax(dmax, fabs(vr_));
        }
        Pr[q][r] = vr_;
        if constexpr (CPLX) Pi[q][r] = vi_;
      }
      __syncthreads();
      // One barrier a column: column q is scaled to L where it is used, and stored scaled a column
      // later, when no wave reads it any more
      auto store_scaled = [&](int q, double il, double l) {
        for (int r = q + tid; r < m; r += NT) {
          Pr[q][r] = r == q ? l : Pr[q][r] * il;
          if constexpr (CPLX) Pi[q][r] = r == q ? 0.0 : Pi[q][r] * il;
        }
      };
      double l = 0.0, il = 0.0;
      for (int q = 0; q < NB; ++q) {
        if (q > 0) store_scaled(q - 1, il, l);
        const double d = Pr[q][q];
        if (!(d > 0.0) || !isfinite(d)) {   // every thread reads the same value: uniform
          ok = false;
          break;
        }
        l = sqrt(d);
        il = 1.0 / l;
        // S[r][q2] -= L[r][q] conj(L[q2][q]) for the panel's later columns q2 <= r (wave per column)
        for (int q2 = q + 1 + wave; q2 < NB; q2 += NW) {
          const double kr = Pr[q][q2] * il, ki = CPLX ? Pi[q][q2] * il : 0.0;
#pragma unroll 4
          for (int r = q2 + lane; r < m; r += 64) {
            const double lr = Pr[q][r] * il;
            if constexpr (CPLX) {
              const double li = Pi[q][r] * il;
              Pr[q2][r] -= fma(lr, kr, li * ki);
              Pi[q2][r] -= fma(li, kr, -lr * ki);
            } else {
              Pr[q2][r] -= lr * kr;
            }
          }
        }
        __syncthreads();
      }
      if (ok) store_scaled(NB - 1, il, l);
      __syncthreads();
      if (!ok) break;
      // sums of |L| along the panel's rows (this thread's rows) and columns (wave per column)
      for (int r = tid; r < m; r += NT) {
        double rs = 0.0;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          if (r < q) continue;
          rs += CPLX ? sqrt(fma(Pr[q][r], Pr[q][r], Pi[q][r] * Pi[q][r])) : fabs(Pr[q][r]);
        }
        rsum[p + r] += rs;
      }
      for (int q = wave; q < NB; q += NW) {
        double cs = 0.0;
        for (int r = q + lane; r < m; r += 64)
          cs += CPLX ? sqrt(fma(Pr[q][r], Pr[q][r], Pi[q][r] * Pi[q][r])) : fabs(Pr[q][r]);
        cs = wave_sum(cs);
        if (lane == 0) csum[q] = cs;
      }
      // trailing update S[i][j] -= sum_q L[i][q] conj(L[j][q]), i, j >= p + NB, of the 16 x 16 blocks on
      // and below the diagonal (what lies above it is not read), on the matrix cores: as vector code it
      // was bound by the LDS reads of four operands per complex product
      const int nb = (m - NB) / 16;
      for (int blk = wave, I = 0, first = 0; blk < nb * (nb + 1) / 2; blk += NW) {
        while (blk - first > I) first += ++I;   // block row I starts at block I (I + 1) / 2
        const int lr = lane >> 4, i = NB + 16 * I + (lane & 15), j = NB + 16 * (blk - first) + (lane & 15);
        const int64_t o = (int64_t)(p + NB + 16 * I + lr) * DE + p + j;
        mfma_f64x4 sr, si;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          sr[r] = -ar[o + 4 * r * DE];
          if constexpr (CPLX) si[r] = -ai[o + 4 * r * DE];
        }
#pragma unroll
        for (int q0 = 0; q0 < NB; q0 += 4) {
          const double xr = Pr[q0 + lr][i], yr_ = Pr[q0 + lr][j];
          sr = __builtin_amdgcn_mfma_f64_16x16x4f64(xr, yr_, sr, 0, 0, 0);
          if constexpr (CPLX) {
            const double xi = Pi[q0 + lr][i], yi_ = Pi[q0 + lr][j];
            sr = __builtin_amdgcn_mfma_f64_16x16x4f64(xi, yi_, sr, 0, 0, 0);
            si = __builtin_amdgcn_mfma_f64_16x16x4f64(xi, yr_, si, 0, 0, 0);
            si = __builtin_amdgcn_mfma_f64_16x16x4f64(-xr, yi_, si, 0, 0, 0);
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          ar[o + 4 * r * DE] = -sr[r];
          if constexpr (CPLX) ai[o + 4 * r * DE] = -si[r];
        }
      }
      __syncthreads();
      if (tid == 0)
        for (int q = 0; q < NB; ++q) cmax = fmax(cmax, csum[q]);
    }
    ok = ok && A.cert_method != 2;
    if (ok) {
      double rmax = 0.0;
      for (int i = tid; i < DE; i += NT) rmax = fmax(rmax, rsum[i]);
      rmax = block_max(rmax, red);
      dmax = block_max(dmax, red);
      if (tid == 0) {
        constexpr double nn = CPLX ? 2.0 * DE + 4.0 : DE + 1.0;
        const double gam = (CPLX ? 1.4142135623730951 : 1.0) * nn * u / (1.0 - nn * u);
        const double c_chol = gam * cmax * rmax * (1.0 + 4.0 * DE * u);
        const double c_shift = 2.0 * u * dmax;
        const double c_asm = 2.0 * (A.maxch + A.maxpar + 1) * u * nf;
        A.scal[gid] = rho;
        A.scal2[gid] = (rho - sigma) + c_chol + c_shift + c_asm;
        if (!isfinite(rho) && A.nonfinite) atomicAdd(A.nonfinite, 1ull);
      }
      __syncthreads();
    } else {
      if (tid == 0 && A.cert_fallback) atomicAdd(A.cert_fallback, 1ull);
      big_assemble<double, double, CPLX, false>(A, c, DE, ar, ai, (double*)nullptr, (double*)nullptr, 0.0, tid, NT);
      tridiag_lambda_min<CPLX, DE>(A, c, ar, ai);
    }
  }
}

// Bits of a placed, lowest first, at the set bits of mask (lowest first).
__device__ __forceinline__ int spread_bits(int a, int mask) {
  int r = 0;
  for (int t = 0; mask != 0; ++t) {
    const int lb = mask & -mask;
    if ((a >> t) & 1) r |= lb;
    mask ^= lb;
  }
  return r;
}

// theta_e at the messages (no extrapolation) into the group's LDS matrix, De lanes per cluster
// (lane i): h_e and the parent messages row by row, then the child messages entry by entry, each
// entry (a, b) of 1 (x) nu_{e->f} scattered to its De / Dc positions (pdep(a, x), pdep(b, x)) over
// the complement bits x.  Children go one after another: two of them can reach one element.
template <bool CPLX, int DE>
__device__ void rows_assemble(const ClusterArgs<double>& A, int64_t c, int i, bool active, double* dr, double* di) {
  constexpr int LD = DE + 1;
  double rr[DE], ri[CPLX ? DE : 1];
#pragma unroll
  for (int j = 0; j < DE; ++j) {
    rr[j] = 0.0;
    if constexpr (CPLX) ri[j] = 0.0;
  }
  const int64_t ho = active ? A.hoff[c] : -1;
  if (ho >= 0) {
    const double* h = A.h + ho;
#pragma unroll
    for (int j = 0; j < DE; ++j) {
      double vr, vi;
      herm_elem<double>([&](int k) { return h[k]; }, i, j, DE, CPLX, vr, vi);
      rr[j] = vr;
      if constexpr (CPLX) ri[j] = vi;
    }
  }
  for (int s = 0; s < A.maxpar; ++s) {
    const int m = active ? A.par[(int64_t)s * A.n + c] : -1;
    if (m < 0) continue;
#pragma unroll
    for (int j = 0; j < DE; ++j) {
      double vr, vi;
      herm_elem<double>([&](int k) { return A.nu_p[(int64_t)k * A.Mp + m]; }, i, j, DE, CPLX, vr, vi);
      rr[j] += vr;
      if constexpr (CPLX) ri[j] += vi;
    }
  }
#pragma unroll
  for (int j = 0; j < DE; ++j) {
    dr[i * LD + j] = rr[j];
    if constexpr (CPLX) di[i * LD + j] = ri[j];
  }
  __syncthreads();
  if (A.Dc <= 0) return;
  const int Dc = A.Dc, ldc = __builtin_ctz(Dc), NE = Dc * Dc;
  for (int s = 0; s < A.maxch; ++s) {   // maxch is the bucket's: the barrier below is uniform
    const int m = active ? A.ch[(int64_t)s * A.n + c] : -1;
    if (m >= 0) {
      const int mask = A.chmask[(int64_t)s * A.n + c] & (DE - 1);
      const int cm = ~mask & (DE - 1);
      for (int ab = i; ab < NE; ab += DE) {
        const int a = ab >> ldc, b = ab & (Dc - 1);
        double er, ei;
        herm_elem<double>([&](int k) { return A.nu_c[(int64_t)k * A.Mc + m]; }, a, b, Dc, CPLX, er, ei);
        const int ia = spread_bits(a, mask), jb = spread_bits(b, mask);
        int x = 0;
        do {   // every subset x of the complement bits
          dr[(ia | x) * LD + (jb | x)] -= er;
          if constexpr (CPLX) di[(ia | x) * LD + (jb | x)] -= ei;
          x = (x - cm) & cm;
        } while (x != 0);
      }
    }
    __syncthreads();
  }
}

// Row-parallel variant for De = 16, 32 (the default there): De lanes per cluster, 64 / De
// clusters per wave, lane i holding row i of theta_e in registers.  Column k below the diagonal
// is then one register per lane, the vectors v and w of each reflection are exchanged through
// LDS, and the reductions stay inside the lane group.  The tridiagonal (d, |e|^2) goes to a
// workspace (structure of arrays: d_k of cluster c at ws[k n + c], |e_k|^2 at ws[(De + k) n + c], and in the
// place of a |e_{De-1}|^2 the exponent of the scaling, or NaN where an entry is not finite) for
// k_sturm_bisect, which brackets lambda_min with one lane per cluster.
template <bool CPLX, int DE>
__global__ __launch_bounds__(64) void k_certify_rows(ClusterArgs<double> A, double* ws) {
  constexpr int LD = DE + 1;
  constexpr int G = 64 / DE;
  __shared__ double sar[G * DE * LD];
  __shared__ double sai[CPLX ? G * DE * LD : 1];
  __shared__ double vbr[G][DE], vbi[G][CPLX ? DE : 1], wbr[G][DE], wbi[G][CPLX ? DE : 1];
  const int l = threadIdx.x, g = l / DE, i = l % DE;
  const int64_t c = (int64_t)blockIdx.x * G + g;
  const bool active = c < A.n;
  double* dr = sar + g * DE * LD;
  double* di = CPLX ? sai + g * DE * LD : sai;
  rows_assemble<CPLX, DE>(A, c, i, active, dr, di);
  double ar[DE], ai[CPLX ? DE : 1];
  double amax = 0.0, n2 = 0.0;
#pragma unroll
  for (int j = 0; j < DE; ++j) {
    ar[j] = active ? dr[i * LD + j] : 0.0;
    amax = fmax(amax, fabs(ar[j]));
    if constexpr (CPLX) {
      ai[j] = active ? di[i * LD + j] : 0.0;
      amax = fmax(amax, fabs(ai[j]));
    }
  }
  const int ex = unit_exponent(seg_max<DE>(amax));
#pragma unroll
  for (int j = 0; j < DE; ++j) {
    ar[j] = ldexp(ar[j], -ex);
    n2 = fma(ar[j], ar[j], n2);
    if constexpr (CPLX) {
      ai[j] = ldexp(ai[j], -ex);
      n2 = fma(ai[j], ai[j], n2);
    }
  }
  const double nrm2 = seg_sum<DE>(n2);
  double e2mine = 0.0;
#pragma unroll
  for (int k = 0; k < DE - 2; ++k) {
    // x = column k below the diagonal: element k of the rows i > k
    const bool below = i > k;
    const double xr = below ? ar[k] : 0.0;
    const double xi = (CPLX && below) ? ai[k] : 0.0;
    const double xn2 = seg_sum<DE>(fma(xr, xr, xi * xi));
    if (i == k) e2mine = xn2;
    // x0 = element k + 1, the first of x, broadcast from lane k + 1 of the group
    const double x0r = __shfl(xr, g * DE + k + 1, 64), x0i = CPLX ? __shfl(xi, g * DE + k + 1, 64) : 0.0;
    double xn, a0, tau;   // uniform in the group
    householder_scalars(xn2, x0r, x0i, xn, a0, tau);
    const double ur = a0 > 0.0 ? x0r / a0 : 1.0, ui = a0 > 0.0 ? x0i / a0 : 0.0;
    // v = x - alpha e_{k+1}, alpha = -(x0 / |x0|) ||x||
    double vr = xr, vi = xi;
    if (i == k + 1) {
      vr = fma(ur, xn, vr);
      vi = fma(ui, xn, vi);
    }
    vbr[g][i] = vr;
    if constexpr (CPLX) vbi[g][i] = vi;
    __syncthreads();
    // p_i = tau sum_{j > k} A_ij v_j
    double pr = 0.0, pim = 0.0;
#pragma unroll
    for (int j = k + 1; j < DE; ++j) {
      const double bjr = vbr[g][j];
      pr = fma(ar[j], bjr, pr);
      if constexpr (CPLX) {
        const double bji = vbi[g][j];
        pr = fma(-ai[j], bji, pr);
        pim = fma(ar[j], bji, fma(ai[j], bjr, pim));
      }
    }
    pr *= tau;
    pim *= tau;
    // K = (tau / 2) v^H p (real), w = p - K v
    const double K = 0.5 * tau * seg_sum<DE>(fma(vr, pr, vi * pim));
    const double wr = fma(-K, vr, pr), wi = fma(-K, vi, pim);
    wbr[g][i] = wr;
    if constexpr (CPLX) wbi[g][i] = wi;
    __syncthreads();
    // A22 -= v w^H + w v^H (lanes i <= k have v_i = w_i = 0: their rows do not change)
#pragma unroll
    for (int j = k + 1; j < DE; ++j) {
      const double vjr = vbr[g][j], wjr = wbr[g][j];
      if constexpr (CPLX) {
        const double vji = vbi[g][j], wji = wbi[g][j];
        ar[j] -= fma(vr, wjr, fma(vi, wji, fma(wr, vjr, wi * vji)));
        ai[j] -= fma(vi, wjr, fma(-vr, wji, fma(wi, vjr, -wr * vji)));
      } else {
        ar[j] -= fma(vr, wjr, wr * vjr);
      }
    }
    __syncthreads();   // before the next step overwrites the broadcast vectors
  }
  // last 2 x 2 block: |e_{De-2}|^2 = |A_{De-2, De-1}|^2, element De - 1 of row De - 2
  if (i == DE - 2) e2mine = fma(ar[DE - 1], ar[DE - 1], CPLX ? ai[DE - 1] * ai[DE - 1] : 0.0);
  double dmine = 0.0;
#pragma unroll
  for (int j = 0; j < DE; ++j)
    if (j == i) dmine = ar[j];
  if (active) {
    ws[(int64_t)i * A.n + c] = dmine;
    ws[(int64_t)(DE + i) * A.n + c] = (i < DE - 1) ? e2mine : isfinite(nrm2) ? (double)ex : nrm2 - nrm2;
    if (i == 0) A.scal2[A.gid[c]] = ldexp(8.0 * DE * DBL_EPSILON * sqrt(nrm2), ex);
  }
}

// lambda_min of every cluster's tridiagonal (d, |e|^2) by bisection on Sturm counts, one lane per
// cluster: from the Gershgorin interval (widened by a few ulps) down to a few ulps of lambda_min;
// the lower end of the final bracket, below which the tridiagonal has no eigenvalue, is returned.
template <int DE>
__global__ __launch_bounds__(256) void k_sturm_bisect(ClusterArgs<double> A, const double* ws) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= A.n) return;
  double d[DE], e2[DE];
#pragma unroll
  for (int k = 0; k < DE; ++k) {
    d[k] = ws[(int64_t)k * A.n + c];
    e2[k] = ws[(int64_t)(DE + k) * A.n + c];
  }
  const double ex = e2[DE - 1];   // NaN: not finite
  e2[DE - 1] = 0.0;
  double lo = INFINITY, hi = -INFINITY, emax = 0.0, re_prev = 0.0;
#pragma unroll
  for (int k = 0; k < DE; ++k) {
    const double re = sqrt(e2[k]);
    lo = fmin(lo, d[k] - (re_prev + re));
    hi = fmax(hi, d[k] + (re_prev + re));
    emax = fmax(emax, e2[k]);
    re_prev = re;
  }
  const double pivmin = DBL_MIN * fmax(1.0, emax);
  const double span0 = fmax(hi - lo, DBL_MIN);
  lo -= 2.0 * DBL_EPSILON * fabs(lo) + span0 * DBL_EPSILON;
  hi += 2.0 * DBL_EPSILON * fabs(hi) + span0 * DBL_EPSILON;
  for (int it = 0; it < 64; ++it) {
    if (hi - lo <= 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi))) break;
    const double x = 0.5 * (lo + hi);
    if (!(x > lo && x < hi)) break;
    bool neg = false;
    double q = d[0] - x;
    if (fabs(q) < pivmin) q = -pivmin;
    neg = q < 0.0;
#pragma unroll
    for (int k = 1; k < DE; ++k) {
      q = (d[k] - x) - e2[k - 1] / q;
      if (fabs(q) < pivmin) q = -pivmin;
      neg = neg || (q < 0.0);
    }
    if (neg) hi = x;   // an eigenvalue below x
    else lo = x;
  }
  const double v = ex == ex ? ldexp(lo, (int)ex) : ex;
  A.scal[A.gid[c]] = v;
  if (!isfinite(v) && A.nonfinite) atomicAdd(A.nonfinite, 1ull);
}

// One-wave variant for De = 16, 32: the matrix in LDS, the De rows of A22 v split over
// 64/De lane groups (partial sums over j = g, g + G, ... combined by shuffles), 64 Sturm
// points per multisection round.
template <bool CPLX, int DE>
__global__ __launch_bounds__(64) void k_cluster_tridiag_w(ClusterArgs<double> A) {
  constexpr int LD = DE + 1;
  constexpr int G = 64 / DE;
  __shared__ double ar[DE * LD];
  __shared__ double ai[CPLX ? DE * LD : 1];
  __shared__ double vr[DE], vi[DE], pr[DE], pi[DE], dg[DE], e2[DE];
  const int64_t c = xcd_cluster(blockIdx.x, A.n);
  const int l = threadIdx.x;
  const int li = l % DE, lg = l / DE;
  lds_assemble<double, CPLX, DE, 64>(A, c, l, A.nu_c, nullptr, A.nu_p, nullptr, 0.0, true, 1.0, ar, ai);
  double amax = 0.0, n2 = 0.0;
  for (int idx = l; idx < DE * DE; idx += 64) {   // the lane's own elements
    const int o = idx / DE * LD + idx % DE;
    amax = fmax(amax, fabs(ar[o]));
    if constexpr (CPLX) amax = fmax(amax, fabs(ai[o]));
  }
  const int ex = __builtin_amdgcn_readfirstlane(unit_exponent(seg_max<64>(amax)));
  for (int idx = l; idx < DE * DE; idx += 64) {
    const int o = idx / DE * LD + idx % DE;
    ar[o] = ldexp(ar[o], -ex);
    n2 = fma(ar[o], ar[o], n2);
    if constexpr (CPLX) {
      ai[o] = ldexp(ai[o], -ex);
      n2 = fma(ai[o], ai[o], n2);
    }
  }
  const double nrm2 = wave_sum_dpp(n2);
  __syncthreads();
  for (int k = 0; k < DE - 2; ++k) {
    const int m = DE - k - 1;
    const int rk = k * LD + k + 1;   // x_i = A[k+1+i][k] = conj(A[k][k+1+i])
    double xs = 0.0;
    if (l < m) {
      xs = ar[rk + l] * ar[rk + l];
      if constexpr (CPLX) xs = fma(ai[rk + l], ai[rk + l], xs);
    }
    const double xn2 = wave_sum_dpp(xs);
    const double x0r = ar[rk], x0i = CPLX ? -ai[rk] : 0.0;
    double xn, a0, tau;
    householder_scalars(xn2, x0r, x0i, xn, a0, tau);
    if (l == 0) {
      dg[k] = ar[k * LD + k];
      e2[k] = xn2;
    }
    if (!(tau > 0.0)) continue;   // wave-uniform
    const double ur = a0 > 0.0 ? x0r / a0 : 1.0, ui = a0 > 0.0 ? x0i / a0 : 0.0;
    if (l < m) {
      double r = ar[rk + l], im = CPLX ? -ai[rk + l] : 0.0;
      if (l == 0) {
        r += ur * xn;
        im += ui * xn;
      }
      vr[l] = r;
      vi[l] = im;
    }
    __syncthreads();
    // p = tau A22 v: lane (li, lg) sums j = lg, lg + G, ... of row li (read as column li)
    double sr = 0.0, si = 0.0;
    if (li < m) {
      for (int j = lg; j < m; j += G) {
        const int o = (k + 1 + j) * LD + (k + 1 + li);
        const double a_r = ar[o];
        sr = fma(a_r, vr[j], sr);
        if constexpr (CPLX) {
          const double a_i = -ai[o];
          sr = fma(-a_i, vi[j], sr);
          si = fma(a_r, vi[j], fma(a_i, vr[j], si));
        }
      }
    }
#pragma unroll
    for (int o = DE; o < 64; o <<= 1) {
      sr += __shfl_xor(sr, o, 64);
      if constexpr (CPLX) si += __shfl_xor(si, o, 64);
    }
    sr *= tau;
    si *= tau;
    const double ks = (l < m) ? fma(vr[l], sr, vi[l] * si) : 0.0;
    const double K = 0.5 * tau * wave_sum_dpp(ks);
    if (l < m) {
      pr[l] = fma(-K, vr[l], sr);
      pi[l] = fma(-K, vi[l], si);
    }
    __syncthreads();
    // A22 -= v w^H + w v^H: lane (li, lg) updates column li of rows lg, lg + G, ... (no division)
    if (li < m) {
#pragma unroll 4
      for (int i = lg; i < m; i += G) {
        const int o = (k + 1 + i) * LD + (k + 1 + li);
        ar[o] -= fma(vr[i], pr[li], fma(vi[i], pi[li], fma(pr[i], vr[li], pi[i] * vi[li])));
        if constexpr (CPLX) ai[o] -= fma(vi[i], pr[li], fma(-vr[i], pi[li], fma(pi[i], vr[li], -pr[i] * vi[li])));
      }
    }
    __syncthreads();
  }
  if (l == 0) {
    dg[DE - 2] = ar[(DE - 2) * LD + DE - 2];
    dg[DE - 1] = ar[(DE - 1) * LD + DE - 1];
    const double xr = ar[(DE - 2) * LD + DE - 1], xi = CPLX ? ai[(DE - 2) * LD + DE - 1] : 0.0;
    e2[DE - 2] = fma(xr, xr, xi * xi);
    e2[DE - 1] = 0.0;
  }
  __syncthreads();
  double lo = INFINITY, hi = -INFINITY, emax = 0.0;
  for (int i = 0; i < DE; ++i) {
    const double r = (i > 0 ? sqrt(e2[i - 1]) : 0.0) + sqrt(e2[i]);
    lo = fmin(lo, dg[i] - r);
    hi = fmax(hi, dg[i] + r);
    emax = fmax(emax, e2[i]);
  }
  const double pivmin = DBL_MIN * fmax(1.0, emax);
  const double span0 = fmax(hi - lo, DBL_MIN);
  lo -= 2.0 * DBL_EPSILON * fabs(lo) + span0 * DBL_EPSILON;
  hi += 2.0 * DBL_EPSILON * fabs(hi) + span0 * DBL_EPSILON;
  for (int round = 0; round < 14; ++round) {
    if (hi - lo <= 2.0 * DBL_EPSILON * fmax(fabs(lo), fabs(hi))) break;   // a few ulps of lambda_min
    const double x = lo + (hi - lo) * (double)(l + 1) / 65.0;
    int cnt = 0;
    double q = dg[0] - x;
    if (fabs(q) < pivmin) q = -pivmin;
    cnt += q < 0.0;
    for (int i = 1; i < DE; ++i) {
      q = (dg[i] - x) - e2[i - 1] / q;
      if (fabs(q) < pivmin) q = -pivmin;
      cnt += q < 0.0;
    }
    const int t = (int)wave_min_dpp(cnt > 0 ? (double)l : 64.0);
    const double nlo = t == 0 ? lo : lo + (hi - lo) * (double)t / 65.0;
    const double nhi = t == 64 ? hi : lo + (hi - lo) * (double)(t + 1) / 65.0;
    if (!(nhi - nlo < hi - lo)) break;
    lo = nlo;
    hi = nhi;
  }
  if (l == 0) store_tridiag_bound(A, A.gid[c], DE, lo, nrm2, ex);
}

// ------------------------------------------------------------------------------------------
// adjoint (a9): VJP of (Q_beta, grad Q_beta) through one cluster
// ------------------------------------------------------------------------------------------
//
// grad Q_beta = B^* rho_beta(B nu + h) with B the linear map from messages to augmented
// Hamiltonians (chain rule of the Lipschitz lemma, Sec. 4.1.2).  For cotangents qbar (per
// instance) and gbar (per message) the cluster's cotangent is
//     Y_e = qbar rho_e + D rho_e[(B gbar)_e],
// with the Daleckii-Krein derivative of the normalised matrix exponential
//     D rho[X] = U [Gamma o (U^H X U)] U^H + beta <rho, X> rho,
//     Gamma_ab = (p_a - p_b)/(l_a - l_b) = p_lo expm1(-beta (l_hi - l_lo)) / (l_hi - l_lo),
//     Gamma_aa = -beta p_a.
// nu_bar = B^* Y is then the message kernel's gradient stage (Y_f - Tr_{e\f} Y_e).  At beta = 0
// the cotangent of Q is Y_e = qbar mu_e (the ground projector; gbar must be absent).
// W lanes per cluster, 64/W clusters per single-wave block.
template <typename T, bool CPLX, int DE, int MODE, int W>
struct VjpLds {
  static constexpr int G = 64 / W, LD = DE + 1, SZ = G * DE * LD, SI = CPLX ? SZ : 1;
  // A wave per cluster: the products' plane only where there are products; without it a third wave of complex
  // 32 x 32 clusters fits a CU.  (Several clusters to a wave keep it: five waves on the four SIMDs of
  // a CU cost more than they bring, 265 us for 8000 real 16 x 16 clusters against 221.)
  static constexpr int ST = MODE == MODE_GIBBS || G > 1 ? SZ : 1, STI = CPLX ? ST : 1;
  static constexpr bool REG = W < 64;   // a wave per cluster: the solver in LDS, on all its lanes
  using Scratch = ScratchFor<T, DE, REG>;
  T ar[SZ], ur[SZ], xr[SZ], yr[ST], ai[SI], ui[SI], xi[SI], yi[STI];
  T p[G * DE], lam[G * DE];
  Scratch J[G];
};
// Where a body finds them: members of one VjpLds, or, a wave per cluster, arrays of their own, which the
// compiler can tell apart (as members, a cluster of 32 or 64 dimensions takes 4 to 9 % longer).
template <typename T, typename Scratch>
struct VjpPlanes {
  T *ar, *ur, *xr, *yr, *ai, *ui, *xi, *yi, *p, *lam;
  Scratch* J;
};
template <typename T, typename L>
__device__ __forceinline__ VjpPlanes<T, typename L::Scratch> vjp_planes(L& v) {
  return {v.ar, v.ur, v.xr, v.yr, v.ai, v.ui, v.xi, v.yi, v.p, v.lam, v.J};
}

template <typename T, bool CPLX, int DE, int MODE, int W>
__device__ void cluster_vjp_body(const ClusterArgs<T>& A, int64_t block, int64_t blocks,
                                 const VjpPlanes<T, typename VjpLds<T, CPLX, DE, MODE, W>::Scratch>& L) {
  constexpr bool REG = VjpLds<T, CPLX, DE, MODE, W>::REG;
  constexpr int LD = DE + 1;
  constexpr int G = 64 / W;
  constexpr int SZ = DE * LD;
  // (one cluster per wave: constants, which are another 4 to 8 % at D = 32, 64)
  const int g = G == 1 ? 0 : threadIdx.x / W, tid = G == 1 ? threadIdx.x : threadIdx.x % W;
  const int64_t c = xcd_cluster(block, blocks) * G + g;
  const bool active = G == 1 || c < A.n;
  T *sar = L.ar + g * SZ, *sur = L.ur + g * SZ, *sxr = L.xr + g * SZ, *str = L.yr + g * SZ;
  T *sai = CPLX ? L.ai + g * SZ : L.ai, *sui = CPLX ? L.ui + g * SZ : L.ui, *sxi = CPLX ? L.xi + g * SZ : L.xi,
    *sti = CPLX ? L.yi + g * SZ : L.yi;
  T *sp = L.p + g * DE, *slam = L.lam + g * DE;
  const bool has_g = (A.gb_c != nullptr || A.gb_p != nullptr);
  T n2 = T(0);
  if (active) {
    n2 = lds_assemble<T, CPLX, DE, W>(A, c, tid, A.nu_c, nullptr, A.nu_p, nullptr, T(0), true, T(1), sar, sai);
    if (has_g) lds_assemble<T, CPLX, DE, W>(A, c, tid, A.gb_c, nullptr, A.gb_p, nullptr, T(0), false,
                                            (T)A.gb_offscale, sxr, sxi);
  }
  const T nrm2 = seg_sum<W>(n2);
  init_vectors<T, CPLX, DE, true, W, REG>(sur, sui, tid, active);
  __syncthreads();
  const bool conv = cluster_jacobi<T, CPLX, DE, true, W, REG>(sar, sai, sur, sui, L.J[g], A.tol, nrm2,
                                                         A.max_sweeps, tid, active);
  if (active && !conv && tid == 0 && A.noconv) atomicAdd(A.noconv, 1ull);
  T lmin = T(INFINITY);
  if (active)
    for (int k = tid; k < DE; k += W) {
      slam[k] = sar[k * LD + k];
      lmin = fmin(lmin, sar[k * LD + k]);
    }
  lmin = seg_min<W>(lmin);
  const T beta = (T)A.beta;
  lds_weights<T, DE, MODE, W>(sar, sp, lmin, beta, (T)A.tau_rel * fmax(T(1), dsqrt<T>(nrm2)), tid, active);
  // rho (or mu) over A
  if (active) lds_rebuild<T, CPLX, DE, W>(sur, sui, sp, sar, sai, tid);
  __syncthreads();
  const int32_t gid = active ? A.gid[c] : 0;
  const T qb = active && A.qbar ? (T)A.qbar[A.cinst[gid]] : T(0);
  if (MODE == MODE_GIBBS && has_g) {
    // <rho, X>
    T rx = T(0);
    for (int idx = tid; active && idx < DE * DE; idx += W) {
      rx = dfma<T>(sar[idx / DE * LD + idx % DE], sxr[idx / DE * LD + idx % DE], rx);
      if constexpr (CPLX) rx = dfma<T>(sai[idx / DE * LD + idx % DE], sxi[idx / DE * LD + idx % DE], rx);
    }
    rx = seg_sum<W>(rx);
    // Tm = U^H X
    for (int idx = tid; active && idx < DE * DE; idx += W) {
      const int a = idx / DE, j = idx % DE;
      T sr = T(0), si = T(0);
      for (int k = 0; k < DE; ++k) {
        const T ur = sur[k * LD + a], ui = CPLX ? -sui[k * LD + a] : T(0);  // conj(U_ka)
        const T xr = sxr[k * LD + j], xi = CPLX ? sxi[k * LD + j] : T(0);
        sr = dfma<T>(ur, xr, sr);
        if constexpr (CPLX) {
          sr = dfma<T>(-ui, xi, sr);
          si = dfma<T>(ur, xi, si);
          si = dfma<T>(ui, xr, si);
        }
      }
      str[a * LD + j] = sr;
      if constexpr (CPLX) sti[a * LD + j] = si;
    }
    __syncthreads();
    // M = (U^H X) U, then Gamma o M (into X)
    for (int idx = tid; active && idx < DE * DE; idx += W) {
      const int a = idx / DE, b = idx % DE;
      T sr = T(0), si = T(0);
      for (int k = 0; k < DE; ++k) {
        const T tr = str[a * LD + k], ti = CPLX ? sti[a * LD + k] : T(0);
        const T ur = sur[k * LD + b], ui = CPLX ? sui[k * LD + b] : T(0);
        sr = dfma<T>(tr, ur, sr);
        if constexpr (CPLX) {
          sr = dfma<T>(-ti, ui, sr);
          si = dfma<T>(tr, ui, si);
          si = dfma<T>(ti, ur, si);
        }
      }
      const int hi = slam[a] >= slam[b] ? a : b, lo = slam[a] >= slam[b] ? b : a;
      const T dl = slam[hi] - slam[lo];
      const T g = (dl == T(0)) ? -beta * sp[lo] : sp[lo] * (T)expm1((double)(-beta * dl)) / dl;
      sxr[a * LD + b] = g * sr;
      if constexpr (CPLX) sxi[a * LD + b] = g * si;
    }
    __syncthreads();
    // Tm = U (Gamma o M)
    for (int idx = tid; active && idx < DE * DE; idx += W) {
      const int i = idx / DE, b = idx % DE;
      T sr = T(0), si = T(0);
      for (int k = 0; k < DE; ++k) {
        const T ur = sur[i * LD + k], ui = CPLX ? sui[i * LD + k] : T(0);
        const T mr = sxr[k * LD + b], mi = CPLX ? sxi[k * LD + b] : T(0);
        sr = dfma<T>(ur, mr, sr);
        if constexpr (CPLX) {
          sr = dfma<T>(-ui, mi, sr);
          si = dfma<T>(ur, mi, si);
          si = dfma<T>(ui, mr, si);
        }
      }
      str[i * LD + b] = sr;
      if constexpr (CPLX) sti[i * LD + b] = si;
    }
    __syncthreads();
    // Y = Tm U^H + (beta <rho,X> + qbar) rho  (into X)
    const T w = beta * rx + qb;
    for (int idx = tid; active && idx < DE * DE; idx += W) {
      const int i = idx / DE, j = idx % DE;
      T sr = T(0), si = T(0);
      for (int k = 0; k < DE; ++k) {
        const T tr = str[i * LD + k], ti = CPLX ? sti[i * LD + k] : T(0);
        const T ur = sur[j * LD + k], ui = CPLX ? -sui[j * LD + k] : T(0);  // conj(U_jk)
        sr = dfma<T>(tr, ur, sr);
        if constexpr (CPLX) {
          sr = dfma<T>(-ti, ui, sr);
          si = dfma<T>(tr, ui, si);
          si = dfma<T>(ti, ur, si);
        }
      }
      sxr[i * LD + j] = dfma<T>(w, sar[i * LD + j], sr);
      if constexpr (CPLX) sxi[i * LD + j] = dfma<T>(w, sai[i * LD + j], si);
    }
    __syncthreads();
    // symmetrise (Y is Hermitian up to rounding): keep the upper triangle mirrored
    for (int idx = tid; active && idx < DE * DE; idx += W) {
      const int i = idx / DE, j = idx % DE;
      if (i < j) {
        sxr[j * LD + i] = sxr[i * LD + j];
        if constexpr (CPLX) sxi[j * LD + i] = -sxi[i * LD + j];
      }
      if constexpr (CPLX) { if (i == j) sxi[i * LD + i] = T(0); }
    }
    __syncthreads();
    if (active) lds_outputs<T, CPLX, DE, W>(A, c, tid, gid, sxr, sxi);
  } else {
    for (int idx = tid; active && idx < DE * DE; idx += W) {
      const int i = idx / DE, j = idx % DE;
      sxr[i * LD + j] = qb * sar[i * LD + j];
      if constexpr (CPLX) sxi[i * LD + j] = qb * sai[i * LD + j];
    }
    __syncthreads();
    if (active) lds_outputs<T, CPLX, DE, W>(A, c, tid, gid, sxr, sxi);
  }
}

template <typename T, bool CPLX, int DE, int MODE, int W>
__global__ __launch_bounds__(64) void k_cluster_vjp(ClusterArgs<T> A) {
  using L = VjpLds<T, CPLX, DE, MODE, W>;
  if constexpr (L::G > 1) {
    __shared__ L lds;
    cluster_vjp_body<T, CPLX, DE, MODE, W>(A, blockIdx.x, gridDim.x, vjp_planes<T>(lds));
  } else {
    // (arrays of one size lie in the order of their names: those of the solver within the reach, 64 KiB, of an
    // LDS instruction's offset; with the products' plane second the adjoint at D = 64 took 5 % longer)
    __shared__ T ar[L::SZ], ur[L::SZ], xr[L::SZ], yr[L::ST], ai[L::SI], ui[L::SI], xi[L::SI], yi[L::STI];
    __shared__ T p[DE], lam[DE];
    __shared__ typename L::Scratch J[1];
    cluster_vjp_body<T, CPLX, DE, MODE, W>(A, blockIdx.x, gridDim.x, {ar, ur, xr, yr, ai, ui, xi, yi, p, lam, J});
  }
}

// Buckets of D = 8, 4 and 2 in one launch, n8, n4, n2 blocks of each, the longest first (LDS: the
// largest of the three).  Each bucket reads the messages and writes its own outputs.
template <bool CPLX>
constexpr int vjp_group_lds() { return (int)sizeof(VjpLds<double, CPLX, 8, MODE_GIBBS, 8>); }
template <bool CPLX, int MODE>
__global__ __launch_bounds__(64) void k_cluster_vjp_group(ClusterArgs<double> A8, ClusterArgs<double> A4,
                                                          ClusterArgs<double> A2, int n8, int n4, int n2) {
  using L8 = VjpLds<double, CPLX, 8, MODE, 8>;
  using L4 = VjpLds<double, CPLX, 4, MODE, 4>;
  using L2 = VjpLds<double, CPLX, 2, MODE, 2>;
  static_assert(sizeof(L4) <= sizeof(L8) && sizeof(L2) <= sizeof(L8), "the largest");
  __shared__ __align__(16) unsigned char lds[sizeof(L8)];
  const int b = blockIdx.x;
  if (b < n8) cluster_vjp_body<double, CPLX, 8, MODE, 8>(A8, b, n8, vjp_planes<double>(*reinterpret_cast<L8*>(lds)));
  else if (b < n8 + n4) cluster_vjp_body<double, CPLX, 4, MODE, 4>(A4, b - n8, n4, vjp_planes<double>(*reinterpret_cast<L4*>(lds)));
  else cluster_vjp_body<double, CPLX, 2, MODE, 2>(A2, b - n8 - n4, n2, vjp_planes<double>(*reinterpret_cast<L2*>(lds)));
}

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------

static inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

// Register (one lane per cluster) instantiations: which (De, precision, field, mode) fit the
// register file (the whole De x De matrix and, with vectors, U live in one lane's VGPRs).
template <typename T, bool CPLX, int DE, int MODE>
constexpr bool reg_ok() {
  constexpr bool dbl = std::is_same<T, double>::value;
  if constexpr (DE <= 4) return true;
  if constexpr (DE == 8) return !(dbl && CPLX && MODE != MODE_CERTIFY);
  return false;  // D_e = 16: H + U exceed the arch VGPR file of one lane; the LDS kernel takes it
}

// Scaling-and-squaring Gibbs kernel (shape code W = 0): dimensions and fields compiled.
static bool expm_ok(int De, bool cplx) { return De == 16 || De == 32 || De == 64 || De == 128 || De == 256; }

// (childless 4 x 4 and 8 x 8 clusters are the overlaps of the two-level family)
static bool reg_pair(int De, int Dc) {
  return (De == 2 && Dc == 0) || (De == 4 && (Dc == 2 || Dc == 0)) || (De == 8 && (Dc == 4 || Dc == 2 || Dc == 0));
}

template <typename T, bool CPLX, int MODE, int DE, int W>
static void launch_lds_w(const ClusterArgs<T>& a, hipStream_t s) {
  constexpr int G = 64 / W;
  hipLaunchKernelGGL((k_cluster_lds<T, CPLX, DE, MODE, W>), dim3((unsigned)((a.n + G - 1) / G)), dim3(64), 0, s, a);
}

template <typename T, bool CPLX, int MODE, int DE, int DC>
static hipError_t launch_reg(const ClusterArgs<T>& a, int block, hipStream_t s) {
  if constexpr (reg_ok<T, CPLX, DE, MODE>()) {
    hipLaunchKernelGGL((k_cluster_reg<T, CPLX, DE, DC, MODE>), dim3(grid_for(a.n, block)), dim3(block), 0, s, a);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <typename T, bool CPLX, int MODE>
static hipError_t launch_cluster_m(const ClusterArgs<T>& a, int block, int W, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  // the register kernels hold one slot per site for single-site children
  if (a.Dc == 2 && (a.maxch < 1 || a.maxch > log2i(a.De))) return hipErrorInvalidValue;
  if (a.Dc == 2 && a.fp != nullptr && a.ch_rslot == nullptr) return hipErrorInvalidValue;
  if (W == 0 || W == 4) {   // 0: one wave per cluster up to D = 32, 4: one workgroup per cluster
    if constexpr (MODE == MODE_GIBBS) {
      if (a.fp != nullptr || a.n > 0x7fffffff) return hipErrorInvalidValue;
      if (a.De == 16 && W == 0)
        hipLaunchKernelGGL((k_cluster_expm<T, CPLX, 16>), dim3((unsigned)a.n), dim3(64), 0, s, a);
      else if (a.De == 32 && W == 0)
        hipLaunchKernelGGL((k_cluster_expm<T, CPLX, 32>), dim3((unsigned)a.n), dim3(64), 0, s, a);
      else if (a.De >= 32 && a.De <= 256 && a.expm_scratch != nullptr && a.expm_blocks > 0) {
        const unsigned grid = (unsigned)std::min<int64_t>(a.n, a.expm_blocks);
        if (a.De == 32)
          hipLaunchKernelGGL((k_cluster_expm_wg<T, CPLX, 32>), dim3(grid), dim3(WgPlan<32>::waves * 64), 0, s, a, a.expm_scratch, a.expm_slab);
        else if (a.De == 64)
          hipLaunchKernelGGL((k_cluster_expm_wg<T, CPLX, 64>), dim3(grid), dim3(WgPlan<64>::waves * 64), 0, s, a, a.expm_scratch, a.expm_slab);
        else if (a.De == 128)
          hipLaunchKernelGGL((k_cluster_expm_wg<T, CPLX, 128>), dim3(grid), dim3(WgPlan<128>::waves * 64), 0, s, a, a.expm_scratch, a.expm_slab);
        else if (a.De == 256)
          hipLaunchKernelGGL((k_cluster_expm_wg<T, CPLX, 256>), dim3(grid), dim3(WgPlan<256>::waves * 64), 0, s, a, a.expm_scratch, a.expm_slab);
        else
          return hipErrorInvalidValue;
      } else
        return hipErrorInvalidValue;
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  if (W == 2) {
    if constexpr (MODE == MODE_CERTIFY && std::is_same<T, double>::value) {
      if ((a.De == 16 || a.De == 32) && a.cert_ws != nullptr) {
        const int G = 64 / a.De;
        if ((a.n + G - 1) / G > 0x7fffffff) return hipErrorInvalidValue;
        const dim3 g1((unsigned)((a.n + G - 1) / G)), g2(grid_for(a.n, 256));
        if (a.De == 16) {
          hipLaunchKernelGGL((k_certify_rows<CPLX, 16>), g1, dim3(64), 0, s, a, a.cert_ws);
          hipLaunchKernelGGL((k_sturm_bisect<16>), g2, dim3(256), 0, s, a, (const double*)a.cert_ws);
        } else {
          hipLaunchKernelGGL((k_certify_rows<CPLX, 32>), g1, dim3(64), 0, s, a, a.cert_ws);
          hipLaunchKernelGGL((k_sturm_bisect<32>), g2, dim3(256), 0, s, a, (const double*)a.cert_ws);
        }
        return hipGetLastError();
      }
      if (a.De == 16 || a.De == 32) {
        if (a.n > 0x7fffffff) return hipErrorInvalidValue;
        if (a.De == 16)
          hipLaunchKernelGGL((k_cluster_tridiag_w<CPLX, 16>), dim3((unsigned)a.n), dim3(64), 0, s, a);
        else
          hipLaunchKernelGGL((k_cluster_tridiag_w<CPLX, 32>), dim3((unsigned)a.n), dim3(64), 0, s, a);
        return hipGetLastError();
      }
      if (a.expm_scratch == nullptr || a.expm_blocks <= 0) return hipErrorInvalidValue;
      const unsigned grid = (unsigned)std::min<int64_t>(a.n, a.expm_blocks);
      // Lanczos + Cholesky certificate at D_e = 256 by default (methods 2 and 3: every D_e >= 64);
      // at 64 and 128 the tridiagonalisation has the matrix in registers and the tighter margin, at 256
      // it goes through the slab and takes 3.9 times the certificate
      if (a.cert_method >= 2 || (a.cert_method == 0 && a.De >= 256)) {
        if (a.De == 64)
          hipLaunchKernelGGL((k_certify_lanczos<CPLX, 64>), dim3(grid), dim3(1024), 0, s, a, a.expm_scratch, a.expm_slab);
        else if (a.De == 128)
          hipLaunchKernelGGL((k_certify_lanczos<CPLX, 128>), dim3(grid), dim3(1024), 0, s, a, a.expm_scratch, a.expm_slab);
        else if (a.De == 256)
          hipLaunchKernelGGL((k_certify_lanczos<CPLX, 256>), dim3(grid), dim3(1024), 0, s, a, a.expm_scratch, a.expm_slab);
        else
          return hipErrorInvalidValue;
        return hipGetLastError();
      }
      if (a.n > 0x7fffffff) return hipErrorInvalidValue;
      if (a.De == 64)
        hipLaunchKernelGGL((k_certify_tridiag<CPLX, 64>), dim3((unsigned)a.n), dim3(256), 0, s, a);
      else if (a.De == 128)
        hipLaunchKernelGGL((k_certify_tridiag<CPLX, 128>), dim3((unsigned)a.n), dim3(512), 0, s, a);
      else if (a.De == 256)
        hipLaunchKernelGGL((k_cluster_tridiag<CPLX, 256>), dim3(grid), dim3(256), 0, s, a, a.expm_scratch, a.expm_slab);
      else
        return hipErrorInvalidValue;
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  if (W == 5) {   // clusters with a spin-1 site: table-driven Jacobi on the padded dimension
    if (a.gtab == nullptr && a.Dc > 0) return hipErrorInvalidValue;
    const int De = a.De;
    if (De <= 4) hipLaunchKernelGGL((k_cluster_gen<T, CPLX, 4, MODE, 4>), dim3((unsigned)((a.n + 15) / 16)), dim3(64), 0, s, a);
    else if (De <= 8) hipLaunchKernelGGL((k_cluster_gen<T, CPLX, 8, MODE, 8>), dim3((unsigned)((a.n + 7) / 8)), dim3(64), 0, s, a);
    else if (De <= 16) hipLaunchKernelGGL((k_cluster_gen<T, CPLX, 16, MODE, 16>), dim3((unsigned)((a.n + 3) / 4)), dim3(64), 0, s, a);
    else if (De <= 32) hipLaunchKernelGGL((k_cluster_gen<T, CPLX, 32, MODE, 32>), dim3((unsigned)((a.n + 1) / 2)), dim3(64), 0, s, a);
    else if (De <= 64) hipLaunchKernelGGL((k_cluster_gen<T, CPLX, 64, MODE, 64>), dim3((unsigned)a.n), dim3(64), 0, s, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  if (W == 1 && a.De >= 8) {
    if (a.De == 8 && a.Dc == 4) return launch_reg<T, CPLX, MODE, 8, 4>(a, block, s);
    if (a.De == 8 && a.Dc == 2) return launch_reg<T, CPLX, MODE, 8, 2>(a, block, s);
    if (a.De == 8 && a.Dc == 0) return launch_reg<T, CPLX, MODE, 8, 0>(a, block, s);
    return hipErrorInvalidValue;
  }
  if (a.De == 2 && a.Dc == 0) {
    hipLaunchKernelGGL((k_cluster_reg<T, CPLX, 2, 0, MODE>), dim3(grid_for(a.n, block)), dim3(block), 0, s, a);
  } else if (a.De == 4 && a.Dc == 2) {
    hipLaunchKernelGGL((k_cluster_reg<T, CPLX, 4, 2, MODE>), dim3(grid_for(a.n, block)), dim3(block), 0, s, a);
  } else if (a.De == 4 && a.Dc == 0 && W == 1) {
    hipLaunchKernelGGL((k_cluster_reg<T, CPLX, 4, 0, MODE>), dim3(grid_for(a.n, block)), dim3(block), 0, s, a);
  } else if (a.fp != nullptr) {
    return hipErrorInvalidValue;  // fused update only in the register kernel
  } else if (a.De == 4 && W == 64) {
    launch_lds_w<T, CPLX, MODE, 4, 64>(a, s);
  } else if (a.De == 8 && W == 16) {
    launch_lds_w<T, CPLX, MODE, 8, 16>(a, s);
  } else if (a.De == 8 && W == 8) {
    launch_lds_w<T, CPLX, MODE, 8, 8>(a, s);
  } else if (a.De == 8 && W == 64) {
    launch_lds_w<T, CPLX, MODE, 8, 64>(a, s);
  } else if (a.De == 16 && W == 16) {
    launch_lds_w<T, CPLX, MODE, 16, 16>(a, s);
  } else if (a.De == 16 && W == 32) {
    launch_lds_w<T, CPLX, MODE, 16, 32>(a, s);
  } else if (a.De == 16 && W == 64) {
    launch_lds_w<T, CPLX, MODE, 16, 64>(a, s);
  } else if (a.De == 32 && W == 32) {
    launch_lds_w<T, CPLX, MODE, 32, 32>(a, s);
  } else if (a.De == 32 && W == 64) {
    launch_lds_w<T, CPLX, MODE, 32, 64>(a, s);
  } else if (a.De == 64 && W == 64) {
    launch_lds_w<T, CPLX, MODE, 64, 64>(a, s);
  } else if ((a.De == 128 || a.De == 256) && a.big_scratch != nullptr) {
    const unsigned grid = (unsigned)std::min<int64_t>(a.n, a.big_blocks);
    hipLaunchKernelGGL((k_cluster_big<T, CPLX, MODE>), dim3(grid), dim3(1024), 0, s, a, (T*)a.big_scratch,
                       a.big_slab);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// k_cluster_lds8_pair with W = 8 or 16 lanes per 8 x 8 cluster.
template <typename T, bool CPLX, int MODE>
hipError_t launch_lds8_pair(const ClusterArgs<T>& a, const ClusterArgs<T>& e, const ClusterArgs<T>& st, int W,
                            hipStream_t s) {
  const int n8 = (int)((a.n + 64 / W - 1) / (64 / W)), nbe = (int)((e.n + 63) / 64), nbs = (int)((st.n + 63) / 64);
  const dim3 g((unsigned)(n8 + nbe + nbs)), b(64);
  if (W == 8) hipLaunchKernelGGL((k_cluster_lds8_pair<T, CPLX, MODE, 8>), g, b, 0, s, a, e, st, n8, nbe);
  else if (W == 16) hipLaunchKernelGGL((k_cluster_lds8_pair<T, CPLX, MODE, 16>), g, b, 0, s, a, e, st, n8, nbe);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// The float Gibbs pass of a 16-dimensional bucket (one wave per cluster) with a bond and a site bucket.
template <typename T, bool CPLX>
hipError_t launch_expm16_pair(const ClusterArgs<T>& a, const ClusterArgs<T>& e, const ClusterArgs<T>& st, hipStream_t s) {
  if (a.De != 16 || e.De != 4 || e.Dc != 2 || st.De != 2 || e.maxch < 1 || e.maxch > 2 || a.fp || e.fp || st.fp)
    return hipErrorInvalidValue;
  const int64_t nbe = grid_for(e.n, 64), nbs = grid_for(st.n, 64);
  if (a.n + nbe + nbs > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_cluster_expm16_pair<T, CPLX>), dim3((unsigned)(a.n + nbe + nbs)), dim3(64), 0, s, a, e, st,
                     (int)nbe, (int)nbs);
  return hipGetLastError();
}

// Entry of the cluster kernels for one (precision, field, mode): explicitly instantiated in
// one translation unit each, so that the kernel families compile in parallel.
template <typename T, bool CPLX, int MODE>
hipError_t launch_cluster_mode(const ClusterArgs<T>& a, int block, int W, hipStream_t s) {
  return launch_cluster_m<T, CPLX, MODE>(a, block, W, s);
}

}  // namespace lrh

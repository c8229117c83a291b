// Small dense complex FP64 problems of FGMRES-DR, each solved by one
// workgroup with its operands in LDS:
//
//   * per Arnoldi step: the implicit residual norm of the small least-squares
//     problem (Section 4.2 and Section 4.6), from a QR factorisation that is
//     carried from step to step: the dense leading block after a deflated
//     restart is factored once by Householder reflections, and every further
//     column, which is of Hessenberg form, adds one Givens rotation;
//   * per cycle: eta = argmin ||c - H^ eta||;
//   * per deflated restart (Lemma 1a, Alg. 4): f from H_m^H f = h_m (LU with
//     partial pivoting), the eigenpairs of H_m + f h_m^H (Householder
//     reduction to Hessenberg form, explicit single-shift QR iteration with
//     Wilkinson shifts, eigenvectors by back substitution in the Schur form),
//     the k eigenvectors of smallest-modulus eigenvalues, G_{k+1}, its QR
//     factorisation and H^_k = Q_{k+1}^H H^ Q_k.
//
// All of it is bound by latency: chains of dependent FP64 operations and LDS
// reads in one workgroup while the rest of the GPU waits. So the chains are
// kept short. Dot products and updates of one row or column go to four lanes
// (a quad), a rotation sweep runs in registers with its scalars read across
// lanes, and serial steps (pivots, shifts) are computed redundantly by every
// wavefront from the same LDS data, so that control flow is uniform over the
// workgroup. Measured at m = 30, k = 10 (us per call): deflated restart 1350
// -> 575, Arnoldi step 50 -> 8, least squares 113 -> 14; at
// m = 20, k = 5: 637 -> 290, 20 -> 4, 47 -> 7.
#include "dw_control.hpp"
#include "dw_kernels.hpp"
#include "dw_types.hpp"

namespace dw {

namespace {

using C = cplx<double>;
constexpr int kL = 64;   // lanes of a wavefront
constexpr int kT = 256;  // threads of a workgroup
// leading dimension of matrices in LDS: with 52 (832 bytes) the four rows (or
// columns) of four neighbouring quads fall into 16 different 16-byte banks
constexpr int kLs = 52;
static_assert(kLs >= kLd, "LDS leading dimension");

__device__ __forceinline__ double cabs(C a) { return sqrt(a.re * a.re + a.im * a.im); }
__device__ __forceinline__ double abs1(C a) { return fabs(a.re) + fabs(a.im); }
__device__ __forceinline__ C cdiv(C a, C b) {
  const double d = b.re * b.re + b.im * b.im;
  return C{(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}
__device__ __forceinline__ C csqrt_(C z) {
  const double r = cabs(z);
  const double re = sqrt(0.5 * (r + z.re));
  double im = sqrt(0.5 * fmax(r - z.re, 0.0));
  if (z.im < 0) im = -im;
  return C{re, im};
}
__device__ __forceinline__ C quad_total(C a) { return C{dw::quad_total(a.re), dw::quad_total(a.im)}; }
__device__ __forceinline__ C lane_value(C v, int lane) { return C{dw::lane_value(v.re, lane), dw::lane_value(v.im, lane)}; }
__device__ __forceinline__ C ldc(const double* p, long long i) { return C{p[2 * i], p[2 * i + 1]}; }
__device__ __forceinline__ void stc(double* p, long long i, C v) {
  p[2 * i] = v.re;
  p[2 * i + 1] = v.im;
}

// 1 / sqrt(t): the hardware estimate (about 24 bits) and one third-order step
__device__ __forceinline__ double rsqrt_(double t) {
  double r = __builtin_amdgcn_rsq(t);
  const double e = fma(-t * r, r, 1.0);
  return fma(r * e, fma(0.375, e, 0.5), r);
}

// Rotation [[conj(a), conj(b)], [-b, a]] that takes (x, y) to (rho, 0),
// rho = sqrt(|x|^2 + |y|^2) real; the identity for x = y = 0.
__device__ __forceinline__ void rotation(C x, C y, C& a, C& b) {
  const double t = fma(x.re, x.re, fma(x.im, x.im, fma(y.re, y.re, y.im * y.im)));
  if (t > 1e-280) {
    const double r = rsqrt_(t);
    a = r * x;
    b = r * y;
  } else {  // too small to square
    const double ax = fmax(fmax(fabs(x.re), fabs(x.im)), fmax(fabs(y.re), fabs(y.im)));
    a = C{1.0, 0.0};
    b = C{0.0, 0.0};
    if (ax > 0) {
      const C xs = C{x.re / ax, x.im / ax}, ys = C{y.re / ax, y.im / ax};
      const double r = 1.0 / sqrt(norm2(xs) + norm2(ys));
      a = r * xs;
      b = r * ys;
    }
  }
}
__device__ __forceinline__ C rot_up(C a, C b, C x, C y) { return cdot(a, x) + cdot(b, y); }
__device__ __forceinline__ C rot_dn(C a, C b, C x, C y) { return a * y - b * x; }

// Householder QR in place of A (rows x cols, column-major, leading dim kLs),
// the reflections applied to columns cols..all-1 and rhs (may be null) too.
// Reflector r is stored in column r of Uv (entries r..rows-1) with beta[r];
// P_r = I - beta_r u_r u_r^H. rows <= 64, all <= 63. One quad per column.
__device__ void hh_qr(C* A, int rows, int cols, int all, C* rhs, C* Uv, double* beta) {
  const int lane = threadIdx.x % kL, quad = threadIdx.x / 4, part = threadIdx.x % 4;
  for (int k = 0; k < cols && k < rows; ++k) {
    const C x = lane < rows ? A[lane + k * kLs] : C{0, 0};
    const double nrm2 = wave_total(lane >= k ? norm2(x) : 0.0);
    const C x0 = A[k + k * kLs];
    const double nrm = sqrt(nrm2);
    const double ax0 = cabs(x0);
    const C ph = ax0 > 0 ? C{x0.re / ax0, x0.im / ax0} : C{1.0, 0.0};
    const C alpha = C{-ph.re * nrm, -ph.im * nrm};
    const C u0 = x0 - alpha;
    const double un2 = nrm2 - ax0 * ax0 + norm2(u0);
    const double bk = (nrm > 0 && un2 > 0) ? 2.0 / un2 : 0.0;
    if (threadIdx.x < rows) Uv[lane + k * kLs] = lane < k ? C{0, 0} : (lane == k ? u0 : x);
    if (threadIdx.x == 0) beta[k] = bk;
    __syncthreads();  // reflector visible; column k read by every wavefront
    if (bk != 0.0) {
      C* col = quad > k && quad < all ? A + quad * kLs : (quad == kT / 4 - 1 ? rhs : nullptr);
      if (col) {
        C s{0, 0};
        for (int i = k + part; i < rows; i += 4) s += cdot(Uv[i + k * kLs], col[i]);
        s = bk * quad_total(s);
        for (int i = k + part; i < rows; i += 4) col[i] -= Uv[i + k * kLs] * s;
      }
      if (threadIdx.x < rows && lane >= k) A[lane + k * kLs] = lane == k ? alpha : C{0, 0};
    }
    __syncthreads();
  }
}

// R eta = rhs(0:cols) by back substitution, R = upper part of A; lane i holds
// unknown i (every wavefront computes the same)
__device__ void back_subst(const C* A, int cols, const C* rhs, C* eta) {
  const int lane = threadIdx.x % kL;
  C r{0, 0}, inv{0, 0};
  if (lane < cols) {
    r = rhs[lane];
    const C d = A[lane + lane * kLs];
    if (!(d.re == 0 && d.im == 0)) inv = cdiv(C{1.0, 0.0}, d);
  }
  __syncthreads();  // eta may be rhs
  C next = lane < cols ? A[lane + (cols - 1) * kLs] : C{0, 0};
  for (int i = cols - 1; i >= 0; --i) {
    const C a = next;
    if (i > 0 && lane < cols) next = A[lane + (i - 1) * kLs];
    const C e = lane_value(r * inv, i);
    if (lane == i) r = e;
    else if (lane < i) r -= a * e;
  }
  if (threadIdx.x < cols) eta[lane] = r;
  __syncthreads();
}

constexpr int kQCols = 25;       // at most k + 1 = 25 columns of Q
constexpr int kQd = 24;          // leading dimension of the leading block's Q^H

// The QR factorisation carried through a cycle (device memory, complex units;
// kept in the buffer of Q_{k+1}, which is written and read between cycles):
// Q^H of the (K+1) x K leading block, the rotations of columns K.. (a, b), the
// right-hand side after the rotations of the final columns, and the sum of
// squares of the final columns (real part).
enum { kStQ = 0, kStA = kQd * kQd, kStB = kStA + kMaxM, kStG = kStB + kMaxM, kStF = kStG + kLd, kStCount = kStF + 1 };
static_assert(kStCount <= kLd * kQCols, "the carried factorisation fits in the buffer of Q");

struct StepSmem {
  C A[kLs * kMaxM];
  C Uv[kLs * kMaxM];
  C rhs[kLd + 1];
  C eta[kLd + 1];
  double beta[kMaxM];
  C Q[kQd * kQd];
  C a[kMaxM], b[kMaxM];
  double red[kT / kL];
};

// Completes Arnoldi step j of a cycle whose first column is K: the norm of the
// new vector from its G partial sums, breakdown test, implicit residual.
// Column j-1 got its second-pass correction in this step and is final now, so
// its rotation is computed and kept; column j is provisional.
__global__ void __launch_bounds__(kT) k_step2(double* H, int j, int K, const double* __restrict__ partials, int G,
                                              const double* c, double* scal, double bd_tol, int* ctl,
                                              const double* ctld, double* st) {
  if (ctl && ctl[kCLive] == 0) return;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  StepSmem& S = *reinterpret_cast<StepSmem*>(smem_raw);
  const int t = threadIdx.x, lane = t % kL;
  const bool first = j == K;
  double part = 0;
  for (int g = t; g < G; g += kT) part += partials[2 * g];
  part = wave_total(part);
  if (lane == 0) S.red[t / kL] = part;
  // columns j-1 and j into rows of eta's neighbours: Uv columns 0 and 1
  C* y0 = S.Uv;
  C* y1 = S.Uv + kLs;
  if (first && K > 0) {
    // leading block, followed by the identity, which becomes Q^H
    for (int q = t; q < (K + 1) * (2 * K + 1); q += kT) {
      const int i = q % (K + 1), col = q / (K + 1);
      S.A[i + col * kLs] = col < K ? ldc(H, i + (long long)col * kLd) : C{col - K == i ? 1.0 : 0.0, 0.0};
    }
    if (t <= K) S.rhs[t] = ldc(c, t);
  } else if (!first) {
    for (int q = t; q < (K + 1) * (K + 1); q += kT) {
      const int i = q % (K + 1), col = q / (K + 1);
      S.Q[i + col * kQd] = ldc(st, kStQ + i + col * kQd);
    }
    for (int q = K + t; q <= j - 2; q += kT) {
      S.a[q] = ldc(st, kStA + q);
      S.b[q] = ldc(st, kStB + q);
    }
  } else if (t == 0) {
    S.Q[0] = C{1.0, 0.0};
  }
  __syncthreads();
  double nrm2 = 0;
  for (int w = 0; w < kT / kL; ++w) nrm2 += S.red[w];
  const double hn = sqrt(fmax(nrm2, 0.0));
  double hf2 = 0;
  if (first) {
    if (K > 0) {
      for (int q = lane; q < (K + 1) * K; q += kL) hf2 += norm2(S.A[q % (K + 1) + (q / (K + 1)) * kLs]);
      hf2 = wave_total(hf2);
      __syncthreads();
      hh_qr(S.A, K + 1, K, 2 * K + 1, S.rhs, S.Uv, S.beta);
      for (int q = t; q < (K + 1) * (K + 1); q += kT) {
        const int i = q % (K + 1), col = q / (K + 1);
        const C v = S.A[i + (K + col) * kLs];
        S.Q[i + col * kQd] = v;
        stc(st, kStQ + i + col * kQd, v);
      }
      __syncthreads();
    }
    if (t < kLd) S.eta[t] = K > 0 && t <= K ? S.rhs[t] : ldc(c, t);
    if (t < kLd) stc(st, kStG + t, S.eta[t]);
    if (t == 0) stc(st, kStF, C{hf2, 0.0});
  } else {
    if (t < kLd) S.eta[t] = ldc(st, kStG + t);
    hf2 = st[2 * kStF];
  }
  C h0{0, 0}, h1{0, 0};
  if (!first && lane <= j) h0 = ldc(H, lane + (long long)(j - 1) * kLd);
  if (lane <= j) h1 = ldc(H, lane + (long long)j * kLd);
  if (lane == j + 1) h1 = C{hn, 0.0};
  if (t < kLs) {
    y0[t] = h0;
    y1[t] = h1;
  }
  if (t == 0) stc(H, j + 1 + (long long)j * kLd, C{hn, 0.0});
  const double f0 = wave_total(norm2(h0)), f1 = wave_total(norm2(h1));
  __syncthreads();
  if (t >= kL) return;  // one wavefront from here on; no barrier follows
  // lanes 0..31: column j-1, lanes 32..63: column j
  const C* y = lane < 32 ? y0 : y1;
  const int i = lane % 32;
  C v = i <= K ? y[i] : C{0, 0};
  if (K > 0) {
    v = C{0, 0};
    if (i <= K)
#pragma unroll 4
      for (int q = 0; q <= K; ++q) v += S.Q[i + q * kQd] * y[q];
  }
  const C v0 = lane_value(v, K), v1 = lane_value(v, 32 + K);
  C u = lane < 32 ? v0 : v1;  // running entry, row K
#pragma unroll 4
  for (int q = K; q <= j - 2; ++q) u = rot_dn(S.a[q], S.b[q], u, y[q + 1]);
  C a0{1, 0}, b0{0, 0}, u1 = lane_value(u, 32);
  C gj = S.eta[j];  // entry j of the right-hand side
  if (!first) {
    const C x0 = lane_value(u, 0);
    rotation(x0, y0[j], a0, b0);
    u1 = rot_dn(a0, b0, u1, y1[j]);
    const C gu = S.eta[j - 1];
    if (lane == 0) {
      stc(st, kStA + j - 1, a0);
      stc(st, kStB + j - 1, b0);
      stc(st, kStG + j - 1, rot_up(a0, b0, gu, gj));
    }
    gj = rot_dn(a0, b0, gu, gj);
    if (lane == 0) {
      stc(st, kStG + j, gj);
      stc(st, kStF, C{hf2 + f0, 0.0});
    }
  }
  C a1, b1;
  rotation(u1, C{hn, 0.0}, a1, b1);
  const double ri = cabs(rot_dn(a1, b1, gj, S.eta[j + 1]));
  const bool broke = !(hn > bd_tol * sqrt(hf2 + f0 + f1));
  if (lane == 0) {
    scal[kSclHnext] = hn;
    scal[kSclHinv] = broke ? 0.0 : 1.0 / hn;
    scal[kSclResImp] = ri;
    scal[kSclBreak] = broke ? 1.0 : 0.0;
    if (ctl) {
      ctl[kCJend] = j + 1;
      ctl[kCBroke] = broke ? 1 : 0;
      if (broke || ri <= ctld[kDTolAbs] || j + 1 >= ctl[kCJlim]) ctl[kCLive] = 0;
    }
  }
}

// eta = argmin ||c - H^ eta||. With st: the factorisation carried through the
// cycle (k_step2) gives R, all columns but the last being rotated in parallel;
// the cycle's first column is dK. Without: Householder QR of a dense H^.
__global__ void __launch_bounds__(kT) k_lsq(const double* H, int cols, const double* c, double* eta, double* scal,
                                            const int* gate, const int* dn, const double* st, const int* dK) {
  if (gate && *gate == 0) return;
  if (dn) cols = *dn;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  StepSmem& S = *reinterpret_cast<StepSmem*>(smem_raw);
  const int t = threadIdx.x, lane = t % kL;
  const int rows = cols + 1;
  for (int q = t; q < rows * cols; q += kT) {
    const int i = q % rows, col = q / rows;
    S.A[i + col * kLs] = ldc(H, i + (long long)col * kLd);
  }
  if (!st) {
    if (t < rows) S.rhs[t] = ldc(c, t);
    __syncthreads();
    hh_qr(S.A, rows, cols, cols, S.rhs, S.Uv, S.beta);
    const double ri = cabs(S.rhs[rows - 1]);
    back_subst(S.A, cols, S.rhs, S.eta);
    if (t < cols) stc(eta, t, S.eta[t]);
    if (t == 0) scal[kSclResImp] = ri;
    return;
  }
  const int K = *dK;
  for (int q = t; q < (K + 1) * (K + 1); q += kT) {
    const int i = q % (K + 1), col = q / (K + 1);
    S.Q[i + col * kQd] = K > 0 ? ldc(st, kStQ + i + col * kQd) : C{1.0, 0.0};
  }
  for (int q = K + t; q <= cols - 2; q += kT) {
    S.a[q] = ldc(st, kStA + q);
    S.b[q] = ldc(st, kStB + q);
  }
  if (t < kLd) S.rhs[t] = ldc(st, kStG + t);
  __syncthreads();
  // leading rows 0..K: Q^H times every column (into Uv, then back)
  if (K > 0) {
    for (int q = t; q < (K + 1) * cols; q += kT) {
      const int i = q % (K + 1), col = q / (K + 1);
      C v{0, 0};
#pragma unroll 4
      for (int p = 0; p <= K; ++p) v += S.Q[i + p * kQd] * S.A[p + col * kLs];
      S.Uv[i + col * kLs] = v;
    }
    __syncthreads();
    for (int q = t; q < (K + 1) * cols; q += kT) {
      const int i = q % (K + 1), col = q / (K + 1);
      S.A[i + col * kLs] = S.Uv[i + col * kLs];
    }
    __syncthreads();
  }
  double ri = 0;
  if (t < cols && t >= K) {  // column t: rotations K..t (the last column's own one follows)
    C* col = S.A + t * kLs;
    C u = col[K];
    const int qe = t < cols - 1 ? t : cols - 2;
    for (int q = K; q <= qe; ++q) {
      const C z = col[q + 1];
      col[q] = rot_up(S.a[q], S.b[q], u, z);
      u = rot_dn(S.a[q], S.b[q], u, z);
    }
    if (t == cols - 1) {
      C a, b;
      const C z = col[cols];
      rotation(u, z, a, b);
      col[cols - 1] = rot_up(a, b, u, z);
      const C g0 = S.rhs[cols - 1], g1 = S.rhs[cols];
      S.rhs[cols - 1] = rot_up(a, b, g0, g1);
      ri = cabs(rot_dn(a, b, g0, g1));
      scal[kSclResImp] = ri;
    }
  }
  __syncthreads();
  back_subst(S.A, cols, S.rhs, S.eta);
  if (t < cols) stc(eta, lane, S.eta[lane]);
}

// Projection onto a deflation space (D Z_k = V_{k+1} H_k): y = argmin ||t - H_k y||
// and s = H_k y, with H_k the (k+1) x k leading block of H.
__global__ void __launch_bounds__(kT) k_project(const double* H, int k, const double* tv, double* y, double* sv,
                                                const int* gate) {
  if (gate && *gate == 0) return;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  StepSmem& S = *reinterpret_cast<StepSmem*>(smem_raw);
  const int t = threadIdx.x;
  const int rows = k + 1;
  for (int q = t; q < rows * k; q += kT) {
    const int i = q % rows, c = q / rows;
    S.A[i + c * kLs] = ldc(H, i + (long long)c * kLd);
  }
  if (t < rows) S.rhs[t] = ldc(tv, t);
  __syncthreads();
  hh_qr(S.A, rows, k, k, S.rhs, S.Uv, S.beta);
  back_subst(S.A, k, S.rhs, S.eta);
  if (t < k) stc(y, t, S.eta[t]);
  if (t < rows) {
    C acc{0, 0};
    for (int c = 0; c < k; ++c) acc += ldc(H, t + (long long)c * kLd) * S.eta[c];
    stc(sv, t, acc);
  }
}

__global__ void __launch_bounds__(kT) k_fresh(double* H, double* c, const double* nrm2, double* scal,
                                              const int* gate) {
  if (gate && *gate == 0) return;
  const double beta = sqrt(fmax(nrm2[0], 0.0));
  for (int t = threadIdx.x; t < kLd * kMaxM; t += kT) stc(H, t, C{0, 0});
  for (int t = threadIdx.x; t < kLd; t += kT) stc(c, t, C{t == 0 ? beta : 0.0, 0.0});
  if (threadIdx.x == 0) {
    scal[kSclBeta] = beta;
    scal[kSclBetaInv] = beta > 0 ? 1.0 / beta : 0.0;
  }
}

struct DeflSmem {
  C Hs[kLs * kMaxM];    // H^ (mm+1) x mm
  C A[kLs * kMaxM];     // B = H_m^H, then H_m + f h^H, its Schur form T, then G_{k+1}, then H^ Q_k
  C Zm[kLs * kMaxM];    // Schur vectors, then Householder vectors of G_{k+1}
  C Qs[kLs * kQCols];   // eigenvectors of T (k x mm), then Q_{k+1}
  C f[kMaxM];
  C u[kLd];
  C lam[kMaxM];
  C eta[kMaxM];
  C ra[kMaxM], rb[kMaxM];  // rotations of one QR sweep
  double beta[kQCols];
  double mod[kMaxM];
  int order[kMaxM];
};

__global__ void __launch_bounds__(kT)
    k_deflate(double* H, int mm, int k, const double* c, const double* etag, double* Qg, double* ritz, double* scal,
              const int* gate, const int* dn) {
  if (gate && *gate == 0) return;
  if (dn) mm = *dn < mm ? *dn : mm;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  DeflSmem& S = *reinterpret_cast<DeflSmem*>(smem_raw);
  const int t = threadIdx.x, lane = t % kL, wave = t / kL, quad = t / 4, part = t % 4;
  const int n = mm;
  const double eps = 2.220446049250313e-16;

  // ---- 1. load H^ and eta
  for (int q = t; q < (mm + 1) * mm; q += kT) {
    const int i = q % (mm + 1), col = q / (mm + 1);
    S.Hs[i + col * kLs] = ldc(H, i + (long long)col * kLd);
  }
  if (t < mm) S.eta[t] = ldc(etag, t);
  __syncthreads();

  // ---- 2. f: H_m^H f = h_m with h_m = conj(last row of H^)
  for (int q = t; q < n * n; q += kT) {
    const int i = q % n, col = q / n;
    S.A[i + col * kLs] = conj(S.Hs[col + i * kLs]);
  }
  if (t < n) S.f[t] = conj(S.Hs[mm + t * kLs]);
  __syncthreads();
  double bmax = 0;
  for (int q = lane; q < n * n; q += kL) bmax = fmax(bmax, norm2(S.A[q % n + (q / n) * kLs]));
  bmax = sqrt(wave_largest(bmax));
  int status = 0;
  for (int q = 0; q < n; ++q) {
    // pivot: the first row of the largest modulus
    const double mine = lane >= q && lane < n ? norm2(S.A[lane + q * kLs]) : -1.0;
    const double best = wave_largest(mine);
    const unsigned long long at = __ballot(mine == best);
    const int p = at ? __ffsll(at) - 1 : q;  // none: a NaN, caught by the test below
    const C piv = S.A[p + q * kLs];
    if (!(cabs(piv) > 1e-14 * bmax)) {
      status = 1;
      break;
    }
    __syncthreads();  // column q read by every wavefront
    if (p != q) {
      if (t < n) {
        const C t0 = S.A[q + t * kLs];
        S.A[q + t * kLs] = S.A[p + t * kLs];
        S.A[p + t * kLs] = t0;
      } else if (t == kT - 1) {
        const C t0 = S.f[q];
        S.f[q] = S.f[p];
        S.f[p] = t0;
      }
      __syncthreads();
    }
    if (quad > q && quad < n) {  // row `quad`
      const C lq = cdiv(S.A[quad + q * kLs], piv);
      for (int jj = q + 1 + part; jj < n; jj += 4) S.A[quad + jj * kLs] -= lq * S.A[q + jj * kLs];
      if (part == 0) S.f[quad] -= lq * S.f[q];
    }
    __syncthreads();
  }
  if (status == 0) back_subst(S.A, n, S.f, S.f);

  // ---- 3. A = H_m + f h_m^H (h_m^H is the last row of H^), Zm = I
  if (status == 0) {
    for (int q = t; q < n * n; q += kT) {
      const int i = q % n, col = q / n;
      S.A[i + col * kLs] = S.Hs[i + col * kLs] + S.f[i] * S.Hs[mm + col * kLs];
      S.Zm[i + col * kLs] = C{i == col ? 1.0 : 0.0, 0.0};
    }
    __syncthreads();
    // ---- 4. Householder reduction to upper Hessenberg form, A <- P A P, Zm <- Zm P
    for (int q = 0; q + 2 < n; ++q) {
      const C x = lane < n ? S.A[lane + q * kLs] : C{0, 0};
      const double nrm2 = wave_total(lane > q ? norm2(x) : 0.0);
      const C x0 = S.A[q + 1 + q * kLs];
      const double nrm = sqrt(nrm2), ax0 = cabs(x0);
      const C ph = ax0 > 0 ? C{x0.re / ax0, x0.im / ax0} : C{1.0, 0.0};
      const C alpha = C{-ph.re * nrm, -ph.im * nrm};
      const C u0 = x0 - alpha;
      const double un2 = nrm2 - ax0 * ax0 + norm2(u0);
      if (!(nrm > 0 && un2 > 0)) continue;  // the same for every wavefront; nothing written since the last barrier
      const double bq = 2.0 / un2;
      if (t < n) S.u[t] = t <= q ? C{0, 0} : (t == q + 1 ? u0 : x);
      __syncthreads();  // u visible; column q read by every wavefront
      if (quad > q && quad < n) {  // left: column `quad`
        C s{0, 0};
        for (int i = q + 1 + part; i < n; i += 4) s += cdot(S.u[i], S.A[i + quad * kLs]);
        s = bq * quad_total(s);
        for (int i = q + 1 + part; i < n; i += 4) S.A[i + quad * kLs] -= S.u[i] * s;
      }
      if (t > q && t < n) S.A[t + q * kLs] = t == q + 1 ? alpha : C{0, 0};  // column q itself
      __syncthreads();
      for (int row = quad; row < 2 * n; row += kT / 4) {  // right: rows of A, then of Zm
        C* M = row < n ? S.A + row : S.Zm + (row - n);
        C s{0, 0};
        for (int jj = q + 1 + part; jj < n; jj += 4) s += M[jj * kLs] * S.u[jj];
        s = bq * quad_total(s);
        for (int jj = q + 1 + part; jj < n; jj += 4) M[jj * kLs] -= s * conj(S.u[jj]);
      }
      __syncthreads();
    }

    // ---- 5. QR iteration with explicit single shifts to upper triangular T.
    // One sweep: A - mu I = Q R by rotations, one wavefront with a lane per
    // column, the running row in registers and the rotation's two entries
    // read across lanes; then R Q + mu I and Zm Q, a lane per row.
    double anorm = 0;
    for (int q = lane; q < n * n; q += kL) anorm = fmax(anorm, abs1(S.A[q % n + (q / n) * kLs]));
    anorm = wave_largest(anorm);
    int hi = n - 1, its = 0, total = 0;
    while (hi > 0) {
      // the active block l..hi starts at the last negligible subdiagonal
      bool neg = false;
      if (lane > 0 && lane <= hi) {
        double sc = abs1(S.A[lane - 1 + (lane - 1) * kLs]) + abs1(S.A[lane + lane * kLs]);
        if (sc == 0) sc = anorm;
        neg = abs1(S.A[lane + (lane - 1) * kLs]) <= eps * sc;
      }
      const unsigned long long mask = __ballot(neg);
      const int l = mask ? 63 - __clzll(mask) : 0;
      if (l == hi) {
        --hi;
        its = 0;
        continue;
      }
      if (++total > 60 * n) {
        status = 2;
        break;
      }
      ++its;
      C mu;
      const C a = S.A[hi - 1 + (hi - 1) * kLs], b = S.A[hi - 1 + hi * kLs];
      const C cc = S.A[hi + (hi - 1) * kLs], d = S.A[hi + hi * kLs];
      if (its % 11 == 10) {
        // exceptional shift to break cycles
        mu = d + C{0.75 * cabs(cc), 0.0};
      } else {
        const C th = 0.5 * (a - d);
        const C disc = csqrt_(th * th + b * cc);
        const C m1 = th + disc, m2 = th - disc;
        mu = d + (norm2(m1) < norm2(m2) ? m1 : m2);
      }
      __syncthreads();  // every wavefront has read the block
      if (wave == 0) {
        const bool on = lane >= l && lane < n;
        C top{0, 0}, nxt{0, 0};
        if (on) {
          top = S.A[l + lane * kLs];
          nxt = S.A[l + 1 + lane * kLs];
        }
        if (lane == l) top -= mu;
        if (l > 0 && lane == 0) S.A[l + (l - 1) * kLs] = C{0, 0};
        for (int q = l; q < hi; ++q) {
          C ahead{0, 0};
          if (on && q + 2 <= hi) ahead = S.A[q + 2 + lane * kLs];
          if (lane == q + 1) nxt -= mu;
          C ra, rb;
          rotation(lane_value(top, q), lane_value(nxt, q), ra, rb);
          if (on) {
            if (lane >= q) S.A[q + lane * kLs] = rot_up(ra, rb, top, nxt);
            if (lane == q) S.A[q + 1 + q * kLs] = C{0, 0};
          }
          if (lane == 0) {
            S.ra[q] = ra;
            S.rb[q] = rb;
          }
          top = rot_dn(ra, rb, top, nxt);
          nxt = ahead;
        }
        if (on && lane >= hi) S.A[hi + lane * kLs] = top;
      }
      __syncthreads();
      if (wave == 0 ? lane <= hi : (wave == 1 && lane < n)) {
        C* M = wave == 0 ? S.A + lane : S.Zm + lane;
        const bool act = wave == 0 && lane >= l;  // rows of the active block get the shift back
        C cur = M[l * kLs], nxt = M[(l + 1) * kLs];
        for (int q = l; q < hi; ++q) {
          C ahead{0, 0};
          if (q + 2 <= hi) ahead = M[(q + 2) * kLs];
          const C ra = S.ra[q], rb = S.rb[q];
          C v = cur * ra + nxt * rb;
          if (act && lane == q) v += mu;
          M[q * kLs] = v;
          cur = cdot(ra, nxt) - cdot(rb, cur);
          nxt = ahead;
        }
        if (act && lane == hi) cur += mu;
        M[hi * kLs] = cur;
      }
      __syncthreads();
    }
  }

  // ---- 6. eigenvalues, stable sort by modulus
  __syncthreads();
  if (status == 0) {
    if (t < n) {
      S.lam[t] = S.A[t + t * kLs];
      S.mod[t] = cabs(S.lam[t]);
    }
    __syncthreads();
    bool nan = false;
    if (lane < n) {
      const double me = S.mod[lane];
      nan = !(me == me);
      int rank = 0;
#pragma unroll 8
      for (int i = 0; i < n; ++i) {
        const double o = S.mod[i];
        if (o < me || (o == me && i < lane)) ++rank;
      }
      if (wave == 0) S.order[rank] = lane;
    }
    if (__ballot(nan)) status = 3;
    __syncthreads();
  }

  if (status == 0) {
    // ---- 7. eigenvectors of T for the k smallest: quad qv back-substitutes,
    // lane `part` of it owning the entries i = part (mod 4)
    double tnorm = 0;
    for (int q = lane; q < n * n; q += kL) tnorm = fmax(tnorm, norm2(S.A[q % n + (q / n) * kLs]));
    const double smin = fmax(eps * sqrt(wave_largest(tnorm)), 1e-300);
    if (quad < k) {
      const int p = S.order[quad];
      const C lp = S.lam[p];
      C* y = S.Qs + quad * kLs;
      for (int i = part; i < n; i += 4) y[i] = C{i == p ? 1.0 : 0.0, 0.0};
      for (int i = p - 1; i >= 0; --i) {
        C s{0, 0};
        for (int jj = i + 1 + ((part - (i + 1)) & 3); jj <= p; jj += 4) s += S.A[i + jj * kLs] * y[jj];
        s = quad_total(s);
        C den = S.A[i + i * kLs] - lp;
        if (cabs(den) < smin) den = C{smin, 0.0};
        if ((i & 3) == part) y[i] = -cdiv(s, den);
      }
    }
    __syncthreads();
    // G_k = Zm Y into A as the first k columns of G_{k+1} ((mm+1) x (k+1))
    for (int q = t; q < (n + 1) * k; q += kT) {
      const int i = q % (n + 1), qv = q / (n + 1);
      const int p = S.order[qv];
      const C* y = S.Qs + qv * kLs;
      C s{0, 0};
      if (i < n)
#pragma unroll 4
        for (int jj = 0; jj <= p; ++jj) s += S.Zm[i + jj * kLs] * y[jj];
      S.A[i + qv * kLs] = s;
    }
    __syncthreads();
    for (int qv = wave; qv < k; qv += kT / kL) {
      const C v = lane < n ? S.A[lane + qv * kLs] : C{0, 0};
      const double nn = wave_total(norm2(v));
      const double inv = nn > 0 ? 1.0 / sqrt(nn) : 0.0;
      if (lane < n) S.A[lane + qv * kLs] = inv * v;
    }
    // ---- 8. last column: the small residual c - H^ eta
    if (t <= mm) {
      C s = ldc(c, t);
#pragma unroll 4
      for (int jj = 0; jj < mm; ++jj) s -= S.Hs[t + jj * kLs] * S.eta[jj];
      S.A[t + k * kLs] = s;
    }
    __syncthreads();
    // ---- 9. QR of G_{k+1}; reflectors into Zm, explicit Q_{k+1} into Qs (lane
    // `part` of a column's quad owns the entries i = part (mod 4))
    hh_qr(S.A, mm + 1, k + 1, k + 1, nullptr, S.Zm, S.beta);
    if (quad <= k) {
      C* col = S.Qs + quad * kLs;
      for (int i = part; i <= mm; i += 4) col[i] = C{i == quad ? 1.0 : 0.0, 0.0};
      for (int r = k; r >= 0; --r) {
        const double br = S.beta[r];
        if (br == 0.0) continue;
        C sacc{0, 0};
        for (int i = r + ((part - r) & 3); i <= mm; i += 4) sacc += cdot(S.Zm[i + r * kLs], col[i]);
        sacc = br * quad_total(sacc);
        for (int i = r + ((part - r) & 3); i <= mm; i += 4) col[i] -= S.Zm[i + r * kLs] * sacc;
      }
    }
    __syncthreads();
    // ---- 10. H^_k = Q^H H^ Q_k (Q_k = Q(0:mm-1, 0:k-1)); T1 = H^ Q_k into A
    for (int q = t; q < (mm + 1) * k; q += kT) {
      const int i = q % (mm + 1), cq = q / (mm + 1);
      C s{0, 0};
#pragma unroll 4
      for (int jj = 0; jj < mm; ++jj) s += S.Hs[i + jj * kLs] * S.Qs[jj + cq * kLs];
      S.A[i + cq * kLs] = s;
    }
    __syncthreads();
    for (int q = t; q < kLd * kMaxM; q += kT) {
      const int i = q % kLd, cq = q / kLd;
      C s{0, 0};
      if (i <= k && cq < k)
#pragma unroll 4
        for (int jj = 0; jj <= mm; ++jj) s += cdot(S.Qs[jj + i * kLs], S.A[jj + cq * kLs]);
      stc(H, q, s);
    }
    for (int q = t; q < (mm + 1) * (k + 1); q += kT) {
      const int i = q % (mm + 1), col = q / (mm + 1);
      stc(Qg, i + (long long)col * kLd, S.Qs[i + col * kLs]);
    }
    if (t < n) stc(ritz, t, S.lam[S.order[t]]);
  }
  if (t == 0) scal[kSclStatus] = (double)status;
}

template <typename K>
dw_status set_lds(K kernel, size_t bytes) {
  if (bytes > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) {
      set_error("hipFuncSetAttribute(LDS %zu) failed: %s", bytes, hipGetErrorString(e));
      return DW_EHIP;
    }
  }
  return DW_OK;
}

}  // namespace

dw_status dense_lsq(const double* H, int cols, const double* c, double* eta, double* scal, hipStream_t s,
                    const int* gate, const int* dn, const double* qr, const int* dK) {
  if (cols < 1 || cols > kMaxM || (qr && !dK)) {
    set_error("dense_lsq: %d columns out of range", cols);
    return DW_EINVAL;
  }
  DW_TRY(set_lds(k_lsq, sizeof(StepSmem)));
  KTimer kt(DW_K_DENSE, s);
  hipLaunchKernelGGL(k_lsq, 1, kT, sizeof(StepSmem), s, H, cols, c, eta, scal, gate, dn, qr, dK);
  DW_CHECK_LAUNCH();
  kt.done(0, 0);
  return DW_OK;
}

dw_status dense_project(const double* H, int k, const double* t, double* y, double* sv, hipStream_t s,
                        const int* gate) {
  if (k < 1 || k >= kMaxM) {
    set_error("dense_project: k = %d out of range", k);
    return DW_EINVAL;
  }
  DW_TRY(set_lds(k_project, sizeof(StepSmem)));
  KTimer kt(DW_K_DENSE, s);
  hipLaunchKernelGGL(k_project, 1, kT, sizeof(StepSmem), s, H, k, t, y, sv, gate);
  DW_CHECK_LAUNCH();
  kt.done(0, 0);
  return DW_OK;
}

dw_status dense_deflate(double* H, int mm, int k, const double* c, const double* eta, double* Q, double* ritz,
                        double* scal, hipStream_t s, const int* gate, const int* dn) {
  if (mm < 1 || mm > kMaxM || k < 1 || k >= mm || k + 1 > kQCols) {
    set_error("dense_deflate: unsupported sizes mm %d, k %d", mm, k);
    return DW_EINVAL;
  }
  DW_TRY(set_lds(k_deflate, sizeof(DeflSmem)));
  KTimer kt(DW_K_DENSE, s);
  hipLaunchKernelGGL(k_deflate, 1, kT, sizeof(DeflSmem), s, H, mm, k, c, eta, Q, ritz, scal, gate, dn);
  DW_CHECK_LAUNCH();
  kt.done(0, 0);
  return DW_OK;
}

dw_status dense_step2(double* H, int j, int j0, const double* partials, int nparts, const double* c, double* scal,
                      double bd_tol, hipStream_t s, double* qr, int* ctl, const double* ctld) {
  if (j < 0 || j >= kMaxM || j0 < 0 || j0 > j || j0 >= kQd) {
    set_error("dense_step2: column %d (first %d) out of range", j, j0);
    return DW_EINVAL;
  }
  DW_TRY(set_lds(k_step2, sizeof(StepSmem)));
  KTimer kt(DW_K_DENSE, s);
  hipLaunchKernelGGL(k_step2, 1, kT, sizeof(StepSmem), s, H, j, j0, partials, nparts, c, scal, bd_tol, ctl, ctld, qr);
  DW_CHECK_LAUNCH();
  kt.done(0, 0);
  return DW_OK;
}

dw_status dense_fresh(double* H, double* c, const double* nrm2, double* scal, hipStream_t s, const int* gate) {
  KTimer kt(DW_K_DENSE, s);
  hipLaunchKernelGGL(k_fresh, 1, kT, 0, s, H, c, nrm2, scal, gate);
  DW_CHECK_LAUNCH();
  kt.done(0, 0);
  return DW_OK;
}

}  // namespace dw

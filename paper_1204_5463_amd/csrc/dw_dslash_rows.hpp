// The Wilson-Dirac operator with two lanes per site (included by k_dslash.hip).
//
// A hop's half spinor has two rows (upper spin components 0 and 1) that the
// link multiplies independently, and row r needs only spins r and one of the
// lower two (3 - r for x and y, 2 + r for z and t). So each site is handled by
// two lanes, 32 apart in one wavefront, one row each: no projection and no
// spinor read is done twice, the two lanes' reads of a link entry are one
// request, and a lane holds half the accumulators. The lower components that
// row r's hops rebuild are spin 3 - r (x, y hops) and spin 2 + r (z, t hops);
// the two lanes exchange the x/y sum after the y hops and lane r stores spins r
// and 2 + r.
//
// As in the one-lane form the block's spinor is staged in LDS, every link is
// read once by its own site, and U_mu(n)^+ (1 + g_mu) psi(n) is handed over to
// site n + mu through LDS.
//
// CANON: x, y and b in the canonical layout (12 contiguous complex numbers per
// site), so that an application on caller fields needs no packing pass: packing,
// the operator on the internal layout and unpacking moved 2.7 times the bytes
// (32^3x64, 12 right-hand sides: 9097 -> 5263 us per application; 8^4: 22.5 ->
// 12.0 us, one launch for three and no allocation).
//
// Bound: traffic beyond the L2. Counted on 32^3x64 with 12 right-hand sides: 600 B
// read and 193 B written per site and side (432 B would do: spinor in and out, a
// twelfth of the links; the rest are faces and links read again), 3.8 TB/s or 0.78 of
// the copy rate, L2 hits 71%, VALU busy 34% of the SIMD cycles at 3.8 waves per SIMD.
#pragma once

#include "dw_clover.hpp"
#include "dw_internal.hpp"
#include "dw_stencil.hpp"

namespace dw {

namespace rows {

// projection coefficient of hop (MU, forward) for row r: i sigma (IMAG) or sigma
template <int MU>
constexpr bool kImag = MU == 0 || MU == 2;

// p + alpha q with alpha = sigma (i sigma if IMAG)
template <bool IMAG, typename T>
__device__ __forceinline__ cplx<T> proj1(cplx<T> p, T sg, cplx<T> q) {
  if constexpr (IMAG) return mk<T>(fma(-sg, q.im, p.re), fma(sg, q.re, p.im));
  else return mk<T>(fma(sg, q.re, p.re), fma(sg, q.im, p.im));
}
// acc += conj(alpha) g
template <bool IMAG, typename T>
__device__ __forceinline__ void rec1(cplx<T>& acc, T sg, cplx<T> g) {
  if constexpr (IMAG) {
    acc.re = fma(sg, g.im, acc.re);
    acc.im = fma(-sg, g.re, acc.im);
  } else {
    acc.re = fma(sg, g.re, acc.re);
    acc.im = fma(sg, g.im, acc.im);
  }
}
// g = W h (DAG false) or W^+ h
template <bool DAG, typename T>
__device__ __forceinline__ void mul1(const cplx<T> w[9], const cplx<T> h[3], cplx<T> g[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    cplx<T> s = mk<T>(0, 0);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if constexpr (DAG) s += cdot(w[b * 3 + a], h[b]);
      else s += w[a * 3 + b] * h[b];
    }
    g[a] = s;
  }
}

template <typename T>
__device__ __forceinline__ T other_row(T v) { return __shfl_xor(v, 32, 64); }
template <typename T>
__device__ __forceinline__ cplx<T> other_row(cplx<T> v) { return mk<T>(other_row(v.re), other_row(v.im)); }

template <typename T, typename SX, typename SG>
struct Ctx {
  const Geom& g;
  int b, l, r;         // block, local site, row
  bool active;
  T rs;                // +1 for row 0, -1 for row 1
  const int* bc;
  const int* lc;
  long long n;         // canonical site (CANON)
  const SX* xr;
  const SX* xsh;       // LDS: block spinor [12][bvol]
  cplx<T>* pb;         // LDS: handed-over half spinors [6][bvol]
  const SG* U;
};

// spinor component k of the site in neighbouring block position c2/nl
// (internal) or at canonical site nn
template <bool CANON, typename T, typename SX, typename SG>
__device__ __forceinline__ cplx<T> face(const Ctx<T, SX, SG>& c, int nb, int nl, long long nn, int k) {
  if constexpr (CANON) return ld<T>(c.xr + nn * 12 + k);
  else return ld<T>(c.xr + spinor_index(c.g, nb, k, nl));
}

template <int MU, bool CANON, int BS, typename T, typename SX, typename SG>
__device__ __forceinline__ void dir(const Ctx<T, SX, SG>& c, cplx<T> up[3], cplx<T> low[3]) {
  constexpr bool IM = kImag<MU>;
  const Geom& g = c.g;
  // x and y on 4^4 blocks: a row of 16 lanes is an x-y plane, so the products go
  // to the neighbour by a lane shift, without LDS and barriers
  constexpr bool SHIFT = BS == 4 && MU < 2;
  const int bvol = BS ? BS * BS * BS * BS : g.bvol, l = c.l, r = c.r;
  const int bm = BS ? BS : g.B[MU];
  const int st = BS ? (MU == 0 ? 1 : MU == 1 ? BS : MU == 2 ? BS * BS : BS * BS * BS) : g.lstride[MU];
  // alpha of the forward hop is sg (times i for x and z): +i, +-1, +-i, -1
  const T sg = MU == 0 ? (T)1 : MU == 3 ? (T)-1 : c.rs;
  const int ks = 3 * r, kp = MU < 2 ? 9 - 3 * r : 6 + 3 * r;
  long long cst = 1;  // canonical site stride
  if constexpr (CANON) {
#pragma unroll
    for (int d = 0; d < MU; ++d) cst *= g.L[d];
  }
  cplx<T> h[3], v[3], handed[3];
  if (c.active) {
    cplx<T> w[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) w[e] = ld<T>(c.U + gauge_index(g, c.b, MU, e, l));
    // U_mu(n)^+ (1 + g_mu) psi(n) for site n + mu
#pragma unroll
    for (int a = 0; a < 3; ++a)
      h[a] = proj1<IM, T>(ld<T>(c.xsh + (ks + a) * bvol + l), -sg, ld<T>(c.xsh + (kp + a) * bvol + l));
    mul1<true, T>(w, h, v);
    if constexpr (SHIFT) {
      // 256 sites: every lane is active
#pragma unroll
      for (int a = 0; a < 3; ++a) handed[a] = lane_shift<MU, -1>(v[a]);
    } else {
#pragma unroll
      for (int a = 0; a < 3; ++a) c.pb[(ks + a) * bvol + l] = v[a];
    }
    // forward hop (1 - g_mu) U_mu(n) psi(n + mu)
    if (c.lc[MU] < bm - 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a)
        h[a] = proj1<IM, T>(ld<T>(c.xsh + (ks + a) * bvol + l + st), sg, ld<T>(c.xsh + (kp + a) * bvol + l + st));
    } else {
      const bool wrap = c.bc[MU] + 1 == g.N[MU];
      int nb = 0;
      long long nn = 0;
      if constexpr (CANON) {
        nn = c.n + (wrap ? cst * (1 - (long long)g.L[MU]) : cst);
      } else {
        int c2[4] = {c.bc[0], c.bc[1], c.bc[2], c.bc[3]};
        c2[MU] = wrap ? 0 : c.bc[MU] + 1;
        nb = encode_block(g, c2);
      }
      const int nl = l - (bm - 1) * st;
#pragma unroll
      for (int a = 0; a < 3; ++a)
        h[a] = proj1<IM, T>(face<CANON>(c, nb, nl, nn, ks + a), sg, face<CANON>(c, nb, nl, nn, kp + a));
    }
    mul1<false, T>(w, h, v);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      up[a] += v[a];
      rec1<IM, T>(low[a], sg, v[a]);
    }
  }
  if constexpr (!SHIFT) __syncthreads();
  if constexpr (BS == 4) __builtin_amdgcn_sched_barrier(0);
  if (c.active) {
    if (c.lc[MU] > 0) {
#pragma unroll
      for (int a = 0; a < 3; ++a) v[a] = SHIFT ? handed[a] : c.pb[(ks + a) * bvol + l - st];
    } else {
      const bool wrap = c.bc[MU] == 0;
      int c2[4] = {c.bc[0], c.bc[1], c.bc[2], c.bc[3]};
      c2[MU] = wrap ? g.N[MU] - 1 : c.bc[MU] - 1;
      const int nb = encode_block(g, c2), nl = l + (bm - 1) * st;
      const long long nn = CANON ? c.n + (wrap ? cst * ((long long)g.L[MU] - 1) : -cst) : 0;
#pragma unroll
      for (int a = 0; a < 3; ++a)
        h[a] = proj1<IM, T>(face<CANON>(c, nb, nl, nn, ks + a), -sg, face<CANON>(c, nb, nl, nn, kp + a));
      cplx<T> w[9];
#pragma unroll
      for (int e = 0; e < 9; ++e) w[e] = ld<T>(c.U + gauge_index(g, nb, MU, e, nl));
      mul1<true, T>(w, h, v);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      up[a] += v[a];
      rec1<IM, T>(low[a], -sg, v[a]);
    }
  }
  if constexpr (MU < 3 && !SHIFT) __syncthreads();
  if constexpr (BS == 4) __builtin_amdgcn_sched_barrier(0);
}

}  // namespace rows

// per-right-hand-side gate and device-side mass (both optional)
struct DCtl {
  const int* gate = nullptr;
  int gstride = 0;
  const double* dmass = nullptr;
  // MODE 1: ||y||^2 of each block's sites to part[rhs * nblk + block]. The squares
  // cost nothing beside the stores; a pass of its own reads y again (32^3x64: 80 us
  // after the 564 us of b - D x)
  s64* part = nullptr;
};

// threads of a workgroup: a block's sites in groups of 32, two lanes each
inline int rows_threads(const Geom& g) { return ((g.bvol + 31) / 32) * 64; }
template <typename T, typename SX>
size_t rows_lds(const Geom& g) {
  return (((size_t)12 * g.bvol * sizeof(SX) + 15) & ~(size_t)15) + (size_t)6 * g.bvol * sizeof(cplx<T>);
}
// blocks the two-lane form takes: one workgroup per block
template <typename T, typename SX>
bool rows_fits(const Geom& g) { return rows_threads(g) <= 1024 && rows_lds<T, SX>(g) <= 160 * 1024; }

// MODE 0: y = scale * D x; MODE 1: y = b - scale * D x
// MAXT: largest workgroup of the instantiation, 1024 for blocks above 256 sites.
// Promising 512 where that holds lets the compiler order the loads for the four
// waves a SIMD has registers for (32^3 x 64, 12 sides: 5525 -> 5260 us).
// BS: 4 for 4^4 blocks known at compile time, else 0. Strides and limits are
// constants, and the x and y products go to the neighbour by lane shifts (four of
// the eight barriers and half of the handing over through LDS less): 8^4, dw_apply:
// 13.5 -> 12.0 us, 16^3x32 33.9 -> 32.8, 12 sides 319.5 -> 314.4, 32^3x64 with 12 5270
// -> 5182. The scheduling fences keep each direction's loads with it: without them
// all loads of a site are hoisted, 188 registers and two waves per SIMD (32^3x64
// with 12 sides 6370 us).
template <typename T, typename SX, typename SG, typename SY, int MODE, int MAXT, int BS, bool CLOV, bool CANON>
__global__ void __launch_bounds__(MAXT)
    k_dslash_rows(Geom g, T diag, const SX* __restrict__ x, T scale, const SG* __restrict__ U, SY* __restrict__ y,
                  const SY* __restrict__ bsrc, long long xs, long long ys, int nr, const int* __restrict__ rlist,
                  const SG* __restrict__ Cl, DCtl dc) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  SX* xsh = reinterpret_cast<SX*>(smem);
  cplx<T>* pb = reinterpret_cast<cplx<T>*>(smem + (((size_t)12 * g.bvol * sizeof(SX) + 15) & ~(size_t)15));
  // work item -> (block, RHS) with the RHS fastest: workgroups that read the
  // same links run together on one XCD. (Two right-hand sides at a time, for
  // all blocks: 5 x 3 x 3 x 5 blocks 57.6 -> 52.5 us, but 16^3 x 8, 12 sides,
  // 76 -> 80 us and 32^3 x 64 5260 -> 5345 us.)
  const int wi = xcd_remap(blockIdx.x, g.nblk * nr);
  if (wi < 0) return;  // uniform for the workgroup
  const int b = wi / nr;
  const int rhs = rlist ? rlist[wi - b * nr] : wi - b * nr;
  if (dc.gate && dc.gate[(long long)rhs * dc.gstride] == 0) return;  // uniform for the workgroup
  if (dc.dmass) diag = (T)(4.0 + *dc.dmass);
  const int l = (threadIdx.x >> 6) * 32 + (threadIdx.x & 31);
  const int r = (threadIdx.x >> 5) & 1;
  const bool active = l < g.bvol;
  const SX* xr = x + (long long)rhs * xs;
  SY* yr = y + (long long)rhs * ys;
  int bc[4], lc[4] = {0, 0, 0, 0};
  decode_block(g, b, bc);
  long long n = 0;
  auto own = [&](int k) { return CANON ? n * 12 + k : spinor_index(g, b, k, l); };
  if (active) {
    decode_local(g, l, lc);
    if constexpr (CANON)
      n = bc[0] * g.B[0] + lc[0] +
          (long long)g.L[0] * (bc[1] * g.B[1] + lc[1] +
                               (long long)g.L[1] * (bc[2] * g.B[2] + lc[2] + (long long)g.L[2] * (bc[3] * g.B[3] + lc[3])));
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      xsh[(3 * r + k) * g.bvol + l] = xr[own(3 * r + k)];
      xsh[(6 + 3 * r + k) * g.bvol + l] = xr[own(6 + 3 * r + k)];
    }
  }
  __syncthreads();
  const rows::Ctx<T, SX, SG> c{g, b, l, r, active, r ? (T)-1 : (T)1, bc, lc, n, xr, xsh, pb, U};
  cplx<T> up[3], lowxy[3], low[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) up[a] = lowxy[a] = mk<T>(0, 0);
  rows::dir<0, CANON, BS>(c, up, lowxy);
  rows::dir<1, CANON, BS>(c, up, lowxy);
  // spin 2 + r: the z and t hops go on from the other lane's x/y sum, so that the
  // hops are added in the order of the one-lane form, to the same bits
#pragma unroll
  for (int a = 0; a < 3; ++a) low[a] = rows::other_row(lowxy[a]);
  rows::dir<2, CANON, BS>(c, up, low);
  rows::dir<3, CANON, BS>(c, up, low);
  if constexpr (CLOV) {
    // lane r takes chirality r (spins 2r and 2r + 1) and the lanes swap the spin
    // that the other one stores. The 18 loads go out in two batches, for which the
    // registers of lowxy are free by now; one or two at a time, 24x16x16x24 with 4
    // sides took 138 us instead of 130, 18x16x16x36 with 3x4x4x6 blocks 240 instead of 189.
    __builtin_amdgcn_sched_barrier(0);
    cplx<T> w[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) w[i] = mk<T>(0, 0);
    if (active) {
      cplx<T> v[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) v[i] = ld<T>(xsh + (6 * r + i) * g.bvol + l);
      clover_chi<T, true>(Cl + ((long long)b * kCloverPairs + 18 * r) * g.bvol + l, g.bvol, v, w);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const cplx<T> got = rows::other_row(r ? w[a] : w[3 + a]);
      up[a] -= (T)2 * (r ? got : w[a]);
      low[a] -= (T)2 * (r ? w[3 + a] : got);
    }
  }
  double sq = 0;
  if (active) {
    const T half = (T)0.5;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int k = 6 * q + 3 * r + a;
        const cplx<T> psi = ld<T>(xsh + k * g.bvol + l);
        const cplx<T> acc = q ? low[a] : up[a];
        cplx<T> d = scale * (diag * psi - half * acc);
        if constexpr (MODE == 1) {
          d = ld<T>(bsrc + (long long)rhs * ys + own(k)) - d;
          sq = fma((double)d.re, (double)d.re, fma((double)d.im, (double)d.im, sq));
        }
        if constexpr (CANON) st(yr + own(k), d);
        else st_nt(yr + own(k), d);
      }
  }
  if constexpr (MODE == 1)
    if (dc.part) {
      sq = wave_total(sq);
      __syncthreads();  // the spinor in LDS is read out
      double* red = reinterpret_cast<double*>(smem);
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
      __syncthreads();
      if (threadIdx.x == 0) {
        double t = red[0];
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) t += red[w];
        dc.part[(long long)rhs * g.nblk + b] = s64{t, 0.0};
      }
    }
}

}  // namespace dw

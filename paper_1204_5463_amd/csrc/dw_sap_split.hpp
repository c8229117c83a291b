// One colour of the Schwarz alternating procedure on 4^4 blocks at FP64 and FP32
// storage: two threads per site, each with two of the four directions and their
// links in registers. Included by dw_sap_kernel.hpp.
//
// With one thread per site the links of a block (147 KB at FP64, 74 KB at FP32)
// are read again by every MR step: from beyond the L2 on large lattices, and by
// one or two wavefronts per SIMD that wait for them on small ones. Here thread 0
// of a site takes x and z, thread 1 y and t (whole wavefronts alike); each holds
// its two links for all MR steps, so a step reads nothing from global memory.
//
// A site projects its own spinor both ways, (1 - g_mu) psi and U_mu^+ (1 + g_mu)
// psi, and its neighbours take these half spinors: for x and y from the lane 1 or
// 4 away in the same row of 16 lanes (data-parallel-primitive moves, no LDS), for
// z and t through LDS. The two threads then swap partial sums: thread 0 owns the
// upper spin components (chirality 0) of the block's vectors, thread 1 the lower
// ones, and each applies the clover term of its chirality.
//
// Four barriers per MR step: residual visible, half spinors visible, partial sums
// visible, block sums visible.
//
// us per colour launch, one thread per site -> now: 16^3x32 nmr 5 FP64 54.5 ->
// 43.7 (clover 81.9 -> 59.1), FP32 38.8 -> 28.9; 8^4 nmr 4 FP64 34.0 -> 25.6;
// 32^3x64 nmr 8 FP64 924 -> 796, FP32 496 -> 339 (clover 783 -> 536). Bound: FP32 by
// VALU issue (5661 instructions per wavefront and launch at nmr 8, about 710 per step:
// busy 86% of the SIMD cycles, two blocks per CU). FP64 (6603, about 780 per step) by the
// chain of phases in turn, at two wavefronts per SIMD and one block per CU (registers of
// the links, 148 KB of LDS): on 32^3x64 VALU busy 45%, LDS 40%, on 16^3x32, one block per
// CU in all, VALU 24%. Reading the halo of the block
// residual ahead of the staging barrier spilled and was slower (nmr 0: 21.6 -> 28.6
// us). The 16-bit storages keep one thread per site: their links fit the
// registers there.
//
// At FP64 it runs whatever the number of right-hand sides, so that a side's result is
// the one of a call on its own. With several sides on more blocks than CUs one thread
// per site would be faster, since the sides find a block's links in the L2 and three
// blocks share a CU (us per two cycles, nmr 2, 5, 8, one thread -> two): 16^3x32 with 4
// sides 421, 605, 785 -> 466, 635, 804, with 12 1259, 1747, 2273 -> 1402, 1904, 2405, with 4
// and the clover term 528, 783, 1043 -> 551, 774, 995; with one side 158, 224 -> 142, 183.
#pragma once

#include "dw_clover.hpp"
#include "dw_internal.hpp"
#include "dw_stencil.hpp"

namespace dw {

namespace sapk {

constexpr int kSV = 256;  // sites of a block
constexpr int kST = 512;  // threads

// upper and lower sums += (SET: =) the spinor rebuilt from the half spinor of hop (MU, DIR)
template <int MU, int DIR, bool SET = false, typename T>
__device__ __forceinline__ void recon_halves(cplx<T> up[6], cplx<T> low[6], const cplx<T> g0[3], const cplx<T> g1[3]) {
  using P = proj_table<MU>;
  constexpr int C = DIR > 0 ? P::c : neg(P::c);
  constexpr int D = DIR > 0 ? P::d : neg(P::d);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const cplx<T> c = coef<C>(P::qc == 0 ? g0[a] : g1[a]), d = coef<D>(P::qd == 0 ? g0[a] : g1[a]);
    up[a] = SET ? g0[a] : up[a] + g0[a];
    up[3 + a] = SET ? g1[a] : up[3 + a] + g1[a];
    low[a] = SET ? c : low[a] + c;
    low[3 + a] = SET ? d : low[3 + a] + d;
  }
}

// LDS: [rho 12 x 256] [half spinors 12 x 512] [reduction 2 x 8 x 3] [||r||^2 8]
template <typename T>
constexpr size_t split_lds() {
  return (size_t)(12 * kSV + 12 * kST) * sizeof(cplx<T>) + (size_t)7 * (kST / 64) * sizeof(T);
}

template <typename T, typename SV, typename SZ, typename SG, bool CLOV>
__global__ void __launch_bounds__(kST) __attribute__((amdgpu_waves_per_eu(std::is_same<T, double>::value ? 2 : 4)))
    k_sap_split(Geom g, int colour, T diag, const SV* __restrict__ v, SZ* __restrict__ z, const SG* __restrict__ U,
                int nmr, int z_zero, long long vs, long long zs, int nr, const int* __restrict__ rlist,
                const SG* __restrict__ Cl, T red2, const int* __restrict__ gate, int gstride,
                const double* __restrict__ dmass) {
  using CT = cplx<T>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  CT* rho_s = reinterpret_cast<CT*>(smem);
  CT* pb = rho_s + 12 * kSV;
  T* red = reinterpret_cast<T*>(pb + 12 * kST);
  constexpr int nw = kST / kWave;
  // work item -> (block, right-hand side) with the RHS index fastest, so that
  // workgroups sharing a block's links run together on one XCD
  const int wi = xcd_remap(blockIdx.x, g.nbc * nr);
  if (wi < 0) return;  // whole workgroup: uniform exit before any barrier
  const int jb = wi / nr;
  const int rhs = rlist ? rlist[wi - jb * nr] : wi - jb * nr;
  if (gate && gate[(long long)rhs * gstride] == 0) return;  // uniform per workgroup, before any barrier
  if (dmass) diag = (T)(4.0 + *dmass);
  const int b = colour_block(g, colour, jb);
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int half = wave / 4;  // 0: x and z, upper components; 1: y and t, lower components
  const int l = tid % kSV;
  const int lc[4] = {l & 3, (l >> 2) & 3, (l >> 4) & 3, wave & 3};
  int bc[4];
  decode_block(g, b, bc);
  const long long own = ((long long)b * 12 + half * 6) * kSV + l;  // component half * 6 of this site
  const SV* vo = v + (long long)rhs * vs + own;
  SZ* zr = z + (long long)rhs * zs;
  SZ* zo = zr + own;
  CT* const ro = rho_s + half * 6 * kSV + l;         // own components in LDS
  CT* const rx = rho_s + (1 - half) * 6 * kSV + l;   // the other thread's
  const T hf = (T)0.5;
  const T diag2 = diag + diag;

  // links of directions half (x or y) and 2 + half (z or t)
  CT w[2][9];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int e = 0; e < 9; ++e) w[d][e] = ld<T>(U + (((long long)b * 4 + 2 * d + half) * 9 + e) * kSV + l);

  // partial sums of this thread's two directions -> own six: the other thread's
  // six go through the LDS rows of its own components. A barrier on both sides
  // (before: every read of rho_s is done).
  auto swap_sums = [&](const CT mine[6], const CT theirs[6], CT s[6]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) rx[k * kSV] = theirs[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] = mine[k] + ro[k * kSV];
  };
  // s -= 2 C x on the own chirality
  auto clover = [&](const CT x[6], CT s[6]) {
    if constexpr (CLOV) {
      // the entries are read in every step: an offset the compiler cannot see
      // through keeps the loads here
      int cofs = 0;
      asm volatile("" : "+v"(cofs));
      CT c[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) c[k] = mk<T>(0, 0);
      clover_chi<T, false>(Cl + ((long long)b * kCloverPairs + 18 * half) * kSV + l + cofs, kSV, x, c);
#pragma unroll
      for (int k = 0; k < 6; ++k) s[k] -= (T)2 * c[k];
    }
  };

  CT y[6], r[6];  // iterate and residual, own components
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    y[k] = mk<T>(0, 0);
    if (z_zero) r[k] = ld<T>(vo + k * kSV);
  }
  if (!z_zero) {
    // block residual r = v - D z: z of this block staged in LDS, the one-site
    // halo of z read from the neighbouring blocks of the other colour
#pragma unroll
    for (int k = 0; k < 6; ++k) ro[k * kSV] = ld<T>(zo + k * kSV);
    __syncthreads();
    CT mine[6], theirs[6];  // hop sums of this thread's directions: own components, the other thread's
#pragma unroll
    for (int k = 0; k < 6; ++k) mine[k] = theirs[k] = mk<T>(0, 0);
    auto first = [&](auto muc, const CT wl[9], CT* out) {
      constexpr int MU = decltype(muc)::value, st = 1 << (2 * MU);
      CT h0[3], h1[3], g0[3], g1[3];
      auto wf = [&](int e) { return wl[e]; };
      proj<MU, -1, T>([&](int k) { return rho_s[k * kSV + l]; }, h0, h1);
      su3_mul<true, true, T>(wf, h0, h1, g0, g1);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        out[a * kST] = g0[a];
        out[(3 + a) * kST] = g1[a];
      }
      if (lc[MU] < 3) {
        proj<MU, +1, T>([&](int k) { return rho_s[k * kSV + l + st]; }, h0, h1);
      } else {
        int c2[4] = {bc[0], bc[1], bc[2], bc[3]};
        c2[MU] = bc[MU] + 1 == g.N[MU] ? 0 : bc[MU] + 1;
        const SZ* zn = zr + (long long)encode_block(g, c2) * 12 * kSV + l - 3 * st;
        proj<MU, +1, T>([&](int k) { return ld<T>(zn + k * kSV); }, h0, h1);
      }
      su3_mul<false, true, T>(wf, h0, h1, g0, g1);
      if constexpr (MU % 2 == 0) recon_halves<MU, +1>(mine, theirs, g0, g1);
      else recon_halves<MU, +1>(theirs, mine, g0, g1);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto second = [&](auto muc, const CT* in) {
      constexpr int MU = decltype(muc)::value, st = 1 << (2 * MU);
      CT h0[3], h1[3], g0[3], g1[3];
      if (lc[MU] > 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          g0[a] = in[a * kST - st];
          g1[a] = in[(3 + a) * kST - st];
        }
      } else {
        int c2[4] = {bc[0], bc[1], bc[2], bc[3]};
        c2[MU] = bc[MU] == 0 ? g.N[MU] - 1 : bc[MU] - 1;
        const int nb = encode_block(g, c2), n = l + 3 * st;
        const SZ* zn = zr + (long long)nb * 12 * kSV + n;
        const SG* un = U + ((long long)nb * 36 + MU * 9) * kSV + n;
        proj<MU, -1, T>([&](int k) { return ld<T>(zn + k * kSV); }, h0, h1);
        su3_mul<true, true, T>([&](int e) { return ld<T>(un + e * kSV); }, h0, h1, g0, g1);
      }
      if constexpr (MU % 2 == 0) recon_halves<MU, -1>(mine, theirs, g0, g1);
      else recon_halves<MU, -1>(theirs, mine, g0, g1);
      __builtin_amdgcn_sched_barrier(0);
    };
    using std::integral_constant;
    if (half == 0) {
      first(integral_constant<int, 0>{}, w[0], pb + tid);
      first(integral_constant<int, 2>{}, w[1], pb + 6 * kST + tid);
    } else {
      first(integral_constant<int, 1>{}, w[0], pb + tid);
      first(integral_constant<int, 3>{}, w[1], pb + 6 * kST + tid);
    }
    __syncthreads();
    if (half == 0) {
      second(integral_constant<int, 0>{}, pb + tid);
      second(integral_constant<int, 2>{}, pb + 6 * kST + tid);
    } else {
      second(integral_constant<int, 1>{}, pb + tid);
      second(integral_constant<int, 3>{}, pb + 6 * kST + tid);
    }
    CT s[6];
    swap_sums(mine, theirs, s);
    CT q[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) q[k] = ld<T>(zo + k * kSV);  // the LDS rows hold partial sums now
    clover(q, s);
#pragma unroll
    for (int k = 0; k < 6; ++k) r[k] = ld<T>(vo + k * kSV) - diag * q[k] + hf * s[k];
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) ro[k * kSV] = r[k];

  // the block operator: a link that leaves the block is zero from here on, so its
  // forward hop adds nothing and neither does what its site hands to the next
  // row of lanes
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    const bool out = (d ? (half ? lc[3] : lc[2]) : (half ? lc[1] : lc[0])) == 3;
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      w[d][e].re = out ? (T)0 : w[d][e].re;
      w[d][e].im = out ? (T)0 : w[d][e].im;
    }
  }

  // sums over the block: this wavefront's values to LDS, then all of them
  T* const rr_s = red + 6 * nw;
  // adaptive stop: rr0 = ||r||^2 over the block, rr = ||rho_it||^2
  const bool adapt = red2 > (T)0;
  T rr0 = 0, rr = 0;
  if (adapt) {
    T sq = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) sq += norm2(r[k]);
    sq = wave_sum(sq);
    if (lane == 0) rr_s[wave] = sq;
    __syncthreads();
    for (int q = 0; q < nw; ++q) rr0 += rr_s[q];
    rr = rr0;
  }
  for (int it = 0; it < nmr; ++it) {
    if (adapt && rr <= red2 * rr0) break;  // uniform over the workgroup
    __syncthreads();                       // rho visible to the whole block
    CT mine[6], theirs[6];
    // direction LD (z or t): half spinors for both neighbours to LDS; direction
    // LN (x or y): all of it, across lanes
    auto send = [&](auto lnc, auto ldc) {
      constexpr int LN = decltype(lnc)::value, LD = decltype(ldc)::value;
      CT psi[12];
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        psi[LN * 6 + k] = r[k];
        psi[(1 - LN) * 6 + k] = rx[k * kSV];
      }
      auto pf = [&](int k) { return psi[k]; };
      CT h0[3], h1[3], g0[3], g1[3];
      {
        auto wf = [&](int e) { return w[1][e]; };
        proj<LD, +1, T>(pf, h0, h1);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          pb[a * kST + tid] = h0[a];
          pb[(3 + a) * kST + tid] = h1[a];
        }
        proj<LD, -1, T>(pf, h0, h1);
        su3_mul<true, true, T>(wf, h0, h1, g0, g1);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          pb[(6 + a) * kST + tid] = g0[a];
          pb[(9 + a) * kST + tid] = g1[a];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      {
        auto wf = [&](int e) { return w[0][e]; };
        proj<LN, -1, T>(pf, h0, h1);
        su3_mul<true, true, T>(wf, h0, h1, g0, g1);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          g0[a] = lane_shift<LN, -1>(g0[a]);
          g1[a] = lane_shift<LN, -1>(g1[a]);
        }
        if constexpr (LN == 0) recon_halves<LN, -1, true>(mine, theirs, g0, g1);
        else recon_halves<LN, -1, true>(theirs, mine, g0, g1);
        __builtin_amdgcn_sched_barrier(0);
        proj<LN, +1, T>(pf, h0, h1);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          h0[a] = lane_shift<LN, +1>(h0[a]);
          h1[a] = lane_shift<LN, +1>(h1[a]);
        }
        su3_mul<false, true, T>(wf, h0, h1, g0, g1);
        if constexpr (LN == 0) recon_halves<LN, +1>(mine, theirs, g0, g1);
        else recon_halves<LN, +1>(theirs, mine, g0, g1);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto take = [&](auto ldc) {
      constexpr int LD = decltype(ldc)::value, st = 1 << (2 * LD);
      CT h0[3], h1[3], g0[3], g1[3];
      if (lc[LD] < 3) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          h0[a] = pb[a * kST + tid + st];
          h1[a] = pb[(3 + a) * kST + tid + st];
        }
        su3_mul<false, true, T>([&](int e) { return w[1][e]; }, h0, h1, g0, g1);
        if constexpr (LD == 2) recon_halves<LD, +1>(mine, theirs, g0, g1);
        else recon_halves<LD, +1>(theirs, mine, g0, g1);
      }
      if (lc[LD] > 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          g0[a] = pb[(6 + a) * kST + tid - st];
          g1[a] = pb[(9 + a) * kST + tid - st];
        }
        if constexpr (LD == 2) recon_halves<LD, -1>(mine, theirs, g0, g1);
        else recon_halves<LD, -1>(theirs, mine, g0, g1);
      }
    };
    using std::integral_constant;
    if (half == 0) send(integral_constant<int, 0>{}, integral_constant<int, 2>{});
    else send(integral_constant<int, 1>{}, integral_constant<int, 3>{});
    __syncthreads();
    if (half == 0) take(integral_constant<int, 2>{});
    else take(integral_constant<int, 3>{});
    CT p[6];
    swap_sums(mine, theirs, p);
    clover(r, p);
    // p2 = 2 D^l rho = 2 diag rho - hops: the factor 2 cancels in the residual
    // update and is restored in the iterate update
    T nre = 0, nim = 0, den = 0;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      p[k] = mk<T>(fma(diag2, r[k].re, -p[k].re), fma(diag2, r[k].im, -p[k].im));
      nre = fma(p[k].re, r[k].re, nre);
      nre = fma(p[k].im, r[k].im, nre);
      nim = fma(p[k].re, r[k].im, nim);
      nim = fma(-p[k].im, r[k].re, nim);
      den = fma(p[k].re, p[k].re, den);
      den = fma(p[k].im, p[k].im, den);
    }
    nre = wave_sum(nre);
    nim = wave_sum(nim);
    den = wave_sum(den);
    T* rb = red + (it & 1) * 3 * nw;
    if (lane == 0) {
      rb[wave * 3 + 0] = nre;
      rb[wave * 3 + 1] = nim;
      rb[wave * 3 + 2] = den;
    }
    __syncthreads();  // also: partial sums read, half spinors read
    nre = nim = den = 0;
#pragma unroll
    for (int q = 0; q < nw; ++q) {
      nre += rb[q * 3 + 0];
      nim += rb[q * 3 + 1];
      den += rb[q * 3 + 2];
    }
    CT alpha = mk<T>(0, 0);
    if constexpr (std::is_same<T, float>::value) {
      const float inv = den > FLT_MIN ? __builtin_amdgcn_rcpf(den) : 0.f;
      alpha = mk<T>(nre * inv, nim * inv);
      if (adapt) rr -= (nre * nre + nim * nim) * inv;
    } else if (den > (T)0) {
      alpha = mk<T>(nre / den, nim / den);
      if (adapt) rr -= (nre * nre + nim * nim) / den;
    }
    const CT alpha_y = mk<T>(alpha.re + alpha.re, alpha.im + alpha.im);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      cmac(y[k], alpha_y, r[k]);
      cmsub(r[k], alpha, p[k]);
      ro[k * kSV] = r[k];
    }
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) st(zo + k * kSV, z_zero ? y[k] : ld<T>(zo + k * kSV) + y[k]);
  // z starts at zero: this workgroup also clears one block of the other colour
  // (same count per colour), which this launch never reads
  if (z_zero) {
    SZ* zc = zr + ((long long)colour_block(g, 1 - colour, jb) * 12 + half * 6) * kSV + l;
#pragma unroll
    for (int k = 0; k < 6; ++k) st(zc + k * kSV, mk<T>(0, 0));
  }
}

template <typename T, typename SV, typename SZ, typename SG, bool CLOV>
dw_status launch_split(const Geom& g, double m0, const void* v, void* z, const void* U, int colour, int nmr,
                       int z_zero, int nrhs, long long vs, long long zs, const int* rlist, hipStream_t s,
                       const void* C, double red2, const int* gate, int gs, const double* dmass) {
  constexpr size_t lds = split_lds<T>();
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)k_sap_split<T, SV, SZ, SG, CLOV>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) {
      set_error("hipFuncSetAttribute(LDS %zu bytes) failed: %s", lds, hipGetErrorString(e));
      return DW_EHIP;
    }
  }
  KTimer kt(DW_K_SAP, s);
  hipLaunchKernelGGL((k_sap_split<T, SV, SZ, SG, CLOV>), (unsigned)xcd_grid(g.nbc * nrhs), kST, lds, s, g, colour,
                     (T)(4.0 + m0), (const SV*)v, (SZ*)z, (const SG*)U, nmr, z_zero, vs, zs, nrhs, rlist,
                     (const SG*)C, (T)red2, gate, gs, dmass);
  DW_CHECK_LAUNCH();
  sap_done<SV, SZ, SG, CLOV>(kt, g, nmr, z_zero, nrhs);
  return DW_OK;
}

}  // namespace sapk

}  // namespace dw

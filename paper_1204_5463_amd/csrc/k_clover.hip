// Builds the clover term of a field from its FP64 links (see dw_clover.hpp).
// One thread per site: F = (Q - Q^+)/8 for each of the six planes from the four
// leaves around the site (periodic), then the two chirality blocks
// (i c_sw / 2) sum sigma^chi_{mu nu} (x) F_{mu nu}, stored packed at all four
// precisions.
//
// Q enters only as Q - Q^+, so a leaf may be replaced by minus its conjugate, and
// the four leaves group into
//   Q' = T(n) U_mu(n)^+ - T(n-mu)^+ U_mu(n-mu),
//   T(n) = U_nu(n-nu)^+ U_mu(n-nu) U_nu(n+mu-nu) - U_nu(n) U_mu(n+nu) U_nu(n+mu)^+,
// the difference of the two staples of U_mu(n). A site computes T(n) once (4
// products, 6 link reads), its own term and, handed to site n+mu through LDS, the
// other site's: 6 products and 7 link reads per plane. Only the Hermitian part is
// handed over, 9 numbers. Where n-mu is outside the workgroup's 256 sites its T is
// computed here as well, by a compact list of such sites (a quarter of them on 4^4
// blocks, one wave per plane, a different one each time).
// A neighbour's offset in the tiled layout is the sum of one term per direction,
// computed once per site (the divisions of the index arithmetic, per link, were
// most of the instructions). In the chiral basis the planes xy and zt fill the
// spin-diagonal blocks and the other four the off-diagonal one, so the two groups
// are accumulated and stored one after the other, which keeps the 42 entries
// of a site out of the registers.
// Bound by the link reads that miss the L2, at two waves per SIMD: counted on 24^3x48
// 4.0 KB read per site for 576 B of links, 1.15 KB written, 5.2 TB/s together; L2 hits
// 63%, VALU busy 33%. 24^3x48: the four leaves of each site by themselves, 10 products
// and 14 link reads per plane, 840 us -> 660 us. (All sites of the lists at the start
// instead, spread over the waves: 288 B of spills, 984 us.)
#include "dw_clover.hpp"
#include "dw_internal.hpp"

namespace dw {

namespace {

constexpr int kThreads = 256;
using C = cplx<double>;

struct M3 {
  C e[9];
};

// r (+)= op(a) op(b), op the conjugate transpose where DA (DB) is set; NEG: r -=.
// a(i, k) is asked for once per entry, row by row, so that a link's rows can be
// read as they are needed. Products are formed apart and added: chained into the
// sums (cmac) they save a third of the instructions, 1-4% of the build's time, and
// cost 7% more rounding error of the term.
template <bool DA, bool DB, bool ACC, bool NEG, typename AF>
__device__ __forceinline__ void mul(M3& r, AF&& a, const M3& b) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    C x[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) x[k] = DA ? conj(a(k * 3 + i)) : a(i * 3 + k);
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      C s = ACC ? r.e[i * 3 + j] : C{0.0, 0.0};
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const C y = DB ? conj(b.e[j * 3 + k]) : b.e[k * 3 + j];
        if constexpr (NEG) s -= x[k] * y;
        else s += x[k] * y;
      }
      r.e[i * 3 + j] = s;
    }
  }
  // each product's loads stay with it: hoisted, they cost the second wave per SIMD
  __builtin_amdgcn_sched_barrier(0);
}

// one of four values by a wave-uniform index (selects, no indexed registers)
__device__ __forceinline__ long long pick(const long long v[4], int i) {
  return i == 0 ? v[0] : i == 1 ? v[1] : i == 2 ? v[2] : v[3];
}

// ALL: all four copies; else FP64 only
template <bool ALL>
struct CloverOut {
  s64* o64;
  s32* o32;
  s16* o16;
  sbf* obf;
  __device__ __forceinline__ void put(long long at, C v, bool on) const {
    if (on) {
      st(o64 + at, v);
      if constexpr (ALL) {
        st(o32 + at, v);
        st(o16 + at, v);
        st(obf + at, v);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
};

template <bool ALL>
__global__ void __launch_bounds__(kThreads, 2)
    k_clover_build(Geom g, const s64* __restrict__ U, SigmaBlocks sb, double csw, CloverOut<ALL> out) {
  __shared__ double own[9][kThreads], far[9][kThreads];  // handed over; by the list, for its site
  __shared__ long long hereL[kThreads], dnL[3][kThreads], upL[3][kThreads], dnN[3][kThreads];
  __shared__ short list[3][kThreads];  // threads whose n - d is outside the workgroup
  __shared__ int count[3];
  const int chunk = xcd_remap(blockIdx.x, (int)((g.V + kThreads - 1) / kThreads));
  if (chunk < 0) return;  // uniform for the workgroup
  const int tid = threadIdx.x;
  const long long s0 = (long long)chunk * kThreads;
  const bool active = s0 + tid < g.V;
  const long long s = active ? s0 + tid : g.V - 1;
  const int b = (int)(s / g.bvol);
  const int l = (int)(s - (long long)b * g.bvol);
  int bc[4], lc[4];
  decode_block(g, b, bc);
  decode_local(g, l, lc);
  // offsets of the neighbours n + d and n - d
  long long up[4], dn[4];
  int before[3];  // thread of n - d, or -1
  if (tid < 3) count[tid] = 0;
  __syncthreads();
  long long bst = g.bvol;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const long long across = (long long)(g.B[d] - 1) * g.lstride[d], turn = (long long)(g.N[d] - 1) * bst;
    const long long ub = bc[d] < g.N[d] - 1 ? bst : -turn, db = bc[d] > 0 ? -bst : turn;
    up[d] = lc[d] < g.B[d] - 1 ? g.lstride[d] : 36 * ub - across;
    dn[d] = lc[d] > 0 ? -g.lstride[d] : 36 * db + across;
    if (d < 3) {
      const long long at = s + (lc[d] > 0 ? -g.lstride[d] : db + across) - s0;
      before[d] = at >= 0 && at < kThreads ? (int)at : -1;
      if (active && before[d] < 0) list[d][atomicAdd(&count[d], 1)] = (short)tid;
      dnL[d][tid] = dn[d];
    }
    if (d > 0) {
      upL[d - 1][tid] = up[d];
      dnN[d - 1][tid] = dn[d];
    }
    bst *= g.N[d];
  }
  hereL[tid] = (long long)b * 36 * g.bvol + l;
  __syncthreads();
  // entry reader of the link U_mu at offset ofs. The pointer goes through an
  // offset the compiler cannot see through: links that appear in two products
  // are read again from the L1 instead of being held
  auto link = [&](long long ofs, int mu) {
    int zero = 0;
    asm volatile("" : "+v"(zero));
    const s64* p = U + ofs + (long long)mu * 9 * g.bvol + zero;
    if constexpr (ALL) {
      return [p, &g](int e) { return ld<double>(p + e * g.bvol); };
    } else {  // small blocks: a link's entries share their lines, so it is read at once
      M3 r;
#pragma unroll
      for (int e = 0; e < 9; ++e) r.e[e] = ld<double>(p + e * g.bvol);
      return [r](int e) { return r.e[e]; };
    }
  };
  auto whole = [](auto&& f) {
    M3 r;
#pragma unroll
    for (int e = 0; e < 9; ++e) r.e[e] = f(e);
    return r;
  };
  // (i csw / 16) (Q' - Q'^+): the diagonal, then (01 02 12) as (re, im)
  auto herm = [&](const M3& q, double h[9]) {
    const double w = 0.0625 * csw;
#pragma unroll
    for (int i = 0; i < 3; ++i) h[i] = -2.0 * w * q.e[4 * i].im;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const C x = q.e[k == 2 ? 5 : 1 + k], y = q.e[k == 0 ? 3 : k == 1 ? 6 : 7];
      h[3 + 2 * k] = -w * (x.im + y.im);
      h[4 + 2 * k] = w * (x.re - y.re);
    }
  };
  // f = (i csw / 2) F of plane (mu, nu), Hermitian
  auto plane = [&](int mu, int nu, int turn, double f[9]) {
    const int k = (tid + 64 * turn) & (kThreads - 1);  // place in the list
    const bool extra = k < count[mu];
#pragma unroll 1
    for (int pass = extra ? 0 : 1; pass < 2; ++pass) {
      const int t = pass ? tid : list[mu][k];  // pass 0: T of the site before t
      const long long down = dnL[mu][t], at = hereL[t] + (pass ? 0 : down);
      const long long pu = pass ? pick(up, mu) : -down, pv = upL[nu - 1][t], mv = dnN[nu - 1][t];
      M3 m, x, q;
      auto rx = [&](int e) { return x.e[e]; };
      mul<false, true, false, true>(m, link(at + pv, mu), whole(link(at + pu, nu)));
      mul<false, false, false, false>(x, link(at, nu), m);
      mul<false, false, false, false>(m, link(at + mv, mu), whole(link(at + pu + mv, nu)));
      mul<true, false, true, false>(x, link(at + mv, nu), m);  // T
      m = whole(link(at, mu));
      mul<true, false, false, true>(q, rx, m);  // - T^+ U
      double h[9];
      herm(q, h);
      double* to = pass ? &own[0][tid] : &far[0][t];
#pragma unroll
      for (int e = 0; e < 9; ++e) to[e * kThreads] = h[e];
      if (pass) {
        mul<false, true, false, false>(q, rx, m);  // T U^+
        herm(q, f);
      }
    }
    __syncthreads();
    const int from = mu == 0 ? before[0] : mu == 1 ? before[1] : before[2];
    const double* h = from >= 0 ? &own[0][from] : &far[0][tid];
#pragma unroll
    for (int e = 0; e < 9; ++e) f[e] += h[e * kThreads];
    __syncthreads();
  };
  // entry (row, column) above the diagonal sits at pair 3 + its number in row-major order
  auto at = [&](int chi, int pair) { return ((long long)b * kCloverPairs + chi * 18 + pair) * g.bvol + l; };
  {
    C f0[6], f5[6];  // (00 11 22 01 02 12) of planes xy and zt
#pragma unroll
    for (int i = 0; i < 6; ++i) f0[i] = f5[i] = C{0.0, 0.0};
#pragma unroll 1
    for (int q = 0; q < 2; ++q) {
      double f[9];
      plane(2 * q, 2 * q + 1, q, f);
      const C v[6] = {{f[0], 0.0}, {f[1], 0.0}, {f[2], 0.0}, {f[3], f[4]}, {f[5], f[6]}, {f[7], f[8]}};
      const double is0 = q == 0 ? 1.0 : 0.0, is5 = 1.0 - is0;  // weights, not branches: a select of 24 registers spills
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        f0[i] += is0 * v[i];
        f5[i] += is5 * v[i];
      }
    }
#pragma unroll
    for (int chi = 0; chi < 2; ++chi) {
      C d[2][6];  // spin, (00 11 22 01 02 12)
#pragma unroll
      for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          d[sp][i] = C{sb.re[0][chi][3 * sp], sb.im[0][chi][3 * sp]} * f0[i];
          cmac(d[sp][i], C{sb.re[5][chi][3 * sp], sb.im[5][chi][3 * sp]}, f5[i]);
        }
      out.put(at(chi, 0), C{d[0][0].re, d[0][1].re}, active);
      out.put(at(chi, 1), C{d[0][2].re, d[1][0].re}, active);
      out.put(at(chi, 2), C{d[1][1].re, d[1][2].re}, active);
      out.put(at(chi, 3), d[0][3], active);
      out.put(at(chi, 4), d[0][4], active);
      out.put(at(chi, 8), d[0][5], active);
      out.put(at(chi, 15), d[1][3], active);
      out.put(at(chi, 16), d[1][4], active);
      out.put(at(chi, 17), d[1][5], active);
    }
  }
  C o[2][9];
#pragma unroll
  for (int i = 0; i < 18; ++i) o[i / 9][i % 9] = C{0.0, 0.0};
#pragma unroll 1
  for (int p = 1; p < 5; ++p) {  // xz, xt, yz, yt: planes 1..4 of the pairs mu < nu
    double f[9];
    plane(p > 2 ? 1 : 0, p % 2 ? 2 : 3, p + 1, f);
    const C full[9] = {{f[0], 0.0}, {f[3], f[4]}, {f[5], f[6]}, {f[3], -f[4]}, {f[1], 0.0}, {f[7], f[8]},
                       {f[5], -f[6]}, {f[7], -f[8]}, {f[2], 0.0}};
#pragma unroll
    for (int chi = 0; chi < 2; ++chi) {
      const C sg = C{sb.re[p][chi][1], sb.im[p][chi][1]};
#pragma unroll
      for (int e = 0; e < 9; ++e) cmac(o[chi][e], sg, full[e]);
    }
  }
#pragma unroll
  for (int chi = 0; chi < 2; ++chi)
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) out.put(at(chi, (a == 0 ? 5 : a == 1 ? 9 : 12) + c), o[chi][a * 3 + c], active);
}

}  // namespace

SigmaBlocks sigma_blocks() {
  // gamma matrices of the chiral basis: g_k = [[0, -i s_k], [i s_k, 0]], g_t = [[0, 1], [1, 0]]
  typedef cplx<double> Cx;
  Cx s[3][4] = {{{0, 0}, {1, 0}, {1, 0}, {0, 0}},     // s_x
                {{0, 0}, {0, -1}, {0, 1}, {0, 0}},    // s_y
                {{1, 0}, {0, 0}, {0, 0}, {-1, 0}}};   // s_z
  Cx gam[4][16];
  for (int mu = 0; mu < 4; ++mu)
    for (int e = 0; e < 16; ++e) gam[mu][e] = Cx{0, 0};
  for (int k = 0; k < 3; ++k)
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j) {
        const Cx v = s[k][i * 2 + j];
        gam[k][i * 4 + (2 + j)] = Cx{v.im, -v.re};       // -i s_k (upper right)
        gam[k][(2 + i) * 4 + j] = Cx{-v.im, v.re};       // +i s_k (lower left)
      }
  for (int i = 0; i < 2; ++i) {
    gam[3][i * 4 + 2 + i] = Cx{1, 0};
    gam[3][(2 + i) * 4 + i] = Cx{1, 0};
  }
  auto mm = [&](const Cx* a, const Cx* b, Cx* r) {
    for (int i = 0; i < 4; ++i)
      for (int j = 0; j < 4; ++j) {
        Cx t{0, 0};
        for (int k = 0; k < 4; ++k) t += a[i * 4 + k] * b[k * 4 + j];
        r[i * 4 + j] = t;
      }
  };
  SigmaBlocks sb;
  int plane = 0;
  for (int mu = 0; mu < 4; ++mu)
    for (int nu = mu + 1; nu < 4; ++nu, ++plane) {
      Cx ab[16], ba[16];
      mm(gam[mu], gam[nu], ab);
      mm(gam[nu], gam[mu], ba);
      for (int chi = 0; chi < 2; ++chi)
        for (int i = 0; i < 2; ++i)
          for (int j = 0; j < 2; ++j) {
            const int e = (2 * chi + i) * 4 + 2 * chi + j;
            const Cx cm = ab[e] - ba[e];
            // sigma = (i/2) [g_mu, g_nu]
            sb.re[plane][chi][i * 2 + j] = -0.5 * cm.im;
            sb.im[plane][chi][i * 2 + j] = 0.5 * cm.re;
          }
    }
  return sb;
}

dw_status launch_clover_build(const Geom& g, const void* U64, double csw, void* const out[4], hipStream_t s) {
  const unsigned grid = (unsigned)xcd_grid((int)((g.V + kThreads - 1) / kThreads));
  s64* o64 = (s64*)out[DW_PREC_F64];
  // On blocks of one or two sites a wavefront's store of a pair touches as many lines
  // as it has lanes, so the other copies are converted from the FP64 one, and a
  // link is read at once: 16^3x32, one site 429 -> 265 us, 1x1x1x2 blocks 272 -> 233.
  if (g.bvol <= 2) {
    hipLaunchKernelGGL(k_clover_build<false>, grid, kThreads, 0, s, g, (const s64*)U64, sigma_blocks(), csw,
                       CloverOut<false>{o64, nullptr, nullptr, nullptr});
    DW_CHECK_LAUNCH();
    for (int p : {DW_PREC_F32, DW_PREC_F16, DW_PREC_BF16})
      DW_TRY(launch_convert(DW_PREC_F64, o64, p, out[p], 1.0, g.V * kCloverPairs, s));
    return DW_OK;
  }
  hipLaunchKernelGGL(k_clover_build<true>, grid, kThreads, 0, s, g, (const s64*)U64, sigma_blocks(), csw,
                     CloverOut<true>{o64, (s32*)out[DW_PREC_F32], (s16*)out[DW_PREC_F16], (sbf*)out[DW_PREC_BF16]});
  DW_CHECK_LAUNCH();
  return DW_OK;
}

}  // namespace dw

// Builds the clover term of a field from its FP64 links (see dw_clover.hpp).
// One thread per site: F = (Q - Q^+)/8 for each of the six planes from the four
// leaves around the site (periodic), then the two chirality blocks
// (i c_sw / 2) sum sigma^chi_{mu nu} (x) F_{mu nu}, stored packed at all four
// precisions.
//
// Q enters only as Q - Q^+, so a leaf may be replaced by minus its conjugate,
// and the four leaves group into
//   Q' = [V A1 + W^+ A2] U^+ + [V B1 + W^+ B2] X,
//   U = U_mu(n), X = U_mu(n-mu), V = U_nu(n), W = U_nu(n-nu),
//   A1 = -U_mu(n+nu) U_nu(n+mu)^+,       A2 = U_mu(n-nu) U_nu(n+mu-nu),
//   B1 = U_mu(n-mu+nu)^+ U_nu(n-mu)^+,   B2 = -U_mu(n-mu-nu)^+ U_nu(n-mu-nu):
// 10 products and 14 link reads per plane instead of 12 and 16. A neighbour's
// offset in the tiled layout is the sum of one term per direction, computed
// once per site (the divisions of the index arithmetic, per link, were most of
// the instructions). In the chiral basis the planes xy and zt fill the spin-
// diagonal blocks and the other four the off-diagonal one, so the two groups
// are accumulated and stored one after the other, which keeps the 42 entries
// of a site out of the registers.
// Bound by the L2: 12 KB of links per site at about 9.5 TB/s. 24^3x48: 886 us and
// 285 us of conversions -> 840 us.
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
// read as they are needed.
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
        if constexpr (NEG) cmsub(s, x[k], y);
        else cmac(s, x[k], y);
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

struct CloverOut {
  s64* o64;
  s32* o32;
  s16* o16;
  sbf* obf;
  __device__ __forceinline__ void put(long long at, C v) const {
    st(o64 + at, v);
    st(o32 + at, v);
    st(o16 + at, v);
    st(obf + at, v);
    __builtin_amdgcn_sched_barrier(0);
  }
};

__global__ void __launch_bounds__(kThreads, 2)
    k_clover_build(Geom g, const s64* __restrict__ U, SigmaBlocks sb, double csw, CloverOut out) {
  const int chunk = xcd_remap(blockIdx.x, (int)((g.V + kThreads - 1) / kThreads));
  if (chunk < 0) return;
  const long long s = (long long)chunk * kThreads + threadIdx.x;
  if (s >= g.V) return;
  const int b = (int)(s / g.bvol);
  const int l = (int)(s - (long long)b * g.bvol);
  int bc[4], lc[4];
  decode_block(g, b, bc);
  decode_local(g, l, lc);
  // offsets of the neighbours n + d and n - d
  long long up[4], dn[4];
  long long bst = (long long)36 * g.bvol;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const long long across = (long long)(g.B[d] - 1) * g.lstride[d], turn = (long long)(g.N[d] - 1) * bst;
    up[d] = lc[d] < g.B[d] - 1 ? g.lstride[d] : (bc[d] < g.N[d] - 1 ? bst : -turn) - across;
    dn[d] = lc[d] > 0 ? -g.lstride[d] : (bc[d] > 0 ? -bst : turn) + across;
    bst *= g.N[d];
  }
  const s64* here = U + (long long)b * 36 * g.bvol + l;
  // entry reader of the link U_mu at offset ofs. The pointer goes through an
  // offset the compiler cannot see through: links that appear in two products
  // are read again from the L1 instead of being held
  auto link = [&](int mu, long long ofs) {
    int zero = 0;
    asm volatile("" : "+v"(zero));
    const s64* p = here + ofs + (long long)mu * 9 * g.bvol + zero;
    return [p, &g](int e) { return ld<double>(p + e * g.bvol); };
  };
  auto whole = [](auto&& f) {
    M3 r;
#pragma unroll
    for (int e = 0; e < 9; ++e) r.e[e] = f(e);
    return r;
  };
  // f = (i csw / 2) F of plane (mu, nu), Hermitian: (i csw / 16) (Q' - Q'^+)
  auto plane = [&](int mu, int nu) {
    const long long pu = pick(up, mu), mm = pick(dn, mu), pv = pick(up, nu), mv = pick(dn, nu);
    M3 q, t, r;
    auto rv = [&](int e) { return r.e[e]; };
    mul<false, true, false, true>(t, link(mu, pv), whole(link(nu, pu)));         // A1
    mul<false, false, false, false>(r, link(nu, 0), t);                          // V A1
    mul<false, false, false, false>(t, link(mu, mv), whole(link(nu, pu + mv)));  // A2
    mul<true, false, true, false>(r, link(nu, mv), t);                           // + W^+ A2
    mul<false, true, false, false>(q, rv, whole(link(mu, 0)));                   // ... U^+
    mul<true, true, false, false>(t, link(mu, mm + pv), whole(link(nu, mm)));    // B1
    mul<false, false, false, false>(r, link(nu, 0), t);                          // V B1
    mul<true, false, false, true>(t, link(mu, mm + mv), whole(link(nu, mm + mv)));  // B2
    mul<true, false, true, false>(r, link(nu, mv), t);                           // + W^+ B2
    mul<false, false, true, false>(q, rv, whole(link(mu, mm)));                  // ... X
    M3 f;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const C x = q.e[i * 3 + j], y = q.e[j * 3 + i];
        const double re = 0.125 * (x.re - y.re), im = 0.125 * (x.im + y.im);
        f.e[i * 3 + j] = C{-0.5 * csw * im, 0.5 * csw * re};
      }
    return f;
  };
  // entry (row, column) above the diagonal sits at pair 3 + its number in row-major order
  auto at = [&](int chi, int pair) { return ((long long)b * kCloverPairs + chi * 18 + pair) * g.bvol + l; };
  {
    C f0[6], f5[6];  // (00 11 22 01 02 12) of planes xy and zt
#pragma unroll
    for (int i = 0; i < 6; ++i) f0[i] = f5[i] = C{0.0, 0.0};
#pragma unroll 1
    for (int q = 0; q < 2; ++q) {
      const M3 f = plane(2 * q, 2 * q + 1);
      const C v[6] = {f.e[0], f.e[4], f.e[8], f.e[1], f.e[2], f.e[5]};
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
      out.put(at(chi, 0), C{d[0][0].re, d[0][1].re});
      out.put(at(chi, 1), C{d[0][2].re, d[1][0].re});
      out.put(at(chi, 2), C{d[1][1].re, d[1][2].re});
      out.put(at(chi, 3), d[0][3]);
      out.put(at(chi, 4), d[0][4]);
      out.put(at(chi, 8), d[0][5]);
      out.put(at(chi, 15), d[1][3]);
      out.put(at(chi, 16), d[1][4]);
      out.put(at(chi, 17), d[1][5]);
    }
  }
  C o[2][9];
#pragma unroll
  for (int i = 0; i < 18; ++i) o[i / 9][i % 9] = C{0.0, 0.0};
#pragma unroll 1
  for (int p = 1; p < 5; ++p) {  // xz, xt, yz, yt: planes 1..4 of the pairs mu < nu
    const M3 f = plane(p > 2 ? 1 : 0, p % 2 ? 2 : 3);
#pragma unroll
    for (int chi = 0; chi < 2; ++chi) {
      const C sg = C{sb.re[p][chi][1], sb.im[p][chi][1]};
#pragma unroll
      for (int e = 0; e < 9; ++e) cmac(o[chi][e], sg, f.e[e]);
    }
  }
#pragma unroll
  for (int chi = 0; chi < 2; ++chi)
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) out.put(at(chi, (a == 0 ? 5 : a == 1 ? 9 : 12) + c), o[chi][a * 3 + c]);
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
  const CloverOut o{(s64*)out[DW_PREC_F64], (s32*)out[DW_PREC_F32], (s16*)out[DW_PREC_F16], (sbf*)out[DW_PREC_BF16]};
  hipLaunchKernelGGL(k_clover_build, grid, kThreads, 0, s, g, (const s64*)U64, sigma_blocks(), csw, o);
  DW_CHECK_LAUNCH();
  return DW_OK;
}

}  // namespace dw

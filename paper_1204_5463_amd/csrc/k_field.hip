// Layout and precision conversion kernels: canonical complex128 fields to
// and from the internal block-tiled layout, and elementwise conversions.
#include "dw_internal.hpp"
#include "dw_types.hpp"

namespace dw {

namespace {

constexpr int kThreads = 256;

// one thread per (internal site, rhs): reads the site's 12 canonical
// complex numbers, writes 12 coalesced internal entries
template <typename S>
__global__ void __launch_bounds__(kThreads) k_pack_spinor(Geom g, const s64* __restrict__ in, S* __restrict__ out,
                                                          double scale, const double* __restrict__ dscale,
                                                          int dstride) {
  long long s = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (s >= g.V) return;
  if (dscale) scale *= dscale[(long long)blockIdx.y * dstride];
  const long long rhs_off = (long long)blockIdx.y * g.V * 12;
  const int b = (int)(s / g.bvol);
  const int l = (int)(s - (long long)b * g.bvol);
  const long long n = canonical_site(g, b, l);
  const s64* src = in + rhs_off + n * 12;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    cplx<double> v = ld<double>(src + c);
    st(out + rhs_off + spinor_index(g, b, c, l), scale * v);
  }
}

template <typename S>
__global__ void __launch_bounds__(kThreads) k_unpack_spinor(Geom g, const S* __restrict__ in, s64* __restrict__ out,
                                                            double scale, const double* __restrict__ dscale,
                                                            int dstride) {
  long long s = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (s >= g.V) return;
  if (dscale) scale *= dscale[(long long)blockIdx.y * dstride];
  const long long rhs_off = (long long)blockIdx.y * g.V * 12;
  const int b = (int)(s / g.bvol);
  const int l = (int)(s - (long long)b * g.bvol);
  const long long n = canonical_site(g, b, l);
  s64* dst = out + rhs_off + n * 12;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    cplx<double> v = ld<double>(in + rhs_off + spinor_index(g, b, c, l));
    st(dst + c, scale * v);
  }
}

// The four storage copies of the links from one read of the canonical field:
// 576 bytes read and 1152 written per site, against 3456 in four passes
// (24^3x48: 684 -> 208 us). One thread per (site, direction), so that the 9
// entries of a link are one contiguous read and every store is coalesced.
// ALL: all four; else FP64 only.
template <bool ALL>
__global__ void __launch_bounds__(kThreads)
    k_pack_gauge(Geom g, const s64* __restrict__ in, s64* __restrict__ o64, s32* __restrict__ o32,
                 s16* __restrict__ o16, sbf* __restrict__ obf) {
  const long long s = (long long)blockIdx.x * kThreads + threadIdx.x;
  if (s >= g.V) return;
  const int mu = blockIdx.y;
  const int b = (int)(s / g.bvol);
  const int l = (int)(s - (long long)b * g.bvol);
  const s64* src = in + ((long long)mu * g.V + canonical_site(g, b, l)) * 9;
  cplx<double> v[9];
#pragma unroll
  for (int e = 0; e < 9; ++e) v[e] = ld<double>(src + e);
  __builtin_amdgcn_sched_barrier(0);  // all 9 loads in flight before the first store
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    const long long at = gauge_index(g, b, mu, e, l);
    st(o64 + at, v[e]);
    if constexpr (ALL) {
      st(o32 + at, v[e]);
      st(o16 + at, v[e]);
      st(obf + at, v[e]);
    }
  }
}

template <typename SI, typename SO>
__global__ void __launch_bounds__(kThreads) k_convert(const SI* __restrict__ in, SO* __restrict__ out, double scale,
                                                      const double* __restrict__ dscale, long long n,
                                                      const int* __restrict__ gate) {
  if (gate && *gate == 0) return;
  if (dscale) scale *= dscale[0];
  long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
  const long long stride = (long long)gridDim.x * kThreads;
  for (; i < n; i += stride) st(out + i, scale * ld<double>(in + i));
}

dim3 site_grid(const Geom& g, int nrhs) { return dim3((unsigned)((g.V + kThreads - 1) / kThreads), (unsigned)nrhs); }

}  // namespace

dw_status launch_pack_spinor(const Geom& g, int prec, const double* in, void* out, double scale, int nrhs,
                             hipStream_t s, const double* dscale, int dstride) {
  const s64* src = reinterpret_cast<const s64*>(in);
  dim3 grid = site_grid(g, nrhs);
  KTimer kt(DW_K_CONVERT, s);
  switch (prec) {
    case DW_PREC_F64: hipLaunchKernelGGL(k_pack_spinor<s64>, grid, kThreads, 0, s, g, src, (s64*)out, scale, dscale, dstride); break;
    case DW_PREC_F32: hipLaunchKernelGGL(k_pack_spinor<s32>, grid, kThreads, 0, s, g, src, (s32*)out, scale, dscale, dstride); break;
    case DW_PREC_F16: hipLaunchKernelGGL(k_pack_spinor<s16>, grid, kThreads, 0, s, g, src, (s16*)out, scale, dscale, dstride); break;
    case DW_PREC_BF16: hipLaunchKernelGGL(k_pack_spinor<sbf>, grid, kThreads, 0, s, g, src, (sbf*)out, scale, dscale, dstride); break;
    default: set_error("unknown precision %d", prec); return DW_EINVAL;
  }
  DW_CHECK_LAUNCH();
  kt.done((double)g.V * 12 * nrhs * (16 + pair_bytes(prec)), 0);
  return DW_OK;
}

dw_status launch_unpack_spinor(const Geom& g, int prec, const void* in, double* out, double scale, int nrhs,
                               hipStream_t s, const double* dscale, int dstride) {
  s64* dst = reinterpret_cast<s64*>(out);
  dim3 grid = site_grid(g, nrhs);
  KTimer kt(DW_K_CONVERT, s);
  switch (prec) {
    case DW_PREC_F64: hipLaunchKernelGGL(k_unpack_spinor<s64>, grid, kThreads, 0, s, g, (const s64*)in, dst, scale, dscale, dstride); break;
    case DW_PREC_F32: hipLaunchKernelGGL(k_unpack_spinor<s32>, grid, kThreads, 0, s, g, (const s32*)in, dst, scale, dscale, dstride); break;
    case DW_PREC_F16: hipLaunchKernelGGL(k_unpack_spinor<s16>, grid, kThreads, 0, s, g, (const s16*)in, dst, scale, dscale, dstride); break;
    case DW_PREC_BF16: hipLaunchKernelGGL(k_unpack_spinor<sbf>, grid, kThreads, 0, s, g, (const sbf*)in, dst, scale, dscale, dstride); break;
    default: set_error("unknown precision %d", prec); return DW_EINVAL;
  }
  DW_CHECK_LAUNCH();
  kt.done((double)g.V * 12 * nrhs * (16 + pair_bytes(prec)), 0);
  return DW_OK;
}

dw_status launch_pack_gauge(const Geom& g, const double* in, void* const out[4], hipStream_t s) {
  // one-site blocks: no store is coalesced there, so the other copies are converted
  // from the FP64 one (import of 16^3x32 268 -> 114 us, of 32^4 2110 -> 990)
  if (g.bvol == 1) {
    {
      KTimer kt(DW_K_CONVERT, s);
      hipLaunchKernelGGL(k_pack_gauge<false>, site_grid(g, 4), kThreads, 0, s, g, (const s64*)in,
                         (s64*)out[DW_PREC_F64], (s32*)nullptr, (s16*)nullptr, (sbf*)nullptr);
      DW_CHECK_LAUNCH();
      kt.done((double)g.V * 36 * 32, 0);
    }
    for (int p : {DW_PREC_F32, DW_PREC_F16, DW_PREC_BF16})
      DW_TRY(launch_convert(DW_PREC_F64, out[DW_PREC_F64], p, out[p], 1.0, g.V * 36, s));
    return DW_OK;
  }
  KTimer kt(DW_K_CONVERT, s);
  hipLaunchKernelGGL(k_pack_gauge<true>, site_grid(g, 4), kThreads, 0, s, g, (const s64*)in, (s64*)out[DW_PREC_F64],
                     (s32*)out[DW_PREC_F32], (s16*)out[DW_PREC_F16], (sbf*)out[DW_PREC_BF16]);
  DW_CHECK_LAUNCH();
  double bytes = 16;
  for (int p = 0; p < 4; ++p) bytes += pair_bytes(p);
  kt.done((double)g.V * 36 * bytes, 0);
  return DW_OK;
}

namespace {
template <typename SI>
dw_status convert_from(const SI* in, int pout, void* out, double scale, const double* ds, long long n,
                       hipStream_t s, const int* gate) {
  long long nb = (n + kThreads - 1) / kThreads;
  unsigned grid = (unsigned)(nb < 8192 ? (nb > 0 ? nb : 1) : 8192);
  KTimer kt(DW_K_CONVERT, s);
  switch (pout) {
    case DW_PREC_F64: hipLaunchKernelGGL((k_convert<SI, s64>), grid, kThreads, 0, s, in, (s64*)out, scale, ds, n, gate); break;
    case DW_PREC_F32: hipLaunchKernelGGL((k_convert<SI, s32>), grid, kThreads, 0, s, in, (s32*)out, scale, ds, n, gate); break;
    case DW_PREC_F16: hipLaunchKernelGGL((k_convert<SI, s16>), grid, kThreads, 0, s, in, (s16*)out, scale, ds, n, gate); break;
    case DW_PREC_BF16: hipLaunchKernelGGL((k_convert<SI, sbf>), grid, kThreads, 0, s, in, (sbf*)out, scale, ds, n, gate); break;
    default: set_error("unknown precision %d", pout); return DW_EINVAL;
  }
  DW_CHECK_LAUNCH();
  kt.done((double)n * (sizeof(SI) + pair_bytes(pout)), 0);
  return DW_OK;
}
}  // namespace

dw_status launch_convert(int pin, const void* in, int pout, void* out, double scale, long long n, hipStream_t s,
                         const double* dscale, const int* gate) {
  switch (pin) {
    case DW_PREC_F64: return convert_from((const s64*)in, pout, out, scale, dscale, n, s, gate);
    case DW_PREC_F32: return convert_from((const s32*)in, pout, out, scale, dscale, n, s, gate);
    case DW_PREC_F16: return convert_from((const s16*)in, pout, out, scale, dscale, n, s, gate);
    case DW_PREC_BF16: return convert_from((const sbf*)in, pout, out, scale, dscale, n, s, gate);
    default: set_error("unknown precision %d", pin); return DW_EINVAL;
  }
}

}  // namespace dw

// 16-bit storage of fine fields, links and prolongator columns: conversions
// and the buffers that hold them (layout and scaling rules in half_field.h).
#include "half_field.h"
#include "internal.h"

namespace wdmg {
namespace {

template <typename H>
__global__ void k_round_h(const cx<float>* __restrict__ in, cxh<H>* __restrict__ out, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    out[i] = f2h<H>(in[i].re, in[i].im);
}

// -v for every stored value: flipping the sign bits of both halves is exact
// (the scales are unchanged).
__global__ void k_neg_h(uint32_t* __restrict__ v, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    v[i] ^= 0x80008000u;
}

__global__ void k_fill32(uint32_t* __restrict__ v, size_t n, uint32_t x) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) v[i] = x;
}
__global__ void k_copy32(uint32_t* __restrict__ d, const uint32_t* __restrict__ s, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    d[i] = s[i];
}

// FP64 or FP32 field -> 16-bit field, one thread per site
template <typename R, typename H>
__global__ void k_to_half(Geom g, const cx<R>* __restrict__ in, cxh<H>* __restrict__ v, float* __restrict__ sc) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (s >= g.vol) return;
  in += (size_t)r * 12 * g.vol;
  v += (size_t)r * 12 * g.vol;
  sc += (size_t)r * g.vol;
  cx<float> a[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) a[k] = cvt<float>(in[(size_t)s * 12 + k]);
  store_site_h(v, sc, s, a);
}

template <typename H, typename R>
__global__ void k_from_half(Geom g, const cxh<H>* __restrict__ v, const float* __restrict__ sc,
                            cx<R>* __restrict__ out) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = blockIdx.y;
  if (s >= g.vol) return;
  out += (size_t)r * 12 * g.vol;
  v += (size_t)r * 12 * g.vol;
  sc += (size_t)r * g.vol;
  cx<float> a[12];
  load_site_h(v, sc, s, a);
#pragma unroll
  for (int k = 0; k < 12; ++k) out[(size_t)s * 12 + k] = cvt<R>(a[k]);
}

template <typename H>
void round_to_half(Ctx& c, const cx<float>* in, void* out, size_t n) {
  size_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL((k_round_h<H>), dim3((unsigned)blocks), dim3(256), 0, c.stream, in, static_cast<cxh<H>*>(out),
                     n);
  WDMG_HIP(hipGetLastError());
}

void round_kind(Ctx& c, int kind, const cx<float>* in, void* out, size_t n) {
  if (kind == WDMG_F16)
    round_to_half<f16_t>(c, in, out, n);
  else
    round_to_half<bf16_t>(c, in, out, n);
}

dim3 site_grid(const Geom& g, int nrhs) { return dim3((g.vol + 255) / 256, nrhs); }

unsigned flat_blocks(size_t n) {
  const size_t b = (n + 255) / 256;
  return (unsigned)(b > 8192 ? 8192 : b);
}

}  // namespace

const void* u16(Ctx& c, int kind) {
  if (kind != WDMG_F16 && kind != WDMG_BF16) throw Error(WDMG_ERR_ARG, "not a 16-bit kind");
  if (c.u16_kind == kind) return c.U16;
  const size_t n = (size_t)c.g0.vpad * kLinkComp;
  if (!c.U16) c.U16 = dev_alloc(c, n * 4);
  round_kind(c, kind, c.U32, c.U16, n);
  c.u16_kind = kind;
  return c.U16;
}

const void* v16(Ctx& c, Level& L, int kind) {
  if (kind != WDMG_F16 && kind != WDMG_BF16) throw Error(WDMG_ERR_ARG, "not a 16-bit kind");
  if (L.v16_kind == kind) return L.V16;
  if (!L.V32) throw Error(WDMG_ERR_ARG, "FP32 prolongator released by wdmg_release_unused");
  const size_t n = (size_t)L.nv * L.n;
  if (!L.V16) L.V16 = dev_alloc(c, n * 4);
  round_kind(c, kind, L.V32, L.V16, n);
  L.v16_kind = kind;
  return L.V16;
}

void hf_renew(Ctx& c, HF& f, int nrhs) {
  const size_t vol = c.g0.vol;
  hf_free(c, f);
  dev_renew(c, f.v, (size_t)nrhs * 12 * vol * 4);
  dev_renew(c, f.s, (size_t)nrhs * vol * sizeof(float));
}

void hf_free(Ctx& c, HF& f) {
  dev_free(c, f.v);
  dev_free(c, f.s);
  f.v = nullptr;
  f.s = nullptr;
}

void hf_copy(Ctx& c, HF dst, HF src, int nrhs) {
  // values (4 bytes each) and scales copied unchanged
  const size_t nv = (size_t)nrhs * 12 * c.g0.vol, ns = (size_t)nrhs * c.g0.vol;
  hipLaunchKernelGGL(k_copy32, dim3(flat_blocks(nv)), dim3(256), 0, c.stream, static_cast<uint32_t*>(dst.v),
                     static_cast<const uint32_t*>(src.v), nv);
  WDMG_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_copy32, dim3(flat_blocks(ns)), dim3(256), 0, c.stream, reinterpret_cast<uint32_t*>(dst.s),
                     reinterpret_cast<const uint32_t*>(src.s), ns);
  WDMG_HIP(hipGetLastError());
}

void hf_neg(Ctx& c, HF f, int nrhs) {
  const size_t n = (size_t)nrhs * 12 * c.g0.vol;
  hipLaunchKernelGGL(k_neg_h, dim3(flat_blocks(n)), dim3(256), 0, c.stream, static_cast<uint32_t*>(f.v), n);
  WDMG_HIP(hipGetLastError());
}

template <typename H>
void hf_zero(Ctx& c, HF f, int nrhs) {
  const size_t nv = (size_t)nrhs * 12 * c.g0.vol, ns = (size_t)nrhs * c.g0.vol;
  hipLaunchKernelGGL(k_fill32, dim3(flat_blocks(nv)), dim3(256), 0, c.stream, static_cast<uint32_t*>(f.v), nv, 0u);
  WDMG_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_fill32, dim3(flat_blocks(ns)), dim3(256), 0, c.stream, reinterpret_cast<uint32_t*>(f.s), ns, 0u);
  WDMG_HIP(hipGetLastError());
}

template <typename R, typename H>
void to_half(Ctx& c, const cx<R>* in, HF out, int nrhs) {
  hipLaunchKernelGGL((k_to_half<R, H>), site_grid(c.g0, nrhs), dim3(256), 0, c.stream, c.g0, in,
                     static_cast<cxh<H>*>(out.v), out.s);
  WDMG_HIP(hipGetLastError());
}

template <typename H, typename R>
void from_half(Ctx& c, HF in, cx<R>* out, int nrhs) {
  hipLaunchKernelGGL((k_from_half<H, R>), site_grid(c.g0, nrhs), dim3(256), 0, c.stream, c.g0,
                     static_cast<const cxh<H>*>(in.v), in.s, out);
  WDMG_HIP(hipGetLastError());
}

#define INST(H)                                                       \
  template void hf_zero<H>(Ctx&, HF, int);                            \
  template void to_half<double, H>(Ctx&, const cx<double>*, HF, int); \
  template void to_half<float, H>(Ctx&, const cx<float>*, HF, int);   \
  template void from_half<H, double>(Ctx&, HF, cx<double>*, int);     \
  template void from_half<H, float>(Ctx&, HF, cx<float>*, int);
INST(f16_t)
INST(bf16_t)
#undef INST

}  // namespace wdmg

// Galerkin coarse operator D_c = P^dagger D P (Sec. 2) as a nearest-neighbour
// stencil of dense complex (2Nv x 2Nv) blocks, and its application.
//
// Storage per coarse site: nine blocks, column-major ([col][row]), in the
// order d = 2 mu (Y_{+mu}, couples to xhat + mu), d = 2 mu + 1 (Y_{-mu},
// couples to xhat - mu), d = 8 (X, the site itself).
//
// Build: a fine-level coupling that leaves an aggregate through its +-mu face
// lands in Y_{+-mu}; every other coupling (the diagonal term and the hops
// that stay inside the aggregate) lands in X.  Each workgroup computes one
// block of one coarse site: it applies the fine hops to the chirality-split
// columns of P at a few sites at a time (staged in LDS) and contracts them
// with the conjugated columns, all in FP64.
#include <type_traits>

#include "half_field.h"
#include "internal.h"
#include "wilson_spin.h"

namespace wdmg {
namespace {

constexpr int kMfmaMinRhs = 2;  // batches of at least this many rhs use the matrix cores

struct AggGeom {
  Geom g;       // geometry of the finer level
  int b[4];     // aggregate extents
  int nb[4];    // aggregates per direction
  int bvol;
};

AggGeom make_agg(const Level& f) {
  AggGeom a;
  a.g = f.g;
  a.bvol = 1;
  for (int mu = 0; mu < 4; ++mu) {
    a.b[mu] = f.block[mu];
    a.nb[mu] = f.dims[mu] / f.block[mu];
    a.bvol *= f.block[mu];
  }
  return a;
}

// Global coordinates of local site `i` of the sites visited for block d of
// aggregate `agg`: the whole aggregate for d = 8, else its (mu, sign) face.
__device__ __forceinline__ void block_site(const AggGeom& a, int agg, int d, int i, int c[4]) {
  int base[4];
  int t = agg;
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    base[mu] = (t % a.nb[mu]) * a.b[mu];
    t /= a.nb[mu];
  }
  const int fmu = d < 8 ? (d >> 1) : -1;
  int u = i;
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    int lc;
    if (mu == fmu) {
      lc = (d & 1) ? 0 : a.b[mu] - 1;
    } else {
      lc = u % a.b[mu];
      u /= a.b[mu];
    }
    c[mu] = base[mu] + lc;
  }
}

__device__ __forceinline__ int nsites_of_block(const AggGeom& a, int d) {
  return d < 8 ? a.bvol / a.b[d >> 1] : a.bvol;
}

// Is the hop (mu, dir) from coordinates c inside the aggregate?
__device__ __forceinline__ bool inside(const AggGeom& a, const int c[4], int mu, int dir) {
  const int lc = c[mu] % a.b[mu];
  return dir > 0 ? (lc < a.b[mu] - 1) : (lc > 0);
}

// ---- level 0: Wilson hops ---------------------------------------------------
template <int MU, int SIGN>
__device__ __forceinline__ void wilson_hop_col(const Geom& g, const int c[4], const cx<double>* __restrict__ U,
                                               const cx<double>* __restrict__ vk, bool neg, int chi,
                                               cx<double> (&t)[12]) {
  int n[4] = {c[0], c[1], c[2], c[3]};  // the neighbour
  n[MU] = SIGN > 0 ? (c[MU] == g.L[MU] - 1 ? 0 : c[MU] + 1) : (c[MU] == 0 ? g.L[MU] - 1 : c[MU] - 1);
  const int nb = canon_site(g, n);
  const int ls = SIGN > 0 ? site_of(g, c[0], c[1], c[2], c[3]) : site_of(g, n[0], n[1], n[2], n[3]);
  cx<double> p[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const bool on = (k / 6) == chi;
    p[k] = on ? vk[(size_t)nb * 12 + k] : mk(0.0, 0.0);
  }
  cx<double> h[6];
  project<MU, SIGN>(p, h);
  cx<double> u[9];
  load_link(U, MU, ls, neg, u);
  cx<double> uh[6];
#pragma unroll
  for (int aa = 0; aa < 2; ++aa) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      cx<double> sacc = mk(0.0, 0.0);
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (SIGN > 0)
          cmadd(sacc, u[i * 3 + b], h[aa * 3 + b]);
        else
          cmaddc(sacc, u[b * 3 + i], h[aa * 3 + b]);
      }
      uh[aa * 3 + i] = sacc;
    }
  }
  expand_add<MU, SIGN>(uh, t);
}

// The hop in direction (mu, dir) at coordinates c.
__device__ void wilson_hop_dispatch(const Geom& g, const int c[4], int mu, int dir, const cx<double>* U,
                                    const cx<double>* vk, bool neg, int chi, cx<double> (&t)[12]) {
  switch (mu * 2 + (dir < 0)) {
    case 0: wilson_hop_col<0, +1>(g, c, U, vk, neg, chi, t); break;
    case 1: wilson_hop_col<0, -1>(g, c, U, vk, neg, chi, t); break;
    case 2: wilson_hop_col<1, +1>(g, c, U, vk, neg, chi, t); break;
    case 3: wilson_hop_col<1, -1>(g, c, U, vk, neg, chi, t); break;
    case 4: wilson_hop_col<2, +1>(g, c, U, vk, neg, chi, t); break;
    case 5: wilson_hop_col<2, -1>(g, c, U, vk, neg, chi, t); break;
    case 6: wilson_hop_col<3, +1>(g, c, U, vk, neg, chi, t); break;
    default: wilson_hop_col<3, -1>(g, c, U, vk, neg, chi, t); break;
  }
}

struct WilsonSide {
  const cx<double>* U;
  double diag;  // 4 + m
  int tneg;     // antiperiodic time: links at t = Lt-1 carry the sign
  static constexpr int kDof = 12;
  // Element offset of dof e at site s in a field of this level.
  __device__ __forceinline__ size_t off(size_t, int s, int e) const { return (size_t)s * 12 + e; }
  __device__ __forceinline__ bool neg(const Geom& g, const int c[4], int mu, int dir) const {
    return tneg && mu == 3 && c[3] == (dir > 0 ? g.L[3] - 1 : 0);
  }
  // T[q][e][cc] for columns col0 .. col0+ncc-1 at the chunk's sites.
  __device__ void columns(const AggGeom& a, int d, const int* sites, const int (*crd)[4], int ncs, int col0, int ncc,
                          int ldt, int nv, const cx<double>* Vv, size_t vstride, cx<double>* T) const {
    for (int w = threadIdx.x; w < ncs * ncc; w += blockDim.x) {
      const int q = w / ncc, cc = w % ncc;
      const int col = col0 + cc, chi = col / nv, k = col % nv;
      const cx<double>* vk = Vv + (size_t)k * vstride;
      const int s = sites[q];
      const int* c = crd[q];
      cx<double> t[12];
#pragma unroll
      for (int e = 0; e < 12; ++e) t[e] = mk(0.0, 0.0);
      if (d < 8) {
        const int mu = d >> 1, dir = (d & 1) ? -1 : 1;
        wilson_hop_dispatch(a.g, c, mu, dir, U, vk, neg(a.g, c, mu, dir), chi, t);
#pragma unroll
        for (int e = 0; e < 12; ++e) t[e] = (-0.5) * t[e];
      } else {
        for (int mu = 0; mu < 4; ++mu) {
          for (int dir = 1; dir >= -1; dir -= 2) {
            if (!inside(a, c, mu, dir)) continue;
            wilson_hop_dispatch(a.g, c, mu, dir, U, vk, neg(a.g, c, mu, dir), chi, t);
          }
        }
#pragma unroll
        for (int e = 0; e < 12; ++e) {
          const bool on = (e / 6) == chi;
          const cx<double> f = on ? vk[(size_t)s * 12 + e] : mk(0.0, 0.0);
          t[e] = mk(diag * f.re - 0.5 * t[e].re, diag * f.im - 0.5 * t[e].im);
        }
      }
#pragma unroll
      for (int e = 0; e < 12; ++e) T[((size_t)q * 12 + e) * ldt + cc] = t[e];
    }
  }
};

// ---- level >= 1: stencil hops ----------------------------------------------
struct StencilSide {
  const cx<double>* Dc;  // finer level's stencil [site][9][col][row]
  int dof;
  __device__ __forceinline__ size_t off(size_t, int s, int e) const { return (size_t)s * dof + e; }
  __device__ void columns(const AggGeom& a, int d, const int* sites, const int (*crd)[4], int ncs, int col0, int ncc,
                          int ldt, int nv, const cx<double>* Vv, size_t vstride, cx<double>* T) const {
    const int half = dof / 2;
    const size_t bsz = (size_t)dof * dof;
    for (int w = threadIdx.x; w < ncs * ncc * dof; w += blockDim.x) {
      const int e = w % dof;
      const int cc = (w / dof) % ncc;
      const int q = w / (dof * ncc);
      const int col = col0 + cc, chi = col / nv, k = col % nv;
      const cx<double>* vk = Vv + (size_t)k * vstride;
      const int s = sites[q];
      const int* c = crd[q];
      cx<double> acc = mk(0.0, 0.0);
      for (int dd = 0; dd < 9; ++dd) {
        int nb;
        if (d < 8) {
          if (dd != d) continue;
        } else if (dd < 8) {
          if (!inside(a, c, dd >> 1, (dd & 1) ? -1 : 1)) continue;
        }
        if (dd == 8)
          nb = s;
        else
          nb = (dd & 1) ? nbr_bwd(a.g, s, c, dd >> 1) : nbr_fwd(a.g, s, c, dd >> 1);
        const cx<double>* blk = Dc + ((size_t)s * 9 + dd) * bsz;
        const cx<double>* f = vk + (size_t)nb * dof + chi * half;
        for (int j = 0; j < half; ++j) cmadd(acc, blk[(size_t)(chi * half + j) * dof + e], f[j]);
      }
      T[((size_t)q * dof + e) * ldt + cc] = acc;
    }
  }
};

// ---- the build kernel ---------------------------------------------------------
// Matrix-core operations on tiles of 16 x 16, four terms at a time; operand
// lanes: A[i][k] at lane i + 16 k, B[k][j] at lane j + 16 k.
template <typename R>
struct Mma;
template <>
struct Mma<double> {
  typedef double acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int r) { return 4 * r + g; }  // of D, lane group g, register r
};
template <>
struct Mma<float> {
  typedef float acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int r) { return 4 * g + r; }
};

// The block is the product of the conjugated columns (n2 rows, chirality by
// chirality) with the hopped ones, summed over the sites: a complex GEMM on
// the FP64 matrix cores, at most 16 tiles, tile t on wave t % 4.  24^3x48,
// 4^4 aggregates, nv 24: 19.4 ms (43.3 ms with the product on the vector units,
// which read two operands from LDS per complex product).  What is left is
// mostly the hops; they take the registers of two workgroups per compute unit.
template <class Side>
__global__ __launch_bounds__(256, 2) void k_coarse_build(Side side, AggGeom a, const cx<double>* __restrict__ Vv,
                                                      size_t vstride, int nv, int dof, int cs, int cc_max,
                                                      cx<double>* __restrict__ Dc) {
  using M = Mma<double>;
  extern __shared__ cx<double> sm[];
  __shared__ int sites[8];
  __shared__ int crd[8][4];
  const int agg = blockIdx.x, d = blockIdx.y;
  const int n2 = 2 * nv, half = dof / 2;
  cx<double>* Vt = sm;                          // [cs][dof][nv]
  cx<double>* T = sm + (size_t)cs * dof * nv;   // [cs][dof][cc_max]
  const int nsites = nsites_of_block(a, d);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const int rt = (nv + 15) / 16;  // row tiles of a chirality
  cx<double>* out = Dc + ((size_t)agg * 9 + d) * n2 * n2;
  for (int col0 = 0; col0 < n2; col0 += cc_max) {
    const int ncc = min(cc_max, n2 - col0);
    const int ntile = 2 * rt * ((ncc + 15) / 16);
    M::acc_t re[4], im[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      re[i] = M::acc_t{0, 0, 0, 0};
      im[i] = M::acc_t{0, 0, 0, 0};
    }
    for (int i0 = 0; i0 < nsites; i0 += cs) {
      const int ncs = min(cs, nsites - i0);
      if (threadIdx.x < ncs) {
        int c[4];
        block_site(a, agg, d, i0 + threadIdx.x, c);
        sites[threadIdx.x] = canon_site(a.g, c);
#pragma unroll
        for (int mu = 0; mu < 4; ++mu) crd[threadIdx.x][mu] = c[mu];
      }
      __syncthreads();
      for (int w = threadIdx.x; w < ncs * dof * nv; w += blockDim.x) {
        const int e = w % dof, k = (w / dof) % nv, q = w / (nv * dof);
        Vt[((size_t)q * dof + e) * nv + k] = Vv[(size_t)k * vstride + side.off(a.g.vol, sites[q], e)];
      }
      side.columns(a, d, sites, crd, ncs, col0, ncc, cc_max, nv, Vv, vstride, T);
      __syncthreads();
      const int nk = ncs * half;  // terms of a chirality in this chunk
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tile = wave + 4 * i;
        if (tile >= ntile) break;
        const int chi = tile & 1, k = 16 * ((tile >> 1) % rt) + li, cc = 16 * ((tile >> 1) / rt) + li;
        const cx<double>* va = Vt + min(k, nv - 1);
        const cx<double>* tb = T + min(cc, ncc - 1);
        for (int r0 = 0; r0 < nk; r0 += 4) {
          const int r = min(r0 + lk, nk - 1);
          const size_t row = (size_t)(r / half) * dof + chi * half + r % half;
          cx<double> v = va[row * nv], t = tb[row * cc_max];
          if (r0 + lk >= nk) v = t = mk(0.0, 0.0);
          re[i] = M::mma(v.re, t.re, re[i]);
          im[i] = M::mma(v.re, t.im, im[i]);
          re[i] = M::mma(v.im, t.im, re[i]);
          im[i] = M::mma(-v.im, t.re, im[i]);
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tile = wave + 4 * i;
      if (tile >= ntile) break;
      const int chi = tile & 1, k0 = 16 * ((tile >> 1) % rt), cc = 16 * ((tile >> 1) / rt) + li;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = k0 + M::row(lk, r);
        if (k < nv && cc < ncc) out[(size_t)(col0 + cc) * n2 + chi * nv + k] = mk(re[i][r], im[i][r]);
      }
    }
  }
}

// ---- application ----------------------------------------------------------------
// One workgroup of nine waves per (coarse site, rhs); wave d applies block d
// (lane = row), and the nine partial rows are summed in a fixed order.
// acc += sum_j blk[j n2] v[j]: one row of a column-major block times a
// vector, in column order, with the loads of 8 columns issued together (20 at
// a time is slower, 256 sites, nv 20, FP64: 11.6 against 10.6 us).
template <typename R>
__device__ __forceinline__ void block_row_madd(const cx<R>* __restrict__ blk, int n2, const cx<R>* v, cx<R>& acc) {
  int jj = 0;
  for (; jj + 8 <= n2; jj += 8) {
    cx<R> a[8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      a[u] = blk[(size_t)(jj + u) * n2];
      b[u] = v[jj + u];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) cmadd(acc, a[u], b[u]);
  }
  for (; jj < n2; ++jj) cmadd(acc, blk[(size_t)jj * n2], v[jj]);
}

template <typename R>
__global__ __launch_bounds__(576) void k_coarse_apply(Geom g, int n2, const cx<R>* __restrict__ Dc,
                                                      const cx<R>* __restrict__ in, cx<R>* __restrict__ out) {
  __shared__ cx<R> part[9][64];
  const int s = blockIdx.x, rhs = blockIdx.y;
  const int d = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const size_t nsite = g.vol;
  in += (size_t)rhs * nsite * n2;
  out += (size_t)rhs * nsite * n2;
  int nb = s;
  if (d < 8) {
    int c[4];
    coords_of(g, s, c);
    nb = (d & 1) ? nbr_bwd(g, s, c, d >> 1) : nbr_fwd(g, s, c, d >> 1);
  }
  cx<R> acc = mk<R>(0, 0);
  if (lane < n2) {
    block_row_madd(Dc + ((size_t)s * 9 + d) * n2 * n2 + lane, n2, in + (size_t)nb * n2, acc);
  }
  part[d][lane] = acc;
  __syncthreads();
  if (d == 0 && lane < n2) {
    cx<R> t = part[8][lane];
#pragma unroll
    for (int dd = 0; dd < 8; ++dd) t = t + part[dd][lane];
    out[(size_t)s * n2 + lane] = t;
  }
}

// Coarse vector layouts: element (rhs q, site, row) of nrhs vectors.
struct RhsMajor {  // [rhs][site][row], the canonical coarse layout
  size_t fs;       // site count x rows
  __device__ __forceinline__ size_t at(int q, int site, int row, int n2) const {
    return (size_t)q * fs + (size_t)site * n2 + row;
  }
};
struct RhsFast {  // [site][row][rhs]: the rhs of one row are adjacent
  int nrhs;
  __device__ __forceinline__ size_t at(int q, int site, int row, int n2) const {
    return ((size_t)site * n2 + row) * nrhs + q;
  }
};

// One right-hand side on the vector units: wave d (of nine) applies block d
// of site s with lane = row; the nine partial rows are added in order.
// Needs blockDim.x >= 576; ends with a block barrier, the result also in `res`.
__device__ __forceinline__ void apply_site_valu1(const Geom& g, int n2, int s, const cx<double>* __restrict__ Dc,
                                                 const cx<double>* in, cx<double>* out, double* lds, cx<double>* res) {
  const int d = threadIdx.x >> 6, lane = threadIdx.x & 63;
  cx<double> acc = mk(0.0, 0.0);
  if (d < 9 && lane < n2) {
    int nb = s, c[4];
    coords_of(g, s, c);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      if (d == 2 * mu) nb = nbr_fwd(g, s, c, mu);
      if (d == 2 * mu + 1) nb = nbr_bwd(g, s, c, mu);
    }
    block_row_madd(Dc + ((size_t)s * 9 + d) * n2 * n2 + lane, n2, in + (size_t)nb * n2, acc);
  }
  if (d < 9) {
    lds[2 * (d * 64 + lane)] = acc.re;
    lds[2 * (d * 64 + lane) + 1] = acc.im;
  }
  __syncthreads();
  if (d == 0 && lane < n2) {
    cx<double> t = mk(lds[2 * (8 * 64 + lane)], lds[2 * (8 * 64 + lane) + 1]);
#pragma unroll
    for (int dd = 0; dd < 8; ++dd) t = t + mk(lds[2 * (dd * 64 + lane)], lds[2 * (dd * 64 + lane) + 1]);
    out[(size_t)s * n2 + lane] = t;
    res[lane] = t;
  }
  __syncthreads();
}

// ---- 16-bit blocks ---------------------------------------------------------------
// Stored [column / 4][row][column % 4] (the padding of the last columns holds
// zeros): four consecutive columns of a row, re and im alternating, are one
// 16-byte load and a matrix-core operand as they stand, and the lanes of
// consecutive rows read one run of memory.
__host__ __device__ inline int h16_chunks(int n2) { return (n2 + 3) / 4; }

// One workgroup per block: scale = largest magnitude of the block's real
// components (after rounding to FP32), stored = fl16(fl32(value * fl32(1/scale))).
template <typename H>
__global__ __launch_bounds__(256) void k_dc_to_half(const cx<double>* __restrict__ Dc, cxh<H>* __restrict__ Dh,
                                                    float* __restrict__ scales, int n2) {
  __shared__ float red[4];
  const size_t b = blockIdx.x;
  const int nn = n2 * n2, np = h16_chunks(n2) * n2 * 4;
  const cx<double>* src = Dc + b * nn;
  float m = 0.0f;
  bool nan = false;
  for (int i = threadIdx.x; i < nn; i += blockDim.x) {
    const cx<float> a = cvt<float>(src[i]);
    m = fmaxf(m, fmaxf(fabsf(a.re), fabsf(a.im)));
    nan = nan || a.re != a.re || a.im != a.im;
  }
  if (nan) m = __builtin_nanf("");
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float o = __shfl_xor(m, off, 64);
    m = (o != o || m != m) ? __builtin_nanf("") : fmaxf(m, o);
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  float mm = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) mm = (red[w] != red[w] || mm != mm) ? __builtin_nanf("") : fmaxf(mm, red[w]);
  float inv;
  const float sc = quant_scale(mm, inv);
  if (threadIdx.x == 0) scales[b] = sc;
  for (int i = threadIdx.x; i < np; i += blockDim.x) {
    const int row = (i >> 2) % n2, col = (i >> 2) / n2 * 4 + (i & 3);
    const cx<float> a = col < n2 ? cvt<float>(src[(size_t)col * n2 + row]) : mk(0.0f, 0.0f);
    Dh[b * np + i] = col < n2 ? quantise<H>(a.re, a.im, inv) : f2h<H>(0.0f, 0.0f);
  }
}

// One right-hand side on the vector units (as k_coarse_apply), 16-bit blocks,
// the vector in FP32.
template <typename H>
__global__ __launch_bounds__(576) void k_coarse_apply_h(Geom g, int n2, const cxh<H>* __restrict__ Dc,
                                                        const float* __restrict__ Dcs,
                                                        const cx<float>* __restrict__ in,
                                                        cx<float>* __restrict__ out) {
  __shared__ cx<float> part[9][64];
  const int s = blockIdx.x, rhs = blockIdx.y;
  const int d = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const size_t nsite = g.vol;
  in += (size_t)rhs * nsite * n2;
  out += (size_t)rhs * nsite * n2;
  int nb = s;
  if (d < 8) {
    int c[4];
    coords_of(g, s, c);
    nb = (d & 1) ? nbr_bwd(g, s, c, d >> 1) : nbr_fwd(g, s, c, d >> 1);
  }
  cx<float> acc = mk(0.0f, 0.0f);
  if (lane < n2) {
    const u4* blk = reinterpret_cast<const u4*>(Dc) + ((size_t)s * 9 + d) * h16_chunks(n2) * n2 + lane;
    const cx<float>* v = in + (size_t)nb * n2;
#pragma unroll 4
    for (int j = 0; j < n2; j += 4) {
      union {
        u4 q;
        cxh<H> v[4];
      } x;
      x.q = blk[(size_t)(j >> 2) * n2];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (j + e < n2) cmadd(acc, h2f(x.v[e]), v[j + e]);
    }
    const float sc = Dcs[(size_t)s * 9 + d];
    acc = mk(sc * acc.re, sc * acc.im);
  }
  part[d][lane] = acc;
  __syncthreads();
  if (d == 0 && lane < n2) {
    cx<float> t = part[8][lane];
#pragma unroll
    for (int dd = 0; dd < 8; ++dd) t = t + part[dd][lane];
    out[(size_t)s * n2 + lane] = t;
  }
}

// ---- batched application on the matrix cores ---------------------------------
// For a batch the coarse operator at one site is, per direction, a complex GEMM
// of the (n2 x n2) block with the neighbour's n2 x nrhs values.  One workgroup
// per site and 16 right-hand sides; its W waves share the nine directions,
// every wave holding all RT = ceil(n2 / 16) row tiles, so a block entry is
// loaded once, straight from memory into the operand's lanes, and no operand
// passes through LDS.  The waves' sums meet in LDS at the end, in wave order.
// Many sites: W = 3 (three directions per wave keep loads in flight while
// products run).  Few sites: W = 9, one direction per wave.  The tiles of
// right-hand sides of a site follow each other on one XCD, whose L2 then holds
// its blocks: two tiles in one workgroup are 1% slower (BF16, 32 rhs), and a wave
// per row tile, which loads the vectors once per wave, takes three times as long.
//
// FP64 / FP32 (v_mfma 16x16x4): four real products per complex one; a lane
// group supplies columns 4 g + u of a block of 16 in step u for both operands,
// so a lane's values of one right-hand side are contiguous.
// 16 bits (v_mfma 16x16x32): a block row's (re, im) pairs are the operand as
// stored; the values enter twice, as (re, -im) for the real and (im, re) for
// the imaginary part.  They are rounded to 16 bits per column and direction:
// in FP16 after scaling the column into [-1, 1] by its largest magnitude (the
// format's range is narrow), in BF16 as they are (it has FP32's range); the
// direction's product is accumulated from zero and added times the block (and
// FP16 column) scale.
//
// Bound: the blocks (215 MB in 16 bits, 430 in FP32, 860 in FP64 at 2592
// sites, nv 24) and the loads of the vectors, nine per value.  BF16 35 us for 2
// right-hand sides, 44 for 16, 73 for 32 (a kernel with both operands staged in
// LDS: 134, 159, 170), FP32 91, 101, 155 (715, 724, 835), FP64 173, 198, 296
// (808, 924, 1249).
template <typename R>
struct BlocksFull {
  using T = R;
  static constexpr bool kHalf = false;
  const cx<R>* Dc;
};
template <typename H>
struct BlocksHalf {
  using T = float;
  using Half = H;
  static constexpr bool kHalf = true;
  const cxh<H>* Dc;
  const float* scale;
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
template <typename H>
__device__ __forceinline__ Mma<float>::acc_t mma32(u4 a, u4 b, Mma<float>::acc_t c) {
  if constexpr (std::is_same<H, bf16_t>::value)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                   0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
}

template <class B, class Lay, int RT, int W>
__global__ __launch_bounds__(64 * W) void k_coarse_mm(Geom g, int n2, int nrhs, B blocks,
                                                      Lay lay, const cx<typename B::T>* __restrict__ in,
                                                      cx<typename B::T>* __restrict__ out,
                                                      cx<typename B::T>* __restrict__ copy) {
  using R = typename B::T;
  using acc_t = typename Mma<R>::acc_t;
  __shared__ acc_t part[W][2][64];
  // the right-hand-side tiles of a site run back to back on one XCD (blocks are
  // dealt to the eight XCDs in turn), each XCD on a contiguous range of sites
  const int ntile = (nrhs + 15) / 16, per = (g.vol + 7) / 8;
  const int s = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3) / ntile;
  const int q0 = (int)(blockIdx.x >> 3) % ntile * 16;
  if (s >= g.vol || (int)(blockIdx.x >> 3) >= per * ntile) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4, q = q0 + li;
  int c[4];
  coords_of(g, s, c);
  acc_t re[RT], im[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    re[i] = acc_t{0, 0, 0, 0};
    im[i] = acc_t{0, 0, 0, 0};
  }
  auto direction = [&](int d) __attribute__((always_inline)) {
    const int nb = d == 8 ? s : ((d & 1) ? nbr_bwd(g, s, c, d >> 1) : nbr_fwd(g, s, c, d >> 1));
    // four consecutive columns of the neighbour's values of rhs q
    auto values = [&](int col, cx<R> (&b)[4]) {
      const int qc = min(q, nrhs - 1);
      if constexpr (sizeof(R) == 4 && std::is_same<Lay, RhsMajor>::value) {
        // two numbers a load (n2 is even); it is the count of loads that bounds FP32 vectors
        typedef float f4 __attribute__((ext_vector_type(4), aligned(8)));
#pragma unroll
        for (int u = 0; u < 4; u += 2) {
          const f4 x = *reinterpret_cast<const f4*>(in + lay.at(qc, nb, min(col + u, n2 - 2), n2));
          const bool on = q < nrhs && col + u < n2;
          b[u] = on ? mk(x.x, x.y) : mk(0.0f, 0.0f);
          b[u + 1] = on ? mk(x.z, x.w) : mk(0.0f, 0.0f);
        }
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const cx<R> x = in[lay.at(qc, nb, min(col + u, n2 - 1), n2)];
          if (copy && d == 8 && q < nrhs && col + u < n2) copy[lay.at(q, s, col + u, n2)] = x;
          b[u] = q < nrhs && col + u < n2 ? x : mk<R>(0, 0);
        }
      }
    };
    if constexpr (!B::kHalf) {
      const cx<R>* blk = blocks.Dc + ((size_t)s * 9 + d) * n2 * n2;
#pragma unroll 1
      for (int kb = 0; kb < RT; ++kb) {
        const int col = 16 * kb + 4 * lk;
        cx<R> b[4], a[4][RT];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < RT; ++i) a[u][i] = blk[(size_t)min(col + u, n2 - 1) * n2 + min(16 * i + li, n2 - 1)];
        values(col, b);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < RT; ++i) {
            re[i] = Mma<R>::mma(a[u][i].re, b[u].re, re[i]);
            im[i] = Mma<R>::mma(a[u][i].re, b[u].im, im[i]);
            re[i] = Mma<R>::mma(-a[u][i].im, b[u].im, re[i]);
            im[i] = Mma<R>::mma(a[u][i].im, b[u].re, im[i]);
          }
      }
    } else {
      using H = typename B::Half;
      const int nch = h16_chunks(n2);
      const u4* blk = reinterpret_cast<const u4*>(blocks.Dc) + ((size_t)s * 9 + d) * nch * n2;
      u4 a[RT][RT];
#pragma unroll
      for (int kb = 0; kb < RT; ++kb)
#pragma unroll
        for (int i = 0; i < RT; ++i) a[kb][i] = blk[(size_t)min(4 * kb + lk, nch - 1) * n2 + min(16 * i + li, n2 - 1)];
      const float f = blocks.scale[(size_t)s * 9 + d];
      cx<float> b[RT][4];
#pragma unroll
      for (int kb = 0; kb < RT; ++kb) values(16 * kb + 4 * lk, b[kb]);
      float fs16 = f, inv = 1.0f;
      if constexpr (!std::is_same<H, bf16_t>::value) {
        // largest magnitude of the column: this lane's values, then the four lane groups
        float m = 0.0f;
#pragma unroll
        for (int kb = 0; kb < RT; ++kb)
#pragma unroll
          for (int u = 0; u < 4; ++u) m = fmaxf(m, fmaxf(fabsf(b[kb][u].re), fabsf(b[kb][u].im)));
        m = fmaxf(m, __shfl_xor(m, 16, 64));
        m = fmaxf(m, __shfl_xor(m, 32, 64));
        fs16 = f * quant_scale(m, inv);
      }
      acc_t tr[RT], ti_[RT];
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        tr[i] = acc_t{0, 0, 0, 0};
        ti_[i] = acc_t{0, 0, 0, 0};
      }
#pragma unroll
      for (int kb = 0; kb < RT; ++kb) {
        u4 b1, b2;  // (re, -im) and (im, re) of four columns
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float br = b[kb][u].re, bi = b[kb][u].im;
          if constexpr (!std::is_same<H, bf16_t>::value) {
            br *= inv;
            bi *= inv;
          }
          const unsigned w = __builtin_bit_cast(unsigned, f2h<H>(br, bi));
          b1[u] = w ^ 0x80000000u;
          b2[u] = (w << 16) | (w >> 16);
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          tr[i] = mma32<H>(a[kb][i], b1, tr[i]);
          ti_[i] = mma32<H>(a[kb][i], b2, ti_[i]);
        }
      }
      // FP16 result columns belong to right-hand side li, as the scale does
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          re[i][r] += fs16 * tr[i][r];
          im[i][r] += fs16 * ti_[i][r];
        }
    }
  };
  // Unrolled, the next direction's loads go out before this one's products: in
  // 16 bits 44 against 53 us (2592 sites, nv 24, 16 rhs); in FP64 its registers
  // cost more than that brings (218 against 198 us).
  if constexpr (B::kHalf) {
#pragma unroll
    for (int k = 0; k < 9 / W; ++k) direction(wave + k * W);
  } else {
#pragma unroll 1
    for (int d = wave; d < 9; d += W) direction(d);
  }
  // row tile i summed over the waves by wave i % W
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    if (i > 0) __syncthreads();
    part[wave][0][lane] = re[i];
    part[wave][1][lane] = im[i];
    __syncthreads();
    if (wave == i % W && q < nrhs) {
      acc_t sr = part[0][0][lane], si = part[0][1][lane];
#pragma unroll
      for (int w = 1; w < W; ++w) {
        sr += part[w][0][lane];
        si += part[w][1][lane];
      }
      if constexpr (sizeof(R) == 4 && std::is_same<Lay, RhsMajor>::value) {
        typedef float f4 __attribute__((ext_vector_type(4), aligned(8)));
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          const int row = 16 * i + Mma<R>::row(lk, r);
          if (row < n2) *reinterpret_cast<f4*>(out + lay.at(q, s, row, n2)) = f4{sr[r], si[r], sr[r + 1], si[r + 1]};
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * i + Mma<R>::row(lk, r);
          if (row < n2) out[lay.at(q, s, row, n2)] = mk<R>(sr[r], si[r]);
        }
      }
    }
  }
}

// ---- coarsest-level GCR in three launches per iteration -------------------------
// GCR(k) on D_c in FP64 for a batch of right-hand sides, each with its own
// coefficients and stopping test (Sec. 2: the coarsest solve).  Iteration j:
//   K1  w_j = D_c r, z_j = r, and per workgroup partial sums of
//       c_i = <W_i, w_j>, d_i = <W_i, r> (i < j), <w_j, w_j>, <w_j, r>, <r, r>
//   K2  (one workgroup per rhs) the sums in a fixed order; h_i = c_i / |W_i|^2;
//       |w'|^2 = <w,w> - sum |c_i|^2 / |W_i|^2 and <w', r> = <w, r> - sum h_i^* d_i
//       for w' = w_j - sum h_i W_i (classical Gram-Schmidt, the W_i orthogonal);
//       a = <w', r> / |w'|^2; a right-hand side with |r| <= tol |b| is frozen
//   K3  w_j = w', z_j -= sum h_i Z_i, x += a z_j, r -= a w_j, and partial sums
//       of the exact |w_j|^2, which K2 of the next iteration stores as |W_j|^2.
// The stopping test is thus lagged by one iteration; the per-rhs active flags
// go to pinned host memory, where the host inspects them two iterations
// later, so it never waits for the GPU inside the solve.
constexpr int kCgcrG1 = 4096;  // workgroups of K1 (one coarse site each up to this many sites)
constexpr int kCgcrG3 = 64;   // chunks per rhs of K3
// Most K1 workgroups whose partials K3 adds up by itself (256 sites, nv 20, 10
// iterations: 6.7 us against 9.6 and a launch with K2 on its own; the partials of
// 4096 workgroups would be 50 MB of reads).
constexpr int kCgcrFusedG1 = 512;

struct CgcrState {  // per-rhs device scalars of one solve (inside the level's scalar block)
  double* h;    // [rhs][2 kMaxKrylov]
  double* nrm;  // [rhs][kMaxKrylov]
  double* a;    // [rhs][2]
  double* rn;   // [rhs]
  double* act;  // [rhs]
  double* tol2; // [rhs]
};

// x = 0, r = b, tol2 = tol^2 |b|^2, active = |b| > 0 (one workgroup per rhs)
__global__ __launch_bounds__(1024) void k_cgcr_init(const cx<double>* __restrict__ b, cx<double>* __restrict__ x,
                                                   cx<double>* __restrict__ r, size_t n, double tol, CgcrState S,
                                                   double* err) {
  __shared__ double red[16];
  const int q = blockIdx.x;
  const size_t o = (size_t)q * n;
  double v[1] = {0.0};
  for (size_t e = threadIdx.x; e < n; e += blockDim.x) {
    const cx<double> bv = b[o + e];
    x[o + e] = mk(0.0, 0.0);
    r[o + e] = bv;
    v[0] += bv.re * bv.re + bv.im * bv.im;
  }
  block_sum<1>(v, red);
  if (threadIdx.x == 0) {
    if (!isfinite(v[0])) err[0] = 1.0;
    S.tol2[q] = tol * tol * v[0];
    S.act[q] = v[0] > 0.0 && isfinite(v[0]) ? 1.0 : 0.0;
    S.rn[q] = v[0];
  }
}

// K1 of a single rhs: grid-stride over sites, nine waves (one per block of
// the stencil), then the dot products of w_j with the basis and r: wave t
// takes basis vectors t, t + 9, ... and the norms come last.  w_j stays in LDS
// for them, and a wave's first basis vector and r are on their way during the
// product (256 sites, nv 20, ten iterations: 13.1 us, 10.6 of them the product
// with its 59 MB of blocks; 13.6 us with w_j read back from memory).
__global__ __launch_bounds__(576) void k_cgcr_apply(Geom g, int n2, int j, int vals,
                                                    const cx<double>* __restrict__ Dc, const cx<double>* r,
                                                    const cx<double>* Wb, cx<double>* w, cx<double>* z,
                                                    double* part) {
  extern __shared__ __align__(16) char dyn1[];
  double* acc = reinterpret_cast<double*>(dyn1);  // [vals]
  __shared__ double lds[2 * 9 * 64];
  __shared__ cx<double> ws[64];
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6, lane = threadIdx.x & 63;
  const size_t bs = (size_t)g.vol * n2;
  const bool on = lane < n2;
  for (int t = threadIdx.x; t < vals; t += blockDim.x) acc[t] = 0.0;
  for (int s = blockIdx.x; s < g.vol; s += gridDim.x) {
    const size_t o = (size_t)s * n2 + lane;
    const cx<double> rv = on ? r[o] : mk(0.0, 0.0);
    cx<double> u = on && wave < j ? Wb[(size_t)wave * bs + o] : mk(0.0, 0.0);
    if (wave == 8 && on) z[o] = rv;
    // ends with a block barrier: w_j of site s is then complete
    apply_site_valu1(g, n2, s, Dc, r, w, lds, ws);
    const cx<double> wv = on ? ws[lane] : mk(0.0, 0.0);
    // a basis vector keeps its wave for every site of the loop, so each
    // accumulator has a single writer
    for (int i = wave; i <= j; i += nw) {
      if (i < j) {
        if (i != wave) u = on ? Wb[(size_t)i * bs + o] : mk(0.0, 0.0);
        const double c_re = wave_sum(u.re * wv.re + u.im * wv.im);
        const double c_im = wave_sum(u.re * wv.im - u.im * wv.re);
        const double d_re = wave_sum(u.re * rv.re + u.im * rv.im);
        const double d_im = wave_sum(u.re * rv.im - u.im * rv.re);
        if (lane == 0) {
          acc[2 * i] += c_re;
          acc[2 * i + 1] += c_im;
          acc[2 * j + 2 * i] += d_re;
          acc[2 * j + 2 * i + 1] += d_im;
        }
      } else {
        const double ww = wave_sum(wv.re * wv.re + wv.im * wv.im);
        const double wr_re = wave_sum(wv.re * rv.re + wv.im * rv.im);
        const double wr_im = wave_sum(wv.re * rv.im - wv.im * rv.re);
        const double rr = wave_sum(rv.re * rv.re + rv.im * rv.im);
        if (lane == 0) {
          acc[4 * j] += ww;
          acc[4 * j + 1] += wr_re;
          acc[4 * j + 2] += wr_im;
          acc[4 * j + 3] += rr;
        }
      }
    }
    __syncthreads();
  }
  for (int t = threadIdx.x; t < vals; t += blockDim.x) part[(size_t)blockIdx.x * vals + t] = acc[t];
}

// K2 on T threads for rhs q.  vals = 4 j + 4 partial values per K1 workgroup;
// p3: K3's g3 partial |w_{j-1}|^2 per rhs (j > 0).  On return h_i is in
// hs[2 i] for every thread, and lane 0 of wave 0 has the rest.
struct CgcrCoef {
  cx<double> a;
  double rr;
  bool on, bad;
};
template <int T>
__device__ __forceinline__ CgcrCoef cgcr_coef(int q, int j, int vals, int g1, const double* __restrict__ part,
                                              const double* __restrict__ p3, int g3, int kmax, const CgcrState& S,
                                              double* tot, double* hs) {
  __shared__ double sub[T];  // [groups][vals]
  const int wave = threadIdx.x >> 6, nw = T / 64, lane = threadIdx.x & 63;
  // thread (group, value) sums every groups-th partial of its value, so that
  // a sweep of the threads reads one run of memory; vals <= 4 kMaxKrylov <= T
  const int groups = T / vals, v0 = threadIdx.x % vals, g0 = threadIdx.x / vals;
  double n3 = 0.0;
  if (wave == nw - 1 && j > 0)
    for (int b = lane; b < g3; b += 64) n3 += p3[(size_t)q * g3 + b];
  if (g0 < groups) {
    const double* p = part + (size_t)q * g1 * vals + v0;
    double s = 0.0;
#pragma unroll 8
    for (int b = g0; b < g1; b += groups) s += p[(size_t)b * vals];
    sub[g0 * vals + v0] = s;
  }
  __syncthreads();
  for (int v = wave; v < vals; v += nw) {
    double s = 0.0;
    for (int b = lane; b < groups; b += 64) s += sub[b * vals + v];
    s = wave_sum(s);
    if (lane == 0) tot[v] = s;
  }
  if (wave == nw - 1) {
    n3 = wave_sum(n3);
    if (lane == 0) tot[vals] = n3;
  }
  __syncthreads();
  CgcrCoef c;
  c.rr = tot[4 * j + 3];
  double ww = 0.0, wr_re = 0.0, wr_im = 0.0;
  if (wave == 0) {
    const double* nrm = S.nrm + (size_t)q * kmax;
    for (int i = lane; i < j; i += 64) {
      const double ni = i == j - 1 ? tot[vals] : nrm[i];
      const double cr = tot[2 * i], ci = tot[2 * i + 1];
      const double hr = ni > 0.0 ? cr / ni : 0.0, hi = ni > 0.0 ? ci / ni : 0.0;
      hs[2 * i] = hr;
      hs[2 * i + 1] = hi;
      ww += hr * cr + hi * ci;  // |c_i|^2 / |W_i|^2
      const double dr = tot[2 * j + 2 * i], di = tot[2 * j + 2 * i + 1];
      wr_re += hr * dr + hi * di;  // conj(h_i) d_i
      wr_im += hr * di - hi * dr;
    }
    ww = tot[4 * j] - wave_sum(ww);
    wr_re = tot[4 * j + 1] - wave_sum(wr_re);
    wr_im = tot[4 * j + 2] - wave_sum(wr_im);
    if (lane == 0) {
      sub[0] = ww;
      sub[1] = wr_re;
      sub[2] = wr_im;
    }
  }
  __syncthreads();
  ww = sub[0];
  c.bad = !isfinite(c.rr) || !isfinite(ww);
  c.on = S.act[q] != 0.0 && c.rr > S.tol2[q];
  const bool ok = c.on && ww > 1e-28 * tot[4 * j];
  c.a = ok ? mk(sub[1] / ww, sub[2] / ww) : mk(0.0, 0.0);
  return c;
}

// What K2 leaves for the host and for later iterations (one thread).
__device__ __forceinline__ void cgcr_record(int q, int j, int kmax, const CgcrCoef& c, double n3, const CgcrState& S,
                                            double* host_act, double* err) {
  if (j > 0) S.nrm[(size_t)q * kmax + j - 1] = n3;
  S.rn[q] = c.rr;
  if (c.bad) err[0] = 1.0;
  S.act[q] = c.on ? 1.0 : 0.0;
  S.a[2 * q] = c.a.re;
  S.a[2 * q + 1] = c.a.im;
  if (host_act) host_act[q] = c.on ? 1.0 : 0.0;
}

// K2 of its own, one workgroup per rhs.
// hist (batched solves, else null): per rhs and iteration j, the h_i of
// iteration j at [2 i], a_j at [2 kmax]; stride 2 kmax + 4 doubles per j.
__global__ __launch_bounds__(1024) void k_cgcr_coef(int j, int vals, int g1, const double* __restrict__ part,
                                                    const double* __restrict__ p3, int g3, int kmax, CgcrState S,
                                                    double* host_act, double* err, double* hist) {
  extern __shared__ __align__(16) char dyn2[];
  double* tot = reinterpret_cast<double*>(dyn2);  // [vals + 1]
  __shared__ double hs[2 * kMaxKrylov];
  const int q = blockIdx.x;
  const CgcrCoef c = cgcr_coef<1024>(q, j, vals, g1, part, p3, g3, kmax, S, tot, hs);
  double* h = S.h + (size_t)q * 2 * kmax;
  double* hj = hist ? hist + ((size_t)q * kmax + j) * (2 * kmax + 4) : nullptr;
  if (threadIdx.x < 2 * j) {
    h[threadIdx.x] = hs[threadIdx.x];
    if (hist) hj[threadIdx.x] = hs[threadIdx.x];
  }
  if (threadIdx.x != 0) return;
  if (hist) {
    hj[2 * kmax] = c.a.re;
    hj[2 * kmax + 1] = c.a.im;
  }
  cgcr_record(q, j, kmax, c, tot[vals], S, host_act, err);
}

// K3: blocks (kCgcrG3 chunks, rhs); p3 and p3n: the partial |w|^2 of the
// iteration before and of this one.  COEF (one rhs): every workgroup does K2
// for itself first, in the same order, and the first records it -- worth a
// launch as long as the partials are few (see kCgcrFusedG1).  The others may
// read act before or after it is recorded: recorded, it only holds what they
// find themselves.
constexpr int kCgcrK3 = 512;
template <bool COEF>
__global__ __launch_bounds__(kCgcrK3) void k_cgcr_update(size_t n, int nrhs, int j, int kmax, const cx<double>* Wb,
                                                         const cx<double>* Zb, cx<double>* w, cx<double>* z,
                                                         cx<double>* x, cx<double>* r, CgcrState S, double* p3n,
                                                         int vals, int g1, const double* __restrict__ part,
                                                         const double* p3, double* host_act, double* err) {
  __shared__ double red[kCgcrK3 / 64];
  __shared__ double hs[2 * kMaxKrylov];
  __shared__ double tot[4 * kMaxKrylov + 1];
  const int q = blockIdx.y;
  cx<double> a;
  bool on;
  if constexpr (COEF) {
    const CgcrCoef c = cgcr_coef<kCgcrK3>(q, j, vals, g1, part, p3, kCgcrG3, kmax, S, tot, hs);
    a = c.a;
    on = c.on;
    if (blockIdx.x == 0 && threadIdx.x == 0) cgcr_record(q, j, kmax, c, tot[vals], S, host_act, err);
  } else {
    on = S.act[q] != 0.0;
    a = mk(S.a[2 * q], S.a[2 * q + 1]);
    const double* h = S.h + (size_t)q * 2 * kmax;
    for (int t = threadIdx.x; t < 2 * j; t += blockDim.x) hs[t] = h[t];
    __syncthreads();
  }
  if (!on) {
    if (threadIdx.x == 0) p3n[(size_t)q * kCgcrG3 + blockIdx.x] = 0.0;
    return;
  }
  const size_t bs = (size_t)nrhs * n, o = (size_t)q * n;
  const size_t cs = (n + kCgcrG3 - 1) / kCgcrG3, e0 = blockIdx.x * cs, e1 = e0 + cs < n ? e0 + cs : n;
  double v[1] = {0.0};
  for (size_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
    cx<double> wv = w[o + e], zv = z[o + e];
#pragma unroll 4
    for (int i = 0; i < j; ++i) {
      const cx<double> hi = mk(hs[2 * i], hs[2 * i + 1]);
      wv = wv - hi * Wb[(size_t)i * bs + o + e];
      zv = zv - hi * Zb[(size_t)i * bs + o + e];
    }
    w[o + e] = wv;
    z[o + e] = zv;
    x[o + e] = x[o + e] + a * zv;
    r[o + e] = r[o + e] - a * wv;
    v[0] += wv.re * wv.re + wv.im * wv.im;
  }
  block_sum<1>(v, red);
  if (threadIdx.x == 0) p3n[(size_t)q * kCgcrG3 + blockIdx.x] = v[0];
}

// ---- the same solve for a batch of rhs in the rhs-fast layout ---------------
// Vectors of the batch are stored [site][row][rhs] for the whole solve, so the
// matrix-core operand of one row and 16 rhs is one contiguous 256-byte run.
// K1 is the batched operator above: 113 us at 2304 sites, nv 24, 16 rhs (135 us
// for a kernel that staged both operands in LDS), 12.7 us (14.4) at 162 sites,
// nv 16.
// Threads of a workgroup form a (rows x nrhs) grid, thread t handling rhs
// t % nrhs at positions (site, row) t / nrhs, t / nrhs + R, ... of the
// workgroup's chunk; sums over those positions meet in LDS, per rhs.
constexpr int kCgcrG3T = 1024;   // workgroups (chunks) of the rhs-fast update: four per CU
constexpr int kCgcrDotIG = 4;    // basis vectors per pass of the dot kernel

// Sums v over the threads of each rhs column; thread q < nrhs receives its total.
__device__ __forceinline__ double rhs_column_sum(double v, int nrhs, int rows, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  double sum = 0.0;
  if ((int)threadIdx.x < nrhs)
    for (int rr = 0; rr < rows; ++rr) sum += red[rr * nrhs + threadIdx.x];
  __syncthreads();
  return sum;
}

// The same for K values per thread at once (red holds K x 256 doubles): value
// k of rhs q is summed by thread k * nrhs + q (looping when K * nrhs > 256)
// and handed to put(k, q, sum).
template <int K, class Put>
__device__ __forceinline__ void rhs_column_sums(const double (&v)[K], int nrhs, int rows, double* red, Put put) {
#pragma unroll
  for (int k = 0; k < K; ++k) red[k * 256 + threadIdx.x] = v[k];
  __syncthreads();
  for (int u = threadIdx.x; u < K * nrhs; u += 256) {
    const int k = u / nrhs, q = u % nrhs;
    double sum = 0.0;
    for (int rr = 0; rr < rows; ++rr) sum += red[k * 256 + rr * nrhs + q];
    put(k, q, sum);
  }
  __syncthreads();
}

// r = b and x = 0 in the rhs-fast layout; partial |b_q|^2 per workgroup.
__global__ __launch_bounds__(256) void k_cgcrT_init(size_t npos, int nrhs, const cx<double>* __restrict__ b,
                                                    cx<double>* __restrict__ xT, cx<double>* __restrict__ rT,
                                                    double* p3) {
  __shared__ double red[256];
  const int rows = 256 / nrhs, q = threadIdx.x % nrhs, rho = threadIdx.x / nrhs;
  const size_t cs = (npos + gridDim.x - 1) / gridDim.x, p0 = blockIdx.x * cs, p1 = p0 + cs < npos ? p0 + cs : npos;
  double v = 0.0;
  if (rho < rows) {
    for (size_t p = p0 + rho; p < p1; p += rows) {
      const cx<double> bv = b[(size_t)q * npos + p];
      rT[p * nrhs + q] = bv;
      xT[p * nrhs + q] = mk(0.0, 0.0);
      v += bv.re * bv.re + bv.im * bv.im;
    }
  }
  const double sum = rhs_column_sum(v, nrhs, rows, red);
  if ((int)threadIdx.x < nrhs) p3[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = sum;
}

// tol2 = tol^2 |b|^2, active = |b| > 0, from the init partials.
// One wave per rhs sums the g partials.
__global__ __launch_bounds__(64) void k_cgcrT_init_fin(int nrhs, int g, const double* __restrict__ p3, double tol,
                                                       CgcrState S, double* err) {
  const int q = blockIdx.x;
  double v = 0.0;
  for (int b = threadIdx.x; b < g; b += 64) v += p3[(size_t)q * g + b];
  v = wave_sum(v);
  if (threadIdx.x != 0) return;
  if (!isfinite(v)) err[0] = 1.0;
  S.tol2[q] = tol * tol * v;
  S.act[q] = v > 0.0 && isfinite(v) ? 1.0 : 0.0;
  S.rn[q] = v;
}

// x (canonical) = xT.
__global__ __launch_bounds__(256) void k_cgcrT_out(size_t npos, int nrhs, const cx<double>* __restrict__ xT,
                                                   cx<double>* __restrict__ x) {
  const size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (e >= npos * nrhs) return;
  const size_t p = e / nrhs;
  const int q = (int)(e % nrhs);
  x[(size_t)q * npos + p] = xT[e];
}

// Dots (rhs-fast): partial c_i = <W_i, w>, d_i = <W_i, r> (i < j) and
// |w|^2, <w, r>, |r|^2 of one chunk of positions, stored in the value order of
// k_cgcr_coef.  Basis vectors are taken kCgcrDotIG per pass over the chunk.
__global__ __launch_bounds__(256) void k_cgcrT_dots(size_t npos, int nrhs, int j, int vals,
                                                    const cx<double>* __restrict__ Wb,
                                                    const cx<double>* __restrict__ w,
                                                    const cx<double>* __restrict__ r, double* part) {
  __shared__ double red[4 * kCgcrDotIG * 256];
  const int rows = 256 / nrhs, q = threadIdx.x % nrhs, rho = threadIdx.x / nrhs;
  const bool on = rho < rows;
  const size_t bs = npos * nrhs;
  const size_t cs = (npos + gridDim.x - 1) / gridDim.x, p0 = blockIdx.x * cs, p1 = p0 + cs < npos ? p0 + cs : npos;
  auto out = [&](int qq) { return part + ((size_t)qq * gridDim.x + blockIdx.x) * vals; };
  for (int i0 = 0; i0 == 0 || i0 < j; i0 += kCgcrDotIG) {
    const int ni = j - i0 < kCgcrDotIG ? j - i0 : kCgcrDotIG;
    double a[kCgcrDotIG][4] = {}, nv[4] = {};
    if (on) {
      for (size_t p = p0 + rho; p < p1; p += rows) {
        const size_t e = p * nrhs + q;
        const cx<double> wv = w[e], rv = r[e];
        if (i0 == 0) {
          nv[0] += wv.re * wv.re + wv.im * wv.im;
          nv[1] += wv.re * rv.re + wv.im * rv.im;
          nv[2] += wv.re * rv.im - wv.im * rv.re;
          nv[3] += rv.re * rv.re + rv.im * rv.im;
        }
#pragma unroll
        for (int u = 0; u < kCgcrDotIG; ++u) {
          if (u < ni) {
            const cx<double> bv = Wb[(size_t)(i0 + u) * bs + e];
            a[u][0] += bv.re * wv.re + bv.im * wv.im;
            a[u][1] += bv.re * wv.im - bv.im * wv.re;
            a[u][2] += bv.re * rv.re + bv.im * rv.im;
            a[u][3] += bv.re * rv.im - bv.im * rv.re;
          }
        }
      }
    }
    // value k = 4 u + c of this pass: c = 0, 1 -> c_i (re, im), 2, 3 -> d_i
    double flat[4 * kCgcrDotIG];
#pragma unroll
    for (int u = 0; u < kCgcrDotIG; ++u)
#pragma unroll
      for (int cc = 0; cc < 4; ++cc) flat[4 * u + cc] = a[u][cc];
    rhs_column_sums<4 * kCgcrDotIG>(flat, nrhs, rows, red, [&](int k, int qq, double sum) {
      const int u = k >> 2, cc = k & 3, i = i0 + u;
      if (u < ni) out(qq)[cc < 2 ? 2 * i + cc : 2 * j + 2 * i + (cc - 2)] = sum;
    });
    if (i0 == 0)
      rhs_column_sums<4>(nv, nrhs, rows, red, [&](int k, int qq, double sum) { out(qq)[4 * j + k] = sum; });
  }
}

// K3 (rhs-fast): w' = w - sum h_i W_i, z' = z - sum h_i Z_i, x += a z',
// r -= a w', partial |w'|^2 per rhs; frozen rhs are left unchanged.
// K3 (rhs-fast): w_j -= sum_i h_i W_i (kept, with |w_j|^2 for the next
// iteration) and r -= a w_j.  The search directions stay unorthogonalised
// (z_j = r_j as K1 copied it) and x is formed once per cycle by
// k_cgcrT_backsolve + k_cgcrT_combine from the recorded h and a.
__global__ __launch_bounds__(256) void k_cgcrT_update(size_t npos, int nrhs, int j, int kmax,
                                                      const cx<double>* __restrict__ Wb, cx<double>* __restrict__ w,
                                                      cx<double>* __restrict__ r, CgcrState S, double* p3) {
  __shared__ double red[256];
  const int rows = 256 / nrhs, q = threadIdx.x % nrhs, rho = threadIdx.x / nrhs;
  const bool on = rho < rows && S.act[q] != 0.0;
  const size_t bs = npos * nrhs;
  const size_t cs = (npos + gridDim.x - 1) / gridDim.x, p0 = blockIdx.x * cs, p1 = p0 + cs < npos ? p0 + cs : npos;
  double v = 0.0;
  if (on) {
    const double* h = S.h + (size_t)q * 2 * kmax;
    const cx<double> a = mk(S.a[2 * q], S.a[2 * q + 1]);
    for (size_t p = p0 + rho; p < p1; p += rows) {
      const size_t e = p * nrhs + q;
      cx<double> wv = w[e];
#pragma unroll 4
      for (int i = 0; i < j; ++i) wv = wv - mk(h[2 * i], h[2 * i + 1]) * Wb[(size_t)i * bs + e];
      w[e] = wv;
      r[e] = r[e] - a * wv;
      v += wv.re * wv.re + wv.im * wv.im;
    }
  }
  const double sum = rhs_column_sum(v, nrhs, rows, red);
  if ((int)threadIdx.x < nrhs) p3[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = sum;
}

// With orthogonalised directions z_m = z~_m - sum_{i<m} h_{m,i} z_i, the
// cycle's update sum_m a_m z_m equals sum_m y_m z~_m for
// y_m = a_m - sum_{i>m} y_i h_{i,m}, taken from the last direction down.
// One thread per rhs; y_m lands at [2 kmax + 2] of row m of the history.
__global__ __launch_bounds__(64) void k_cgcrT_backsolve(int nrhs, int J, int kmax, double* __restrict__ hist) {
  const int q = threadIdx.x;
  if (q >= nrhs) return;
  const size_t st = 2 * (size_t)kmax + 4;
  double* hq = hist + (size_t)q * kmax * st;
  for (int m = J - 1; m >= 0; --m) {
    cx<double> y = mk(hq[m * st + 2 * kmax], hq[m * st + 2 * kmax + 1]);
    for (int i = m + 1; i < J; ++i)
      y = y - mk(hq[i * st + 2 * kmax + 2], hq[i * st + 2 * kmax + 3]) * mk(hq[i * st + 2 * m], hq[i * st + 2 * m + 1]);
    hq[m * st + 2 * kmax + 2] = y.re;
    hq[m * st + 2 * kmax + 3] = y.im;
  }
}

// x += sum_{m<J} y_m z~_m (rhs-fast vectors, element e belongs to rhs e % nrhs).
__global__ __launch_bounds__(256) void k_cgcrT_combine(size_t npos, int nrhs, int J, int kmax,
                                                       const cx<double>* __restrict__ Zb,
                                                       const double* __restrict__ hist, cx<double>* __restrict__ x) {
  const size_t bs = npos * nrhs;
  const size_t st = 2 * (size_t)kmax + 4;
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < bs; e += (size_t)gridDim.x * blockDim.x) {
    const double* yq = hist + (size_t)(e % nrhs) * kmax * st + 2 * kmax + 2;
    cx<double> xv = x[e];
    for (int m = 0; m < J; ++m) xv = xv + mk(yq[m * st], yq[m * st + 1]) * Zb[(size_t)m * bs + e];
    x[e] = xv;
  }
}

template <int RT, int W, class B, class Lay>
void launch_coarse_mm(Ctx& c, const Level& cl, const B& blocks, const Lay& lay, const cx<typename B::T>* in,
                      cx<typename B::T>* out, cx<typename B::T>* copy, int nrhs) {
  hipLaunchKernelGGL((k_coarse_mm<B, Lay, RT, W>), dim3(8 * ((cl.nsite + 7) / 8) * ((nrhs + 15) / 16)), dim3(64 * W),
                     0, c.stream, cl.g, cl.dof, nrhs, blocks, lay, in, out, copy);
}

// out = D_c in for a batch, and copy = in where given (dof <= 64).
template <class B, class Lay>
void coarse_mm(Ctx& c, const Level& cl, const B& blocks, const Lay& lay, const cx<typename B::T>* in,
               cx<typename B::T>* out, cx<typename B::T>* copy, int nrhs) {
  // Nine waves per workgroup pay where a workgroup has a compute unit to itself
  // (256 sites, nv 20, 16 rhs: FP32 14.0 us against 16.2, FP64 22.9 against
  // 24.9; at 32 rhs FP32 25.1 against 24.3).
  const bool nine = (long long)cl.nsite * ((nrhs + 15) / 16) <= c.ncu;
#define MM(RT)                                                             \
  do {                                                                     \
    if (nine)                                                              \
      launch_coarse_mm<RT, 9>(c, cl, blocks, lay, in, out, copy, nrhs);    \
    else                                                                   \
      launch_coarse_mm<RT, 3>(c, cl, blocks, lay, in, out, copy, nrhs);    \
  } while (0)
  switch ((cl.dof + 15) / 16) {
    case 1: MM(1); break;
    case 2: MM(2); break;
    case 3: MM(3); break;
    default: MM(4); break;
  }
#undef MM
  WDMG_HIP(hipGetLastError());
}

template <typename R>
__global__ void k_coarse_shift(cx<R>* Dc, int nsite, int n2, double dm) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nsite * n2) return;
  const int s = i / n2, r = i % n2;
  cx<R>* x = Dc + ((size_t)s * 9 + 8) * n2 * n2;
  x[(size_t)r * n2 + r].re += (R)dm;
}

template <class Side>
void launch_build(Ctx& c, const Side& side, const Level& f, Level& cl, int dof) {
  const AggGeom a = make_agg(f);
  const int n2 = 2 * f.nv;
  // LDS budget ~48 KiB: cs sites of V (dof x nv) and T (dof x cc) columns.
  int cc = n2;
  int cs = 4;
  auto bytes = [&](int cs_, int cc_) { return (size_t)cs_ * dof * (f.nv + cc_) * sizeof(cx<double>); };
  while (cs > 1 && (bytes(cs, cc) > 48 * 1024 || cs * cc > 256)) --cs;
  while (cc > 1 && (bytes(cs, cc) > 48 * 1024 || n2 * cc > 16 * 256)) cc = (cc + 1) / 2;
  const int nagg = cl.nsite;
  ProfScope ps(c, WDMG_K_DC_BUILD, nagg);
  hipLaunchKernelGGL((k_coarse_build<Side>), dim3(nagg, 9), dim3(256), bytes(cs, cc), c.stream, side, a, f.V64,
                     f.n, f.nv, dof, cs, cc, cl.Dc64);
  WDMG_HIP(hipGetLastError());
}

}  // namespace

void coarse_build0(Ctx& c, const Level& f, Level& cl) {
  WilsonSide side{c.U64, 4.0 + c.mass, c.t_bc < 0 ? 1 : 0};
  launch_build(c, side, f, cl, 12);
}

void coarse_buildC(Ctx& c, const Level& f, Level& cl) {
  StencilSide side{f.Dc64, f.dof};
  launch_build(c, side, f, cl, f.dof);
}

template <typename R>
void coarse_apply(Ctx& c, const Level& cl, const cx<R>* Dc, cx<R>* out, const cx<R>* in, int nrhs) {
  c.n_Dc[cl.l] += nrhs;
  if (nrhs >= kMfmaMinRhs && cl.dof <= 64) {
    ProfScope ps(c, sizeof(R) == 8 ? WDMG_K_DC_MFMA_F64 : WDMG_K_DC_MFMA_F32, (long long)cl.nsite * nrhs);
    coarse_mm(c, cl, BlocksFull<R>{Dc}, RhsMajor{(size_t)cl.nsite * cl.dof}, in, out, nullptr, nrhs);
    return;
  }
  ProfScope ps(c, sizeof(R) == 8 ? WDMG_K_DC_F64 : WDMG_K_DC_F32, (long long)cl.nsite * nrhs);
  hipLaunchKernelGGL((k_coarse_apply<R>), dim3(cl.nsite, nrhs), dim3(576), 0, c.stream, cl.g, cl.dof, Dc, in, out);
  WDMG_HIP(hipGetLastError());
}

void coarse_shift(Ctx& c, Level& cl, double dm) {
  if (!cl.Dc64 || !cl.Dc32) throw Error(WDMG_ERR_ARG, "coarse blocks released by wdmg_release_unused");
  const int n = cl.nsite * cl.dof;
  hipLaunchKernelGGL((k_coarse_shift<double>), dim3((n + 255) / 256), dim3(256), 0, c.stream, cl.Dc64, cl.nsite,
                     cl.dof, dm);
  WDMG_HIP(hipGetLastError());
  hipLaunchKernelGGL((k_coarse_shift<float>), dim3((n + 255) / 256), dim3(256), 0, c.stream, cl.Dc32, cl.nsite,
                     cl.dof, dm);
  WDMG_HIP(hipGetLastError());
  cl.dc16_kind = 0;  // the 16-bit copy is remade from the shifted FP64 blocks on next use
}

void ensure_dc16(Ctx& c, Level& cl, int kind) {
  const int n2 = cl.dof;
  const size_t nblk = (size_t)cl.nsite * 9, nn = (size_t)h16_chunks(n2) * n2 * 4;
  if (cl.dc16_kind != kind) {
    if (!cl.Dc64) throw Error(WDMG_ERR_ARG, "FP64 coarse blocks released by wdmg_release_unused");
    if (!cl.Dc16) cl.Dc16 = dev_alloc(c, nblk * nn * 4);
    if (!cl.Dc16s) cl.Dc16s = static_cast<float*>(dev_alloc(c, nblk * sizeof(float)));
    if (kind == WDMG_F16)
      hipLaunchKernelGGL((k_dc_to_half<f16_t>), dim3((unsigned)nblk), dim3(256), 0, c.stream, cl.Dc64,
                         static_cast<cxh<f16_t>*>(cl.Dc16), cl.Dc16s, n2);
    else
      hipLaunchKernelGGL((k_dc_to_half<bf16_t>), dim3((unsigned)nblk), dim3(256), 0, c.stream, cl.Dc64,
                         static_cast<cxh<bf16_t>*>(cl.Dc16), cl.Dc16s, n2);
    WDMG_HIP(hipGetLastError());
    cl.dc16_kind = kind;
  }
}

template <typename H>
void coarse_apply_16(Ctx& c, Level& cl, cx<float>* out, const cx<float>* in, int nrhs) {
  const cxh<H>* d16 = static_cast<const cxh<H>*>(cl.Dc16);
  if (nrhs >= kMfmaMinRhs && cl.dof <= 64) {
    ProfScope ps(c, WDMG_K_DC_MFMA_H, (long long)cl.nsite * nrhs);
    coarse_mm(c, cl, BlocksHalf<H>{d16, cl.Dc16s}, RhsMajor{(size_t)cl.nsite * cl.dof}, in, out, nullptr, nrhs);
    return;
  }
  ProfScope ps(c, WDMG_K_DC_H, (long long)cl.nsite * nrhs);
  hipLaunchKernelGGL((k_coarse_apply_h<H>), dim3(cl.nsite, nrhs), dim3(576), 0, c.stream, cl.g, cl.dof, d16, cl.Dc16s,
                     in, out);
  WDMG_HIP(hipGetLastError());
}

void coarse_apply_h(Ctx& c, Level& cl, int kind, cx<float>* out, const cx<float>* in, int nrhs) {
  ensure_dc16(c, cl, kind);
  c.n_Dc[cl.l] += nrhs;
  if (kind == WDMG_F16)
    coarse_apply_16<f16_t>(c, cl, out, in, nrhs);
  else
    coarse_apply_16<bf16_t>(c, cl, out, in, nrhs);
}

void coarsest_gcr(Ctx& c, Level& L, cx<double>* x, const cx<double>* b, int nrhs, double tol, int k, int maxit) {
  const int n2 = L.dof;
  const size_t n = L.n, bs = (size_t)nrhs * n;
  double* gb = c.dsc + gcr_base(L.l);
  CgcrState S{gb + G_H, gb + G_NRM, gb + G_A, gb + G_RN, gb + G_ACT, gb + G_TOL};
  const int g1 = L.nsite < kCgcrG1 ? L.nsite : kCgcrG1;
  if (nrhs == 1 && (size_t)(4 * k + 4) * sizeof(double) > 96 * 1024)
    throw Error(WDMG_ERR_ARG, "coarse_restart too long (LDS)");
  static bool lds_attr = false;
  if (!lds_attr) {  // the single-rhs K1 keeps 4 j + 4 partial sums in LDS
    WDMG_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_cgcr_apply),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
    lds_attr = true;
  }
  // a batch keeps its vectors rhs-fast for the whole solve (x in L.xT)
  const bool fast = nrhs >= 2;
  const size_t npos = (size_t)L.nsite * n2;
  long long g1t = ((long long)npos * nrhs + 511) / 512;
  if (g1t > 1024) g1t = 1024;
  const int g1f = (int)g1t;
  cx<double>* r = L.w64[1];
  if (fast) {
    hipLaunchKernelGGL(k_cgcrT_init, dim3(kCgcrG3T), dim3(256), 0, c.stream, npos, nrhs, b, L.xT, r, L.cpart3);
    WDMG_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_cgcrT_init_fin, dim3(nrhs), dim3(64), 0, c.stream, nrhs, kCgcrG3T, L.cpart3, tol, S,
                       c.dsc + S_ERR);
  } else {
    hipLaunchKernelGGL(k_cgcr_init, dim3(nrhs), dim3(1024), 0, c.stream, b, x, r, n, tol, S, c.dsc + S_ERR);
  }
  WDMG_HIP(hipGetLastError());
  // The active flags of iteration it land in pinned memory and are inspected
  // `lag` iterations later, so the stream never drains while the host waits.
  const int lag = 2;
  auto done_at = [&](int i) {
    WDMG_HIP(hipEventSynchronize(c.ring_ev[i % kRing]));
    const double* f = c.hring + (size_t)(i % kRing) * kMaxRhs;
    for (int q = 0; q < nrhs; ++q)
      if (f[q] != 0.0) return false;
    return true;
  };
  // batch: x += sum_m y_m z~_m over the J directions of the cycle just ended
  auto combine = [&](int J) {
    hipLaunchKernelGGL(k_cgcrT_backsolve, dim3(1), dim3(64), 0, c.stream, nrhs, J, k, L.chist);
    WDMG_HIP(hipGetLastError());
    const size_t nb = (npos * nrhs + 255) / 256;
    hipLaunchKernelGGL(k_cgcrT_combine, dim3((unsigned)(nb < 4096 ? nb : 4096)), dim3(256), 0, c.stream, npos, nrhs,
                       J, k, L.basisZ, L.chist, L.xT);
    WDMG_HIP(hipGetLastError());
  };
  const int fixed = c.capturing ? (c.coarse_fixed_iters < maxit ? c.coarse_fixed_iters : maxit) : 0;
  int it = 0;
  for (; it < (c.capturing ? fixed : maxit); ++it) {
    const int j = it % k;
    cx<double>* w = L.basisW + (size_t)j * bs;
    cx<double>* z = L.basisZ + (size_t)j * bs;
    const int vals = 4 * j + 4;
    if (fast) {
      {
        ProfScope ps(c, WDMG_K_COARSE_GCR, (long long)L.nsite * nrhs);
        coarse_mm(c, L, BlocksFull<double>{L.Dc64}, RhsFast{nrhs}, r, w, z, nrhs);  // also z = r
      }
      hipLaunchKernelGGL(k_cgcrT_dots, dim3(g1f), dim3(256), 0, c.stream, npos, nrhs, j, vals, L.basisW, w, r,
                         L.cpart);
      WDMG_HIP(hipGetLastError());
      hipLaunchKernelGGL(k_cgcr_coef, dim3(nrhs), dim3(1024), (size_t)(vals + 1) * sizeof(double), c.stream, j, vals,
                         g1f, L.cpart, L.cpart3, kCgcrG3T, k, S,
                         c.capturing ? nullptr : c.dring + (size_t)(it % kRing) * kMaxRhs, c.dsc + S_ERR, L.chist);
      WDMG_HIP(hipGetLastError());
      if (!c.capturing) WDMG_HIP(hipEventRecord(c.ring_ev[it % kRing], c.stream));
      hipLaunchKernelGGL(k_cgcrT_update, dim3(kCgcrG3T), dim3(256), 0, c.stream, npos, nrhs, j, k, L.basisW, w, r, S,
                         L.cpart3);
      WDMG_HIP(hipGetLastError());
      if (j == k - 1) combine(k);
      c.n_Dc[L.l] += nrhs;
      if (!c.capturing && it >= lag && done_at(it - lag)) {
        ++it;
        break;
      }
      continue;
    }
    {
      ProfScope ps(c, WDMG_K_COARSE_GCR, (long long)L.nsite * nrhs);
      hipLaunchKernelGGL(k_cgcr_apply, dim3(g1), dim3(576), (size_t)vals * sizeof(double), c.stream, L.g, n2, j, vals,
                         L.Dc64, r, L.basisW, w, z, L.cpart);
      WDMG_HIP(hipGetLastError());
    }
    double* host_act = c.capturing ? nullptr : c.dring + (size_t)(it % kRing) * kMaxRhs;
    double* err = c.dsc + S_ERR;
    // the partial |w|^2 of an iteration are read while the next one's are written
    double* p3 = L.cpart3 + (size_t)(it & 1) * kCgcrG3;
    double* p3n = L.cpart3 + (size_t)(~it & 1) * kCgcrG3;
    const dim3 grid(kCgcrG3, nrhs), block(kCgcrK3);
    if (g1 <= kCgcrFusedG1) {
      hipLaunchKernelGGL(k_cgcr_update<true>, grid, block, 0, c.stream, n, nrhs, j, k, L.basisW, L.basisZ, w, z, x, r,
                         S, p3n, vals, g1, L.cpart, p3, host_act, err);
      WDMG_HIP(hipGetLastError());
      if (!c.capturing) WDMG_HIP(hipEventRecord(c.ring_ev[it % kRing], c.stream));
    } else {
      hipLaunchKernelGGL(k_cgcr_coef, dim3(nrhs), dim3(1024), (size_t)(vals + 1) * sizeof(double), c.stream, j, vals,
                         g1, L.cpart, p3, kCgcrG3, k, S, host_act, err, nullptr);
      WDMG_HIP(hipGetLastError());
      if (!c.capturing) WDMG_HIP(hipEventRecord(c.ring_ev[it % kRing], c.stream));
      hipLaunchKernelGGL(k_cgcr_update<false>, grid, block, 0, c.stream, n, nrhs, j, k, L.basisW, L.basisZ, w, z, x, r,
                         S, p3n, vals, g1, L.cpart, p3, host_act, err);
      WDMG_HIP(hipGetLastError());
    }
    c.n_Dc[L.l] += nrhs;
    if (!c.capturing && it >= lag && done_at(it - lag)) {
      ++it;
      break;
    }
  }
  if (fast) {
    if (it > 0 && (it - 1) % k != k - 1) combine((it - 1) % k + 1);
    hipLaunchKernelGGL(k_cgcrT_out, dim3((unsigned)((npos * nrhs + 255) / 256)), dim3(256), 0, c.stream, npos, nrhs,
                       L.xT, x);
    WDMG_HIP(hipGetLastError());
  }
  if (it > c.last_coarse_iters) c.last_coarse_iters = it;
}

size_t coarsest_gcr_partials(int nrhs, int k) {
  return (size_t)nrhs * kCgcrG1 * (4 * k + 4);
}
size_t coarsest_gcr_history(int nrhs, int k) { return (size_t)nrhs * k * (2 * (size_t)k + 4); }
size_t coarsest_gcr_partials3(int nrhs) { return (size_t)nrhs * (kCgcrG3T > kCgcrG3 ? kCgcrG3T : kCgcrG3); }

template void coarse_apply<double>(Ctx&, const Level&, const cx<double>*, cx<double>*, const cx<double>*, int);
template void coarse_apply<float>(Ctx&, const Level&, const cx<float>*, cx<float>*, const cx<float>*, int);

}  // namespace wdmg

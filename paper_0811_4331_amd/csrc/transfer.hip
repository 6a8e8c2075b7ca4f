// Restriction P^dagger, prolongation P and the FP64 block orthonormalisation
// that builds P (Sec. 2: P V_c = V, P^dagger P = I through a QR of the
// aggregated candidates; Sec. 3: geometric aggregates with chirality kept
// intact, so R = P^dagger).
//
// P is stored as its Nv orthonormal block columns laid out like Nv fields of
// the finer level; the column (xhat, chi, k) is field k restricted to the
// aggregate xhat and to the dofs of chirality chi.  A coarse field is
// [rhs][xhat][chi * Nv + k].
//
// Fields of every level are [site][dof] in lexicographic site order, dof = 12
// at level 0; the two chiralities are the two halves of dof.
#include <algorithm>
#include <type_traits>

#include "half_field.h"
#include "internal.h"

namespace wdmg {
namespace {

constexpr int KC = 8;  // coarse columns reduced per block-wide sum

// Sites of aggregate `agg` of a level with geometry g and aggregate block b.
struct AggMap {
  Geom g;
  int b[4];
  int nb[4];   // aggregates per direction
  int bvol;
  __device__ __forceinline__ int site(int agg, int l) const {
    int a[4], lc[4];
    int t = agg;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      a[mu] = t % nb[mu];
      t /= nb[mu];
    }
    int u = l;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      lc[mu] = u % b[mu];
      u /= b[mu];
    }
    const int c[4] = {a[0] * b[0] + lc[0], a[1] * b[1] + lc[1], a[2] * b[2] + lc[2], a[3] * b[3] + lc[3]};
    return canon_site(g, c);
  }
  __device__ __forceinline__ int agg_of(int s) const {
    int c[4];
    canon_coords(g, s, c);
    return (c[0] / b[0]) + nb[0] * ((c[1] / b[1]) + nb[1] * ((c[2] / b[2]) + nb[2] * (c[3] / b[3])));
  }
};

AggMap make_map(const Level& f) {
  AggMap m;
  m.g = f.g;
  m.bvol = 1;
  for (int mu = 0; mu < 4; ++mu) {
    m.b[mu] = f.block[mu];
    m.nb[mu] = f.dims[mu] / f.block[mu];
    m.bvol *= f.block[mu];
  }
  return m;
}

// Row accessor: row r = l * half + d (site l of the aggregate, dof d of the
// chirality) of an (aggregate, chirality) block -> element offset.  A site's
// numbers of one chirality are consecutive rows and consecutive in memory.
struct Rows {
  AggMap map;
  int dof;
  int nrows() const { return map.bvol * (dof / 2); }
  __device__ __forceinline__ size_t off(int agg, int chi, int r) const {
    const int half = dof / 2, l = r / half, d = r - l * half;
    return (size_t)map.site(agg, l) * dof + chi * half + d;
  }
};

// Workgroup -> (aggregate, rhs) for a one-dimensional grid of nagg * nrhs
// workgroups.  The hardware sends workgroup b to XCD b % 8; the mapping gives
// every XCD a contiguous run of aggregates and runs all right-hand sides of
// an aggregate back to back there, so its P columns come from HBM once and
// are re-read from that XCD's L2.
__device__ __forceinline__ void agg_rhs_block(int nagg, int nrhs, int& agg, int& rhs) {
  const int b = blockIdx.x;
  if (nagg & 7) {
    agg = b % nagg;
    rhs = b / nagg;
    return;
  }
  const int xcd = b & 7, local = b >> 3;
  agg = xcd * (nagg >> 3) + local / nrhs;
  rhs = local % nrhs;
}

// ---- batched restriction on the matrix cores --------------------------------
// For a batch of right-hand sides P^dagger is, per (aggregate, chirality), the
// complex GEMM out[k][q] = sum_row conj(V[row][k]) f[row][q], done as four real
// products of 16 columns x 4 rows x 16 right-hand sides:
//   re += Re V . Re f + Im V . Im f,   im += Re V . Im f - Im V . Re f.
// A lane's operand of V is one complex number, so V goes straight from memory
// to registers (two rows per lane and load); it is read once per 32 rhs.  The
// fields go through LDS: their rows are columns of the product and are shared
// by the column tiles.  Workgroup = (aggregate, up to 16 QT rhs), four waves =
// (chirality, half of the chunk's rows) with all column tiles in registers;
// the two halves add up at the end.  Chunk c + 1 is on its way while the
// products of chunk c run.
//
// A is the type of products and sums: FP32 for FP32 and 16-bit operands at
// level 0 on aggregates of whole 64 sites, FP64 on all others (see
// launch_restrict_mm).
//
// Bound: the matrix cores (FP32 products, 1.0 of 1.7 M cycles at nv 24, whose
// columns fill 24 of 32) and the vector units around them.  24^3x48, nv 24,
// bf16, 32 FP32 right-hand sides in: 783 us, 950 us before the site table (a
// kernel that staged V in LDS for vector-unit products, with a conversion pass
// before it: 2019 us).
constexpr int kMmTable = 512;  // sites of an aggregate whose indices are kept in LDS
constexpr int kMmRows = 48;  // rows of a chunk (of each chirality): eight sites at level 0

template <typename R>
struct Mm;
template <>
struct Mm<float> {
  typedef float acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // row of D held by lane group g = lane / 16 in register r
  static __device__ __forceinline__ int row(int g, int r) { return 4 * g + r; }
};
template <>
struct Mm<double> {
  typedef double acc_t __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int r) { return 4 * r + g; }
};

// Prolongator columns [k][element]; two consecutive rows of a site at `off`.
template <typename R>
struct VFull {
  using T = R;
  const cx<R>* v;
  size_t stride;
  struct Raw {
    cx<R> a, b;
  };
  __device__ __forceinline__ cx<R> one(int k, size_t off) const { return v[(size_t)k * stride + off]; }
  __device__ __forceinline__ Raw pair(int k, size_t off) const {
    const cx<R>* p = v + (size_t)k * stride + off;
    return {p[0], p[1]};
  }
  static __device__ __forceinline__ cx<R> first(Raw r) { return r.a; }
  static __device__ __forceinline__ cx<R> second(Raw r) { return r.b; }
};
template <typename H>
struct VHalf {
  using T = float;
  const cxh<H>* v;
  size_t stride;
  struct Raw {
    cxh<H> a, b;
  };
  __device__ __forceinline__ Raw pair(int k, size_t off) const {
    const cxh<H>* p = v + (size_t)k * stride + off;
    return {p[0], p[1]};
  }
  static __device__ __forceinline__ cx<float> first(Raw r) { return h2f(r.a); }
  static __device__ __forceinline__ cx<float> second(Raw r) { return h2f(r.b); }
};

// Prolonged fields: as they are, or in 16 bits.
template <typename R>
struct OutFull {
  using T = R;
  static constexpr bool kHalf = false;
  cx<R>* f;
};
template <typename H>
struct OutHalf {
  using T = float;
  static constexpr bool kHalf = true;
  cxh<H>* v;
  float* s;
  __device__ __forceinline__ void store(int q, int vol, int site, const cx<float> (&x)[12]) const {
    store_site_h(v + (size_t)q * 12 * vol, s + (size_t)q * vol, site, x);
  }
};

// Fields of level 0, half a site (the six numbers of one chirality) of one
// right-hand side per item; lanes 2 i, 2 i + 1 hold the two halves of a site.
// load() issues the loads, get() gives the values.
template <typename R>
struct SiteFull {
  using T = R;
  static constexpr bool kSite = true;
  const cx<R>* f;
  int vol;
  struct Raw {
    cx<R> x[6];
  };
  __device__ __forceinline__ Raw load(int q, int site, int chi) const {
    Raw r;
    const cx<R>* p = f + ((size_t)q * vol + site) * 12 + 6 * chi;
#pragma unroll
    for (int m = 0; m < 6; ++m) r.x[m] = p[m];
    return r;
  }
  static __device__ __forceinline__ void get(const Raw& r, cx<R> (&x)[6]) {
#pragma unroll
    for (int m = 0; m < 6; ++m) x[m] = r.x[m];
  }
};
// FP32 fields taken as if stored in 16 bits (rounded with their site's scale).
template <typename H>
struct SiteRound {
  using T = float;
  static constexpr bool kSite = true;
  const cx<float>* f;
  int vol;
  using Raw = typename SiteFull<float>::Raw;
  __device__ __forceinline__ Raw load(int q, int site, int chi) const {
    return SiteFull<float>{f, vol}.load(q, site, chi);
  }
  static __device__ __forceinline__ void get(const Raw& r, cx<float> (&x)[6]) {
    float a[12];
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      a[2 * m] = r.x[m].re;
      a[2 * m + 1] = r.x[m].im;
    }
    float s = site_scale<12>(a), inv;
    s = scale_join(s, __shfl_xor(s, 1, 64));
    s = quant_scale(s, inv);
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      const cx<float> z = h2f(quantise<H>(a[2 * m], a[2 * m + 1], inv));
      x[m] = mk(s * z.re, s * z.im);
    }
  }
};
template <typename H>
struct SiteHalf {  // 16-bit fields with per-site scales
  using T = float;
  static constexpr bool kSite = true;
  const cxh<H>* v;
  const float* sc;
  int vol;
  struct Raw {
    cxh<H> x[6];
    float s;
  };
  __device__ __forceinline__ Raw load(int q, int site, int chi) const {
    Raw r;
    const cxh<H>* p = v + ((size_t)q * vol + site) * 12 + 6 * chi;
#pragma unroll
    for (int m = 0; m < 6; ++m) r.x[m] = p[m];
    r.s = sc[(size_t)q * vol + site];
    return r;
  }
  static __device__ __forceinline__ void get(const Raw& r, cx<float> (&x)[6]) {
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      const cx<float> z = h2f(r.x[m]);
      x[m] = mk(r.s * z.re, r.s * z.im);
    }
  }
};
// Fields of any level, two consecutive rows of a site per item.
template <typename R>
struct PairFull {
  using T = R;
  static constexpr bool kSite = false;
  const cx<R>* f;
  size_t n;  // elements of a field
  struct Raw {
    cx<R> a, b;
  };
  __device__ __forceinline__ Raw load(int q, size_t off) const {
    const cx<R>* p = f + (size_t)q * n + off;
    return {p[0], p[1]};
  }
};

template <class VL, class FL, typename A, int CT, int QT>
__global__ __launch_bounds__(256) void k_restrict_mm(AggMap map, int dof, VL V, FL F,
                                                     cx<typename VL::T>* __restrict__ out, int nagg, int nv,
                                                     int nrhs) {
  using R = typename VL::T;
  using acc_t = typename Mm<A>::acc_t;
  constexpr int QN = 16 * QT, LD = QN + 1;
  __shared__ __align__(16) cx<R> Fs[2][2][kMmRows][LD];
  __shared__ int table[kMmTable];
  int agg, tile;
  agg_rhs_block(nagg, gridDim.x / nagg, agg, tile);
  // a site's index takes a dozen divisions, five times per thread and chunk
  const bool tab = map.bvol <= kMmTable;
  for (int l = threadIdx.x; tab && l < map.bvol; l += 256) table[l] = map.site(agg, l);
  __syncthreads();
  auto site = [&](int l) { return tab ? table[l] : map.site(agg, l); };
  const int q0 = tile * QN, nq = min(QN, nrhs - q0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int chi = wave >> 1, kh = wave & 1;
  const int half = FL::kSite ? 6 : dof / 2, nrows = map.bvol * half;
  const int nch = (nrows + kMmRows - 1) / kMmRows;
  const int li = lane & 15, lk = lane >> 4;
  // items of the fields per chunk and thread
  constexpr int NI = FL::kSite ? QN * (kMmRows / 6) * 2 / 256 : QN * kMmRows / 256;
  typename FL::Raw fr[NI];
  typename VL::Raw vr[3][CT];
  auto load = [&](int c) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int e = i * 256 + threadIdx.x;
      if constexpr (FL::kSite) {
        const int q = e >> 4, l = c * 8 + ((e >> 1) & 7);
        if (q < nq && l < map.bvol) fr[i] = F.load(q0 + q, site(l), e & 1);
      } else {
        const int q = e / kMmRows, p = e % kMmRows, row = c * kMmRows + 2 * (p % (kMmRows / 2));
        const int l = row / half;
        if (q < nq && row < nrows)
          fr[i] = F.load(q0 + q, (size_t)site(l) * dof + (p / (kMmRows / 2)) * half + (row - l * half));
      }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int row = min(c * kMmRows + kh * 24 + t * 8 + 2 * lk, nrows - 2), l = row / half;
      const size_t off = (size_t)site(l) * dof + chi * half + (row - l * half);
#pragma unroll
      for (int j = 0; j < CT; ++j) vr[t][j] = V.pair(min(16 * j + li, nv - 1), off);
    }
  };
  auto stage = [&](int c, int b) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int e = i * 256 + threadIdx.x;
      if constexpr (FL::kSite) {
        const int q = e >> 4, s = (e >> 1) & 7;
        cx<R> x[6];
        FL::get(fr[i], x);
        const bool on = q < nq && c * 8 + s < map.bvol;
#pragma unroll
        for (int m = 0; m < 6; ++m) Fs[b][e & 1][s * 6 + m][q] = on ? x[m] : mk<R>(0, 0);
      } else {
        const int q = e / kMmRows, p = e % kMmRows, r = 2 * (p % (kMmRows / 2));
        const bool on = q < nq && c * kMmRows + r < nrows;
        Fs[b][p / (kMmRows / 2)][r][q] = on ? fr[i].a : mk<R>(0, 0);
        Fs[b][p / (kMmRows / 2)][r + 1][q] = on ? fr[i].b : mk<R>(0, 0);
      }
    }
  };
  acc_t re[CT][QT], im[CT][QT];
#pragma unroll
  for (int j = 0; j < CT; ++j)
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      re[j][t] = acc_t{0, 0, 0, 0};
      im[j][t] = acc_t{0, 0, 0, 0};
    }
  load(0);
  for (int c = 0; c < nch; ++c) {
    const int b = c & 1;
    stage(c, b);
    typename VL::Raw vc[3][CT];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int j = 0; j < CT; ++j) vc[t][j] = vr[t][j];
    __syncthreads();  // chunk c is staged; the other buffer (chunk c - 1) has been read
    if (c + 1 < nch) load(c + 1);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // rows 2 lk + h of the step: the same pairing on both operands
        cx<A> f[QT];
#pragma unroll
        for (int u = 0; u < QT; ++u) f[u] = cvt<A>(Fs[b][chi][kh * 24 + t * 8 + 2 * lk + h][16 * u + li]);
#pragma unroll
        for (int j = 0; j < CT; ++j) {
          const cx<A> v = cvt<A>(h == 0 ? VL::first(vc[t][j]) : VL::second(vc[t][j]));
#pragma unroll
          for (int u = 0; u < QT; ++u) {
            re[j][u] = Mm<A>::mma(v.re, f[u].re, re[j][u]);
            im[j][u] = Mm<A>::mma(v.re, f[u].im, im[j][u]);
            re[j][u] = Mm<A>::mma(v.im, f[u].im, re[j][u]);
            im[j][u] = Mm<A>::mma(-v.im, f[u].re, im[j][u]);
          }
        }
      }
    }
  }
  // the second half's sums join the first's
  cx<A>* part = reinterpret_cast<cx<A>*>(&Fs[0][0][0][0]);
  static_assert(sizeof(Fs) >= 2 * 64 * 4 * sizeof(cx<A>), "one tile of both chiralities");
#pragma unroll
  for (int j = 0; j < CT; ++j) {
#pragma unroll
    for (int u = 0; u < QT; ++u) {
      __syncthreads();
      if (kh == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) part[(chi * 4 + r) * 64 + lane] = mk<A>(re[j][u][r], im[j][u][r]);
      }
      __syncthreads();
      const int q = 16 * u + li;
      if (kh == 0 && q < nq) {
        cx<R>* o = out + ((size_t)(q0 + q) * nagg + agg) * 2 * nv + chi * nv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * j + Mm<A>::row(lk, r);
          const cx<A> p = part[(chi * 4 + r) * 64 + lane];
          if (k < nv) o[k] = mk<R>((R)(re[j][u][r] + p.re), (R)(im[j][u][r] + p.im));
        }
      }
    }
  }
}

// ---- prolongation on the vector units -----------------------------------------
// A launch over nb blocks of the field and ng groups of right-hand sides.  A
// block's groups run on one XCD, whose L2 they share V in (rows of eight blocks;
// without the padding 20x12x20x12, nv 20, FP16, 4 groups of one 49 us against
// 35).  Where V is longer than the Infinity Cache they run back to back (x: 8
// XCDs x groups, y: rows), so that it comes from memory once (24^3x48, nv 20,
// BF16, 8 rhs 522 us against 560), else the blocks are swept once per group
// (20^4, 133 against 142).
struct BlockMap {
  int b0;  // first block, or -1: x blocks, y groups
  __device__ __forceinline__ int block() const {
    return b0 < 0 ? (int)blockIdx.x : b0 + 8 * (int)blockIdx.y + (int)(blockIdx.x & 7);
  }
  __device__ __forceinline__ int group() const { return (int)(b0 < 0 ? blockIdx.y : blockIdx.x >> 3); }
};
template <class Launch>
void over_blocks(size_t nb, int ng, size_t vbytes, Launch launch) {
  const size_t rows = (nb + 7) / 8, most = 65535;  // rows of a grid
  if (ng == 1 || vbytes <= ((size_t)256 << 20)) {
    launch(dim3((unsigned)(8 * rows), ng), BlockMap{-1});
    return;
  }
  for (size_t r = 0; r < rows; r += most)
    launch(dim3(8 * ng, (unsigned)std::min(most, rows - r)), BlockMap{(int)(8 * r)});
}

// One thread per EP consecutive elements of a finer-level field, which belong to
// one chirality of a site, and NB right-hand sides.
constexpr int RB = 8;
template <class VL, int NB, int EP>
__global__ __launch_bounds__(256) void k_prolong(AggMap map, int dof, VL V, const cx<typename VL::T>* __restrict__ in,
                                                 cx<typename VL::T>* __restrict__ out, int nagg, int nv, int nrhs,
                                                 BlockMap bm) {
  using R = typename VL::T;
  const size_t n = (size_t)map.g.vol * dof;
  const size_t idx = ((size_t)bm.block() * 256 + threadIdx.x) * EP;
  const int r0 = bm.group() * NB, nr = min(NB, nrhs - r0);
  if (idx >= n) return;
  const int s = (int)(idx / dof), e = (int)(idx % dof);
  const int chi = e >= dof / 2;
  const cx<R>* ec = in + ((size_t)r0 * nagg + map.agg_of(s)) * 2 * nv + chi * nv;
  cx<R> acc[NB][EP];
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int m = 0; m < EP; ++m) acc[q][m] = mk<R>(0, 0);
#pragma unroll 4
  for (int k = 0; k < nv; ++k) {
    cx<R> w[EP];
#pragma unroll
    for (int m = 0; m < EP; ++m) w[m] = V.one(k, idx + m);
#pragma unroll
    for (int q = 0; q < NB; ++q)
      if (q < nr) {
        const cx<R> x = ec[(size_t)q * nagg * 2 * nv + k];
#pragma unroll
        for (int m = 0; m < EP; ++m) cmadd(acc[q][m], w[m], x);
      }
  }
#pragma unroll
  for (int q = 0; q < NB; ++q)
    if (q < nr) {
#pragma unroll
      for (int m = 0; m < EP; ++m) out[(size_t)(r0 + q) * n + idx + m] = acc[q][m];
    }
}

// The same into a 16-bit field, one thread per site.
template <typename H, int NB>
__global__ __launch_bounds__(256) void k_prolong0_h(AggMap map, VHalf<H> V, const cx<float>* __restrict__ in,
                                                    OutHalf<H> O, int nagg, int nv, int nrhs, BlockMap bm) {
  const int s = bm.block() * 256 + threadIdx.x, r0 = bm.group() * NB, vol = map.g.vol;
  if (s >= vol) return;
  const cx<float>* ec = in + ((size_t)r0 * nagg + map.agg_of(s)) * 2 * nv;
  cx<float> acc[NB][12];
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int m = 0; m < 12; ++m) acc[q][m] = mk(0.0f, 0.0f);
  constexpr int kUnroll = NB == 4 ? 1 : 2;  // columns at a time (BF16, 24^3x48, nv 20, 8 rhs: 523 us, 563 with two)
#pragma unroll kUnroll
  for (int k = 0; k < nv; ++k) {
    cx<float> w[12];
    const u4* vk = reinterpret_cast<const u4*>(V.v + (size_t)k * V.stride) + (size_t)s * 3;
#pragma unroll
    for (int m = 0; m < 3; ++m) unpack_h<H>(vk[m], m, w);
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      if (r0 + q >= nrhs) break;
      const cx<float>* e = ec + (size_t)q * nagg * 2 * nv;
      const cx<float> e0 = e[k], e1 = e[nv + k];
#pragma unroll
      for (int m = 0; m < 6; ++m) cmadd(acc[q][m], w[m], e0);
#pragma unroll
      for (int m = 6; m < 12; ++m) cmadd(acc[q][m], w[m], e1);
    }
  }
#pragma unroll
  for (int q = 0; q < NB; ++q)
    if (r0 + q < nrhs) O.store(r0 + q, vol, s, acc[q]);
}

// ---- batched prolongation on the matrix cores (level 0) -----------------------
// Per (aggregate, chirality) f[row][q] = sum_k V[row][k] c[k][q], as four real
// products of 16 rows x 4 columns x 16 right-hand sides per complex one.  The
// coarse values of the aggregate stay in registers; V goes from memory to
// registers, two consecutive rows of a column per lane (so a wave's product
// covers 32 rows, even and odd ones in two tiles) and is read once per 16 QT
// rhs.  Six waves (chirality x 32-row parts) cover a unit of 16 sites, whose
// results cross LDS to be stored as rows of sites; a 16-bit field gets its
// site's scale there.  The next unit's columns are on their way during the
// products.
//
// Bound: memory (V and the result once).
constexpr int kPmSites = 16, kPmThreads = 384, kPmLd = kPmSites * 12 + 2;

template <class VL, class OUT, int KT, int QT>
__global__ __launch_bounds__(kPmThreads) void k_prolong_mm(AggMap map, VL V, const cx<typename VL::T>* __restrict__ in,
                                                           OUT O, int nagg, int nv, int nrhs, int nsplit) {
  using R = typename VL::T;
  using acc_t = typename Mm<R>::acc_t;
  __shared__ __align__(16) cx<R> tile[16][kPmLd];  // [rhs][site x 12]
  __shared__ int table[2][kPmSites];
  int agg, qt;
  agg_rhs_block(nagg, gridDim.x / nagg, agg, qt);
  const int split = qt % nsplit;
  qt /= nsplit;
  const int q0 = qt * 16 * QT, nq = min(16 * QT, nrhs - q0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int chi = wave & 1, part = wave >> 1;
  const int li = lane & 15, lk = lane >> 4;
  const int nu = map.bvol / kPmSites, vol = map.g.vol;
  const int u0 = split * nu / nsplit, u1 = (split + 1) * nu / nsplit;  // this workgroup's units
  // coarse values: lane (q = li, column 4 t + lk)
  cx<R> c[KT][QT];
#pragma unroll
  for (int t = 0; t < KT; ++t)
#pragma unroll
    for (int u = 0; u < QT; ++u) {
      const int q = 16 * u + li, k = 4 * t + lk;
      c[t][u] = q < nq && k < nv ? in[((size_t)(q0 + q) * nagg + agg) * 2 * nv + chi * nv + k] : mk<R>(0, 0);
    }
  // this lane's row pair of a unit
  const int row = 32 * part + 2 * li, ls = row / 6, lm = row - 6 * ls;
  typename VL::Raw vr[KT];
  auto load = [&](int un) {
    const size_t off = (size_t)map.site(agg, un * kPmSites + ls) * 12 + 6 * chi + lm;
#pragma unroll
    for (int t = 0; t < KT; ++t) vr[t] = V.pair(min(4 * t + lk, nv - 1), off);
  };
  load(u0);
  for (int un = u0; un < u1; ++un) {
    acc_t re[2][QT], im[2][QT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int u = 0; u < QT; ++u) {
        re[h][u] = acc_t{0, 0, 0, 0};
        im[h][u] = acc_t{0, 0, 0, 0};
      }
    if (threadIdx.x < kPmSites) table[un & 1][threadIdx.x] = map.site(agg, un * kPmSites + threadIdx.x);
    typename VL::Raw vc[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) vc[t] = vr[t];
    if (un + 1 < u1) load(un + 1);
#pragma unroll
    for (int t = 0; t < KT; ++t) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const cx<R> v = h == 0 ? VL::first(vc[t]) : VL::second(vc[t]);
#pragma unroll
        for (int u = 0; u < QT; ++u) {
          re[h][u] = Mm<R>::mma(v.re, c[t][u].re, re[h][u]);
          im[h][u] = Mm<R>::mma(v.re, c[t][u].im, im[h][u]);
          re[h][u] = Mm<R>::mma(-v.im, c[t][u].im, re[h][u]);
          im[h][u] = Mm<R>::mma(v.im, c[t][u].re, im[h][u]);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < QT; ++u) {
      __syncthreads();  // the previous tile of 16 rhs has been stored
#pragma unroll
      for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int rr = 32 * part + 2 * Mm<R>::row(lk, r) + h;
          tile[li][(rr / 6) * 12 + 6 * chi + rr % 6] = mk<R>(re[h][u][r], im[h][u][r]);
        }
      }
      __syncthreads();
      const int* tb = table[un & 1];
      const int nqu = min(16, nq - 16 * u);
      if constexpr (OUT::kHalf) {
        for (int e = threadIdx.x; e < nqu * kPmSites; e += kPmThreads) {
          const int q = e / kPmSites, sl = e % kPmSites;
          cx<float> x[12];
#pragma unroll
          for (int m = 0; m < 12; ++m) x[m] = tile[q][sl * 12 + m];
          O.store(q0 + 16 * u + q, vol, tb[sl], x);
        }
      } else {
        constexpr int N = 16 / sizeof(cx<R>), PER = kPmSites * 12 / N;  // numbers per chunk, chunks per rhs
        for (int e = threadIdx.x; e < nqu * PER; e += kPmThreads) {
          const int q = e / PER, p = (e % PER) * N, sl = p / 12, m = p % 12;
          cx<R>* o = O.f + ((size_t)(q0 + 16 * u + q) * vol + tb[sl]) * 12 + m;
#pragma unroll
          for (int w = 0; w < N; ++w) o[w] = tile[q][p + w];
        }
      }
    }
  }
}

// ---- restriction of one right-hand side -------------------------------------
// Every element of V is used once, so V is streamed: one workgroup per
// (aggregate, rhs, column range), thread t on component t % dof of every S-th
// site (a row of sites is one run of memory), KC columns at a time in double.
// The site table of the aggregate replaces a dozen integer divisions per
// element.  The column ranges fill the chip (about 2048 workgroups); those of
// one (aggregate, rhs) run back to back on one XCD and re-read the field from
// its L2.
constexpr int kSiteTable = 1024;

template <typename R>
struct OneFull {
  const cx<R>* v;
  size_t vstride;
  const cx<R>* f;
  size_t n;  // elements of a field
  using T = R;
  __device__ __forceinline__ cx<R> column(int k, size_t off) const { return v[(size_t)k * vstride + off]; }
  __device__ __forceinline__ cx<R> field(int rhs, int, size_t off) const { return f[(size_t)rhs * n + off]; }
};
template <typename H>
struct OneHalf {
  const cxh<H>* v;
  size_t vstride;
  const cxh<H>* f;
  const float* sc;
  int vol;
  using T = float;
  __device__ __forceinline__ cx<float> column(int k, size_t off) const { return h2f(v[(size_t)k * vstride + off]); }
  __device__ __forceinline__ cx<float> field(int rhs, int site, size_t off) const {
    const cx<float> z = h2f(f[(size_t)rhs * 12 * vol + off]);
    const float s = sc[(size_t)rhs * vol + site];
    return mk(s * z.re, s * z.im);
  }
};

template <class D, int KC>
__global__ __launch_bounds__(256) void k_restrict_one(AggMap map, int dof, int S, D io, cx<typename D::T>* __restrict__ out,
                                                      int nagg, int nv, int nsplit, int kper) {
  using R = typename D::T;
  __shared__ int table[kSiteTable];
  __shared__ double red[2 * KC][256];
  int agg, item;
  agg_rhs_block(nagg, gridDim.x / nagg, agg, item);
  const int rhs = item / nsplit, split = item % nsplit;
  const int kbeg = split * kper, kend = min(nv, kbeg + kper);
  out += ((size_t)rhs * nagg + agg) * 2 * nv;
  const int half = dof / 2;
  const int e = threadIdx.x % dof, l0 = threadIdx.x / dof;
  for (int k0 = kbeg; k0 < kend; k0 += KC) {
    double v[2 * KC];
#pragma unroll
    for (int q = 0; q < 2 * KC; ++q) v[q] = 0.0;
    for (int c0 = 0; c0 < map.bvol; c0 += kSiteTable) {
      const int nc = min(kSiteTable, map.bvol - c0);
      if (k0 == kbeg || map.bvol > kSiteTable) {
        __syncthreads();
        for (int l = threadIdx.x; l < nc; l += blockDim.x) table[l] = map.site(agg, c0 + l);
        __syncthreads();
      }
#pragma unroll 2
      for (int l = l0; l < nc; l += S) {
        const int site = table[l];
        const size_t o = (size_t)site * dof + e;
        const cx<R> f = io.field(rhs, site, o);
        cx<R> w[KC];
#pragma unroll
        for (int q = 0; q < KC; ++q) w[q] = io.column(min(k0 + q, kend - 1), o);
#pragma unroll
        for (int q = 0; q < KC; ++q) {
          v[2 * q] += (double)w[q].re * f.re + (double)w[q].im * f.im;
          v[2 * q + 1] += (double)w[q].re * f.im - (double)w[q].im * f.re;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 2 * KC; ++q) red[q][threadIdx.x] = v[q];
    __syncthreads();
    // value u = 2 KC chi + q summed over the S x half threads of its chirality:
    // 16 threads each, then across them
    constexpr int G = 16;
    for (int u = threadIdx.x / G; u < 4 * KC; u += blockDim.x / G) {
      const int chi = u / (2 * KC), q = u % (2 * KC);
      double t = 0.0;
      for (int i = threadIdx.x % G; i < S * half; i += G) t += red[q][(i / half) * dof + chi * half + i % half];
#pragma unroll
      for (int m = G / 2; m > 0; m >>= 1) t += __shfl_xor(t, m, 64);
      if (threadIdx.x % G == 0 && k0 + (q >> 1) < kend)
        reinterpret_cast<R*>(out + chi * nv + k0 + (q >> 1))[q & 1] = (R)t;
    }
    __syncthreads();
  }
}

// ---- block orthonormalisation (FP64): block Gram-Schmidt, two passes --------
// One workgroup per (aggregate, chirality); column j is orthogonalised against
// columns 0..j-1 twice, QB of them at a time, then normalised by its (real,
// positive) norm, which makes diag(R) real positive and Q unique.  A thread
// keeps its NR rows' offsets and the current column's values in registers and
// reads the QB earlier columns once per pass (they feed the dot products and,
// still in registers, the update).
constexpr int QB = 4;
template <int NR>
__global__ __launch_bounds__(256) void k_block_qr(Rows rows, int nrows, cx<double>* Vv, size_t vstride, int nv,
                                                  double* dsc) {
  __shared__ double lds[2 * QB * 4];
  __shared__ double coef[2 * QB];
  const int agg = blockIdx.x, chi = blockIdx.y;
  size_t off[NR];
  bool on[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int r = threadIdx.x + i * blockDim.x;
    on[i] = r < nrows;
    off[i] = rows.off(agg, chi, on[i] ? r : 0);
  }
  auto norm2 = [&](const cx<double> (&a)[NR]) {
    double v[1] = {0.0};
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (on[i]) v[0] += a[i].re * a[i].re + a[i].im * a[i].im;
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) coef[0] = v[0];
    __syncthreads();
    const double t = coef[0];
    __syncthreads();
    return t;
  };
  for (int j = 0; j < nv; ++j) {
    cx<double>* vj = Vv + (size_t)j * vstride;
    cx<double> a[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) a[i] = on[i] ? vj[off[i]] : mk(0.0, 0.0);
    const double norm0 = norm2(a);
    for (int pass = 0; pass < 2; ++pass) {
      for (int i0 = 0; i0 < j; i0 += QB) {
        cx<double> b[QB][NR];
        double v[2 * QB];
#pragma unroll
        for (int q = 0; q < QB; ++q) {
          v[2 * q] = v[2 * q + 1] = 0.0;
          const cx<double>* vi = Vv + (size_t)(i0 + q) * vstride;
#pragma unroll
          for (int i = 0; i < NR; ++i) b[q][i] = i0 + q < j && on[i] ? vi[off[i]] : mk(0.0, 0.0);
        }
#pragma unroll
        for (int q = 0; q < QB; ++q)
#pragma unroll
          for (int i = 0; i < NR; ++i) {
            v[2 * q] += b[q][i].re * a[i].re + b[q][i].im * a[i].im;
            v[2 * q + 1] += b[q][i].re * a[i].im - b[q][i].im * a[i].re;
          }
        block_sum<2 * QB>(v, lds);
        if (threadIdx.x == 0) {
#pragma unroll
          for (int q = 0; q < 2 * QB; ++q) coef[q] = v[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < QB; ++q) {
          const cx<double> h = mk(coef[2 * q], coef[2 * q + 1]);
#pragma unroll
          for (int i = 0; i < NR; ++i) a[i] = a[i] - h * b[q][i];
        }
        __syncthreads();
      }
    }
    const double n1 = norm2(a), nr = sqrt(n1);
    if (threadIdx.x == 0 && !(nr > 1e-12 * sqrt(norm0))) dsc[S_ERR + 1] = 1.0;  // rank lost (or NaN)
    const double inv = nr > 0.0 ? 1.0 / nr : 0.0;
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (on[i]) vj[off[i]] = mk(a[i].re * inv, a[i].im * inv);
  }
}

// The same for blocks of more rows than the registers of a workgroup hold,
// column values re-read from memory.
__global__ __launch_bounds__(256) void k_block_qr_long(Rows rows, int nrows, cx<double>* Vv, size_t vstride, int nv,
                                                       double* dsc) {
  __shared__ double lds[2 * KC * 4];
  __shared__ double coef[2 * 64];
  __shared__ double scal;
  const int agg = blockIdx.x, chi = blockIdx.y;
  for (int j = 0; j < nv; ++j) {
    cx<double>* vj = Vv + (size_t)j * vstride;
    double n0[1] = {0.0};
    for (int r = threadIdx.x; r < nrows; r += blockDim.x) {
      const cx<double> a = vj[rows.off(agg, chi, r)];
      n0[0] += a.re * a.re + a.im * a.im;
    }
    block_sum<1>(n0, lds);
    if (threadIdx.x == 0) scal = sqrt(n0[0]);
    __syncthreads();
    const double norm0 = scal;
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
      for (int i0 = 0; i0 < j; i0 += KC) {
        double v[2 * KC];
#pragma unroll
        for (int q = 0; q < 2 * KC; ++q) v[q] = 0.0;
        for (int r = threadIdx.x; r < nrows; r += blockDim.x) {
          const size_t o = rows.off(agg, chi, r);
          const cx<double> a = vj[o];
#pragma unroll
          for (int q = 0; q < KC; ++q) {
            if (i0 + q < j) {
              const cx<double> b = Vv[(size_t)(i0 + q) * vstride + o];
              v[2 * q] += b.re * a.re + b.im * a.im;
              v[2 * q + 1] += b.re * a.im - b.im * a.re;
            }
          }
        }
        block_sum<2 * KC>(v, lds);
        if (threadIdx.x == 0) {
          for (int q = 0; q < 2 * KC; ++q) coef[2 * i0 + q] = v[q];
        }
        __syncthreads();
      }
      for (int r = threadIdx.x; r < nrows; r += blockDim.x) {
        const size_t o = rows.off(agg, chi, r);
        cx<double> a = vj[o];
        for (int i = 0; i < j; ++i) a = a - mk(coef[2 * i], coef[2 * i + 1]) * Vv[(size_t)i * vstride + o];
        vj[o] = a;
      }
      __syncthreads();
    }
    double n1[1] = {0.0};
    for (int r = threadIdx.x; r < nrows; r += blockDim.x) {
      const cx<double> a = vj[rows.off(agg, chi, r)];
      n1[0] += a.re * a.re + a.im * a.im;
    }
    block_sum<1>(n1, lds);
    if (threadIdx.x == 0) {
      const double nr = sqrt(n1[0]);
      if (!(nr > 1e-12 * norm0)) dsc[S_ERR + 1] = 1.0;  // rank lost (or NaN)
      scal = nr > 0.0 ? 1.0 / nr : 0.0;
    }
    __syncthreads();
    const double inv = scal;
    for (int r = threadIdx.x; r < nrows; r += blockDim.x) {
      const size_t o = rows.off(agg, chi, r);
      const cx<double> a = vj[o];
      vj[o] = mk(a.re * inv, a.im * inv);
    }
    __syncthreads();
  }
}

inline int nagg_of(const Level& f) {
  int n = 1;
  for (int mu = 0; mu < 4; ++mu) n *= f.dims[mu] / f.block[mu];
  return n;
}

inline int tpb_for(int nrows) {
  int t = ((nrows + 63) / 64) * 64;
  return t > 256 ? 256 : t;
}

// Column ranges per (aggregate, rhs) of k_restrict_one: enough workgroups to
// fill the chip (about 2048), ranges of at least one column.
struct RestrictSplit {
  int nsplit, kper;
};
inline RestrictSplit restrict_split(int nagg, int nrhs, int nv) {
  const long long have = (long long)nagg * nrhs;
  int want = (int)((2048 + have - 1) / have);
  if (want > nv) want = nv;
  if (want < 1) want = 1;
  const int kper = (nv + want - 1) / want;
  return {(nv + kper - 1) / kper, kper};
}

template <class D>
void launch_restrict_one(Ctx& c, const Level& f, const D& io, cx<typename D::T>* out, int nrhs) {
  const int nagg = nagg_of(f);
  const RestrictSplit sp = restrict_split(nagg, nrhs, f.nv);
  // S sites per sweep, a power of two; whole groups of 16 threads for the sums
  int S = 1;
  while (2 * S * f.dof <= 256) S *= 2;
  const dim3 grid(nagg * nrhs * sp.nsplit), block(S * f.dof % 16 ? (S * f.dof + 15) / 16 * 16 : S * f.dof);
  if (sp.kper <= 4)
    hipLaunchKernelGGL((k_restrict_one<D, 4>), grid, block, 0, c.stream, make_map(f), f.dof, S, io, out, nagg, f.nv,
                       sp.nsplit, sp.kper);
  else
    hipLaunchKernelGGL((k_restrict_one<D, 8>), grid, block, 0, c.stream, make_map(f), f.dof, S, io, out, nagg, f.nv,
                       sp.nsplit, sp.kper);
  WDMG_HIP(hipGetLastError());
}

}  // namespace

// The matrix-core restriction where it applies: two rows of a site in a pair,
// at most 32 columns (two column tiles of registers).  One right-hand side
// would fill one of a tile's 16 columns: it streams V instead.
inline bool mm_fits(const Level& f) { return f.dof % 4 == 0 && f.nv <= 32; }

template <typename A, class VL, class FL>
void launch_restrict_sums(Ctx& c, const Level& f, const VL& V, const FL& F, cx<typename VL::T>* out, int nrhs) {
  const AggMap map = make_map(f);
  const int nagg = nagg_of(f);
  const dim3 block(256);
#define RM(CT, QT)                                                                                                  \
  hipLaunchKernelGGL((k_restrict_mm<VL, FL, A, CT, QT>), grid, block, 0, c.stream, map, f.dof, V, F, out, nagg, f.nv, \
                     nrhs)
  if (nrhs <= 16) {
    const dim3 grid(nagg);
    if (f.nv <= 16)
      RM(1, 1);
    else
      RM(2, 1);
  } else {
    const dim3 grid(nagg * ((nrhs + 31) / 32));
    if (f.nv <= 16)
      RM(1, 2);
    else
      RM(2, 2);
  }
#undef RM
  WDMG_HIP(hipGetLastError());
}

// Sums of FP32 and 16-bit operands: in FP32 at level 0 on aggregates of whole
// 64 sites (the 4^4 ones of every production hierarchy: 24^3x48, nv 24, bf16,
// 32 rhs 783 us), in FP64 on smaller or odd aggregates and on the coarse
// levels, as a single right-hand side sums everywhere.  FP64 products run at
// half the FP32 rate: 2592 sites of 48 numbers, nv 16, 16 rhs 20 us (17 with
// FP32 sums, 160 with FP64 sums on the vector units); 24^4, 3^4 aggregates, nv
// 20, FP32, 32 rhs 692 us (430, 11500).
template <class VL, class FL>
void launch_restrict_mm(Ctx& c, const Level& f, const VL& V, const FL& F, cx<typename VL::T>* out, int nrhs) {
  if (sizeof(typename VL::T) == 4 && f.l == 0 && make_map(f).bvol % 64 == 0)
    launch_restrict_sums<typename VL::T>(c, f, V, F, out, nrhs);
  else
    launch_restrict_sums<double>(c, f, V, F, out, nrhs);
}

template <typename R>
void restrict_any(Ctx& c, const Level& f, const cx<R>* V, const cx<R>* in, cx<R>* out, int nrhs) {
  if (nrhs >= 2 && mm_fits(f)) {
    if (f.dof == 12)
      launch_restrict_mm(c, f, VFull<R>{V, f.n}, SiteFull<R>{in, f.nsite}, out, nrhs);
    else
      launch_restrict_mm(c, f, VFull<R>{V, f.n}, PairFull<R>{in, f.n}, out, nrhs);
    return;
  }
  launch_restrict_one(c, f, OneFull<R>{V, f.n, in, f.n}, out, nrhs);
}

template <typename R>
void restrict0(Ctx& c, const Level& f, const cx<R>* V, const cx<R>* in, cx<R>* out, int nrhs) {
  ProfScope ps(c, sizeof(R) == 8 ? WDMG_K_RESTRICT_F64 : WDMG_K_RESTRICT_F32, (long long)f.nsite * nrhs);
  restrict_any<R>(c, f, V, in, out, nrhs);
}

template <typename R>
void restrictC(Ctx& c, const Level& f, const cx<R>* V, const cx<R>* in, cx<R>* out, int nrhs) {
  restrict_any<R>(c, f, V, in, out, nrhs);
}

// The matrix-core prolongation where it applies: level 0, aggregates of whole
// units, at most 32 columns, and a batch that fills enough of a tile's 16
// columns: from 6 right-hand sides in FP64, 3 in FP32 (vector units / matrix
// cores, us, 24^3x48, nv 20: FP64 4 rhs 789 / 965, 6 rhs 1089 / 1005, 16 rhs
// 2752 / 1233; FP32 2 rhs 411 / 380, 16 rhs 2151 / 506; 16^4: FP32 2 rhs 36 / 42,
// 3 rhs 46 / 43).
enum { kPmMinF64 = 6, kPmMinF32 = 3 };
// In 16 bits by blocks of 256 sites: up to half a block per compute unit from 17,
// under two from 13, else from 12 in BF16 and 10 in FP16 (BF16 12x16x8x16: 14 rhs
// 42 / 49; 16^4: 12 rhs 72 / 83, 13 rhs 88 / 85; 20^4: 14 rhs 228 / 220; 24^3x48:
// BF16 11 rhs 664 / 688, 12 rhs 744 / 713, FP16 9 rhs 635 / 655, 10 rhs 693 / 680).
template <typename H>
int pm_min_half(const Ctx& c, const Level& f) {
  const int nblk = (f.nsite + 255) / 256;
  if (nblk <= c.ncu / 2) return 17;
  if (nblk < 2 * c.ncu) return 13;
  return std::is_same<H, bf16_t>::value ? 12 : 10;
}
inline bool pm_fits(const Level& f, int nrhs, int least) {
  return nrhs >= least && f.dof == 12 && make_map(f).bvol % kPmSites == 0 && f.nv <= 32;
}

template <class VL, class OUT>
void launch_prolong_mm(Ctx& c, const Level& f, const VL& V, const cx<typename VL::T>* in, const OUT& O, int nrhs) {
  const AggMap map = make_map(f);
  const int nagg = nagg_of(f);
  // 32 rhs per workgroup read V half as often; FP64 has registers for 16
  constexpr int Q2 = sizeof(typename VL::T) == 4 ? 2 : 1;
  const int qt = nrhs <= 16 ? 1 : Q2;
  const int ntile = (nrhs + 16 * qt - 1) / (16 * qt);
  // an aggregate's units go over several workgroups where the aggregates do not
  // fill the chip (32 aggregates, nv 20, FP32, 16 rhs: 45 us unsplit, 11 us in
  // 16; 256 of them: 50 us unsplit, 58 us in 4)
  const int nu = map.bvol / kPmSites, want = (c.ncu + nagg * ntile - 1) / (nagg * ntile);
  const int nsplit = want < nu ? want : nu;
  const dim3 block(kPmThreads), grid(nagg * ntile * nsplit);
#define PM(KT)                                                                                                 \
  do {                                                                                                         \
    if (qt == 1)                                                                                               \
      hipLaunchKernelGGL((k_prolong_mm<VL, OUT, KT, 1>), grid, block, 0, c.stream, map, V, in, O, nagg, f.nv,  \
                         nrhs, nsplit);                                                                        \
    else                                                                                                       \
      hipLaunchKernelGGL((k_prolong_mm<VL, OUT, KT, Q2>), grid, block, 0, c.stream, map, V, in, O, nagg, f.nv, \
                         nrhs, nsplit);                                                                        \
  } while (0)
  if (f.nv <= 16)
    PM(4);
  else if (f.nv <= 24)
    PM(6);
  else
    PM(8);
#undef PM
  WDMG_HIP(hipGetLastError());
}

template <typename R>
void launch_prolong(Ctx& c, const Level& f, const cx<R>* V, const cx<R>* in, cx<R>* out, int nrhs) {
  if (pm_fits(f, nrhs, sizeof(R) == 8 ? kPmMinF64 : kPmMinF32)) {
    launch_prolong_mm(c, f, VFull<R>{V, f.n}, in, OutFull<R>{out}, nrhs);
    return;
  }
  const size_t vbytes = (size_t)f.nv * f.n * sizeof(cx<R>);
#define PV(NB, EP)                                                                                             \
  over_blocks((f.n / (EP) + 255) / 256, (nrhs + (NB) - 1) / (NB), vbytes, [&](dim3 grid, BlockMap bm) {        \
    hipLaunchKernelGGL((k_prolong<VFull<R>, NB, EP>), grid, dim3(256), 0, c.stream, make_map(f), f.dof,        \
                       VFull<R>{V, f.n}, in, out, nagg_of(f), f.nv, nrhs, bm);                                 \
  })
  if (nrhs > 1)
    PV(RB, 1);
  else if (sizeof(R) == 4 && f.dof % 4 == 0)
    PV(1, 2);
  else
    PV(1, 1);
#undef PV
  WDMG_HIP(hipGetLastError());
}

template <typename R>
void prolong0(Ctx& c, const Level& f, const cx<R>* V, const cx<R>* in, cx<R>* out, int nrhs) {
  ProfScope ps(c, sizeof(R) == 8 ? WDMG_K_PROLONG_F64 : WDMG_K_PROLONG_F32, (long long)f.nsite * nrhs);
  launch_prolong<R>(c, f, V, in, out, nrhs);
}

template <typename R>
void prolongC(Ctx& c, const Level& f, const cx<R>* V, const cx<R>* in, cx<R>* out, int nrhs) {
  launch_prolong<R>(c, f, V, in, out, nrhs);
}

template <typename H>
bool restrict0_round(Ctx& c, const Level& f, const void* V16, const cx<float>* in, cx<float>* out, int nrhs) {
  if (nrhs < 2 || !mm_fits(f)) return false;
  ProfScope ps(c, WDMG_K_RESTRICT_H, (long long)f.nsite * nrhs);
  launch_restrict_mm(c, f, VHalf<H>{static_cast<const cxh<H>*>(V16), f.n}, SiteRound<H>{in, f.nsite}, out, nrhs);
  return true;
}

template <typename H>
void restrict0_h(Ctx& c, const Level& f, const void* V16, HF in, cx<float>* out, int nrhs) {
  if (nrhs >= 2 && mm_fits(f)) {
    ProfScope ps(c, WDMG_K_RESTRICT_H, (long long)f.nsite * nrhs);
    launch_restrict_mm(c, f, VHalf<H>{static_cast<const cxh<H>*>(V16), f.n},
                       SiteHalf<H>{static_cast<const cxh<H>*>(in.v), in.s, f.nsite}, out, nrhs);
    return;
  }
  ProfScope ps(c, WDMG_K_RESTRICT_H, (long long)f.nsite * nrhs);
  launch_restrict_one(c, f, OneHalf<H>{static_cast<const cxh<H>*>(V16), f.n, static_cast<const cxh<H>*>(in.v), in.s,
                                       f.nsite}, out, nrhs);
}

template <typename H>
void prolong0_h(Ctx& c, const Level& f, const void* V16, const cx<float>* in, HF out, int nrhs) {
  ProfScope ps(c, WDMG_K_PROLONG_H, (long long)f.nsite * nrhs);
  const VHalf<H> V{static_cast<const cxh<H>*>(V16), f.n};
  const OutHalf<H> O{static_cast<cxh<H>*>(out.v), out.s};
  if (pm_fits(f, nrhs, pm_min_half<H>(c, f))) {
    launch_prolong_mm(c, f, V, in, O, nrhs);
    return;
  }
  // Right-hand sides per thread, which share its part of V: one where that fills
  // the chip no more than four workgroups a compute unit (8x8x8x16, 8 rhs: 15 us
  // against 18 with two, 24 with four), two in FP16 and for the next larger
  // lattices (20x12x20x12, 8 rhs: 50 us, 57 with one, 54 with four; FP16 20^4, 4
  // rhs: 69, 73, 86), else four (BF16 24^3x48, 8 rhs: 522, 572 with two).
  const int nblk = (f.nsite + 255) / 256;
#define PH(NB)                                                                                                  \
  over_blocks(nblk, (nrhs + (NB) - 1) / (NB), (size_t)f.nv * f.n * 4, [&](dim3 grid, BlockMap bm) {             \
    hipLaunchKernelGGL((k_prolong0_h<H, NB>), grid, dim3(256), 0, c.stream, make_map(f), V, in, O, nagg_of(f),  \
                       f.nv, nrhs, bm);                                                                         \
  })
  if ((long long)nblk * nrhs <= 4 * c.ncu)
    PH(1);
  else if (std::is_same<H, f16_t>::value || (long long)nblk * ((nrhs + 3) / 4) <= 2 * c.ncu)
    PH(2);
  else
    PH(4);
#undef PH
  WDMG_HIP(hipGetLastError());
}

template bool restrict0_round<f16_t>(Ctx&, const Level&, const void*, const cx<float>*, cx<float>*, int);
template bool restrict0_round<bf16_t>(Ctx&, const Level&, const void*, const cx<float>*, cx<float>*, int);
template void restrict0_h<f16_t>(Ctx&, const Level&, const void*, HF, cx<float>*, int);
template void restrict0_h<bf16_t>(Ctx&, const Level&, const void*, HF, cx<float>*, int);
template void prolong0_h<f16_t>(Ctx&, const Level&, const void*, const cx<float>*, HF, int);
template void prolong0_h<bf16_t>(Ctx&, const Level&, const void*, const cx<float>*, HF, int);

void launch_qr(Ctx& c, const Level& f, cx<double>* V) {
  Rows rows{make_map(f), f.dof};
  const int nrows = rows.nrows();
  const dim3 grid(nagg_of(f), 2), block(tpb_for(nrows));
  const int nr = (nrows + block.x - 1) / block.x;
#define QR(N) hipLaunchKernelGGL((k_block_qr<N>), grid, block, 0, c.stream, rows, nrows, V, f.n, f.nv, c.dsc)
  if (nr <= 1)
    QR(1);
  else if (nr <= 2)
    QR(2);
  else if (nr <= 4)
    QR(4);
  else if (nr <= 6)
    QR(6);
  else
    hipLaunchKernelGGL(k_block_qr_long, grid, block, 0, c.stream, rows, nrows, V, f.n, f.nv, c.dsc);
#undef QR
  WDMG_HIP(hipGetLastError());
}

void block_qr0(Ctx& c, const Level& f, cx<double>* V) {
  ProfScope ps(c, WDMG_K_BLOCK_QR, (long long)nagg_of(f) * 2);
  launch_qr(c, f, V);
}

void block_qrC(Ctx& c, const Level& f, cx<double>* V) { launch_qr(c, f, V); }

#define INST(R)                                                                                 \
  template void restrict0<R>(Ctx&, const Level&, const cx<R>*, const cx<R>*, cx<R>*, int);     \
  template void restrictC<R>(Ctx&, const Level&, const cx<R>*, const cx<R>*, cx<R>*, int);     \
  template void prolong0<R>(Ctx&, const Level&, const cx<R>*, const cx<R>*, cx<R>*, int);      \
  template void prolongC<R>(Ctx&, const Level&, const cx<R>*, const cx<R>*, cx<R>*, int);
INST(double)
INST(float)
#undef INST

}  // namespace wdmg

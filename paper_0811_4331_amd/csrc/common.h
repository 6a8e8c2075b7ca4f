// Device-side building blocks shared by every kernel of libwdmg (gfx950).
//
// * cx<R>: complex number, 8- or 16-byte aligned so a wavefront's loads of
//   consecutive elements coalesce into full 64-lane transactions.
// * Geom: lattice geometry of one multigrid level.  Fields are stored in
//   lexicographic site order (canon_site).  The links of the fine level are
//   stored tile-major: the lattice is cut into (Bx,By,Bz,Bt) tiles (the 4^4
//   aggregates of the multigrid, Sec. 3), tiles are numbered
//   lexicographically and sites inside a tile lexicographically.  Coarse
//   levels use B = 1 (both orders are the same).
// * wave / block reductions with a fixed summation order (deterministic).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace wdmg {

template <typename R>
struct __align__(2 * sizeof(R)) cx {
  R re, im;
};

template <typename R>
__host__ __device__ __forceinline__ cx<R> mk(R a, R b) {
  cx<R> z;
  z.re = a;
  z.im = b;
  return z;
}
template <typename R>
__host__ __device__ __forceinline__ cx<R> operator+(cx<R> a, cx<R> b) { return mk(a.re + b.re, a.im + b.im); }
template <typename R>
__host__ __device__ __forceinline__ cx<R> operator-(cx<R> a, cx<R> b) { return mk(a.re - b.re, a.im - b.im); }
template <typename R>
__host__ __device__ __forceinline__ cx<R> operator*(cx<R> a, cx<R> b) {
  return mk(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re);
}
template <typename R>
__host__ __device__ __forceinline__ cx<R> operator*(R s, cx<R> a) { return mk(s * a.re, s * a.im); }
// conj(a) * b
template <typename R>
__host__ __device__ __forceinline__ cx<R> cmulc(cx<R> a, cx<R> b) {
  return mk(a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re);
}
// acc += a * b
template <typename R>
__host__ __device__ __forceinline__ void cmadd(cx<R>& acc, cx<R> a, cx<R> b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
}
// acc += conj(a) * b
template <typename R>
__host__ __device__ __forceinline__ void cmaddc(cx<R>& acc, cx<R> a, cx<R> b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(-a.im, b.re, acc.im);
}
// i * a and -i * a
template <typename R>
__host__ __device__ __forceinline__ cx<R> ti(cx<R> a) { return mk(-a.im, a.re); }
template <typename R>
__host__ __device__ __forceinline__ cx<R> tmi(cx<R> a) { return mk(a.im, -a.re); }

template <typename Rout, typename Rin>
__host__ __device__ __forceinline__ cx<Rout> cvt(cx<Rin> a) {
  return mk((Rout)a.re, (Rout)a.im);
}

// ---------------------------------------------------------------------------
// Geometry.
struct Geom {
  int L[4];    // extents x, y, z, t
  int B[4];    // tile extents (1, 2 or 4)
  int lb[4];   // log2 B
  int nT[4];   // tiles per direction
  int sl[4];   // stride of a local coordinate inside a tile
  int st[4];   // stride (in sites) of a tile coordinate
  int vol;     // sites
  int vpad;    // sites rounded up to a multiple of 64 (link blocks)
  int tvol;    // sites per tile
  int ltvol;   // log2 tvol
};

__host__ __device__ __forceinline__ int site_of(const Geom& g, int x, int y, int z, int t) {
  const int c[4] = {x, y, z, t};
  int tile = 0, loc = 0;
#pragma unroll
  for (int mu = 3; mu >= 0; --mu) {
    const int tc = c[mu] >> g.lb[mu];
    const int lc = c[mu] & (g.B[mu] - 1);
    tile = tile * g.nT[mu] + tc;
    loc += lc * g.sl[mu];
  }
  return (tile << g.ltvol) + loc;
}

__host__ __device__ __forceinline__ void coords_of(const Geom& g, int s, int c[4]) {
  int tile = s >> g.ltvol;
  const int loc = s & (g.tvol - 1);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    const int tc = tile % g.nT[mu];
    tile /= g.nT[mu];
    const int lc = (loc >> (g.lb[0] * (mu > 0) + g.lb[1] * (mu > 1) + g.lb[2] * (mu > 2))) & (g.B[mu] - 1);
    c[mu] = (tc << g.lb[mu]) + lc;
  }
}

// Canonical (lexicographic, x fastest) index of coordinates c, and back: the
// site order of every field.  The tile-major order above numbers the links.
__host__ __device__ __forceinline__ int canon_site(const Geom& g, const int (&c)[4]) {
  return c[0] + g.L[0] * (c[1] + g.L[1] * (c[2] + g.L[2] * c[3]));
}
__host__ __device__ __forceinline__ void canon_coords(const Geom& g, int i, int (&c)[4]) {
#pragma unroll
  for (int mu = 0; mu < 3; ++mu) {
    c[mu] = i % g.L[mu];
    i /= g.L[mu];
  }
  c[3] = i;
}

// Neighbour of site s (with coordinates c) one step forward / backward in mu,
// periodic.  No division: local step inside the tile, else tile step.
__host__ __device__ __forceinline__ int nbr_fwd(const Geom& g, int s, const int c[4], int mu) {
  const int lc = c[mu] & (g.B[mu] - 1);
  if (lc < g.B[mu] - 1) return s + g.sl[mu];
  s -= (g.B[mu] - 1) * g.sl[mu];
  const int tc = c[mu] >> g.lb[mu];
  return (tc < g.nT[mu] - 1) ? s + g.st[mu] : s - (g.nT[mu] - 1) * g.st[mu];
}

__host__ __device__ __forceinline__ int nbr_bwd(const Geom& g, int s, const int c[4], int mu) {
  const int lc = c[mu] & (g.B[mu] - 1);
  if (lc > 0) return s - g.sl[mu];
  s += (g.B[mu] - 1) * g.sl[mu];
  const int tc = c[mu] >> g.lb[mu];
  return (tc > 0) ? s - g.st[mu] : s + (g.nT[mu] - 1) * g.st[mu];
}

// ---------------------------------------------------------------------------
// Reductions (wave64).
// v of the lane that DPP control CTRL names (0 where there is none, or outside
// the rows of ROWS).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, ROWS, 0xf, true);
  const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, ROWS, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
// Sum over groups of N = 8, 16 or 32 lanes, in the last lane of each; all 64
// lanes take part.
template <int N>
__device__ __forceinline__ double group_sum(double v) {
  static_assert(N == 8 || N == 16 || N == 32, "a DPP row, its half or two rows");
  v += dpp<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8
  v += dpp<0x112, 0xf>(v);
  v += dpp<0x114, 0xf>(v);
  if constexpr (N >= 16) v += dpp<0x118, 0xf>(v);
  if constexpr (N == 32) v += dpp<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
  return v;
}
// Sum over the wave, in every lane; all 64 lanes take part.  Row shifts and
// broadcasts on the vector unit: the same sum by lane permutes goes through
// the LDS pipe twelve times (Wilson operator with the sums of an MR step, 16^4,
// FP32, 8 rhs: 47.8 against 53.4 us).
__device__ __forceinline__ double wave_sum(double v) {
  v = group_sum<32>(v);
  v += dpp<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3: lane 63 holds the sum
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, 63);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), 63);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Sums K values over the block; the result is valid in thread 0.  `lds` must
// hold K * (blockDim.x / 64) doubles.
template <int K>
__device__ __forceinline__ void block_sum(double (&v)[K], double* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) lds[wave * K + k] = v[k];
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = wave_sum(lane < nw ? lds[lane * K + k] : 0.0);
  }
  __syncthreads();
}

}  // namespace wdmg

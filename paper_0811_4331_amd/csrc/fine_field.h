// Fine-lattice field layout and link storage.
//
// Fields are stored as the caller hands them in: sites in lexicographic order
// (x fastest), a site's 12 numbers (spin, colour) in one run, right-hand sides
// one after another.  Element (site i, component k) sits at 12 i + k.
//
// Links are SU(3) (Sec. 3: unitary connections).  Only their first two rows
// are stored (6 complex per link, 24 per site); the third row is rebuilt as
// the complex conjugate of the cross product of the first two.  The
// antiperiodic time sign is folded into the stored rows of U_t at t = Lt-1,
// so the rebuilt row takes the same sign explicitly.  Sites are numbered
// tile-major (see Geom) and stored in blocks of 64 -- one wavefront -- with
// the components of a block contiguous: element (site s, component k) of
// ncomp sits at ((s / 64) * ncomp + k) * 64 + s % 64, so that a wavefront's
// load of one component is one contiguous run.  The site count is padded to a
// multiple of 64 (Geom::vpad); padding sites hold zeros.
#pragma once

#include "common.h"

namespace wdmg {

constexpr int kLinkComp = 24;  // stored complex numbers per site (4 links x 2 rows)

// 16 bytes: the unit in which sites are moved
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
template <typename R>
union ChunkOf {
  static constexpr int N = 16 / (2 * sizeof(R));  // complex numbers in it
  u4 q;
  R v[2 * N];
};
// chunk c of a site's numbers
template <typename R>
__device__ __forceinline__ u4 chunk_of(const cx<R> (&a)[12], int c) {
  constexpr int N = ChunkOf<R>::N;
  ChunkOf<R> q;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    q.v[2 * e] = a[c * N + e].re;
    q.v[2 * e + 1] = a[c * N + e].im;
  }
  return q.q;
}

// Element of the blocked link storage.
__host__ __device__ __forceinline__ size_t fidx(int s, int k, int ncomp) {
  return ((size_t)(s >> 6) * ncomp + k) * 64 + (s & 63);
}

// Third row of an SU(3) link from its first two: conj(row0 x row1), with
// the folded boundary sign when neg.
template <typename R>
__device__ __forceinline__ void recon_third_row(cx<R> (&u)[9], bool neg) {
  const cx<R> c0 = u[1] * u[5] - u[2] * u[4];
  const cx<R> c1 = u[2] * u[3] - u[0] * u[5];
  const cx<R> c2 = u[0] * u[4] - u[1] * u[3];
  const R sg = neg ? (R)-1 : (R)1;
  u[6] = mk<R>(sg * c0.re, -sg * c0.im);
  u[7] = mk<R>(sg * c1.re, -sg * c1.im);
  u[8] = mk<R>(sg * c2.re, -sg * c2.im);
}

template <typename R>
__device__ __forceinline__ void load_link(const cx<R>* __restrict__ U, int mu, int s, bool neg, cx<R> (&u)[9]) {
  const cx<R>* base = U + fidx(s, mu * 6, kLinkComp);
#pragma unroll
  for (int e = 0; e < 6; ++e) u[e] = base[e * 64];
  recon_third_row(u, neg);
}

}  // namespace wdmg

// Wilson-Dirac operator on gfx950 (Sec. 1):
//   (D psi)(x) = (4 + m) psi(x)
//              - 1/2 sum_mu [ (1 - gamma_mu) U_mu(x) psi(x+mu) + (1 + gamma_mu) U_mu(x-mu)^+ psi(x-mu) ]
// in the chiral basis (gamma5 = diag(1,1,-1,-1)).  Each hop projects the
// neighbour spinor onto the two-dimensional image of (1 -+ gamma_mu), applies
// the SU(3) link to the two colour vectors of that half spinor, and expands
// back to four spins.  The antiperiodic time sign is folded into the stored
// links U_t(x) at t = Lt-1, so it reaches both hop directions.
//
// Layout: fields in site order (a site's 12 numbers in one run), links as
// their first two rows in tile-major blocks of 64 sites (see fine_field.h).
// A thread that loaded its own neighbour would touch one memory line per lane
// and load, so both kernels fetch spinors in 16-byte chunks with consecutive
// lanes on consecutive chunks and hand every thread its site through LDS:
//   k_wilson_gather  any lattice, every precision; one wave per direction
//   k_wilson_tile    4^4 tiles, FP32 arithmetic; a tile and its faces in LDS,
//                    links in registers over a batch of right-hand sides
#include "half_field.h"
#include "internal.h"
#include "wilson_spin.h"

namespace wdmg {
namespace {

// ---- fields ---------------------------------------------------------------
// Full<R>: FP64 or FP32 fields and links.  Half<H>: 16-bit fields with a scale
// per site and 16-bit links, arithmetic in FP32.
template <typename R>
struct Full {
  using T = R;
  static constexpr bool kDots = true;
  static constexpr bool kHalf = false;
  static constexpr int NC = 12 * 2 * sizeof(R) / 16;  // stored chunks per site
  const u4* in;
  u4* out;
  const cx<R>* U;
  __device__ __forceinline__ void link(int mu, int s, bool neg, cx<R> (&u)[9]) const { load_link(U, mu, s, neg, u); }
  __device__ __forceinline__ void rows(int mu, int s, cx<R> (&u)[6]) const {
    const cx<R>* base = U + fidx(s, mu * 6, kLinkComp);
#pragma unroll
    for (int e = 0; e < 6; ++e) u[e] = base[e * 64];
  }
};

template <typename H>
struct Half {
  using T = float;
  static constexpr bool kDots = true;
  static constexpr bool kHalf = true;
  static constexpr int NC = 3;
  const u4* in;
  const float* isc;
  u4* out;
  float* osc;
  const cxh<H>* U;
  __device__ __forceinline__ void link(int mu, int s, bool neg, cx<float> (&u)[9]) const {
    load_link_h(U, mu, s, neg, u);
  }
  __device__ __forceinline__ void raw(int mu, int s, unsigned (&u)[6]) const {
    const unsigned* base = reinterpret_cast<const unsigned*>(U) + fidx(s, mu * 6, kLinkComp);
#pragma unroll
    for (int e = 0; e < 6; ++e) u[e] = base[e * 64];
  }
  static __device__ __forceinline__ void whole(const unsigned (&l)[6], bool neg, cx<float> (&u)[9]) {
#pragma unroll
    for (int e = 0; e < 6; ++e) u[e] = h2f(__builtin_bit_cast(cxh<H>, l[e]));
    recon_third_row(u, neg);
  }
};

// The numbers of stored chunk c of a site (16 bits: unscaled).
template <typename R>
__device__ __forceinline__ void unpack_chunk(const Full<R>*, u4 q, int c, cx<R> (&p)[12]) {
  ChunkOf<R> x;
  x.q = q;
#pragma unroll
  for (int e = 0; e < ChunkOf<R>::N; ++e) p[c * ChunkOf<R>::N + e] = mk<R>(x.v[2 * e], x.v[2 * e + 1]);
}
template <typename H>
__device__ __forceinline__ void unpack_chunk(const Half<H>*, u4 q, int c, cx<float> (&p)[12]) {
  unpack_h<H>(q, c, p);
}
template <class S>
__device__ __forceinline__ void unpack(u4 q, int c, cx<typename S::T> (&p)[12]) {
  unpack_chunk(static_cast<const S*>(nullptr), q, c, p);
}

// n complex numbers in 16 bits at v (4-byte aligned), unscaled; and stored.
template <typename H, int N>
__device__ __forceinline__ void load_numbers(const Half<H>*, const unsigned* v, float (&p)[N]) {
#pragma unroll
  for (int k = 0; k < N / 2; ++k) {
    const cx<float> z = h2f(__builtin_bit_cast(cxh<H>, v[k]));
    p[2 * k] = z.re;
    p[2 * k + 1] = z.im;
  }
}
// Half's result as FP32 numbers, each what 16-bit storage would have held: for
// callers with FP32 fields (24^3x48, BF16, 1 rhs: 98 us with a pass that reads
// the stored result back, 72 us so).
template <typename H>
struct HalfOut32 : Half<H> {
  static constexpr bool kDots = false;
  cx<float>* f32;
};

// N / 2 numbers of a site from the first on, in 16 bits with the site's scale
// so = 1 / inv, which the site's first thread stores.
template <typename H, int N>
__device__ __forceinline__ void store_numbers(const Half<H>& io, int r, int vol, int site, int first,
                                              const float (&a)[N], float so, float inv) {
  if (first == 0) io.osc[(size_t)r * vol + site] = so;
  unsigned* v = reinterpret_cast<unsigned*>(io.out) + ((size_t)r * vol + site) * 12 + first;
#pragma unroll
  for (int k = 0; k < N / 2; ++k)
    v[k] = __builtin_bit_cast(unsigned, quantise<H>(a[2 * k], a[2 * k + 1], inv));
}
template <typename H, int N>
__device__ __forceinline__ void store_numbers(const HalfOut32<H>& io, int r, int vol, int site, int first,
                                              const float (&a)[N], float so, float inv) {
  cx<float>* v = io.f32 + ((size_t)r * vol + site) * 12 + first;
#pragma unroll
  for (int k = 0; k < N / 2; ++k) {
    const cx<float> z = h2f(quantise<H>(a[2 * k], a[2 * k + 1], inv));
    v[k] = mk(so * z.re, so * z.im);
  }
}

// U h (SIGN > 0) or U^+ h of the two colour vectors of a half spinor.
template <int SIGN, typename R>
__device__ __forceinline__ void link_half(const cx<R> (&u)[9], const cx<R> (&h)[6], cx<R> (&uh)[6]) {
#pragma unroll
  for (int a = 0; a < 2; ++a) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      cx<R> t = mk<R>(0, 0);
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (SIGN > 0)
          cmadd(t, u[i * 3 + b], h[a * 3 + b]);
        else
          cmaddc(t, u[b * 3 + i], h[a * 3 + b]);
      }
      uh[a * 3 + i] = t;
    }
  }
}

template <int MU, int SIGN, typename R>
__device__ __forceinline__ void hop_add(const cx<R> (&u)[9], const cx<R> (&p)[12], cx<R> (&acc)[12]) {
  cx<R> h[6], uh[6];
  project<MU, SIGN>(p, h);
  link_half<SIGN>(u, h, uh);
  expand_add<MU, SIGN>(uh, acc);
}

template <int MU, int SIGN>
__device__ __forceinline__ void hop_add_scaled(const cx<float> (&u)[9], const cx<float> (&p)[12], float sc,
                                               cx<float> (&acc)[12]) {
  cx<float> h[6], uh[6];
  project<MU, SIGN>(p, h);
  link_half<SIGN>(u, h, uh);
  expand_add_scaled<MU, SIGN>(uh, sc, acc);
}

typedef __attribute__((address_space(1))) const void glb_t;
typedef __attribute__((address_space(3))) void lds_t;

// 16 bytes per lane straight into LDS at dst + 16 lane (dst uniform over the wave).
__device__ __forceinline__ void load_to_lds(const void* src, void* dst) {
  __builtin_amdgcn_global_load_lds((glb_t*)src, (lds_t*)dst, 16, 0, 0);
}
// vmcnt(0): this wave's loads have landed (LDS ones included)
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt(0x0f70);
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// lgkmcnt(0): this wave's LDS reads have returned
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_wave_barrier();
}

// Sums of three values over a wave, in its lanes 60, 61 and 62.  The first two
// exchanges also hand the values out to the lanes, so the rest is done for one
// value a lane instead of three.
__device__ __forceinline__ double wave_sums3(const double (&d)[3]) {
  const int lane = threadIdx.x & 63;
  const bool b0 = lane & 1, b1 = lane & 2;
  const double x = (b0 ? d[1] : d[0]) + dpp<0xb1, 0xf>(b0 ? d[0] : d[1]);  // quad_perm 1 0 3 2
  const double z = d[2] + dpp<0xb1, 0xf>(d[2]);
  double y = (b1 ? z : x) + dpp<0x4e, 0xf>(b1 ? x : z);  // quad_perm 2 3 0 1
  y += dpp<0x114, 0xf>(y);                               // row_shr 4, 8
  y += dpp<0x118, 0xf>(y);
  y += __shfl_xor(y, 16, 64);
  return y + __shfl_xor(y, 32, 64);
}

// MR step-size sums of one thread (Sec. 3 smoother): Re and Im of <out, in>
// and |out|^2 over n numbers of the operator's result and input.
template <typename R>
__device__ __forceinline__ void mr_dots(const R* o, const R* i, int n, double (&d)[3]) {
#pragma unroll
  for (int k = 0; k < n; k += 2) {
    const double ore = o[k], oim = o[k + 1], ire = i[k], iim = i[k + 1];
    d[0] += ore * ire + oim * iim;
    d[1] += ore * iim - oim * ire;
    d[2] += ore * ore + oim * oim;
  }
}

// ---- any lattice: one wave per direction ------------------------------------
// A workgroup of four waves covers one block of 64 sites of the link layout;
// wave mu takes the two hops along mu.  Lane l of load i fetches position
// (64 i + l) of the wave's buffer of 64 rows, whose site index comes from the
// lane that owns the row; rows of 6 (12) chunks would put rows four (two)
// apart on the same banks, so a row's chunks are exchanged by swz (rows of 3
// chunks spread by themselves).  The backward neighbours are on their way
// while the forward hop is worked on.  The four directions meet in the same
// buffers, where all 256 threads sum and store.
//
// A workgroup takes a group of right-hand sides.  FP32 and 16 bits keep the
// links and offsets of the wave in registers over the group; FP64 keeps the two
// stored rows of the links (166 registers, three waves per SIMD) and finds the
// rest anew.  ONE: a single right-hand side.  In 16 bits its rows are half as
// long as the sums that follow them in the buffer: both neighbours' rows are
// fetched at once, and with the links' rows held as stored the kernel has 76
// registers instead of 125.  In FP64 the backward link is loaded with the
// backward rows, so that less is waited for before the first hop.
//
// Bound: instructions (one wave takes 700 to 900 vector instructions for 64
// sites and a direction), in FP64 also the L2.  Measured, kernel alone:
//   FP64  24^3x48 32 rhs 3770 us (4480 with one rhs per workgroup), 8 rhs 933
//         (1102), 1 rhs 156; 32^4 8 rhs 1442 (1665); each inside a solve
//   BF16  24^3x48 1 rhs 55 us (66 as a group of one), 32^4 86 us (102)
// and with the layout conversions that it makes unnecessary in brackets: 32^4
// FP64 1 rhs 222 us (398), 12x20x10x18 FP32 5 rhs 22 us (53), 32^4 FP32 1 rhs
// 120 us (210).
template <typename R>
__device__ __forceinline__ int swz(int j) {
  return sizeof(R) == 4 ? (j >> 2) & 1 : (j >> 1) & 3;
}
template <class S>
__device__ __forceinline__ int row_pos(int j, int c) {  // position of stored chunk c of row j
  return j * S::NC + (S::kHalf ? c : (c ^ swz<typename S::T>(j)));
}

template <class S>
__device__ __forceinline__ void gather_offsets(int nb, int lane, unsigned (&off)[S::NC]) {
#pragma unroll
  for (int i = 0; i < S::NC; ++i) {
    const int e = i * 64 + lane, j = e / S::NC, c = e % S::NC;
    off[i] = (unsigned)(__shfl(nb, j, 64) * S::NC + (S::kHalf ? c : (c ^ swz<typename S::T>(j))));
  }
}

template <class S>
__device__ __forceinline__ void fetch_sites(const u4* f, const unsigned (&off)[S::NC], u4* buf) {
#pragma unroll
  for (int i = 0; i < S::NC; ++i) load_to_lds(f + off[i], buf + i * 64);
}

template <class S>
__device__ __forceinline__ void read_row(const u4* buf, int lane, cx<typename S::T> (&p)[12]) {
#pragma unroll
  for (int c = 0; c < S::NC; ++c) unpack<S>(buf[row_pos<S>(lane, c)], c, p);
}

template <int MU, int SIGN>
__device__ __forceinline__ void read_half_f64(const u4* buf, int lane, cx<double> (&h)[6]) {
  // one colour at a time, so that four numbers of the row, not twelve, are held
  const cx<double>* row = reinterpret_cast<const cx<double>*>(buf) + lane * 12;
  const int sw = swz<double>(lane);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    cx<double> p[12];
#pragma unroll
    for (int k = 0; k < 4; ++k) p[3 * k + c] = row[(3 * k + c) ^ sw];
    project_colour<MU, SIGN>(p, c, h);
  }
}

// acc as the row of this lane in working precision (rows of Full<R>)
template <typename R>
__device__ __forceinline__ void write_row(u4* buf, int lane, const cx<R> (&acc)[12]) {
#pragma unroll
  for (int c = 0; c < Full<R>::NC; ++c) buf[row_pos<Full<R>>(lane, c)] = chunk_of<R>(acc, c);
}

template <int MU>
__device__ __forceinline__ int stride_of(const Geom& g) {
  return MU == 0 ? 1 : (MU == 1 ? g.L[0] : (MU == 2 ? g.L[0] * g.L[1] : g.L[0] * g.L[1] * g.L[2]));
}
template <int MU>
__device__ __forceinline__ int canon_fwd(const Geom& g, const int (&c)[4], int me) {
  return c[MU] == g.L[MU] - 1 ? me - (g.L[MU] - 1) * stride_of<MU>(g) : me + stride_of<MU>(g);
}
template <int MU>
__device__ __forceinline__ int canon_bwd(const Geom& g, const int (&c)[4], int me) {
  return c[MU] == 0 ? me + (g.L[MU] - 1) * stride_of<MU>(g) : me - stride_of<MU>(g);
}

template <int MU, class S, bool ONE, class Finish>
__device__ __forceinline__ void gather_wave(const Geom& g, const S& io, int tneg, int s, const int (&c)[4], int me,
                                            int r0, int r1, u4* buf, Finish finish) {
  using R = typename S::T;
  const int lane = threadIdx.x & 63;
  const size_t fs = (size_t)g.vol * S::NC;
  const bool last = MU == 3 && tneg && c[3] == g.L[3] - 1, first = MU == 3 && tneg && c[3] == 0;
  const int nf = canon_fwd<MU>(g, c, me), nb = canon_bwd<MU>(g, c, me);
  if constexpr (sizeof(R) == 8 && ONE) {
    const u4* f = io.in + r0 * fs;
    cx<R> h[6], uh[6], u[9], acc[12];
    {
      unsigned off[S::NC];
      gather_offsets<S>(nf, lane, off);
      fetch_sites<S>(f, off, buf);
    }
    io.link(MU, s, last, u);
    wait_loads();
    read_half_f64<MU, +1>(buf, lane, h);
    wait_lds();
    __builtin_amdgcn_sched_barrier(0);
    {
      unsigned off[S::NC];
      gather_offsets<S>(nb, lane, off);
      fetch_sites<S>(f, off, buf);
    }
    link_half<+1>(u, h, uh);
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = mk<R>(0, 0);
    expand_add<MU, +1>(uh, acc);
    __builtin_amdgcn_sched_barrier(0);
    io.link(MU, nbr_bwd(g, s, c, MU), first, u);
    wait_loads();
    read_half_f64<MU, -1>(buf, lane, h);
    link_half<-1>(u, h, uh);
    expand_add<MU, -1>(uh, acc);
    write_row<R>(buf, lane, acc);
    finish(r0);
  } else if constexpr (sizeof(R) == 8) {
    cx<R> lf[6], lb[6];
    io.rows(MU, s, lf);
    io.rows(MU, nbr_bwd(g, s, c, MU), lb);
    auto whole = [](const cx<R> (&l)[6], bool neg, cx<R> (&u)[9]) {
#pragma unroll
      for (int k = 0; k < 6; ++k) u[k] = l[k];
      recon_third_row(u, neg);
    };
    for (int r = r0; r < r1; ++r) {
      const u4* f = io.in + r * fs;
      cx<R> h[6], uh[6], u[9], acc[12];
      // nothing derived from these is kept from one right-hand side to the next:
      // there are no registers for it
      int nfr = nf, nbk = nb, lane = threadIdx.x & 63;
      asm volatile("" : "+v"(nfr), "+v"(nbk), "+v"(lane));
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        asm volatile("" : "+v"(lf[k].re), "+v"(lf[k].im));
        asm volatile("" : "+v"(lb[k].re), "+v"(lb[k].im));
      }
      {
        unsigned off[S::NC];
        gather_offsets<S>(nfr, lane, off);
        fetch_sites<S>(f, off, buf);
      }
      wait_loads();
      read_half_f64<MU, +1>(buf, lane, h);
      wait_lds();
      __builtin_amdgcn_sched_barrier(0);
      {
        unsigned off[S::NC];
        gather_offsets<S>(nbk, lane, off);
        fetch_sites<S>(f, off, buf);
      }
      whole(lf, last, u);
      link_half<+1>(u, h, uh);
#pragma unroll
      for (int k = 0; k < 12; ++k) acc[k] = mk<R>(0, 0);
      expand_add<MU, +1>(uh, acc);
      __builtin_amdgcn_sched_barrier(0);
      whole(lb, first, u);
      wait_loads();
      read_half_f64<MU, -1>(buf, lane, h);
      link_half<-1>(u, h, uh);
      expand_add<MU, -1>(uh, acc);
      write_row<R>(buf, lane, acc);
      finish(r);
    }
  } else if constexpr (ONE) {
    const u4* f = io.in + r0 * fs;
    {
      unsigned of[S::NC], ob[S::NC];
      gather_offsets<S>(nf, lane, of);
      gather_offsets<S>(nb, lane, ob);
      fetch_sites<S>(f, of, buf);
      fetch_sites<S>(f, ob, buf + 64 * S::NC);
    }
    unsigned lf[6], lb[6];
    io.raw(MU, s, lf);
    io.raw(MU, nbr_bwd(g, s, c, MU), lb);
    const float sf = io.isc[(size_t)r0 * g.vol + nf], sb = io.isc[(size_t)r0 * g.vol + nb];
    cx<R> p[12], acc[12], u[9];
    wait_loads();
    read_row<S>(buf, lane, p);
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = mk<R>(0, 0);
    io.whole(lf, last, u);
    hop_add_scaled<MU, +1>(u, p, sf, acc);
    __builtin_amdgcn_sched_barrier(0);
    read_row<S>(buf + 64 * S::NC, lane, p);
    io.whole(lb, first, u);
    hop_add_scaled<MU, -1>(u, p, sb, acc);
    wait_lds();
    write_row<R>(buf, lane, acc);
    finish(r0);
  } else {
    unsigned of[S::NC], ob[S::NC];
    gather_offsets<S>(nf, lane, of);
    gather_offsets<S>(nb, lane, ob);
    fetch_sites<S>(io.in + r0 * fs, of, buf);
    cx<R> uf[9], ub[9];
    io.link(MU, s, last, uf);
    io.link(MU, nbr_bwd(g, s, c, MU), first, ub);
    for (int r = r0; r < r1; ++r) {
      const u4* f = io.in + r * fs;
      if (r > r0) fetch_sites<S>(f, of, buf);
      float sf = 1.0f, sb = 1.0f;
      if constexpr (S::kHalf) {
        sf = io.isc[(size_t)r * g.vol + nf];
        sb = io.isc[(size_t)r * g.vol + nb];
      }
      cx<R> p[12], acc[12];
      wait_loads();
      read_row<S>(buf, lane, p);
      wait_lds();
      __builtin_amdgcn_sched_barrier(0);
      fetch_sites<S>(f, ob, buf);
#pragma unroll
      for (int k = 0; k < 12; ++k) acc[k] = mk<R>(0, 0);
      if constexpr (S::kHalf)
        hop_add_scaled<MU, +1>(uf, p, sf, acc);
      else
        hop_add<MU, +1>(uf, p, acc);
      __builtin_amdgcn_sched_barrier(0);
      wait_loads();
      read_row<S>(buf, lane, p);
      if constexpr (S::kHalf) {
        hop_add_scaled<MU, -1>(ub, p, sb, acc);
        wait_lds();  // the row of sums is longer than the stored row it replaces
      } else {
        hop_add<MU, -1>(ub, p, acc);
      }
      write_row<R>(buf, lane, acc);
      finish(r);
    }
  }
}

template <class S, bool DOTS, bool ONE, typename R = typename S::T>
__global__ __launch_bounds__(256) void k_wilson_gather(Geom g, S io, R diag, int tneg, int nsb, int nrhs, int nper,
                                                       int g5, double* dots) {
  constexpr int NW = Full<R>::NC, N = ChunkOf<R>::N;  // chunks of a working-precision row, numbers in one
  __shared__ u4 buf[4][64 * NW];
  __shared__ double red[2][4][3];
  // blocks of one rhs group in XCD-contiguous order (workgroup b runs on XCD
  // b % 8), the groups of a block back to back (a sweep of the blocks per group:
  // FP64 24^3x48 32 rhs 3560 us against 3640, but FP32 12x20x10x18 32 rhs 105
  // against 96)
  const int ngrp = (nrhs + nper - 1) / nper;
  int sb, grp;
  {
    const int b = blockIdx.x;
    if (nsb & 7) {
      sb = b / ngrp;
      grp = b % ngrp;
    } else {
      const int local = b >> 3;
      sb = (b & 7) * (nsb >> 3) + local / ngrp;
      grp = local % ngrp;
    }
  }
  const int r0 = grp * nper, r1 = min(nrhs, r0 + nper);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int s = sb * 64 + lane < g.vol ? sb * 64 + lane : 0;
  int c[4];
  coords_of(g, s, c);
  const int me = canon_site(g, c);
  const size_t fs = (size_t)g.vol * S::NC;
  auto flush = [&](int r) {  // the four waves' sums of right-hand side r, written before the last barrier
    if (threadIdx.x < 3) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < 4; ++w) t += red[r & 1][w][threadIdx.x];
      dots[((size_t)r * nsb + sb) * 3 + threadIdx.x] = t;
    }
  };
  // the four directions of right-hand side r summed and stored
  auto finish = [&](int r) {
    __syncthreads();
    const u4* f = io.in + r * fs;
    double d[3] = {0.0, 0.0, 0.0};
    if constexpr (!S::kHalf) {
#pragma unroll
      for (int i = 0; i < (NW + 3) / 4; ++i) {
        int tid = threadIdx.x;
        if constexpr (sizeof(R) == 8 && !ONE) asm volatile("" : "+v"(tid));  // as in gather_wave
        const int e = i * 256 + tid, j = e / NW;
        const int site = __shfl(me, j & 63, 64);
        if (e < 64 * NW && sb * 64 + j < g.vol) {
          const size_t o = (size_t)site * NW + ((e % NW) ^ swz<R>(j));
          ChunkOf<R> a, p;
          p.q = f[o];
          a.q = buf[0][e];
#pragma unroll
          for (int w = 1; w < 4; ++w) {
            ChunkOf<R> b;
            b.q = buf[w][e];
#pragma unroll
            for (int k = 0; k < 2 * N; ++k) a.v[k] += b.v[k];
          }
#pragma unroll
          for (int k = 0; k < 2 * N; ++k) a.v[k] = diag * p.v[k] - (R)0.5 * a.v[k];
          if constexpr (sizeof(R) == 8) {  // a chunk is one number: components 6..11 take gamma5's sign
            if (g5 && ((e % NW) ^ swz<R>(j)) >= 6) {
              a.v[0] = -a.v[0];
              a.v[1] = -a.v[1];
            }
          }
          io.out[r * fs + o] = a.q;
          if constexpr (DOTS) mr_dots(a.v, p.v, 2 * N, d);
        }
      }
    } else {
      // four threads per site, three numbers each; the scale needs all twelve
      const int j = threadIdx.x >> 2, q = threadIdx.x & 3;
      const int site = __shfl(me, j, 64);
      const bool live = sb * 64 + j < g.vol;
      float a[6], p[6];
      float sc = 0.0f;
      if (live) {
        sc = io.isc[(size_t)r * g.vol + site];
        load_numbers(&io, reinterpret_cast<const unsigned*>(f) + ((size_t)site * 12 + 3 * q), p);
      }
      const float dg = diag * sc;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int n = 3 * q + k, pos = 2 * row_pos<Full<float>>(j, n >> 1) + (n & 1);
        float re = 0.0f, im = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const cx<float> b = reinterpret_cast<const cx<float>*>(buf[w])[pos];
          re += b.re;
          im += b.im;
        }
        a[2 * k] = live ? dg * p[2 * k] - 0.5f * re : 0.0f;
        a[2 * k + 1] = live ? dg * p[2 * k + 1] - 0.5f * im : 0.0f;
      }
      float m = site_scale<6>(a);
      m = scale_join(m, __shfl_xor(m, 1, 64));
      m = scale_join(m, __shfl_xor(m, 2, 64));
      if (live) {
        float inv;
        const float so = quant_scale(m, inv);
        store_numbers(io, r, g.vol, site, 3 * q, a, so, inv);
        if constexpr (DOTS) {
          mr_dots(a, p, 6, d);
          d[0] *= (double)sc;
          d[1] *= (double)sc;
        }
      }
    }
    if constexpr (DOTS) {
      const double t = wave_sums3(d);
      if (lane >= 60 && lane < 63) red[r & 1][wave][lane - 60] = t;
    }
    if (DOTS || r + 1 < r1) __syncthreads();
    if constexpr (DOTS) flush(r);
  };
  switch (wave) {
    case 0: gather_wave<0, S, ONE>(g, io, tneg, s, c, me, r0, r1, buf[0], finish); break;
    case 1: gather_wave<1, S, ONE>(g, io, tneg, s, c, me, r0, r1, buf[1], finish); break;
    case 2: gather_wave<2, S, ONE>(g, io, tneg, s, c, me, r0, r1, buf[2], finish); break;
    default: gather_wave<3, S, ONE>(g, io, tneg, s, c, me, r0, r1, buf[3], finish); break;
  }
}

// ---- 4^4 tiles, FP32 arithmetic: persistent workgroups over (tile, rhs) ------
// A tile's 256 spinors and the 8 x 64 of its faces are staged in LDS per
// right-hand side, as FP32 rows in `slots`: own sites first, then the faces
// (x+, x-, y+, ...).  Three site reads per site instead of nine, the faces in
// runs of four sites (384 bytes in FP32).  512 threads: thread (half, site)
// takes the two directions 2 half, 2 half + 1 of its site with their four
// links in registers for every right-hand side of the tile; the two halves'
// sums meet in the face slots once those have been read.  Two LDS buffers: the
// next right-hand side's chunks are loaded while the current one is worked on
// (147 KB, one workgroup per compute unit, no spilled registers).
//
// The grid is one workgroup per compute unit, and each walks its tiles
// (TileWork): the work per unit is equal to one right-hand side, and the
// prologue of a tile (links, offsets) overlaps the previous tile's last
// right-hand side.  Neighbouring workgroups of an XCD are in step: L2 misses are
// at most 1.07 of the algorithmic bytes, where one read of every spinor is 0.53
// (an upper bound: hits in the Infinity Cache count, and so does the counter's
// factor for a copy's long requests).  24^3x48, 32 rhs, FP32: 1300 us against
// 2018 us for the best earlier kernel (3717 us with its layout conversions); one
// workgroup per tile and 8 right-hand sides: 1493 us.
// Bound: two waves per SIMD, which hide neither all of the loads (3.3 TB/s of the
// 4.7 TB/s a copy reaches; with the hops taken out 4% faster) nor all of the
// instructions (vector units 53% busy in FP32, 61% in BF16).
constexpr int kTileSlots = 256 + 8 * 64;
constexpr int kTileChunks = kTileSlots * 6;
constexpr int kTileThreads = 512;
constexpr size_t kTileLds = 2 * (size_t)kTileChunks * 16;

__device__ __forceinline__ int tile_nbr(int l, int mu, int dir) {
  const int c = (l >> (2 * mu)) & 3;
  const int lo = l & ((1 << (2 * mu)) - 1), hi = l >> (2 * mu + 2);
  const int j = lo | (hi << (2 * mu));  // the other three coordinates
  if (dir > 0) return c < 3 ? l + (1 << (2 * mu)) : 256 + (2 * mu) * 64 + j;
  return c > 0 ? l - (1 << (2 * mu)) : 256 + (2 * mu + 1) * 64 + j;
}

__device__ __forceinline__ void slot_read(const u4* sm, int slot, cx<float> (&p)[12]) {
#pragma unroll
  for (int c = 0; c < 6; ++c) unpack<Full<float>>(sm[row_pos<Full<float>>(slot, c)], c, p);
}

// The four hops of a thread: directions 2 H and 2 H + 1.
template <int H>
__device__ __forceinline__ void tile_hops(const u4* sm, const cx<float> (&u)[4][9], const int (&nbs)[4],
                                          cx<float> (&acc)[12]) {
  cx<float> p[12];
  slot_read(sm, nbs[0], p);
  hop_add<2 * H, +1>(u[0], p, acc);
  slot_read(sm, nbs[1], p);
  hop_add<2 * H, -1>(u[1], p, acc);
  slot_read(sm, nbs[2], p);
  hop_add<2 * H + 1, +1>(u[2], p, acc);
  slot_read(sm, nbs[3], p);
  hop_add<2 * H + 1, -1>(u[3], p, acc);
}

__device__ __forceinline__ void tile_base(const Geom& g, int tile, int (&base)[4]) {
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    base[mu] = (tile % g.nT[mu]) * 4;
    tile /= g.nT[mu];
  }
}

// Canonical site of a slot of the tile at `base`.
__device__ __forceinline__ int tile_site(const Geom& g, const int (&base)[4], int slot) {
  int x[4];
  if (slot < 256) {
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) x[mu] = base[mu] + ((slot >> (2 * mu)) & 3);
  } else {
    const int face = (slot - 256) >> 6, mu0 = face >> 1;
    int j = slot & 63;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      if (mu == mu0) {
        const int v = (face & 1) ? base[mu] - 1 : base[mu] + 4;
        x[mu] = v < 0 ? g.L[mu] - 1 : (v >= g.L[mu] ? 0 : v);
      } else {
        x[mu] = base[mu] + (j & 3);
        j >>= 2;
      }
    }
  }
  return canon_site(g, x);
}

// Work of a persistent workgroup: whole tiles in rounds (all right-hand sides
// of a tile, the workgroups of one XCD on neighbouring tiles), then an equal
// share of the (tile, rhs) pairs of the last, partly filled round.
struct TileWork {
  int t0, nwg, full, nrhs;  // first tile of the XCD, its workgroups, whole rounds
  int a, b;                 // pairs of the last round
  int round, j;
  __device__ __forceinline__ bool next(int& tile, int& r0, int& r1) {
    if (round < full) {
      tile = t0 + round * nwg + j;
      ++round;
      r0 = 0;
      r1 = nrhs;
      return true;
    }
    if (a >= b) return false;
    tile = t0 + full * nwg + a / nrhs;
    r0 = a % nrhs;
    r1 = min(nrhs, r0 + b - a);
    a += r1 - r0;
    return true;
  }
};

template <class S, bool DOTS>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_wilson_tile(
    Geom g, S io, float diag, int tneg, int ntile, int nrhs, int nxcd, double* dots) {
  extern __shared__ __align__(16) u4 smem[];  // 2 x kTileChunks
  __shared__ double red[2][8][3];
  constexpr int NL = (kTileSlots * S::NC + kTileThreads - 1) / kTileThreads;  // loads per thread (9, 5)
  constexpr int kBytes = S::NC * 16;
  TileWork w;
  {
    const int x = blockIdx.x % nxcd, per = ntile / nxcd;
    w.nwg = gridDim.x / nxcd;
    w.j = blockIdx.x / nxcd;
    w.t0 = x * per;
    w.full = per / w.nwg;
    w.nrhs = nrhs;
    w.round = 0;
    const long long rest = (long long)(per - w.full * w.nwg) * nrhs;
    w.a = (int)(rest * w.j / w.nwg);
    w.b = (int)(rest * (w.j + 1) / w.nwg);
  }
  int tile, r, r1;
  if (!w.next(tile, r, r1)) return;
  const int tid = threadIdx.x, l = tid & 255, half = tid >> 8, lane = tid & 63, wave = tid >> 6;
  const size_t fs = (size_t)g.vol * kBytes;  // bytes of a field
  const char* fin = reinterpret_cast<const char*>(io.in);
  char* fout = reinterpret_cast<char*>(io.out);
  cx<float> u[4][9];
  int nbs[4];
#pragma unroll
  for (int m2 = 0; m2 < 2; ++m2) {
    nbs[2 * m2] = tile_nbr(l, 2 * half + m2, +1);
    nbs[2 * m2 + 1] = tile_nbr(l, 2 * half + m2, -1);
  }
  auto links = [&](int t) {
    int base[4], c[4];
    tile_base(g, t, base);
    const int s = t * 256 + l;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) c[mu] = base[mu] + ((l >> (2 * mu)) & 3);
#pragma unroll
    for (int m2 = 0; m2 < 2; ++m2) {
      const int mu = 2 * half + m2;
      const bool last = tneg && mu == 3 && c[3] == g.L[3] - 1, first = tneg && mu == 3 && c[3] == 0;
      io.link(mu, s, last, u[2 * m2]);
      io.link(mu, nbr_bwd(g, s, c, mu), first, u[2 * m2 + 1]);
    }
  };
  // byte offsets in a field of the chunks this thread stages (FP32: the first
  // three are the tile's own), 16 bits: also the site it finishes half of
  unsigned off[NL];
  int own = 0;
  auto offsets = [&](int t) {
    int base[4];
    tile_base(g, t, base);
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int p = min(k * kTileThreads + tid, kTileSlots * S::NC - 1);
      const int slot = p / S::NC, c = S::kHalf ? p % S::NC : (p % S::NC) ^ swz<float>(slot);
      off[k] = (unsigned)tile_site(g, base, slot) * (unsigned)kBytes + (unsigned)c * 16u;
    }
    if constexpr (S::kHalf) own = tile_site(g, base, tid >> 1);
  };
  u4 v[NL];
  float vs[S::kHalf ? NL : 1];
  auto fetch = [&](int rr) {
    const char* f = fin + rr * fs;
#pragma unroll
    for (int k = 0; k < NL; ++k) v[k] = *reinterpret_cast<const u4*>(f + off[k]);
    if constexpr (S::kHalf) {
      const float* sc = io.isc + (size_t)rr * g.vol;
#pragma unroll
      for (int k = 0; k < NL; ++k) vs[k] = sc[off[k] / kBytes];
    }
  };
  auto stage = [&](u4* dst) {
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int p = k * kTileThreads + tid;
      if constexpr (!S::kHalf) {
        dst[p] = v[k];
      } else if (p < kTileSlots * S::NC) {  // four numbers: two FP32 chunks, scaled
        const int slot = p / 3, c = p % 3;
        cx<float> q[12];
        unpack<S>(v[k], 0, q);
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e] = vs[k] * q[e];
        dst[row_pos<Full<float>>(slot, 2 * c)] = chunk_of<float>(q, 0);
        dst[row_pos<Full<float>>(slot, 2 * c + 1)] = chunk_of<float>(q, 1);
      }
    }
  };
  int fr = -1, ft = 0;  // pair whose sums wait in red
  auto flush = [&](int buf) {
    if (fr >= 0 && tid < 3) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < 8; ++q) t += red[buf][q][tid];
      dots[((size_t)fr * ntile + ft) * 3 + tid] = t;
    }
  };
  offsets(tile);
  fetch(r);
  links(tile);
  stage(smem);
  __syncthreads();
  int cur = 0;
  for (;;) {
    u4* sm = smem + cur * kTileChunks;
    u4* nx = smem + (cur ^ 1) * kTileChunks;
    unsigned o3[3];
    int oown = own;
    if constexpr (!S::kHalf) {
#pragma unroll
      for (int k = 0; k < 3; ++k) o3[k] = off[k];
    }
    // the next pair's chunks, in flight while this one is worked on
    int nt = tile, nr = r + 1, nr1 = r1;
    bool more = true;
    if (nr == r1) {
      more = w.next(nt, nr, nr1);
      if (more && nt != tile) offsets(nt);
    }
    if (more) fetch(nr);
    cx<float> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = mk(0.0f, 0.0f);
    if (half == 0)
      tile_hops<0>(sm, u, nbs, acc);
    else
      tile_hops<1>(sm, u, nbs, acc);
    if (more && nt != tile) links(nt);
    __syncthreads();  // every neighbour has been read: the face slots take the sums
    if constexpr (DOTS) flush(cur ^ 1);
    {
      u4* ex = sm + (256 + half * 256) * 6;
#pragma unroll
      for (int c = 0; c < 6; ++c) ex[row_pos<Full<float>>(l, c)] = chunk_of<float>(acc, c);
    }
    if (more) stage(nx);
    __syncthreads();
    double d[3] = {0.0, 0.0, 0.0};
    char* o = fout + r * fs;
    if constexpr (!S::kHalf) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int p = k * kTileThreads + tid;
        ChunkOf<float> a, b, c;
        c.q = sm[p];
        a.q = sm[256 * 6 + p];
        b.q = sm[512 * 6 + p];
#pragma unroll
        for (int e = 0; e < 4; ++e) a.v[e] = diag * c.v[e] - 0.5f * (a.v[e] + b.v[e]);
        *reinterpret_cast<u4*>(o + o3[k]) = a.q;
        if constexpr (DOTS) mr_dots(a.v, c.v, 4, d);
      }
    } else {
      // two threads per site, six numbers each; the scale needs all twelve
      const int j = tid >> 1, h = tid & 1;
      float a[12], p[12];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int pos = row_pos<Full<float>>(j, 3 * h + k);
        ChunkOf<float> x, y, z;
        x.q = sm[pos];
        y.q = sm[256 * 6 + pos];
        z.q = sm[512 * 6 + pos];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[4 * k + e] = x.v[e];
          a[4 * k + e] = diag * x.v[e] - 0.5f * (y.v[e] + z.v[e]);
        }
      }
      float m = site_scale<12>(a);
      m = scale_join(m, __shfl_xor(m, 1, 64));
      float inv;
      const float so = quant_scale(m, inv);
      store_numbers(io, r, g.vol, oown, 6 * h, a, so, inv);
      if constexpr (DOTS) mr_dots(a, p, 12, d);
    }
    if constexpr (DOTS) {
      const double t = wave_sums3(d);
      if (lane >= 60 && lane < 63) red[cur][wave][lane - 60] = t;
      fr = r;
      ft = tile;
    }
    cur ^= 1;
    if (!more) break;
    tile = nt;
    r = nr;
    r1 = nr1;
  }
  if constexpr (DOTS) {
    __syncthreads();
    flush(cur ^ 1);
  }
}

// ---- dispatch ---------------------------------------------------------------
// Forced values of WDMG_TUNE_DSLASH: 5 and 9 name the tile kernel, the others
// the gather kernel.  Automatic choice, from the (lattice, batch) sweep of
// both kernels (us, tile / gather):
//   24^3x48: 2 rhs 124 / 123, 3 rhs 162 / 179, 8 rhs 337 / 426, 32 rhs 1299 / 1649
//   32^4:    2 rhs 189 / 191, 3 rhs 244 / 262     20^4: 6 rhs 71 / 74, 8 rhs 87 / 96
//   16^4:    8 rhs 35 / 34, 12 rhs 47 / 49        28x12x16x36: 6 rhs 82 / 77, 8 rhs 107 / 117
// (FP32).  The tile kernel pays for a prologue per tile, so it needs several
// right-hand sides per tile and enough pairs per compute unit.
constexpr int kFormGather = 1, kFormTile = 5;

template <class S>
bool tile_fits(const Geom& g) {
  if (sizeof(typename S::T) == 8) return false;
  for (int mu = 0; mu < 4; ++mu)
    if (g.B[mu] != 4) return false;
  return (long long)g.vol * S::NC * 16 <= 0xffffffffll;  // 32-bit byte offsets in a field
}

// 16 bits (BF16): 24^3x48: 6 rhs 284 / 286, 8 rhs 363 / 377; 32^4: 3 rhs 251 / 234,
//   8 rhs 557 / 568; 16^4: 12 rhs 52 / 52, 16 rhs 65 / 66; 20x12x20x12: 16 rhs 69 / 68,
//   24 rhs 91 / 95; 28x12x16x36: 12 rhs 158 / 154, 16 rhs 210 / 212.  The gather
//   kernel moves half the bytes there, so it takes a larger batch to beat it.
template <class S>
int auto_form(const Geom& g, int nrhs) {
  if (!tile_fits<S>(g) || nrhs < (S::kHalf ? 6 : 2)) return kFormGather;
  const long long pairs = (long long)(g.vol / 256) * nrhs;
  const long long least = S::kHalf ? (nrhs >= 16 ? 4000 : 15000) : (nrhs >= 8 ? 3000 : 5000);
  return pairs >= least ? kFormTile : kFormGather;
}

// Right-hand sides per workgroup of the gather kernel, at most `most` (16; FP64
// 4: 20x12x20x12, 8 rhs 81 us at 4, 89 at 8; 24^3x48, 32 rhs 3640 at 4, 3540 at
// 8), in groups of equal size.  Two
// site blocks per compute unit are enough workgroups: then the whole batch
// shares its links and offsets (12x20x10x18, 675 blocks, FP32, 5 rhs: 20.8 us in
// one group, 24.1 in two).  With fewer blocks, as many as leave about four
// workgroups per compute unit (8^4, 32 rhs: 13 us at 2, 32 us at 16).
inline int gather_group(const Ctx& c, int nsb, int nrhs, int forced, int most) {
  long long n = forced > 0 ? forced : nsb >= 2 * c.ncu ? most : (long long)nsb * nrhs / (4 * c.ncu);
  if (forced <= 0 && n > most) n = most;
  if (n < 1) n = 1;
  if (n > nrhs) n = nrhs;
  const int groups = (int)((nrhs + n - 1) / n);
  return (nrhs + groups - 1) / groups;
}

template <class S>
void allow_tile_lds() {
  auto allow = [](const void* f) {
    WDMG_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTileLds));
  };
  allow(reinterpret_cast<const void*>(&k_wilson_tile<S, false>));
  if constexpr (S::kDots) allow(reinterpret_cast<const void*>(&k_wilson_tile<S, true>));
}

// Runs the operator; with `dots` the launch also writes the MR partial sums,
// and the return value is the number of slots per rhs.  With g5 (FP64) the
// result is gamma5 D in.
template <class S>
int launch_dslash(Ctx& c, const S& io, int nrhs, int prof_id, int prec_index, double* dots = nullptr, int g5 = 0) {
  using R = typename S::T;
  const Geom& g = c.g0;
  const int key = nrhs < kMaxRhs ? nrhs : kMaxRhs;
  signed char& fslot = c.tune_dslash[prec_index][key];
  signed char& gslot = c.tune_group[prec_index][key];
  int v = c.tune_force[WDMG_TUNE_DSLASH] >= 0 ? c.tune_force[WDMG_TUNE_DSLASH] : fslot;
  if (v < 0) fslot = (signed char)(v = auto_form<S>(g, nrhs));
  const bool tile = (v == 5 || v == 9) && tile_fits<S>(g);
  const int nsb = g.vpad / 64;
  int rg = c.tune_force[WDMG_TUNE_DSLASH_GROUP] >= 0 ? c.tune_force[WDMG_TUNE_DSLASH_GROUP] : gslot;
  const int nper = gather_group(c, nsb, nrhs, rg, sizeof(R) == 8 ? 4 : 16);
  if (rg < 0) gslot = (signed char)(nper < kMaxRhs ? nper : kMaxRhs);
  const bool with_dots = dots != nullptr;
  const int tneg = c.t_bc < 0 ? 1 : 0;
  const R diag = (R)(4.0 + c.mass);
  ProfScope ps(c, prof_id, (long long)g.vol * nrhs);
  c.n_D += nrhs;
  if constexpr (sizeof(R) == 4) {
    if (tile) {
      const int nt = g.vol / 256, nx = nt % 8 == 0 ? 8 : 1;
      const dim3 grid(c.ncu / 8 * 8), block(kTileThreads);
      const auto k = with_dots ? &k_wilson_tile<S, S::kDots> : &k_wilson_tile<S, false>;
      hipLaunchKernelGGL(k, grid, block, kTileLds, c.stream, g, io, diag, tneg, nt, nrhs, nx, dots);
      WDMG_HIP(hipGetLastError());
      return nt;
    }
  }
  const dim3 grid((unsigned)((long long)nsb * ((nrhs + nper - 1) / nper))), block(256);
  auto k = with_dots ? &k_wilson_gather<S, S::kDots, false, R> : &k_wilson_gather<S, false, false, R>;
  if constexpr (S::kHalf || sizeof(R) == 8) {
    // FP64: where all workgroups run at once the latency of the first loads counts, and
    // the backward link is better loaded later (12x20x10x18, 1 rhs 13.1 us against 13.4);
    // with more of them the loop's lighter link rows are (24^3x48, 1 rhs 147 against 141)
    if (nper == 1 && (S::kHalf || (long long)nsb * nrhs <= 4 * c.ncu))
      k = with_dots ? &k_wilson_gather<S, S::kDots, true, R> : &k_wilson_gather<S, false, true, R>;
  }
  hipLaunchKernelGGL(k, grid, block, 0, c.stream, g, io, diag, tneg, nsb, nrhs, nper, g5, dots);
  WDMG_HIP(hipGetLastError());
  return nsb;
}

template <typename R>
Full<R> full_io(Ctx& c, cx<R>* out, const cx<R>* in) {
  Full<R> io;
  io.in = reinterpret_cast<const u4*>(in);
  io.out = reinterpret_cast<u4*>(out);
  if constexpr (sizeof(R) == 8)
    io.U = c.U64;
  else
    io.U = c.U32;
  return io;
}

template <typename H>
Half<H> half_io(Ctx& c, HF out, HF in) {
  Half<H> io;
  io.in = static_cast<const u4*>(in.v);
  io.isc = in.s;
  io.out = static_cast<u4*>(out.v);
  io.osc = out.s;
  io.U = static_cast<const cxh<H>*>(u16(c, half_kind<H>()));
  return io;
}

}  // namespace

void init_dslash() {
  allow_tile_lds<Full<float>>();
  allow_tile_lds<Half<f16_t>>();
  allow_tile_lds<Half<bf16_t>>();
  allow_tile_lds<HalfOut32<f16_t>>();
  allow_tile_lds<HalfOut32<bf16_t>>();
}

template <typename R>
void dslash(Ctx& c, cx<R>* out, const cx<R>* in, int nrhs) {
  launch_dslash(c, full_io<R>(c, out, in), nrhs, sizeof(R) == 8 ? WDMG_K_DSLASH_F64 : WDMG_K_DSLASH_F32,
                sizeof(R) == 8 ? WDMG_F64 : WDMG_F32);
}

void dslash_g5(Ctx& c, cx<double>* out, const cx<double>* in, int nrhs) {
  launch_dslash(c, full_io<double>(c, out, in), nrhs, WDMG_K_DSLASH_F64, WDMG_F64, nullptr, 1);
}

template <typename H>
void dslash_h(Ctx& c, HF out, HF in, int nrhs) {
  launch_dslash(c, half_io<H>(c, out, in), nrhs, half_kind<H>() == WDMG_F16 ? WDMG_K_DSLASH_F16 : WDMG_K_DSLASH_BF16,
                half_kind<H>());
}

double* dots_buffer(Ctx& c, int nrhs) {
  const size_t need = ((size_t)c.g0.vpad / 64 + 2) * 3 * (size_t)nrhs;
  if (need > c.dots_cap) {
    if (c.capturing) throw Error(WDMG_ERR_ARG, "MR partial-sum buffer too small inside a graph capture");
    WDMG_HIP(hipStreamSynchronize(c.stream));
    c.dots_cap = 0;
    dev_renew(c, c.dots, need * sizeof(double));
    c.dots_cap = need;
  }
  return c.dots;
}

template <typename R>
void dslash_mr(Ctx& c, cx<R>* out, const cx<R>* in, int nrhs, double scale, int slot) {
  double* d = dots_buffer(c, nrhs);
  const int nparts = launch_dslash(c, full_io<R>(c, out, in), nrhs,
                                   sizeof(R) == 8 ? WDMG_K_DSLASH_F64 : WDMG_K_DSLASH_F32,
                                   sizeof(R) == 8 ? WDMG_F64 : WDMG_F32, d);
  step_alpha_fin(c, d, nparts, nrhs, scale, slot);
}

template <typename H>
void dslash_h_f32(Ctx& c, cx<float>* out, HF in, int nrhs) {
  HalfOut32<H> io;
  static_cast<Half<H>&>(io) = half_io<H>(c, in, in);
  io.f32 = out;
  launch_dslash(c, io, nrhs, half_kind<H>() == WDMG_F16 ? WDMG_K_DSLASH_F16 : WDMG_K_DSLASH_BF16, half_kind<H>());
}
template <typename H>
void dslash_h_mr(Ctx& c, HF out, HF in, int nrhs, double scale, int slot) {
  double* d = dots_buffer(c, nrhs);
  const int nparts = launch_dslash(c, half_io<H>(c, out, in), nrhs,
                                   half_kind<H>() == WDMG_F16 ? WDMG_K_DSLASH_F16 : WDMG_K_DSLASH_BF16,
                                   half_kind<H>(), d);
  step_alpha_fin(c, d, nparts, nrhs, scale, slot);
}

template void dslash<double>(Ctx&, cx<double>*, const cx<double>*, int);
template void dslash<float>(Ctx&, cx<float>*, const cx<float>*, int);
template void dslash_h<f16_t>(Ctx&, HF, HF, int);
template void dslash_h<bf16_t>(Ctx&, HF, HF, int);
template void dslash_h_f32<f16_t>(Ctx&, cx<float>*, HF, int);
template void dslash_h_f32<bf16_t>(Ctx&, cx<float>*, HF, int);
template void dslash_mr<double>(Ctx&, cx<double>*, const cx<double>*, int, double, int);
template void dslash_mr<float>(Ctx&, cx<float>*, const cx<float>*, int, double, int);
template void dslash_h_mr<f16_t>(Ctx&, HF, HF, int, double, int);
template void dslash_h_mr<bf16_t>(Ctx&, HF, HF, int, double, int);

}  // namespace wdmg

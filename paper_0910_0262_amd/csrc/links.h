// Links as the kernels that read or write all of them see them: the packed
// full matrices, the copies derived from them, and the tile of the caller's
// site-major arrays that one workgroup moves through LDS.
#pragma once
#include "qcd_internal.h"

namespace qcd {

// ------------------------------------------------------------------ derived copies
// Link q = mu * 2 + par at checkerboard site cb, entries r[9]: the copies that
// `c` holds (null: not written).  binary16 entries are rounded float64 ->
// float32 -> binary16, both to nearest even.
__device__ __forceinline__ void store_copies(const LinkCopies& c, int stride, int q, int cb, const double2 (&r)[9]) {
  if (c.u12 != nullptr) {
#pragma unroll
    for (int k = 0; k < 6; ++k) *elem(c.u12, (size_t)(q * 6 + k) * stride, cb) = r[k];
  }
  if (c.uh != nullptr) {  // rows 0, 1: halves 0-7 in a 16-byte chunk, 8-11 in an 8-byte one
    h8_t a;
    h4_t b;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a[2 * k] = (_Float16)(float)r[k].x;
      a[2 * k + 1] = (_Float16)(float)r[k].y;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      b[2 * k] = (_Float16)(float)r[4 + k].x;
      b[2 * k + 1] = (_Float16)(float)r[4 + k].y;
    }
    uint4* p4 = (uint4*)c.uh;
    *elem(p4, (size_t)q * stride, cb) = from_h8(a);
    *elem((uint2*)(p4 + (size_t)8 * stride), (size_t)q * stride, cb) = from_h4(b);
  }
  if (c.uh18 != nullptr) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      unsigned int w[3];
#pragma unroll
      for (int j = 0; j < 3; ++j)
        w[j] = from_h2(h2_t{(_Float16)(float)r[3 * k + j].x, (_Float16)(float)r[3 * k + j].y});
      *elem(c.uh18, (size_t)(q * 3 + k) * stride, cb) = LinkRow{w[0], w[1], w[2]};
    }
  }
}

// ------------------------------------------------------------------ one tile of the caller's arrays
// A workgroup of 256 takes 64 consecutive sites, i.e. 32 checkerboard sites of
// each parity, with one work-item per link: wavefront mu, lanes 0-31 the even
// sites and 32-63 the odd ones.  The caller's site-major arrays are read and
// written in one contiguous run through LDS (N double2 per link; a site's 4 N
// are followed by one of padding against bank conflicts); the packed fields
// are touched in runs of 32 elements.
constexpr int kTileSites = 64;
struct TileLink {
  int mu, par, cb, site;  // site: of the tile, 0 .. 63
  bool live;
};
inline int tile_blocks(const Geom& g) { return (g.V + kTileSites - 1) / kTileSites; }
__device__ __forceinline__ TileLink tile_link(const Geom& g) {
  TileLink t;
  const int lane = threadIdx.x & 63;
  t.mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  t.par = lane >> 5;
  t.cb = (int)blockIdx.x * 32 + (lane & 31);
  t.live = t.cb < g.Vh;
  int x[4];
  cb_coords(t.live ? t.cb : 0, t.par, g, x);
  t.site = 2 * (lane & 31) + (x[0] & 1);
  return t;
}
template <int N>
struct TileLds {
  double2 v[kTileSites * (4 * N + 1)];
  __device__ __forceinline__ double2& at(const TileLink& t, int k) { return v[t.site * (4 * N + 1) + t.mu * N + k]; }
};
// T: the caller's pairs of doubles, by the alignment the caller's array is known to have
template <int N, class T>
__device__ __forceinline__ void tile_read(TileLds<N>& l, const Geom& g, const T* __restrict__ user) {
  const size_t base = (size_t)blockIdx.x * (kTileSites * 4 * N), end = (size_t)g.V * 4 * N;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const int e = c * 256 + (int)threadIdx.x;
    if (base + e < end) {
      const T d = user[base + e];
      l.v[e + e / (4 * N)] = make_double2(d.x, d.y);
    }
  }
  __syncthreads();
}
template <int N>
__device__ __forceinline__ void tile_write(const TileLds<N>& l, const Geom& g, double2* __restrict__ user) {
  __syncthreads();
  const size_t base = (size_t)blockIdx.x * (kTileSites * 4 * N), end = (size_t)g.V * 4 * N;
#pragma unroll
  for (int c = 0; c < N; ++c) {
    const int e = c * 256 + (int)threadIdx.x;
    if (base + e < end) user[base + e] = l.v[e + e / (4 * N)];
  }
}

}  // namespace qcd

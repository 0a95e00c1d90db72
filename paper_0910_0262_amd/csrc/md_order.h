// Work order and gathers of the molecular-dynamics kernels that read
// neighbouring links (gauge force, clover force, hopping force, clover build).
//
// Each link is read by up to 18 work-items of these kernels, so what they
// cost is decided by where those reads are served.
//  * One parity per wavefront.  The fields are kept by checkerboard; with 64
//    lexicographic sites (alternating parity) every load of a wavefront fell
//    into two runs of 512 bytes in steps of two lanes, 34 L1 accesses per
//    load instruction where 1024 contiguous bytes need 16 (counted on the
//    gauge force at 32^3x64: 7.4e8 accesses, 1.2 of its 1.75 ms at one per
//    cycle and CU).  Here 64 lanes are 64 consecutive checkerboard sites.
//  * Tiles in y and z.  Sites go x, y inside a tile, z inside a tile, t, then
//    the next tile; each XCD takes one contiguous range, so that a link's
//    neighbours in every direction are read from the same L2 soon after it.
//    MD_TILE_SITES per t-slice of a tile: 256, 512, 1024, 2048 and 4096
//    measured 1921, 1969, 1920, 1863 and 1750 us (gauge force) and 2884, 2840,
//    2831, 2820 and 2750 us (determinant force) at 32^3x64.
//  * The four directions and two parities of 64 checkerboard positions are
//    eight consecutive workgroups, so that they share their gathers in L2.
// At 32^3x64 the gathers of the gauge force, the clover force and the clover
// build all arrive at about 15.5 TB/s, with one to four wavefronts per SIMD
// alike: what these kernels cost now is the number of matrices they read.
#pragma once
#include "qcd_internal.h"

namespace qcd {

constexpr int MD_TILE_SITES = 4096;

struct MdGeom {
  Geom g;
  int S[4];           // lexicographic strides
  int ty, tz, nty;    // tile extents in y and z (dividing Ly, Lz), tiles along y
  double inv_ty, inv_tz, inv_t, inv_nty;
};

inline MdGeom md_geom(const Geom& g) {
  MdGeom m;
  m.g = g;
  m.S[0] = 1;
  for (int d = 1; d < 4; ++d) m.S[d] = m.S[d - 1] * g.X[d - 1];
  // the largest tile of at most MD_TILE_SITES sites; of equal ones the squarer
  int best = 0;
  m.ty = m.tz = 1;
  for (int ty = 1; ty <= g.X[1]; ++ty) {
    if (g.X[1] % ty != 0) continue;
    for (int tz = 1; tz <= g.X[2]; ++tz) {
      if (g.X[2] % tz != 0) continue;
      const int n = g.X[0] * ty * tz;
      if (n > MD_TILE_SITES) continue;
      const int d = ty > tz ? ty - tz : tz - ty, db = m.ty > m.tz ? m.ty - m.tz : m.tz - m.ty;
      if (n > best || (n == best && d < db)) {
        best = n;
        m.ty = ty;
        m.tz = tz;
      }
    }
  }
  m.nty = g.X[1] / m.ty;
  m.inv_ty = 1.0 / m.ty;
  m.inv_tz = 1.0 / m.tz;
  m.inv_t = 1.0 / g.X[3];
  m.inv_nty = 1.0 / m.nty;
  return m;
}

struct MdSite {
  int x[4];
  int i, cb;  // lexicographic and checkerboard index
};

// The site of parity par at work position j, 0 <= j < Vh, of the tiled order.
__device__ __forceinline__ MdSite md_site(const MdGeom& m, int j, int par) {
  MdSite s;
  int xh, yi, zi, yt;
  int q = fdivmod(j, m.g.Xh, m.g.inv_xh, xh);
  q = fdivmod(q, m.ty, m.inv_ty, yi);
  q = fdivmod(q, m.tz, m.inv_tz, zi);
  q = fdivmod(q, m.g.X[3], m.inv_t, s.x[3]);
  const int zt = fdivmod(q, m.nty, m.inv_nty, yt);
  s.x[1] = yt * m.ty + yi;
  s.x[2] = zt * m.tz + zi;
  s.x[0] = 2 * xh + ((s.x[1] + s.x[2] + s.x[3] + par) & 1);
  s.i = lex(s.x, m.g);
  s.cb = s.i >> 1;
  return s;
}

// Lexicographic index steps from site s to its neighbours in direction d
// (the same for every wavefront lane except across the periodic edge).
__device__ __forceinline__ int md_coord(const MdSite& s, int d) {
  return d == 0 ? s.x[0] : (d == 1 ? s.x[1] : (d == 2 ? s.x[2] : s.x[3]));
}
__device__ __forceinline__ int md_fwd(const MdGeom& m, const MdSite& s, int d) {
  const int st = m.S[d];
  return md_coord(s, d) + 1 == m.g.X[d] ? st - st * m.g.X[d] : st;
}
__device__ __forceinline__ int md_bwd(const MdGeom& m, const MdSite& s, int d) {
  const int st = m.S[d];
  return md_coord(s, d) == 0 ? st * m.g.X[d] - st : -st;
}

// Per-site launches: workgroups of 64, workgroup w takes parity w & 1 of the
// positions 64 (w >> 1) ...; per-link launches: direction (w >> 1) & 3, parity
// w & 1 of the positions 64 (w >> 3) ... (w the XCD-contiguous index).
inline int md_site_blocks(const Geom& g) { return 2 * ((g.Vh + 63) / 64); }
inline int md_link_blocks(const Geom& g) { return 8 * ((g.Vh + 63) / 64); }

// Links are gathered by many neighbouring work-items here, so they are read
// with ordinary (cached) loads, unlike the stencil's streaming loads.  mu and
// par are uniform over the wavefront: a scalar base and a 32-bit lane offset.
__device__ __forceinline__ Mat<double> md_link(const double2* __restrict__ u18, int stride, int mu, int par, int cb) {
  const double2* base = u18 + (size_t)((mu * 2 + par) * 9) * stride;
  Mat<double> u;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 d = *elem(base, (size_t)k * stride, cb);
    u.m[k / 3][k % 3] = {d.x, d.y};
  }
  return u;
}

// c += a b
template <typename R>
__device__ __forceinline__ void mm_acc(Mat<R>& c, const Mat<R>& a, const Mat<R>& b) {
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      c.m[i][j] = cfma(a.m[i][2], b.m[2][j], cfma(a.m[i][1], b.m[1][j], cfma(a.m[i][0], b.m[0][j], c.m[i][j])));
}

}  // namespace qcd

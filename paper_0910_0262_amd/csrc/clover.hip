// Clover term: field strength from the four-leaf clover and the two 6x6
// Hermitian blocks of A = 1 - kappa c_sw sum_{mu<nu} sigma_mu,nu (x) F_mu,nu,
// then the inverse of the odd-site blocks for the even-odd preconditioner.
//
// In the chiral basis sigma_mu,nu = diag(B_up, B_dn) with 2x2 blocks
//   (0,1): -s3, -s3   (0,2): s2, s2   (0,3): s1, -s1
//   (1,2): -s1, -s1   (1,3): s2, -s2  (2,3): s3, -s3
// so sum sigma (x) F = s1 (x) X + s2 (x) Y + s3 (x) Z per chirality with
//   upper: X = F03 - F12, Y = F02 + F13, Z = F23 - F01
//   lower: X = -F12 - F03, Y = F02 - F13, Z = -F01 - F23,
// and s1 (x) X + s2 (x) Y + s3 (x) Z = [[Z, X - iY], [X + iY, -Z]].
#include "md_order.h"

namespace qcd {

// F_mu,nu(x) = traceless part of (Q - Q^dag) / (8i), Q the sum of the four
// counter-clockwise leaves in the mu-nu plane starting at x.
struct FHerm {  // Hermitian 3x3: diagonal, then entries 01, 02, 12
  double d[3];
  Cx<double> x[3];
};
__device__ __forceinline__ FHerm field_strength(const double2* __restrict__ u18, const MdGeom& m,
                                                const MdSite& s, int par, int mu, int nu) {
  const int st = m.g.stride, np = 1 - par;
  const int fm = md_fwd(m, s, mu), fn = md_fwd(m, s, nu), bm = md_bwd(m, s, mu), bn = md_bwd(m, s, nu);
  auto U = [&](int d, int p, int step) { return md_link(u18, st, d, p, (s.i + step) >> 1); };
  const Mat<double> un_x = U(nu, par, 0);
  Mat<double> q, t;
  // U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
  t = mm(U(mu, par, 0), U(nu, np, fm));
  t = mm(t, adj(U(mu, np, fn)));
  q = mm(t, adj(un_x));
  __builtin_amdgcn_sched_barrier(0);
  // U_nu(x) U_mu(x-mu+nu)^dag U_nu(x-mu)^dag U_mu(x-mu)
  t = mm(un_x, adj(U(mu, par, bm + fn)));
  t = mm(t, adj(U(nu, np, bm)));
  const Mat<double> um_xm = U(mu, np, bm);
  mm_acc(q, t, um_xm);
  __builtin_amdgcn_sched_barrier(0);
  // U_mu(x-mu)^dag U_nu(x-mu-nu)^dag U_mu(x-mu-nu) U_nu(x-nu)
  t = mm(adj(um_xm), adj(U(nu, par, bm + bn)));
  t = mm(t, U(mu, par, bm + bn));
  const Mat<double> un_xm = U(nu, np, bn);
  mm_acc(q, t, un_xm);
  __builtin_amdgcn_sched_barrier(0);
  // U_nu(x-nu)^dag U_mu(x-nu) U_nu(x+mu-nu) U_mu(x)^dag
  t = mm(adj(un_xm), U(mu, np, bn));
  t = mm(t, U(nu, par, fm + bn));
  int own = s.cb;  // read again rather than kept: two wavefronts per SIMD leave no registers for it
  asm volatile("" : "+v"(own));
  mm_acc(q, t, adj(md_link(u18, st, mu, par, own)));

  FHerm f;
  const double tr = (q.m[0][0].im + q.m[1][1].im + q.m[2][2].im) / 3.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) f.d[a] = 0.25 * (q.m[a][a].im - tr);
  // (q_ab - conj q_ba) / (8 i)
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const Cx<double> d = q.m[k == 2][k == 0 ? 1 : 2] - conj(q.m[k == 0 ? 1 : 2][k == 2]);
    f.x[k] = {d.im / 8.0, -d.re / 8.0};
  }
  return f;
}

// sa a + sb b
__device__ __forceinline__ FHerm fsum(const FHerm& a, double sa, const FHerm& b, double sb) {
  FHerm f;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    f.d[k] = sa * a.d[k] + sb * b.d[k];
    f.x[k] = sa * a.x[k] + sb * b.x[k];
  }
  return f;
}

// ------------------------------------------------------------------ inversion
// Hermitian positive-definite 6x6 inverse by Cholesky A = L L^dag:
// A^{-1} = L^{-dag} L^{-1}, and ln det A = sum_j ln L_jj^2.  Returns false if
// a pivot is not positive.
__device__ __forceinline__ bool invert_block(const Block<double>& a, Block<double>& inv, double& logdet) {
  Cx<double> L[6][6];
  logdet = 0.0;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    double d = a.d[j];
#pragma unroll
    for (int k = 0; k < j; ++k) d -= norm2(L[j][k]);
    if (!(d > 0.0)) return false;
    logdet += log(d);
    const double ljj = sqrt(d), rinv = 1.0 / ljj;
    L[j][j] = {ljj, 0.0};
#pragma unroll
    for (int i = j + 1; i < 6; ++i) {
      Cx<double> s = conj(a.o[offd(j, i)]);  // A_ij for i > j
#pragma unroll
      for (int k = 0; k < j; ++k) s = s - L[i][k] * conj(L[j][k]);
      L[i][j] = rinv * s;
    }
  }
  // T = L^{-1}, lower triangular
  Cx<double> T[6][6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    T[i][i] = {1.0 / L[i][i].re, 0.0};
#pragma unroll
    for (int j = 0; j < i; ++j) {
      Cx<double> s = {0.0, 0.0};
#pragma unroll
      for (int k = j; k < i; ++k) s = s + L[i][k] * T[k][j];
      T[i][j] = (-1.0 / L[i][i].re) * s;
    }
  }
  // inv = T^dag T: inv_rc = sum_{k >= max(r,c)} conj(T_kr) T_kc
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    double d = 0.0;
#pragma unroll
    for (int k = r; k < 6; ++k) d += norm2(T[k][r]);
    inv.d[r] = d;
#pragma unroll
    for (int c = r + 1; c < 6; ++c) {
      Cx<double> s = {0.0, 0.0};
#pragma unroll
      for (int k = c; k < 6; ++k) s = s + cmulc(T[k][r], T[k][c]);
      inv.o[offd(r, c)] = s;
    }
  }
  return true;
}

__device__ void store_block_f64(double2* base, int stride, int i, const Block<double>& b) {
#pragma unroll
  for (int k = 0; k < 3; ++k) base[(size_t)k * stride + i] = make_double2(b.d[2 * k], b.d[2 * k + 1]);
#pragma unroll
  for (int k = 0; k < 15; ++k) base[(size_t)(3 + k) * stride + i] = make_double2(b.o[k].re, b.o[k].im);
}
__device__ void block_reals(const Block<double>& b, double r[36]) {
#pragma unroll
  for (int k = 0; k < 6; ++k) r[k] = b.d[k];
#pragma unroll
  for (int k = 0; k < 15; ++k) {
    r[6 + 2 * k] = b.o[k].re;
    r[7 + 2 * k] = b.o[k].im;
  }
}
// The 36 reals of one block in FP32, and their max |real|.
__device__ __forceinline__ float block_reals32(const Block<double>& b, float r[36]) {
  double rr[36];
  block_reals(b, rr);
  float m = 0.f;
#pragma unroll
  for (int k = 0; k < 36; ++k) {
    r[k] = float(rr[k]);
    m = fmaxf(m, fabsf(r[k]));
  }
  return m;
}
// binary16 copy of block B, with its scale (max |real|): halves 36 B .. 36 B + 35
// of a site's 72 in nine 16-byte chunks, of which the fifth is shared.
template <int B>
__device__ __forceinline__ void store_half_block(const float r[36], float sc, uint4* h16, float2* hs, int stride, int i) {
  const float inv = sc > 0.f ? 1.0f / sc : 0.f;
  _Float16 h[36];
#pragma unroll
  for (int k = 0; k < 36; ++k) h[k] = (_Float16)(r[k] * inv);
  constexpr int first = B == 0 ? 0 : 4;  // of the halves, in the four whole chunks
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    h8_t c;
#pragma unroll
    for (int j = 0; j < 8; ++j) c[j] = h[first + 8 * k + j];
    h16[(size_t)(5 * B + k) * stride + i] = from_h8(c);
  }
  constexpr int rest = B == 0 ? 32 : 0;
  const h4_t c = {h[rest], h[rest + 1], h[rest + 2], h[rest + 3]};
  ((uint2*)(h16 + (size_t)4 * stride + i))[B] = from_h4(c);
  ((float*)(hs + i))[B] = sc;
}

// Odd-site block B: A_oo^{-1} in FP64 and binary16 (zero if A is not positive
// definite).  Compile-time B: a loop over the blocks indexed its arrays at run
// time, which put both blocks and both inverses in scratch memory.
template <int B>
__device__ __forceinline__ bool invert_site_block(const Block<double>& a, int i, double2* clov_inv, uint4* h16,
                                                  float2* hs, int stride, double& ld) {
  Block<double> inv;
  const bool ok = invert_block(a, inv, ld);
  if (!ok) {
    ld = 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) inv.d[k] = 0.0;
#pragma unroll
    for (int k = 0; k < 15; ++k) inv.o[k] = {0.0, 0.0};
  }
  store_block_f64(clov_inv + (size_t)(B * 18) * stride, stride, i, inv);
  float r[36];
  const float sc = block_reals32(inv, r);
  store_half_block<B>(r, sc, h16, hs, stride, i);
  return ok;
}

// For a loaded clover term (one built from links gets all of this where it is built).
__global__ void __launch_bounds__(64) clover_invert_k(Geom g, const double2* __restrict__ clov, CloverOut o) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.Vh) return;
  const CloverF64 ce{clov, g.stride}, co{clov + (size_t)36 * g.stride, g.stride};
  Block<double> a;
  float r[36];
  load_block(ce, i, 0, a);
  float sc = block_reals32(a, r);
  store_half_block<0>(r, sc, o.h_e, o.h_es, g.stride, i);
  load_block(ce, i, 1, a);
  sc = block_reals32(a, r);
  store_half_block<1>(r, sc, o.h_e, o.h_es, g.stride, i);
  // odd sites: A_oo^{-1}
  double ld0 = 0.0, ld1 = 0.0;
  load_block(co, i, 0, a);
  const bool ok0 = invert_site_block<0>(a, i, o.inv, o.hinv_o, o.hinv_os, g.stride, ld0);
  load_block(co, i, 1, a);
  const bool ok1 = invert_site_block<1>(a, i, o.inv, o.hinv_o, o.hinv_os, g.stride, ld1);
  const bool ok = ok0 && ok1;
  o.logdet[i] = ok ? ld0 + ld1 : 0.0;
  if (!ok) o.status[0] = 1;
}

// FP32 copies of A_ee and A_oo^{-1} (for the FP32 clover option): 18 float4
// chunks, reals [b * 36 + r].
__global__ void __launch_bounds__(64) clover_copy32_k(Geom g, const double2* __restrict__ clov,
                                                      const double2* __restrict__ inv, float4* e32, float4* inv32) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.Vh) return;
#pragma unroll 1
  for (int f = 0; f < 2; ++f) {
    const CloverF64 src{f == 0 ? clov : inv, g.stride};
    float4* const dst = f == 0 ? e32 : inv32;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      Block<double> a;
      load_block(src, i, b, a);
      float r[36];
      (void)block_reals32(a, r);
#pragma unroll
      for (int k = 0; k < 9; ++k)
        dst[(size_t)(9 * b + k) * g.stride + i] = make_float4(r[4 * k], r[4 * k + 1], r[4 * k + 2], r[4 * k + 3]);
    }
  }
}
hipError_t launch_clover_copy32(const Geom& g, const double2* clov, const double2* inv, float4* e32, float4* inv32,
                                hipStream_t s) {
  hipLaunchKernelGGL(clover_copy32_k, dim3(blocks_for(g.Vh, 64)), dim3(64), 0, s, g, clov, inv, e32, inv32);
  return hipGetLastError();
}

// ------------------------------------------------------------------ compact copies of A_ee
// (the site term of k2): per chiral block X3 and W of 1 - [[X3, W], [W^dag,
// -X3]], 26 reals, in FP64 and in binary16 with a per-block scale: halves
// 26 B .. 26 B + 25 of a site's 52, in six chunks of eight and one of four, of
// which the fourth is shared.
template <int B>
__device__ __forceinline__ void store_compact_block(const double r[26], const CloverOut& o, int stride, int i) {
#pragma unroll
  for (int k = 0; k < 13; ++k) o.c64[(size_t)(B * 13 + k) * stride + i] = make_double2(r[2 * k], r[2 * k + 1]);
  float f[26], m = 0.f;
#pragma unroll
  for (int k = 0; k < 26; ++k) {
    f[k] = float(r[k]);
    m = fmaxf(m, fabsf(f[k]));
  }
  const float inv = m > 0.f ? 1.0f / m : 0.f;
  _Float16 h[26];
#pragma unroll
  for (int k = 0; k < 26; ++k) h[k] = (_Float16)(f[k] * inv);
  constexpr int first = B == 0 ? 0 : 6;  // of the halves, in the whole chunks 0 .. 2 or 4, 5
#pragma unroll
  for (int k = 0; k < (B == 0 ? 3 : 2); ++k) {
    h8_t c;
#pragma unroll
    for (int j = 0; j < 8; ++j) c[j] = h[first + 8 * k + j];
    o.ch[(size_t)(4 * B + k) * stride + i] = from_h8(c);
  }
  unsigned int* const mid = (unsigned int*)(o.ch + (size_t)3 * stride + i);
  if constexpr (B == 0) {
    mid[0] = from_h2(h2_t{h[24], h[25]});
  } else {
#pragma unroll
    for (int j = 0; j < 3; ++j) mid[1 + j] = from_h2(h2_t{h[2 * j], h[2 * j + 1]});
    const h4_t t = {h[22], h[23], h[24], h[25]};
    ((uint2*)(o.ch + (size_t)6 * stride))[i] = from_h4(t);
  }
  ((float*)(o.chs + i))[B] = m;
}
// Of a loaded clover term: the form holds for one built from links; for any
// other, status[1] is set and the caller keeps the full blocks.
template <int B>
__device__ __forceinline__ double compact_loaded(const CloverF64& ce, const CloverOut& o, int stride, int i) {
  Block<double> a;
  load_block(ce, i, B, a);
  double r[26];
  r[0] = 0.5 * (a.d[3] - a.d[0]);
  r[1] = 0.5 * (a.d[4] - a.d[1]);
  const Cx<double> x01 = 0.5 * (a.o[offd(3, 4)] - a.o[offd(0, 1)]);
  const Cx<double> x02 = 0.5 * (a.o[offd(3, 5)] - a.o[offd(0, 2)]);
  const Cx<double> x12 = 0.5 * (a.o[offd(4, 5)] - a.o[offd(1, 2)]);
  r[2] = x01.re;
  r[3] = x01.im;
  r[4] = x02.re;
  r[5] = x02.im;
  r[6] = x12.re;
  r[7] = x12.im;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const Cx<double> w = a.o[offd(k / 3, 3 + k % 3)];
    r[8 + 2 * k] = -w.re;
    r[9 + 2 * k] = -w.im;
  }
  store_compact_block<B>(r, o, stride, i);
  // B00 + B11 = 2 and tr X3 = 0
  double dev = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) dev = fmax(dev, fabs(a.d[k] + a.d[3 + k] - 2.0));
  const Cx<double> s01 = a.o[offd(0, 1)] + a.o[offd(3, 4)], s02 = a.o[offd(0, 2)] + a.o[offd(3, 5)],
                   s12 = a.o[offd(1, 2)] + a.o[offd(4, 5)];
  dev = fmax(dev, fmax(fmax(fabs(s01.re), fabs(s01.im)), fmax(fabs(s02.re), fabs(s02.im))));
  dev = fmax(dev, fmax(fabs(s12.re), fabs(s12.im)));
  return fmax(dev, fabs(a.d[3] + a.d[4] + a.d[5] - a.d[0] - a.d[1] - a.d[2]));
}
__global__ void __launch_bounds__(64) clover_compact_k(Geom g, const double2* __restrict__ clov, CloverOut o) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.Vh) return;
  const CloverF64 ce{clov, g.stride};
  const double d0 = compact_loaded<0>(ce, o, g.stride, i), d1 = compact_loaded<1>(ce, o, g.stride, i);
  if (fmax(d0, d1) > 1e-12) o.status[1] = 1;
}

hipError_t launch_clover_invert(const Geom& g, const double2* clov, const CloverOut& o, hipStream_t s) {
  hipLaunchKernelGGL(clover_invert_k, dim3(blocks_for(g.Vh, 64)), dim3(64), 0, s, g, clov, o);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(clover_compact_k, dim3(blocks_for(g.Vh, 64)), dim3(64), 0, s, g, clov, o);
  return hipGetLastError();
}

// ------------------------------------------------------------------ build
// F per plane, A, and all that is derived from A, in one launch: A and A^{-1}
// are written once and never read back (inversion and copies as two launches
// of their own read 1.8 GB of the 32^3x64 term again).  The F of 64 sites of
// one parity (9 reals each) meet in LDS; then one wavefront per chiral block
// writes the block of A and, on even sites, its compact and binary16 copies
// or, on odd sites, A^{-1}, its binary16 copy and ln det A.
//
// Two forms.  TILES = 2: four wavefronts take the even and the odd sites of
// the same place, three planes each, then one block each: all four stay busy,
// two workgroups fill a CU's eight places, and one gathers links while the
// other inverts.  TILES = 1: six wavefronts take one parity, one plane each;
// two of them go on to the blocks, and one workgroup fits a CU.  It has the
// shorter chain of dependent loads, which is all that counts while a workgroup
// gets a CU to itself anyway: us for the whole call, TILES = 1 and 2:
//   8^4 26 | 32, 8^2 x16^2 (512 units) 29 | 35, 12^3x24 (648 units) 59 | 55,
//   16^4 76 | 68, 24^3x48 750 | 627, 32^3x64 2320 | 1850.
// The line lies at 512 units (64 sites of a parity), two per CU.  With three
// launches the call took 91 us at 16^4 and 2350 us at 32^3x64.  Bound by the
// links' way from L2 to the CUs (78 of 144 bytes per site, 1.05 ms at 32^3x64)
// and 2.6 GB of results (0.45 ms).  Three wavefronts per SIMD (24 KB of LDS
// per tile) lose: 2093 us.
struct BuildLds {
  double f[6][9][64];
};
__device__ __forceinline__ FHerm lds_f(const BuildLds& l, int p, int lane) {
  FHerm f;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    f.d[k] = l.f[p][k][lane];
    f.x[k] = {l.f[p][3 + 2 * k][lane], l.f[p][4 + 2 * k][lane]};
  }
  return f;
}
// The plane sums of one chiral half times kappa c_sw: block entries 1 -+ Z on
// the diagonal sub-blocks and -(X - iY) beside them.
//   upper half X = F03 - F12, Y = F02 + F13, Z = F23 - F01;
//   lower half X = -F03 - F12, Y = F02 - F13, Z = -F23 - F01
__device__ __forceinline__ FHerm half_z(const BuildLds& l, int h, double kc, int lane) {
  return fsum(lds_f(l, 5, lane), h == 0 ? kc : -kc, lds_f(l, 0, lane), -kc);
}
__device__ __forceinline__ void half_offdiag(const BuildLds& l, int h, double kc, int lane, Cx<double> w[3][3]) {
  const double sg = h == 0 ? kc : -kc;
  const FHerm x = fsum(lds_f(l, 2, lane), sg, lds_f(l, 3, lane), -kc);
  const FHerm y = fsum(lds_f(l, 1, lane), kc, lds_f(l, 4, lane), sg);
#pragma unroll
  for (int a = 0; a < 3; ++a) w[a][a] = {-x.d[a], y.d[a]};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int a = k == 2 ? 1 : 0, b = k == 0 ? 1 : 2;
    w[a][b] = ti(y.x[k]) - x.x[k];
    w[b][a] = ti(conj(y.x[k])) - conj(x.x[k]);
  }
}
__device__ __forceinline__ void half_block(const FHerm& z, const Cx<double> (&w)[3][3], Block<double>& b) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    b.d[a] = 1.0 - z.d[a];
    b.d[3 + a] = 1.0 + z.d[a];
#pragma unroll
    for (int c = 0; c < 3; ++c) b.o[offd(a, 3 + c)] = w[a][c];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int a = k == 2 ? 1 : 0, c = k == 0 ? 1 : 2;
    b.o[offd(a, c)] = -z.x[k];
    b.o[offd(3 + a, 3 + c)] = z.x[k];
  }
}
// Block B of 64 sites of parity par: A, then what is derived from it; ln det A
// and whether it could be inverted go to the plane sums' place in LDS, which
// no other wavefront reads any more.
template <int B>
__device__ __forceinline__ void finish_block(const BuildLds& lds, int par, int cb, double kc, int lane, int stride,
                                             double2* clov, const CloverOut& o, double& ld, bool& ok) {
  const FHerm z = half_z(lds, B, kc, lane);
  Cx<double> w[3][3];
  half_offdiag(lds, B, kc, lane, w);
  Block<double> a;
  half_block(z, w, a);
  store_block_f64(clov + (size_t)(par * 36 + B * 18) * stride, stride, cb, a);
  if (par == 1) {
    ok = invert_site_block<B>(a, cb, o.inv, o.hinv_o, o.hinv_os, stride, ld);
    return;
  }
  float f[36];
  const float sc = block_reals32(a, f);
  store_half_block<B>(f, sc, o.h_e, o.h_es, stride, cb);
  double r[26];
  r[0] = z.d[0];
  r[1] = z.d[1];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    r[2 + 2 * k] = z.x[k].re;
    r[3 + 2 * k] = z.x[k].im;
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    r[8 + 2 * k] = -w[k / 3][k % 3].re;
    r[9 + 2 * k] = -w[k / 3][k % 3].im;
  }
  store_compact_block<B>(r, o, stride, cb);
}

template <int TILES>
__global__ void __launch_bounds__(TILES == 1 ? 384 : 256) clover_build_k(MdGeom m, const double2* __restrict__ u18,
                                                                         double kc, double2* __restrict__ clov,
                                                                         CloverOut o) {
  __shared__ BuildLds lds[TILES];
  constexpr int kPlanes = TILES == 1 ? 1 : 3;
  const Geom& g = m.g;
  const int w = xcd_block(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = ((TILES == 1 ? w >> 1 : w) << 6) + lane;
  const bool live = j < g.Vh;
  auto parity = [&](int tile) { return TILES == 1 ? w & 1 : tile; };
  {
    const int tile = TILES == 1 ? 0 : wave >> 1, par = parity(tile);
    const MdSite s = md_site(m, min(j, g.Vh - 1), par);
#pragma unroll 1
    for (int q = 0; q < kPlanes; ++q) {
      const int p = TILES == 1 ? wave : 3 * (wave & 1) + q;
      // planes 01 02 03 12 13 23
      const int mu = p < 3 ? 0 : (p < 5 ? 1 : 2), nu = p < 3 ? p + 1 : (p < 5 ? p - 1 : 3);
      const FHerm f = field_strength(u18, m, s, par, mu, nu);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        lds[tile].f[p][k][lane] = f.d[k];
        lds[tile].f[p][3 + 2 * k][lane] = f.x[k].re;
        lds[tile].f[p][4 + 2 * k][lane] = f.x[k].im;
      }
    }
  }
  __syncthreads();
  const int tile = wave >> 1, par = parity(tile);
  const int cb = md_site(m, min(j, g.Vh - 1), par).cb;
  double ld = 0.0;
  bool ok = true;
  if (live && wave < 2 * TILES) {
    if ((wave & 1) == 0)
      finish_block<0>(lds[tile], par, cb, kc, lane, g.stride, clov, o, ld, ok);
    else
      finish_block<1>(lds[tile], par, cb, kc, lane, g.stride, clov, o, ld, ok);
  }
  // ln det A of both blocks (none where either failed)
  if (TILES == 1 && par == 0) return;  // the whole workgroup
  BuildLds& odd = lds[TILES - 1];
  __syncthreads();
  if (wave == 2 * TILES - 1) {
    odd.f[0][0][lane] = ld;
    odd.f[0][1][lane] = ok ? 1.0 : 0.0;
  }
  __syncthreads();
  if (wave == 2 * TILES - 2 && live) {
    const bool both = ok && odd.f[0][1][lane] != 0.0;
    o.logdet[cb] = both ? ld + odd.f[0][0][lane] : 0.0;
    if (!both) o.status[0] = 1;
  }
}

hipError_t launch_clover_build(const Geom& g, const double2* u18, double kappa, double csw, double2* clov,
                               const CloverOut& o, hipStream_t s) {
  const int units = md_site_blocks(g);
  if (units <= 512)
    hipLaunchKernelGGL(clover_build_k<1>, dim3(units), dim3(384), 0, s, md_geom(g), u18, kappa * csw, clov, o);
  else
    hipLaunchKernelGGL(clover_build_k<2>, dim3(units / 2), dim3(256), 0, s, md_geom(g), u18, kappa * csw, clov, o);
  return hipGetLastError();
}

}  // namespace qcd

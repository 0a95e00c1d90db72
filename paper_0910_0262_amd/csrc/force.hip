// Fermion force for S = phi^dag (Mhat^dag Mhat)^{-1} phi and the HMD link and
// momentum updates.
//
// With X = (Mhat^dag Mhat)^{-1} phi, Y = Mhat X, Z = A_oo^{-1} H_oe X and
// W = A_oo^{-1} H_eo^dag Y, the first-order change of S is
//   dS = 2 kappa^2 Re[l^dag dH r] + 2 kappa c_sw Re sum_x,mu<nu tr[dF_mu,nu(x) Gamma_mu,nu(x)]
// with full-lattice l = (Y even, W odd), r = (X even, Z odd) and
// Gamma_mu,nu(x)_ba = sum_s,s' (sigma_mu,nu)_ss' Lambda(x)_(s'b),(sa),
// Lambda = X Y^dag on even sites and kappa^2 Z W^dag on odd sites.
// The kernels write G = dS/dRe U + i dS/dIm U per link (dS = Re sum conj(G) dU).
//
// Hopping part, per link U_mu(x) (eta = boundary sign of the hop):
//   G = 2 kappa^2 eta (B^dag + C),
//   B = sum_k h-_k(r(x+mu)) h-_k(l(x))^dag,  C = sum_k h+_k(r(x)) h+_k(l(x+mu))^dag,
// where h-(v), h+(v) are the upper spin pair of (1 -+ gamma_mu) v: the
// projectors are rank two, so the spin trace reduces to two colour outer products.
//
// Clover part: Re tr[dF Gamma] = (1/4) Im tr[dQ Xi] with Xi the Hermitian part
// of the traceless part of Gamma; each link enters the leaves of 6 plaquettes
// at 4 corners each, and a leaf derivative is the product of the other three
// links with Xi inserted at the leaf's corner.
#include "links.h"
#include "md_order.h"

namespace qcd {

// ------------------------------------------------------------------ helpers
__device__ __forceinline__ void spinor_at(SpF64 e, SpF64 o, int par, int cb, Spinor<double>& v) {
  load(par ? o : e, cb, v);
}
// out += sum_k a_k (x) b_k^dag  (colour outer products, out[row][col] = a_row conj(b_col))
__device__ __forceinline__ void outer_acc(Mat<double>& out, const Half<double>& a, const Half<double>& b) {
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) out.m[r][c] = out.m[r][c] + a.h[k][r] * conj(b.h[k][c]);
}
__device__ __forceinline__ void store_mat(double2* base, int stride, int i, const Mat<double>& m) {
#pragma unroll
  for (int k = 0; k < 9; ++k) base[(size_t)k * stride + i] = make_double2(m.m[k / 3][k % 3].re, m.m[k / 3][k % 3].im);
}
__device__ __forceinline__ Mat<double> load_mat(const double2* base, int stride, int i) {
  Mat<double> m;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 d = base[(size_t)k * stride + i];
    m.m[k / 3][k % 3] = {d.x, d.y};
  }
  return m;
}

int md_link_partials(const Geom& g) { return md_link_blocks(g); }

// ------------------------------------------------------------------ output of a force pass
// A workgroup of NW wavefronts holds G of one direction at 64 sites of one
// parity, in wavefront 0.  The caller's arrays are site-major, so a lane's own
// 16-byte stores would each be a write request of their own (a separate output
// kernel that made them took 1.2 ms for G and F at 32^3x64); the values pass
// through LDS instead and go out as runs of one link (144 bytes of G, 64 of F).
// F^a = Re{ i tr[T^a U G^dag] } = -Im(tr[lambda^a W]) / 2, W = U G^dag.
template <int NW>
struct MdLds {
  double2 v[(NW > 2 ? 2 * 576 : 576 + 256)];
};
// F and P are arrays of double in the caller's memory: pairs of them, 8-byte aligned
typedef double d2_a8 __attribute__((ext_vector_type(2), aligned(8)));
// run(e, at): double2 number e of the 64 links' N double2 values each, element `at` of the caller's array
template <int N, int NW, class F>
__device__ __forceinline__ void md_runs(int lex_site, int n_live, int mu, F run) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int c0 = 0; c0 < N; c0 += NW) {
    const int c = c0 + (NW > 1 ? (int)(threadIdx.x >> 6) : 0);
    if (c >= N) break;
    const int e = c * 64 + lane, l = e / N;
    const int i = __shfl(lex_site, l, 64);
    if (l < n_live) run(e, ((size_t)i * 4 + mu) * N + (e - l * N));
  }
}
// G = gin + i mt^dag, mt the sum of the wavefronts' parts (in their order).
// Every thread of the workgroup calls it.
template <int NW>
__device__ __forceinline__ void md_emit(const MdOut& o, const double2* gin, MdLds<NW>& lds, const Geom& g, const MdSite& s,
                                        int n_live, int mu, int par, const double2* __restrict__ u18,
                                        const Mat<double>& part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const size_t field = (size_t)((mu * 2 + par) * 9) * g.stride;
  double2* const other = lds.v + 576;
  if constexpr (NW > 1) {
    if (wave > 0) {
#pragma unroll
      for (int k = 0; k < 9; ++k)
        lds.v[(wave - 1) * 576 + k * 64 + lane] = make_double2(part.m[k / 3][k % 3].re, part.m[k / 3][k % 3].im);
    }
    __syncthreads();
  }
  if (wave == 0) {
    Mat<double> mt = part, G = gin != nullptr ? load_mat(gin + field, g.stride, s.cb) : mzero<double>();
#pragma unroll
    for (int w = 1; w < NW; ++w)
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const double2 d = lds.v[(w - 1) * 576 + k * 64 + lane];
        mt.m[k / 3][k % 3] = mt.m[k / 3][k % 3] + Cx<double>{d.x, d.y};
      }
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) G.m[r][c] = G.m[r][c] + ti(conj(mt.m[c][r]));
    if (o.g_user != nullptr) {
#pragma unroll
      for (int k = 0; k < 9; ++k) lds.v[lane * 9 + k] = make_double2(G.m[k / 3][k % 3].re, G.m[k / 3][k % 3].im);
    }
    if (o.f_user != nullptr || o.p_user != nullptr) {
      const Mat<double> W = mm(md_link(u18, g.stride, mu, par, s.cb), adj(G));
      const double r3 = 0.57735026918962576451;  // 1 / sqrt(3)
      double f[8];
      f[0] = W.m[0][1].im + W.m[1][0].im;
      f[1] = (W.m[0][1] - W.m[1][0]).re;  // Im(i z) = Re z
      f[2] = W.m[0][0].im - W.m[1][1].im;
      f[3] = W.m[0][2].im + W.m[2][0].im;
      f[4] = (W.m[0][2] - W.m[2][0]).re;
      f[5] = W.m[1][2].im + W.m[2][1].im;
      f[6] = (W.m[1][2] - W.m[2][1]).re;
      f[7] = (W.m[0][0].im + W.m[1][1].im - 2.0 * W.m[2][2].im) * r3;
#pragma unroll
      for (int k = 0; k < 4; ++k) other[lane * 4 + k] = make_double2(-0.5 * f[2 * k], -0.5 * f[2 * k + 1]);
    }
  }
  __syncthreads();
  if (o.g_user != nullptr) md_runs<9, NW>(s.i, n_live, mu, [&](int e, size_t at) { o.g_user[at] = lds.v[e]; });
  if (o.f_user == nullptr && o.p_user == nullptr) return;
  md_runs<4, NW>(s.i, n_live, mu, [&](int e, size_t at) {
    const double2 v = other[e];
    if (o.f_user != nullptr) ((d2_a8*)o.f_user)[at] = d2_a8{v.x, v.y};
    if (o.p_user != nullptr) {  // P <- P - dt F
      const d2_a8 p = ((const d2_a8*)o.p_user)[at];
      ((d2_a8*)o.p_user)[at] = d2_a8{p.x - o.dt * v.x, p.y - o.dt * v.y};
    }
  });
}
// Common start of a per-link kernel: direction, parity and site of this
// work-item (lanes past the lattice repeat its last site and store nothing).
__device__ __forceinline__ void md_link_site(const MdGeom& m, int& w, int& mu, int& par, int& n_live, MdSite& s) {
  w = xcd_block(blockIdx.x, gridDim.x);
  mu = (w >> 1) & 3;
  par = w & 1;
  const int j0 = (w >> 3) << 6;
  n_live = min(64, m.g.Vh - j0);
  s = md_site(m, min(j0 + (int)(threadIdx.x & 63), m.g.Vh - 1), par);
}

// G taken from the accumulator alone (no accumulator: zero)
__global__ void __launch_bounds__(64) force_finish_k(MdGeom m, const double2* __restrict__ u18,
                                                     const double2* gin, MdOut o) {
  __shared__ MdLds<1> lds;
  int w, mu, par, n_live;
  MdSite s;
  md_link_site(m, w, mu, par, n_live, s);
  md_emit<1>(o, gin, lds, m.g, s, n_live, mu, par, u18, mzero<double>());
}
hipError_t launch_force_finish(const Geom& g, const double2* u18, const double2* gin, const MdOut& o, hipStream_t s) {
  hipLaunchKernelGGL(force_finish_k, dim3(md_link_blocks(g)), dim3(64), 0, s, md_geom(g), u18, gin, o);
  return hipGetLastError();
}

// ------------------------------------------------------------------ hopping force
template <int MU>
__device__ __forceinline__ Mat<double> hop_force_dir(const MdGeom& m, const MdSite& s, int par, SpF64 le, SpF64 lo,
                                                     SpF64 re, SpF64 ro) {
  const int ny = (s.i + md_fwd(m, s, MU)) >> 1;
  Spinor<double> l_x, r_x, l_y, r_y;
  spinor_at(le, lo, par, s.cb, l_x);
  spinor_at(re, ro, par, s.cb, r_x);
  spinor_at(le, lo, 1 - par, ny, l_y);
  spinor_at(re, ro, 1 - par, ny, r_y);
  Half<double> a, b;
  Mat<double> B = mzero<double>(), C = mzero<double>();
  project<MU, -1>(r_y, a);
  project<MU, -1>(l_x, b);
  outer_acc(B, a, b);
  project<MU, +1>(r_x, a);
  project<MU, +1>(l_y, b);
  outer_acc(C, a, b);
  return madd(adj(B), C);
}

__global__ void __launch_bounds__(64) force_hop_k(MdGeom m, SpF64 le, SpF64 lo, SpF64 re, SpF64 ro, double coef,
                                                  double2* __restrict__ gint) {
  const int w = xcd_block(blockIdx.x, gridDim.x), par = w & 1;
  const int j = ((w >> 1) << 6) + threadIdx.x;
  if (j >= m.g.Vh) return;
  const MdSite s = md_site(m, j, par);
  Mat<double> f[4];
  f[0] = hop_force_dir<0>(m, s, par, le, lo, re, ro);
  f[1] = hop_force_dir<1>(m, s, par, le, lo, re, ro);
  f[2] = hop_force_dir<2>(m, s, par, le, lo, re, ro);
  f[3] = hop_force_dir<3>(m, s, par, le, lo, re, ro);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    const double eta = (mu == 3 && m.g.tb < 0 && s.x[3] == m.g.X[3] - 1) ? -coef : coef;
    Mat<double> g;
#pragma unroll
    for (int k = 0; k < 9; ++k) g.m[k / 3][k % 3] = eta * f[mu].m[k / 3][k % 3];
    store_mat(gint + (size_t)((mu * 2 + par) * 9) * m.g.stride, m.g.stride, s.cb, g);
  }
}

hipError_t launch_force_hop(const Geom& g, SpF64 ell_e, SpF64 ell_o, SpF64 rho_e, SpF64 rho_o, double coef,
                            double2* gint, hipStream_t s) {
  hipLaunchKernelGGL(force_hop_k, dim3(md_site_blocks(g)), dim3(64), 0, s, md_geom(g), ell_e, ell_o, rho_e, rho_o,
                     coef, gint);
  return hipGetLastError();
}

// ------------------------------------------------------------------ clover force: Xi per site
// plane p: 0 (0,1), 1 (0,2), 2 (0,3), 3 (1,2), 4 (1,3), 5 (2,3)
// Xi of a plane is the traceless Hermitian part of
//   Gamma_ab = sum_s,s' (sigma_mu,nu)_ss' Lambda_(s'a),(sb),
// with sigma_mu,nu = sgn times a Pauli matrix on each chiral half.  sigma is
// Hermitian, so the Hermitian part may be taken of Lambda first: of each
// half's 6x6 Lambda only D = Lambda_00 - Lambda_11 and O = Lambda_01 enter,
//   T1 = O + O^dag,  T2 = i (O - O^dag),  T3 = D,
// and the six planes are sums and differences of the two halves' T.
// Stored packed: 4 double2 per plane and site, (d0, d1), x01, x02, x12 of
// [[d0, x01, x02], [., d1, x12], [., ., -d0 - d1]] (64 bytes instead of the
// 144 of a general matrix, which the clover force gathers 18 times per link).
struct Herm {
  double d0, d1;
  Cx<double> x01, x02, x12;
};
__device__ __forceinline__ void store_xi(double2* xi, int stride, int par, int p, int cb, const Herm& h) {
  double2* b = xi + (size_t)((par * 6 + p) * kXiChunks) * stride;
  *elem(b, 0, cb) = make_double2(h.d0, h.d1);
  *elem(b, (size_t)stride, cb) = make_double2(h.x01.re, h.x01.im);
  *elem(b, (size_t)2 * stride, cb) = make_double2(h.x02.re, h.x02.im);
  *elem(b, (size_t)3 * stride, cb) = make_double2(h.x12.re, h.x12.im);
}

// D and O of one chiral half, as the three T matrices' independent entries
struct Tri {
  double d[3][3];  // d[k]: diagonal of T_{k+1}, trace removed (two entries used)
  Cx<double> x[3][3];  // x[k]: entries 01, 02, 12 of T_{k+1}
};
template <bool FERM, bool DET>
__device__ __forceinline__ Tri half_tri(const Cx<double> (&l)[2][3], const Cx<double> (&r)[2][3], double w,
                                        const double2* __restrict__ inv, int stride, int cb, double w_det, int half,
                                        bool odd) {
  const double hw = 0.5 * w;
  double dd[3] = {0.0, 0.0, 0.0};
  Cx<double> dx[3] = {}, o[3][3] = {};
  if constexpr (FERM) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      // Re(r_a conj l_a) of spin 0 minus spin 1
      dd[a] = w * ((r[0][a].re * l[0][a].re + r[0][a].im * l[0][a].im) -
                   (r[1][a].re * l[1][a].re + r[1][a].im * l[1][a].im));
#pragma unroll
      for (int b = 0; b < 3; ++b)
        o[a][b] = hw * cfma(l[0][a], conj(r[1][b]), r[0][a] * conj(l[1][b]));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int a = k == 2 ? 1 : 0, b = k == 0 ? 1 : 2;
      const Cx<double> up = cfma(l[0][a], conj(r[0][b]), r[0][a] * conj(l[0][b]));
      const Cx<double> dn = cfma(l[1][a], conj(r[1][b]), r[1][a] * conj(l[1][b]));
      dx[k] = hw * (up - dn);
    }
  }
  if constexpr (DET) {
    if (odd) {
      Block<double> B;
      load_block(CloverF64{inv, stride}, cb, half, B);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        dd[a] += w_det * (B.d[a] - B.d[3 + a]);
#pragma unroll
        for (int b = 0; b < 3; ++b) o[a][b] = o[a][b] + w_det * B.o[offd(a, 3 + b)];
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int a = k == 2 ? 1 : 0, b = k == 0 ? 1 : 2;
        dx[k] = dx[k] + w_det * (B.o[offd(a, b)] - B.o[offd(3 + a, 3 + b)]);
      }
    }
  }
  Tri t;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    t.d[0][a] = 2.0 * o[a][a].re;
    t.d[1][a] = -2.0 * o[a][a].im;
    t.d[2][a] = dd[a];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int a = k == 2 ? 1 : 0, b = k == 0 ? 1 : 2;
    t.x[0][k] = o[a][b] + conj(o[b][a]);
    t.x[1][k] = ti(o[a][b] - conj(o[b][a]));
    t.x[2][k] = dx[k];
  }
  return t;
}

// Xi per site and plane.  FERM: Lambda = r l^dag with weight w_e (even) or w_o
// (odd).  DET: Lambda += w_det A_oo^{-1} on odd sites (the derivative of
// -2 sum_odd ln det A has the same form as the fermion clover term, with
// A_oo^{-1} in place of kappa^2 Z W^dag).
template <bool FERM, bool DET>
__global__ void __launch_bounds__(64) clover_xi_k(Geom g, SpF64 le, SpF64 lo, SpF64 re, SpF64 ro, double w_e,
                                                  double w_o, const double2* __restrict__ cinv, double w_det,
                                                  double2* __restrict__ xi) {
  // one parity per workgroup: the determinant part (odd sites) runs on whole wavefronts
  const int w = xcd_block(blockIdx.x, gridDim.x), par = w & 1;
  const int cb = ((w >> 1) << 6) + threadIdx.x;
  if (cb >= g.Vh) return;
  const double wt = par ? w_o : w_e;
  Tri t[2];
  Spinor<double> l, r;
  if constexpr (FERM) {
    load(par ? lo : le, cb, l);
    load(par ? ro : re, cb, r);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    Cx<double> lh[2][3] = {}, rh[2][3] = {};
    if constexpr (FERM) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          lh[s][c] = l.v[2 * h + s][c];
          rh[s][c] = r.v[2 * h + s][c];
        }
    }
    t[h] = half_tri<FERM, DET>(lh, rh, wt, cinv, g.stride, cb, w_det, h, par == 1);
  }
  // plane p: (T of the upper half) su + (T of the lower half) sd, T of Pauli matrix k + 1
  constexpr int kk[6] = {2, 1, 0, 0, 1, 2};
  constexpr double su[6] = {-1, 1, 1, -1, 1, 1}, sd[6] = {-1, 1, -1, -1, -1, -1};
#pragma unroll
  for (int p = 0; p < 6; ++p) {
    const int k = kk[p];
    double d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) d[a] = su[p] * t[0].d[k][a] + sd[p] * t[1].d[k][a];
    const double tr = (d[0] + d[1] + d[2]) / 3.0;
    Herm h;
    h.d0 = d[0] - tr;
    h.d1 = d[1] - tr;
    h.x01 = su[p] * t[0].x[k][0] + sd[p] * t[1].x[k][0];
    h.x02 = su[p] * t[0].x[k][1] + sd[p] * t[1].x[k][1];
    h.x12 = su[p] * t[0].x[k][2] + sd[p] * t[1].x[k][2];
    store_xi(xi, g.stride, par, p, cb, h);
  }
}

hipError_t launch_clover_xi(const Geom& g, SpF64 ell_e, SpF64 ell_o, SpF64 rho_e, SpF64 rho_o, double w_e,
                            double w_o, const double2* cinv, double w_det, double2* xi, hipStream_t s) {
  const dim3 grid(md_site_blocks(g)), block(64);
  const bool ferm = ell_e.p != nullptr, det = cinv != nullptr;
  if (ferm && det)
    hipLaunchKernelGGL((clover_xi_k<true, true>), grid, block, 0, s, g, ell_e, ell_o, rho_e, rho_o, w_e, w_o, cinv,
                       w_det, xi);
  else if (ferm)
    hipLaunchKernelGGL((clover_xi_k<true, false>), grid, block, 0, s, g, ell_e, ell_o, rho_e, rho_o, w_e, w_o, cinv,
                       w_det, xi);
  else if (det)
    hipLaunchKernelGGL((clover_xi_k<false, true>), grid, block, 0, s, g, ell_e, ell_o, rho_e, rho_o, w_e, w_o, cinv,
                       w_det, xi);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// ------------------------------------------------------------------ clover force: leaf derivatives
__device__ __forceinline__ int plane_index(int a, int b) {  // a < b
  return a == 0 ? b - 1 : (a == 1 ? b + 1 : 5);
}
// sgn Xi of plane p at checkerboard site cb of parity par
__device__ __forceinline__ Mat<double> xi_at(const double2* __restrict__ xi, int stride, int p, int par, int cb,
                                             double sgn) {
  const double2* b = xi + (size_t)((par * 6 + p) * kXiChunks) * stride;
  const double2 d = *elem(b, 0, cb), a = *elem(b, (size_t)stride, cb), e = *elem(b, (size_t)2 * stride, cb),
                f = *elem(b, (size_t)3 * stride, cb);
  Mat<double> m;
  const double d0 = sgn * d.x, d1 = sgn * d.y;
  m.m[0][0] = {d0, 0.0};
  m.m[1][1] = {d1, 0.0};
  m.m[2][2] = {-d0 - d1, 0.0};
  m.m[0][1] = {sgn * a.x, sgn * a.y};
  m.m[0][2] = {sgn * e.x, sgn * e.y};
  m.m[1][2] = {sgn * f.x, sgn * f.y};
  m.m[1][0] = conj(m.m[0][1]);
  m.m[2][0] = conj(m.m[0][2]);
  m.m[2][1] = conj(m.m[1][2]);
  return m;
}
// Products with a Hermitian matrix h (real diagonal): c = h b, c += b h
__device__ __forceinline__ Mat<double> hm(const Mat<double>& h, const Mat<double>& b) {
  Mat<double> c;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      Cx<double> v = h.m[i][i].re * b.m[i][j];
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k != i) v = cfma(h.m[i][k], b.m[k][j], v);
      c.m[i][j] = v;
    }
  return c;
}
__device__ __forceinline__ void hm_acc(Mat<double>& c, const Mat<double>& h, const Mat<double>& b) {  // c += h b
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      Cx<double> v = axpy(c.m[i][j], h.m[i][i].re, b.m[i][j]);
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k != i) v = cfma(h.m[i][k], b.m[k][j], v);
      c.m[i][j] = v;
    }
}
__device__ __forceinline__ void mh_acc(Mat<double>& c, const Mat<double>& b, const Mat<double>& h) {  // c += b h
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      Cx<double> v = axpy(c.m[i][j], h.m[j][j].re, b.m[i][j]);
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k != j) v = cfma(b.m[i][k], h.m[k][j], v);
      c.m[i][j] = v;
    }
}

// S_g = beta sum_{x, mu<nu} (1 - Re tr U_mu,nu(x) / 3).  For one link the
// plaquettes through it sum to Re tr(U_mu(x) A_mu(x)) with the staple sum
//   A_mu(x) = sum_{nu != mu} U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
//                          + U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu),
// so dS_g = -(beta/3) Re tr(dU A) and G = -(beta/3) A^dag.  A plaquette's
// share of the action is taken from the up staple of its mu < nu link.
__device__ __forceinline__ double plaquette_share(const Mat<double>& U, const Mat<double>& up) {
  double re = 0.0;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      re = fmar(U.m[r][c].re, up.m[c][r].re, re);
      re = fmar(-U.m[r][c].im, up.m[c][r].im, re);
    }
  return fmar(re, -1.0 / 3.0, 1.0);
}
// U_nu(y+mu) U_mu(y+nu)^dag U_nu(y)^dag as A = U_mu(y+nu)^dag U_nu(y)^dag, then L1 A
__device__ __forceinline__ Mat<double> up_staple(const double2* __restrict__ u18, int st, int mu, int nu, int par,
                                                 int cb, int cbm, int cbn) {
  const Mat<double> A = mm(adj(md_link(u18, st, mu, 1 - par, cbn)), adj(md_link(u18, st, nu, par, cb)));
  return mm(md_link(u18, st, nu, 1 - par, cbm), A);
}

// For one link U_mu(y) and each nu the two plaquettes of the plane close
// with the staples L1 L2 L3 (up: U_nu(y+mu) U_mu(y+nu)^dag U_nu(y)^dag, down:
// U_nu(y+mu-nu)^dag U_mu(y-nu)^dag U_nu(y-nu)).  With C0 .. C3 the plane's Xi
// (sign reversed for mu > nu) at y, y+mu and the two far corners after L1 and
// L2, the leaf derivatives of a plaquette sum to
//   L1 L2 L3 C0 + C1 L1 L2 L3 + L1 (C2 L2 + L2 C3) L3,
// up minus down; C0 and C1 are the same for both, so their products are
// taken once, of the difference of the staples.  GAUGE adds the Wilson gauge
// force from the staples' sum, as gauge_force_k does, and its action.
//
// 14 3x3 products per plane (6 of them with a Hermitian factor) and 42 gathered
// matrices per link.
//
// The weights go in with the factors (Xi with coef, the staples with
// i coef_g), so that one sum mt holds both forces: dS = Im tr(dU mt), hence
// G = i mt^dag.
//
// One work-item per link, the planes in the order nu = mu ^ q (at each step the
// four directions of a site pair up on two planes, whose Xi and links they
// then gather at about the same time).  Two wavefronts per SIMD; with a
// wavefront per (link, nu), summed in LDS as in the gauge force, the pass took
// 3.25 instead of 2.46 ms at 32^3x64 (with the gauge force).
template <bool GAUGE>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
force_clover_k(MdGeom m, const double2* __restrict__ u18, const double2* __restrict__ xi, double coef, double coef_g,
               const double2* gin, MdOut o, double* __restrict__ partial) {
  __shared__ MdLds<1> lds;
  int w, mu, par, n_live;
  MdSite s;
  md_link_site(m, w, mu, par, n_live, s);
  const int st = m.g.stride;
  const int um = md_fwd(m, s, mu), cbm = (s.i + um) >> 1;
  Mat<double> mt = mzero<double>();
  double act = 0.0;
#pragma unroll 1
  for (int q = 1; q < 4; ++q) {
    const int nu = mu ^ q;
    const int p = mu < nu ? plane_index(mu, nu) : plane_index(nu, mu);
    const double sc = mu < nu ? coef : -coef;
    const int un = md_fwd(m, s, nu), dn = md_bwd(m, s, nu);
    Mat<double> D;
    {
      const int n = (s.i + un) >> 1, mn = (s.i + um + un) >> 1;
      Mat<double> T, A;
      {
        const Mat<double> L2 = adj(md_link(u18, st, mu, 1 - par, n));
        T = hm(xi_at(xi, st, p, par, mn, sc), L2);
        mh_acc(T, L2, xi_at(xi, st, p, 1 - par, n, sc));
        const Mat<double> L3 = adj(md_link(u18, st, nu, par, s.cb));
        A = mm(L2, L3);
        T = mm(T, L3);
      }
      const Mat<double> L1 = md_link(u18, st, nu, 1 - par, cbm);
      mm_acc(mt, L1, T);
      D = mm(L1, A);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (GAUGE) {
      // U is read again for each plane: kept over the loop it would cost the registers of a matrix
      int own = s.cb;
      asm volatile("" : "+v"(own));
      const double share = plaquette_share(md_link(u18, st, mu, par, own), D);
      act += mu < nu ? share : 0.0;
      __builtin_amdgcn_sched_barrier(0);
    }
    {
      const int n = (s.i + dn) >> 1, mn = (s.i + um + dn) >> 1;
      Mat<double> T, A;
      {
        const Mat<double> L2 = adj(md_link(u18, st, mu, 1 - par, n));
        T = hm(xi_at(xi, st, p, par, mn, -sc), L2);
        mh_acc(T, L2, xi_at(xi, st, p, 1 - par, n, -sc));
        const Mat<double> L3 = md_link(u18, st, nu, 1 - par, n);
        A = mm(L2, L3);
        T = mm(T, L3);
      }
      const Mat<double> L1 = adj(md_link(u18, st, nu, par, mn));
      mm_acc(mt, L1, T);
      A = mm(L1, A);
      if constexpr (GAUGE) {
        const Mat<double> sum = madd(D, A);
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int c = 0; c < 3; ++c) mt.m[r][c] = axpy_i(mt.m[r][c], coef_g, sum.m[r][c]);
      }
      D = msub(D, A);
    }
    mh_acc(mt, D, xi_at(xi, st, p, par, s.cb, sc));
    hm_acc(mt, xi_at(xi, st, p, 1 - par, cbm, sc), D);
  }
  if constexpr (GAUGE) block_sum_store((int)threadIdx.x < n_live ? act : 0.0, partial, w);
  md_emit<1>(o, gin, lds, m.g, s, n_live, mu, par, u18, mt);
}

hipError_t launch_force_clover(const Geom& g, const double2* u18, const double2* xi, double coef, double coef_g,
                               const double2* gin, const MdOut& o, double* partial, hipStream_t s) {
  const dim3 grid(md_link_blocks(g)), block(64);
  if (coef_g != 0.0 && partial == nullptr) return hipErrorInvalidValue;
  if (coef_g != 0.0)
    hipLaunchKernelGGL(force_clover_k<true>, grid, block, 0, s, md_geom(g), u18, xi, coef, coef_g, gin, o, partial);
  else
    hipLaunchKernelGGL(force_clover_k<false>, grid, block, 0, s, md_geom(g), u18, xi, coef, 0.0, gin, o, partial);
  return hipGetLastError();
}

// ------------------------------------------------------------------ Wilson gauge action and force
// G (+)= coef A_mu(x)^dag, and (ACTION) per-workgroup partial sums of the
// action from the same staples.  A workgroup of three wavefronts takes 64
// links, each wavefront one nu: at 16^4, where there are few wavefronts, 67
// instead of 77 us per call with a wavefront per plane and both its links, and
// 158 with a work-item per link and separate action and output kernels; at
// 32^3x64 1.70, 1.66 and 3.68 ms (of the last, 1.75 in the staples alone, 0.73
// in the action and 1.23 in the output).
template <bool ACTION>
__global__ void __launch_bounds__(192) gauge_force_k(MdGeom m, const double2* __restrict__ u18, double coef,
                                                     const double2* gin, MdOut o, double* __restrict__ partial) {
  __shared__ MdLds<3> lds;
  int w, mu, par, n_live;
  MdSite s;
  md_link_site(m, w, mu, par, n_live, s);
  const int st = m.g.stride;
  const int nu = mu ^ (1 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  const int um = md_fwd(m, s, mu), un = md_fwd(m, s, nu), dn = md_bwd(m, s, nu), cbm = (s.i + um) >> 1;
  const int n = (s.i + un) >> 1, b = (s.i + dn) >> 1, mb = (s.i + um + dn) >> 1;
  Mat<double> a = up_staple(u18, st, mu, nu, par, s.cb, cbm, n);
  if constexpr (ACTION) {
    const double act = mu < nu ? plaquette_share(md_link(u18, st, mu, par, s.cb), a) : 0.0;
    block_sum_store((int)(threadIdx.x & 63) < n_live ? act : 0.0, partial, w);
  }
  const Mat<double> down = adj(mm(md_link(u18, st, mu, 1 - par, b), md_link(u18, st, nu, par, mb)));
  mm_acc(a, down, md_link(u18, st, nu, 1 - par, b));
  // coef a^dag = i (i coef a)^dag
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) a.m[r][c] = coef * ti(a.m[r][c]);
  md_emit<3>(o, gin, lds, m.g, s, n_live, mu, par, u18, a);
}

hipError_t launch_gauge_force(const Geom& g, const double2* u18, double coef, const double2* gin, const MdOut& o,
                              double* partial, hipStream_t s) {
  const dim3 grid(md_link_blocks(g)), block(192);
  if (partial != nullptr)
    hipLaunchKernelGGL(gauge_force_k<true>, grid, block, 0, s, md_geom(g), u18, coef, gin, o, partial);
  else
    hipLaunchKernelGGL(gauge_force_k<false>, grid, block, 0, s, md_geom(g), u18, coef, gin, o, partial);
  return hipGetLastError();
}

// The action alone, from the up staples alone: the partial sums of
// gauge_force_k, bit for bit (force_clover_k adds a link's planes before it
// sums over links).  One work-item per site, four partial sums per workgroup.
__global__ void __launch_bounds__(64) plaquette_k(MdGeom m, const double2* __restrict__ u18, double* partial) {
  const int w = xcd_block(blockIdx.x, gridDim.x), par = w & 1;
  const int j = ((w >> 1) << 6) + threadIdx.x;
  const bool live = j < m.g.Vh;
  const MdSite s = md_site(m, min(j, m.g.Vh - 1), par);
  const int st = m.g.stride;
#pragma unroll 1
  for (int mu = 0; mu < 4; ++mu) {
    const int cbm = (s.i + md_fwd(m, s, mu)) >> 1;
    double sum = 0.0;
#pragma unroll 1
    for (int q = 1; q < 4; ++q) {
      const int nu = mu ^ q;
      if (nu < mu) continue;
      const Mat<double> up = up_staple(u18, st, mu, nu, par, s.cb, cbm, (s.i + md_fwd(m, s, nu)) >> 1);
      const double act = plaquette_share(md_link(u18, st, mu, par, s.cb), up);
      sum += wave_sum(live ? act : 0.0);
    }
    if (threadIdx.x == 0) partial[((w >> 1) * 4 + mu) * 2 + par] = sum;
  }
}

hipError_t launch_plaquette(const Geom& g, const double2* u18, double* partial, hipStream_t s) {
  hipLaunchKernelGGL(plaquette_k, dim3(md_site_blocks(g)), dim3(64), 0, s, md_geom(g), u18, partial);
  return hipGetLastError();
}

// Per-block partial sums of a checkerboard array of doubles.
__global__ void __launch_bounds__(256) sum_cb_k(int n, const double* __restrict__ v, double* partial) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  block_sum_store(t < n ? v[t] : 0.0, partial, blockIdx.x);
}

hipError_t launch_sum_cb(const Geom& g, const double* v, double* partial, int block, hipStream_t s) {
  hipLaunchKernelGGL(sum_cb_k, dim3(blocks_for(g.Vh, block)), dim3(block), 0, s, g.Vh, v, partial);
  return hipGetLastError();
}

// ------------------------------------------------------------------ HMD updates
// f_j of exp(iQ) = f0 + f1 Q + f2 Q^2 in closed form (c1 > 0)
__device__ void expi_closed(double c0, double c1, Cx<double>& f0, Cx<double>& f1, Cx<double>& f2) {
  const bool neg = c0 < 0.0;
  const double c0a = fabs(c0);
  const double c0max = 2.0 * pow(c1 / 3.0, 1.5);
  double ratio = c0a / c0max;
  ratio = ratio > 1.0 ? 1.0 : ratio;
  const double theta = acos(ratio);
  const double u = sqrt(c1 / 3.0) * cos(theta / 3.0);
  const double w = sqrt(c1) * sin(theta / 3.0);
  const double u2 = u * u, w2 = w * w;
  const double xi0 = fabs(w) < 0.05 ? 1.0 - w2 / 6.0 * (1.0 - w2 / 20.0 * (1.0 - w2 / 42.0)) : sin(w) / w;
  const double cw = cos(w);
  const Cx<double> e2iu = {cos(2.0 * u), sin(2.0 * u)}, emiu = {cos(u), -sin(u)};
  Cx<double> h0 = (u2 - w2) * e2iu + emiu * Cx<double>{8.0 * u2 * cw, 2.0 * u * (3.0 * u2 + w2) * xi0};
  Cx<double> h1 = (2.0 * u) * e2iu - emiu * Cx<double>{2.0 * u * cw, -(3.0 * u2 - w2) * xi0};
  Cx<double> h2 = e2iu - emiu * Cx<double>{cw, 3.0 * u * xi0};
  const double den = 1.0 / (9.0 * u2 - w2);
  f0 = den * h0;
  f1 = den * h1;
  f2 = den * h2;
  if (neg) {  // f_j(-c0) = (-1)^j conj(f_j(c0))
    f0 = conj(f0);
    f1 = -conj(f1);
    f2 = conj(f2);
  }
}
// exp(i Q) = f0 + f1 Q + f2 Q^2 for Hermitian traceless Q, with f_j from
// c0 = det Q = tr(Q^3)/3 and c1 = tr(Q^2)/2 (Cayley-Hamilton: Q^3 = c1 Q + c0).
// For |Q| <= 1/2 (the eigenvalues are at most 2 sqrt(c1/3)) the power series
// to order 15, whose remainder is below 1e-18, by Horner's rule on the three
// coefficients: a step of the integrator is far inside, and the closed form's
// arc cosine, power and six sines and cosines were most of what a link's
// update computed.  Beyond, the closed form of Morningstar and Peardon (Phys.
// Rev. D 69 (2004) 054501).
__device__ Mat<double> expi_herm(const Mat<double>& q) {
  const Mat<double> q2 = mm(q, q);
  const double c1 = 0.5 * (q2.m[0][0].re + q2.m[1][1].re + q2.m[2][2].re);
  Mat<double> out;
  const Mat<double> q3 = mm(q2, q);
  const double c0 = (q3.m[0][0].re + q3.m[1][1].re + q3.m[2][2].re) / 3.0;
  Cx<double> f0, f1, f2;
  if (c1 <= 0.1875) {
    f0 = {1.0, 0.0};
    f1 = f2 = {0.0, 0.0};
#pragma unroll
    for (int k = 15; k >= 1; --k) {  // f <- 1 + (i Q / k) f
      const double w = 1.0 / k;
      const Cx<double> t0 = c0 * f2, t1 = axpy(f0, c1, f2);
      f2 = w * ti(f1);
      f1 = w * ti(t1);
      f0 = {1.0 - w * t0.im, w * t0.re};
    }
  } else {
    expi_closed(c0, c1, f0, f1, f2);
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      out.m[a][b] = f1 * q.m[a][b] + f2 * q2.m[a][b];
      if (a == b) out.m[a][b] = out.m[a][b] + f0;
    }
  return out;
}

// Back to SU(3): row 0 normalised, row 1 orthogonalised against it and
// normalised, row 2 = conj(row 0 x row 1).
__device__ __forceinline__ void reunitarize(Mat<double>& u) {
  double n0 = 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c) n0 += norm2(u.m[0][c]);
  n0 = 1.0 / sqrt(n0);
#pragma unroll
  for (int c = 0; c < 3; ++c) u.m[0][c] = n0 * u.m[0][c];
  Cx<double> d = {0.0, 0.0};
#pragma unroll
  for (int c = 0; c < 3; ++c) d = d + cmulc(u.m[0][c], u.m[1][c]);  // conj(a) b
  double n1 = 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    u.m[1][c] = u.m[1][c] - d * u.m[0][c];
    n1 += norm2(u.m[1][c]);
  }
  n1 = 1.0 / sqrt(n1);
#pragma unroll
  for (int c = 0; c < 3; ++c) u.m[1][c] = n1 * u.m[1][c];
  u.m[2][0] = conj(u.m[0][1] * u.m[1][2] - u.m[0][2] * u.m[1][1]);
  u.m[2][1] = conj(u.m[0][2] * u.m[1][0] - u.m[0][0] * u.m[1][2]);
  u.m[2][2] = conj(u.m[0][0] * u.m[1][1] - u.m[0][1] * u.m[1][0]);
}

// U <- E U with E = exp(i h P), P = sum_a P^a lambda^a / 2; reunitarisation; E
// once more (the end of a step and the start of the next move the links by the
// same momenta); the copies.  Bound by the bytes of U, P and the copies, so
// all of it is one pass: exponential, reunitarisation and copies as three
// passes took 0.66 + 0.40 + 0.55 ms at 32^3x64 and, twice in a pure-gauge step
// of 142 us at 16^4, 77 us (the step now 77 us in all).
__global__ void __launch_bounds__(256) move_links_k(Geom g, double2* __restrict__ u18, const double* __restrict__ p_user,
                                                    double h, int reunit, int twice, LinkCopies c) {
  __shared__ TileLds<4> lds;
  if (h != 0.0) tile_read<4>(lds, g, (const d2_a8*)p_user);
  const TileLink t = tile_link(g);
  if (!t.live) return;
  double2* const base = u18 + (size_t)((t.mu * 2 + t.par) * 9) * g.stride;
  Mat<double> U = load_mat(base, g.stride, t.cb);
  if (h != 0.0) {
    double P[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double2 d = lds.at(t, k);
      P[2 * k] = 0.5 * h * d.x;
      P[2 * k + 1] = 0.5 * h * d.y;
    }
    const double r3 = 0.57735026918962576451;  // 1 / sqrt(3)
    Mat<double> q;
    q.m[0][0] = {P[2] + P[7] * r3, 0.0};
    q.m[1][1] = {-P[2] + P[7] * r3, 0.0};
    q.m[2][2] = {-2.0 * P[7] * r3, 0.0};
    q.m[0][1] = {P[0], -P[1]};
    q.m[1][0] = {P[0], P[1]};
    q.m[0][2] = {P[3], -P[4]};
    q.m[2][0] = {P[3], P[4]};
    q.m[1][2] = {P[5], -P[6]};
    q.m[2][1] = {P[5], P[6]};
    const Mat<double> E = expi_herm(q);
    U = mm(E, U);
    if (reunit) reunitarize(U);
    if (twice) U = mm(E, U);
  } else if (reunit) {
    reunitarize(U);
  }
  double2 r[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) r[k] = make_double2(U.m[k / 3][k % 3].re, U.m[k / 3][k % 3].im);
  if (h != 0.0 || reunit) {
#pragma unroll
    for (int k = 0; k < 9; ++k) base[(size_t)k * g.stride + t.cb] = r[k];
  }
  store_copies(c, g.stride, t.mu * 2 + t.par, t.cb, r);
}

hipError_t launch_move_links(const Geom& g, double2* u18, const double* p_user, double h, bool reunit, bool twice,
                             const LinkCopies& c, hipStream_t s) {
  hipLaunchKernelGGL(move_links_k, dim3(tile_blocks(g)), dim3(256), 0, s, g, u18, p_user, h, reunit ? 1 : 0,
                     twice ? 1 : 0, c);
  return hipGetLastError();
}

}  // namespace qcd

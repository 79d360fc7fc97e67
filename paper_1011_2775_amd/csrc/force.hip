// Gauge-link gradient ("force") of a real loss through x = D(U)^-1 eta.
//
// With lambda = D^-dag g for the upstream gradient g of x, the loss changes by
// dL = -Re <lambda, dD x>.  Gradients follow PyTorch's convention for complex
// variables (dL = Re sum conj(G) dU).  Derivation from Eq.(1):
//
//  hop:    G_mu(y) = 1/2 ph sum_s [ lambda(y)_s chi_s^dag + phi_s lambda(y+mu)_s^dag ]
//          chi = (1 - gamma_mu) x(y+mu), phi = (1 + gamma_mu) x(y), ph the time
//          boundary phase of the link;
//  clover: with S_s(mu,nu) = csw (i/2) sigma_mu_nu on chirality s (mu < nu),
//          Xi(y)[i][j] = sum_s sum_{a,b} S_s[a][b] x(y)_{s,b,i} conj(lambda(y)_{s,a,j}),
//          Z = (Xi^dag - Xi)/8, the loss changes by Re sum_y tr(dQ_mu_nu(y) Z(y))
//          with Q the sum of the four plaquette leaves.  Every leaf of Q at y
//          is one elementary square of the plane read from its corner y, so
//          sum_y tr(Q(y) Z(y)) = sum_squares sum_corners tr(loop from corner c
//          times Z(c)).  For the square L1 L2 L3 L4 = U_a(z) U_b(z+a)
//          U_a(z+b)^dag U_b(z)^dag with corners c1..c4 = z, z+a, z+a+b, z+b,
//          the derivative with respect to factor k is
//          K_k = Z1 A B C + A Z2 B C + A B Z3 C + A B C Z0,
//          (A, B, C) = (L_k+1, L_k+2, L_k+3), Z1..Z3 at the corners before
//          them and Z0 at corner k; a plain link collects K^dag, an adjoint
//          link collects K.
//
// All arithmetic is FP64; fields use the canonical lexicographic layout.
#include "kernels.h"
#include "hop_core.h"
#include "su3.h"

namespace wcmg {

namespace {
constexpr int kT = 128;

__device__ __forceinline__ void load12(const double2* v, size_t site, cpx<double> o[12]) {
  const double2* p = v + site * 12;
#pragma unroll
  for (int k = 0; k < 12; ++k) o[k] = mk(p[k].x, p[k].y);
}

// out = (1 - gamma_mu) v (BACK = false) or (1 + gamma_mu) v (BACK = true)
template <int MU, bool BACK>
__device__ __forceinline__ void one_pm_gamma(const cpx<double> v[12], cpx<double> out[12]) {
  cpx<double> h[6];
  project<double, MU, BACK>(v, h);
#pragma unroll
  for (int k = 0; k < 12; ++k) out[k] = mk(0.0, 0.0);
  accumulate<double, MU, BACK>(out, h);
}

template <int MU>
__device__ __forceinline__ void hop_force_mu(const double2* x, const double2* lam, int nrhs, size_t V,
                                             size_t y, size_t yp, double ph, cpx<double> acc[9]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = mk(0.0, 0.0);
  for (int r = 0; r < nrhs; ++r) {
    const size_t off = (size_t)r * V;
    cpx<double> v[12], w[12], l[12];
    // lambda(y)_s chi_s^dag,  chi = (1 - gamma) x(y+mu)
    load12(x, off + yp, v);
    one_pm_gamma<MU, false>(v, w);
    load12(lam, off + y, l);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        cpx<double> t = mk(0.0, 0.0);
#pragma unroll
        for (int s = 0; s < 4; ++s) cfmac(t, w[s * 3 + b], l[s * 3 + a]);
        acc[a * 3 + b] = acc[a * 3 + b] + t;
      }
    // phi_s lambda(y+mu)_s^dag,  phi = (1 + gamma) x(y)
    load12(x, off + y, v);
    one_pm_gamma<MU, true>(v, w);
    load12(lam, off + yp, l);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        cpx<double> t = mk(0.0, 0.0);
#pragma unroll
        for (int s = 0; s < 4; ++s) cfmac(t, l[s * 3 + b], w[s * 3 + a]);
        acc[a * 3 + b] = acc[a * 3 + b] + t;
      }
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = (0.5 * ph) * acc[k];
}

template <int MU>
__device__ __forceinline__ void hop_force_store(double2* G, const double2* x, const double2* lam, int nrhs, size_t V,
                                                size_t y, size_t yp, double ph) {
  cpx<double> acc[9];
  hop_force_mu<MU>(x, lam, nrhs, V, y, yp, ph, acc);
  double2* o = G + (y * 4 + MU) * 9;
#pragma unroll
  for (int k = 0; k < 9; ++k) o[k] = make_double2(acc[k].r, acc[k].i);
}

// The hop part of all four links of a site by one thread, which reads the site's
// own spinors once.  Bound by the gather of four neighbours a pair of spinors.
// k_link_force<false>, a wavefront per direction, reads the site's spinors four
// times: three pairs at 16^3x32 190 us here and 234 us there, at 32^2x8^2 80 and
// 116 us.
__global__ void __launch_bounds__(kT) k_hop_force(double2* G, const double2* x, const double2* lam, int nrhs,
                                                  DGeom g) {
  const int y = blockIdx.x * blockDim.x + threadIdx.x, V = 2 * g.Vh;
  if (y >= V) return;
  int c[4], n[4];
  coords_of(g.L, y, c);
  // spatial hops carry the coefficient hs (1 on isotropic lattices), the last time slice its phase
  shift(g.L, c, 0, 1, n);
  hop_force_store<0>(G, x, lam, nrhs, V, y, lex_of(g.L, n), g.hs);
  shift(g.L, c, 1, 1, n);
  hop_force_store<1>(G, x, lam, nrhs, V, y, lex_of(g.L, n), g.hs);
  shift(g.L, c, 2, 1, n);
  hop_force_store<2>(G, x, lam, nrhs, V, y, lex_of(g.L, n), g.hs);
  shift(g.L, c, 3, 1, n);
  hop_force_store<3>(G, x, lam, nrhs, V, y, lex_of(g.L, n), c[3] == g.L[3] - 1 ? g.t_bc : 1.0);
}

// site of place t (parity p = t / Vh, checkerboard index t mod Vh): coordinates and lexicographic index
__device__ __forceinline__ int force_site(const DGeom& g, int t, int c[4]) {
  const int p = t >= g.Vh, i = t - p * g.Vh;
  cb_coords(g, i, p, c);
  return 2 * i + (c[0] & 1);
}

// Z = (Xi^dag - Xi) / 8 per site and plane mu < nu.  It is antihermitian: nine
// doubles, [plane] of (01), (02), (12), (im 00, im 11) as double2[parity][Vh],
// then im 22 as double[parity][Vh]
// (ONE: one pair, whose spinors are loaded once for the six planes)
template <bool ONE>
__global__ void __launch_bounds__(kT) k_clover_insertion(double* Z, const double2* x, const double2* lam,
                                                         int nrhs, CloverCoef cc, DGeom g) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x, V = 2 * g.Vh;
  if (t >= V) return;
  int c[4];
  const int y = force_site(g, t, c);
  cpx<double> v[12], l[12];
  if constexpr (ONE) {
    load12(x, y, v);
    load12(lam, y, l);
  }
  for (int pl = 0; pl < 6; ++pl) {
    cpx<double> xi[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) xi[k] = mk(0.0, 0.0);
    for (int r = 0; r < (ONE ? 1 : nrhs); ++r) {
      if constexpr (!ONE) {
        load12(x, (size_t)r * V + y, v);
        load12(lam, (size_t)r * V + y, l);
      }
#pragma unroll
      for (int chi = 0; chi < 2; ++chi)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const cpx<double> s = mk(cc.s[pl][chi][a * 2 + b][0], cc.s[pl][chi][a * 2 + b][1]);
            const int sa = 2 * chi + a, sb = 2 * chi + b;
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
              for (int j = 0; j < 3; ++j) {
                // s * x_{sb,i} * conj(lambda_{sa,j})
                cpx<double> u = mk(0.0, 0.0);
                cfmac(u, l[sa * 3 + j], v[sb * 3 + i]);
                cfma(xi[i * 3 + j], s, u);
              }
          }
    }
    double* zp = Z + (size_t)pl * 9 * V;
    double2* zo = reinterpret_cast<double2*>(zp);
    constexpr int kRow[3] = {0, 0, 1}, kCol[3] = {1, 2, 2};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const cpx<double> z = 0.125 * (cconj(xi[kCol[k] * 3 + kRow[k]]) - xi[kRow[k] * 3 + kCol[k]]);
      zo[(size_t)k * V + t] = make_double2(z.r, z.i);
    }
    zo[(size_t)3 * V + t] = make_double2(-0.25 * xi[0].i, -0.25 * xi[4].i);
    zp[(size_t)8 * V + t] = -0.25 * xi[8].i;
  }
}

__device__ __forceinline__ int plane_index(int a, int b) {  // a < b
  return a == 0 ? b - 1 : (a == 1 ? b + 1 : 5);
}

__device__ __forceinline__ C3 madd(const C3& a, const C3& b) {
  C3 r;
#pragma unroll
  for (int k = 0; k < 9; ++k) r.m[k] = a.m[k] + b.m[k];
  return r;
}

// One wavefront per direction mu of 64 sites, the four of a workgroup on the
// same sites: they share links and Z through the L1, mu and nu are scalar (a
// thread per link with mu in the low bits of its index had the lanes of a
// wavefront in different directions: every load four groups of sites, both
// branches of every square), the sites of a wavefront are neighbours in the
// checkerboard layout, and a link's two parts are written once.
//
// For link U_mu(x) and direction nu, with Z of the plane (antihermitian) and
// the path x -> x +- nu -> x +- nu + mu -> x + mu of links A, B, C (A and C
// adjoint where the path runs against them),
//   K = Z(x) A B C + A Z(x +- nu) B C + A B Z(x +- nu + mu) C + A B C Z(x + mu)
// is the derivative of the square on that side with the link taken out: the
// square above nu contributes -K and the one below +K for mu < nu (the reverse
// orientation, mu > nu, the negative), written as
//   A (Z B + B Z) C + Z(x) A B C + A B C Z(x + mu)
// with products formed in place: the sum over both sides kept apart (four more
// matrices alive) took 372 registers, one wavefront per SIMD and 316 us; loads
// held behind what stands before them (fewer registers still) 390 us; 256
// registers, two wavefronts, loads free within a square, 251 us.
// 48 products of 3x3 matrices a link (90 us of FP64 arithmetic at this size)
// and the gather of 18 links and 24 Z of 72 bytes through L1 and L2 bound it.
// 16^3x32, one pair of spinors: hop part 87 us and clover part 614 us as
// launches of their own, 251 us now; the insertion 63 us, 27 us now.
struct ForceLinks {
  const double2* gauge;
  const double* Z;
  DGeom g;
};
__device__ __forceinline__ C3 load_zc(const ForceLinks& f, int pl, const int c[4]) {
  const int p = (c[0] + c[1] + c[2] + c[3]) & 1;
  const size_t V = 2 * (size_t)f.g.Vh, t = (size_t)p * f.g.Vh + cb_index(f.g, c);
  const double* zp = f.Z + (size_t)pl * 9 * V;
  const double2* b = reinterpret_cast<const double2*>(zp) + t;
  const double2 z01 = b[0], z02 = b[V], z12 = b[2 * V], d = b[3 * V];
  const double d2 = zp[8 * V + t];
  C3 m;
  m.m[0] = mk(0.0, d.x);
  m.m[1] = mk(z01.x, z01.y);
  m.m[2] = mk(z02.x, z02.y);
  m.m[3] = mk(-z01.x, z01.y);
  m.m[4] = mk(0.0, d.y);
  m.m[5] = mk(z12.x, z12.y);
  m.m[6] = mk(-z02.x, z02.y);
  m.m[7] = mk(-z12.x, z12.y);
  m.m[8] = mk(0.0, d2);
  return m;
}

// acc += s A B, each row of the product from zero: terms added to acc one by one would be rounded
// at the size of the whole sum
__device__ __forceinline__ void mul_add(C3& acc, double s, const C3& A, const C3& B) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    cpx<double> t[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) t[j] = mk(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int j = 0; j < 3; ++j) cfma(t[j], A.m[i * 3 + k], B.m[k * 3 + j]);
#pragma unroll
    for (int j = 0; j < 3; ++j)
      acc.m[i * 3 + j] = mk(fma(s, t[j].r, acc.m[i * 3 + j].r), fma(s, t[j].i, acc.m[i * 3 + j].i));
  }
}
// B <- A B, column by column; B <- B A, row by row
__device__ __forceinline__ void left_mul(const C3& A, C3& B) {
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    cpx<double> t[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      t[i] = mk(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < 3; ++k) cfma(t[i], A.m[i * 3 + k], B.m[k * 3 + j]);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) B.m[i * 3 + j] = t[i];
  }
}
__device__ __forceinline__ void right_mul(C3& B, const C3& A) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    cpx<double> t[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      t[j] = mk(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < 3; ++k) cfma(t[j], B.m[i * 3 + k], A.m[k * 3 + j]);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) B.m[i * 3 + j] = t[j];
  }
}

template <bool up>
__device__ __forceinline__ void clover_force_side(const ForceLinks& f, const int x[4], const int xm[4], int mu, int nu,
                                                  C3& acc) {
  const int pl = mu < nu ? plane_index(mu, nu) : plane_index(nu, mu);
  const double sgn = (mu < nu) != up ? 1.0 : -1.0;
  int z[4], zm[4];
  shift(f.g.L, x, nu, up ? 1 : -1, z);
  shift(f.g.L, xm, nu, up ? 1 : -1, zm);
  C3 B = load_u(f.gauge, f.g, z, mu), M;
#pragma unroll
  for (int k = 0; k < 9; ++k) M.m[k] = mk(0.0, 0.0);
  mul_add(M, 1.0, load_zc(f, pl, z), B);
  mul_add(M, 1.0, B, load_zc(f, pl, zm));
  {
    const C3 A = up ? load_u(f.gauge, f.g, x, nu) : dagm(load_u(f.gauge, f.g, z, nu));
    left_mul(A, M);
    left_mul(A, B);
  }
  {
    const C3 C = up ? dagm(load_u(f.gauge, f.g, xm, nu)) : load_u(f.gauge, f.g, zm, nu);
    mul_add(acc, sgn, M, C);
    right_mul(B, C);
  }
  mul_add(acc, sgn, load_zc(f, pl, x), B);
  mul_add(acc, sgn, B, load_zc(f, pl, xm));
}

template <bool CLOVER>
__global__ void __launch_bounds__(256, 2) k_link_force(double2* G, const double2* x, const double2* lam, int nrhs,
                                                    ForceLinks f) {
  const int V = 2 * f.g.Vh, nblocks = (V + 63) / 64, b = xcd_block(nblocks);
  const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = b * 64 + (threadIdx.x & 63);
  if (b >= nblocks || t >= V) return;
  int c[4], cm[4];
  const int y = force_site(f.g, t, c);
  shift(f.g.L, c, mu, 1, cm);
  const size_t yp = lex_of(f.g.L, cm);
  // spatial hops carry the coefficient hs (1 on isotropic lattices), the last time slice its phase
  const double ph = mu < 3 ? f.g.hs : (c[3] == f.g.L[3] - 1 ? f.g.t_bc : 1.0);
  C3 acc, cl;
  if constexpr (CLOVER) {
    // first, from zero: added to the hop part term by term it would be rounded at the sum's size
#pragma unroll
    for (int k = 0; k < 9; ++k) cl.m[k] = mk(0.0, 0.0);
#pragma unroll 1
    for (int k = 1; k < 4; ++k) {
      const int nu = (mu + k) & 3;
      clover_force_side<true>(f, c, cm, mu, nu, cl);
      clover_force_side<false>(f, c, cm, mu, nu, cl);
    }
  }
  if (mu == 0) hop_force_mu<0>(x, lam, nrhs, V, y, yp, ph, acc.m);
  else if (mu == 1) hop_force_mu<1>(x, lam, nrhs, V, y, yp, ph, acc.m);
  else if (mu == 2) hop_force_mu<2>(x, lam, nrhs, V, y, yp, ph, acc.m);
  else hop_force_mu<3>(x, lam, nrhs, V, y, yp, ph, acc.m);
  if constexpr (CLOVER) acc = madd(acc, cl);
  double2* o = G + ((size_t)y * 4 + mu) * 9;
#pragma unroll
  for (int k = 0; k < 9; ++k) o[k] = make_double2(acc.m[k].r, acc.m[k].i);
}

// Sites from which the hop part alone is done by a thread a site: a wavefront for each of the 256
// compute units.  Below, a wavefront per direction finds idle units (three pairs at 12288 sites 30.5
// against 31.7 us, twelve 112 against 134); above, its workgroups come in a second round (three pairs
// at 16800 sites 46 against 39 us).
constexpr int kSiteThreads = 64 * 256;
}  // namespace

void force_compute(void* G, const void* x, const void* lam, int nrhs, const void* gauge64, const Geom& g,
                   const CloverCoef* cc, void* zbuf, hipStream_t st) {
  ForceLinks f{reinterpret_cast<const double2*>(gauge64), reinterpret_cast<const double*>(zbuf), dgeom(g)};
  const double2* xs = reinterpret_cast<const double2*>(x);
  const double2* ls = reinterpret_cast<const double2*>(lam);
  const dim3 gz((g.V + kT - 1) / kT);
  if (!cc && g.V >= kSiteThreads) {
    hipLaunchKernelGGL(k_hop_force, gz, dim3(kT), 0, st, reinterpret_cast<double2*>(G), xs, ls, nrhs, f.g);
    HIPCHK(hipGetLastError());
    return;
  }
  if (cc) {
    if (nrhs == 1)
      hipLaunchKernelGGL(k_clover_insertion<true>, gz, dim3(kT), 0, st, reinterpret_cast<double*>(zbuf), xs, ls, nrhs,
                         *cc, f.g);
    else
      hipLaunchKernelGGL(k_clover_insertion<false>, gz, dim3(kT), 0, st, reinterpret_cast<double*>(zbuf), xs, ls,
                         nrhs, *cc, f.g);
    HIPCHK(hipGetLastError());
  }
  const dim3 grid(xcd_grid((g.V + 63) / 64));
  if (cc)
    hipLaunchKernelGGL(k_link_force<true>, grid, dim3(256), 0, st, reinterpret_cast<double2*>(G), xs, ls, nrhs, f);
  else
    hipLaunchKernelGGL(k_link_force<false>, grid, dim3(256), 0, st, reinterpret_cast<double2*>(G), xs, ls, nrhs, f);
  HIPCHK(hipGetLastError());
}

}  // namespace wcmg

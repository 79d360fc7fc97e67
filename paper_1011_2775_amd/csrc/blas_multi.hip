// Several-vector kernels of the Krylov solvers: the multi-dot, the GCR step
// and the solution update, over one right-hand side or a lockstep batch
// (grid row blockIdx.y is the right-hand side, vectors vs elements apart).
//
// All three stream k + 2 vectors once and do a few flops an element, so they
// are bound by memory, and what they need is enough loads in flight: each
// thread loads 16 bytes of eight vectors (padding slots read y again) before
// the first of them is used, where a loop with a test per vector waits for
// every load in turn.  Setup on 16^3x32 (FP32, 1.57 M complex, GCR(30), mean
// over a cycle): multi-dot 77 -> 47 us, step 73 -> 44 us a step, and in pairs
// of steps 49 and 46 us a pair; outer GCR (FP64, 0.79 M complex, mean over 17
// steps) 52 -> 32 us, 38 -> 29 us.
//
// Sums accumulate in double in a fixed order: per thread, per wavefront, per
// block, then over the blocks by the last one to arrive, so results are
// bitwise reproducible.
#include "blas_common.h"

namespace wcmg {

namespace {

using namespace blas_detail;

constexpr int kVecs = 72;     // vectors per launch (GCR slots, y and r fit)
constexpr int kGroup = 8;     // vectors whose loads are in flight together
constexpr int kDotChunks = 256;

struct VecList {
  const void* v[kVecs];
};
struct HostCoefs {
  double c[2 * kVecs];
};

// W complex elements in one load
template <typename T, int W>
struct Pack;
template <>
struct Pack<double, 1> {
  using V = double2;
  __device__ __forceinline__ static cpx<double> get(const V& v, int) { return mk(v.x, v.y); }
  __device__ __forceinline__ static void set(V& v, int, cpx<double> c) { v = make_double2(c.r, c.i); }
};
template <>
struct Pack<float, 1> {
  using V = float2;
  __device__ __forceinline__ static cpx<double> get(const V& v, int) { return mk((double)v.x, (double)v.y); }
  __device__ __forceinline__ static void set(V& v, int, cpx<double> c) { v = make_float2((float)c.r, (float)c.i); }
};
template <>
struct Pack<float, 2> {
  using V = float4;
  __device__ __forceinline__ static cpx<double> get(const V& v, int w) {
    return w ? mk((double)v.z, (double)v.w) : mk((double)v.x, (double)v.y);
  }
  __device__ __forceinline__ static void set(V& v, int w, cpx<double> c) {
    if (w) {
      v.z = (float)c.r;
      v.w = (float)c.i;
    } else {
      v.x = (float)c.r;
      v.y = (float)c.i;
    }
  }
};

// res[2j..2j+1] = <v_j, y>; NY = 3: res[6j..6j+5] = <v_j, y>, <v_j, y2>, <v_j, y3>.
// Workgroups of one chunk of elements and the ng groups of kGroup vectors are numbered so that they run together on one
// XCD (y is then read once from memory and found in that XCD's L2).
template <typename T, int W, int NY = 1>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, NY == 3 ? 2 : 8))) k_multi_cdot(VecList m, int k, int ng, int nc, const void* y,
                                                         const void* y2, const void* y3, size_t vs, size_t n, RedB o) {
  using P = Pack<T, W>;
  using V = typename P::V;
  constexpr int NV = 2 * NY;
  const int t = blockIdx.x >> 3, g = t % ng, chunk = (t / ng) * 8 + (blockIdx.x & 7);
  const int j0 = g * kGroup, kb = min(kGroup, k - j0);
  const size_t ro = (size_t)blockIdx.y * vs * sizeof(typename C2<T>::V), nv = n / W;
  const void* ys[3] = {y, y2, y3};
  const V* yp[NY];
#pragma unroll
  for (int c = 0; c < NY; ++c) yp[c] = reinterpret_cast<const V*>(reinterpret_cast<const char*>(ys[c]) + ro);
  const V* vp[kGroup];
#pragma unroll
  for (int j = 0; j < kGroup; ++j)
    vp[j] = j < kb ? reinterpret_cast<const V*>(reinterpret_cast<const char*>(m.v[j0 + j]) + ro) : yp[0];
  double s[NV * kGroup];
#pragma unroll
  for (int j = 0; j < NV * kGroup; ++j) s[j] = 0.0;
  for (size_t i = (size_t)chunk * kThreads + threadIdx.x; i < nv; i += (size_t)nc * kThreads) {
    V yv[NY], q[kGroup];
#pragma unroll
    for (int c = 0; c < NY; ++c) yv[c] = yp[c][i];
#pragma unroll
    for (int j = 0; j < kGroup; ++j) q[j] = vp[j][i];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      cpx<double> b[NY];
#pragma unroll
      for (int c = 0; c < NY; ++c) b[c] = P::get(yv[c], w);
#pragma unroll
      for (int j = 0; j < kGroup; ++j) {
        const cpx<double> a = P::get(q[j], w);
#pragma unroll
        for (int c = 0; c < NY; ++c) {
          double* d = s + NV * j + 2 * c;
          d[0] = fma(a.r, b[c].r, fma(a.i, b[c].i, d[0]));
          d[1] = fma(a.r, b[c].i, fma(-a.i, b[c].r, d[1]));
        }
      }
    }
  }
  const int row = blockIdx.y * ng + g;
  block_reduce_row<NV * kGroup>(s, o.part + (size_t)row * nc * (NV * kGroup), o.counter + row * kCounterRow, nc,
                                chunk, o.res + (size_t)blockIdx.y * o.rs + NV * j0, nullptr, NV * kb);
}

// acc -= sum_j c_j v_j (SUB) or += at pack index i; c padded with zeros to a multiple of kGroup
template <typename T, int W, bool SUB>
__device__ __forceinline__ void combine(const VecList& m, int k, size_t ro, const void* pad, size_t i,
                                        const double2* c, cpx<double> (&acc)[W]) {
  using P = Pack<T, W>;
  using V = typename P::V;
  for (int j0 = 0; j0 < k; j0 += kGroup) {
    V q[kGroup];
#pragma unroll
    for (int j = 0; j < kGroup; ++j)
      q[j] = reinterpret_cast<const V*>(reinterpret_cast<const char*>(j0 + j < k ? m.v[j0 + j] : pad) + ro)[i];
#pragma unroll
    for (int j = 0; j < kGroup; ++j) {
      const double2 cj = c[j0 + j];
      const double cr = SUB ? -cj.x : cj.x, ci = SUB ? -cj.y : cj.y;
#pragma unroll
      for (int w = 0; w < W; ++w) cfma(acc[w], mk(cr, ci), P::get(q[j], w));
    }
  }
}

__device__ __forceinline__ cpx<double> alpha_of(const double* qa) {
  const double d = qa[0];
  return d > 0.0 ? mk(qa[1] / d, qa[2] / d) : mk(0.0, 0.0);
}

// One GCR step after the multi-dot: beta[2j] = <q_j, y> for the k basis slots,
// beta[2k] = <y, y>, beta[2k+2] = <r, y>.  y -= sum_j c_j q_j with
// c_j = <q_j, y> / ||q_j||^2;
//   ||y_orth||^2 = <y, y> - sum_j |<q_j, y>|^2 / ||q_j||^2   (in order of j),
//   <y_orth, r>  = <y, r>                                    (r is orthogonal to every q_j);
// rout = rin - alpha y_orth with alpha = <y_orth, r> / ||y_orth||^2, ||rout||^2
// into o, {||y_orth||^2, <y_orth, r>} to qa[4k ..] and the c_j to cj.  Elements
// are visited from the end: what the multi-dot read last is still in the
// Infinity Cache when the basis does not fit there.
template <typename T, int W>
__global__ void __launch_bounds__(kThreads) k_gcr_step(VecList m, int k, void* y, const void* rin, void* rout,
                                                       size_t vs, size_t n, const double* beta, size_t bs, double* qa,
                                                       size_t qs, double* cj, size_t cjs, RedB o) {
  using P = Pack<T, W>;
  using V = typename P::V;
  __shared__ double2 c[kVecs + kGroup];
  __shared__ double term[kVecs];
  const double* be = beta + (size_t)blockIdx.y * bs;
  double* q4 = qa + (size_t)blockIdx.y * qs;
  for (int j = threadIdx.x; j < k + kGroup; j += kThreads) {
    const double d = j < k ? q4[4 * j] : 0.0;
    double2 v = make_double2(0.0, 0.0);
    double tj = 0.0;
    if (d > 0.0) {
      const double br = be[2 * j], bi = be[2 * j + 1];
      v = make_double2(br / d, bi / d);
      tj = (br * br + bi * bi) / d;
    }
    c[j] = v;
    if (j < k) term[j] = tj;
  }
  __syncthreads();
  double qq = be[2 * k];
  for (int j = 0; j < k; ++j) qq -= term[j];
  const cpx<double> qr = mk(be[2 * k + 2], -be[2 * k + 3]);
  const cpx<double> alpha = qq > 0.0 ? mk(qr.r / qq, qr.i / qq) : mk(0.0, 0.0);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      q4[4 * k] = qq;
      q4[4 * k + 1] = qr.r;
      q4[4 * k + 2] = qr.i;
    }
    double* cr = cj + (size_t)blockIdx.y * cjs;
    for (int j = threadIdx.x; j < k; j += kThreads) {
      cr[2 * j] = c[j].x;
      cr[2 * j + 1] = c[j].y;
    }
  }
  const size_t ro = (size_t)blockIdx.y * vs * sizeof(typename C2<T>::V), nv = n / W;
  V* yp = reinterpret_cast<V*>(reinterpret_cast<char*>(y) + ro);
  const V* ip = reinterpret_cast<const V*>(reinterpret_cast<const char*>(rin) + ro);
  V* op = reinterpret_cast<V*>(reinterpret_cast<char*>(rout) + ro);
  double s[1] = {0.0};
  for (size_t l = (size_t)blockIdx.x * kThreads + threadIdx.x; l < nv; l += (size_t)gridDim.x * kThreads) {
    const size_t i = nv - 1 - l;
    const V yv = yp[i];
    V rv = ip[i];
    cpx<double> a[W];
#pragma unroll
    for (int w = 0; w < W; ++w) a[w] = P::get(yv, w);
    combine<T, W, true>(m, k, ro, y, i, c, a);
    V ys;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      P::set(ys, w, a[w]);
      const cpx<double> as = P::get(ys, w);  // as stored
      const cpx<double> b = P::get(rv, w) - alpha * as;
      P::set(rv, w, b);
      const cpx<double> bv = P::get(rv, w);
      s[0] += bv.r * bv.r + bv.i * bv.i;
    }
    yp[i] = ys;
    op[i] = rv;
  }
  block_reduce_row<1>(s, o.part + (size_t)blockIdx.y * gridDim.x, o.counter + blockIdx.y * kCounterRow, gridDim.x,
                      blockIdx.x, o.res + (size_t)blockIdx.y * o.rs, nullptr, 1);
}

// Two GCR steps after one multi-dot with a pair: y1 = A z_k (which is the raw
// direction z_k+1 and stays), y2 = A y1, and beta[6j..] = {<v_j, y1>, <v_j, y2>,
// <v_j, r>} of v = {q_0 .. q_k-1, y1, y2}.  q_k = y1 - sum_j b1_j q_j,
// q_k+1 = y2 - sum_j b2_j q_j - g q_k, rout = rin - alpha1 q_k - alpha2 q_k+1;
// with q_k orthogonal to the q_j
//   <q_k, y2> = <y1, y2> - sum_j conj(b1_j) <q_j, y2>,
//   <q_k, r> = <y1, r> - sum_j conj(b1_j) <q_j, r>,
//   <q_k+1, r> = <y2, r> - sum_j conj(b2_j) <q_j, r> - conj(g) <q_k, r>.
// r is orthogonal to the q_j only as far as it has not come down to rounding.
// Taken for granted there, every further pair multiplied it: GCR(64) on a
// spectrum of radius 0.5 about 1 ended at 2e-4 (FP32) and 2e-7 (FP64) of the
// start instead of 8e-8 and 3e-15.
// The span of {r, A r} is that of two steps (r after a step is r - alpha A r),
// so a pair costs the basis two reads instead of four.  A y2 of whose square no
// more than `lost` is outside the basis adds no direction: FP64 1e-14, a
// hundred roundings of the difference that says so (1e-10 dropped directions
// that eigenvalues in narrow clusters need: residuals of 2.3e-6 where 1.6e-6
// was to be had); FP32 1e-10, above which a higher line did the same although
// vectors stored in FP32 are orthogonal to 1e-7 only.
template <typename T, int W>
__global__ void __launch_bounds__(kThreads) k_gcr_step_pair(VecList m, int k, const void* y1, void* q1, void* y2,
                                                            const void* rin, void* rout, size_t n, const double* be,
                                                            double* q4, double* cj1, double* cj2) {
  using P = Pack<T, W>;
  using V = typename P::V;
  __shared__ double2 c1[kVecs + kGroup], c2[kVecs + kGroup];
  // terms of the sums over the basis: ||q_k||^2, ||q_k+1||^2, <q_k, y2>, <q_k, r>, <q_k+1, r>
  constexpr int kSums = 8;
  __shared__ double term[kSums][kVecs + 1], sum[kSums];
  for (int j = threadIdx.x; j < k + kGroup; j += kThreads) {
    const double d = j < k ? q4[4 * j] : 0.0;
    double2 u = make_double2(0.0, 0.0), v = u;
    double t[kSums];
#pragma unroll
    for (int i = 0; i < kSums; ++i) t[i] = 0.0;
    if (d > 0.0) {
      const double* e = be + 6 * j;
      u = make_double2(e[0] / d, e[1] / d);
      v = make_double2(e[2] / d, e[3] / d);
      t[0] = (e[0] * e[0] + e[1] * e[1]) / d;
      t[1] = (e[2] * e[2] + e[3] * e[3]) / d;
      t[2] = u.x * e[2] + u.y * e[3];
      t[3] = u.x * e[3] - u.y * e[2];
      t[4] = u.x * e[4] + u.y * e[5];
      t[5] = u.x * e[5] - u.y * e[4];
      t[6] = v.x * e[4] + v.y * e[5];
      t[7] = v.x * e[5] - v.y * e[4];
    }
    c1[j] = u;
    c2[j] = v;
    if (j < k)
#pragma unroll
      for (int i = 0; i < kSums; ++i) term[i][j] = t[i];
  }
  __syncthreads();
  if (threadIdx.x < kSums) {
    double t = 0.0;
    for (int j = 0; j < k; ++j) t += term[threadIdx.x][j];
    sum[threadIdx.x] = t;
  }
  __syncthreads();
  const double* e1 = be + 6 * k;  // <y1, y1>, <y1, y2>, <y1, r>
  const double* e2 = e1 + 6;      // <y2, y1>, <y2, y2>, <y2, r>
  double qq1 = e1[0] - sum[0], qq2 = e2[2] - sum[1];
  cpx<double> g = mk(e1[2] - sum[2], e1[3] - sum[3]);
  const cpx<double> r1 = mk(e1[4] - sum[4], e1[5] - sum[5]);
  cpx<double> alpha1 = mk(0.0, 0.0), alpha2 = alpha1;
  if (qq1 > 0.0) {
    alpha1 = mk(r1.r / qq1, r1.i / qq1);
    qq2 -= (g.r * g.r + g.i * g.i) / qq1;
    g = mk(g.r / qq1, g.i / qq1);
  } else {
    g = mk(0.0, 0.0);
  }
  const cpx<double> r2 = mk(e2[4] - sum[6] - (g.r * r1.r + g.i * r1.i), e2[5] - sum[7] - (g.r * r1.i - g.i * r1.r));
  constexpr double lost = sizeof(T) == 8 ? 1e-14 : 1e-10;
  if (!(qq2 > lost * e2[2])) qq2 = 0.0;
  if (qq2 > 0.0) alpha2 = mk(r2.r / qq2, r2.i / qq2);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      q4[4 * k] = qq1;
      q4[4 * k + 1] = r1.r;
      q4[4 * k + 2] = r1.i;
      q4[4 * k + 4] = qq2;
      q4[4 * k + 5] = r2.r;
      q4[4 * k + 6] = r2.i;
      cj2[2 * k] = g.r;
      cj2[2 * k + 1] = g.i;
    }
    for (int j = threadIdx.x; j < k; j += kThreads) {
      cj1[2 * j] = c1[j].x;
      cj1[2 * j + 1] = c1[j].y;
      cj2[2 * j] = c2[j].x;
      cj2[2 * j + 1] = c2[j].y;
    }
  }
  const size_t nv = n / W;
  const V* y1p = reinterpret_cast<const V*>(y1);
  V* q1p = reinterpret_cast<V*>(q1);
  V* y2p = reinterpret_cast<V*>(y2);
  const V* ip = reinterpret_cast<const V*>(rin);
  V* op = reinterpret_cast<V*>(rout);
  for (size_t l = (size_t)blockIdx.x * kThreads + threadIdx.x; l < nv; l += (size_t)gridDim.x * kThreads) {
    const size_t i = nv - 1 - l;
    V v1 = y1p[i], v2 = y2p[i], rv = ip[i];
    cpx<double> a1[W], a2[W];
#pragma unroll
    for (int w = 0; w < W; ++w) {
      a1[w] = P::get(v1, w);
      a2[w] = P::get(v2, w);
    }
    for (int j0 = 0; j0 < k; j0 += kGroup) {
      V q[kGroup];
#pragma unroll
      for (int j = 0; j < kGroup; ++j) q[j] = reinterpret_cast<const V*>(j0 + j < k ? m.v[j0 + j] : y1)[i];
#pragma unroll
      for (int j = 0; j < kGroup; ++j) {
        const double2 u = c1[j0 + j], v = c2[j0 + j];
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const cpx<double> qv = P::get(q[j], w);
          cfma(a1[w], mk(-u.x, -u.y), qv);
          cfma(a2[w], mk(-v.x, -v.y), qv);
        }
      }
    }
#pragma unroll
    for (int w = 0; w < W; ++w) {
      P::set(v1, w, a1[w]);
      const cpx<double> s1 = P::get(v1, w);  // as stored
      P::set(v2, w, a2[w] - g * s1);
      P::set(rv, w, P::get(rv, w) - alpha1 * s1 - alpha2 * P::get(v2, w));
    }
    q1p[i] = v1;
    y2p[i] = v2;
    op[i] = rv;
  }
}

// x += sum_j c_j v_j, c from the device (row r at coef + r cs) or the launch's arguments
template <typename T, int W, bool DEV>
__global__ void __launch_bounds__(kThreads) k_multi_axpy(VecList m, HostCoefs h, int k, void* x, size_t vs, size_t n,
                                                         const double* coef, size_t cs) {
  using P = Pack<T, W>;
  using V = typename P::V;
  __shared__ double2 c[kVecs + kGroup];
  for (int j = threadIdx.x; j < k + kGroup; j += kThreads) {
    double2 v = make_double2(0.0, 0.0);
    if (j < k) {
      if constexpr (DEV) {
        const double* cf = coef + (size_t)blockIdx.y * cs;
        v = make_double2(cf[2 * j], cf[2 * j + 1]);
      } else {
        v = make_double2(h.c[2 * j], h.c[2 * j + 1]);
      }
    }
    c[j] = v;
  }
  __syncthreads();
  const size_t ro = (size_t)blockIdx.y * vs * sizeof(typename C2<T>::V), nv = n / W;
  V* xp = reinterpret_cast<V*>(reinterpret_cast<char*>(x) + ro);
  for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < nv; i += (size_t)gridDim.x * kThreads) {
    V xv = xp[i];
    cpx<double> a[W];
#pragma unroll
    for (int w = 0; w < W; ++w) a[w] = P::get(xv, w);
    combine<T, W, false>(m, k, ro, x, i, c, a);
#pragma unroll
    for (int w = 0; w < W; ++w) P::set(xv, w, a[w]);
    xp[i] = xv;
  }
}

// Coefficients of the solution update of a GCR cycle whose directions are kept
// as the raw preconditioned vectors z_j: with z~_j = z_j - sum_{i<j} c_ij z~_i
// (c_ij in cmat[j][i], complex) and x += sum_j alpha_j z~_j, x += sum_j y_j z_j
// where y solves (I + C) y = alpha by back substitution (alpha_j = 0 for the
// nf fixed slots, whose vectors are not orthogonalised).  One workgroup a
// right-hand side; lane i of the first wavefront keeps y_i, the triangle is
// staged in LDS (one thread reading it entry by entry took 67 us for 30 slots).
constexpr int kMaxSlots = 64;
__global__ void __launch_bounds__(kThreads) k_gcr_coef_solve(const double* qa, size_t qs, const double* cmat,
                                                             size_t cms, int ldc, double* y, size_t ys, int nf,
                                                             int kt) {
  __shared__ double2 c[kMaxSlots * (kMaxSlots - 1) / 2];
  const double* q4 = qa + (size_t)blockIdx.x * qs;
  const double* cm = cmat + (size_t)blockIdx.x * cms;
  for (int e = threadIdx.x; e < kt * kt; e += kThreads) {
    const int j = e / kt, i = e - j * kt;
    if (i < j && j >= nf) c[j * (j - 1) / 2 + i] = make_double2(cm[2 * ((size_t)j * ldc + i)], cm[2 * ((size_t)j * ldc + i) + 1]);
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const int i = threadIdx.x;
  cpx<double> s = (i < nf || i >= kt) ? mk(0.0, 0.0) : alpha_of(q4 + 4 * i);
  for (int j = kt - 1; j >= nf; --j) {
    const cpx<double> yj = mk(__shfl(s.r, j), __shfl(s.i, j));
    if (i < j) {
      const double2 v = c[j * (j - 1) / 2 + i];
      s = s - mk(v.x, v.y) * yj;
    }
  }
  if (i < kt) {
    double* o = y + (size_t)blockIdx.x * ys;
    o[2 * i] = s.r;
    o[2 * i + 1] = s.i;
  }
}

// two FP32 elements a load where lengths, strides and addresses allow it
bool wide_ok(const void* const* v, int k, const void* a, const void* b, const void* c, size_t vs, size_t n, int nrhs) {
  if (n % 2 || (nrhs > 1 && vs % 2)) return false;
  uintptr_t bits = (uintptr_t)a | (uintptr_t)b | (uintptr_t)c;
  for (int j = 0; j < k; ++j) bits |= (uintptr_t)v[j];
  return bits % 16 == 0;
}

VecList vec_list(const void* const* v, int k) {
  if (k > kVecs) fail(WCMG_EINVAL, "too many vectors for one launch");
  VecList m{};
  for (int j = 0; j < k; ++j) m.v[j] = v[j];
  return m;
}

void check_rows(int nrhs) {
  if (nrhs < 1 || nrhs > kMaxBatch) fail(WCMG_EINVAL, "batch size out of range");
}

size_t packs(int prec, bool wide, size_t n) { return prec == WCMG_F32 && wide ? n / 2 : n; }

// workgroups along the elements: enough to fill the chip (about `most` over
// the batch), every thread with at least one element
unsigned rows_grid(size_t nv, int nrhs, size_t most) {
  const size_t b = std::min((nv + kThreads - 1) / kThreads, std::max<size_t>(most / nrhs, 1));
  return (unsigned)std::max<size_t>(b, 1);
}

}  // namespace

#define DISPATCH_W(prec, wide, KERNEL, grid, ...)                                                \
  do {                                                                                           \
    if ((prec) == WCMG_F64)                                                                      \
      hipLaunchKernelGGL((KERNEL<double, 1>), grid, dim3(kThreads), 0, st, __VA_ARGS__);         \
    else if (wide)                                                                               \
      hipLaunchKernelGGL((KERNEL<float, 2>), grid, dim3(kThreads), 0, st, __VA_ARGS__);          \
    else                                                                                         \
      hipLaunchKernelGGL((KERNEL<float, 1>), grid, dim3(kThreads), 0, st, __VA_ARGS__);          \
    HIPCHK(hipGetLastError());                                                                   \
  } while (0)

void blas_multi_cdot_b(int prec, const void* const* v, int k, const void* y, size_t vs, size_t n, int nrhs,
                       const RedB& o, hipStream_t st) {
  check_rows(nrhs);
  for (int j0 = 0; j0 < k; j0 += kVecs) {
    const int kk = std::min(kVecs, k - j0), ng = (kk + kGroup - 1) / kGroup;
    const VecList m = vec_list(v + j0, kk);
    const bool wide = wide_ok(v + j0, kk, y, nullptr, nullptr, vs, n, nrhs);
    const size_t nv = packs(prec, wide, n);
    // chunks in multiples of eight (one per XCD); the finish adds nc partials
    // per value, so not more of them than keep the chip busy
    size_t nc = std::min<size_t>((nv + kThreads - 1) / kThreads, kDotChunks);
    nc = std::min<size_t>(nc, std::max<size_t>(4096 / ((size_t)ng * nrhs), 8));
    nc = (nc + 7) / 8 * 8;
    const RedB oo{o.res + 2 * j0, o.rs, o.part, o.counter};
    DISPATCH_W(prec, wide, k_multi_cdot, dim3((unsigned)(nc * ng), nrhs), m, kk, ng, (int)nc, y, nullptr, nullptr,
               vs, n, oo);
  }
}

void blas_multi_cdot(int prec, const void* const* v, int k, const void* y, size_t n, const RedOut& o,
                     hipStream_t st) {
  blas_multi_cdot_b(prec, v, k, y, 0, n, 1, RedB{o.res, 0, o.partial, o.counter}, st);
}

void blas_multi_cdot_pair(int prec, const void* const* v, int k, const void* y1, const void* y2, const void* r,
                          size_t n, const RedOut& o, hipStream_t st) {
  const int ng = (k + kGroup - 1) / kGroup;
  const VecList m = vec_list(v, k);
  const bool wide = wide_ok(v, k, y1, y2, r, 0, n, 1);
  const size_t nv = packs(prec, wide, n);
  // as blas_multi_cdot_b, with the partials of three times the values in the same space
  size_t nc = (std::min<size_t>((nv + kThreads - 1) / kThreads, kDotChunks) + 7) / 8 * 8;
  nc = std::min<size_t>(nc, kRedPartials / (6 * kGroup) / ng / 8 * 8);
  const RedB oo{o.res, 0, o.partial, o.counter};
  const dim3 grid((unsigned)(nc * ng)), block(kThreads);
#define WCMG_DP(T, W)                                                                                          \
  hipLaunchKernelGGL((k_multi_cdot<T, W, 3>), grid, block, 0, st, m, k, ng, (int)nc, y1, y2, r, (size_t)0, n, oo)
  if (prec == WCMG_F64) WCMG_DP(double, 1);
  else if (wide) WCMG_DP(float, 2);
  else WCMG_DP(float, 1);
#undef WCMG_DP
  HIPCHK(hipGetLastError());
}

void blas_gcr_step_pair(int prec, const void* const* q, int k, const void* y1, void* q1, void* y2, const void* rin,
                        void* rout, size_t n, const double* beta, double* qa, double* cj1, double* cj2,
                        hipStream_t st) {
  const VecList m = vec_list(q, k);
  const void* ends[2] = {y2, rin};
  const bool wide = wide_ok(q, k, y1, q1, rout, 0, n, 1) && wide_ok(ends, 2, nullptr, nullptr, nullptr, 0, n, 1);
  const dim3 grid(rows_grid(packs(prec, wide, n), 1, 2048));
  DISPATCH_W(prec, wide, k_gcr_step_pair, grid, m, k, y1, q1, y2, rin, rout, n, beta, qa, cj1, cj2);
}

void blas_gcr_step_b(int prec, const void* const* q, int k, void* y, const void* rin, void* rout, size_t vs, size_t n,
                     int nrhs, const double* beta, size_t bs, double* qa, size_t qs, double* cj, size_t cjs,
                     const RedB& o, hipStream_t st) {
  check_rows(nrhs);
  const VecList m = vec_list(q, k);
  const bool wide = wide_ok(q, k, y, rin, rout, vs, n, nrhs);
  const dim3 grid(rows_grid(packs(prec, wide, n), nrhs, 2048), nrhs);
  DISPATCH_W(prec, wide, k_gcr_step, grid, m, k, y, rin, rout, vs, n, beta, bs, qa, qs, cj, cjs, o);
}

void blas_gcr_step_dev(int prec, const void* const* q, int k, void* y, const void* rin, void* rout, size_t n,
                       const double* beta, double* qa, double* cj, const RedOut& o, hipStream_t st) {
  blas_gcr_step_b(prec, q, k, y, rin, rout, 0, n, 1, beta, 0, qa, 0, cj, 0, RedB{o.res, 0, o.partial, o.counter}, st);
}

static void multi_axpy_rows(int prec, const void* const* v, int k, void* x, size_t vs, size_t n, int nrhs,
                            const double* host, const double* dev, size_t cs, hipStream_t st) {
  check_rows(nrhs);
  for (int j0 = 0; j0 < k; j0 += kVecs) {
    const int kk = std::min(kVecs, k - j0);
    const VecList m = vec_list(v + j0, kk);
    HostCoefs h{};
    if (host) std::copy(host + 2 * j0, host + 2 * (j0 + kk), h.c);
    const double* d = dev ? dev + 2 * j0 : nullptr;
    const bool wide = wide_ok(v + j0, kk, x, nullptr, nullptr, vs, n, nrhs);
    const dim3 grid(rows_grid(packs(prec, wide, n), nrhs, 4096), nrhs);
#define WCMG_MA(T, W)                                                                                            \
  do {                                                                                                           \
    if (dev)                                                                                                     \
      hipLaunchKernelGGL((k_multi_axpy<T, W, true>), grid, dim3(kThreads), 0, st, m, h, kk, x, vs, n, d, cs);    \
    else                                                                                                         \
      hipLaunchKernelGGL((k_multi_axpy<T, W, false>), grid, dim3(kThreads), 0, st, m, h, kk, x, vs, n, d, cs);   \
  } while (0)
    if (prec == WCMG_F64) WCMG_MA(double, 1);
    else if (wide) WCMG_MA(float, 2);
    else WCMG_MA(float, 1);
#undef WCMG_MA
    HIPCHK(hipGetLastError());
  }
}

void blas_multi_axpy(int prec, const double* c, const void* const* v, int k, void* y, size_t n, hipStream_t st) {
  multi_axpy_rows(prec, v, k, y, 0, n, 1, c, nullptr, 0, st);
}

void blas_multi_axpy_dev(int prec, const double* coef, const void* const* v, int k, void* y, size_t n,
                         hipStream_t st) {
  multi_axpy_rows(prec, v, k, y, 0, n, 1, nullptr, coef, 0, st);
}

static void coef_solve(const double* qa, size_t qs, const double* cmat, size_t cms, int ldc, double* y, size_t ys,
                       int nf, int kt, int nrhs, hipStream_t st) {
  if (kt > kMaxSlots) fail(WCMG_EINVAL, "too many GCR slots");
  hipLaunchKernelGGL(k_gcr_coef_solve, dim3(nrhs), dim3(kThreads), 0, st, qa, qs, cmat, cms, ldc, y, ys, nf, kt);
  HIPCHK(hipGetLastError());
}

void blas_gcr_update_x_raw(int prec, const void* const* z, int nf, int kt, void* x, size_t n, const double* qa,
                           const double* cmat, int ldc, double* y, hipStream_t st) {
  if (kt <= 0) return;
  coef_solve(qa, 0, cmat, 0, ldc, y, 0, nf, kt, 1, st);
  multi_axpy_rows(prec, z, kt, x, 0, n, 1, nullptr, y, 0, st);
}

void blas_gcr_update_x_raw_b(int prec, const void* const* z, int kt, void* x, size_t vs, size_t n, int nrhs,
                             const double* qa, size_t qs, const double* cmat, size_t cms, int ldc, double* y,
                             size_t ys, hipStream_t st) {
  check_rows(nrhs);
  if (kt <= 0) return;
  coef_solve(qa, qs, cmat, cms, ldc, y, ys, 0, kt, nrhs, st);
  multi_axpy_rows(prec, z, kt, x, vs, n, nrhs, nullptr, y, ys, st);
}

}  // namespace wcmg

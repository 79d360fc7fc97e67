// Transfer between the fine lattice and the first coarse level
// (red-black paragraph): P from the null vectors split into space-time
// blocks x 2 chiralities, R = P^dag gamma5, and the pieces of the coarse
// operator construction Yhat = R D_p P.
//
//   R:  c(b, s, k) = (+1 | -1)_s  sum_{x in b, chirality(a) = s} conj(V_k(x,a)) r(x,a)
//   P:  e(x, a)    = sum_k V_k(x, a) c(block(x), chirality(a), k)
//
// V_k are the block-orthonormalised vectors, kept block by block:
//   V[k][parity][block][chirality][site of the block's half][6]  complex,
// so that everything R and P read of a vector for one block is contiguous.
// In the fine layouts a block's row is two sites (32 bytes a component plane)
// and a read of one block's share touched four times the bytes.
//
// The kernels walk "units" of a block's half: one complex (FP64 vectors) or
// two (FP32 and FP16), 16 or 8 bytes.  The fine side is the caller's canonical
// layout (read and written in place of a converted copy) or one of the
// solvers', for one parity or both, for one right-hand side or a batch: the
// vectors, by far the larger operand, are read once.
#include "kernels.h"
#include "hop_core.h"

#include <type_traits>

namespace wcmg {

namespace {

__device__ __forceinline__ int coarse_internal(const BlockGeom& bg, int clex) {
  if (!bg.coarse_cb) return clex;
  int c0 = clex % bg.nb[0];
  int r = clex / bg.nb[0];
  int c1 = r % bg.nb[1];
  r /= bg.nb[1];
  int c2 = r % bg.nb[2];
  int c3 = r / bg.nb[2];
  int cp = (c0 + c1 + c2 + c3) & 1;
  return cp * (bg.Vc / 2) + (clex >> 1);
}

// lexicographic index of the l-th site of parity p of block clex
__device__ __forceinline__ int block_lex(const DGeom& g, const BlockGeom& bg, int clex, int p, int l) {
  int r = clex, cc[4];
  cc[0] = r % bg.nb[0];
  r /= bg.nb[0];
  cc[1] = r % bg.nb[1];
  r /= bg.nb[1];
  cc[2] = r % bg.nb[2];
  cc[3] = r / bg.nb[2];
  const int bxh = bg.b[0] / 2;
  int lxh = l % bxh;
  r = l / bxh;
  int c[4];
  c[1] = cc[1] * bg.b[1] + r % bg.b[1];
  r /= bg.b[1];
  c[2] = cc[2] * bg.b[2] + r % bg.b[2];
  c[3] = cc[3] * bg.b[3] + r / bg.b[2];
  c[0] = cc[0] * bg.b[0] + 2 * lxh + ((p + c[1] + c[2] + c[3]) & 1);
  return ((c[3] * g.L[2] + c[2]) * g.L[1] + c[1]) * g.L[0] + c[0];
}

// block of a site and its place in the block's half (the inverse of block_lex)
__device__ __forceinline__ void site_block(const DGeom& g, const BlockGeom& bg, const int c[4], int& clex, int& l) {
  clex = (((c[3] / bg.b[3]) * bg.nb[2] + c[2] / bg.b[2]) * bg.nb[1] + c[1] / bg.b[1]) * bg.nb[0] + c[0] / bg.b[0];
  l = (((c[3] % bg.b[3]) * bg.b[2] + c[2] % bg.b[2]) * bg.b[1] + c[1] % bg.b[1]) * (bg.b[0] / 2) +
      (c[0] % bg.b[0]) / 2;
}

// first complex of (vector k, parity p, block b, chirality s)
__device__ __forceinline__ size_t vec_at(const BlockGeom& bg, int k, int p, int b, int s) {
  return ((((size_t)k * 2 + p) * bg.Vc + b) * 2 + s) * (size_t)(bg.bvol / 2) * 6;
}

// vector storage: E complex elements a unit, arithmetic type C of the
// transfer; L: what a lane of the restriction loads at once, G units
template <typename VT>
struct VecUnit;
template <>
struct VecUnit<double> {
  using U = double2;
  using L = double2;
  using C = double;
  static constexpr int E = 1, G = 1;
  __device__ __forceinline__ static U unit(const L& l, int) { return l; }
  __device__ __forceinline__ static void get(const U& u, cpx<double> v[1]) { v[0] = mk(u.x, u.y); }
};
template <>
struct VecUnit<float> {
  using U = float4;
  using L = float4;
  using C = float;
  static constexpr int E = 2, G = 1;
  __device__ __forceinline__ static U unit(const L& l, int) { return l; }
  __device__ __forceinline__ static void get(const U& u, cpx<float> v[2]) {
    v[0] = mk(u.x, u.y);
    v[1] = mk(u.z, u.w);
  }
};
template <>
struct VecUnit<__half> {
  using U = uint2;
  using L = uint4;
  using C = float;
  static constexpr int E = 2, G = 2;
  __device__ __forceinline__ static U unit(const L& l, int g) {
    return g ? make_uint2(l.z, l.w) : make_uint2(l.x, l.y);
  }
  __device__ __forceinline__ static void get(const U& u, cpx<float> v[2]) {
    const float2 a = __half22float2(*reinterpret_cast<const __half2*>(&u.x));
    const float2 b = __half22float2(*reinterpret_cast<const __half2*>(&u.y));
    v[0] = mk(a.x, a.y);
    v[1] = mk(b.x, b.y);
  }
};

// The fine side of a unit.  The restriction reads it at an offset from its
// block: CANON the canonical complex128 layout (rounded to C on reading; off
// in complexes), else the block layout of the vectors in C (off in units).
template <typename C, int E, bool CANON>
struct FineIn;
template <typename C, int E>
struct FineIn<C, E, true> {
  double2 t[E];
  __device__ __forceinline__ void load(const void* base, int off) {
    const double2* q = reinterpret_cast<const double2*>(base) + off;
#pragma unroll
    for (int e = 0; e < E; ++e) t[e] = q[e];
  }
  __device__ __forceinline__ void get(cpx<C> v[E]) const {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = mk((C)t[e].x, (C)t[e].y);
  }
};
template <typename C, int E>
struct FineIn<C, E, false> {
  typename VecUnit<C>::U t;
  __device__ __forceinline__ void load(const void* base, int off) {
    t = reinterpret_cast<const typename VecUnit<C>::U*>(base)[off];
  }
  __device__ __forceinline__ void get(cpx<C> v[E]) const { VecUnit<C>::get(t, v); }
};
// The prolongation writes the canonical layout or the parity-split one of C.
template <typename C, int E, bool CANON>
__device__ __forceinline__ void store_fine(void* base, int Vh, int lex, int s, int cu,
                                           const cpx<C> v[E]) {
  if constexpr (CANON) {
    double2* q = reinterpret_cast<double2*>(base) + (size_t)lex * 12 + s * 6 + cu * E;
#pragma unroll
    for (int e = 0; e < E; ++e) q[e] = make_double2((double)v[e].r, (double)v[e].i);
  } else {
    typename VecUnit<C>::U u;
    if constexpr (E == 1)
      u = make_double2(v[0].r, v[0].i);
    else
      u = make_float4(v[0].r, v[0].i, v[1].r, v[1].i);
    reinterpret_cast<typename VecUnit<C>::U*>(base)[(size_t)(s * (6 / E) + cu) * Vh + (lex >> 1)] = u;
  }
}

// component re/im `part` of row `row` of coarse site b, rounded to the transfer's arithmetic
template <typename C, bool CANON>
__device__ __forceinline__ void put_coarse(const RestrictArgs& a, int n, int b, int row, int part, double v) {
  const size_t site = a.internal_sites ? coarse_internal(a.bg, b) : b;
  const size_t at = (site * a.site_stride + row) * 2 + part;
  if constexpr (CANON)
    reinterpret_cast<double*>(a.out[n])[at] = (double)(C)v;
  else
    reinterpret_cast<C*>(a.out[n])[at] = (C)v;
}

// the block's site table: lexicographic index of site l of parity p at [p half + l]
__device__ __forceinline__ void fill_sites(int* sites, const DGeom& g, const BlockGeom& bg, int b, int p0, int np) {
  const int half = bg.bvol / 2;
  for (int t = threadIdx.x; t < np * half; t += blockDim.x)
    sites[t] = block_lex(g, bg, b, p0 + t / half, t % half);
}
// where the restriction finds unit t of the block's parities: canonical offset
// in complexes (chirality 0), else the unit's place in the block layout
template <bool CANON, int E>
__device__ __forceinline__ void fill_offsets(int* off, const RestrictArgs& a, int b, int U) {
  constexpr int P = 6 / E;
  for (int t = threadIdx.x; t < a.np * U; t += blockDim.x) {
    const int ip = t >= U, u = t - ip * U;
    if constexpr (CANON) {
      const int l = u / P;
      off[t] = block_lex(a.g, a.bg, b, a.p0 + ip, l) * 12 + (u - l * P) * E;
    } else {
      off[t] = ip * (a.bg.Vc * 2 * U) + u;
    }
  }
}
template <bool CANON, int E>
__device__ __forceinline__ const void* fine_base(const RestrictArgs& a, const void* in, int b, int s) {
  if constexpr (CANON)
    return reinterpret_cast<const double2*>(in) + s * 6;
  else
    return reinterpret_cast<const cpx<typename std::conditional<E == 1, double, float>::type>*>(in) +
           vec_at(a.bg, 0, a.p0, b, s);
}
// ------------------------------------------------------------ restriction
// One right-hand side: a wavefront takes eight vectors of one chirality of a
// block, its lanes the units; the sixteen sums (FP64) are added over the lanes
// by halving (each exchange carries half of the values, 17 of them where a
// butterfly per value takes 96), without LDS or barriers.  Bound by the read
// of the vectors.  16^3x32, Nv 24: FP64, both parities, from the canonical layout
// 435 -> 116 us (5.2 TB/s, a large copy's rate); FP32 even half with FP16 vectors
// (the cycle) 35 -> 26 us.
// FP64 sums: a lane's 24 units added in a row had an error of 2.7e-16 against
// 1.8e-16 of a thread per site; three units at a time into a sum of two words
// 1.6e-16, at the same speed.
constexpr int kRV = 8;

// PARTS: FP64 results from blocks of at least 192 units, summed in parts
template <typename VT, bool CANON, bool PARTS>
__global__ void __launch_bounds__(128) k_restrict(RestrictArgs a) {
  using X = VecUnit<VT>;
  using C = typename X::C;
  using L = typename X::L;
  constexpr int E = X::E, P = 6 / E, G = X::G;
  extern __shared__ int off[];
  const int b = xcd_block(a.bg.Vc);
  if (b >= a.bg.Vc) return;
  const int lane = threadIdx.x & 63, s = threadIdx.x >> 6, k0 = blockIdx.y * kRV;
  const int U = a.bg.bvol / 2 * P;
  if constexpr (CANON) {
    fill_offsets<CANON, E>(off, a, b, U);
    __syncthreads();
  }
  double acc[2 * kRV], low[2 * kRV];
#pragma unroll
  for (int j = 0; j < 2 * kRV; ++j) acc[j] = low[j] = 0.0;
  for (int ip = 0; ip < a.np; ++ip) {
    const void* in = fine_base<CANON, E>(a, a.in[0], b, s);
    const L* v[kRV];
#pragma unroll
    for (int j = 0; j < kRV; ++j)
      v[j] = reinterpret_cast<const L*>(a.vecs) + vec_at(a.bg, min(k0 + j, a.nvec - 1), a.p0 + ip, b, s) / (E * G);
    auto add = [&](int u, double (&sum)[2 * kRV]) {
      FineIn<C, E, CANON> w[G];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        if constexpr (CANON)
          w[h].load(in, off[ip * U + u * G + h]);
        else
          w[h].load(in, ip * (a.bg.Vc * 2 * U) + u * G + h);
      }
      L t[kRV];
#pragma unroll
      for (int j = 0; j < kRV; ++j) t[j] = v[j][u];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        cpx<C> wv[E];
        w[h].get(wv);
#pragma unroll
        for (int j = 0; j < kRV; ++j) {
          cpx<C> vv[E];
          X::get(X::unit(t[j], h), vv);
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const double wr = (double)wv[e].r, wi = (double)wv[e].i, vr = (double)vv[e].r, vi = (double)vv[e].i;
            sum[2 * j] = fma(vr, wr, fma(vi, wi, sum[2 * j]));
            sum[2 * j + 1] = fma(vr, wi, fma(-vi, wr, sum[2 * j + 1]));
          }
        }
      }
    };
    int u = lane;
    // three units from zero, added to a sum of two words: a lane's chain of roundings stays short
    if constexpr (PARTS)
      for (; u + 128 < U; u += 192) {
        double part[2 * kRV];
#pragma unroll
        for (int j = 0; j < 2 * kRV; ++j) part[j] = 0.0;
#pragma unroll
        for (int h = 0; h < 3; ++h) add(u + 64 * h, part);
#pragma unroll
        for (int j = 0; j < 2 * kRV; ++j) {
          const double t = acc[j] + part[j], w = t - acc[j];
          low[j] += (acc[j] - (t - w)) + (part[j] - w);
          acc[j] = t;
        }
      }
#pragma unroll 3
    for (; u < U / G; u += 64) add(u, acc);
  }
  if constexpr (PARTS)
#pragma unroll
    for (int j = 0; j < 2 * kRV; ++j) acc[j] = isfinite(low[j]) ? acc[j] + low[j] : acc[j];
  // after the exchange over lane bit m the lanes with the bit set hold the upper half of the values
#pragma unroll
  for (int h = kRV, m = 32; h >= 1; h >>= 1, m >>= 1) {
    const bool up = lane & m;
#pragma unroll
    for (int j = 0; j < h; ++j) {
      const double give = up ? acc[j] : acc[j + h], keep = up ? acc[j + h] : acc[j];
      acc[j] = keep + __shfl_xor(give, m);
    }
  }
  double r = acc[0];
  r += __shfl_xor(r, 2);
  r += __shfl_xor(r, 1);
  const int idx = lane >> 2, k = k0 + (idx >> 1);
  if ((lane & 3) == 0 && k < a.nvec)
    put_coarse<C, CANON>(a, 0, b, s * a.nvec + k, idx & 1, s ? -r : r);
}

// Several right-hand sides (up to 16 a launch): per block and chirality the
// product [nvec x K] [K x nin] of complex numbers, K the block's half-spinor
// components, on the FP64 matrix instructions 16x16x4.  With re and im of a
// vector as consecutive K entries, column 2n is the right-hand side (the real
// part of conj(V) W) and column 2n + 1 is it times -i (the imaginary part), so
// no product is wasted.  The four wavefronts of a workgroup split K and are
// added in LDS; every vector and every right-hand side is read once.
// Fragments: A row = lane mod 16, B column = lane mod 16, K = lane / 16;
// result row = 4 r + lane / 16, column = lane mod 16.
// The matrix work of two row and two column tiles is 82 us at 16^3x32, Nv 24;
// measured there, 12 right-hand sides: FP32 from the canonical layout 1170 ->
// 240 us (from 9 to 16 inputs it grows by 13 us each, so the rows of 768 bytes
// scattered over twelve fields bound it), the cycle's even half with FP16
// vectors 400 -> 86 us; nine FP64 inputs in the block layout (a column of the
// coarse build) 3830 -> 241 us.  One input stays on k_restrict: there the tiles
// are mostly padding (FP32 84 us against 117 us with two inputs).
// FP64 sums: accumulated through the instructions, K / 4 roundings in a row,
// they had an error of 9.3e-16 (blocks of 256 sites) where one vector had
// 1.8e-16; the products of two steps from zero, added to a sum of two words,
// have 1.6e-16 (of one step 1.3e-16, but a few blocks then wait for the adds: 75
// us where 60 had been, now 65).  The second words take the registers of two
// wavefronts per SIMD with two row and two column tiles, and the time stays (12
// inputs, Nv 24: 291 and 292 us).
typedef double d4 __attribute__((ext_vector_type(4)));

template <typename VT, bool CANON, int MT, int NT>
__global__ void __launch_bounds__(256, MT * NT <= (sizeof(VT) == 8 ? 2 : 4) ? 4 : 2) k_restrict_mfma(RestrictArgs a) {
  using X = VecUnit<VT>;
  using C = typename X::C;
  using L = typename X::L;
  constexpr int E = X::E, P = 6 / E, G = X::G;
  extern __shared__ int off[];
  __shared__ double red[4][256];
  const int b = xcd_block(a.bg.Vc);
  if (b >= a.bg.Vc) return;
  const int U = a.bg.bvol / 2 * P, total = a.np * U;
  fill_offsets<CANON, E>(off, a, b, U);
  __syncthreads();
  // the wavefront's number in a scalar register: the loop's bounds are then scalar too
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), s = blockIdx.y;
  const int q = lane >> 4, j = lane & 15;
  // row and column tiles of this workgroup, when they are shared out over several
  const int zr = (int)gridDim.z / a.col_groups, k0 = ((int)blockIdx.z % zr) * 16 * MT, n0 = ((int)blockIdx.z / zr) * 8 * NT;
  const bool im = j & 1;
  const L* v[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
    v[m] = reinterpret_cast<const L*>(a.vecs) + vec_at(a.bg, min(k0 + 16 * m + j, a.nvec - 1), a.p0, b, s) / (E * G);
  const int pstep = a.bg.Vc * 2 * U / G;  // loads from one parity to the other
  const void* w[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) w[n] = fine_base<CANON, E>(a, a.in[min(n0 + 8 * n + (j >> 1), a.nin - 1)], b, s);
  d4 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[m][n] = (d4){0.0, 0.0, 0.0, 0.0};
  // loads of a step: each lane G units of its vectors and right-hand sides
  struct Step {
    L v[MT];
    FineIn<C, E, CANON> w[NT][G];
  };
  auto load = [&](int t0, Step& st) {
    const int t = t0 + q * G, at = t >= U ? pstep + (t - U) / G : t / G;
#pragma unroll
    for (int m = 0; m < MT; ++m) st.v[m] = v[m][at];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const int o = off[t + h];
#pragma unroll
      for (int n = 0; n < NT; ++n) st.w[n][h].load(w[n], o);
    }
  };
  auto multiply = [&](const Step& st, d4 (&acc)[MT][NT]) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      // B fragments: the right-hand side, or -i times it in odd columns
      double b0[NT][E], b1[NT][E];
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        cpx<C> wv[E];
        st.w[n][h].get(wv);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const C re = wv[e].r, ii = wv[e].i, nr = -re;
          b0[n][e] = (double)(im ? ii : re);
          b1[n][e] = (double)(im ? nr : ii);
        }
      }
      cpx<C> vv[MT][E];
#pragma unroll
      for (int m = 0; m < MT; ++m) X::get(X::unit(st.v[m], h), vv[m]);
#pragma unroll
      for (int e = 0; e < E; ++e) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int n = 0; n < NT; ++n)
            acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)vv[m][e].r, b0[n][e], acc[m][n], 0, 0, 0);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int n = 0; n < NT; ++n)
            acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)vv[m][e].i, b1[n][e], acc[m][n], 0, 0, 0);
      }
    }
  };
  // loads run two steps ahead of the products; no branch inside a turn of the
  // loop, or every wait becomes one for all loads
  constexpr int kStep = 16 * G;
  const int first = wave * 4 * G, steps = (total - first + kStep - 1) / kStep;
  if (steps > 0) {
    auto at = [&](int i) { return first + min(i, steps - 1) * kStep; };
    Step s0, s1, s2;
    load(at(0), s0);
    load(at(1), s1);
    int i = 0;
    auto three = [&](auto&& each) {
      load(at(i + 2), s2);
      each(s0);
      load(at(i + 3), s0);
      each(s1);
      load(at(i + 4), s1);
      each(s2);
      i += 3;
    };
    // FP64 results: the products of two steps are summed from zero and added to a sum of two words
    if constexpr (sizeof(VT) == 8) {
      d4 low[MT][NT], part[MT][NT];
      auto clear = [&](d4 (&sum)[MT][NT]) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int n = 0; n < NT; ++n) sum[m][n] = (d4){0.0, 0.0, 0.0, 0.0};
      };
      auto exact_add = [&]() {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            const d4 t = acc[m][n] + part[m][n], v = t - acc[m][n];
            low[m][n] += (acc[m][n] - (t - v)) + (part[m][n] - v);
            acc[m][n] = t;
          }
      };
      clear(low);
      while (i + 6 <= steps) {
        clear(part);
        load(at(i + 2), s2);
        multiply(s0, part);
        load(at(i + 3), s0);
        multiply(s1, part);
        exact_add();
        clear(part);
        load(at(i + 4), s1);
        multiply(s2, part);
        load(at(i + 5), s2);
        multiply(s0, part);
        exact_add();
        clear(part);
        load(at(i + 6), s0);
        multiply(s1, part);
        load(at(i + 7), s1);
        multiply(s2, part);
        exact_add();
        i += 6;
      }
      auto one = [&](const Step& st) {
        clear(part);
        multiply(st, part);
        exact_add();
      };
      while (i + 3 <= steps) three(one);
      if (i < steps) one(s0);
      if (i + 1 < steps) one(s1);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
          for (int r = 0; r < 4; ++r)  // an infinite sum has no low word
            acc[m][n][r] = isfinite(low[m][n][r]) ? acc[m][n][r] + low[m][n][r] : acc[m][n][r];
    } else {
      auto add = [&](const Step& st) { multiply(st, acc); };
      while (i + 3 <= steps) three(add);
      if (i < steps) add(s0);
      if (i + 1 < steps) add(s1);
    }
  }
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < NT; ++n) {
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][r * 64 + lane] = acc[m][n][r];
      __syncthreads();
      const int tid = threadIdx.x;
      const double sum = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
      const int k = k0 + 16 * m + 4 * wave + q, rhs = n0 + 8 * n + (j >> 1);
      if (k < a.nvec && rhs < a.nin) put_coarse<C, CANON>(a, rhs, b, s * a.nvec + k, j & 1, s ? -sum : sum);
      __syncthreads();
    }
}

// ------------------------------------------------------------ prolongation
// A thread takes one unit of a block and all right-hand sides (NT >= nin): the
// vectors are read once, coalesced, the block's coarse values come from LDS,
// and the sums over k run in order in the transfer's arithmetic.  Bound by the
// vectors and the output.  16^3x32, Nv 24, to the canonical layout: FP64 192 ->
// 124 us; FP32, 12 right-hand sides 856 -> 219 us; the cycle's even half (FP16
// vectors) 26 -> 17 us.
template <typename VT, bool CANON, int NT>
__global__ void __launch_bounds__(256) k_prolong(ProlongArgs a) {
  using X = VecUnit<VT>;
  using C = typename X::C;
  using V2 = typename Vec2<C>::T;
  constexpr int E = X::E, P = 6 / E;
  extern __shared__ __align__(16) char shm[];
  const int b = xcd_block(a.bg.Vc);
  if (b >= a.bg.Vc) return;
  const int half = a.bg.bvol / 2, U = half * P, n2 = 2 * a.nvec;
  V2* cf = reinterpret_cast<V2*>(shm);                    // [2 nvec][NT]
  int* sites = reinterpret_cast<int*>(cf + n2 * NT);      // [np half]
  fill_sites(sites, a.g, a.bg, b, a.p0, a.np);
  const size_t site = a.internal_sites ? coarse_internal(a.bg, b) : b;
  for (int t = threadIdx.x; t < n2 * NT; t += 256) {
    const int n = t / n2, row = t - n * n2;
    V2 c;
    c.x = (C)0;
    c.y = (C)0;
    if (n < a.nin) {
      if constexpr (CANON) {
        const double2 d = reinterpret_cast<const double2*>(a.in[n])[site * n2 + row];
        c.x = (C)d.x;
        c.y = (C)d.y;
      } else {
        c = reinterpret_cast<const V2*>(a.in[n])[site * n2 + row];
      }
    }
    cf[row * NT + n] = c;
  }
  __syncthreads();
  const size_t kstep = (size_t)a.bg.Vc * 4 * U;  // units from one vector to the next
  for (int t = blockIdx.y * 256 + threadIdx.x; t < a.np * 2 * U; t += gridDim.y * 256) {
    const int ip = t >= 2 * U, r = t - ip * 2 * U, s = r >= U, u = r - s * U, l = u / P, cu = u - l * P;
    const typename X::U* v = reinterpret_cast<const typename X::U*>(a.vecs) + vec_at(a.bg, 0, a.p0 + ip, b, s) / E + u;
    const V2* cs = cf + s * a.nvec * NT;
    cpx<C> o[NT][E];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int e = 0; e < E; ++e) o[n][e] = mk((C)0, (C)0);
#pragma unroll 4
    for (int k = 0; k < a.nvec; ++k) {
      cpx<C> vv[E];
      X::get(v[(size_t)k * kstep], vv);
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const V2 c = cs[k * NT + n];
#pragma unroll
        for (int e = 0; e < E; ++e) cfma(o[n][e], vv[e], mk((C)c.x, (C)c.y));
      }
    }
#pragma unroll
    for (int n = 0; n < NT; ++n)
      if (n < a.nin)
        store_fine<C, E, CANON>(a.out[n], a.g.Vh, sites[ip * half + l], s, cu, o[n]);
  }
}

// ------------------------------------------------------------ cycle input
// Even halves of FP64 spinors rounded to C, in the fine layout (the smoother's)
// and in the block layout (the restriction's), right-hand side blockIdx.y.
template <typename C>
__global__ void __launch_bounds__(256) k_round_even(void* fine, void* block, size_t stride, const void* in64,
                                                    size_t stride64, DGeom g, BlockGeom bg) {
  using V2 = typename Vec2<C>::T;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.Vh) return;
  cpx<double> v[12];
  cpx<C> w[12];
  SpinorIO<double>::load(reinterpret_cast<const char*>(in64) + blockIdx.y * stride64, g.Vh, i, v);
#pragma unroll
  for (int k = 0; k < 12; ++k) w[k] = mk((C)v[k].r, (C)v[k].i);
  SpinorIO<C>::store(reinterpret_cast<char*>(fine) + blockIdx.y * stride, g.Vh, i, w);
  int c[4], b, l;
  cb_coords(g, i, 0, c);
  site_block(g, bg, c, b, l);
  V2* o = reinterpret_cast<V2*>(reinterpret_cast<char*>(block) + blockIdx.y * stride) + vec_at(bg, 0, 0, b, 0) + l * 6;
  const size_t chi = (size_t)(bg.bvol / 2) * 6;
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    V2 t;
    t.x = w[k].r;
    t.y = w[k].i;
    o[(k >= 6 ? chi - 6 : 0) + k] = t;
  }
}

// ------------------------------------------------------------ vectors
// fine FP64 vectors (parity-split layout) block by block
__global__ void k_vec_to_block(const double2* __restrict__ raw, double2* __restrict__ out, int nvec, DGeom g,
                               BlockGeom bg) {
  const int half = bg.bvol / 2;
  const size_t total = (size_t)nvec * 2 * bg.Vc * half;
  for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (size_t)gridDim.x * blockDim.x) {
    const int l = (int)(t % half);
    size_t r = t / half;
    const int b = (int)(r % bg.Vc);
    r /= bg.Vc;
    const int p = (int)(r % 2), k = (int)(r / 2);
    const double2* src = raw + (size_t)(2 * k + p) * 12 * g.Vh + (block_lex(g, bg, b, p, l) >> 1);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      double2* dst = out + vec_at(bg, k, p, b, s) + (size_t)l * 6;
#pragma unroll
      for (int c = 0; c < 6; ++c) dst[c] = src[(size_t)(6 * s + c) * g.Vh];
    }
  }
}

// chirality s of vector k as a fine FP64 spinor (the other chirality zero), both halves
__global__ void k_block_column(const double2* __restrict__ vecs, double2* __restrict__ out, int k, int s, DGeom g,
                               BlockGeom bg) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 2 * g.Vh) return;
  const int p = t >= g.Vh, i = t - p * g.Vh;
  int c[4], b, l;
  cb_coords(g, i, p, c);
  site_block(g, bg, c, b, l);
  const double2* src = vecs + vec_at(bg, k, p, b, s) + (size_t)l * 6;
  double2* dst = out + (size_t)p * 12 * g.Vh + i;
#pragma unroll
  for (int a = 0; a < 6; ++a) {
    dst[(size_t)(6 * s + a) * g.Vh] = src[a];
    dst[(size_t)(6 * (1 - s) + a) * g.Vh] = make_double2(0.0, 0.0);
  }
}

// FP32 copy of the vectors with the rounding of half-precision spinors (one scale a site)
__global__ void k_vec_half_rounded(const double2* __restrict__ v64, float2* __restrict__ out, int nvec, BlockGeom bg) {
  const int half = bg.bvol / 2;
  const size_t total = (size_t)nvec * 2 * bg.Vc * half;
  for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (size_t)gridDim.x * blockDim.x) {
    const int l = (int)(t % half);
    const size_t kpb = t / half;
    const size_t at = kpb * 2 * half * 6 + (size_t)l * 6;
    cpx<float> v[12];
#pragma unroll
    for (int a = 0; a < 12; ++a) {
      const double2 d = v64[at + (a >= 6 ? (size_t)half * 6 - 6 : 0) + a];
      v[a] = mk((float)d.x, (float)d.y);
    }
    round_half_spinor(v);
#pragma unroll
    for (int a = 0; a < 12; ++a) out[at + (a >= 6 ? (size_t)half * 6 - 6 : 0) + a] = make_float2(v[a].r, v[a].i);
  }
}

// Gram-Schmidt (classical, twice) per (block, chirality) on FP64 vectors.  The
// vector being orthogonalised sits in LDS; each wavefront forms whole dot
// products with every eighth earlier vector (no barrier per group of them),
// then every thread subtracts the combination from the elements it owns.
// Bound by re-reading the earlier vectors from L2.  16^3x32, Nv 24: 21.8 ->
// 4.6 ms.
constexpr int kOrthoThreads = 512;

__global__ void __launch_bounds__(kOrthoThreads) k_block_ortho(double2* vecs, int nvec, BlockGeom bg, int* flag) {
  extern __shared__ __align__(16) char shm[];
  __shared__ double2 cf[64];
  __shared__ double2 nrm[kOrthoThreads / 64];
  double2* v = reinterpret_cast<double2*>(shm);  // [2][half * 6]
  const int b = blockIdx.x, s = blockIdx.y, run = bg.bvol / 2 * 6, len = 2 * run;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const size_t pstep = vec_at(bg, 0, 1, 0, 0), kstep = 2 * pstep;
  double2* base = vecs + vec_at(bg, 0, 0, b, s);
  auto at = [&](int e) { return e < run ? (size_t)e : pstep + (e - run); };
  // sum of squares of v over the workgroup (every thread gets it), carried in two words: an error
  // of a norm scales a whole vector and does not average out in a product with it
  auto norm2 = [&]() {
#pragma clang fp contract(off)
    double t = 0.0, low = 0.0;
    auto add = [&](double p, double l) {
      const double u = t + p, w = u - t;
      low += ((t - (u - w)) + (p - w)) + l;
      t = u;
    };
    for (int e = threadIdx.x; e < len; e += kOrthoThreads) {
      const double x = v[e].x, y = v[e].y;
      add(x * x, fma(x, x, -(x * x)));
      add(y * y, fma(y, y, -(y * y)));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) add(__shfl_xor(t, off), __shfl_xor(low, off));
    __syncthreads();
    if (lane == 0) nrm[wave] = make_double2(t, low);
    __syncthreads();
    t = low = 0.0;
    for (int q = 0; q < kOrthoThreads / 64; ++q) add(nrm[q].x, nrm[q].y);
    return t + low;
  };
  for (int k = 0; k < nvec; ++k) {
    double2* vk = base + (size_t)k * kstep;
    for (int e = threadIdx.x; e < len; e += kOrthoThreads) v[e] = vk[at(e)];
    const double n0 = norm2();
    for (int pass = 0; pass < 2 && k > 0; ++pass) {
      for (int j = wave; j < k; j += kOrthoThreads / 64) {
        const double2* qj = base + (size_t)j * kstep;
        double pr[4] = {0.0, 0.0, 0.0, 0.0}, pi[4] = {0.0, 0.0, 0.0, 0.0};
        int e = lane;
        for (; e + 192 < len; e += 256)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const double2 t = qj[at(e + 64 * u)], x = v[e + 64 * u];
            pr[u] += t.x * x.x + t.y * x.y;
            pi[u] += t.x * x.y - t.y * x.x;
          }
        for (; e < len; e += 64) {
          const double2 t = qj[at(e)], x = v[e];
          pr[0] += t.x * x.x + t.y * x.y;
          pi[0] += t.x * x.y - t.y * x.x;
        }
        double sr = (pr[0] + pr[1]) + (pr[2] + pr[3]), si = (pi[0] + pi[1]) + (pi[2] + pi[3]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
          sr += __shfl_xor(sr, off);
          si += __shfl_xor(si, off);
        }
        if (lane == 0) cf[j] = make_double2(sr, si);
      }
      __syncthreads();
      for (int e = threadIdx.x; e < len; e += kOrthoThreads) {
        cpx<double> x = mk(v[e].x, v[e].y);
        const double2* q = base + at(e);
#pragma unroll 4
        for (int j = 0; j < k; ++j) {
          const double2 t = q[(size_t)j * kstep];
          x = x - mk(cf[j].x, cf[j].y) * mk(t.x, t.y);
        }
        v[e] = make_double2(x.r, x.i);
      }
      __syncthreads();
    }
    const double nk = sqrt(norm2());
    if (!(nk > 1e-12 * sqrt(n0)) && threadIdx.x == 0) *flag = 1;
    const double inv = nk > 0.0 ? 1.0 / nk : 0.0;
    for (int e = threadIdx.x; e < len; e += kOrthoThreads) vk[at(e)] = make_double2(inv * v[e].x, inv * v[e].y);
    __syncthreads();
  }
}

// Nine buckets of D_p = A A^-1 + H A^-1 acting on (v, u = A^-1 v), split by the
// block the hop comes from: bucket 0 collects v and every hop that stays in
// the block, bucket 1+d the hop from direction d when it crosses the block face.
struct SplitArgs {
  double2* bucket[9];
  const void* v;
  const void* u;
  const void* gauge;
  DGeom g;
  BlockGeom bg;
};

// the buckets are in the block layout that the restriction reads: a site's half-spinors at `at`
__device__ __forceinline__ void store_block(const SplitArgs& a, double2* bucket, size_t at, const cpx<double> w[12]) {
  const size_t chi = (size_t)(a.bg.bvol / 2) * 6;
#pragma unroll
  for (int k = 0; k < 12; ++k) bucket[at + (k >= 6 ? chi - 6 : 0) + k] = make_double2(w[k].r, w[k].i);
}

template <int MU>
__device__ __forceinline__ void split_mu(const SplitArgs& a, int p, int i, const int c[4], size_t at,
                                         cpx<double> acc0[12]) {
  const DGeom& g = a.g;
  const size_t hb = (size_t)12 * g.Vh * 16;  // bytes of one FP64 parity half
  const void* u_op = reinterpret_cast<const char*>(a.u) + (size_t)(1 - p) * hb;
  const bool coarse_extent = a.bg.nb[MU] > 1;
#pragma unroll
  for (int back = 0; back < 2; ++back) {
    int n[4] = {c[0], c[1], c[2], c[3]};
    int nb;
    cpx<double> psi[12], h[6], hu[6], U[9], hd[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) hd[k] = mk(0.0, 0.0);
    bool cross;
    if (!back) {
      n[MU] = (n[MU] + 1 == g.L[MU]) ? 0 : n[MU] + 1;
      nb = cb_index(g, n);
      SpinorIO<double>::load(u_op, g.Vh, nb, psi);
      load_link<double, double>(a.gauge, g.Vh, p, MU, i, U);
      project<double, MU, false>(psi, h);
      link_mul<double, false>(U, h, hu);
      if (MU == 3 && c[3] == g.L[3] - 1)
        for (int k = 0; k < 6; ++k) hu[k] = g.t_bc * hu[k];
      if (MU < 3)
        for (int k = 0; k < 6; ++k) hu[k] = g.hs * hu[k];
      accumulate<double, MU, false>(hd, hu);
      cross = coarse_extent && (c[MU] % a.bg.b[MU] == a.bg.b[MU] - 1);
    } else {
      n[MU] = (n[MU] == 0) ? g.L[MU] - 1 : n[MU] - 1;
      nb = cb_index(g, n);
      SpinorIO<double>::load(u_op, g.Vh, nb, psi);
      load_link<double, double>(a.gauge, g.Vh, 1 - p, MU, nb, U);
      project<double, MU, true>(psi, h);
      link_mul<double, true>(U, h, hu);
      if (MU == 3 && c[3] == 0)
        for (int k = 0; k < 6; ++k) hu[k] = g.t_bc * hu[k];
      if (MU < 3)
        for (int k = 0; k < 6; ++k) hu[k] = g.hs * hu[k];
      accumulate<double, MU, true>(hd, hu);
      cross = coarse_extent && (c[MU] % a.bg.b[MU] == 0);
    }
    cpx<double> w[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      hd[k] = -0.5 * hd[k];
      w[k] = cross ? hd[k] : mk(0.0, 0.0);
      if (!cross) acc0[k] = acc0[k] + hd[k];
    }
    store_block(a, a.bucket[1 + 2 * MU + back], at, w);
  }
}

__global__ void __launch_bounds__(128) k_hop_split(SplitArgs a) {
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= 2 * a.g.Vh) return;
  const int p = gid / a.g.Vh, i = gid % a.g.Vh;
  int c[4];
  cb_coords(a.g, i, p, c);
  const size_t hb = (size_t)12 * a.g.Vh * 16;
  int b, l;
  site_block(a.g, a.bg, c, b, l);
  const size_t at = vec_at(a.bg, 0, p, b, 0) + (size_t)l * 6;
  cpx<double> acc0[12];
  SpinorIO<double>::load(reinterpret_cast<const char*>(a.v) + (size_t)p * hb, a.g.Vh, i, acc0);
  split_mu<0>(a, p, i, c, at, acc0);
  split_mu<1>(a, p, i, c, at, acc0);
  split_mu<2>(a, p, i, c, at, acc0);
  split_mu<3>(a, p, i, c, at, acc0);
  store_block(a, a.bucket[0], at, acc0);
}

}  // namespace

int coarse_internal_index_host(const BlockGeom& bg, int clex) {
  if (!bg.coarse_cb) return clex;
  int c0 = clex % bg.nb[0];
  int r = clex / bg.nb[0];
  int c1 = r % bg.nb[1];
  r /= bg.nb[1];
  int c2 = r % bg.nb[2];
  int c3 = r / bg.nb[2];
  int cp = (c0 + c1 + c2 + c3) & 1;
  return cp * (bg.Vc / 2) + (clex >> 1);
}


namespace {
inline int transfer_tiles(int n, int per) { return (n + per - 1) / per; }

void check_transfer(int nvec, const BlockGeom& bg) {
  if (nvec < 1 || nvec > 64) fail(WCMG_EDIM, "nvec must be in 1..64");
  if (bg.bvol > 1024 || bg.bvol % 16) fail(WCMG_EDIM, "block volume must be a multiple of 16, at most 1024");
}

template <typename VT, bool CANON>
void restrict_t(const RestrictArgs& a, hipStream_t st) {
  const size_t shm = (size_t)a.np * (a.bg.bvol / 2) * (6 / VecUnit<VT>::E) * sizeof(int);
  if (a.nin == 1) {
    const dim3 g1(xcd_grid(a.bg.Vc), transfer_tiles(a.nvec, kRV));
    if (sizeof(VT) == 8 && a.bg.bvol / 2 * 6 >= 192)
      hipLaunchKernelGGL((k_restrict<VT, CANON, sizeof(VT) == 8>), g1, dim3(128), CANON ? shm : 0, st, a);
    else
      hipLaunchKernelGGL((k_restrict<VT, CANON, false>), g1, dim3(128), CANON ? shm : 0, st, a);
    HIPCHK(hipGetLastError());
    return;
  }
  if (sizeof(VT) < 8 && a.nin == 2 && a.bg.Vc < 256 && a.bg.bvol > 512) {
    // few large blocks: two single launches have more workgroups than the tiles (64 blocks of 1024
    // sites, Nv 20 / 40 / 64: 93 / 134 / 190 us, tiles 129 / 164 / 267; blocks of 256 and less lose)
    RestrictArgs h = a;
    h.nin = 1;
    restrict_t<VT, CANON>(h, st);
    h.in[0] = a.in[1];
    h.out[0] = a.out[1];
    restrict_t<VT, CANON>(h, st);
    return;
  }
  const int mt = transfer_tiles(a.nvec, 16);
  dim3 grid(xcd_grid(a.bg.Vc), 2);
#define WCMG_RM(M)                                                                                    \
  do {                                                                                                \
    if (a.nin <= 8)                                                                                   \
      hipLaunchKernelGGL((k_restrict_mfma<VT, CANON, M, 1>), grid, dim3(256), shm, st, a);            \
    else                                                                                              \
      hipLaunchKernelGGL((k_restrict_mfma<VT, CANON, M, 2>), grid, dim3(256), shm, st, a);            \
  } while (0)
  if (sizeof(VT) == 8 && a.nin > 8 && mt <= 2 && a.bg.Vc <= 64) {
    // so few blocks that the column tiles find compute units of their own
    RestrictArgs h = a;
    h.col_groups = 2;
    grid.z = 2;
    if (mt == 1)
      hipLaunchKernelGGL((k_restrict_mfma<VT, CANON, 1, 1>), grid, dim3(256), shm, st, h);
    else
      hipLaunchKernelGGL((k_restrict_mfma<VT, CANON, 2, 1>), grid, dim3(256), shm, st, h);
  } else if (mt == 1) {
    WCMG_RM(1);
  } else if (mt == 2) {
    WCMG_RM(2);
  } else if (mt == 3) {
    WCMG_RM(3);
  } else if (sizeof(VT) == 8 && a.nin > 8) {
    // four row tiles, two column tiles and their low words exceed the registers: two rows each
    grid.z = 2;
    WCMG_RM(2);
  } else {
    WCMG_RM(4);
  }
#undef WCMG_RM
  HIPCHK(hipGetLastError());
}

template <typename VT, bool CANON, int NT>
void prolong_n(const ProlongArgs& a, hipStream_t st) {
  using X = VecUnit<VT>;
  const int units = a.np * a.bg.bvol / 2 * 2 * (6 / X::E);
  const size_t shm = (size_t)2 * a.nvec * NT * 2 * sizeof(typename X::C) + (size_t)a.np * (a.bg.bvol / 2) * sizeof(int);
  // one pass of each thread where the coarse values are few, else longer runs
  // of a workgroup over its block (their load into LDS is then paid once)
  const int pieces = std::max(1, std::min(transfer_tiles(units, 256), NT > 4 ? 3 : 6));
  hipLaunchKernelGGL((k_prolong<VT, CANON, NT>), dim3(xcd_grid(a.bg.Vc), pieces), dim3(256), shm, st, a);
  HIPCHK(hipGetLastError());
}
template <typename VT, bool CANON>
void prolong_t(const ProlongArgs& a, hipStream_t st) {
  if (a.nin == 1) prolong_n<VT, CANON, 1>(a, st);
  else if (a.nin <= 4) prolong_n<VT, CANON, 4>(a, st);
  else if (a.nin <= 8) prolong_n<VT, CANON, 8>(a, st);
  else if (a.nin <= 12) prolong_n<VT, CANON, 12>(a, st);
  else prolong_n<VT, CANON, 16>(a, st);
}
}  // namespace

void launch_restrict(int vprec, bool canonical, const RestrictArgs& a, hipStream_t st) {
  check_transfer(a.nvec, a.bg);
  if (a.nin < 1 || a.nin > kMaxTransfer) fail(WCMG_EINVAL, "restriction of 1..16 vectors at once");
  if (vprec == WCMG_F64) canonical ? restrict_t<double, true>(a, st) : restrict_t<double, false>(a, st);
  else if (vprec == WCMG_F32) canonical ? restrict_t<float, true>(a, st) : restrict_t<float, false>(a, st);
  else if (!canonical) restrict_t<__half, false>(a, st);
  else fail(WCMG_EINVAL, "FP16 vectors serve the cycle only");
}

void launch_prolong(int vprec, bool canonical, const ProlongArgs& a, hipStream_t st) {
  check_transfer(a.nvec, a.bg);
  if (a.nin < 1 || a.nin > kMaxTransfer) fail(WCMG_EINVAL, "prolongation of 1..16 vectors at once");
  if (!canonical && a.np != 1) fail(WCMG_EINVAL, "prolongation of one parity to the parity-split layout");
  if (vprec == WCMG_F64) canonical ? prolong_t<double, true>(a, st) : prolong_t<double, false>(a, st);
  else if (vprec == WCMG_F32) canonical ? prolong_t<float, true>(a, st) : prolong_t<float, false>(a, st);
  else if (!canonical) prolong_t<__half, false>(a, st);
  else fail(WCMG_EINVAL, "FP16 vectors serve the cycle only");
}

void launch_round_even(int prec, void* fine, void* block, const void* in64, const Geom& g, const BlockGeom& bg,
                       int nrhs, hipStream_t st) {
  const dim3 grid((g.Vh + 255) / 256, nrhs);
  const size_t h64 = spinor_bytes(WCMG_F64, g.Vh), h = spinor_bytes(prec, g.Vh);
  if (prec == WCMG_F64)
    hipLaunchKernelGGL(k_round_even<double>, grid, dim3(256), 0, st, fine, block, h, in64, h64, dgeom(g), bg);
  else
    hipLaunchKernelGGL(k_round_even<float>, grid, dim3(256), 0, st, fine, block, h, in64, h64, dgeom(g), bg);
  HIPCHK(hipGetLastError());
}

void launch_vec_to_block(void* out, const void* raw, int nvec, const Geom& g, const BlockGeom& bg, hipStream_t st) {
  const size_t total = (size_t)nvec * 2 * bg.Vc * (bg.bvol / 2);
  const int blocks = (int)std::min<size_t>((total + 255) / 256, 65536);
  hipLaunchKernelGGL(k_vec_to_block, dim3(blocks), dim3(256), 0, st, reinterpret_cast<const double2*>(raw),
                     reinterpret_cast<double2*>(out), nvec, dgeom(g), bg);
  HIPCHK(hipGetLastError());
}

void launch_block_column(void* out, const void* v64, int k, int s, const Geom& g, const BlockGeom& bg,
                         hipStream_t st) {
  hipLaunchKernelGGL(k_block_column, dim3((2 * g.Vh + 255) / 256), dim3(256), 0, st,
                     reinterpret_cast<const double2*>(v64), reinterpret_cast<double2*>(out), k, s, dgeom(g), bg);
  HIPCHK(hipGetLastError());
}

void launch_vec_half_rounded(void* out32, const void* v64, int nvec, const BlockGeom& bg, hipStream_t st) {
  const size_t total = (size_t)nvec * 2 * bg.Vc * (bg.bvol / 2);
  const int blocks = (int)std::min<size_t>((total + 255) / 256, 65536);
  hipLaunchKernelGGL(k_vec_half_rounded, dim3(blocks), dim3(256), 0, st, reinterpret_cast<const double2*>(v64),
                     reinterpret_cast<float2*>(out32), nvec, bg);
  HIPCHK(hipGetLastError());
}

void launch_block_orthonormalize(void* vecs, int nvec, const BlockGeom& bg, int* flag, hipStream_t st) {
  check_transfer(nvec, bg);
  const size_t shm = (size_t)bg.bvol * 6 * 16;
  if (shm > 64 * 1024)  // blocks of more than 682 sites
    HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_block_ortho),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
  hipLaunchKernelGGL(k_block_ortho, dim3(bg.Vc, 2), dim3(kOrthoThreads), shm, st, reinterpret_cast<double2*>(vecs),
                     nvec, bg, flag);
  HIPCHK(hipGetLastError());
}

void launch_hop_split(void* const* buckets, const void* v, const void* u, const void* gauge64, const Geom& g,
                      const BlockGeom& bg, hipStream_t st) {
  SplitArgs a;
  for (int k = 0; k < 9; ++k) a.bucket[k] = reinterpret_cast<double2*>(buckets[k]);
  a.v = v;
  a.u = u;
  a.gauge = gauge64;
  a.g = dgeom(g);
  a.bg = bg;
  dim3 grid((2 * g.Vh + 127) / 128), block(128);
  hipLaunchKernelGGL(k_hop_split, grid, block, 0, st, a);
  HIPCHK(hipGetLastError());
}

}  // namespace wcmg

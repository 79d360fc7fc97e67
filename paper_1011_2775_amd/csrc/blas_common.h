// Shared pieces of the BLAS-1 kernels: complex loads/stores in double or
// float storage, the block reduction into per-block partials, and the grid
// sizes (which depend only on the vector length, so results are bitwise
// reproducible run to run).
#pragma once

#include <algorithm>

#include "kernels.h"

namespace wcmg {
namespace blas_detail {

constexpr int kThreads = 256;

template <typename T>
struct C2;
template <>
struct C2<double> {
  using V = double2;
};
template <>
struct C2<float> {
  using V = float2;
};

template <typename T>
__device__ __forceinline__ cpx<double> ld(const void* p, size_t i) {
  auto v = reinterpret_cast<const typename C2<T>::V*>(p)[i];
  return mk((double)v.x, (double)v.y);
}
template <typename T>
__device__ __forceinline__ void st(void* p, size_t i, cpx<double> c) {
  using V = typename C2<T>::V;
  V v;
  v.x = (T)c.r;
  v.y = (T)c.i;
  reinterpret_cast<V*>(p)[i] = v;
}

// Sum of NR doubles over nb blocks in one launch: every block stores its
// partials (device-coherent), counts itself in *counter, and the last block to
// arrive adds the partials in block order (TPV threads per value over fixed
// strided subsets of the blocks, then a fixed shuffle tree) and writes the
// first nvalid sums to res (and hres); it then rearms the counter.  The
// order of the additions never depends on which block finishes last.
// block: this block's place 0 .. nb-1 in the sum; partial: nb x NR doubles.
// Several sums share a launch (one per right-hand side or group of vectors)
// when each has partials and a row of counters of its own.
//
// Atomic adds to one cache line take turns (about 10 ns each), so a row holds
// eight counters on lines of their own, each counting every eighth block, and
// one that counts the eight: 4608 adds to one line had cost k_cdot_norm_b with
// twelve right-hand sides 45 of its 70 us.
template <int NR>
__device__ __forceinline__ void block_reduce_row(double (&v)[NR], double* partial, unsigned* counter, int nb,
                                                 int block, double* res, double* hres, int nvalid) {
  __shared__ double sh[NR][kThreads / 64];
  __shared__ double shw[kThreads / 64];
  __shared__ int last_s;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if constexpr (NR % 16 == 0 && NR > 16) {
    // many values: each exchange hands the lanes on either side half of them (the same sums bit for
    // bit; 51 exchanges for 48 values where six each are 288)
    int base = 0;
#pragma unroll
    for (int off = 32, h = NR / 2; off >= 4; off >>= 1, h >>= 1) {
      const bool up = lane & off;
      base += up ? h : 0;
#pragma unroll
      for (int k = 0; k < h; ++k) {
        const double give = up ? v[k] : v[k + h], keep = up ? v[k + h] : v[k];
        v[k] = keep + __shfl_xor(give, off);
      }
    }
#pragma unroll
    for (int k = 0; k < NR / 16; ++k) {
      v[k] += __shfl_xor(v[k], 2);
      v[k] += __shfl_xor(v[k], 1);
      if ((lane & 3) == 0) sh[base + k][wave] = v[k];
    }
  } else {
#pragma unroll
    for (int k = 0; k < NR; ++k) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off);
    }
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < NR; ++k) sh[k][wave] = v[k];
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < NR) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) s += sh[threadIdx.x][w];
    __hip_atomic_store(partial + (size_t)block * NR + threadIdx.x, s, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  // the partial stores are complete (and coherent) before the block counts itself
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const int sub = block & 7;
    const unsigned mine = (nb - sub + 7) >> 3, subs = nb < 8 ? nb : 8;
    bool last = __hip_atomic_fetch_add(counter + (sub + 1) * kCounterLine, 1u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT) == mine - 1;
    if (last)
      last = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == subs - 1;
    last_s = last;
  }
  __syncthreads();
  if (!last_s) return;
  int tpv = 1;
  while (tpv * 2 * nvalid <= kThreads && tpv < nb) tpv *= 2;
  const int t = threadIdx.x, vv = t / tpv, j = t - vv * tpv;
  double s = 0.0;
  if (vv < nvalid) {
    // eight loads in flight, then added in block order
    int b = j;
    for (; b + 7 * tpv < nb; b += 8 * tpv) {
      double p[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        p[u] = __hip_atomic_load(partial + (size_t)(b + u * tpv) * NR + vv, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int u = 0; u < 8; ++u) s += p[u];
    }
    for (; b < nb; b += tpv)
      s += __hip_atomic_load(partial + (size_t)b * NR + vv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const int width = tpv < 64 ? tpv : 64;
  for (int off = width >> 1; off > 0; off >>= 1) s += __shfl_down(s, off, width);
  if (tpv > 64) {
    if (lane == 0) shw[wave] = s;
    __syncthreads();
    if (j == 0 && vv < nvalid) {
      double u = 0.0;
      for (int q = 0; q < tpv / 64; ++q) u += shw[wave + q];
      s = u;
    }
  }
  if (j == 0 && vv < nvalid) {
    res[vv] = s;
    if (hres) hres[vv] = s;
  }
  if (threadIdx.x < 9)
    __hip_atomic_store(counter + threadIdx.x * kCounterLine, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int NR>
__device__ __forceinline__ void block_reduce(double (&v)[NR], const RedOut& o) {
  block_reduce_row<NR>(v, o.partial, o.counter, gridDim.x, blockIdx.x, o.res, o.hres, NR);
}

// enough blocks that every thread handles about 8 elements, at most
// kRedBlocks; short vectors (the coarse levels) spread over up to 64 blocks
// with at least one element per thread, so that a pass is not limited by the
// latency of a handful of compute units
inline dim3 red_grid(size_t n) {
  size_t b = (n + 8 * kThreads - 1) / (8 * kThreads);
  const size_t spread = std::min<size_t>((n + kThreads - 1) / kThreads, 64);
  if (b < spread) b = spread;
  if (b < 1) b = 1;
  if (b > (size_t)kRedBlocks) b = kRedBlocks;
  return dim3((unsigned)b);
}
inline dim3 ew_grid(size_t n) {
  size_t b = (n + kThreads - 1) / kThreads;
  if (b > 65536) b = 65536;
  if (b == 0) b = 1;
  return dim3((unsigned)b);
}

#define GRID_STRIDE(i, n) \
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (size_t)gridDim.x * blockDim.x)


}  // namespace blas_detail
}  // namespace wcmg

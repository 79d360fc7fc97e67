// Batched BLAS-1 kernels for the lockstep multi-right-hand-side solvers.
//
// A batch holds nrhs vectors of n complex elements, vstride elements apart.
// Grid row blockIdx.y is the right-hand side; every reduction of a batch
// keeps its per-block partials at part[rhs][block][NR] and the last block of
// a right-hand side to arrive adds them (fixed tree, as in the single-vector
// kernels) into res[rhs * rs + k], so a reduction is one launch.
#include "blas_common.h"

namespace wcmg {

namespace {

using namespace blas_detail;

template <int NR>
__device__ __forceinline__ void reduce_rhs(double (&v)[NR], const RedB& o) {
  block_reduce_row<NR>(v, o.part + (size_t)blockIdx.y * gridDim.x * NR, o.counter + blockIdx.y * kCounterRow,
                       gridDim.x, blockIdx.x, o.res + (size_t)blockIdx.y * o.rs, nullptr, NR);
}
template <typename T>
__device__ __forceinline__ const void* row(const void* p, size_t vs) {
  return reinterpret_cast<const char*>(p) + (size_t)blockIdx.y * vs * sizeof(typename C2<T>::V);
}
template <typename T>
__device__ __forceinline__ void* row(void* p, size_t vs) {
  return reinterpret_cast<char*>(p) + (size_t)blockIdx.y * vs * sizeof(typename C2<T>::V);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_norm2_b(const void* x, size_t vs, size_t n, RedB o) {
  double v[1] = {0.0};
  const void* xr = row<T>(x, vs);
  GRID_STRIDE(i, n) {
    cpx<double> a = ld<T>(xr, i);
    v[0] += a.r * a.r + a.i * a.i;
  }
  reduce_rhs(v, o);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_cdot_norm_b(const void* x, const void* y, size_t vs, size_t n, RedB o) {
  double v[3] = {0.0, 0.0, 0.0};
  const void* xr = row<T>(x, vs);
  const void* yr = row<T>(y, vs);
  GRID_STRIDE(i, n) {
    cpx<double> a = ld<T>(xr, i), b = ld<T>(yr, i);
    v[0] += a.r * b.r + a.i * b.i;
    v[1] += a.r * b.i - a.i * b.r;
    v[2] += a.r * a.r + a.i * a.i;
  }
  reduce_rhs(v, o);
}

template <typename T>
__global__ void k_zero_b(void* x, size_t vs, size_t n) {
  void* xr = row<T>(x, vs);
  GRID_STRIDE(i, n) st<T>(xr, i, mk(0.0, 0.0));
}
template <typename T>
__global__ void k_copy_b(void* y, const void* x, size_t vs, size_t n) {
  void* yr = row<T>(y, vs);
  const void* xr = row<T>(x, vs);
  GRID_STRIDE(i, n) st<T>(yr, i, ld<T>(xr, i));
}
// out = b - y (out may be y)
template <typename T>
__global__ void k_residual_b(void* out, const void* b, const void* y, size_t vs, size_t n) {
  void* o = row<T>(out, vs);
  const void* br = row<T>(b, vs);
  const void* yr = row<T>(y, vs);
  GRID_STRIDE(i, n) st<T>(o, i, ld<T>(br, i) - ld<T>(yr, i));
}

// MR step of every right-hand side with alpha = coef[0..1] / coef[2] (row r at coef + r * cs)
template <typename T>
__global__ void k_mr_update_b(const double* coef, size_t cs, void* x, void* r, const void* Ar, size_t vs, size_t n) {
  const double* cf = coef + (size_t)blockIdx.y * cs;
  const double d = cf[2];
  const cpx<double> a = d > 0.0 ? mk(cf[0] / d, cf[1] / d) : mk(0.0, 0.0);
  void* xr = row<T>(x, vs);
  void* rr = row<T>(r, vs);
  const void* ar = row<T>(Ar, vs);
  GRID_STRIDE(i, n) {
    st<T>(xr, i, ld<T>(xr, i) + a * ld<T>(rr, i));
    st<T>(rr, i, ld<T>(rr, i) - a * ld<T>(ar, i));
  }
}

}  // namespace

#define DISPATCH_B(prec, KERNEL, grid, ...)                                                 \
  do {                                                                                      \
    if ((prec) == WCMG_F64)                                                                 \
      hipLaunchKernelGGL(KERNEL<double>, grid, dim3(kThreads), 0, st, __VA_ARGS__);         \
    else                                                                                    \
      hipLaunchKernelGGL(KERNEL<float>, grid, dim3(kThreads), 0, st, __VA_ARGS__);          \
    HIPCHK(hipGetLastError());                                                              \
  } while (0)

static dim3 red_grid_b(size_t n, int nrhs) { return dim3(red_grid(n).x, nrhs); }
static dim3 ew_grid_b(size_t n, int nrhs) { return dim3(ew_grid(n).x, nrhs); }

static void check_batch(int nrhs) {
  if (nrhs < 1 || nrhs > kMaxBatch) fail(WCMG_EINVAL, "batch size out of range");
}

void blas_norm2_b(int prec, const void* x, size_t vs, size_t n, int nrhs, const RedB& o, hipStream_t st) {
  check_batch(nrhs);
  DISPATCH_B(prec, k_norm2_b, red_grid_b(n, nrhs), x, vs, n, o);
}

void blas_cdot_norm_b(int prec, const void* x, const void* y, size_t vs, size_t n, int nrhs, const RedB& o,
                      hipStream_t st) {
  check_batch(nrhs);
  DISPATCH_B(prec, k_cdot_norm_b, red_grid_b(n, nrhs), x, y, vs, n, o);
}

void blas_zero_b(int prec, void* x, size_t vs, size_t n, int nrhs, hipStream_t st) {
  check_batch(nrhs);
  if (n) DISPATCH_B(prec, k_zero_b, ew_grid_b(n, nrhs), x, vs, n);
}
void blas_copy_b(int prec, void* y, const void* x, size_t vs, size_t n, int nrhs, hipStream_t st) {
  check_batch(nrhs);
  if (n) DISPATCH_B(prec, k_copy_b, ew_grid_b(n, nrhs), y, x, vs, n);
}
void blas_residual_b(int prec, void* out, const void* b, const void* y, size_t vs, size_t n, int nrhs,
                     hipStream_t st) {
  check_batch(nrhs);
  if (n) DISPATCH_B(prec, k_residual_b, ew_grid_b(n, nrhs), out, b, y, vs, n);
}

void blas_mr_update_b(int prec, const double* coef, size_t cs, void* x, void* r, const void* Ar, size_t vs, size_t n,
                      int nrhs, hipStream_t st) {
  check_batch(nrhs);
  DISPATCH_B(prec, k_mr_update_b, ew_grid_b(n, nrhs), coef, cs, x, r, Ar, vs, n);
}

}  // namespace wcmg

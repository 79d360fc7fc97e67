// BLAS-1 kernels for the Krylov solvers (GCR, BiCGStab, MR).
//
// Vectors are flat arrays of complex numbers in double or float storage;
// every reduction accumulates in double, first per wavefront with lane
// shuffles, then across the 4 wavefronts of a block in LDS; the last block
// of the grid to finish then sums the per-block partials in a fixed tree and
// writes the result to device memory, all in the one launch.  The grids
// depend only on the vector length, so results are bitwise reproducible run
// to run.
#include "blas_common.h"

namespace wcmg {

namespace {

using namespace blas_detail;

// complex vector in storage D from storage T (rounding to nearest)
template <typename D, typename T>
__global__ void k_convert(void* y, const void* x, size_t n) {
  GRID_STRIDE(i, n) st<D>(y, i, ld<T>(x, i));
}

template <typename T>
__global__ void k_zero(void* x, size_t n) {
  GRID_STRIDE(i, n) st<T>(x, i, mk(0.0, 0.0));
}
template <typename T>
__global__ void k_copy(void* y, const void* x, size_t n) {
  GRID_STRIDE(i, n) st<T>(y, i, ld<T>(x, i));
}
template <typename T>
__global__ void k_axpby(double ar, double ai, const void* x, double br, double bi, void* y, size_t n) {
  cpx<double> a = mk(ar, ai), b = mk(br, bi);
  GRID_STRIDE(i, n) st<T>(y, i, a * ld<T>(x, i) + b * ld<T>(y, i));
}
template <typename T>
__global__ void __launch_bounds__(kThreads) k_norm2(const void* x, size_t n, const RedOut o) {
  double v[1] = {0.0};
  GRID_STRIDE(i, n) {
    cpx<double> a = ld<T>(x, i);
    v[0] += a.r * a.r + a.i * a.i;
  }
  block_reduce<1>(v, o);
}
template <typename T>
__global__ void __launch_bounds__(kThreads) k_cdot(const void* x, const void* y, size_t n, const RedOut o) {
  double v[2] = {0.0, 0.0};
  GRID_STRIDE(i, n) {
    cpx<double> a = ld<T>(x, i), b = ld<T>(y, i);
    v[0] += a.r * b.r + a.i * b.i;
    v[1] += a.r * b.i - a.i * b.r;
  }
  block_reduce<2>(v, o);
}
template <typename T>
__global__ void __launch_bounds__(kThreads) k_cdot_norm(const void* x, const void* y, size_t n, const RedOut o) {
  double v[3] = {0.0, 0.0, 0.0};
  GRID_STRIDE(i, n) {
    cpx<double> a = ld<T>(x, i), b = ld<T>(y, i);
    v[0] += a.r * b.r + a.i * b.i;
    v[1] += a.r * b.i - a.i * b.r;
    v[2] += a.r * a.r + a.i * a.i;
  }
  block_reduce<3>(v, o);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_axpy_norm(double ar, double ai, const void* x, void* y, size_t n,
                                                        const RedOut o) {
  double v[1] = {0.0};
  cpx<double> a = mk(ar, ai);
  GRID_STRIDE(i, n) {
    cpx<double> b = ld<T>(y, i) + a * ld<T>(x, i);
    st<T>(y, i, b);
    cpx<double> bs = ld<T>(y, i);
    v[0] += bs.r * bs.r + bs.i * bs.i;
  }
  block_reduce<1>(v, o);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_bicg_update(double ar, double ai, double wr, double wi, const void* p,
                                                          const void* s, const void* t, void* x, void* r,
                                                          const void* rhat, size_t n, const RedOut o) {
  double v[3] = {0.0, 0.0, 0.0};
  cpx<double> a = mk(ar, ai), w = mk(wr, wi);
  GRID_STRIDE(i, n) {
    cpx<double> sv = ld<T>(s, i);
    st<T>(x, i, ld<T>(x, i) + a * ld<T>(p, i) + w * sv);
    st<T>(r, i, sv - w * ld<T>(t, i));
    cpx<double> rv = ld<T>(r, i), h = ld<T>(rhat, i);
    v[0] += rv.r * rv.r + rv.i * rv.i;
    v[1] += h.r * rv.r + h.i * rv.i;
    v[2] += h.r * rv.i - h.i * rv.r;
  }
  block_reduce<3>(v, o);
}

template <typename T>
__global__ void k_bicg_p(double br, double bi, double wr, double wi, const void* r, const void* v, void* p,
                         size_t n) {
  cpx<double> b = mk(br, bi), w = mk(wr, wi);
  GRID_STRIDE(i, n) st<T>(p, i, ld<T>(r, i) + b * (ld<T>(p, i) - w * ld<T>(v, i)));
}

// MR step with alpha = <Ar, r> / ||Ar||^2 read from coef = [re, im, ||Ar||^2]
template <typename T>
__global__ void k_mr_update_dev(const double* coef, void* x, void* r, const void* Ar, size_t n) {
  const double d = coef[2];
  cpx<double> a = d > 0.0 ? mk(coef[0] / d, coef[1] / d) : mk(0.0, 0.0);
  GRID_STRIDE(i, n) {
    st<T>(x, i, ld<T>(x, i) + a * ld<T>(r, i));
    st<T>(r, i, ld<T>(r, i) - a * ld<T>(Ar, i));
  }
}

template <typename T>
__global__ void k_mr_update(double ar, double ai, void* x, void* r, const void* Ar, size_t n) {
  cpx<double> a = mk(ar, ai);
  GRID_STRIDE(i, n) {
    st<T>(x, i, ld<T>(x, i) + a * ld<T>(r, i));
    st<T>(r, i, ld<T>(r, i) - a * ld<T>(Ar, i));
  }
}

}  // namespace

#define DISPATCH(prec, KERNEL, grid, ...)                                                       \
  do {                                                                                          \
    if ((prec) == WCMG_F64)                                                                     \
      hipLaunchKernelGGL(KERNEL<double>, grid, dim3(kThreads), 0, st, __VA_ARGS__);             \
    else                                                                                        \
      hipLaunchKernelGGL(KERNEL<float>, grid, dim3(kThreads), 0, st, __VA_ARGS__);              \
    HIPCHK(hipGetLastError());                                                                  \
  } while (0)


void blas_zero(int prec, void* x, size_t n, hipStream_t st) { DISPATCH(prec, k_zero, ew_grid(n), x, n); }
void blas_convert(int prec_dst, void* y, int prec_src, const void* x, size_t n, hipStream_t st) {
  const dim3 g = ew_grid(n);
  if (prec_dst == WCMG_F64 && prec_src == WCMG_F64)
    hipLaunchKernelGGL((k_convert<double, double>), g, dim3(kThreads), 0, st, y, x, n);
  else if (prec_dst == WCMG_F64)
    hipLaunchKernelGGL((k_convert<double, float>), g, dim3(kThreads), 0, st, y, x, n);
  else if (prec_src == WCMG_F64)
    hipLaunchKernelGGL((k_convert<float, double>), g, dim3(kThreads), 0, st, y, x, n);
  else
    hipLaunchKernelGGL((k_convert<float, float>), g, dim3(kThreads), 0, st, y, x, n);
  HIPCHK(hipGetLastError());
}
void blas_copy(int prec, void* y, const void* x, size_t n, hipStream_t st) {
  DISPATCH(prec, k_copy, ew_grid(n), y, x, n);
}
void blas_axpby(int prec, double ar, double ai, const void* x, double br, double bi, void* y, size_t n,
                hipStream_t st) {
  DISPATCH(prec, k_axpby, ew_grid(n), ar, ai, x, br, bi, y, n);
}
void blas_norm2(int prec, const void* x, size_t n, const RedOut& o, hipStream_t st) {
  DISPATCH(prec, k_norm2, red_grid(n), x, n, o);
}
void blas_cdot(int prec, const void* x, const void* y, size_t n, const RedOut& o, hipStream_t st) {
  DISPATCH(prec, k_cdot, red_grid(n), x, y, n, o);
}
void blas_cdot_norm(int prec, const void* x, const void* y, size_t n, const RedOut& o, hipStream_t st) {
  DISPATCH(prec, k_cdot_norm, red_grid(n), x, y, n, o);
}
void blas_axpy_norm(int prec, double ar, double ai, const void* x, void* y, size_t n, const RedOut& o,
                    hipStream_t st) {
  DISPATCH(prec, k_axpy_norm, red_grid(n), ar, ai, x, y, n, o);
}
void blas_bicg_update(int prec, double ar, double ai, double wr, double wi, const void* p, const void* s,
                      const void* t, void* x, void* r, const void* rhat, size_t n, const RedOut& o, hipStream_t st) {
  DISPATCH(prec, k_bicg_update, red_grid(n), ar, ai, wr, wi, p, s, t, x, r, rhat, n, o);
}
void blas_bicg_p(int prec, double br, double bi, double wr, double wi, const void* r, const void* v, void* p,
                 size_t n, hipStream_t st) {
  DISPATCH(prec, k_bicg_p, ew_grid(n), br, bi, wr, wi, r, v, p, n);
}
void blas_mr_update(int prec, double ar, double ai, void* x, void* r, const void* Ar, size_t n, hipStream_t st) {
  DISPATCH(prec, k_mr_update, ew_grid(n), ar, ai, x, r, Ar, n);
}

void blas_mr_update_dev(int prec, const double* coef, void* x, void* r, const void* Ar, size_t n, hipStream_t st) {
  DISPATCH(prec, k_mr_update_dev, ew_grid(n), coef, x, r, Ar, n);
}

}  // namespace wcmg

// Small kernels: residual-norm finalisation and stop test (Alg. 2 E update
// and loop condition), identity fill for the explicit Q, copies.

#include "finalize_body.h"
#include "rrf_internal.h"

namespace rrf {
namespace {

// The one-workgroup finalisation (finalize_body.h) from plain partials.
__global__ __launch_bounds__(256) void finalize_kernel(const double* np, FinalizeArgs f) {
  finalize_plain(np, f);
}

// [I; 0], and nw words from gsrc to gdst (the first workgroup).
template <typename T>
__global__ void fill_identity_kernel(T* Q, int64_t ldq, int64_t m, int64_t k,
                                     const unsigned* gsrc, unsigned* gdst, int nw) {
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int i = (int)threadIdx.x; i < nw; i += (int)blockDim.x) gdst[i] = gsrc[i];
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= m) return;
  for (int64_t c = blockIdx.y; c < k; c += gridDim.y)
    Q[r + c * ldq] = (r == c) ? T(1) : T(0);
}

template <typename T>
__global__ void copy_kernel(const T* src, int64_t lds, T* dst, int64_t ldd,
                            int64_t rows, int64_t cols) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  for (int64_t c = blockIdx.y; c < cols; c += gridDim.y)
    dst[r + c * ldd] = src[r + c * lds];
}

template <typename Ts, typename Td>
__global__ void convert_kernel(const Ts* src, int64_t lds, Td* dst, int64_t ldd,
                               int64_t rows, int64_t cols) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  for (int64_t c = blockIdx.y; c < cols; c += gridDim.y)
    dst[r + c * ldd] = (Td)src[r + c * lds];
}

// A caller's reflector to the plan's binary64 V (m x bp) and T (64 rows, bp
// columns), zero past its b columns, in one launch (grid rows x bp).
template <typename T>
__global__ __launch_bounds__(256) void reflector_in_kernel(const T* V, int64_t ldv, const T* Tm,
                                                           int64_t ldt, int64_t m, int b,
                                                           double* Vw, int64_t ldw, double* Tw) {
  const int c = (int)blockIdx.y;
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r < m) Vw[r + c * ldw] = c < b ? (double)V[r + (int64_t)min(c, b - 1) * ldv] : 0.0;
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    const int i = (int)threadIdx.x;
    Tw[i + c * 64] = (i < b && c < b) ? (double)Tm[i + (int64_t)c * ldt] : 0.0;
  }
}

// A factored panel to the caller's V (m x b), T (b x b) and tau, and the run
// state to its pinned copy, in one launch (grid rows x b).
template <typename T>
__global__ __launch_bounds__(256) void panel_out_kernel(const double* Vw, int64_t ldw,
                                                        const double* Tw, const double* tauw,
                                                        int64_t m, int b, T* V, int64_t ldv,
                                                        T* Tm, int64_t ldt, T* tau,
                                                        const DevState* st, DevState* h) {
  const int c = (int)blockIdx.y;
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r < m) V[r + c * ldv] = (T)Vw[r + c * ldw];
  if (blockIdx.x == 0) {
    const int i = (int)threadIdx.x;
    if (i < b) Tm[i + c * ldt] = (T)Tw[i + c * 64];
    if (i == 0) tau[c] = (T)tauw[c];
    if (c == 0 && i == 0) *h = *st;
  }
}

// The run state and the traces (blk blocks, the estimates of nspec) to pinned
// host memory.
__global__ __launch_bounds__(256) void export_kernel(const DevState* st, DevState* h,
                                                     const double* tt, const double* ts,
                                                     const double* tp, int blk, int nspec,
                                                     double* th, size_t stride) {
  if (threadIdx.x == 0) {
    DevState v = *st;
    v.barrier_err = __hip_atomic_load(&st->barrier_err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *h = v;
  }
  for (int i = (int)threadIdx.x; i < blk; i += 256) {
    th[i] = tt[i];
    th[stride + i] = ts[i];
    if (i < nspec) th[2 * stride + i] = tp[i];
  }
}

// Rows [r0, r0 + b) of b columns to rows [0, b), one thread per column (b at
// most 64; a row is read before a thread writes it or any row past it).
__global__ __launch_bounds__(64) void lift_rows_kernel(double* T, int64_t ldt, int64_t r0, int b) {
  const int c = (int)threadIdx.x;
  if (c >= b) return;
  double* t = T + c * ldt;
  for (int i = 0; i < b; ++i) t[i] = t[r0 + i];
}

}  // namespace

hipError_t launch_finalize(const double* normpart, int nparts, DevState* st,
                           DevState* mirror, double* trace_trail, double* trace_sub, int block,
                           int64_t k_after, int64_t k_cap, int mode,
                           double tol, int init, hipStream_t s) {
  FinalizeArgs f{};
  f.nparts = nparts; f.st = st; f.mirror = mirror; f.tt = trace_trail; f.ts = trace_sub; f.block = block;
  f.k_after = k_after; f.k_cap = k_cap; f.mode = mode; f.tol = tol; f.init = init;
  hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(256), 0, s, normpart, f);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fill_identity(T* Q, int64_t ldq, int64_t m, int64_t k, const void* gsrc,
                                void* gdst, size_t gbytes, hipStream_t s) {
  if (m <= 0 || k <= 0) return hipSuccess;
  dim3 grid((unsigned)ceil_div(m, 256), (unsigned)(k < 4096 ? k : 4096));
  hipLaunchKernelGGL(fill_identity_kernel<T>, grid, dim3(256), 0, s, Q, ldq, m, k,
                     (const unsigned*)gsrc, (unsigned*)gdst, (int)(gbytes / 4));
  return hipGetLastError();
}

template <typename T>
hipError_t launch_copy(const T* src, int64_t lds, T* dst, int64_t ldd,
                       int64_t rows, int64_t cols, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  dim3 grid((unsigned)ceil_div(rows, 256), (unsigned)(cols < 4096 ? cols : 4096));
  hipLaunchKernelGGL(copy_kernel<T>, grid, dim3(256), 0, s, src, lds, dst, ldd,
                     rows, cols);
  return hipGetLastError();
}

template <typename Ts, typename Td>
hipError_t launch_convert(const Ts* src, int64_t lds, Td* dst, int64_t ldd,
                          int64_t rows, int64_t cols, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  dim3 grid((unsigned)ceil_div(rows, 256), (unsigned)(cols < 4096 ? cols : 4096));
  hipLaunchKernelGGL((convert_kernel<Ts, Td>), grid, dim3(256), 0, s, src, lds,
                     dst, ldd, rows, cols);
  return hipGetLastError();
}

template hipError_t launch_fill_identity<double>(double*, int64_t, int64_t, int64_t, const void*, void*, size_t, hipStream_t);
template hipError_t launch_copy<float>(const float*, int64_t, float*, int64_t, int64_t, int64_t, hipStream_t);
template hipError_t launch_copy<double>(const double*, int64_t, double*, int64_t, int64_t, int64_t, hipStream_t);
template hipError_t launch_convert<double, float>(const double*, int64_t, float*, int64_t, int64_t, int64_t, hipStream_t);

template <typename T>
hipError_t launch_reflector_in(const T* V, int64_t ldv, const T* Tm, int64_t ldt, int64_t m,
                               int b, int bp, double* Vw, int64_t ldw, double* Tw,
                               hipStream_t s) {
  hipLaunchKernelGGL(reflector_in_kernel<T>, dim3((unsigned)ceil_div(m, 256), (unsigned)bp),
                     dim3(256), 0, s, V, ldv, Tm, ldt, m, b, Vw, ldw, Tw);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_panel_out(const double* Vw, int64_t ldw, const double* Tw, const double* tauw,
                            int64_t m, int b, T* V, int64_t ldv, T* Tm, int64_t ldt, T* tau,
                            const DevState* st, DevState* h, hipStream_t s) {
  hipLaunchKernelGGL(panel_out_kernel<T>, dim3((unsigned)ceil_div(m, 256), (unsigned)b),
                     dim3(256), 0, s, Vw, ldw, Tw, tauw, m, b, V, ldv, Tm, ldt, tau, st, h);
  return hipGetLastError();
}

template hipError_t launch_reflector_in<float>(const float*, int64_t, const float*, int64_t, int64_t, int, int, double*, int64_t, double*, hipStream_t);
template hipError_t launch_reflector_in<double>(const double*, int64_t, const double*, int64_t, int64_t, int, int, double*, int64_t, double*, hipStream_t);
template hipError_t launch_panel_out<float>(const double*, int64_t, const double*, const double*, int64_t, int, float*, int64_t, float*, int64_t, float*, const DevState*, DevState*, hipStream_t);
template hipError_t launch_panel_out<double>(const double*, int64_t, const double*, const double*, int64_t, int, double*, int64_t, double*, int64_t, double*, const DevState*, DevState*, hipStream_t);

hipError_t launch_export(const DevState* st, DevState* h, const double* tt, const double* ts,
                         const double* tp, int blk, int nspec, double* th, size_t stride,
                         hipStream_t s) {
  hipLaunchKernelGGL(export_kernel, dim3(1), dim3(256), 0, s, st, h, tt, ts, tp, blk, nspec, th,
                     stride);
  return hipGetLastError();
}

hipError_t launch_lift_rows(double* T, int64_t ldt, int64_t r0, int b, hipStream_t s) {
  if (b < 1 || b > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(lift_rows_kernel, dim3(1), dim3(64), 0, s, T, ldt, r0, b);
  return hipGetLastError();
}

}  // namespace rrf

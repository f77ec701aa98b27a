// Spectral-norm estimate of the rows not yet in B (the alternative stopping
// test of Sec. 3, proposed as future work in the conclusion), and the scaled
// identity that power iterations use as their W factor.
//
// With Bt the trailing rows after a block and Y = Bt Omega' the sample of
// the next sketch block (first min(b, 64) columns), Z = Bt^T Y, the estimate
// is the largest eigenvalue of the pencil (Z^T Z, Y^T Y):
//   max over x in span(Y) of ||Bt^T x||^2 / ||x||^2
// (one step of randomized subspace iteration; a lower bound of ||Bt||_2^2,
// exact when rank(Bt) <= the block width).  Y and Z arrive from the gather
// and the reduce kernel (Z as split partials); here:
//   spec_gram_kernel   partial Gram matrices G_Y = Y^T Y and G_Z = Z^T Z
//                      over row ranges, f64 MFMA, values scaled by ||A||_F
//                      (1/sqrt(E0) for Y, 1/E0 for Z) so nothing overflows;
//   spec_sum_kernel    sums the partials in a fixed order;
//   spec_finish_kernel one workgroup: L = chol(G_Y + delta I), M = L^-1 G_Z
//                      L^-T, and the largest eigenvalue of M by repeated
//                      squaring, then a Rayleigh quotient; writes E_spec
//                      (times E0) to the run state and the trace.  16 x 16
//                      blocks: the diagonal blocks of L in one wavefront's
//                      registers, everything else tile products on f64 MFMA
//                      (12 squarings of 64 x 64, 64 MFMAs a wavefront each).
// Measured at 3001 x 1733 fp64, b = 48, per estimate: the estimate's kernels
// 780 -> 83 us (finish 410 -> 60: every step had run on LDS entries, most of
// them in one wavefront; Gram sums 366 -> 19: too few workgroups, one load in
// flight).

#include <utility>

#include "lanes.h"
#include "mfma.h"
#include "rrf_internal.h"

namespace rrf {
namespace {

constexpr int kSpecRows = 64;   // rows per staged chunk

template <typename T>
__global__ __launch_bounds__(256) void spec_gram_kernel(SpecGramArgs<T> a) {
  __shared__ double X[kSpecRows][65];
  const int t = threadIdx.x;
  const int lane = t & 63, wv = t >> 6, l16 = lane >> 4, m16 = lane & 15;
  const int w = (int)blockIdx.x;
  const bool isY = w < a.gy;
  const int64_t rows = isY ? a.my : a.nz;
  const int64_t rpw = isY ? a.rows_per_wg_y : a.rows_per_wg_z;
  const int64_t r_begin = (int64_t)(isY ? w : w - a.gy) * rpw;
  const int64_t r_end = min(rows, r_begin + rpw);
  const double E0 = a.st->E0;
  const double sc = E0 > 0.0 ? (isY ? 1.0 / sqrt(E0) : 1.0 / E0) : 0.0;

  d4_t acc[4];
#pragma unroll
  for (int ct = 0; ct < 4; ++ct) acc[ct] = d4_t{0.0, 0.0, 0.0, 0.0};
  for (int64_t r0 = r_begin; r0 < r_end; r0 += kSpecRows) {
    __syncthreads();
    if (isY) {
      // Column-major Y: thread t loads row t % 64 of columns t / 64 + 4 i.
      const int rr = t % 64, c0 = t / 64;
      const int64_t r = r0 + rr;
      const bool ok = r < r_end;
      double v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int c = c0 + 4 * i;
        v[i] = (ok && c < a.bp) ? a.Y[r + (int64_t)c * a.ldy] : 0.0;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) X[rr][c0 + 4 * i] = sc * v[i];
    } else {
      // Row-major Z partials Z_s[row * bp + c]: thread t loads column t % 64
      // of rows t / 64 + 4 i, summed over the splits in split order, 32 loads
      // in flight (clamped split and row, surplus values not added).
      const int cc = t % 64, q0 = t / 64;
      constexpr int RB = 4, SB = 8;
#pragma unroll 1
      for (int i0 = 0; i0 < 16; i0 += RB) {
        double z[RB];
        const T* zp[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          z[i] = 0.0;
          const int64_t r = r0 + q0 + 4 * (i0 + i);
          zp[i] = a.Z + (r < r_end ? r : r_begin) * a.bp + (cc < a.bp ? cc : 0);
        }
        for (int s0 = 0; s0 < a.nsplit; s0 += SB) {
          T v[RB][SB];
#pragma unroll
          for (int u = 0; u < SB; ++u)
#pragma unroll
            for (int i = 0; i < RB; ++i)
              v[i][u] = zp[i][(int64_t)min(s0 + u, a.nsplit - 1) * a.split_stride];
#pragma unroll
          for (int u = 0; u < SB; ++u)
            if (s0 + u < a.nsplit)
#pragma unroll
              for (int i = 0; i < RB; ++i) z[i] += (double)v[i][u];
        }
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          const int rr = q0 + 4 * (i0 + i);
          X[rr][cc] = (r0 + rr < r_end && cc < a.bp) ? sc * z[i] : 0.0;
        }
      }
    }
    __syncthreads();
    // G[16 pt + m][16 ct + n] += sum_r X[r][16 pt + m] X[r][16 ct + n],
    // pt = this wavefront, over the chunk's rows in K steps of 4.
#pragma unroll 4
    for (int s4 = 0; s4 < kSpecRows / 4; ++s4) {
      const double av = X[4 * s4 + l16][16 * wv + m16];
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
        acc[ct] = Mfma<double>::op(av, X[4 * s4 + l16][16 * ct + m16], acc[ct]);
    }
  }
  // Lane holds G[16 wv + l16 + 4 i][16 ct + m16].
  double* out = a.part + (int64_t)w * 4096;
#pragma unroll
  for (int ct = 0; ct < 4; ++ct)
#pragma unroll
    for (int i = 0; i < 4; ++i) out[(16 * wv + l16 + 4 * i) * 64 + 16 * ct + m16] = acc[ct][i];
}

// sum[w][e] = the partials of one Gram matrix (w = 0: Y, 1: Z) added in
// workgroup order; grid 32 x 256 threads, one entry each.
__global__ __launch_bounds__(256) void spec_sum_kernel(SpecFinishArgs a, double* sum) {
  const int e = (int)(blockIdx.x * 256 + threadIdx.x);   // < 2 x 4096
  const bool isY = e < 4096;
  const double* p = a.part + (isY ? 0 : (int64_t)a.gy * 4096) + (e & 4095);
  const int nw = isY ? a.gy : a.gz;
  double s = 0.0;
  for (int w0 = 0; w0 < nw; w0 += 16) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[(int64_t)min(w0 + u, nw - 1) * 4096];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (w0 + u < nw) s += v[u];
  }
  sum[e] = s;
}

// Cholesky of a 16 x 16 block (pivots at least delta) with the inverse of its
// factor, on one wavefront: lane (h, k) holds rows 4 h + i of column k; row j
// of L^-1 goes to inv when it is final.  (As the blocks of the Gram panel.)
template <int J>
__device__ __forceinline__ void chol16_step(double (&f)[4], double (&aux)[4], double* inv,
                                            const double delta, const int h, const int k) {
  constexpr int QJ = J / 4, IJ = J % 4;
  const double piv = fmax(lane_value<16 * QJ + J>(f[IJ]), delta);
  const double y = fast_rsqrt(piv);
  const double fc = row_of<QJ>(f[IJ]) * (y * y);
  const double ak = row_of<QJ>(aux[IJ]) * y;
  if (h == QJ) inv[J * 17 + k] = ak;
  const double ac = ak * y;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double fr = row_lane<J>(f[i]);
    f[i] = fma(-fr, fc, f[i]);
    aux[i] = fma(-fr, ac, aux[i]);
  }
}
template <int... Js>
__device__ __forceinline__ void chol16(double (&f)[4], double (&aux)[4], double* inv,
                                       const double delta, const int h, const int k,
                                       std::integer_sequence<int, Js...>) {
  (chol16_step<Js>(f, aux, inv, delta, h, k), ...);
}

constexpr int kSl = 66;   // row stride of a 64 x 64 matrix in LDS

__global__ __launch_bounds__(256) void spec_finish_kernel(SpecFinishArgs a, const double* sum) {
  __shared__ double A[64 * kSl];   // G_Y, its factor R above the diagonal; then powers
  __shared__ double B[64 * kSl];   // G_Z, X = L^-1 G_Z; then powers
  __shared__ double M[64 * kSl];   // X^T, then M
  __shared__ double inv[4][16 * 17];
  __shared__ double red[4];
  __shared__ int jmax;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6, g = lane >> 4, m16 = lane & 15;
  {
    double v[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) v[q] = sum[t + 256 * q];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int e = t + 256 * q;
      A[(e / 64) * kSl + e % 64] = v[q];
      B[(e / 64) * kSl + e % 64] = v[16 + q];
    }
  }
  __syncthreads();
  // delta = 64 u max diag(G_Y); an all-zero G_Y means Y = 0: estimate 0.
  double dmax = A[lane * kSl + lane];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, off));
  dmax = fmax(dmax, 0.0);
  if (!(dmax > 0.0)) {   // uniform: every wavefront has the same diagonal
    if (t == 0) {
      a.st->E_spec = 0.0;
      if (a.block >= 0) a.trace[a.block] = 0.0;
    }
    return;
  }
  const double delta = 64.0 * 1.1102230246251565e-16 * dmax;
  const d4_t zero = d4_t{0.0, 0.0, 0.0, 0.0};
  // c + op(A) B of 16 x 16 tiles with row stride la, lb; D[g + 4 i][m16].
  auto mm = [&](const double* P, const int la, const bool at, const double* Q, const int lb,
                d4_t c) __attribute__((always_inline)) -> d4_t {
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
      const int kk = 4 * s4 + g;
      c = Mfma<double>::op(at ? P[kk * la + m16] : P[m16 * la + kk], Q[kk * lb + m16], c);
    }
    return c;
  };
  // G_Y + delta I = L L^T by 16-column blocks, R = L^T in A's upper blocks:
  // R_JK = L_JJ^-1 F_JK, F_KL -= R_JK^T R_JL.
#pragma unroll 1
  for (int J = 0; J < 4; ++J) {
    if (wv == 0) {
      double f[4], aux[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * g + i;
        f[i] = A[(16 * J + r) * kSl + 16 * J + m16] + (r == m16 ? delta : 0.0);
        aux[i] = r == m16 ? 1.0 : 0.0;
      }
      chol16(f, aux, inv[J], delta, g, m16, std::make_integer_sequence<int, 16>{});
    }
    __syncthreads();
    const int nk = 3 - J;
    if (wv < nk) {
      double* F = A + 16 * J * kSl + 16 * (J + 1 + wv);
      const d4_t d = mm(inv[J], 17, false, F, kSl, zero);
#pragma unroll
      for (int i = 0; i < 4; ++i) F[(g + 4 * i) * kSl + m16] = d[i];
    }
    __syncthreads();
    for (int u = wv; u < nk * (nk + 1) / 2; u += 4) {
      int v = u, ti = 0;
      while (v >= nk - ti) {
        v -= nk - ti;
        ++ti;
      }
      const int K = J + 1 + ti, N = K + v;
      const d4_t d = mm(A + 16 * J * kSl + 16 * K, kSl, true, A + 16 * J * kSl + 16 * N, kSl, zero);
#pragma unroll
      for (int i = 0; i < 4; ++i) A[(16 * K + g + 4 * i) * kSl + 16 * N + m16] -= d[i];
    }
    __syncthreads();
  }
  // S <- L^-1 S by block rows (wavefront w: the 16 columns of block w, no
  // barrier): S_J = L_JJ^-1 (S_J - sum_{I < J} R_IJ^T S_I); the result also
  // goes, transposed, to D.
  auto solve = [&](double* S, double* D) __attribute__((always_inline)) {
#pragma unroll 1
    for (int J = 0; J < 4; ++J) {
      double* Sj = S + 16 * J * kSl + 16 * wv;
      d4_t d = zero;
      for (int I = 0; I < J; ++I)
        d = mm(A + 16 * I * kSl + 16 * J, kSl, true, S + 16 * I * kSl + 16 * wv, kSl, d);
      d4_t x = zero;   // d's layout is the next product's operand
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4)
        x = Mfma<double>::op(inv[J][m16 * 17 + 4 * s4 + g],
                             Sj[(4 * s4 + g) * kSl + m16] - d[s4], x);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        Sj[(g + 4 * i) * kSl + m16] = x[i];
        if (D) D[(16 * wv + m16) * kSl + 16 * J + g + 4 * i] = x[i];
      }
      // The wavefront's own LDS writes are read by its other lanes next.
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
  };
  solve(B, M);            // X = L^-1 G_Z; M = X^T
  __syncthreads();
  solve(M, nullptr);      // M = L^-1 X^T (symmetric)
  __syncthreads();
  // Repeated squaring P <- P^2 / trace(P^2) (P stays positive semidefinite),
  // 12 times: P ~ M^4096, whose columns lie along the top eigenvector.
  // Wavefront w computes block row w; P is read from src and written to dst.
  const double* src = M;
  double* dst = A;
#pragma unroll 1
  for (int it = 0; it < 12; ++it) {
    d4_t o[4] = {zero, zero, zero, zero};
#pragma unroll 4
    for (int s4 = 0; s4 < 16; ++s4) {
      const double av = src[(16 * wv + m16) * kSl + 4 * s4 + g];
#pragma unroll
      for (int c = 0; c < 4; ++c)
        o[c] = Mfma<double>::op(av, src[(4 * s4 + g) * kSl + 16 * c + m16], o[c]);
    }
    double tr = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) tr += (c == wv && g + 4 * i == m16) ? o[c][i] : 0.0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off);
    if (lane == 0) red[wv] = tr;
    __syncthreads();
    const double s = (red[0] + red[1]) + (red[2] + red[3]);
    const double sc = s > 0.0 ? 1.0 / s : 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) dst[(16 * wv + g + 4 * i) * kSl + 16 * c + m16] = o[c][i] * sc;
    __syncthreads();
    src = dst;
    dst = dst == A ? B : A;
  }
  // v = the column of P with the largest diagonal entry; estimate
  // v^T M v / v^T v.
  if (wv == 0) {
    double best = src[lane * kSl + lane];
    int jb = lane;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double ob = __shfl_xor(best, off);
      const int oj = __shfl_xor(jb, off);
      if (ob > best || (ob == best && oj < jb)) {
        best = ob;
        jb = oj;
      }
    }
    if (lane == 0) jmax = jb;
  }
  __syncthreads();
  const int jb = jmax;
  if (wv == 0) {
    const double vc = src[lane * kSl + jb];
    double m4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int i = 0; i < 64; i += 4)
#pragma unroll
      for (int u = 0; u < 4; ++u) m4[u] += M[(i + u) * kSl + lane] * src[(i + u) * kSl + jb];
    double num = vc * ((m4[0] + m4[1]) + (m4[2] + m4[3])), den = vc * vc;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      num += __shfl_xor(num, off);
      den += __shfl_xor(den, off);
    }
    if (lane == 0) {
      const double lam = den > 0.0 ? num / den : 0.0;
      const double E = fmax(lam, 0.0) * a.st->E0;
      a.st->E_spec = E;
      if (a.block >= 0) a.trace[a.block] = E;
    }
  }
}

__global__ void scaled_identity_kernel(double* Tm, int64_t ldt, const DevState* st) {
  const int i = threadIdx.x % 64, j = threadIdx.x / 64;
  const double E0 = st->E0;
  const double d = E0 > 0.0 ? 1.0 / E0 : 0.0;
  for (int jj = j; jj < 64; jj += 4) Tm[i + jj * ldt] = (i == jj) ? d : 0.0;
}

}  // namespace

template <typename T>
hipError_t launch_spec_gram(SpecGramArgs<T>* ap, hipStream_t s) {
  SpecGramArgs<T>& a = *ap;
  if (a.bp < 1 || a.bp > 64) return hipErrorInvalidValue;
  a.gy = (int)std::max<int64_t>(1, std::min<int64_t>(kMaxSpecWGs / 2, ceil_div(a.my, kSpecRows)));
  a.rows_per_wg_y = round_up(ceil_div(std::max<int64_t>(a.my, 1), a.gy), kSpecRows);
  a.gy = (int)std::max<int64_t>(1, ceil_div(std::max<int64_t>(a.my, 1), a.rows_per_wg_y));
  a.gz = (int)std::max<int64_t>(1, std::min<int64_t>(kMaxSpecWGs / 2, ceil_div(a.nz, kSpecRows)));
  a.rows_per_wg_z = round_up(ceil_div(std::max<int64_t>(a.nz, 1), a.gz), kSpecRows);
  a.gz = (int)std::max<int64_t>(1, ceil_div(std::max<int64_t>(a.nz, 1), a.rows_per_wg_z));
  hipLaunchKernelGGL((spec_gram_kernel<T>), dim3((unsigned)(a.gy + a.gz)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_spec_finish(const SpecFinishArgs& a, hipStream_t s) {
  // The sums follow the partials in their buffer.
  double* sum = a.part + (int64_t)(a.gy + a.gz) * 4096;
  hipLaunchKernelGGL(spec_sum_kernel, dim3(32), dim3(256), 0, s, a, sum);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(spec_finish_kernel, dim3(1), dim3(256), 0, s, a, sum);
  return hipGetLastError();
}

hipError_t launch_scaled_identity(double* Tm, int64_t ldt, const DevState* st, hipStream_t s) {
  hipLaunchKernelGGL(scaled_identity_kernel, dim3(1), dim3(256), 0, s, Tm, ldt, st);
  return hipGetLastError();
}

template hipError_t launch_spec_gram<float>(SpecGramArgs<float>*, hipStream_t);
template hipError_t launch_spec_gram<double>(SpecGramArgs<double>*, hipStream_t);

}  // namespace rrf

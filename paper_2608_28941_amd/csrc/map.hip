// GaLore subspace-consistency map (Sec. 7): a low-rank optimizer state M
// (r_old x n) expressed in the basis Q_old is carried to the next basis as
// out = Q_new^T (Q_old M) = C M with C = Q_new^T Q_old (r_new x r_old).
//
// Three launches, MFMA 16x16x4 in the plan's dtype:
//   map_tn_kernel   C_s = Q_new[rows of split s]^T Q_old[rows of split s]
//                   (the reduction over the m rows is split so that the small
//                   r_new x r_old output fills the device);
//   map_sum_kernel  C^T = sum_s C_s^T in a fixed order (deterministic);
//   map_tn_kernel   out = (C^T)^T M, the same product.
// Both products contract the index that is contiguous in memory, so operands
// move in 16-byte packs along it from HBM to LDS ([output index][k]) to the
// registers: a pack feeds the K steps of 4 (f32) or 2 (f64) MFMAs, the K
// order permuted alike on both sides.  A workgroup computes a TI x 64 tile of
// the output, a wavefront TI/2 x 32 of it, from double-buffered chunks (one
// barrier each).  The MFMA runs in the transposed frame (its output rows
// index the output's columns), so the 16 lanes of an output column write 16
// consecutive rows of the column-major result.
//
// Bound: MFMA.  4096 x (512, 448), n = 11008, f32 (7 GFLOP): 87 us for the
// three launches, against 138 with a 64 x 64 tile, one scalar LDS read per
// operand and two barriers per chunk (and operand loads behind per-value
// branches).

#include <type_traits>

#include "mfma.h"
#include "rrf_internal.h"

namespace rrf {
namespace {

constexpr int kMapTJ = 64;   // output columns per workgroup

// Values of a 16-byte pack, and the chunk of the contracted index.
template <typename T> constexpr int map_vec() { return 16 / (int)sizeof(T); }
template <typename T> constexpr int map_chunk() { return 128 / (int)sizeof(T); }

template <typename T>
struct alignas(16) MapPack {
  T v[map_vec<T>()];
};

// Dpart_s[i + j ldd] = sum over k of split s of A[k + i lda] B[k + j ldb],
// i < M, j < N; grid (ceil(M / TI) x ceil(N / 64) tiles, splits of
// rows_per_split, a multiple of the chunk).  ALIGNED: A, B, lda and ldb allow 16-byte packs.
template <typename T, int TI, bool ALIGNED>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 3 : 2) void map_tn_kernel(const T* A, int64_t lda, const T* B,
                                                        int64_t ldb, int64_t M, int64_t N,
                                                        int64_t K, int64_t rows_per_split,
                                                        T* Dpart, int64_t ldd,
                                                        int64_t split_stride) {
  typedef typename Mfma<T>::acc_t acc_t;
  typedef MapPack<T> pack_t;
  constexpr int VEC = map_vec<T>();
  constexpr int KC = map_chunk<T>();       // 8 packs
  constexpr int NP = KC / VEC;             // packs per row of a chunk (8)
  constexpr int PA = TI * NP / 256;        // packs per thread
  constexpr int PB = kMapTJ * NP / 256;
  constexpr int WI = TI / 32;              // 16-row tiles of a wavefront, along i
  // Rows of 8 packs, pack p of row r at p ^ (r % 8): reads of one pack column
  // over 16 rows and writes of whole rows are both free of bank conflicts, and
  // three workgroups fit a compute unit.
  __shared__ pack_t As[2][TI * NP];
  __shared__ pack_t Bs[2][kMapTJ * NP];
  auto at = [](int r, int p) __attribute__((always_inline)) { return r * NP + (p ^ (r & 7)); };
  const int t = threadIdx.x;
  const int lane = t & 63, wv = t >> 6, g = lane >> 4, m16 = lane & 15;
  const int wi = (wv & 1) * (TI / 2), wj = (wv >> 1) * 32;
  const unsigned nti = (unsigned)((M + TI - 1) / TI);
  const int64_t i0 = (int64_t)(blockIdx.x % nti) * TI, j0 = (int64_t)(blockIdx.x / nti) * kMapTJ;
  const int64_t k_begin = (int64_t)blockIdx.y * rows_per_split;
  const int64_t k_end = min(K, k_begin + rows_per_split);
  // Staging: pack t % 8 of output index t / 8 + 32 q.
  const int pk = t % NP, pr = t / NP;
  acc_t acc[2][WI];
#pragma unroll
  for (int jt = 0; jt < 2; ++jt)
#pragma unroll
    for (int it = 0; it < WI; ++it) acc[jt][it] = Mfma<T>::zero();
  pack_t pa[PA], pb[PB];
  // Whole chunks load unconditional packs; the last one of a ragged K (and
  // every chunk of unaligned operands) clamped single values, zero past the
  // end.  Output rows and columns past M and N read clamped addresses and are
  // not stored.
  const T* Ap[PA];
  const T* Bp[PB];
#pragma unroll
  for (int q = 0; q < PA; ++q) Ap[q] = A + min(i0 + pr + 32 * q, M - 1) * lda;
#pragma unroll
  for (int q = 0; q < PB; ++q) Bp[q] = B + min(j0 + pr + 32 * q, N - 1) * ldb;
  auto load_packs = [&](int64_t k0) __attribute__((always_inline)) {
    const int64_t k = k0 + VEC * pk;
#pragma unroll
    for (int q = 0; q < PA; ++q) pa[q] = *reinterpret_cast<const pack_t*>(Ap[q] + k);
#pragma unroll
    for (int q = 0; q < PB; ++q) pb[q] = *reinterpret_cast<const pack_t*>(Bp[q] + k);
  };
  auto load_values = [&](int64_t k0) __attribute__((always_inline)) {
    const int64_t k = k0 + VEC * pk;
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      const int64_t kc = min(k + v, k_end - 1);
#pragma unroll
      for (int q = 0; q < PA; ++q) pa[q].v[v] = Ap[q][kc];
#pragma unroll
      for (int q = 0; q < PB; ++q) pb[q].v[v] = Bp[q][kc];
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      const bool in = k + v < k_end;
#pragma unroll
      for (int q = 0; q < PA; ++q) pa[q].v[v] = in ? pa[q].v[v] : T(0);
#pragma unroll
      for (int q = 0; q < PB; ++q) pb[q].v[v] = in ? pb[q].v[v] : T(0);
    }
  };
  auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < PA; ++q) As[buf][at(pr + 32 * q, pk)] = pa[q];
#pragma unroll
    for (int q = 0; q < PB; ++q) Bs[buf][at(pr + 32 * q, pk)] = pb[q];
  };
  // D[j][i] of the chunk in buffer cur: lane (g, m) supplies k = 4 VEC u +
  // VEC g + h at K step h of pack u on both sides.
  auto compute = [&](int cur) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NP / 4; ++u) {
      pack_t bo[2], ao[WI];
#pragma unroll
      for (int jt = 0; jt < 2; ++jt)
        bo[jt] = Bs[cur][at(wj + 16 * jt + m16, 4 * u + g)];
#pragma unroll
      for (int it = 0; it < WI; ++it)
        ao[it] = As[cur][at(wi + 16 * it + m16, 4 * u + g)];
#pragma unroll
      for (int h = 0; h < VEC; ++h)
#pragma unroll
        for (int jt = 0; jt < 2; ++jt)
#pragma unroll
          for (int it = 0; it < WI; ++it)
            acc[jt][it] = Mfma<T>::op(bo[jt].v[h], ao[it].v[h], acc[jt][it]);
    }
  };
  if (k_begin < k_end) {
    // The whole chunks' loop has no branch inside (a branch between the two
    // forms of the loads made the compiler wait for them at the join).
    int cur = 0;
    int64_t k0 = k_begin;
    if (ALIGNED && k0 + KC <= k_end) {
      load_packs(k0);
      stage(0);
      __syncthreads();
      for (k0 += KC; k0 + KC <= k_end; k0 += KC) {
        load_packs(k0);
        compute(cur);
        stage(cur ^ 1);
        __syncthreads();
        cur ^= 1;
      }
    } else {
      load_values(k0);
      stage(0);
      __syncthreads();
      k0 += KC;
    }
    for (; k0 < k_end; k0 += KC) {
      load_values(k0);
      compute(cur);
      stage(cur ^ 1);
      __syncthreads();
      cur ^= 1;
    }
    compute(cur);
  }
  // Lane (g, m16) item q holds D[i0 + wi + 16 it + m16][j0 + wj + 16 jt + drow(g, q)].
  T* D = Dpart + (int64_t)blockIdx.y * split_stride;
#pragma unroll
  for (int it = 0; it < WI; ++it) {
    const int64_t i = i0 + wi + 16 * it + m16;
    if (i >= M) continue;
#pragma unroll
    for (int jt = 0; jt < 2; ++jt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t j = j0 + wj + 16 * jt + Mfma<T>::drow(g, q);
        if (j < N) D[i + j * ldd] = acc[jt][it][q];
      }
  }
}

// C[e] = sum_s Cpart_s[e], e < count, in split order.
template <typename T>
__global__ void map_sum_kernel(const T* Cpart, int nsplit, int64_t split_stride, T* C,
                               int64_t count) {
  constexpr int ZB = 8;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= count) return;
  double s = 0.0;
  for (int q0 = 0; q0 < nsplit; q0 += ZB) {
    T v[ZB];
#pragma unroll
    for (int u = 0; u < ZB; ++u) v[u] = Cpart[(int64_t)min(q0 + u, nsplit - 1) * split_stride + e];
#pragma unroll
    for (int u = 0; u < ZB; ++u)
      if (q0 + u < nsplit) s += (double)v[u];
  }
  C[e] = (T)s;
}

// D = A^T B in nsplit splits of the contracted index.  Tiles of 128 rows
// where they still fill the device (256 workgroups), else 64.
template <typename T>
hipError_t map_tn(const T* A, int64_t lda, const T* B, int64_t ldb, int64_t M, int64_t N,
                  int64_t K, int64_t rows, int ns, T* D, int64_t ldd, int64_t stride,
                  hipStream_t s) {
  constexpr int VEC = map_vec<T>();
  const bool al = reinterpret_cast<uintptr_t>(A) % 16 == 0 &&
                  reinterpret_cast<uintptr_t>(B) % 16 == 0 && lda % VEC == 0 && ldb % VEC == 0;
  const bool big = ceil_div(M, 128) * ceil_div(N, kMapTJ) * ns >= 256;
  const dim3 grid((unsigned)(ceil_div(M, big ? 128 : 64) * ceil_div(N, kMapTJ)), (unsigned)ns);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, A, lda, B, ldb, M, N, K, rows, D, ldd, stride);
  };
  if (big && al) go(map_tn_kernel<T, 128, true>);
  else if (big) go(map_tn_kernel<T, 128, false>);
  else if (al) go(map_tn_kernel<T, 64, true>);
  else go(map_tn_kernel<T, 64, false>);
  return hipGetLastError();
}

}  // namespace

int map_splits(int64_t r_new, int64_t r_old, int64_t m, int num_cus) {
  // About two workgroups per compute unit, splits of at least 128 rows.
  const int64_t tiles = ceil_div(r_old, r_old > 64 ? 128 : 64) * ceil_div(r_new, kMapTJ);
  int64_t s = ceil_div(2 * (int64_t)num_cus, std::max<int64_t>(tiles, 1));
  s = std::min<int64_t>({s, kMaxMapSplits, std::max<int64_t>(1, m / 128)});
  return (int)std::max<int64_t>(s, 1);
}

template <typename T>
hipError_t launch_subspace_map(const T* Qnew, int64_t ldqn, int64_t r_new, const T* Qold,
                               int64_t ldqo, int64_t r_old, const T* M, int64_t ldm,
                               int64_t m, int64_t n, T* out, int64_t ldo, T* Cpart,
                               T* C, int nsplit, hipStream_t s) {
  const int64_t rows = round_up(ceil_div(m, nsplit), map_chunk<T>());
  const int ns = (int)ceil_div(m, rows);
  // C^T (r_old x r_new), so that its contiguous index is the one the second
  // product contracts; its columns padded to whole packs (the padding is
  // never read).
  const int64_t ldc = round_up(r_old, kMapPad);
  const int64_t stride = map_c_elems(r_new, r_old);
  hipError_t e = map_tn<T>(Qold, ldqo, Qnew, ldqn, r_old, r_new, m, rows, ns, Cpart, ldc,
                           stride, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((map_sum_kernel<T>), dim3((unsigned)ceil_div(stride, 256)), dim3(256), 0,
                     s, Cpart, ns, stride, C, stride);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return map_tn<T>(C, ldc, M, ldm, r_new, n, r_old, round_up(r_old, map_chunk<T>()), 1, out,
                   ldo, 0, s);
}

template hipError_t launch_subspace_map<float>(const float*, int64_t, int64_t, const float*,
                                               int64_t, int64_t, const float*, int64_t,
                                               int64_t, int64_t, float*, int64_t, float*,
                                               float*, int, hipStream_t);
template hipError_t launch_subspace_map<double>(const double*, int64_t, int64_t,
                                                const double*, int64_t, int64_t,
                                                const double*, int64_t, int64_t, int64_t,
                                                double*, int64_t, double*, double*, int,
                                                hipStream_t);

}  // namespace rrf

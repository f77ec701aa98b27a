// Panel Householder QR with T factor (Alg. 2, geqrt step) from the panel's
// Gram matrix: one grid-wide exchange per sweep of columns instead of one per
// column, and the column recurrence of a sweep on 16 x 16 blocks.
//
// The reflectors are those of LAPACK dlarfg / geqr2 (same signs, tau, V with
// unit diagonal); only the inner products they need come from a different
// place.  A sweep starts at column j0 with the current panel X (finished
// reflector columns before j0) and F = X^T X over the rows >= j0, exchanged
// across the grid, and runs on F and on the panel's top BP rows alone:
//
//   * Householder steps are orthogonal, so the Gram matrix of the remaining
//     columns over the rows >= j0 stays what it was and R (the rows the steps
//     make final) is its Cholesky factor, with the signs of dlarfg:
//     R_jj = beta_j = -sign(alpha_j) |R_jj|, alpha_j the current top entry.
//   * With J the 16 columns of a block, X_JJ their rows of the top block,
//     X_JJ - R_JJ = V_JJ W_JJ is an LU factorisation (V_JJ unit lower, the
//     pivots alpha_j - beta_j do not cancel), and below it V = X_J W_JJ^-1.
//   * The columns K right of J: R_JK = R_JJ^-T F_JK, W_JK = V_JJ^-1 (X_JK -
//     R_JK), X_K -= V_J W_JK, F_KL -= R_JK^T R_JL.
//
// So one wavefront factors the 16 x 16 block in registers (Cholesky and LU
// together, with R^-T, V^-1 and W^-1 built in the same steps; rows of 16
// lanes hold a block row's 16 columns, four block rows per lane group, so a
// step needs lane broadcasts only, no LDS and no barrier), and everything
// else is 16 x 16 tile products on f64 MFMA: the top block and F in LDS, the
// bulk rows in registers.  Every workgroup runs the sweep on its own copy of
// F and of the top block, all of them bit for bit alike.
//
// Downdating a norm loses relative accuracy when the column has shrunk: the
// rounding error of F[j][j] after s steps is about s u nu_j, nu_j being the
// column's norm^2 (rows >= sweep start) when F was last formed.  When the
// norm^2 below the diagonal falls below theta nu_j the sweep ends and F is
// formed again from the current rows (the safeguard LAPACK's dgeqp3 applies
// to its downdated column norms), so the norm behind each reflector has
// relative error <= ~64 u / theta and the reflector is orthogonal to that
// accuracy; a well-conditioned panel needs one exchange.  The first column of
// a sweep takes its norm below the diagonal straight from the exchange, so a
// column that is zero there is seen exactly (tau = 0, H = I; the sweep ends
// after it).  T (Eq. (4)) comes from the Gram matrix of the finished V (one
// more exchange, read by one workgroup) and tau.
//
// Layout: 256 threads; a wavefront owns RT tiles of 16 rows, kept in
// registers as f64 MFMA operands of the transposed frame: lane (g, m) holds
// row m, columns 16 c + 4 i + g at x[rt][c][i]; the output of a tile product
// has the same layout, so it is the next product's operand.  Rows 0 .. BP-1
// (workgroup 0's first tiles) live in the top block; their registers are not
// used.
//
// What bounds it: the exchanges (about 5 us each at 64 workgroups) and the
// serial 16-column factorisations (5 us each, about 650 cycles a column: one
// chain of a reciprocal square root, a reciprocal and lane broadcasts).
// Measured (rrf_panel_qr with this panel, the whole call): 16384 x 64 of
// condition 1e2, six sweeps, 173 us, against 409 us for the column-by-column
// grid (which that call takes by default: V here is two to three times as far
// from the exact one; a run's Q and B do not show it); 3000 x 32 of
// condition 1e2 89 us against 115 for the recurrence on all of F with two
// workgroup barriers per column.  In the look-ahead launch at 4096 x 4096 fp32,
// b = 32: 58 -> 35 us per block.
//
// The body runs as a kernel of its own (panel_gram.hip) or on the first
// workgroups of the look-ahead launch (lookahead.hip); w is the panel
// workgroup's index.

#pragma once

#include <utility>

#include "lanes.h"
#include "mfma.h"
#include "xchg.h"

namespace rrf {
namespace {

constexpr double kGramTheta = 0.125;

// A lane index the compiler cannot see through: the masks and addresses of
// one phase of the body are formed there instead of being hoisted out of the
// sweep loop, where they spill.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Exchanged Gram values: the upper-triangle 16 x 16 tiles of F in the MFMA
// output layout (tile x, item i, lane l holds F[16 ti + l/16 + 4 i][16 tj +
// l%16]), so that each lane's tagged stores are coalesced.
template <int BP>
struct GramGeom {
  static constexpr int N16 = BP / 16;
  static constexpr int NTL = N16 * (N16 + 1) / 2;
  static constexpr int NSLOT = NTL * 256;
  static constexpr __host__ __device__ __forceinline__ int tile(int ti, int tj) {
    return ti * N16 - ti * (ti - 1) / 2 + (tj - ti);
  }
};

constexpr int kTs = 17;   // row stride of a 16 x 16 tile in LDS

template <int BP>
struct GramLds {
  static constexpr int LS = BP + 2;   // staged rows
  static constexpr int LT = BP + 1;   // top block and W
  struct Work {
    double F[GramGeom<BP>::NTL][16 * kTs];   // upper tiles of F; R_JK in place
    double W[16 * LT];                       // W_JK of the current block
    double inv[3][16 * kTs];                 // R^-T, V^-1, W^-1
  };
  union {
    double S[64 * LS];            // staged rows for the Gram sums
    Work k;
  };
  double top[BP * LT];            // rows 0..BP-1: V below the diagonal, current
                                  // columns from the sweep's column on
  double tau[BP], nu[BP];
  double red2[256];
  double fx;                      // norm^2 below the diagonal, sweep's first column
  int js, stopped;                // of the block just factored
  int je;                         // end of its rows of R and W: js, or the sweep's
                                  // first column where that is left as it is
};

// One 16 x 16 block of a sweep: lane (h, k) holds rows 4 h + i of column k.
// The four wavefronts run the same Cholesky and LU, and each but the first
// one of the inverses beside it: R^-T and V^-1 (roles 1 and 2; a row is
// written to LDS when it is final) and W^-1 (role 3).  V's and W^-1's columns
// stay unscaled until the block ends (rwl), and entries a later step no
// longer reads may hold anything, so a step has no per-entry selects.
struct GramBlock {
  double f[4], x[4], aux[4];
  double tau, rwl;  // of the lane's column: tau, and 1 / (alpha - beta)
  double thr;       // least norm^2 below the diagonal the lane's column may have
  unsigned todo;    // bit mask of the columns to do
  int unchecked;    // the column whose norm came straight from the exchange
  int js;           // columns [o, js) done when the block ends
};

template <int J>
__device__ __forceinline__ void gram_block_step(GramBlock& s, double* inv, const int role,
                                                const int h, const int k) {
  if (!((s.todo >> J) & 1u)) return;   // uniform
  constexpr int QJ = J / 4, IJ = J % 4;
  const double alpha = lane_value<16 * QJ + J>(s.x[IJ]);
  const double nrm2 = lane_value<16 * QJ + J>(s.f[IJ]);
  const double xn2 = nrm2 - alpha * alpha;
  if (J != s.unchecked && !(xn2 >= lane_value<J>(s.thr))) {
    s.js = J;
    s.todo = 0;
    return;
  }
  const double fk = row_of<QJ>(s.f[IJ]);    // row J of F and X at the lane's column
  const double xk = row_of<QJ>(s.x[IJ]);
  double fr[4], xr[4];                      // column J of F and X at the lane's rows
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    fr[i] = row_lane<J>(s.f[i]);            // (R[J][row] R_JJ, by symmetry)
    xr[i] = row_lane<J>(s.x[i]);
  }
  const double y = fast_rsqrt(nrm2);
  const double rb = (alpha >= 0.0) ? -y : y;        // 1 / beta
  const double wjj = fma(-nrm2, rb, alpha);         // alpha - beta
  const double rw = fast_rcp(wjj);
  // (y^2 would overflow for column norms below 7.5e-155.)
  const double fc = (fk * y) * y;
#pragma unroll
  for (int i = 0; i < 4; ++i) s.f[i] = fma(-fr[i], fc, s.f[i]);
  const double wk = (k > J) ? fma(-fk, rb, xk) : 0.0;   // W_Jk = X_Jk - R_Jk
  const double wc = rw * wk;
#pragma unroll
  for (int i = 0; i < 4; ++i) s.x[i] = fma(-xr[i], wc, s.x[i]);
  s.tau = (k == J) ? -wjj * rb : s.tau;
  s.rwl = (k == J) ? rw : s.rwl;
  if (role == 3) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s.aux[i] = fma(-row_lane<J>(s.aux[i]), wc, s.aux[i]);
  } else if (role != 0) {
    const bool r1 = role == 1;
    const double a0 = row_of<QJ>(s.aux[IJ]);
    const double ak = r1 ? a0 * rb : a0;
    if (h == QJ) inv[J * kTs + k] = ak;
    const double rs = r1 ? rb : rw;
#pragma unroll
    for (int i = 0; i < 4; ++i) s.aux[i] = fma(-((r1 ? fr[i] : xr[i]) * rs), ak, s.aux[i]);
  }
}

template <int... Js>
__device__ __forceinline__ void gram_block_steps(GramBlock& s, double* inv, const int role,
                                                 const int h, const int k,
                                                 std::integer_sequence<int, Js...>) {
  (gram_block_step<Js>(s, inv, role, h, k), ...);
}

template <int BP, int RT>
__device__ __forceinline__ void panel_gram_body(GramLds<BP>& L, const GramPanelArgs& ga,
                                                const int w) {
  typedef GramGeom<BP> Geo;
  typedef GramLds<BP> Lds;
  constexpr int NB = BP / 16;
  constexpr int LS = Lds::LS, LT = Lds::LT;
  constexpr int RW = 64 * RT;
  // Gram tiles of a wavefront: with one tile the wavefronts split the rows.
  constexpr bool kSplitRows = Geo::NTL == 1;
  constexpr int NTW = kSplitRows ? 1 : (Geo::NTL + 3) / 4;

  const PanelArgs& a = ga.p;
  const int t0 = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(t0 >> 6);
  const int64_t base = (int64_t)w * RW;
  const int b = a.b, G = a.G;
  const bool forced = waits_forced(a.st);
  if (forced && G == 1) {   // no wait below: record the forced give-up
    unsigned spins = 0;
    keep_waiting(&spins, a.st);
  }

  // This wavefront's rows, and the top block (every workgroup).
  d4_t x[RT][NB];
  {
  const int t = opaque(t0), lane = t & 63, g = lane >> 4, m16 = lane & 15;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const double* Yr = a.Y + base + 16 * (wv * RT + rt) + m16 + (int64_t)g * a.ldy;
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[rt][c][i] = Yr[(int64_t)(16 * c + 4 * i) * a.ldy];
  }
  {
    constexpr int NTOP = BP * BP / 256;
    double tv[NTOP];
#pragma unroll
    for (int q = 0; q < NTOP; ++q) {
      const int e = t + 256 * q;
      tv[q] = a.Y[e % BP + (int64_t)(e / BP) * a.ldy];
    }
#pragma unroll
    for (int q = 0; q < NTOP; ++q) {
      const int e = t + 256 * q;
      L.top[(e % BP) * LT + e / BP] = tv[q];
    }
  }
  if (t < BP) L.tau[t] = 0.0;
  }

  unsigned exch = 0;
  // Gram matrix of the current rows into L.k.F.  FINAL: of V (unit diagonal,
  // zeros above), read by workgroup G - 1 only; else over the rows > j0, then
  // row j0 added (nu, and fx before it is added).
  auto form_gram = [&](const int j0, auto final_tag) __attribute__((always_inline)) {
    constexpr bool FINAL = decltype(final_tag)::value;
    const int t = opaque(t0), lane = t & 63, g = lane >> 4, m16 = lane & 15;
    const unsigned epoch = a.epoch_base + 1u + exch;
    const int par = (int)(exch & 1u);
    ++exch;
    d4_t acc[NTW];
#pragma unroll
    for (int u = 0; u < NTW; ++u) acc[u] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      __syncthreads();
      // Rows below BP come from the top block.
      const int64_t r = base + 16 * (wv * RT + rt) + m16;
      double* Sr = L.S + (16 * wv + m16) * LS;
      if (w == 0 && 16 * (wv * RT + rt) < BP) {   // uniform per wavefront
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int k = 16 * c + 4 * i + g;
            const double v = L.top[r * LT + k];
            if (FINAL) Sr[k] = (r > k) ? v : (r == k && k < b ? 1.0 : 0.0);
            else Sr[k] = (r > j0) ? v : 0.0;
          }
      } else {
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) Sr[16 * c + 4 * i + g] = x[rt][c][i];
      }
      __syncthreads();
      if constexpr (kSplitRows) {
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
          const double v = L.S[(16 * wv + 4 * s4 + g) * LS + m16];
          acc[0] = Mfma<double>::op(v, v, acc[0]);
        }
      } else {
#pragma unroll
        for (int u = 0; u < NTW; ++u) {
          const int tl = wv + 4 * u;
          if (tl < Geo::NTL) {   // uniform
            int ti = 0, r0 = tl;
            while (r0 >= NB - ti) {
              r0 -= NB - ti;
              ++ti;
            }
            const int tj = ti + r0;
#pragma unroll 8
            for (int s4 = 0; s4 < 16; ++s4)
              acc[u] = Mfma<double>::op(L.S[(4 * s4 + g) * LS + 16 * ti + m16],
                                        L.S[(4 * s4 + g) * LS + 16 * tj + m16], acc[u]);
          }
        }
      }
    }
    // One tile: the wavefronts' shares of the rows are added first.
    if constexpr (kSplitRows) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i) L.S[wv * 256 + i * 64 + lane] = acc[0][i];
      __syncthreads();
      if (wv == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[0][i] = (L.S[i * 64 + lane] + L.S[256 + i * 64 + lane]) +
                      (L.S[512 + i * 64 + lane] + L.S[768 + i * 64 + lane]);
      }
    }
    __syncthreads();   // L.S is free: L.k may be written
    auto put_f = [&](const int slot, double v) __attribute__((always_inline)) {
      const int tl = slot >> 8, i = (slot >> 6) & 3, ln = slot & 63;
      const int rr = (ln >> 4) + 4 * i, cc = ln & 15;
      if (!FINAL) {
        int ti = 0, r0 = tl;
        while (r0 >= NB - ti) {
          r0 -= NB - ti;
          ++ti;
        }
        const int gr = 16 * ti + rr, gc = 16 * (ti + r0) + cc;
        if (gr == j0 && gc == j0) L.fx = v;
        v += L.top[j0 * LT + gr] * L.top[j0 * LT + gc];
        if (gr == gc) L.nu[gr] = v;
      }
      L.k.F[tl][rr * kTs + cc] = v;
    };
    if (G == 1) {
#pragma unroll
      for (int u = 0; u < NTW; ++u) {
        const int tl = wv + 4 * u;
        if (tl < Geo::NTL) {
#pragma unroll
          for (int i = 0; i < 4; ++i) put_f(tl * 256 + i * 64 + lane, acc[u][i]);
        }
      }
      __syncthreads();
      return;
    }
    {
      u64* dst = ga.part + ((int64_t)par * G + w) * Geo::NSLOT * 2;
#pragma unroll
      for (int u = 0; u < NTW; ++u) {
        const int tl = wv + 4 * u;
        if (tl < Geo::NTL) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            put_tagged(&dst[(tl * 256 + i * 64 + lane) * 2], acc[u][i], epoch);
        }
      }
    }
    u64* sums = ga.sums + (int64_t)par * Geo::NSLOT * 2;
    // This workgroup's slice of slots, summed over all workgroups in a fixed
    // order (nsub threads per slot, then in LDS).
    {
      constexpr int NS = Geo::NSLOT;
      const int se = (NS + G - 1) / G;
      const int e0 = w * se;
      const int ne = max(0, min(NS, e0 + se) - e0);
      const int nsub = max(1, min(16, 256 / max(ne, 1)));
      const int per = 256 / nsub;
      for (int p0 = 0; p0 < ne; p0 += per) {
        const int el = p0 + t % per, sub = t / per;
        double s = 0.0;
        if (el < ne && sub < nsub) {
          const u64* src = ga.part + ((int64_t)par * G * NS + e0 + el) * 2;
          unsigned spins = 0;
          for (int w0 = sub; w0 < G; w0 += 8 * nsub) {
            u64 hi[8], lo[8];
            bool ok;
            do {
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                const int ww = w0 + u * nsub;
                const u64* q = src + (int64_t)(ww < G ? ww : 0) * NS * 2;
                hi[u] = get_word(q);
                lo[u] = get_word(q + 1);
              }
              ok = true;
#pragma unroll
              for (int u = 0; u < 8; ++u) ok = ok && tagged(hi[u], epoch) && tagged(lo[u], epoch);
            } while ((!ok || forced) && keep_waiting(&spins, a.st));
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (w0 + u * nsub < G) s += untag(hi[u], lo[u]);
          }
        }
        L.red2[t] = s;
        __syncthreads();
        if (t < per && p0 + t < ne) {
          double tot = 0.0;
          for (int sb = 0; sb < nsub; ++sb) tot += L.red2[sb * per + t];
          put_tagged(&sums[(int64_t)(e0 + p0 + t) * 2], tot, epoch);
        }
        __syncthreads();
      }
    }
    if (FINAL && w != G - 1) return;
    // The sums (every workgroup that goes on reads all of them).
    {
      u64 hi[Geo::NTL], lo[Geo::NTL];
      unsigned spins = 0;
      bool ok;
      do {
#pragma unroll
        for (int q = 0; q < Geo::NTL; ++q) {
          const u64* p = sums + (int64_t)(t + 256 * q) * 2;
          hi[q] = get_word(p);
          lo[q] = get_word(p + 1);
        }
        ok = true;
#pragma unroll
        for (int q = 0; q < Geo::NTL; ++q) ok = ok && tagged(hi[q], epoch) && tagged(lo[q], epoch);
      } while ((!ok || forced) && keep_waiting(&spins, a.st));
#pragma unroll
      for (int q = 0; q < Geo::NTL; ++q) put_f(t + 256 * q, untag(hi[q], lo[q]));
    }
    __syncthreads();
  };

  // Tile product D[g + 4 i][m16] of LDS tiles (row strides la, lb), added to
  // c; AT: the transpose of A.
  auto mm = [&](const double* A, const int la, const bool at, const double* B, const int lb,
                const int g, const int m16, d4_t c) __attribute__((always_inline)) -> d4_t {
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
      const int kk = 4 * s4 + g;
      const double av = at ? A[kk * la + m16] : A[m16 * la + kk];
      c = Mfma<double>::op(av, B[kk * lb + m16], c);
    }
    return c;
  };

  // The bulk rows under the column operations of block J (a compile-time
  // constant: x stays in registers): X_J <- X_J a4, X_K <- X_K - V_J W_JK.
  auto bulk = [&](auto jtag) __attribute__((always_inline)) {
    constexpr int J = decltype(jtag)::value;
    const int t = opaque(t0), lane = t & 63, g = lane >> 4, m16 = lane & 15;
    (void)t;
    double av[4];
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) av[s4] = L.k.inv[2][(4 * s4 + g) * kTs + m16];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      d4_t d = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) d = Mfma<double>::op(av[s4], x[rt][J][s4], d);
      x[rt][J] = d;
    }
#pragma unroll
    for (int K = J + 1; K < NB; ++K) {
      double wvv[4];
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) wvv[s4] = -L.k.W[(4 * s4 + g) * LT + 16 * K + m16];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4)
          x[rt][K] = Mfma<double>::op(wvv[s4], x[rt][J][s4], x[rt][K]);
    }
  };

  const int nbb = (b + 15) / 16;   // blocks with a column of the panel
  int j0 = 0;
  while (j0 < b) {                 // sweeps (uniform)
    form_gram(j0, std::false_type{});
    bool first = true;
    int J = j0 / 16;
    for (; J < nbb; ++J) {
      const int o = max(j0 - 16 * J, 0);
      double* topJ = L.top + 16 * J * LT;
      {
        const int t = opaque(t0), lane = t & 63, g = lane >> 4, m16 = lane & 15;
        GramBlock s;
        const double* Fj = L.k.F[Geo::tile(J, J)];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 4 * g + i;
          s.f[i] = Fj[r * kTs + m16];
          s.x[i] = topJ[r * LT + 16 * J + m16];
          s.aux[i] = (r == m16) ? 1.0 : 0.0;
        }
        // (At least the least positive number: a norm of zero ends the sweep.)
        s.thr = fmax(kGramTheta * L.nu[16 * J + m16], 4.9406564584124654e-324);
        s.tau = 0.0;
        s.rwl = 1.0;
        const int nb = min(16, b - 16 * J);
        s.js = nb;
        s.unchecked = first ? o : -1;
        const bool none = first && !(L.fx > 0.0);
        s.todo = ((1u << nb) - 1u) & ~((1u << o) - 1u);
        if (none) {
          // Nothing below the diagonal in the sweep's first column: H = I,
          // V's column zero, tau = 0, and the sweep ends after it.  No step
          // runs, so the inverses have no rows: R and W have none either.
          s.js = o + 1;
          s.todo = 0;
          if (m16 == o) s.rwl = 0.0;
        }
        const bool whole = s.js == nb;
        __syncthreads();   // every wavefront has read the block
        gram_block_steps(s, L.k.inv[max(wv - 1, 0)], wv, g, m16,
                         std::make_integer_sequence<int, 16>{});
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 4 * g + i;
          // Rows above the diagonal of a finished column are not read again.
          if (wv == 0) topJ[r * LT + 16 * J + m16] = s.x[i] * s.rwl;
          if (wv == 3) L.k.inv[2][r * kTs + m16] = s.aux[i] * s.rwl;
        }
        if (t >= o && t < s.js) L.tau[16 * J + t] = s.tau;
        if (t == 0) {
          L.js = s.js;
          L.je = none ? o : s.js;
          L.stopped = (whole && s.todo != 0) ? 0 : 1;
        }
      }
      __syncthreads();
      const int js = L.js, je = L.je;
      const bool stopped = L.stopped != 0;
      first = false;
      // R_JK over F_JK (rows [o, je), the others zero) and V in the top rows
      // below the block.
      {
        const int t = opaque(t0), lane = t & 63, g = lane >> 4, m16 = lane & 15;
        (void)t;
        const int nk = NB - 1 - J;
        for (int u = wv; u < 2 * nk; u += 4) {
          if (u < nk) {
            double* Fk = L.k.F[Geo::tile(J, J + 1 + u)];
            const d4_t d = mm(L.k.inv[0], kTs, false, Fk, kTs, g, m16, d4_t{0.0, 0.0, 0.0, 0.0});
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int r = g + 4 * i;
              Fk[r * kTs + m16] = (r >= o && r < je) ? d[i] : 0.0;
            }
          } else {
            double* X = L.top + 16 * (J + 1 + u - nk) * LT + 16 * J;
            const d4_t d = mm(X, LT, false, L.k.inv[2], kTs, g, m16, d4_t{0.0, 0.0, 0.0, 0.0});
#pragma unroll
            for (int i = 0; i < 4; ++i) X[(g + 4 * i) * LT + m16] = d[i];
          }
        }
        if (nk > 0) __syncthreads();
        // W_JK = V_JJ^-1 (X_JK - R_JK), rows [o, je).
        for (int u = wv; u < nk; u += 4) {
          const int K = J + 1 + u;
          const double* Fk = L.k.F[Geo::tile(J, K)];
          d4_t d = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int s4 = 0; s4 < 4; ++s4) {
            const int kk = 4 * s4 + g;
            d = Mfma<double>::op(L.k.inv[1][m16 * kTs + kk],
                                 topJ[kk * LT + 16 * K + m16] - Fk[kk * kTs + m16], d);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r = g + 4 * i;
            L.k.W[r * LT + 16 * K + m16] = (r >= o && r < je) ? d[i] : 0.0;
          }
        }
        if (nk > 0) __syncthreads();
        // X_IK -= V_IJ W_JK in the top rows below the block (and in the
        // block's own rows >= js when the sweep ends here); F_KL -= R_JK^T
        // R_JL when it goes on.
        const int nt = nk * nk;
        const int extra = stopped ? nk : nk * (nk + 1) / 2;
        for (int u = wv; u < nt + extra; u += 4) {
          if (u < nt) {
            const int I = J + 1 + u / nk, K = J + 1 + u % nk;
            double* X = L.top + 16 * I * LT;
            const d4_t d = mm(X + 16 * J, LT, false, L.k.W + 16 * K, LT,
                              g, m16, d4_t{0.0, 0.0, 0.0, 0.0});
#pragma unroll
            for (int i = 0; i < 4; ++i) X[(g + 4 * i) * LT + 16 * K + m16] -= d[i];
          } else if (stopped) {
            const int K = J + 1 + u - nt;
            d4_t d = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
              const int kk = 4 * s4 + g;
              const double v = topJ[m16 * LT + 16 * J + kk];
              d = Mfma<double>::op((kk >= o && kk < je) ? v : 0.0, L.k.W[kk * LT + 16 * K + m16], d);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int r = g + 4 * i;
              if (r >= js) topJ[r * LT + 16 * K + m16] -= d[i];
            }
          } else {
            int v = u - nt, ti = 0;
            while (v >= nk - ti) {
              v -= nk - ti;
              ++ti;
            }
            const int K = J + 1 + ti, M = K + v;
            double* Fk = L.k.F[Geo::tile(K, M)];
            const d4_t d = mm(L.k.F[Geo::tile(J, K)], kTs, true, L.k.F[Geo::tile(J, M)], kTs,
                              g, m16, d4_t{0.0, 0.0, 0.0, 0.0});
#pragma unroll
            for (int i = 0; i < 4; ++i) Fk[(g + 4 * i) * kTs + m16] -= d[i];
          }
        }
      }
      if (J == 0) bulk(std::integral_constant<int, 0>{});
      if constexpr (NB > 1)
        if (J == 1) bulk(std::integral_constant<int, 1>{});
      if constexpr (NB > 2) {
        if (J == 2) bulk(std::integral_constant<int, 2>{});
        if (J == 3) bulk(std::integral_constant<int, 3>{});
      }
      __syncthreads();
      if (stopped) {
        j0 = 16 * J + js;
        break;
      }
    }
    if (J == nbb) j0 = b;
  }

  const int t = opaque(t0), lane = t & 63, g = lane >> 4, m16 = lane & 15;
  // V with explicit unit diagonal and zeros above / beyond b.
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int64_t r = base + 16 * (wv * RT + rt) + m16;
    if (r < a.m) {
      const bool top = w == 0 && 16 * (wv * RT + rt) < BP;
#pragma unroll
      for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = 16 * c + 4 * i + g;
          double v = x[rt][c][i];
          if (top) v = (r > k) ? L.top[r * LT + k] : (r == k && k < b ? 1.0 : 0.0);
          a.V[r + (int64_t)k * a.ldv] = v;
        }
    }
  }

  // T (Eq. (4)) from S = V^T V and tau: T[c][c] = tau_c, T[i][c] = -tau_i
  // sum_{i < p <= c} S[i][p] T[p][c] (tau_i = 0 gives a zero row); within the
  // diagonal blocks by back substitution, one column per thread, then
  // T_JK = -T_JJ sum_{J < M <= K} S_JM T_MK by block diagonals.
  form_gram(0, std::true_type{});
  if (w != G - 1) return;
  double* Tl = L.top;
  if (t < BP) {
    const int J = t / 16, cc = t % 16;
    const double* Sj = L.k.F[Geo::tile(J, J)];
    double tc[16];
#pragma unroll
    for (int i = 15; i >= 0; --i) {
      double s0 = 0.0, s1 = 0.0;
#pragma unroll
      for (int p = i + 1; p < 16; p += 2) {
        s0 += Sj[i * kTs + p] * tc[p];
        if (p + 1 < 16) s1 += Sj[i * kTs + p + 1] * tc[p + 1];
      }
      const double ti = L.tau[16 * J + i];
      tc[i] = (i < cc) ? -ti * (s0 + s1) : (i == cc ? ti : 0.0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) Tl[(16 * J + i) * LT + t] = tc[i];
  }
  __syncthreads();
#pragma unroll 1
  for (int d = 1; d < NB; ++d) {
    for (int J = wv; J < NB - d; J += 4) {
      const int K = J + d;
      d4_t s = d4_t{0.0, 0.0, 0.0, 0.0};
      for (int M = J + 1; M <= K; ++M)
        s = mm(L.k.F[Geo::tile(J, M)], kTs, false, Tl + 16 * M * LT + 16 * K, LT, g, m16, s);
      d4_t o = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4)
        o = Mfma<double>::op(-Tl[(16 * J + m16) * LT + 16 * J + 4 * s4 + g], s[s4], o);
#pragma unroll
      for (int i = 0; i < 4; ++i) Tl[(16 * J + g + 4 * i) * LT + 16 * K + m16] = o[i];
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < BP * BP / 256; ++q) {
    const int e = t + 256 * q;
    const int i = e % BP, c = e / BP;
    a.Tm[i + (int64_t)c * a.ldt] = (i / 16 <= c / 16) ? Tl[i * LT + c] : 0.0;
  }
  if (t < b) a.tau[t] = L.tau[t];
}

}  // namespace
}  // namespace rrf

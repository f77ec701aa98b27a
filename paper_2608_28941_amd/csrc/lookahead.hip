// Look-ahead kernel: the one-GPU form of the paper's two-queue overlap
// (Sec. 5, Fig. 2(b)).  While the update of block i streams over B, the panel
// of block i + 1 is factored on a few compute units: the first G workgroups
// of the launch run the panel (panel_gram_body), the others the update tiles
// (update_body).  Workgroups are dispatched in order, so the panel's
// workgroups are resident from the start; the update's workgroups never wait
// on anything, so the panel's grid-wide waits always complete.
//
// The panel's input is the sample of block i + 1 taken one update earlier
// and brought up to date with Q_i^T before this launch (see rrf_run).
//
// Block 0 has no update to hide its panel in, but its panel and the first
// look-ahead sample S_1 = A Omega_1 are independent: the same launch shape
// runs them together (SAMPLE_ONLY: the non-panel workgroups only sample,
// update_body with no reflectors and no store).

#include "panel_gram_body.h"
#include "update_body.h"

namespace rrf {
namespace {

template <typename T, int BP, int RT, bool SAMPLE_ONLY>
__global__ __launch_bounds__(256, 2) void update_gram_kernel(UpdateArgs<T> ua,
                                                             GramPanelArgs ga,
                                                             unsigned nrb) {
  constexpr int UBP = SAMPLE_ONLY ? 0 : BP;
  // A workgroup is one or the other: the two parts share their LDS.
  __shared__ union {
    GramLds<BP> g;
    UpdLds<T, UBP, BP> u;
  } L;
  if ((int)blockIdx.x < ga.p.G) {
    panel_gram_body<BP, RT>(L.g, ga, (int)blockIdx.x);
    return;
  }
  const unsigned t = blockIdx.x - (unsigned)ga.p.G;
  update_body<T, UBP, BP, !SAMPLE_ONLY>(L.u, ua, t % nrb, t / nrb, nrb);
}

template <typename T, int BP, int RT, bool SO>
hipError_t ug_go(const UpdateArgs<T>& ua, int nsplit, const GramPanelArgs& ga,
                 hipStream_t s) {
  const unsigned nrb = (unsigned)ceil_div(ua.mr, kUpdRows);
  const dim3 grid((unsigned)ga.p.G + nrb * (unsigned)nsplit);
  hipLaunchKernelGGL((update_gram_kernel<T, BP, RT, SO>), grid, dim3(256), 0, s, ua, ga, nrb);
  return hipGetLastError();
}

template <typename T, int BP, int RT, bool SO>
int ug_occ() {
  static const int occ = [] {
    int o = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &o, reinterpret_cast<const void*>(update_gram_kernel<T, BP, RT, SO>), 256, 0) !=
        hipSuccess)
      o = 0;
    return o;
  }();
  return occ;
}

// Dispatch over the panel's width and row tiles: go(BP, RT) as integral
// constants for a built shape, else fallback.
template <int BP, typename F, typename R>
R ug_rt(int rt, F&& go, R fallback) {
  typedef std::integral_constant<int, BP> bp_t;
  switch (rt) {
    case 1: return go(bp_t{}, std::integral_constant<int, 1>{});
    case 2: return go(bp_t{}, std::integral_constant<int, 2>{});
    case 4: return go(bp_t{}, std::integral_constant<int, 4>{});
    case 8: if constexpr (8 * BP <= kGramFusedRegs) return go(bp_t{}, std::integral_constant<int, 8>{}); break;
    case 16: if constexpr (16 * BP <= kGramFusedRegs) return go(bp_t{}, std::integral_constant<int, 16>{}); break;
  }
  return fallback;
}
template <typename F, typename R>
R ug_shape(const PanelShape& sh, F&& go, R fallback) {
  switch (sh.bp) {
    case 16: return ug_rt<16>(sh.rpt, go, fallback);
    case 32: return ug_rt<32>(sh.rpt, go, fallback);
    case 64: return ug_rt<64>(sh.rpt, go, fallback);
  }
  return fallback;
}

}  // namespace

bool update_gram_supported(int bp, int qp, const PanelShape& sh) {
  return (bp == 0 || bp == qp) && qp == sh.bp && sh.G >= 1 && sh.G <= kMaxGramWGs &&
         ug_shape(sh, [](auto, auto) { return true; }, false);
}

template <typename T>
int update_gram_occupancy(const PanelShape& sh, bool sample_only) {
  return ug_shape(sh, [&](auto b, auto r) {
    return sample_only ? ug_occ<T, decltype(b)::value, decltype(r)::value, true>()
                       : ug_occ<T, decltype(b)::value, decltype(r)::value, false>();
  }, 0);
}

template int update_gram_occupancy<float>(const PanelShape&, bool);
template int update_gram_occupancy<double>(const PanelShape&, bool);

template <typename T>
hipError_t launch_update_gram(const UpdateArgs<T>& ua, int nsplit, const GramPanelArgs& ga,
                              const PanelShape& sh, hipStream_t s) {
  const bool so = ua.bp == 0;
  if (!update_gram_supported(ua.bp, ua.qp, sh) || so != (ua.dst == nullptr) || ua.mr <= 0 ||
      ua.n <= 0 || ga.p.G != sh.G || ga.p.b < 1 || ga.p.b > sh.bp)
    return hipErrorNotSupported;
  // 32-bit buffer offsets, as in launch_update.
  const int64_t ld = ua.dst ? std::max(ua.lds, ua.ldd) : ua.lds;
  if (ld < ua.mr || (int64_t)kUpdChunk * ld * (int64_t)sizeof(T) > ((int64_t)1 << 30))
    return hipErrorInvalidValue;
  return ug_shape(sh, [&](auto b, auto r) {
    return so ? ug_go<T, decltype(b)::value, decltype(r)::value, true>(ua, nsplit, ga, s)
              : ug_go<T, decltype(b)::value, decltype(r)::value, false>(ua, nsplit, ga, s);
  }, hipErrorNotSupported);
}

template hipError_t launch_update_gram<float>(const UpdateArgs<float>&, int, const GramPanelArgs&, const PanelShape&, hipStream_t);
template hipError_t launch_update_gram<double>(const UpdateArgs<double>&, int, const GramPanelArgs&, const PanelShape&, hipStream_t);

}  // namespace rrf

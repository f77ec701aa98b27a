// Panel Householder QR with T factor from the panel's Gram matrix, as a
// kernel of its own (the body and its description are in panel_gram_body.h).

#include "panel_gram_body.h"

namespace rrf {
namespace {

template <int BP, int RT>
__global__ __launch_bounds__(256) void panel_gram_kernel(GramPanelArgs ga) {
  __shared__ GramLds<BP> L;
  panel_gram_body<BP, RT>(L, ga, (int)blockIdx.x);
}

// Row tiles per wavefront: the panel's registers (RT BP / 2 of the 512) leave
// room for everything else up to RT BP = 512.
constexpr int kGramRegs = 512;

template <int BP, int RT>
hipError_t gram_go(const GramPanelArgs& a, hipStream_t s) {
  auto fn = panel_gram_kernel<BP, RT>;
  int occ = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
      &occ, reinterpret_cast<const void*>(fn), 256, 0);
  if (e != hipSuccess) return e;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return hipErrorInvalidDevice;
  if (occ < 1 || a.p.G > occ * cus) return hipErrorCooperativeLaunchTooLarge;
  GramPanelArgs arg = a;
  void* params[] = {&arg};
  return launch_resident(reinterpret_cast<const void*>(fn), dim3(a.p.G), dim3(256), params, s);
}

template <int BP>
hipError_t gram_rt(const GramPanelArgs& a, int rt, hipStream_t s) {
  switch (rt) {
    case 1: return gram_go<BP, 1>(a, s);
    case 2: return gram_go<BP, 2>(a, s);
    case 4: return gram_go<BP, 4>(a, s);
    case 8: if constexpr (8 * BP <= kGramRegs) return gram_go<BP, 8>(a, s); break;
    case 16: if constexpr (16 * BP <= kGramRegs) return gram_go<BP, 16>(a, s); break;
    case 32: if constexpr (32 * BP <= kGramRegs) return gram_go<BP, 32>(a, s); break;
  }
  return hipErrorInvalidValue;
}

// The fewest row tiles per wavefront, at most rt_max, whose grid has at most
// max_wgs workgroups.
bool gram_shape_within(int64_t m, int bp, int rt_max, int64_t max_wgs, PanelShape* out) {
  for (int rt = 1; rt <= rt_max; rt *= 2) {
    const int64_t G = ceil_div(m, (int64_t)64 * rt);
    if (G <= max_wgs && G <= kMaxGramWGs) {
      out->bp = bp;
      out->rpt = rt;
      out->G = (int)G;
      out->rows_pad = G * 64 * rt;
      return true;
    }
  }
  return false;
}

}  // namespace

bool gram_panel_shape(int64_t m, int b, int num_cus, PanelShape* out) {
  if (b < 1 || b > kMaxBlock || m < b) return false;
  const int bp = pad16(b);
  // One workgroup (no exchange) up to 128 columns x row tiles, else the
  // fewest rows per wavefront within half the compute units (a smaller grid
  // exchanges less), failing that within one workgroup per compute unit.
  return gram_shape_within(m, bp, 128 / bp, 1, out) ||
         gram_shape_within(m, bp, kGramRegs / bp, std::max(1, num_cus / 2), out) ||
         gram_shape_within(m, bp, kGramRegs / bp, num_cus, out);
}

bool gram_fused_shape(int64_t m, int b, int max_wgs, PanelShape* out) {
  if (b < 1 || b > kMaxBlock || m < b) return false;
  const int bp = pad16(b);
  return gram_shape_within(m, bp, 128 / bp, 1, out) ||
         gram_shape_within(m, bp, kGramFusedRegs / bp, max_wgs, out);
}

hipError_t launch_panel_gram(const GramPanelArgs& a, const PanelShape& sh, hipStream_t s) {
  if (a.p.G != sh.G || a.p.b < 1 || a.p.b > sh.bp) return hipErrorInvalidValue;
  switch (sh.bp) {
    case 16: return gram_rt<16>(a, sh.rpt, s);
    case 32: return gram_rt<32>(a, sh.rpt, s);
    case 64: return gram_rt<64>(a, sh.rpt, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace rrf

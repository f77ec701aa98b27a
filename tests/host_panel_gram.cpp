// The Gram panel's body (panel_gram_body.h) on the CPU: reads a panel, runs G
// workgroups of it and writes V, T and tau.  LDS starts as the byte given, so
// that a value read before it is written shows.
//   host_panel_gram BP RT G b m fill in.bin out.bin
// in: m x b doubles, column-major; out: V (m x b), T (b x b), tau (b), the
// number of grid exchanges (G > 1) and the wait error.

#include "host_wavefront.h"

#include <cstdio>
#include <cstdlib>

#include "panel_gram_body.h"

template <int BP, int RT>
static int go(int G, int b, int64_t m, int fill, const char* in, const char* out) {
  using namespace rrf;
  const int64_t rows = (int64_t)G * 64 * RT, ld = rows;
  if (m > rows || b > BP || b > m) return 2;
  std::vector<double> Y(ld * BP, 0.0), V(ld * BP, 0.0), T(64 * BP, 0.0), tau(BP, 0.0);
  FILE* f = std::fopen(in, "rb");
  if (!f) return 3;
  for (int c = 0; c < b; ++c)
    if (std::fread(&Y[c * ld], 8, (size_t)m, f) != (size_t)m) return 3;
  std::fclose(f);
  std::vector<unsigned long long> part((size_t)2 * G * kGramSlots * 2, 0), sums(2 * kGramSlots * 2, 0);
  DevState st{};
  st.spin_limit = 1u << 20;
  std::vector<std::unique_ptr<GramLds<BP>>> lds;
  for (int g = 0; g < G; ++g) {
    lds.push_back(std::make_unique<GramLds<BP>>());
    std::memset((void*)lds.back().get(), fill, sizeof(GramLds<BP>));
  }
  GramPanelArgs a{};
  a.p.Y = Y.data(); a.p.ldy = ld; a.p.m = m; a.p.b = b;
  a.p.V = V.data(); a.p.ldv = ld; a.p.Tm = T.data(); a.p.ldt = 64; a.p.tau = tau.data();
  a.p.epoch_base = 128; a.p.st = &st; a.p.G = G;
  a.part = part.data(); a.sums = sums.data();
  hostwave::run(G, [&](int w) { panel_gram_body<BP, RT>(*lds[w], a, w); });
  f = std::fopen(out, "wb");
  if (!f) return 3;
  for (int c = 0; c < b; ++c) std::fwrite(&V[c * ld], 8, (size_t)m, f);
  for (int c = 0; c < b; ++c) std::fwrite(&T[c * 64], 8, (size_t)b, f);
  std::fwrite(tau.data(), 8, (size_t)b, f);
  // The exchanges are numbered by their words' epochs.
  unsigned last = a.p.epoch_base;
  for (unsigned long long x : sums) last = std::max(last, (unsigned)x);
  const double exchanges = last - a.p.epoch_base, err = st.barrier_err;
  std::fwrite(&exchanges, 8, 1, f);
  std::fwrite(&err, 8, 1, f);
  std::fclose(f);
  return 0;
}

int main(int argc, char** argv) {
  if (argc != 9) return 1;
  const int bp = std::atoi(argv[1]), rt = std::atoi(argv[2]), G = std::atoi(argv[3]),
            b = std::atoi(argv[4]), m = std::atoi(argv[5]), fill = std::atoi(argv[6]);
  if (bp == 16 && rt == 1) return go<16, 1>(G, b, m, fill, argv[7], argv[8]);
  if (bp == 32 && rt == 1) return go<32, 1>(G, b, m, fill, argv[7], argv[8]);
  if (bp == 64 && rt == 1) return go<64, 1>(G, b, m, fill, argv[7], argv[8]);
  if (bp == 64 && rt == 2) return go<64, 2>(G, b, m, fill, argv[7], argv[8]);
  return 1;
}

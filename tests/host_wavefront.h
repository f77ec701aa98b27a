// A host stand-in for the wavefront operations that the Gram panel's body
// uses, so that the body itself runs on the CPU: every lane is a fiber, the
// fibers of a grid run round robin on one thread, and a cross-lane operation
// exchanges its operands at a barrier of the wavefront's 64 lanes.
// Include it before the kernel's header (compiled as plain C++).
#pragma once

#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <functional>
#include <memory>
#include <vector>

namespace hostwave {

struct Wave {
  int count = 0;
  unsigned gen = 0;
  unsigned long long ex[2][3][64];   // operands, by parity of the operation
};
struct Group {
  int count = 0;
  unsigned gen = 0;
  Wave wave[4];
};
struct Fiber {
  ucontext_t ctx;
  std::unique_ptr<char[]> stack;
  Group* group;
  unsigned tid;
  unsigned ops = 0;
  bool done = false;
};

inline ucontext_t main_ctx;
inline std::vector<std::unique_ptr<Fiber>> fibers;
inline Fiber* cur = nullptr;
inline std::function<void(int)> body;   // body(workgroup) of the current fiber

inline void yield() { swapcontext(&cur->ctx, &main_ctx); }

template <typename B>
inline void barrier(B& b, int n) {
  const unsigned g = b.gen;
  if (++b.count == n) {
    b.count = 0;
    ++b.gen;
  } else {
    while (b.gen == g) yield();
  }
}

inline int lane() { return (int)(cur->tid & 63); }
inline Wave& wave() { return cur->group->wave[cur->tid >> 6]; }

// Publishes this lane's operand(s); returns the wavefront's, by lane.
inline unsigned long long (*exchange(unsigned long long a, unsigned long long b = 0,
                                     unsigned long long c = 0))[64] {
  Wave& w = wave();
  auto* e = w.ex[cur->ops++ & 1];
  e[0][lane()] = a;
  e[1][lane()] = b;
  e[2][lane()] = c;
  barrier(w, 64);
  return e;
}

inline double as_double(unsigned long long u) {
  double d;
  std::memcpy(&d, &u, 8);
  return d;
}
inline unsigned long long as_bits(double d) {
  unsigned long long u;
  std::memcpy(&u, &d, 8);
  return u;
}

inline void entry(int wg) {
  body(wg);
  cur->done = true;
  while (true) yield();
}

// Runs fn(workgroup) on groups x 256 lanes until all have returned.
inline void run(int groups, std::function<void(int)> fn) {
  body = std::move(fn);
  std::vector<std::unique_ptr<Group>> gs;
  fibers.clear();
  for (int g = 0; g < groups; ++g) {
    gs.push_back(std::make_unique<Group>());
    for (unsigned t = 0; t < 256; ++t) {
      auto f = std::make_unique<Fiber>();
      f->stack.reset(new char[1 << 17]);
      f->group = gs.back().get();
      f->tid = t;
      getcontext(&f->ctx);
      f->ctx.uc_stack.ss_sp = f->stack.get();
      f->ctx.uc_stack.ss_size = 1 << 17;
      makecontext(&f->ctx, reinterpret_cast<void (*)()>(entry), 1, g);
      fibers.push_back(std::move(f));
    }
  }
  for (bool live = true; live;) {
    live = false;
    for (auto& f : fibers)
      if (!f->done) {
        live = true;
        cur = f.get();
        swapcontext(&main_ctx, &f->ctx);
      }
  }
  fibers.clear();
}

struct Pair {
  unsigned v[2];
  unsigned operator[](int i) const { return v[i]; }
};
struct ThreadIdx {
  struct X {
    operator unsigned() const { return cur->tid; }
  } x;
};

// The operations, by their documented lane layouts.
inline int mov_dpp(int v, int ctrl) {   // row_newbcast: lane ctrl - 0x150 of the row
  return (int)exchange((unsigned)v)[0][(lane() & 48) + (ctrl - 0x150)];
}
inline int readlane(int v, int l) { return (int)exchange((unsigned)v)[0][l]; }
inline int readfirstlane(int v) { return readlane(v, 0); }
inline Pair permlane32_swap(unsigned a, unsigned b) {
  auto* e = exchange(a, b);
  const int l = lane(), h = l & 31;
  return l < 32 ? Pair{{(unsigned)e[0][h], (unsigned)e[0][h + 32]}}
                : Pair{{(unsigned)e[1][h], (unsigned)e[1][h + 32]}};
}
inline Pair permlane16_swap(unsigned a, unsigned b) {
  auto* e = exchange(a, b);
  const int l = lane(), base = (l & 32) + (l & 15);
  return (l & 16) == 0 ? Pair{{(unsigned)e[0][base], (unsigned)e[0][base + 16]}}
                       : Pair{{(unsigned)e[1][base], (unsigned)e[1][base + 16]}};
}
template <typename V>
inline V mfma_f64_16x16x4(double a, double b, V c) {
  auto* e = exchange(as_bits(a), as_bits(b));
  const int g = lane() >> 4, m = lane() & 15;
  for (int i = 0; i < 4; ++i)
    for (int k = 0; k < 4; ++k)
      c[i] = std::fma(as_double(e[0][16 * k + g + 4 * i]), as_double(e[1][16 * k + m]), c[i]);
  return c;
}
// An estimate with a relative error of about 2^-15.
inline double coarse(double v) { return v * (1.0 + 0x1p-15); }

}  // namespace hostwave

static hostwave::ThreadIdx threadIdx;
static inline void __syncthreads() { hostwave::barrier(*hostwave::cur->group, 256); }
static inline double __longlong_as_double(long long u) { return hostwave::as_double((unsigned long long)u); }
static inline long long __double_as_longlong(double d) { return (long long)hostwave::as_bits(d); }
using std::max;
using std::min;

#define __builtin_amdgcn_mov_dpp(v, c, r, b, z) hostwave::mov_dpp(v, c)
#define __builtin_amdgcn_readlane(v, l) hostwave::readlane(v, l)
#define __builtin_amdgcn_readfirstlane(v) hostwave::readfirstlane(v)
#define __builtin_amdgcn_permlane32_swap(a, b, f, g) hostwave::permlane32_swap(a, b)
#define __builtin_amdgcn_permlane16_swap(a, b, f, g) hostwave::permlane16_swap(a, b)
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, x, y, z) hostwave::mfma_f64_16x16x4(a, b, c)
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, x, y, z) (c)
#define __builtin_amdgcn_rsq(v) hostwave::coarse(1.0 / std::sqrt(v))
#define __builtin_amdgcn_rcp(v) hostwave::coarse(1.0 / (v))
#define __builtin_amdgcn_s_sleep(n) hostwave::yield()
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_store(p, v, o, s) (*(p) = (v))
#define __hip_atomic_load(p, o, s) (*(p))

// The kernels of csrc/slice_build.h on the CPU: every GPU thread is a fiber,
// wavefront votes and barriers are switch points.  Built with the address and
// bounds sanitizers, so that an index outside a shared array or outside the
// workspace ranges of the slices ends the program; what the kernels wrote is
// then compared with the CSR rows they were given.
#include <ucontext.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <numeric>
#include <random>
#include <set>
#include <vector>

#define __host__
#define __device__
#define __global__
#define __shared__ static
#define __launch_bounds__(n)
#define __forceinline__ inline

struct int2 {
  int32_t x, y;
};
struct uint4 {
  uint32_t x, y, z, w;
};
static int2 make_int2(int32_t x, int32_t y) { return {x, y}; }
static uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
struct Dim {
  uint32_t x, y, z;
};
static Dim threadIdx, blockIdx, blockDim;
using std::max;
using std::min;

// ---------------------------------------------------------------- the fibers
enum State { READY, AT_WAVE, AT_BLOCK, ENDED };
struct Fiber {
  ucontext_t ctx;
  std::unique_ptr<char[]> stack;
  State state;
  unsigned votes;  // parity picks the buffer, so that one switch per vote is enough
};
constexpr size_t STACK = 64 << 10;
static std::vector<Fiber> fibers;
static ucontext_t scheduler;
static std::function<void()> body;
static uint32_t now;
static uint64_t vote_buf[16][2][64];

static void wait_at(State s) {
  const uint32_t me = now;
  fibers[me].state = s;
  swapcontext(&fibers[me].ctx, &scheduler);
  now = me;
  threadIdx = {me, 0, 0};
}
static void __syncthreads() { wait_at(AT_BLOCK); }
static void __builtin_wave_barrier_host() { wait_at(AT_WAVE); }
static const uint64_t *vote(uint64_t v) {
  const uint32_t me = now;
  uint64_t *buf = vote_buf[me >> 6][fibers[me].votes++ & 1];
  buf[me & 63] = v;
  wait_at(AT_WAVE);
  return buf;
}
static unsigned long long __ballot(bool p) {
  const uint64_t *b = vote(p);
  unsigned long long m = 0;
  for (int i = 0; i < 64; ++i) m |= (unsigned long long)(b[i] != 0) << i;
  return m;
}
static int32_t __shfl(int32_t v, int lane, int) { return (int32_t)vote((uint32_t)v)[lane]; }
static int32_t __shfl_xor(int32_t v, int d, int) {
  const uint32_t lane = now & 63;
  return (int32_t)vote((uint32_t)v)[lane ^ d];
}
static int32_t readfirstlane_host(int32_t v) { return __shfl(v, 0, 64); }
static int __popc(uint32_t x) { return __builtin_popcount(x); }
static uint32_t atomicAdd(uint32_t *p, uint32_t v) {
  const uint32_t o = *p;
  *p += v;
  return o;
}
static uint32_t atomicMax(uint32_t *p, uint32_t v) {
  const uint32_t o = *p;
  *p = std::max(*p, v);
  return o;
}
#define __builtin_amdgcn_wave_barrier __builtin_wave_barrier_host
#define __builtin_amdgcn_readfirstlane readfirstlane_host

#include "slice_build.h"

static void fiber_main() {
  threadIdx = {now, 0, 0};
  body();
  fibers[now].state = ENDED;
}

static void run_block(uint32_t threads, uint32_t bx, uint32_t by) {
  blockDim = {threads, 1, 1};
  blockIdx = {bx, by, 0};
  if (fibers.size() < threads) fibers.resize(threads);
  std::memset(vote_buf, 0, sizeof(vote_buf));
  for (uint32_t t = 0; t < threads; ++t) {
    Fiber &f = fibers[t];
    if (!f.stack) f.stack.reset(new char[STACK]);
    getcontext(&f.ctx);
    f.ctx.uc_stack.ss_sp = f.stack.get();
    f.ctx.uc_stack.ss_size = STACK;
    f.ctx.uc_link = &scheduler;
    makecontext(&f.ctx, fiber_main, 0);
    f.state = READY;
    f.votes = 0;
  }
  auto all = [&](uint32_t a, uint32_t b, State s) {
    bool some = false;
    for (uint32_t t = a; t < b; ++t) {
      if (fibers[t].state != s && fibers[t].state != ENDED) return false;
      some |= fibers[t].state == s;
    }
    return some;
  };
  for (;;) {
    bool ran = false;
    for (uint32_t w = 0; w < threads; w += 64) {
      const uint32_t e = std::min(threads, w + 64);
      do {
        for (uint32_t t = w; t < e; ++t)
          if (fibers[t].state == READY) {
            ran = true;
            now = t;
            swapcontext(&scheduler, &fibers[t].ctx);
          }
        if (!all(w, e, AT_WAVE)) break;
        for (uint32_t t = w; t < e; ++t)
          if (fibers[t].state == AT_WAVE) fibers[t].state = READY;
      } while (true);
    }
    if (all(0, threads, AT_BLOCK)) {
      for (uint32_t t = 0; t < threads; ++t)
        if (fibers[t].state == AT_BLOCK) fibers[t].state = READY;
      continue;
    }
    bool ended = true;
    for (uint32_t t = 0; t < threads; ++t) ended &= fibers[t].state == ENDED;
    if (ended) return;
    if (!ran) {
      std::printf("a barrier that not every thread reaches\n");
      std::exit(1);
    }
  }
}

// ---------------------------------------------------------------- the graphs
using Rows = std::vector<std::vector<int32_t>>;  // local columns, ascending

static Rows from_edges(int32_t n, const std::set<std::pair<int32_t, int32_t>> &edges) {
  Rows r(n);
  for (auto [a, b] : edges) {
    r[a].push_back(b);
    r[b].push_back(a);
  }
  for (auto &x : r) std::sort(x.begin(), x.end());
  return r;
}

static Rows graph(const char *kind, int32_t n, std::mt19937 &rng) {
  std::set<std::pair<int32_t, int32_t>> e;
  auto add = [&](int32_t a, int32_t b) {
    if (a != b) e.insert({std::min(a, b), std::max(a, b)});
  };
  if (!std::strcmp(kind, "regular")) {
    for (int32_t v = 0; v < n; ++v)
      for (int32_t d = 1; d <= 3; ++d) add(v, (v + d) % n);
  } else if (!std::strcmp(kind, "random")) {
    for (int64_t i = 0; i < 12 * (int64_t)n; ++i) add((int32_t)(rng() % n), (int32_t)(rng() % n));
  } else if (!std::strcmp(kind, "hub_first")) {
    for (int32_t v = 1; v < n; ++v) add(0, v);
  } else {  // hub_last: a star around the last row and a few pairs
    for (int32_t v = 0; v + 1 < n; ++v) add(n - 1, v);
    for (int32_t v = 0; v + 1 < n; v += 5) add(v, v + 1);
  }
  return from_edges(n, e);
}

static int failures = 0;
#define EXPECT(c, ...)                 \
  do {                                 \
    if (!(c)) {                        \
      std::printf("FAIL " __VA_ARGS__); \
      std::printf("\n");               \
      ++failures;                      \
      return;                          \
    }                                  \
  } while (0)

static void check(const std::vector<Rows> &gs, int32_t log2T, const char *what) {
  const int32_t G = (int32_t)gs.size();
  std::vector<int64_t> off(1, 0);
  std::vector<int32_t> rp(1, 0), ci;
  int32_t n_max = 0;
  for (const Rows &r : gs) {
    const int32_t lo = (int32_t)off.back();
    for (const auto &row : r) {
      for (int32_t u : row) ci.push_back(lo + u);
      rp.push_back((int32_t)ci.size());
    }
    off.push_back(lo + (int64_t)r.size());
    n_max = std::max(n_max, (int32_t)r.size());
  }
  const int64_t n = off.back(), nnz = (int64_t)ci.size();
  const bool wide = log2T >= 4;
  // heap blocks of exactly the workspace's sizes
  std::vector<uint16_t> ord(n, 0xffff);
  std::vector<int2> slices(std::max(mqo::ell_slice_base(n, G), mqo::wide_slice_base(n, G)), int2{-1, -1});
  std::vector<uint4> blocks(mqo::ell_block_base(n, nnz, G) * 64, uint4{~0u, ~0u, ~0u, ~0u});
  const int32_t zrow = (std::max(n_max, 256) + 31) & ~31;
  ci.push_back(0);  // (an empty vector has no address)
  for (int32_t g = 0; g < G; ++g) {
    body = [&] { mqo::k_ell_order(rp.data(), off.data(), ord.data(), slices.data()); };
    run_block(1024, g, 0);
  }
  for (int32_t g = 0; g < G; ++g) {
    if (wide) {
      body = [&] {
        mqo::k_wide_build(rp.data(), ci.data(), off.data(), log2T, zrow, ord.data(), slices.data(), blocks.data());
      };
      run_block(1024, g, 0);
    } else {
      body = [&] {
        mqo::k_ell_slots(rp.data(), ci.data(), off.data(), log2T, zrow, ord.data(), slices.data(), blocks.data());
      };
      for (int32_t y = 0; y < (n_max + 255) / 256; ++y) run_block(256, g, y);
    }
  }
  const int32_t R = wide ? mqo::wide_rows(log2T) : 64, sh = log2T + 2;
  for (int32_t g = 0; g < G; ++g) {
    const Rows &r = gs[g];
    const int32_t ng = (int32_t)r.size();
    std::vector<char> seen(ng, 0);
    for (int32_t i = 0; i < ng; ++i) {
      const int32_t v = ord[off[g] + i];
      EXPECT(v < ng && !seen[v], "%s T %d graph %d of %d rows: place %d holds row %d", what, 1 << log2T, g, ng, i, v);
      seen[v] = 1;
    }
    const int2 *sl = slices.data() + (wide ? mqo::wide_slice_base(off[g], g) : mqo::ell_slice_base(off[g], g));
    const uint4 *bl = blocks.data() + mqo::ell_block_base(off[g], rp[off[g]], g) * 64;
    for (int32_t i = 0; i < ng; ++i) {
      const std::vector<int32_t> &row = r[ord[off[g] + i]];
      const int2 s = sl[i / R];
      std::vector<int32_t> got;
      for (int32_t b = 0; b < s.y; ++b) {
        const uint4 q = bl[(int64_t)(s.x + b) * R + i % R];
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
        for (int32_t k = 0; k < (wide ? 4 : 8); ++k) {
          const uint32_t at = wide ? w[k] : (w[k >> 1] >> (16 * (k & 1))) & 0xffffu;
          EXPECT((at & ((1u << sh) - 1)) == 0, "%s T %d rows %d: entry inside a row", what, 1 << log2T, ng);
          const int32_t u = (int32_t)(at >> sh);
          if (u < zrow) got.push_back(u);  // else a row of zeros
          EXPECT(u < zrow + (wide ? 1 : 32), "%s T %d rows %d: entry past the zero rows", what, 1 << log2T, ng);
        }
      }
      EXPECT(got == row, "%s T %d graph %d of %d rows: row %d has other entries", what, 1 << log2T, g, ng,
             (int)ord[off[g] + i]);
    }
  }
  std::printf("ok %s T %d rows %d\n", what, 1 << log2T, n_max);
}

int main(int argc, char **argv) {
  const int32_t log2T = std::atoi(argv[1]);
  std::mt19937 rng(12345u + (unsigned)log2T);
  for (int a = 2; a < argc; ++a) {
    const int32_t n = std::atoi(argv[a]);
    for (const char *kind : {"regular", "random", "hub_first", "hub_last"}) {
      check({graph(kind, n, rng)}, log2T, kind);
      if (failures) return 1;
    }
    // neighbours in the workspace: ranges that overlap would show
    check({graph("hub_first", std::max(1, n / 2), rng), graph("random", n, rng), graph("random", 1, rng),
           graph("hub_last", std::max(1, n / 3), rng), graph("regular", n, rng)},
          log2T, "batch");
    if (failures) return 1;
  }
  std::printf("0 failure(s)\n");
  return 0;
}

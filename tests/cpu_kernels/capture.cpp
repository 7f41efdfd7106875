// Plan builds and applies recorded into graphs or left in flight, on a host build of
// libsalt: the sequence named by argv[1] with argv[2] tokens, every replay compared with the
// eager result of the same maps (integer inputs, bit for bit).  The maps differ
// in their group sizes, at equal tile counts, as a graph's launches need.
// Prints "ok" or the first difference.  Test infrastructure only.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <random>
#include <vector>

#include "salt.h"

namespace {
constexpr int IN = 72, OUT = 40, C = 4, RC = 8, SLOTS = 12;
std::mt19937 rng(2608);

void need(bool ok, const char* what, int a = 0) {
  if (ok) return;
  printf("FAIL %s (%d)\n", what, a);
  exit(1);
}
// bf16 integers of -2 .. 2
std::vector<uint16_t> ints(size_t n) {
  std::vector<uint16_t> v(n);
  for (auto& x : v) {
    const float f = (float)((int)(rng() % 5) - 2);
    uint32_t u;
    memcpy(&u, &f, 4);
    x = (uint16_t)(u >> 16);
  }
  return v;
}

struct Maps {
  std::vector<int32_t> c, u;
};
// T tokens in C groups of T / C plus skew[g]: no group's tile count changes with
// the skews used here
Maps make_maps(int T, const int (&skew)[C]) {
  Maps m;
  for (int g = 0; g < C; ++g) m.c.insert(m.c.end(), T / C + skew[g], g);
  for (int t = 0; t < T; ++t) m.u.push_back(t % 13 == 5 ? -1 : (int)(rng() % SLOTS));
  m.u[0] = 1;                                   // (slot 1 has the largest rank)
  for (int t = T - 1; t > 0; --t) {
    const int k = (int)(rng() % (t + 1));
    std::swap(m.c[t], m.c[k]);
    std::swap(m.u[t], m.u[k]);
  }
  return m;
}

struct Bench {
  salt_ctx* ctx = nullptr;
  salt_plan* plan = nullptr;
  hipStream_t s = nullptr;
  std::vector<uint16_t> x, y0, y;
  explicit Bench(int max_T) : x(ints((size_t)max_T * IN)), y0(ints((size_t)max_T * OUT)), y(y0) {
    salt_shape sh{IN, OUT};
    salt_config cfg{};
    cfg.dtype = SALT_BF16;
    cfg.n_tables = 1;
    cfg.tables = &sh;
    cfg.n_centroids = C;
    cfg.r_c = RC;
    cfg.n_slots = SLOTS;
    cfg.r_u_max = 2;
    cfg.max_tokens = max_T;
    need(salt_create(&cfg, &ctx) == SALT_OK, "create");
    const auto at = ints((size_t)C * RC * IN), b = ints((size_t)C * RC * OUT);
    need(salt_pin_centroids(ctx, 0, 0, C, at.data(), b.data()) == SALT_OK, "pin");
    for (int i = 0; i < SLOTS; ++i) {
      const int r = 1 + i % 2;
      void* p = nullptr;
      const auto v = ints((size_t)r * (IN + OUT));
      need(salt_host_alloc(2 * v.size(), &p) == SALT_OK, "host alloc");
      memcpy(p, v.data(), 2 * v.size());
      need(salt_load_residual(ctx, i, r, p, 2 * v.size()) == SALT_OK, "load");
      need(salt_wait_loads(ctx) == SALT_OK, "wait");
      salt_host_free(p);
    }
    need(salt_plan_create(ctx, &plan) == SALT_OK, "plan");
    need(hipStreamCreateWithFlags(&s, hipStreamNonBlocking) == hipSuccess, "stream");
  }
  salt_status set(const Maps& m) {
    return salt_plan_set_maps(ctx, plan, (int)m.c.size(), m.c.data(), m.u.data(), nullptr, s);
  }
  salt_status build() { return salt_plan_build(ctx, plan, s); }
  salt_status apply() { return salt_apply(ctx, 0, plan, x.data(), y.data(), s); }
  void reset() { memcpy(y.data(), y0.data(), 2 * y.size()); }   // (the launches keep y's address)
  std::vector<uint16_t> eager(const Maps& m) {
    reset();
    need(set(m) == SALT_OK && build() == SALT_OK && apply() == SALT_OK, salt_last_error(ctx));
    return y;
  }
};

// of the same batch on a context of its own
std::vector<std::vector<uint16_t>> expected(Bench& b, const std::vector<Maps>& maps) {
  salt_plan* p = nullptr;
  need(salt_plan_create(b.ctx, &p) == SALT_OK, "plan");
  std::swap(p, b.plan);
  std::vector<std::vector<uint16_t>> out;
  for (const Maps& m : maps) out.push_back(b.eager(m));
  std::swap(p, b.plan);
  salt_plan_destroy(b.ctx, p);
  return out;
}
std::vector<Maps> all_maps(int T) {
  return {make_maps(T, {0, 0, 0, 0}), make_maps(T, {-1, 2, -2, 1}), make_maps(T, {3, -1, 0, -2})};
}
}  // namespace

int main(int argc, char** argv) {
  need(argc == 3, "usage: capture SEQUENCE TOKENS");
  const char* seq = argv[1];
  const int T = atoi(argv[2]);
  Bench b(std::max(T, 200));
  const auto maps = all_maps(T);
  const auto want = expected(b, maps);
  auto same = [&](int k, const char* what) { need(b.y == want[(size_t)k], what, k); };
  if (!strcmp(seq, "apply_then_build")) {
    // an apply recorded before any build of the plan is
    b.eager(maps[0]);
    salt_cpu_begin_capture(b.s);
    need(b.apply() == SALT_OK, "captured apply");
    salt_cpu::Graph* apply = salt_cpu_end_capture();
    need(b.set(maps[1]) == SALT_OK, "set");
    salt_cpu_begin_capture(b.s);
    need(b.build() == SALT_OK, "captured build");
    salt_cpu::Graph* build = salt_cpu_end_capture();
    for (int k : {1, 2, 0, 1}) {
      need(b.set(maps[k]) == SALT_OK, "set");
      b.reset();
      salt_cpu_replay(*build);
      salt_cpu_replay(*apply);
      same(k, "replayed build and apply");
    }
    for (int k : {2, 0}) {
      need(b.set(maps[k]) == SALT_OK && b.build() == SALT_OK, "eager build");
      b.reset();
      salt_cpu_replay(*apply);
      same(k, "eager build, replayed apply");
    }
  } else if (!strcmp(seq, "two_sizes")) {
    // graphs of two batch sizes on one plan, replayed in turn
    const auto small = all_maps(200);
    const auto want_small = expected(b, small);
    salt_cpu::Graph* g[2];
    for (int i = 0; i < 2; ++i) {
      need(b.set(i ? small[0] : maps[0]) == SALT_OK, "set");
      salt_cpu_begin_capture(b.s);
      need(b.build() == SALT_OK && b.apply() == SALT_OK, "captured build and apply");
      g[i] = salt_cpu_end_capture();
    }
    for (int k : {0, 1, 2, 0})
      for (int i = 0; i < 2; ++i) {
        need(b.set(i ? small[k] : maps[k]) == SALT_OK, "set");
        b.reset();
        salt_cpu_replay(*g[i]);
        need(b.y == (i ? want_small : want)[(size_t)k], i ? "small batch" : "large batch", k);
      }
  } else if (!strcmp(seq, "maps_in_capture")) {
    // the maps of a fresh plan set inside the capture; a second batch there is
    // refused and leaves plan, context and capture as they were
    salt_cpu_begin_capture(b.s);
    need(b.set(maps[0]) == SALT_OK, "captured set");
    need(b.build() == SALT_OK && b.apply() == SALT_OK, "captured build and apply");
    need(b.set(maps[1]) == SALT_ERR_BAD_STATE, "a second batch in the capture");
    need(b.apply() == SALT_OK, "captured apply");
    salt_cpu::Graph* g = salt_cpu_end_capture();
    g->pop_back(), g->pop_back();                 // (the second apply's two launches)
    int last = 0;
    for (int k : {-1, -1, 1, 2, -1, 0, 1}) {      // (-1: no new maps)
      if (k >= 0) need(b.set(maps[last = k]) == SALT_OK, "set");
      b.reset();
      salt_cpu_replay(*g);
      same(last, "replay");
    }
    salt_cpu_begin_capture(b.s);
    need(b.set(maps[0]) == SALT_ERR_BAD_STATE, "maps in a second capture");
    salt_cpu_end_capture();
    need(b.eager(maps[2]) == want[2], "eager after the captures");
  } else if (!strcmp(seq, "batches_in_flight")) {
    // many batches of one plan, none waited for by the caller: each must find its
    // own maps in the staging buffers; and no event stands between a build and the
    // shrink behind it
    salt_cpu::g_lazy = true;
    std::vector<std::vector<uint16_t>> ys(9, b.y0);
    for (int i = 0; i < 9; ++i) {
      need(b.set(maps[i % 3]) == SALT_OK, "set", i);
      const int events = salt_cpu::g_events_recorded;
      need(b.build() == SALT_OK, "build", i);
      if (i == 4) need(b.build() == SALT_OK, "second build", i);
      need(salt_apply(b.ctx, 0, b.plan, b.x.data(), ys[i].data(), b.s) == SALT_OK, "apply", i);
      need(salt_cpu::g_events_recorded == events, "an event among build and apply", i);
    }
    need(hipStreamSynchronize(b.s) == hipSuccess, "synchronize");
    for (int i = 0; i < 9; ++i) need(ys[i] == want[i % 3], "batch", i);
    salt_cpu::g_lazy = false;
  } else if (!strcmp(seq, "maps_in_capture_built_outside")) {
    salt_cpu_begin_capture(b.s);
    need(b.set(maps[0]) == SALT_OK, "captured set");
    salt_cpu_end_capture();
    b.reset();
    need(b.build() == SALT_OK && b.apply() == SALT_OK, "eager build");
    same(0, "eager build of captured maps");
    need(b.eager(maps[1]) == want[1], "eager after it");
  } else {
    need(false, "no such sequence");
  }
  printf("ok\n");
  return 0;
}

// salt_adapter_gram's host side, on a host build of libsalt, over tables of which one
// is much wider than the others: what argv[1] names, with adapters of ranks argv[2]
// and argv[3] (integer factors; every result bit for bit).
//   first_call  the first call of a context allocates no page-locked memory
//   scratch     the scratch holds the tables' own K chunks, not the widest table's for each
//   no_memory   a device without room for the chunks' Grams still answers
// Prints "ok" or what failed.  Test infrastructure only.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <random>
#include <vector>

#include "salt.h"

namespace {
std::mt19937 rng(2608);
void need(bool ok, const char* what, double a = 0) {
  if (ok) return;
  printf("FAIL %s (%g)\n", what, a);
  exit(1);
}
struct Adapter {
  std::vector<uint16_t> bits;     // bf16
  std::vector<double> v;
  explicit Adapter(size_t n) : bits(n), v(n) {
    for (size_t i = 0; i < n; ++i) {
      const float f = (float)((int)(rng() % 5) - 2);
      uint32_t u;
      memcpy(&u, &f, 4);
      bits[i] = (uint16_t)(u >> 16);
      v[i] = f;
    }
  }
};
// sum over i, j of (X1_i . X2_j) (Y1_i . Y2_j)
double trace(const double* x1, const double* x2, int in, const double* y1, const double* y2, int out, int r1, int r2) {
  double s = 0;
  for (int i = 0; i < r1; ++i)
    for (int j = 0; j < r2; ++j) {
      double a = 0, b = 0;
      for (int k = 0; k < in; ++k) a += x1[(size_t)i * in + k] * x2[(size_t)j * in + k];
      for (int k = 0; k < out; ++k) b += y1[(size_t)i * out + k] * y2[(size_t)j * out + k];
      s += a * b;
    }
  return s;
}
}  // namespace

int main(int argc, char** argv) {
  need(argc == 4, "usage: gram CHECK R1 R2");
  const char* check = argv[1];
  const int r1 = atoi(argv[2]), r2 = atoi(argv[3]);
  const std::vector<salt_shape> tabs = {{8, 24}, {40, 8}, {1032, 64}, {16, 12288}, {24, 8}, {64, 1024}};
  salt_config cfg{};
  cfg.dtype = SALT_BF16;
  cfg.n_tables = (int)tabs.size();
  cfg.tables = tabs.data();
  cfg.n_slots = cfg.max_tokens = 1;
  salt_ctx* ctx = nullptr;
  need(salt_create(&cfg, &ctx) == SALT_OK, "create");
  size_t sum = 0, chunks = 0;
  for (const salt_shape& s : tabs) {
    sum += s.in_dim + s.out_dim;
    chunks += (s.in_dim + 1023) / 1024 + (s.out_dim + 1023) / 1024;
  }
  const Adapter a(sum * r1), b(sum * r2);
  std::vector<double> got(3 * tabs.size());
  const size_t p1 = (r1 + 15) / 16 * 16, p2 = (r2 + 15) / 16 * 16, side = 4 * (p1 * p2 + p1 * p1 + p2 * p2);
  if (!strcmp(check, "no_memory")) salt_cpu::g_malloc_limit = 2 * tabs.size() * side;
  const int before = salt_cpu::g_host_mallocs;
  salt_cpu::g_last_malloc = 0;
  need(salt_adapter_gram(ctx, a.bits.data(), r1, b.bits.data(), r2, got.data(), nullptr) == SALT_OK, salt_last_error(ctx));
  if (!strcmp(check, "first_call")) need(salt_cpu::g_host_mallocs == before, "page-locked memory allocated");
  if (!strcmp(check, "scratch")) need(salt_cpu::g_last_malloc <= chunks * side, "scratch bytes", (double)salt_cpu::g_last_malloc);
  size_t o = 0;
  for (size_t t = 0; t < tabs.size(); ++t) {
    const int in = tabs[t].in_dim, out = tabs[t].out_dim;
    const double *a1 = &a.v[o * r1], *b1 = a1 + (size_t)r1 * in, *a2 = &b.v[o * r2], *b2 = a2 + (size_t)r2 * in;
    const double want[3] = {trace(a1, a2, in, b1, b2, out, r1, r2), trace(a1, a1, in, b1, b1, out, r1, r1),
                            trace(a2, a2, in, b2, b2, out, r2, r2)};
    for (int k = 0; k < 3; ++k) need(got[3 * t + k] == want[k], "result", (double)(3 * t + k));
    o += in + out;
  }
  salt_destroy(ctx);
  printf("ok\n");
  return 0;
}

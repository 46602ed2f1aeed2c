// CPU driver of the library's work splits (fd_plans.hpp), built with the address
// and undefined-behaviour sanitizers by tests/test_host_plans.py.  A mode per
// property; the exit status is 0 when it holds, and the first failures are
// printed.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>

#include "fd_plans.hpp"

using namespace fd;

static int failures = 0;
static void fail(const char* what, long long a, long long b, long long need, long long have) {
  if (++failures <= 5)
    std::fprintf(stderr, "%s: %lld within %lld needs %lld, has %lld\n", what, a, b, need, have);
}

// Every plan of a prefix fits the partial sums carved for the longest one:
// all pairs of block counts up to 800, and prefixes of long sets.
static void prefixes() {
  const int64_t block = 4 * SYM_NIB * TILE;
  auto check = [&](int64_t k, int64_t nmax) {
    const size_t have = std::max(part_rows_bound(nmax * block, nmax * block),
                                 sym_part_rows_within(nmax * block, SYM_NIB));
    const size_t sym = sym_part_rows(k * block, SYM_NIB);
    if (sym > have) fail("symmetric row sums", k, nmax, (long long)sym, (long long)have);
    const KVPlan p = plan_rowsum(k * block, nmax * block, 4);
    const size_t plain = size_t(p.nsplit) * size_t(k * block);
    if (plain > have) fail("row sums", k, nmax, (long long)plain, (long long)have);
  };
  size_t running = 0;
  for (int64_t nmax = 1; nmax <= 800; ++nmax) {
    running = std::max(running, sym_part_rows(nmax * block, SYM_NIB));
    if (running != sym_part_rows_within(nmax * block, SYM_NIB))
      fail("maximum", nmax, nmax, (long long)running,
           (long long)sym_part_rows_within(nmax * block, SYM_NIB));
    for (int64_t k = 1; k <= nmax; k += nmax < 200 ? 1 : 7) check(k, nmax);
  }
  for (int64_t nmax : {2047, 2048, 2049, 2050, 4096, 5000})
    for (int64_t k = 1; k <= nmax; ++k) check(k, nmax);
  const int64_t top = (int64_t(1) << 30) / block;
  for (int64_t k = 2049; k <= top; k += 997) check(k, top);
  check(top, top);
}

// Products of every width in the partial products carved for the largest sizes.
static void products() {
  for (int64_t nr : {1, 300, 512, 513, 5000, 20000, 65536, 300000})
    for (int64_t nc : {1, 513, 16384, 30011, 65536, 262145, 4000000})
      for (int b : {2, 16, 17, 64})
        for (int dp : {4, 12, 64})
          for (int64_t grow : {1, 2, 3}) {
            const KVPlan p = plan_product(nr, nc, dp, b);
            const int64_t npad = round_up(nr, ROW_PAD);
            const size_t have = part_rows_bound(round_up(nr * grow, ROW_PAD), nc * grow);
            if (size_t(p.nsplit) * size_t(npad) > have)
              fail("product", nr, nc, (long long)p.nsplit * npad, (long long)have);
          }
}

// The single column's sums: contributions of waves next to the smallest weight of
// the widest column, one per 256 rows, rounded, gathered four at a time, split
// into two words and put together again, against their exact sum; and the
// largest contributions a workgroup gathers.
static void columns() {
  std::mt19937_64 rng(7);
  const double unit = std::ldexp(1.0, WIDE_FRAC);
  auto total = [&](int64_t count, auto value, long double& exact) {
    uint64_t hi = 0, lo = 0;
    exact = 0;
    for (int64_t k = 0; k < count; k += 4) {
      uint64_t word = 0;
      for (int e = 0; e < 4; ++e) {
        const float v = value();
        exact += (long double)v;
        word += uint64_t(std::llrint(double(v) * unit));
      }
      hi += uint64_t(int64_t(word) >> WIDE_SPLIT);
      lo += word & ((uint64_t(1) << WIDE_SPLIT) - 1);
    }
    return (double(int64_t(hi)) * double(uint64_t(1) << WIDE_SPLIT) + double(lo)) / unit;
  };
  for (int e = 9; e <= 30; ++e) {
    const int64_t npad = int64_t(1) << e, count = std::max<int64_t>(4, npad / 256);
    const double own = 0.5 / double(column_range(npad));
    for (double spread : {1.0, 1e-3, 1e-7}) {
      std::uniform_real_distribution<double> u(-1.0, 1.0);
      long double exact = 0;
      const double got = total(count, [&] { return float(own * spread * u(rng)); }, exact);
      const double err = std::fabs(double((long double)got - exact));
      if (err > std::ldexp(own, -18)) fail("column sum, 2^-60", e, 0, (long long)(err * 0x1p60), (long long)(std::ldexp(own, -18) * 0x1p60));
    }
  }
  // 128 rows of the largest weight, with kernel values a little above 1
  for (float v : {128.f * 1.0001f, -128.f * 1.0001f}) {
    long double exact = 0;
    const double got = total(1 << 20, [&] { return v; }, exact);
    if (std::fabs(got - double(exact)) > std::fabs(double(exact)) * 1e-15)
      fail("largest column", 0, 0, (long long)exact, (long long)got);
  }
}

int main(int argc, char** argv) {
  if (argc == 2 && !std::strcmp(argv[1], "prefixes")) prefixes();
  else if (argc == 2 && !std::strcmp(argv[1], "products")) products();
  else if (argc == 2 && !std::strcmp(argv[1], "columns")) columns();
  else return 2;
  std::printf("%d failures\n", failures);
  return failures ? 1 : 0;
}

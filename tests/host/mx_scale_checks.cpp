// Scale of the matrix-core pair kernel's whole numbers: for the longest launches
// and series that alternate, jump or have one large value, the numbers fit their
// four digits, the energies by digit products are exact, and every sum of
// squared differences stays below 2^64 (and so is what the kernel's arithmetic
// modulo 2^64 gives).
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <functional>
#include <random>
#include <vector>

#include "pair_matrix.hpp"

using namespace nfs;

static long long g_fail = 0, g_checks = 0;
#define CHECK(c, ...)                                             \
  do {                                                            \
    ++g_checks;                                                   \
    if (!(c) && ++g_fail <= 20) {                                 \
      std::printf("FAIL %s:%d: ", #c, __LINE__);                  \
      std::printf(__VA_ARGS__);                                   \
      std::printf("\n");                                          \
    }                                                             \
  } while (0)

namespace {

// Most targets of one launch over all spans of delays.
int64_t longest_launch() {
  int64_t best = 0;
  for (int64_t ta = 1; ta < 3; ++ta)
    for (int64_t tb : {ta, ta + 15, ta + 100, ta + 599})
      for (int64_t n = 1500; n < 2400; ++n)
        best = std::max(best, mx_cut(ta, ta + n, ta, std::min(tb, ta + n - 1)) - ta);
  return best;
}

void check_series(const char* what, const std::vector<float>& x, const std::vector<float>& y) {
  float energy = 0.f;
  for (size_t t = 0; t < x.size(); ++t) energy = std::fma(x[t], x[t], std::fma(y[t], y[t], energy));
  if (!(energy <= kMxMost) || energy < kMxFew) return;
  uint32_t bits;
  const float roomy = kMxRoom * energy;
  std::memcpy(&bits, &roomy, 4);
  const int ex = mx_exponent(bits);
  std::vector<int64_t> q[2];
  double squares = 0.0;
  for (int comp = 0; comp < 2; ++comp)
    for (size_t t = 0; t < x.size(); ++t) {
      const int64_t v = int64_t(std::rint(std::ldexp(comp ? y[t] : x[t], ex)));
      CHECK(std::llabs(v) < (int64_t(1) << 31) - (1 << 24), "%s: %lld", what, (long long)v);
      const uint32_t w = (uint32_t(int32_t(v)) + 0x808080u) ^ 0x808080u;
      int64_t back = 0;
      for (int d = 0; d < 4; ++d) back += int64_t(int8_t(w >> (8 * d))) * (int64_t(1) << (8 * d));
      CHECK(back == v, "%s: digits of %lld", what, (long long)v);
      q[comp].push_back(v);
      squares += double(v) * double(v);
    }
  CHECK(squares > 0x1.dp59 && squares < 0x1.fp61, "%s: squares %g", what, squares);
  for (size_t tau : {size_t(1), size_t(2), size_t(3), x.size() / 2, x.size() - 1}) {
    uint64_t S = 0;
    long double exact = 0;
    for (size_t t = tau; t < x.size(); ++t)
      for (int comp = 0; comp < 2; ++comp) {
        const int64_t d = q[comp][t] - q[comp][t - tau];
        S += uint64_t(d) * uint64_t(d);
        exact += (long double)(d) * (long double)(d);
      }
    CHECK(exact < 0x1p64L && std::fabs((long double)(S) - exact) <= exact * 0x1p-50L,
          "%s: delay %zu sum %.6Lg", what, tau, exact);
  }
}

}  // namespace

int main() {
  const int64_t most = longest_launch();
  CHECK(most > 2048, "longest launch %lld", (long long)most);
  std::mt19937 rng(3);
  std::normal_distribution<float> normal;
  const float top = std::nextafter(2.f, 0.f);  // the top of a binade
  for (int64_t n : {int64_t(2), int64_t(17), int64_t(900), int64_t(2048), most + 1})
    for (int shift : {-40, -3, 0, 9, 40}) {
      const float u = std::ldexp(1.f, shift);
      auto series = [&](const char* what, std::function<float(int64_t)> f,
                        std::function<float(int64_t)> g) {
        std::vector<float> x, y;
        for (int64_t t = 0; t < n; ++t) {
          x.push_back(f(t) * u);
          y.push_back(g(t) * u);
        }
        check_series(what, x, y);
      };
      auto sign = [](int64_t t) { return t % 2 ? -1.f : 1.f; };
      series("alternating at a binade's top", [&](int64_t t) { return top * sign(t); },
             [&](int64_t t) { return top * sign(t); });
      series("alternating", [&](int64_t t) { return 1.4143f * sign(t); },
             [&](int64_t t) { return -1.4141f * sign(t); });
      series("halves", [&](int64_t t) { return t < n / 2 ? top : -top; }, [](int64_t) { return 0.f; });
      series("one large value", [&](int64_t t) { return t == n / 2 ? 3e4f : normal(rng); },
             [&](int64_t) { return normal(rng); });
      series("noise", [&](int64_t) { return normal(rng); }, [&](int64_t) { return normal(rng); });
    }
  std::printf("%lld checks, %lld failures, longest launch %lld\n", g_checks, g_fail,
              (long long)most);
  return g_fail ? 1 : 0;
}

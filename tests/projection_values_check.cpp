// Host-only check of the projection's vectorised values (built by
// tests/test_projection_values.py): the library's source is included, so that
// its internal evaluations can be compared with the definition through the C
// library's log, cos and sqrt.  Every value must have the definition's bits,
// with and without wide vectors, and the polynomials must stay within the
// margin that decides when the definition is evaluated instead.
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "arc_projection.cpp"

int main(int argc, char** argv) {
  const long blocks = argc > 1 ? std::atol(argv[1]) : 20000;
  double worst = 0.0;
  long bad = 0, again = 0, total = 0;
  double u1[arc::kBoxMullerBlock], u2[arc::kBoxMullerBlock];
  float got[arc::kBoxMullerBlock], plain[arc::kBoxMullerBlock];
  int32_t sure[arc::kBoxMullerBlock];
  auto check = [&](int n) {
    arc::box_muller_block(u1, u2, n, got);
    arc::box_muller_lanes(u1, u2, n, plain, sure);
    for (int k = 0; k < n; ++k) {
      const double radius = std::sqrt(-2.0 * std::log(u1[k]));
      const double z = radius * std::cos(arc::kTwoPi * u2[k]);
      const float want = static_cast<float>(z);
      const double fast =
          std::sqrt(-2.0 * arc::fast_log(u1[k])) * arc::fast_cos(arc::kTwoPi * u2[k]);
      if (radius > 0.0) worst = std::max(worst, std::fabs(fast - z) / radius);
      uint32_t a, b, c;
      std::memcpy(&a, &want, 4);
      std::memcpy(&b, &got[k], 4);
      std::memcpy(&c, &plain[k], 4);
      if (a != b || (sure[k] && a != c)) {
        if (bad++ < 10) std::printf("u1 %a u2 %a: %a, want %a\n", u1[k], u2[k], got[k], want);
      }
      again += !sure[k];
      ++total;
    }
  };
  const double ulp = 0x1p-53;
  // The ends of both intervals, the neighbourhoods of sqrt(1/2) and of powers
  // of two, and the angles around every multiple of pi/4.
  int n = 0;
  for (int i = 0; i < 200; ++i)
    for (int j = 0; j < 200; ++j) {
      const double e1[8] = {1.0 - i * ulp, (i + 1) * ulp, 0.5 + (i - 100) * ulp,
                            0.7071067811865475 + (i - 100) * ulp, 0x1p-20 + (i - 100) * ulp,
                            (i + 1) / 201.0, 1.0 - (i + 1) * 0x1p-30, 0.25 + (i - 100) * ulp};
      for (int s = 0; s < 8; ++s) {
        u1[n] = e1[s];
        const double at = (j % 9) / 8.0 + (j / 9 - 11) * ulp * (s < 4 ? 1.0 : 1e6);
        u2[n] = std::min(std::max(at, 0.0), 1.0 - ulp);
        if (++n == arc::kBoxMullerBlock) {
          check(n);
          n = 0;
        }
      }
    }
  for (long b = 0; b < blocks; ++b) {
    arc::SplitMix64 gen(static_cast<uint64_t>(b) * 1000003u + 17u, 0);
    const int cnt = 1 + static_cast<int>(b % arc::kBoxMullerBlock);
    for (int k = 0; k < cnt; ++k) {
      u1[k] = static_cast<double>((gen.next() >> 11) + 1) * ulp;
      u2[k] = static_cast<double>(gen.next() >> 11) * ulp;
    }
    check(cnt);
  }
  std::printf("values %ld, evaluated again %ld, worst %.3g of the radius\n", total, again, worst);
  const bool ok = bad == 0 && worst < 3e-15;
  std::printf("%s\n", ok ? "ok" : "FAIL");
  return !ok;
}

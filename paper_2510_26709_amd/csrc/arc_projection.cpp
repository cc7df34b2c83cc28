// Shared Gaussian projection V_t of ARC-Top-K (Sec. IV, Alg. 1: every node
// derives the same V in R^{n x r}, vec(V) ~ N(0, I), from a shared seed).
//
// Generator: SplitMix64 (Steele, Lea & Flood, OOPSLA 2014).  Its state starts
// at the seed and advances by the golden gamma before each output, which is
// the state passed through the variant-13 mixer.  Entry (j, k) of step t uses
// outputs 2c and 2c+1 of the stream, c = (t*n + j)*r + k, as two 53-bit
// uniforms u1 in (0, 1] and u2 in [0, 1), and the cosine branch of the
// Box-Muller transform in binary64, rounded once to binary32.  The result is
// fully determined by (seed, t, n, r) and is identical on every node.
//
// The values are those of the C library's log, cos and sqrt.  Calling them
// costs 44 ns a value, so blocks of values go through polynomials that the
// compiler vectorises, and only a value whose rounding to binary32 their
// error could change is computed again with the library's functions.
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

#include "arc_internal.h"

namespace arc {
namespace {

constexpr uint64_t kGoldenGamma = 0x9E3779B97F4A7C15ull;

inline uint64_t splitmix_mix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// Generator positioned just before output number x of the seeded stream.
struct SplitMix64 {
  uint64_t state;
  SplitMix64(uint64_t seed, uint64_t x) : state(seed + x * kGoldenGamma) {}
  uint64_t next() {
    state += kGoldenGamma;
    return splitmix_mix(state);
  }
};

}  // namespace

namespace {

constexpr double kTwoPi = 6.283185307179586476925286766559;
constexpr double kTwoToMinus53 = 1.0 / 9007199254740992.0;

// The definition of one value.
float box_muller(double u1, double u2) {
  const double radius = std::sqrt(-2.0 * std::log(u1));
  return static_cast<float>(radius * std::cos(kTwoPi * u2));
}

inline uint64_t bits_of(double v) {
  uint64_t b;
  std::memcpy(&b, &v, sizeof b);
  return b;
}
inline double from_bits(uint64_t b) {
  double v;
  std::memcpy(&v, &b, sizeof v);
  return v;
}

// ln u for u in (0, 1], to a few units in the last place: u = m 2^e with m in
// [sqrt(1/2), sqrt 2), ln u = e ln 2 + 2 artanh(x), x = (m - 1) / (m + 1), by
// the series x + x^3/3 + x^5/5 + ... up to x^21 (|x| < 0.1716: the rest is
// below 2^-58 of the first term).
inline double fast_log(double u) {
  const uint64_t b = bits_of(u);
  // Exponent of u / sqrt(1/2), so that m lands in the interval above.
  const int64_t e =
      static_cast<int64_t>((b - 0x3fe6a09e667f3bcdull) >> 52) -
      static_cast<int64_t>(b < 0x3fe6a09e667f3bcdull ? 4096 : 0);
  const double m = from_bits(b - (static_cast<uint64_t>(e) << 52));
  // e as a double: |e| < 2^51, through the low bits of 1.5 * 2^52.
  const double ed = from_bits(0x4338000000000000ull + static_cast<uint64_t>(e)) -
                    6755399441055744.0;
  const double x = (m - 1.0) / (m + 1.0), q = x * x;
  double p = 1.0 / 21.0;
  p = p * q + 1.0 / 19.0;
  p = p * q + 1.0 / 17.0;
  p = p * q + 1.0 / 15.0;
  p = p * q + 1.0 / 13.0;
  p = p * q + 1.0 / 11.0;
  p = p * q + 1.0 / 9.0;
  p = p * q + 1.0 / 7.0;
  p = p * q + 1.0 / 5.0;
  p = p * q + 1.0 / 3.0;
  const double ln_m = 2.0 * x + 2.0 * x * (q * p);
  // ln 2 in two parts, the first of 24 bits: e times it is exact.
  return ed * 0x1.62e43p-1 + (ed * -0x1.05c610ca86c39p-29 + ln_m);
}

// cos a for a in [0, 2 pi], within a few 2^-53: a = k pi/2 + y with |y| <=
// pi/4, and the Taylor series of cos y or sin y (up to y^16 and y^17: the
// rest is below 2^-58).
inline double fast_cos(double a) {
  const double kShift = 6755399441055744.0;  // 1.5 * 2^52
  const double t = a * 0x1.45f306dc9c883p-1 + kShift;  // a / (pi/2), to a whole number
  const double k = t - kShift;
  const uint64_t quadrant = bits_of(t);  // its low two bits
  // pi/2 in three parts, the first two of 24 bits: k times them is exact.
  const double y =
      ((a - k * 0x1.921fb6p+0) - k * -0x1.777a5cp-25) - k * -0x1.ee59d9cceba4p-50;
  const double q = y * y;
  double c = 1.0 / 20922789888000.0;
  c = c * q - 1.0 / 87178291200.0;
  c = c * q + 1.0 / 479001600.0;
  c = c * q - 1.0 / 3628800.0;
  c = c * q + 1.0 / 40320.0;
  c = c * q - 1.0 / 720.0;
  c = c * q + 1.0 / 24.0;
  c = c * q - 0.5;
  c = c * q + 1.0;
  double s = 1.0 / 355687428096000.0;
  s = s * q - 1.0 / 1307674368000.0;
  s = s * q + 1.0 / 6227020800.0;
  s = s * q - 1.0 / 39916800.0;
  s = s * q + 1.0 / 362880.0;
  s = s * q - 1.0 / 5040.0;
  s = s * q + 1.0 / 120.0;
  s = s * q - 1.0 / 6.0;
  s = y + y * (q * s);
  // cos(k pi/2 + y): cos y, -sin y, -cos y, sin y for k = 0..3.
  const double v = quadrant & 1 ? s : c;
  return from_bits(bits_of(v) ^ (((quadrant + 1) & 2) << 62));
}

// Values of a block, as far as the polynomials decide them: sure[k] is 0
// where another evaluation in binary64 could round out[k] differently.  Both
// evaluations of z lie within 3e-15 radius of each other (rounding of the
// logarithm, the angle's reduction and the series, and the library's own
// units in the last place), so a margin of 1e-14 radius leaves no doubt.
inline void box_muller_lanes(const double* u1, const double* u2, int n, float* out,
                             int32_t* sure) {
  for (int k = 0; k < n; ++k) {
    const double radius = std::sqrt(-2.0 * fast_log(u1[k]));
    const double z = radius * fast_cos(kTwoPi * u2[k]);
    const double margin = radius * 1e-14;
    const float lo = static_cast<float>(z - margin), hi = static_cast<float>(z + margin);
    out[k] = lo;
    // (radius 0, for u1 = 1: the sign of the zero is the library's.)
    sure[k] = (lo == hi) & (radius > 0.0);
  }
}

#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
__attribute__((target("avx2"), flatten)) void box_muller_avx2(const double* u1, const double* u2,
                                                              int n, float* out, int32_t* sure) {
  box_muller_lanes(u1, u2, n, out, sure);
}
bool have_avx2() {
  static const bool yes = __builtin_cpu_supports("avx2");
  return yes;
}
#endif

}  // namespace

void box_muller_block(const double* u1, const double* u2, int n, float* out) {
  int32_t sure[kBoxMullerBlock];
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
  if (have_avx2())
    box_muller_avx2(u1, u2, n, out, sure);
  else
#endif
    box_muller_lanes(u1, u2, n, out, sure);
  for (int k = 0; k < n; ++k)
    if (!sure[k]) out[k] = box_muller(u1[k], u2[k]);
}

void generate_projection_rows(uint64_t seed, int64_t t, int64_t n, int32_t r, int64_t j0,
                              int64_t j1, float* V) {
  const uint64_t un = static_cast<uint64_t>(n), ur = static_cast<uint64_t>(r);
  // Entries (j, k) in order are c = (t*n + j)*r + k in order.
  const uint64_t base = static_cast<uint64_t>(t) * un * ur;
  const uint64_t end = static_cast<uint64_t>(j1) * ur;
  double u1[kBoxMullerBlock], u2[kBoxMullerBlock];
  for (uint64_t i = static_cast<uint64_t>(j0) * ur; i < end; i += kBoxMullerBlock) {
    const int cnt =
        static_cast<int>(end - i < kBoxMullerBlock ? end - i : uint64_t{kBoxMullerBlock});
    for (int k = 0; k < cnt; ++k) {
      SplitMix64 gen(seed, 2 * (base + i + static_cast<uint64_t>(k)));
      const uint64_t w1 = gen.next();
      const uint64_t w2 = gen.next();
      u1[k] = static_cast<double>(static_cast<int64_t>((w1 >> 11) + 1)) * kTwoToMinus53;
      u2[k] = static_cast<double>(static_cast<int64_t>(w2 >> 11)) * kTwoToMinus53;
    }
    box_muller_block(u1, u2, cnt, V + i);
  }
}

void generate_projection(uint64_t seed, int64_t t, int64_t n, int32_t r, float* V) {
  generate_projection_rows(seed, t, n, r, 0, n, V);
}

// ---------------------------------------------------------------------------
// ProjectionPool: the rows of every width's V_t split evenly over a few
// threads.  Each entry is a pure function of (seed, t, j, k), so the split
// changes no value.
// ---------------------------------------------------------------------------
ProjectionPool::ProjectionPool(int threads) {
  if (threads < 1) threads = 1;
  // Each thread gets the count by value: threads_ is still growing while the
  // first ones start.
  threads_.reserve(static_cast<size_t>(threads));
  for (int i = 0; i < threads; ++i) threads_.emplace_back([this, i, threads] { run(i, threads); });
}

ProjectionPool::~ProjectionPool() {
  {
    std::lock_guard<std::mutex> lk(mu_);
    quit_ = true;
  }
  cv_job_.notify_all();
  for (std::thread& th : threads_) th.join();
}

void ProjectionPool::start(uint64_t seed, int64_t t, int32_t r,
                           const std::vector<ProjectionBlock>* blocks, float* dst) {
  wait();
  std::lock_guard<std::mutex> lk(mu_);
  seed_ = seed;
  t_ = t;
  r_ = r;
  blocks_ = blocks;
  dst_ = dst;
  total_rows_ = 0;
  for (const ProjectionBlock& b : *blocks) total_rows_ += b.width;
  remaining_ = static_cast<int>(threads_.size());
  ++job_;
  cv_job_.notify_all();
}

void ProjectionPool::wait() {
  std::unique_lock<std::mutex> lk(mu_);
  cv_done_.wait(lk, [this] { return remaining_ == 0; });
}

void ProjectionPool::run(int id, int nthreads) {
  uint64_t seen = 0;
  for (;;) {
    std::unique_lock<std::mutex> lk(mu_);
    cv_job_.wait(lk, [&] { return quit_ || job_ != seen; });
    if (quit_) return;
    seen = job_;
    const uint64_t seed = seed_;
    const int64_t t = t_, total = total_rows_;
    const int32_t r = r_;
    const std::vector<ProjectionBlock>& blocks = *blocks_;
    float* dst = dst_;
    lk.unlock();
    // This thread's share [lo, hi) of the rows of all widths, in block order.
    const int64_t lo = total * id / nthreads, hi = total * (id + 1) / nthreads;
    int64_t first = 0;
    for (const ProjectionBlock& b : blocks) {
      const int64_t j0 = lo > first ? lo - first : 0;
      const int64_t j1 = hi - first < b.width ? hi - first : b.width;
      if (j0 < j1) generate_projection_rows(seed, t, b.width, r, j0, j1, dst + b.offset);
      first += b.width;
    }
    lk.lock();
    if (--remaining_ == 0) cv_done_.notify_all();
  }
}

}  // namespace arc

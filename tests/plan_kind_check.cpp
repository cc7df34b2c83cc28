// Host-only check of the static entry point's plans (built by
// tests/test_plan_kind.py, linked against the library): the kind chosen for a
// configuration near the scratch limit, and that the number of row groups by
// which it was chosen is the number in its tables, for every kind.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "arc_context.h"

namespace {
bool ok = true;
const char* const kNames[] = {"fast", "aligned", "general"};

void check(arc_config cfg, int want) {
  int64_t m = 0;
  if (arc::check_config(&cfg, &m) != ARC_OK) {
    std::printf("rejected: %s\n", arc_last_error());
    ok = false;
    return;
  }
  // Every kind in turn: refuse the first `skip` of them.
  for (int skip = 0; skip < 3; ++skip) {
    int asked = 0;
    int64_t counted = -1;
    arc_ctx c;
    const arc_status st = arc::plan_context(
        &cfg, m, nullptr,
        [&](const arc_ctx&, int64_t groups) {
          counted = groups;
          return asked++ == skip;
        },
        &c);
    if (st != ARC_OK || static_cast<int>(c.plan) != skip ||
        counted != static_cast<int64_t>(c.groups.size())) {
      std::printf("d=%lld n=%lld %s: counted %lld, filled %zu\n", (long long)cfg.d,
                  (long long)cfg.n, kNames[skip], (long long)counted, c.groups.size());
      ok = false;
    }
  }
  if (want < 0) return;
  int kinds = 0;
  arc_ctx c;
  const arc_status st = arc::plan_context(
      &cfg, m, nullptr,
      [&](const arc_ctx& p, int64_t groups) {
        ++kinds;
        return arc::static_scratch_bytes(p, groups) <= ARC_STATIC_SCRATCH_BYTES;
      },
      &c);
  const size_t bytes = arc::static_scratch_bytes(c, static_cast<int64_t>(c.groups.size()));
  if (st != ARC_OK || static_cast<int>(c.plan) != want || kinds != want + 1 ||
      bytes > ARC_STATIC_SCRATCH_BYTES) {
    std::printf("d=%lld n=%lld r=%d: %s, want %s (%zu bytes)\n", (long long)cfg.d,
                (long long)cfg.n, cfg.r, kNames[static_cast<int>(c.plan)], kNames[want], bytes);
    ok = false;
  }
}

arc_config view(int64_t d, int64_t n, int32_t N, int32_t r) {
  arc_config cfg{};
  cfg.d = d;
  cfg.n = n;
  cfg.K = 5;
  cfg.N = N;
  cfg.r = r;
  cfg.eta = 0.1f;
  return cfg;
}
}  // namespace

int main() {
  // The configurations that tests/test_zz_no_alloc.py runs on a device.
  check(view(160ll * 1'700'000 + 4, 160, 1, 8), 0);
  check(view(160ll * 1'800'000 + 4, 160, 1, 8), 1);
  check(view(260ll * 1'750'000, 260, 1, 8), 2);
  check(view(819ll * 6'900'000, 819, 1, 1), 1);
  // Counts of every kernel: rows of one to three values, spans, lines, strided
  // windows, ragged rows, r without vectorised kernels.
  for (const int64_t n : {1, 3, 4, 27, 64, 333, 819, 820, 1001, 1024, 2048, 2307, 4099, 8192})
    for (const int64_t rows : {0, 1, 7, 64, 257, 1000})
      for (const int64_t tail : {0, 1, 4, 33})
        for (const int32_t r : {3, 4}) {
          const int64_t d = n * rows + (tail < n ? tail : 0);
          if (d > 0) check(view(d, n, 2, r), -1);
        }
  std::vector<arc_tensor> t;
  int64_t d = 0;
  for (int i = 0; i < 40; ++i) {
    t.push_back({1 + i * i, 1 + (i * 37) % 900 * (i % 5 + 1), 1});
    d += t.back().rows * t.back().cols;
  }
  arc_config cfg = view(d, 0, 3, 4);
  cfg.K = 0;
  cfg.tensors = t.data();
  cfg.num_tensors = static_cast<int32_t>(t.size());
  check(cfg, 0);
  std::printf("%s\n", ok ? "ok" : "FAIL");
  return !ok;
}

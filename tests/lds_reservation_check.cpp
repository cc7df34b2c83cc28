// Host-only check of the rule for LDS reservations (built by
// tests/test_lds_reservation.py): each launch that reserves LDS to cap its
// occupancy does so only where the device gives one workgroup that much.
#include <cstdio>

#include "arc_internal.h"

int main() {
  const int64_t cu = arc::kLdsPerCu;
  bool ok = true;
  auto expect = [&](bool want, int64_t lds_per_cu, int64_t per_block, int64_t bytes) {
    if (arc::may_reserve_lds(lds_per_cu, per_block, bytes) == want) return;
    ok = false;
    std::printf("%lld of %lld, %lld a workgroup: want %d\n", (long long)bytes,
                (long long)lds_per_cu, (long long)per_block, want);
  };
  for (const int64_t bytes : {(int64_t)arc::kDenseLdsCap, (int64_t)arc::kOptLdsCap}) {
    expect(true, cu, cu, bytes);
    expect(true, cu, bytes, bytes);
    expect(false, cu, bytes - 1, bytes);
    expect(false, cu / 2, cu, bytes);
  }
  // 160 KB a compute unit, 64 KB a workgroup: room for the x update's, not for
  // the dense iteration's.
  expect(true, cu, 64 * 1024, arc::kOptLdsCap);
  expect(false, cu, 64 * 1024, arc::kDenseLdsCap);
  std::printf("%s\n", ok ? "ok" : "FAIL");
  return !ok;
}

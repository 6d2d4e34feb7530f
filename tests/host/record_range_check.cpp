// Host check of the adjoint gathers' index ranges: whatever an overflowed sort
// left in first[] and rows, the clipped range lies inside the record slots,
// keeps its values if it did so before, and the 16-byte flag reads over it (from
// its start's 16-byte boundary on, while below its end) stay inside the flag
// array, which has the capacity rounded up to 16 bytes.
#include <cstdio>

#include "blend.hpp"

static bool check(uint32_t first, uint32_t count, int64_t cap) {
  uint32_t e0 = first, cnt = count;
  pvg::clip_range(e0, cnt, cap);
  const bool inside = static_cast<int64_t>(first) + count <= cap;
  if (inside ? cnt != count || (cnt && e0 != first) : cnt != 0) return false;
  const int64_t flags = (cap + 15) / 16 * 16, end = static_cast<int64_t>(e0) + cnt;
  int reads = 0;
  for (int64_t b = e0 & ~15u; b < end && reads < 8; b += 16, ++reads)
    if (b + 16 > flags) return false;
  return cnt != 0 || reads == 0;
}

int main() {
  const int64_t caps[] = {0, 1, 15, 16, 17, 100, 4095, 4096, 1000003, 0x7fffffffll, 0xfffffff1ll, 0xffffffffll};
  for (const int64_t cap : caps) {
    for (int64_t base : {int64_t{0}, cap, int64_t{0x80000000ll}, int64_t{0xffffffc0ll}})
      for (int64_t d = -70; d <= 70; ++d)
        for (uint32_t cnt : {0u, 1u, 15u, 16u, 17u, 48u, 49u, 0x80000000u, 0xffffffffu}) {
          const int64_t e0 = base + d;
          if (e0 < 0 || e0 > 0xffffffffll) continue;
          if (!check(static_cast<uint32_t>(e0), cnt, cap)) {
            std::printf("first %lld, count %u, capacity %lld\n", (long long)e0, cnt, (long long)cap);
            return 1;
          }
        }
  }
  std::printf("record range ok\n");
  return 0;
}

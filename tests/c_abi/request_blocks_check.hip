// CPU check of the number of block table entries that a request needs over
// all groups (request_blocks) and of its limit: sums that a 32-bit total
// would wrap to nothing, or to a few entries, lie beyond kMaxRequestBlocks,
// and up to it the finishing kernel's index plus its stride fits 32 bits.
// Host code only: no GPU.
#include <cstdint>
#include <cstdio>

#include "bsr_device.h"

static int bad = 0;
static void expect(const char* what, uint64_t got, uint64_t want) {
  if (got == want) return;
  printf("MISMATCH %s: %llu, expected %llu\n", what, (unsigned long long)got, (unsigned long long)want);
  ++bad;
}

int main() {
  const uint32_t ones[8] = {1, 1, 1, 1, 1, 1, 1, 1};
  const uint32_t mixed[8] = {1, 2, 3, 64, 1, 1, 7, 128};
  expect("no tokens", bsr::request_blocks(0, mixed, 8), 0);
  expect("eight groups, 1000 tokens", bsr::request_blocks(1000, mixed, 8), 1000 + 500 + 334 + 16 + 1000 + 1000 + 143 + 8);
  expect("wraps to 0", bsr::request_blocks(1ull << 29, ones, 8), 1ull << 32);
  expect("wraps to 8", bsr::request_blocks((1ull << 29) + 1, ones, 8), (1ull << 32) + 8);
  expect("wraps to 16384", bsr::request_blocks((1ull << 29) + 2048, ones, 8), (1ull << 32) + 16384);
  expect("largest", bsr::request_blocks((1ull << 32) - 3, ones, 8), 8 * ((1ull << 32) - 3));
  const uint64_t stride = static_cast<uint64_t>(bsr::kFinishMaxGrid) * bsr::kFinishThreads;
  expect("last index plus stride fits 32 bits", bsr::kMaxRequestBlocks - 1 + stride <= 0xFFFFFFFFull, 1);
  expect("the limit itself", bsr::kMaxRequestBlocks, (1ull << 32) - (1ull << 18));
  if (!bad) printf("ok\n");
  return bad != 0;
}

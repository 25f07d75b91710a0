// Rules of the launches that hold on any device, checked on the host (test
// infrastructure, built and run by tests/test_launch_rules.py). Exit status 0
// when every check held.
#include "moray_internal.h"

#include <cstdio>

using namespace moray;

static int failures = 0;
#define CHECK(cond)                                                   \
  do {                                                                \
    if (!(cond)) {                                                    \
      std::printf("FAILED line %d: %s\n", __LINE__, #cond);          \
      ++failures;                                                     \
    }                                                                 \
  } while (0)

// Units of a level: all rays in them, counted in 32 bits.
static void units() {
  const unsigned chunks[] = {1, 63, 64, 100, 256, 4096, 1u << 20}, waves[] = {4, 1024, 3072};
  const unsigned long long sizes[] = {1, 63, 64, 65, 1024, 196608, 262144, 262145, 786432, 786433,
                                      1ull << 30, (1ull << 30) + 1, 1ull << 31, 1ull << 32, 6442450944ull, 3ull << 35};
  for (unsigned w : waves)
    for (unsigned c : chunks)
      for (unsigned long long all : sizes) {
        const unsigned span = unit_rays(all, c, w);
        CHECK(span >= 1);
        const unsigned long long n = (all + span - 1) / span;
        CHECK(n + kSegMax < 1ull << 31);                       // each segment may end in a partial unit
        CHECK((unsigned long long)(unsigned)n * span >= all);  // as the kernel counts them
        if (all <= (unsigned long long)c * w) CHECK(n <= w && span % kWave == 0);
        else if (all >> 30 < c) CHECK(span == c);
      }
}

// Blocks of a launch: a context that asks for fewer blocks than a variant holds gets
// them all (one a compute unit leaves none without), one that asks for more gets
// as many as stay resident.
static void blocks() {
  CHECK(launch_blocks(256, 2, 256) == 256);
  CHECK(launch_blocks(512, 2, 256) == 512);
  CHECK(launch_blocks(768, 2, 256) == 512);
  CHECK(launch_blocks(768, 3, 256) == 768);
  CHECK(launch_blocks(1024, 3, 256) == 768);
  CHECK(launch_blocks(1, 4, 256) == 1);
}

// The level the seeds enter at: never beyond the finest level, the queue or half the lanes
// of the launch, and no coarser than these ask for.
static void entries() {
  moray_ctx c;
  c.num_cu = 256;
  c.blocks_per_cu = 3;
  CHECK(launch_lanes(&c) == 196608);
  c.blocks_per_cu = 1;
  CHECK(launch_lanes(&c) == 65536);
  const long long lanes[] = {1024, 65536, 196608}, trees[] = {1, 2, 7, 64, 5000};
  const size_t caps[] = {256, 4096, 1u << 20};
  for (long long n : lanes)
    for (long long t : trees)
      for (size_t cap : caps)
        for (int l0 = 0; l0 <= 3; ++l0)
          for (int top = l0; top <= 8; ++top) {
            const int l = descend_level(t, l0, top, cap, n);
            auto fits = [&](int k) { return t * (12ll << (2 * k)) <= n / 2 && (size_t)(t * (12ll << (2 * k))) <= cap; };
            CHECK(l >= l0 && l <= top && (l == l0 || fits(l)) && (l == top || !fits(l + 1)));
          }
}

int main() {
  units();
  blocks();
  entries();
  std::printf("%s\n", failures ? "SOME CHECK FAILED" : "ALL OK");
  return failures ? 1 : 0;
}

// The rules by which a step's launches are split (csrc/step_rules.h, host code), over all sizes that they tell apart.  Built
// with sanitizers by tests/test_step_rules.py.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "../../paper_2605_04450_amd/csrc/step_rules.h"

#define CHECK(cond)                                                              \
  do {                                                                           \
    if (!(cond)) {                                                               \
      std::fprintf(stderr, "rules.cpp:%d: check failed: %s\n", __LINE__, #cond); \
      std::exit(1);                                                              \
    }                                                                            \
  } while (0)

using namespace racer;

// Column slices divide a front half's d / 32 tiles per wavefront, never bring more blocks than the chip holds at once, and
// leave no half of the CUs idle where one more halving fits.
static void join_slices_fit_one_round() {
  for (uint32_t d : {64u, 128u, 256u, 512u})
    for (uint32_t groups = 1; groups <= (join_max_rows(d, 0, 1, 0) + 31) / 32; ++groups) {
      const uint32_t s = join_slices(d, groups);
      CHECK(s >= 1 && (d / 32) % s == 0);
      CHECK(s == 1 || groups * s <= join_per_cu(d) * kCus);
      CHECK(s == d / 32 || 2 * groups * s > kCus);
    }
}

// Wavefronts of the fp32 attention: never more than the chip holds at once, unless one request stands out.
static void f32_waves_fit() {
  for (uint32_t dh : {16u, 32u, 48u, 64u})
    for (uint32_t blocks : {1u, 200u, 256u, 257u, 384u, 512u, 513u, 5000u})
      for (uint32_t longest : {1u, 64u, 65u, 192u, 193u, 512u, 513u, 4000u})
        for (uint64_t mean : {uint64_t(1), uint64_t(longest) / 9, uint64_t(longest) / 2, uint64_t(longest)}) {
          const uint32_t w = f32_waves(dh, blocks, longest, mean);
          CHECK(w == 4 || w == 8 || (w == 16 && dh <= 32));
          CHECK(longest > 64 || w == 4);
          CHECK(blocks <= 2 * kCus || w == 4);
          if (blocks > kCus && 2 * mean >= longest) CHECK(w <= (dh <= 32 ? 8 : 4));
        }
  CHECK(f32_waves(32, 256, 256, 136) == 16 && f32_waves(32, 402, 1024, 19) == 16 && f32_waves(64, 201, 1024, 20) == 8 && f32_waves(64, 402, 1024, 20) == 8);
}

// Many short steps behind more than they bring: separate halves where 64 row tiles of 128 fill the chip.
static void joined_limits() {
  CHECK(join_max_rows(512, 8192, 128, 128 * 64) == 8192 && join_max_rows(512, 8192, 128, 128 * 64 + 1) == 8064);
  CHECK(join_max_rows(512, 8192, 64, 1 << 20) == 8064 && join_max_rows(512, 8192, 63, 1 << 20) == 8192);
  CHECK(join_max_rows(256, 20000, 300, 1 << 20) == 24576 && join_max_rows(64, 1, 1, 0) == 65536 && join_max_rows(128, 1, 1, 0) == 65536);
}

// Sums by rows: more than eight partials a tile, and no more than two and a half blocks per CU.
static void sums_limits() {
  CHECK(sums_by_rows(640, 4 * 9, 4) && !sums_by_rows(641, 4 * 9, 4) && !sums_by_rows(640, 4 * 8, 4));
  CHECK(sums_by_rows(1, 9, 1) && !sums_by_rows(1, 2, 1) && !sums_by_rows(0, 0, 0));
}

int main() {
  sums_limits();
  join_slices_fit_one_round();
  joined_limits();
  f32_waves_fit();
  std::puts("step rules: ok");
  return 0;
}

// Rules by which a step's launches are split (host code).
#pragma once

#include <cstdint>

namespace racer {

constexpr uint32_t kCus = 256;

// ---- joined layer halves (layer_join): 32 rows a block ------------------------------------------------------------
// Blocks of layer_join that a CU holds: by their registers (of 512 per SIMD and lane: at d = 256 174 to 236, at 512 318 to 459,
// the back half alone the most) two, or one at d = 512, where 53 to 92 KB of the 160 KB of LDS would allow one or two.
constexpr uint32_t join_per_cu(uint32_t d) { return d <= 256 ? 2 : 1; }

// Slices of the front half's columns, down to one tile per wavefront, while there are CUs without a block, but no more
// blocks than the chip holds at once.  2048 rows of d = 256: 84 us with 256 blocks, 94 with 128, 91 with 1024.  d = 512, four
// layers, two rounds of blocks and one: 576 rows 160 and 115 us, 2112 rows 223 and 170, 6144 rows 297 and 246, 8128 rows 317
// and 258.
constexpr uint32_t join_slices(uint32_t d, uint32_t groups) {
  uint32_t slices = 1;
  while (slices < d / 32 && groups * slices < kCus && 2 * groups * slices <= join_per_cu(d) * kCus) slices *= 2;
  return slices;
}

// Up to how many rows a step's layer halves are joined: a block of 32 rows reads all of W2 and its part of W1, one of
// layer_half_fused does so for 128, and from some number of rounds of blocks on that weighs more than the launches.  Steps of
// four layers, joined and not, prefills of 256 tokens each: d = 64, 65 536 rows 174 and 190 us, 98 304 rows 202 and 213,
// 131 072 rows 252 and 249; d = 128, 65 536 rows 261 and 284, 81 920 rows 360 and 379, 98 304 rows 415 and 409; d = 256,
// 16 384 rows 202 and 232, 24 576 rows 259 and 269, 32 768 rows 329 and 330; d = 512, 8192 rows 286 and 299, 12 288 rows 457 and
// 434.
// With 64 tiles of 128 rows the separate halves of d = 512 fill the chip evenly, and are ahead where many short steps lie
// behind more than they bring, whose attention leaves neither weights nor pages in the caches: 128 x 64 behind 512 397 and
// 418 us, behind 3072 881 and 901 (but behind 64 281 and 269; and with 63 tiles, cut into uneven rounds, 124 x 64 behind
// 3072 1014 and 930).
constexpr uint32_t join_max_rows(uint32_t d, uint64_t rows, uint64_t requests, uint64_t cached) {
  if (d == 512) return cached > rows && 128 * requests >= rows ? 63 * 128 : 64 * 128;
  return d <= 128 ? 65536 : 24576;
}

// ---- sums of the partial outputs of cut query tiles ---------------------------------------------------------------
// Both kernels add in the order of the keys.  attention_reduce_rows waits for memory once where attention_reduce waits for each
// four partials, but asks for four times as many pieces of memory: it is ahead where partials are many and its blocks (of four
// rows of a tile and head) few.  Steps of eight layers, attention_reduce and attention_reduce_rows, us:
//   partials (d = 64, a request of 64): 2 141 and 143, 8 139 and 139, 12 135 and 132, 40 153 and 136, 94 198 and 158
//   blocks, 24 partials (d = 256, 64 new tokens each): 64 176 and 166, 256 204 and 194, 512 253 and 246, 640 273 and 268
//   blocks, 16 partials: 640 228 and 226, 960 302 and 303;  12: 640 208 and 207;  8: 512 187 and 187, 1024 222 and 224
constexpr bool sums_by_rows(uint64_t blocks, uint64_t partials, uint64_t tiles) {
  return 2 * blocks <= 5 * kCus && partials > 8 * tiles;
}

// ---- fp32 attention: wavefronts per block, which take groups of 16 keys in turn -----------------------------------
// blocks: query tiles times heads.  longest: tokens of the longest request.  mean_keys: keys that a query tile sees, on average.
// Up to a block per CU, about a wavefront per group of the longest request, 16 at most (eight where heads are wider than 32: 16
// would spill).  4 requests x 256 tokens, 2 heads of 32, whole step: 26.2 us with four, 23.9 with eight, 23.1 with 16.
// Up to two blocks per CU, the neighbours' wavefronts already fill it: eight, or four where heads are wider (16 requests x
// 256 tokens, 2 heads of 32: 39.8 us with four, 37.9 with eight, 40.8 with 16; 448 blocks of one request's last 64 tokens of 256 each, 2
// heads of 64: 68.1 and 71.3), unless the longest request is a chain that the others do not cover (one of 1024 among 200 of
// 16: heads of 32 59.3, 48.9 and 45.6, of 64 94.7 and 80.7; 24 ragged ones of 250, heads of 64, 73.6 and 67.8).
constexpr uint32_t f32_waves(uint32_t dh, uint64_t blocks, uint32_t longest, uint64_t mean_keys) {
  if (blocks > 2 * kCus || longest <= 64) return 4;
  if (dh > 32) return blocks <= kCus || 5ull * longest > 12 * mean_keys ? 8 : 4;
  if (longest <= 192) return 8;
  return blocks <= kCus || (longest > 512 && longest > 8 * mean_keys) ? 16 : 8;
}

}  // namespace racer

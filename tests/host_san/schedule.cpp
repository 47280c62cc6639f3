// The attention schedule (csrc/attn_schedule.h, host code) over random and edge steps, built with sanitizers by
// tests/test_attn_schedule.py: every key tile of every query tile and head is covered once, by pieces whose pages fit a
// workgroup's table; partial outputs have slots of their own in the order of the keys; the stated bounds hold; a step that is
// cut has no more pieces than places, or no more work per place than a piece with its cost; its dies take the largest pieces
// first; the dies' loads differ by no more than a unit of work; and blocks take turns where places that progress alike, the
// largest pieces first, end within a quarter of the mean.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <queue>
#include <random>

#include "../../paper_2605_04450_amd/csrc/attn_schedule.h"
#include "../../paper_2605_04450_amd/csrc/step_rules.h"

#define CHECK(cond)                                                                 \
  do {                                                                              \
    if (!(cond)) {                                                                  \
      std::fprintf(stderr, "schedule.cpp:%d: check failed: %s\n", __LINE__, #cond); \
      std::exit(1);                                                                 \
    }                                                                               \
  } while (0)

using namespace racer;

static void check(const std::vector<ReqDev>& reqs, uint32_t H, uint32_t pt, AttnSchedule& s) {
  uint64_t N = 0, longest = 1;
  for (const ReqDev& r : reqs) {
    N += r.new_len;
    longest = std::max<uint64_t>(longest, r.prefix_len + r.new_len);
  }
  s.build(reqs.data(), static_cast<uint32_t>(reqs.size()), H, pt);
  const AttnBounds b = attn_bounds(reqs.size(), N, longest, H, pt);
  CHECK(s.items.size() <= b.items && s.work.size() <= b.work && s.n_slots <= b.work && s.groups.size() <= b.items);
  // the lists of the dies, and a workgroup for every entry
  CHECK(s.begin[0] == 0 && s.begin[kXcds] == s.work.size());
  for (uint32_t x = 0; x < kXcds; ++x) CHECK(s.begin[x] <= s.begin[x + 1] && (s.begin[x + 1] - s.begin[x]) * kXcds <= s.blocks);
  struct Piece { uint32_t k, kt_begin, kt_end; };
  std::vector<std::vector<Piece>> of(s.items.size() * H);
  for (const AttnWork& w : s.work) {
    CHECK((w.item_head >> 4) < s.items.size() && (w.item_head & 15) < H);
    const AttnItem& t = s.items[w.item_head >> 4];
    const uint32_t kt_begin = w.k * s.piece, kt_end = w.k + 1 == t.pieces ? attn_tiles(t) : kt_begin + s.piece;
    CHECK(w.k < t.pieces && kt_begin < kt_end && (kt_end * 64ull - 1) / pt - kt_begin * 64ull / pt < kAttnMaxItemPages);
    // the loop asks for the page of tile kt_end + 1, and the last word of the list is not a page's
    if (pt >= 64 && (pt & (pt - 1)) == 0) CHECK((kt_end + 1) * 64ull / pt - kt_begin * 64ull / pt < kAttnMaxItemPages);
    CHECK((kt_end * 64ull - 1) / pt - kt_begin * 64ull / pt < kAttnMaxItemPages - 1);
    of[(w.item_head >> 4) * H + (w.item_head & 15)].push_back({w.k, kt_begin, kt_end});
  }
  // the loads of the dies: each unit went to the least loaded one, and is closed when it weighs more than a 32nd of a head's work
  auto size_of = [&](const AttnWork& w) {
    const AttnItem& t = s.items[w.item_head >> 4];
    return static_cast<uint64_t>(w.k + 1 == t.pieces ? attn_tiles(t) - w.k * s.piece : s.piece);
  };
  uint64_t least = ~0ull, most = 0, largest = 0, total = 0, all = 0;
  for (uint32_t x = 0; x < kXcds; ++x) {
    uint64_t load = 0;
    for (uint32_t i = s.begin[x]; i < s.begin[x + 1]; ++i) {
      const uint64_t size = size_of(s.work[i]);
      CHECK(s.groups.empty() || i == s.begin[x] || size_of(s.work[i - 1]) >= size);
      load += size + kAttnItemCost;
      largest = std::max(largest, size);
    }
    least = std::min(least, load);
    most = std::max(most, load);
  }
  for (const AttnItem& t : s.items) {
    total += attn_tiles(t) + kAttnItemCost;
    all += attn_tiles(t) + kAttnItemCost * t.pieces;
  }
  CHECK(most - least <= total / (4 * kXcds) + largest + kAttnItemCost);
  if (!s.groups.empty() && s.piece < attn_page_cap(pt)) {
    CHECK(all * H <= (s.piece + kAttnItemCost) * static_cast<uint64_t>(kAttnBlocks));
    if (2 * s.items.size() * H <= kAttnBlocks) CHECK(s.work.size() <= kAttnBlocks);
  }
  if (s.work.size() <= kAttnBlocks) {
    CHECK(s.turns);
  } else {
    std::vector<uint64_t> sizes;
    for (const AttnWork& w : s.work) sizes.push_back(size_of(w) + kAttnItemCost);
    std::sort(sizes.begin(), sizes.end(), std::greater<>());
    std::priority_queue<uint64_t, std::vector<uint64_t>, std::greater<>> places(std::greater<>(), std::vector<uint64_t>(kAttnBlocks, 0));
    uint64_t end = 0;
    for (uint64_t size : sizes) {
      const uint64_t at = places.top() + size;
      places.pop();
      places.push(at);
      end = std::max(end, at);
    }
    CHECK(s.turns == (4 * end <= 5 * ((all * H + kAttnBlocks - 1) / kAttnBlocks)));
  }
  uint64_t slots = 0;
  size_t n_cut = 0;
  for (uint32_t i : s.groups) {
    CHECK(i < s.items.size() && s.items[i].pieces >= 2 && s.items[i].slot0 == slots);
    slots += s.items[i].pieces * H;
  }
  for (const AttnItem& t : s.items) n_cut += t.pieces > 1;
  CHECK(slots == s.n_slots && n_cut == s.groups.size());
  size_t item = 0;
  for (uint32_t r = 0; r < reqs.size(); ++r)
    for (uint32_t q0 = 0; q0 < reqs[r].new_len; q0 += 128, ++item) {
      const AttnItem& t = s.items[item];
      CHECK(t.req == r && t.qt == q0 / 128 && t.prefix_len == reqs[r].prefix_len && t.new_len == reqs[r].new_len && t.x_off == reqs[r].x_off);
      const uint32_t last = t.prefix_len + std::min(q0 + 127, t.new_len - 1);
      for (uint32_t h = 0; h < H; ++h) {
        auto& p = of[item * H + h];
        std::sort(p.begin(), p.end(), [](const Piece& a, const Piece& c) { return a.k < c.k; });
        CHECK(p.size() == t.pieces);
        uint32_t at = 0;
        for (size_t k = 0; k < p.size(); ++k) {
          CHECK(p[k].k == k && p[k].kt_begin == at);
          at = p[k].kt_end;
        }
        CHECK(at == last / 64 + 1);
      }
    }
  CHECK(item == s.items.size());
}

static std::vector<ReqDev> requests(const std::vector<std::pair<uint32_t, uint32_t>>& lens) {
  std::vector<ReqDev> r;
  uint32_t x = 0;
  for (const auto& l : lens) {
    r.push_back({l.first, l.second, 0, 0, x});
    x += l.second;
  }
  return r;
}

// Entries of the positional window against the distance in 64 bits, also where distance or table pass 2^30 and 2^31 entries: at
// the item's first key, around its middle and at its last tile, for items of a few tiles and of the most there are.
static void positions() {
  for (uint64_t top : {127ull, 128ull, 190ull, 400ull, 5000ull, (1ull << 29) + 255, (1ull << 29) + 256, (1ull << 29) + 257, (1ull << 30) - 1, 1ull << 30,
                       (1ull << 30) + 300, (1ull << 31) - 2, (1ull << 31) + 126})
    for (uint64_t n_pos : {1ull, 2ull, 100ull, 256ull, 4999ull, (1ull << 29) + 1, (1ull << 30) - 1, 1ull << 30, (1ull << 30) + 1, 1ull << 31,
                           (1ull << 31) + 127, (1ull << 32) - 1}) {
      const PosEntries e = pos_entries(static_cast<uint32_t>(top), static_cast<uint32_t>(n_pos));
      CHECK((e.last + 1ull) * 4 <= 1ull << 32);
      for (uint64_t tiles : {1ull, 2ull, 606ull, static_cast<unsigned long long>(kAttnMaxItemTiles)}) {
        const uint64_t end = std::min(64 * tiles + 191, top + 255);
        for (uint64_t from : {uint64_t(0), end / 2, end > 600 ? end - 600 : 0})
          for (uint64_t x = from; x < std::min(from + 600, end); ++x) {
            const int64_t want = std::min<int64_t>(std::max<int64_t>(static_cast<int64_t>(top) - static_cast<int64_t>(x), 0), static_cast<int64_t>(n_pos) - 1);
            CHECK(e.base + std::min(std::max(e.first - static_cast<uint32_t>(x), 256u), e.last) == want);
          }
      }
    }
  CHECK(attn_page_cap(0xFFFFFFF8u) == kAttnMaxItemTiles && attn_page_cap(64) == kAttnMaxItemPages - kAttnSparePages);
}

int main() {
  positions();
  AttnSchedule s;  // one object over all steps, as in a pool
  for (uint32_t H : {1u, 4u, 16u})
    for (uint32_t pt : {8u, 24u, 64u, 800u}) {
      check(requests({{0, 1}}), H, pt, s);
      check(requests({{0, 0}, {5, 0}, {63, 1}, {64, 128}, {0, 129}}), H, pt, s);
      check(requests({{2973, 64}}), H, pt, s);
      check(requests({{1u << 20, 3}, {0, 5000}}), H, pt, s);
      check(requests(std::vector<std::pair<uint32_t, uint32_t>>(700, {0, 1})), H, pt, s);
      check(requests(std::vector<std::pair<uint32_t, uint32_t>>(32, {16384, 512})), H, pt, s);
    }
  // items as long as a page list allows: of 606 tiles of 64 tokens, or from inside a page on
  for (uint32_t pt : {64u, 128u, 256u, 8u, 24u}) {
    check(requests(std::vector<std::pair<uint32_t, uint32_t>>(40, {1u << 20, 500})), 8, pt, s);
    CHECK(s.piece == attn_page_cap(pt) || pt > 64);
  }
  // equal query tiles that fill more than half of the places: one each, not one of a share and a remainder
  for (uint32_t n : {130u, 144u, 160u, 192u})
    for (uint32_t prefix : {1024u, 3072u}) {
      check(requests(std::vector<std::pair<uint32_t, uint32_t>>(n, {prefix, 64})), 4, 64, s);
      CHECK(s.work.size() == 4 * n && s.groups.empty());
    }
  // but one that is many times as long as the others is cut
  {
    std::vector<std::pair<uint32_t, uint32_t>> l(160, {1024, 64});
    l[17].first = 16384;
    check(requests(l), 4, 64, s);
    CHECK(!s.groups.empty());
  }
  // steps of tests/test_gpu_attention_tiles.py: they are cut into as many pieces as it says, and added up by attention_reduce_rows
  // or not; first those whose keys lie in pieces of two key tiles
  struct Sums { uint32_t H, n, pieces, len; bool by_rows; };
  for (const Sums& c : {Sums{1, 1, 5, 1, false}, {1, 1, 6, 64, false}, {2, 2, 7, 33, false}, {4, 1, 8, 64, false}, {4, 16, 12, 64, false},
                        {1, 1, 9, 64, true}, {1, 2, 16, 3, true}, {4, 1, 17, 64, true}, {4, 1, 24, 64, true}, {8, 1, 32, 128, true},
                        {1, 1, 33, 64, true}, {2, 1, 48, 2, true}, {1, 1, 49, 100, true}, {4, 1, 94, 1, true}}) {
    check(requests(std::vector<std::pair<uint32_t, uint32_t>>(c.n, {128 * c.pieces - c.len, c.len})), c.H, 64, s);
    CHECK(s.piece == 2 && s.groups.size() == c.n && s.n_slots == c.n * c.H * c.pieces);
    CHECK(sums_by_rows((c.len + 3) / 4 * c.n * c.H, s.n_slots, c.n * c.H) == c.by_rows);
  }
  struct Cut { uint32_t H, n, prefix, len, pieces; bool by_rows; };
  for (const Cut& c : {Cut{1, 40, 1100, 64, 9, true}, {1, 41, 1100, 64, 9, false}, {2, 20, 1100, 61, 9, true}, {2, 21, 1100, 61, 9, false},
                       {1, 41, 1000, 64, 8, false}, {1, 40, 1000, 64, 8, false}, {1, 64, 520, 64, 5, false}, {2, 33, 600, 1, 5, false},
                       {1, 1, 4500, 64, 36, true}, {1, 1, 4000, 64, 32, true}, {1, 1, 1000, 128, 9, true}, {1, 64, 200, 64, 2, false},
                       {4, 1, 300, 3, 2, false}, {4, 1, 200, 2, 2, false}}) {
    check(requests(std::vector<std::pair<uint32_t, uint32_t>>(c.n, {c.prefix, c.len})), c.H, 64, s);
    CHECK(s.groups.size() == c.n && s.n_slots == c.n * c.H * c.pieces);
    CHECK(sums_by_rows((c.len + 3) / 4 * c.n * c.H, s.n_slots, c.n * c.H) == c.by_rows);
  }
  {  // of tests/test_gpu_step_capture.py: a prefill of 2300 tokens, one head: 17 of its 18 query tiles are cut, into 2 to 18 pieces
    check(requests({{0, 2300}}), 1, 64, s);
    CHECK(s.groups.size() == 17 && s.n_slots == 170 && sums_by_rows(17 * 32 - 1, 170, 17));
  }
  std::mt19937 g(1);
  auto log_size = [&](double e) { return static_cast<uint32_t>(std::exp((g() % 10000) / 10000.0 * e)); };
  const uint32_t pts[] = {8, 16, 24, 40, 64, 256, 800};
  for (int it = 0; it < 1500; ++it) {
    std::vector<std::pair<uint32_t, uint32_t>> l(1 + g() % (it % 50 == 0 ? 300 : 12));
    for (auto& p : l) p = {g() % 4 ? log_size(10.0) - 1 : 0, g() % 8 ? log_size(8.0) : g() % 2};
    check(requests(l), 1 + g() % 16, pts[g() % 7], s);
  }
  std::puts("attention schedule: ok");
  return 0;
}

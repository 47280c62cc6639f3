// Which attention workgroup of a step does what (host code).
//
// The score matrix of a request is a staircase: a query tile (128 new tokens) sees as many 64-key tiles as lie before its
// last query.  A workgroup takes a range of one query tile's key tiles for one head, and as many are resident as the chip
// has places for (kAttnPlaces per die); the others start as places become free.
//   - Workgroup ids go round-robin over the chip's dies, each with an L2 of its own, so every die has a list.  Units of
//     work that read the same keys of the same head go to one die, where they lie one behind the other, heaviest unit onto
//     the least loaded die.
//   - The units with the largest items come first, so that what starts last is small (64 users back with 64 tokens behind
//     2048 and 64 new histories, where the long cached ones used to start last: 424 -> 355 us a launch).
//   - If a query tile has clearly more than a place's share of the work, those with more than that are cut over their keys
//     into pieces of it (or larger ones, one for each place), and the pieces sorted by size.  They leave fp32 partial outputs that attention_reduce adds up in the
//     order of the keys.
// Tried instead and slower: one workgroup per place with a list dealt beforehand (places do not progress alike: 131k-token
// prefill 327 -> 366 us, 349 with wavefront priorities by progress; 128 x 64 behind 3072 99 -> 104), or with items
// taken from a queue per die (390 and 120 us: what a workgroup does between two items takes longer than a new one's start).
// Pieces of 4/5, 3/5 or 2/5 of the share: 107, 100, 105 us instead of 97 for 128 x 64 behind 3072.
#pragma once

#include <algorithm>
#include <cstdint>
#include <iterator>
#include <vector>

namespace racer {

constexpr uint32_t kXcds = 8;
constexpr uint32_t kAttnPlaces = 128;  // workgroups resident per die: 32 CUs, four each
constexpr uint32_t kAttnBlocks = kXcds * kAttnPlaces;
constexpr uint32_t kAttnItemCost = 2;  // what an item costs besides its key tiles, in key tiles
// Small steps: a workgroup needs about 3 us before its first tile and 1.1 us per tile, so two tiles an item, spread over
// idle CUs, beat eight in one (one request of 64 new tokens 18 -> 11 us, 13 ragged prefills 35 -> 14 us).
constexpr uint32_t kAttnMinTiles = 2;
constexpr uint32_t kAttnMaxItemPages = 608;  // words of a workgroup's page list
// Words of it beyond the pages that an item's tiles would fill if they began with a page: the item may begin inside one, and the
// loop asks for the page of the second tile behind the item's last one (a word that may hold anything, and is not used).
constexpr uint32_t kAttnSparePages = 2;

struct ReqDev {  // device copy of one request
  uint32_t prefix_len, new_len;
  uint32_t page_table_off, ts_off, x_off;
};

// A query tile: 128 new tokens (or what is left of them) of one request
struct AttnItem {
  uint32_t prefix_len, new_len, page_table_off, ts_off, x_off;  // of the request
  uint32_t req, qt;
  uint32_t slot0, pieces;  // cut into more than one: piece k of head h leaves its partial output in slot slot0 + h * pieces + k
};

// What one workgroup does: piece k of a query tile (key tiles k * piece up to the next piece, the last one up to the last
// tile) for one head.  A list entry is as short as it can be: steps whose lists fit a kernel argument are the ones that
// need no staging, and that a graph can capture.
struct AttnWork {
  uint32_t item_head, k;  // item << 4 | head
};
constexpr uint32_t kMaxHeads = 16;

// key tiles that a query tile sees
constexpr uint32_t attn_tiles(const AttnItem& t) {
  const uint32_t last = t.qt * 128 + 127 < t.new_len ? t.qt * 128 + 127 : t.new_len - 1;
  return (t.prefix_len + last) / 64 + 1;
}

// Where the positional biases of an item are.  Entry x of its window is the bias of distance top - x, held within the table's
// n_pos entries (negative distances belong to keys after the query, which the causal select removes).  It sits at
// base + min(max(first - x, 256), last): a base in 64 bits and, since an item has no more than kAttnMaxItemTiles key tiles, an
// offset of less than 2^30 entries, 2^32 bytes.  top is below 2^31 + 127, n_pos any number but 0, x at most 191 past the
// item's last key.
constexpr uint32_t kAttnMaxItemTiles = 1u << 23;
struct PosEntries {
  int64_t base;
  uint32_t first, last;
};
constexpr PosEntries pos_entries(uint32_t top, uint32_t n_pos) {
  constexpr uint32_t span = kAttnMaxItemTiles * 64 + 256;
  const uint32_t nearest = top > span ? top - span : 0;  // no entry of the item is of a shorter distance, or of more than 0
  const uint32_t from = nearest < n_pos - 1 ? nearest : n_pos - 1;
  const uint32_t entries = n_pos - 1 - from < span ? n_pos - 1 - from : span;
  return {static_cast<int64_t>(from) - 256, top - from + 256, entries + 256};  // 256 and up: so that nothing is negative
}

// key tiles whose pages an item's slice of the page table can name
inline uint32_t attn_page_cap(uint32_t page_tokens) {
  return static_cast<uint32_t>(std::max<uint64_t>(1, std::min<uint64_t>(kAttnMaxItemTiles, (kAttnMaxItemPages - kAttnSparePages) * static_cast<uint64_t>(page_tokens) / 64)));
}

// Upper bounds for up to B requests, N new tokens and sequences of up to max_seq tokens: query tiles, and entries of all lists
struct AttnBounds { uint64_t items, work; };
inline AttnBounds attn_bounds(uint64_t B, uint64_t N, uint64_t max_seq, uint32_t H, uint32_t page_tokens) {
  const uint64_t q = N / 128 + B, visits = q * H * (max_seq / 64 + 1);
  // one per query tile and head, and one more per cut: at a place's share, or at the page cap
  const uint64_t cuts = std::min<uint64_t>(2 * kAttnBlocks, visits / kAttnMinTiles) + 2 * (visits / attn_page_cap(page_tokens));
  return {q, q * H + cuts};
}

class AttnSchedule {
 public:
  std::vector<AttnItem> items;
  std::vector<AttnWork> work;      // die x's list: entries [begin[x], begin[x + 1])
  uint32_t begin[kXcds + 1] = {};
  uint32_t blocks = 0;             // workgroups to launch
  std::vector<uint32_t> groups;    // the query tiles whose partial outputs are to be added up
  uint32_t piece = 0;              // key tiles of a piece
  uint32_t n_slots = 0;
  bool turns = true;               // the blocks of a CU take turns at going first (ends_evenly)

  // Memory for steps within these bounds (touched, so that the first of them pays for none of it).
  void reserve(const AttnBounds& b, uint32_t H) {
    auto have = [](auto& v, uint64_t n) {
      if (v.capacity() >= n) return;
      v.resize(n);
      v.clear();
    };
    have(items, b.items);
    have(work, b.work);
    have(sorted_, b.work);
    have(groups, b.items);
    have(atoms_, b.work / H + b.items);
    have(units_, b.work / H + b.items);
    have(die_, b.work + b.items * H);
  }

  void build(const ReqDev* reqs, uint32_t B, uint32_t H, uint32_t page_tokens) {
    items.clear(); work.clear(); groups.clear(); atoms_.clear(); units_.clear();
    n_slots = blocks = 0;
    uint64_t total = 0;
    uint32_t largest = 0;
    for (uint32_t r = 0; r < B; ++r)
      for (uint32_t q0 = 0; q0 < reqs[r].new_len; q0 += 128) {
        const ReqDev& q = reqs[r];
        items.push_back({q.prefix_len, q.new_len, q.page_table_off, q.ts_off, q.x_off, r, q0 / 128, 0, 1});
        const uint32_t n = attn_tiles(items.back());
        total += n + kAttnItemCost;
        largest = std::max(largest, n);
      }
    const uint32_t page_cap = attn_page_cap(page_tokens);
    uint64_t share = std::max<uint64_t>(kAttnMinTiles + kAttnItemCost, (total * H + kAttnBlocks - 1) / kAttnBlocks);
    // Cut at all?  Then into the smallest pieces of which all places together can take one each, or into pieces of a place's
    // share with what the pieces cost included.  The first where query tiles fill at most half of the places, and up to three
    // quarters of them where its pieces are about equal: the second would cut them into a share and a remainder.  (One each and
    // shares, 64 new tokens behind 3072, d = 256, four layers: 96 requests 382 and 419 us, 144 523 and 616, 160 557 and 627;
    // 192 x 128 behind 2048, two layers, 335 and 393.  With places for no more than a fifth of them besides it depends on
    // the shape: 200 x 64 behind 3072 702 and 757, but d = 128, 100 x 512 behind 3000, 427 and 411; and unequal ones lose: 70
    // prefills of 300 151 and 136, 16 of 1500 211 and 200, 250 x 64 behind 3072 with a spread of 0.3 477 and 457.)
    const bool cut = largest + kAttnItemCost > share + share / 4 || largest > page_cap;
    if (cut) {
      const uint64_t tiles = static_cast<uint64_t>(items.size()) * H, even = share_of(share, ~0ull, H, false);
      uint64_t one_each = 0;
      if (2 * tiles <= kAttnBlocks) one_each = share_of(share, ~0ull, H, true);
      else if (4 * tiles <= 3 * kAttnBlocks) one_each = share_of(share, 2 * even, H, true);
      share = one_each ? one_each : even;
    }
    piece = static_cast<uint32_t>(std::min<uint64_t>(share - kAttnItemCost, page_cap));
    if (cut)
      for (uint32_t i = 0; i < items.size(); ++i) {
        AttnItem& t = items[i];
        t.pieces = pieces_of(attn_tiles(t), piece, page_cap);
        if (t.pieces < 2) continue;
        t.slot0 = n_slots;
        n_slots += t.pieces * H;
        groups.push_back(i);
      }
    // units: query tiles of one request (cut ones: their pieces with the same keys), and, of one that is a large part of
    // the whole step, runs of them
    for (uint32_t i0 = 0; i0 < items.size();) {
      uint32_t i1 = i0, most = 0;
      while (i1 < items.size() && items[i1].req == items[i0].req) most = std::max(most, items[i1++].pieces);
      for (uint32_t k = 0; k < most; ++k) {
        Unit u{0, 0, static_cast<uint32_t>(atoms_.size()), 0};
        for (uint32_t i = i1; i-- > i0;) {  // the largest first
          if (k >= items[i].pieces) continue;
          atoms_.push_back({i, k});
          const uint32_t size = size_of(items[i], k);
          u.weight += size + kAttnItemCost;
          u.largest = std::max(u.largest, size);
          ++u.n;
          if (u.weight > total / (4 * kXcds)) {
            units_.push_back(u);
            u = Unit{0, 0, static_cast<uint32_t>(atoms_.size()), 0};
          }
        }
        if (u.n) units_.push_back(u);
      }
      i0 = i1;
    }
    std::sort(units_.begin(), units_.end(), [](const Unit& a, const Unit& b) {
      return a.largest != b.largest ? a.largest > b.largest : a.weight != b.weight ? a.weight > b.weight : a.atom0 < b.atom0;
    });
    uint64_t load[kXcds] = {};
    uint32_t at[kXcds + 1] = {};  // entries of the dies before x, then where the next one of die x goes
    die_.resize(units_.size() * H);
    for (size_t u = 0; u < units_.size(); ++u)
      for (uint32_t h = 0; h < H; ++h) {
        uint32_t best = 0;
        for (uint32_t x = 1; x < kXcds; ++x)
          if (load[x] < load[best]) best = x;
        load[best] += units_[u].weight;
        at[best + 1] += units_[u].n;
        die_[u * H + h] = static_cast<uint8_t>(best);
      }
    for (uint32_t x = 0; x < kXcds; ++x) {
      blocks = std::max(blocks, kXcds * at[x + 1]);
      at[x + 1] += at[x];
    }
    std::copy(at, at + kXcds + 1, begin);
    work.resize(begin[kXcds]);
    for (size_t u = 0; u < units_.size(); ++u)
      for (uint32_t h = 0; h < H; ++h) {
        uint32_t& to = at[die_[u * H + h]];
        for (uint32_t a = 0; a < units_[u].n; ++a) {
          const Atom& t = atoms_[units_[u].atom0 + a];
          work[to++] = {t.item << 4 | h, t.k};
        }
      }
    turns = work.size() <= kAttnBlocks || ends_evenly(H, largest);
    if (!cut) return;
    sorted_.resize(work.size());
    for (uint32_t x = 0; x < kXcds; ++x) {  // by size, else in the order they have
      count_.assign(piece + kAttnMinTiles + 1, 0);
      auto place = [&](const AttnWork& w) -> uint32_t& { return count_[piece + kAttnMinTiles - size_of(items[w.item_head >> 4], w.k)]; };
      for (uint32_t i = begin[x]; i < begin[x + 1]; ++i) ++place(work[i]);
      uint32_t to = begin[x];
      for (uint32_t& c : count_) {
        const uint32_t n = c;
        c = to;
        to += n;
      }
      for (uint32_t i = begin[x]; i < begin[x + 1]; ++i) sorted_[place(work[i])++] = work[i];
    }
    work.swap(sorted_);
  }

 private:
  struct Atom { uint32_t item, k; };
  struct Unit { uint64_t weight; uint32_t largest, atom0, n; };
  std::vector<Atom> atoms_;
  std::vector<Unit> units_;
  std::vector<uint8_t> die_;  // [unit][head]
  std::vector<uint32_t> count_, ends_;
  std::vector<AttnWork> sorted_;

  // The least share from `from` on with which there are no more pieces than places (one_each), or no more work, the
  // pieces' cost included, than a share per place.  With a limit `most`: 0 if there is none, or its pieces are not about equal.
  uint64_t share_of(uint64_t from, uint64_t most, uint32_t H, bool one_each) const {
    for (uint64_t share = from; share <= most; share += one_each && most == ~0ull ? 1 : 1 + share / 32) {
      uint64_t count = 0, all = 0;
      for (const AttnItem& t : items) {
        const uint64_t n = (attn_tiles(t) + share - kAttnItemCost - 1) / (share - kAttnItemCost);
        count += n;
        all += attn_tiles(t) + kAttnItemCost * n;
      }
      if (one_each ? count * H <= kAttnBlocks : all * H <= share * kAttnBlocks)
        return most == ~0ull || 20 * all >= 17 * share * count ? share : 0;
    }
    return 0;
  }

  // Places that progress alike all end a round of workgroups together, which is best where the last round is full, and where it
  // is not leaves few workgroups to run alone: there it is better that they progress as they happen to.  Do places that
  // progress alike end within a quarter of the mean?  (With turns and without, d = 256, two layers: 128 x 200 new tokens behind
  // 3072, two even rounds, 463 and 483 us; 700 x 64 behind 1024, 1.10 of the mean, 539 and 544; 160 x 128 behind 2048, 1.18, 343 and
  // 347; 600 x 64 behind 1024, 1.28, 490 and 488; 75 x 256 behind 3000, 1.33, 408 and 388; 96 x 512 behind 2048, 1.33, 618 and
  // 576; 70 x 512 behind 2000, 1.83, 566 and 502.)
  bool ends_evenly(uint32_t H, uint32_t largest) {
    count_.assign(largest + 1, 0);
    uint64_t all = 0;
    for (const AttnItem& t : items) {
      const uint32_t last = size_of(t, t.pieces - 1);
      if (t.pieces > 1) count_[piece] += (t.pieces - 1) * H;
      count_[last] += H;
      all += attn_tiles(t) + static_cast<uint64_t>(kAttnItemCost) * t.pieces;
    }
    // places by when they become free, the largest pieces first
    const uint64_t mean = (all * H + kAttnBlocks - 1) / kAttnBlocks;
    ends_.assign(mean + largest + kAttnItemCost + 1, 0);
    ends_[0] = kAttnBlocks;
    uint64_t free = 0, end = 0;
    for (uint32_t size = largest; size > 0; --size)
      for (uint32_t left = count_[size]; left > 0;) {
        while (ends_[free] == 0) ++free;
        const uint32_t n = std::min(left, ends_[free]);
        ends_[free] -= n;
        ends_[free + size + kAttnItemCost] += n;
        end = std::max(end, free + size + kAttnItemCost);
        left -= n;
      }
    return 4 * end <= 5 * mean;
  }

  uint32_t size_of(const AttnItem& t, uint32_t k) const { return k + 1 == t.pieces ? attn_tiles(t) - k * piece : piece; }
  // How many pieces a query tile of n key tiles is cut into, at multiples of `piece`; a last piece of less than
  // kAttnMinTiles joins the one before it.
  static uint32_t pieces_of(uint32_t n, uint32_t piece, uint32_t page_cap) {
    uint32_t k = (n + piece - 1) / piece;
    if (k > 1 && n - (k - 1) * piece < kAttnMinTiles && n - (k - 2) * piece <= page_cap) --k;
    return k;
  }
};

}  // namespace racer

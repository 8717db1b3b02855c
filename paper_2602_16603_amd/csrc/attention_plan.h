// How an attention launch of few query tiles over many keys is cut over the keys.  Plain C++17 with no GPU dependency:
// the plan can be built and checked on the CPU.
#pragma once
#include <algorithm>
#include <array>
#include <cstdint>
#include <vector>

namespace fp {

// Bytes of partial outputs a task's attention may leave at most.  The plan alone would reach 0.75 GB (32 heads of 128,
// 6200 tokens behind 110000 cached ones) for a gain of a few per cent; a chunk of up to 2048 tokens behind up to 24576
// asks for 102 MB at 32 heads, 224 MB at 40.
constexpr int64_t kAttnPartBytes = 256ll << 20;

// A workgroup walks its keys one tile after the other and a CU holds one workgroup, so a launch of few
// query tiles over many keys -- a chunk of a long prompt -- keeps most CUs idle for the whole walk.  Cut
// over the keys it ends when its longest part does, plus the merge.  Times in key tiles (about 1.4 us): a query
// tile pays kWholeCost on top of its keys (prologue, first loads), a part kPartCost (and storing its output: 133 KB
// per head), the merge kMergeCost and the reading of all parts (50 (part, head) pairs in the time of a tile).
// All heads of a query tile take equally long, so the 256 CUs count as 256 / heads places that each
// take one (query tile, every head) at a time, longest first.  More than four such rounds balance
// themselves.  No part is shorter than kMinPart tiles (its first key must be visible to all 256 queries
// of the tile, which five tiles ensure).  512 tokens behind 15872 cached ones, 32 heads of 128: 365 us
// whole (64 workgroups of 256 tiles), 125 + 8 us in four parts per query tile; 128 behind 24576 461 -> 81 us, 1100
// behind 20000 434 -> 323, 2048 behind 2048 stays whole (101; in parts 106).  With 5 to 64 heads of 64 and 128, prompts
// of 1024 to 4100 tokens and chunks behind 600 to 40000: none slower than whole, 1.39 times as fast on average.
//
// Number of key tiles a part of a query tile should hold so that the launch ends soonest: `tiles` = key tiles of every
// query tile, most first; at most `max_parts` parts in all.  0: leave the query tiles whole.
inline int attention_part_tiles(const std::vector<int32_t>& tiles, int n_q_heads, int64_t max_parts) {
  constexpr int kPlaces = 256, kMaxPlaces = 64, kRounds = 4, kMinPart = 8, kWholeCost = 3, kPartCost = 5, kMergeCost = 4, kMaxParts = 16;
  const int places = std::min(kMaxPlaces, std::max(1, kPlaces / n_q_heads));
  if (tiles.empty() || (int)tiles.size() > kRounds * places || tiles[0] < 2 * kMinPart) return 0;
  auto parts_of = [](int n, int limit) { return limit ? (n + limit - 1) / limit : 1; };
  // Parts of at most `limit` tiles: how many of them leave their output, and when the last one is done -- not gone
  // through for a limit whose work alone, spread evenly over the places, takes until `give_up`.
  int64_t stored = 0;
  auto end_of = [&](int limit, int64_t give_up) {
    int64_t work = 0;
    stored = 0;
    for (int32_t n : tiles) {
      const int parts = parts_of(n, limit);
      if (parts > 1) stored += parts;
      work += (int64_t)parts * ((n + parts - 1) / parts + (parts > 1 ? kPartCost : kWholeCost));
    }
    const int64_t merge = stored ? kMergeCost + stored * n_q_heads / 50 : 0;
    if (work / places + merge >= give_up) return give_up;
    std::array<int64_t, kMaxPlaces> at{};           // a heap: the place that is free soonest in front
    for (int32_t n : tiles) {
      const int parts = parts_of(n, limit);
      for (int p = 0; p < parts; ++p) {
        const int64_t end = at[0] + (n + parts - 1) / parts + (parts > 1 ? kPartCost : kWholeCost);
        int i = 0;
        for (int c = 1; c < places; c = 2 * i + 1) {
          if (c + 1 < places && at[c + 1] < at[c]) ++c;
          if (at[c] >= end) break;
          at[i] = at[c];
          i = c;
        }
        at[i] = end;
      }
    }
    return *std::max_element(at.begin(), at.begin() + places) + merge;
  };
  int best = 0;
  int64_t best_end = end_of(0, INT64_MAX);
  best_end -= best_end / 16;                        // worth it from about a sixteenth on
  int last = 0;
  for (int parts = 2; parts <= kMaxParts; ++parts) {
    const int limit = std::max(2 * kMinPart - 1, (tiles[0] + parts - 1) / parts);   // (then no part is below kMinPart)
    if (limit == last || limit >= tiles[0]) continue;
    last = limit;
    const int64_t end = end_of(limit, best_end);
    if (stored <= max_parts && end < best_end) { best_end = end; best = limit; }
  }
  return best;
}

}  // namespace fp

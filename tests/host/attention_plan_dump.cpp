// Prints what the attention plan (csrc/attention_plan.h) makes of launches read from standard input, one per line:
//   heads max_parts n_sequences new cached [new cached ...]
// Output per line: part size in key tiles (0: whole), parts of every query tile, and the smallest part in key tiles.
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>

#include "../../paper_2602_16603_amd/csrc/attention_plan.h"

int main() {
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    long long heads, max_parts, n_seqs;
    if (!(in >> heads >> max_parts >> n_seqs)) continue;
    std::vector<int32_t> tiles;
    for (long long s = 0; s < n_seqs; ++s) {
      int n = 0, cached = 0;
      in >> n >> cached;
      for (int q = 0; q < n; q += 256) tiles.push_back((cached + std::min(n, q + 256) + 63) / 64);
    }
    std::sort(tiles.rbegin(), tiles.rend());
    const int limit = fp::attention_part_tiles(tiles, (int)heads, max_parts);
    int parts = 0, least = 1 << 30;
    for (int32_t n : tiles) {
      const int p = limit ? (n + limit - 1) / limit : 1;
      if (p > 1) parts += p;
      for (int i = 0; p > 1 && i < p; ++i)
        least = std::min(least, (int)((int64_t)n * (i + 1) / p - (int64_t)n * i / p));
    }
    std::printf("%d %d %d\n", limit, parts, parts ? least : 0);
  }
  return 0;
}

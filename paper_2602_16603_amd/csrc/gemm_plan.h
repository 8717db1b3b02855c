// Which tile a GEMM runs on.  Plain C++17 with no GPU dependency: the rules can be built and checked on the CPU.
#pragma once
#include <cstdint>

namespace fp {

constexpr uint32_t kOffOutOfRange = 0x80000000u;   // a byte offset no buffer descriptor here covers

// Row tile of a grouped launch whose experts receive `mean_rows` rows on average: the smallest that holds most
// experts in one tile, up to 128 rows of the ring kernel; from about 100 rows on the matrix pipes bound the
// launch and the 256-row tile is ahead.  experts_up / experts_down (with the combine) of the 30B-A3B shape, us, with tiles
// of 256, 128, 64 and 32 rows: 6 rows per expert 214/110, 186/97, 170/82, 159/80; 37 rows 224/121, 198/99,
// 187/99, 192/108; with every tile's own start in K: 50 rows -, 194/104, 178/102, -; 64 rows -, 194/109,
// 215/118, -; 119 rows 217/140, 244/145, -, -.
// The smaller tiles reach an expert's gate and up rows through one 32-bit offset, as the dense fused kernel does
// ([2 ffn][hidden] below 2 GiB); the 256-row tile has a base for each.
inline int moe_tile_rows(int64_t mean_rows, int64_t ffn, int64_t hidden) {
  if ((ffn + 256) * hidden * 2 >= (int64_t)kOffOutOfRange) return 256;
  return mean_rows <= 18 ? 32 : mean_rows <= 52 ? 64 : mean_rows <= 100 ? 128 : 256;
}

}  // namespace fp

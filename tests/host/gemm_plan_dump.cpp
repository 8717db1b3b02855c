// Prints what the GEMM dispatch rules (csrc/gemm_plan.h) say to the lines read from standard input:
//   moe mean_rows ffn hidden      -> rows per tile of the experts' grouped launches
#include <iostream>
#include <sstream>
#include <string>

#include "../../paper_2602_16603_amd/csrc/gemm_plan.h"

int main() {
  std::string line, kind;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    if (!(in >> kind)) continue;
    if (kind == "moe") {
      long long rows, ffn, hidden;
      in >> rows >> ffn >> hidden;
      std::cout << fp::moe_tile_rows(rows, ffn, hidden) << "\n";
    }
  }
  return 0;
}

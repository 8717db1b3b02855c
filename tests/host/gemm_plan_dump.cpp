// Prints what the GEMM dispatch rules (csrc/gemm_plan.h) say to the lines read from standard input:
//   moe mean_rows ffn hidden      -> rows per tile of the experts' grouped launches
//   tile m n k residual           -> tile of a problem too small for the large tiles: ring32, ring64, ring128, any128, large
//   rows m n k bf16|swiglu|residual -> rows of the large tile for an uncut problem (swiglu: n outputs)
//   f32 m n k residual            -> rows of the fp32 tile
//   few m n k                     -> 1 if the problem runs on the few-rows kernel
//   starts m n k                  -> groups of columns that start at different k (0: all at the beginning)
//   forms m f k workspace aligned -> the starts that the plain projection of 2 f columns and the fused one of f outputs run with
//                                    (operands on the 16-byte grid or only on the dword grid), whether all of their columns
//                                    start alike (1), and whether the plain one is cut (1) or there is no fused one (2)
//   warm row_tiles                -> shares of a W panel in the large tile's L2 warm-up
//   warm3 k swiglu                -> 1 if the large tile on three stages asks for the warm-up
//   swiglu m f k                  -> rows per tile of its fused gate_up projection (0: two operators)
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
    } else if (kind == "tile") {
      static const char* const names[] = {"ring32", "ring64", "ring128", "any128", "large"};
      long long m, n, k;
      int residual;
      in >> m >> n >> k >> residual;
      std::cout << names[(int)fp::small_problem_tile(m, n, k, residual != 0)] << "\n";
    } else if (kind == "f32") {
      long long m, n, k;
      int residual;
      in >> m >> n >> k >> residual;
      std::cout << fp::f32_tile_rows(m, n, k, residual != 0) << "\n";
    } else if (kind == "few") {
      long long m, n, k;
      in >> m >> n >> k;
      std::cout << fp::few_rows(m, n, k) << "\n";
    } else if (kind == "starts") {
      long long m, n, k;
      in >> m >> n >> k;
      std::cout << fp::start_groups(m, n, k) << "\n";
    } else if (kind == "forms") {
      long long m, f, k, workspace;
      int aligned;
      in >> m >> f >> k >> workspace >> aligned;
      fp::W4Shape p = fp::w4_plan(1, m, 2 * f, k, (size_t)workspace);
      if (p.splits > 1) p = fp::w4_cut(m, 2 * f, k, false, p);
      const bool fusable = fp::swiglu_fusable(m, f, k);
      // (splits 0: the tiles of small problems, which start at the beginning)
      const int plain = p.splits == 1 ? fp::uncut_starts(m, 2 * f, k, p.nj, fp::few_rows(m, 2 * f, k) && aligned) : 0;
      const int fused = fusable ? fp::uncut_starts(m, 2 * f, k, fp::swiglu_nj(m, f), fp::swiglu_few_rows(m, f) && aligned) : 0;
      bool alike = true;
      for (long long col = 0; col < f; col += 8)
        for (long long half : {0LL, f}) alike &= fp::k_start((int)(half + col), (int)k, plain) == fp::k_start((int)col, (int)k, fused);
      std::cout << plain << " " << fused << " " << alike << " " << (fusable ? p.splits > 1 : 2) << "\n";
    } else if (kind == "warm") {
      int row_tiles;
      in >> row_tiles;
      std::cout << fp::warm_shares(row_tiles) << "\n";
    } else if (kind == "warm3") {
      int k, swiglu;
      in >> k >> swiglu;
      std::cout << fp::warm_three_stages(k, swiglu != 0) << "\n";
    } else if (kind == "rows") {
      long long m, n, k;
      std::string epilogue;
      in >> m >> n >> k >> epilogue;
      const bool swiglu = epilogue == "swiglu";
      std::cout << fp::large_tile_rows(m, (n + (swiglu ? 127 : 255)) / (swiglu ? 128 : 256), k,
                                       swiglu ? fp::LargeEpilogue::kSwiGLU : epilogue == "residual" ? fp::LargeEpilogue::kResidual
                                                                                                    : fp::LargeEpilogue::kBf16) << "\n";
    } else if (kind == "swiglu") {
      long long m, f, k;
      in >> m >> f >> k;
      std::cout << fp::swiglu_tile_rows(m, f, k) << "\n";
    }
  }
  return 0;
}

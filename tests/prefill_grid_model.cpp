// The grid of the masked attention's kernels played through on the host (bc_prefill_grid.h): workgroups go to the eight XCDs in
// turn, and inside an XCD to its four shader engines in turn.  Prints for every number of (trajectory, KV head) pairs in a padded
// grid and every number of head splits
//   once      whether every row of the grid has every place once
//   engines   fewest engines that a pair's workgroups come to
//   most      workgroups of a pair that come to one engine, of a thousand, at most
//   run       fewest engines in any four workgroups of a pair that follow one another in the grid
#include <cstdio>
#include <vector>

#include "bc_prefill_grid.h"

using namespace bc;

int main() {
  for (int npairs = 8; npairs <= 400; ++npairs) {
    const int stride = pair_stride(npairs);
    if (stride % 8) continue;
    for (int splits = 1; splits <= 5; ++splits) {
      const int rows = 3 * 5 * 16;
      std::vector<std::vector<int>> engines(stride);
      bool once = true;
      for (int y = 0; y < rows; ++y)
        for (int x = 0; x < splits * stride; ++x) {
          const int pair = pair_in_turn(x % stride, stride, y);
          const long long linear = (long long)y * splits * stride + x;
          if (pair < 0 || pair >= stride || (int)engines[pair].size() != y * splits + x / stride) { once = false; continue; }
          engines[pair].push_back((int)(linear / 8 % 4));
        }
      int fewest = 4, most = 0, run = 4;
      for (const auto& e : engines) {
        int count[4] = {0, 0, 0, 0}, met = 0;
        for (int x : e) ++count[x];
        for (int c : count) { met += c > 0; most = c > most ? c : most; }
        fewest = met < fewest ? met : fewest;
        for (size_t i = 0; i + 4 <= e.size(); ++i) {
          int seen = 0;
          for (int k = 0; k < 4; ++k) seen |= 1 << e[i + k];
          const int n = __builtin_popcount(seen);
          run = n < run ? n : run;
        }
      }
      std::printf("npairs=%d stride=%d splits=%d once=%d engines=%d most=%d run=%d\n", npairs, stride, splits, once, fewest,
                  most * 1000 / (rows * splits), run);
    }
  }
}

// What bc_prefill_grid.h says of the masked attention's launches, on the host.
// "pairs": the grid played through: workgroups go to the eight XCDs in
// turn, and inside an XCD to its four shader engines in turn.  Prints for every number of (trajectory, KV head) pairs in a padded
// grid and every number of head splits
//   once      whether every row of the grid has every place once
//   engines   fewest engines that a pair's workgroups come to
//   most      workgroups of a pair that come to one engine, of a thousand, at most
//   run       fewest engines in any four workgroups of a pair that follow one another in the grid
// Otherwise, for every line "B Hq Hkv d total_rows max_rows rows P c" of the input, what the backward cuts the key blocks of such a
// trajectory into:
//   parts, band   of a dense block and of a response block
//   tiles, bytes  of the chain of the longest dense block, and of one part's sums of all pairs
//   sums, room    rows of partial sums, and of the trajectory's share of the workspace
//   groups, grid  workgroups that have work in a column of the grid, and rows of it
//   one           whether the dq kernel's workgroups go out in the same launch
#include <cstdio>
#include <cstring>
#include <vector>

#include "bc_prefill_grid.h"

using namespace bc;

static void pairs() {
  for (int npairs = 8; npairs <= 400; ++npairs) {
    const int stride = pair_stride(npairs);
    if (stride % 8) continue;
    for (int splits = 1; splits <= 5; ++splits) {
      const int rows = 3 * 5 * 16;
      std::vector<std::vector<int>> engines(stride);
      bool once = true;
      for (int y = 0; y < rows; ++y)
        for (int x = 0; x < splits * stride; ++x) {
          const int pair = pair_in_turn(x % stride, stride, pair_turn(stride), y);
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

static void parts(const long long* a) {
  const int B = (int)a[0], Hq = (int)a[1], Hkv = (int)a[2], d = (int)a[3], max_rows = (int)a[5], rows = (int)a[6], P = (int)a[7], c = (int)a[8];
  const int g = Hq / Hkv, splits = dense_splits(B, Hq, Hkv, a[4]), most = most_parts(splits), band = band_splits(B, Hq, Hkv, a[4], splits);
  const int prompt = c > 0 && P < rows ? P : rows, beacons = c > 0 ? (rows - prompt) / (c + 1) : 0, keys = prompt + beacons;
  const auto blocks = [](int n) { return (n + kDkvKeys - 1) / kDkvKeys; };
  const int dense = blocks(prompt) + blocks(beacons);
  const int n = dense_parts(splits, most, band, least_tiles(g, band), B * Hkv, g, d, rows, keys, dense);
  std::printf("splits=%d parts=%d band=%d tiles=%d bytes=%lld sums=%lld room=%lld groups=%d grid=%lld one=%d\n", splits, n, band, rows / kTileRows * g,
              8ll * d * B * Hkv * keys,
              (long long)(n > 1 ? n * keys : 0) + (band > 1 ? band * (rows - keys) : 0), splits > 1 ? (long long)splits * rows : 0,
              dense * n + blocks(rows - prompt) * band, (long long)dkv_grid_rows(B * Hkv, most, band, blocks(max_rows)),
              (int)in_one_launch(B, B * Hkv, head_tiling(g), a[4]));
}

int main(int argc, char** argv) {
  if (argc == 2 && !std::strcmp(argv[1], "pairs")) return pairs(), 0;
  long long a[9];          // (one trajectory a line of the input)
  while (std::scanf("%lld %lld %lld %lld %lld %lld %lld %lld %lld", a, a + 1, a + 2, a + 3, a + 4, a + 5, a + 6, a + 7, a + 8) == 9) parts(a);
}

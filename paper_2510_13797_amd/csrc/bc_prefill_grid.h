// Which workgroup of the masked attention's kernels works on what, and where the hardware puts it.  Plain arithmetic without
// memory, shared by the kernels, the calls that launch them and a host test that plays a grid through.
#pragma once
#include <cmath>
#include <cstdint>

#ifndef BC_HOST_DEVICE
#if defined(__HIPCC__)
#define BC_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define BC_HOST_DEVICE inline
#endif
#endif

namespace bc {

constexpr int kTileRows = 32;         // rows of a staged tile; query rows of a wave
constexpr int kTileWaves = 4;         // waves of a workgroup

// ---------------------------------------------------------------------------
// how the heads of a group are dealt to the waves of a workgroup
// ---------------------------------------------------------------------------
struct HeadTiling {
  int32_t heads;        // query heads per workgroup: 4, 2 or 1
  int32_t splits;       // workgroups that share a group's heads
  int32_t row_blocks;   // blocks of 32 query rows per workgroup: kTileWaves / heads
};
// Four waves, one per SIMD: three workgroups then fit a CU whatever SIMD each starts on (six waves
// per workgroup, all heads of a group of six: 1.22 against 0.77 ms, the second workgroup found no
// SIMD with room for two more waves).  As many heads as divide the group into fours or twos without a
// remainder, since more rows per workgroup mean a longer masked band: groups of six with one head and
// 128 rows took 0.75, with two heads and 64 rows 0.70 ms; groups of four with two heads 0.523, with
// four heads and 32 rows 0.511 ms.
inline HeadTiling head_tiling(int g) {
  const int heads = g % 4 == 0 || g == 7 ? 4 : g % 2 == 0 ? 2 : 1;
  return {heads, (g + heads - 1) / heads, kTileWaves / heads};
}

// ---------------------------------------------------------------------------
// where a (trajectory, KV head) pair stands in a row of the grid
// ---------------------------------------------------------------------------
// Workgroups go to the 8 XCDs in turn.  With the pairs of a row tile (and its head splits) padded to a
// multiple of 8, all tiles of a pair - which read the same prompt and beacon rows - share an L2; for
// few pairs that would leave XCDs idle (three trajectories with two KV heads: six of eight XCDs at
// work), and the tiles are dealt out evenly instead.
inline int pair_stride(int npairs) { return npairs % 8 == 0 || npairs > 64 ? (npairs + 7) & ~7 : npairs; }
// Inside an XCD they go to its four shader engines in turn, and a workgroup waits for a place in the engine whose turn it is.  With an
// even number of pairs an XCD, a pair at the same place in every row of the grid has its workgroups on one engine or two, and
// trajectories of different length or ratio then wait for the engine of the heaviest while the others stand idle (8 of 1482 to 5617 rows, ratios
// of 2 to 32, 32/8 heads, forward with workspace: a third of the compute units idle, a call takes 487 us; 394 with the pairs of an XCD
// changing places from row to row; 16 equal trajectories take what they took).  Two pairs an XCD change places every other row:
// every row, a step of two workgroups and one back, they came to two engines again, and gradients in one launch of both kinds of workgroup
// lost by it (eight of 26 to 2364 rows, 8/2 heads, 172 us in two launches, 185 in one, 134 now; two of 1058 and 4362, 32/8 heads, forward 82 and
// 60).  An odd number comes to all four in turn by itself, and changing places
// would undo that (130 trajectories, 129 of some 50 rows and one of 14,046, 5/1 heads, ratio 4: forward 590 us, 469 at the same place, gradients 2503 and
// 2067; 27 of which one has 956 rows, 32/8 heads: forward 31.8 and 27.0).
// pair_turn(): eight times the places of a row, which the launch works out (chosen in the kernel: 383.4 us for that forward, 381.9 so, 381.2 before).
inline int pair_turn(int pstride) { return pstride % 16 ? 0 : pstride == 16 ? 4 : 8; }
BC_HOST_DEVICE int pair_in_turn(int at, int pstride, int turn, unsigned row) {
  return turn ? (int)((at + (row * (unsigned)turn & ~7u)) % (unsigned)pstride) : at;
}

// ---------------------------------------------------------------------------
// what the backward's key blocks are cut into
// ---------------------------------------------------------------------------
constexpr int kDkvKeys = 64;          // keys of a workgroup: two pairs of waves with 32 keys each
constexpr int kDkvAtOnce = 3 * 256;   // workgroups that run at once at d = 128; at 64 it would be four a compute unit, which no rule here uses
constexpr int kMostSplits = 8, kMostParts = 16;

// Partial sums the workspace has room for, of every row: what dense_parts() chooses from.
// A dense block streams all later rows of all heads, a chain of up to g * rows/32 tiles, and there are few of
// them: they are cut until as many as run at once (three per CU) are there, taking one key in eight for dense
// (ratios and prompt lengths are on the device).  Backward of 6 trajectories, 14/2 heads, d = 64, 12,966 rows: two
// parts 523 us, six 300; one trajectory of 6631 rows, 24/8 heads: 597, three 372; three short trajectories: 118,
// six 62; more parts than that cost work (16 trajectories of 8688 rows: two 2.70 ms, three 2.66, six 2.82; 8 of
// 3389 rows, 32/8 heads: 2.37, 2.40, 2.55).  Parts of fewer than eight tiles are not worth their partial sums.
inline int dense_splits(int B, int Hq, int Hkv, int64_t total_rows) {
  constexpr int64_t kMost = kMostSplits;
  const int64_t blocks = total_rows * Hkv / (8 * kDkvKeys) + 1;
  const int64_t tiles = total_rows / B * (Hq / Hkv) / kTileRows;      // of a chain
  const int64_t n = (kDkvAtOnce + blocks - 1) / blocks, least = Hq > Hkv ? 2 : 1;
  const int64_t most = tiles / 8 < kMost ? tiles / 8 : kMost;
  return (int)(n < least || most < least ? least : n > most ? most : n);
}

// Workgroups that share a response block: a chain of about three tiles for each head of a group, which is what a launch of
// a few trajectories takes where the chip is not full.  As many as run at once beside the dense blocks' parts, at least
// two heads each.  Three trajectories of 336 to 795 rows, 12/2 heads, whole 69.3 us a pass, in three parts 67.1
// (the dense blocks' chains are as long); three of 300 rows, 14/2 heads, d = 64, 56.9 and 50.2; of 380 rows (forward and gradients in one
// graph), 12/2 heads 59.5 and 51.9, d = 64 45.9 and 40.0, but three of 830 rows 69.4 and 71.0.  Groups of fewer than six heads stay
// whole: two trajectories of 216 rows, 4/1 heads, 44.5 and in two parts 44.9, called one by one.  In one graph groups of five gain as those of six do (two of
// 270 rows, 5/1 heads 51.8 and 45.7, three of 830 64.6 and 65.1), groups of four half as much (43.0 and 40.1, 55.5 and 56.0).
inline int band_splits(int B, int Hq, int Hkv, int64_t total_rows, int splits) {
  const int64_t pairs = (int64_t)B * Hkv, g = Hq / Hkv;
  if (g < 6) return 1;
  const int64_t blocks = total_rows * Hkv / kDkvKeys;        // one in eight dense, as above
  const int64_t n = (kDkvAtOnce - (blocks / 8 + 2 * pairs) * splits) / (blocks - blocks / 8 + pairs);
  const int64_t most = g / 2 < splits ? g / 2 : splits;
  return (int)(n < 1 ? 1 : n > most ? most : n);
}

// Most workgroups that share a dense key block: more than there is room for of every row only where the chip is not full.
BC_HOST_DEVICE int most_parts(int splits) { return splits == kMostSplits ? kMostParts : splits; }

// Parts of a trajectory's dense key blocks: as many as run at once if all trajectories are like this one, and two where the heads of a
// group make the chain long.  One part stores its result directly.  (The host does not know how many keys are dense, and reckons with
// one in eight.  Cut by that alone, 4 uncompressed trajectories of 2200 rows, 8/8 heads, had six parts of 1120 blocks and took
// 376 us, 318 whole.)
// A trajectory has room for `splits` sums of every row, and the fewer of its rows are dense the more parts fit, up to `most`.  The n-th part takes
// some tiles / n^2 off the chain and costs one more sum of all dense keys: worth it up to kSumBytes for a tile, and for parts of eight
// tiles that are no shorter than a part of a response block (least_tiles()).  Both from 600 batches of up to 48 trajectories, each with at
// most 8, 10, 12, 14 and 16 parts; of 234 others, the gradients of which take 0.68 to 1.10 of the time with at most eight
// (mean 0.964).  By parts of eight tiles and 18 MB together, which is what one batch had said, it was 0.69 to 1.20 (0.987): ten of 450 to 1153 rows,
// 4/1 heads, d = 64, 49.4 us with eight, 50.0 now, 52.6 so; one of 1229, 24/8 heads, 50.5, 50.4 and 57.1.  (The root and the quotient exactly, in front of
// every workgroup's first load: 0.2 us of a small pass.  All of this with sums that cost some twice what they do now on small launches: a part more may pay there
// where it does not get one.)
constexpr float kSumBytes = 0.5e6f;
inline int least_tiles(int g, int band) { return 3 * ((g + band - 1) / band) > 8 ? 3 * ((g + band - 1) / band) : 8; }
BC_HOST_DEVICE float approximate_root(float a, float b) {        // of a / b
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_sqrtf(a * __builtin_amdgcn_rcpf(b));
#else
  return sqrtf(a / b);
#endif
}
BC_HOST_DEVICE int dense_parts(int splits, int most, int band, int least, int npairs, int g, int D, int rows, int dense_keys, int dense_blocks) {
  const int some = dense_blocks < 1 ? 1 : dense_blocks > kDkvAtOnce ? kDkvAtOnce : dense_blocks, blocks = some * npairs;
  const int n = (kDkvAtOnce + blocks - 1) / blocks, wanted = n < 2 && g > 1 ? 2 : n;
  int fit = splits;                // (room for `splits` there always is: the tokens have band <= splits)
  if (most > splits) {
    const int keys = dense_keys < 1 ? 1 : dense_keys;
    const int room = (splits * rows - (band > 1 ? band * (rows - dense_keys) : 0)) / keys;
    const int tiles = rows / kTileRows * g, long_enough = tiles / least;
    const int few = (int)approximate_root(kSumBytes * tiles, 8.f * D * npairs * keys);
    int more = room < few ? room : few;
    more = more < long_enough ? more : long_enough;
    more = more < most ? more : most;
    fit = fit < more ? more : fit;
  }
  return wanted < fit ? wanted : fit;
}

// Rows of the dkv grid.  Key blocks of a trajectory: at most `key_blocks` of response rows, and of prompt keys and gathered beacons,
// which are rows of it too, one more.  The parts of the latter together are at most two each, or as many workgroups as run at once and
// the last of each block's (dense_parts()).  A workgroup that finds no part costs 1 us in a thousand.
inline int64_t dkv_grid_rows(int npairs, int most, int band, int key_blocks) {
  const int dense_blocks = key_blocks + 1;
  const int64_t at_once = kDkvAtOnce / npairs + dense_blocks, all = (int64_t)dense_blocks * most;
  const int64_t least = (int64_t)dense_blocks * (most < 2 ? most : 2);
  return (all < at_once ? all : at_once < least ? least : at_once) + (int64_t)key_blocks * band;
}

// The waves that add the parts up: keys a wave takes at a time where a key's row of dk (all KV heads) has less than 64 units of 16 bytes, slices
// of 64 units where it has more.
BC_HOST_DEVICE int reduce_keys(int per_row) { return per_row < 64 ? 64 / per_row : 1; }
BC_HOST_DEVICE int reduce_slices(int per_row) { return per_row <= 64 ? 1 : (per_row + 63) / 64; }
// Workgroups (of four waves) a trajectory at most.
inline int reduce_blocks(int B) { return B <= 4 ? 1024 : B >= 32 ? 128 : 4096 / B; }

// ---------------------------------------------------------------------------
// the backward's launches
// ---------------------------------------------------------------------------
// Whether dq and dkv blocks go out in one launch: where the dq kernel's workgroups (of trajectories of the mean length) are no more than
// the compute units, and for four pairs and fewer, whose dkv kernel does not fill the chip either, no more than run at once.  Otherwise the
// chip has work for one kernel after the other, with three dkv workgroups a compute unit in place of two (d = 64: four, three) and none
// for Delta.  712 batches in one launch, most of them of one or two long trajectories beside short ones (which the mean does not tell), take 0.73
// of the time of the gradients before there was one, the worst 1.04.  Forward and gradients, us a pass behind other work, in two launches and in one, ratio 16, 4, 0 (those rows of a ratio
// that lie on the other side of the line in brackets).  The line was drawn for a joined kernel that was 2 to 6 % slower: from 240 to 290 workgroups of 12/2 heads some
// would gain up to 11 % beyond it, others (32/8 heads, 480 workgroups) lose 2 to 4 %.
//   trajectories x tokens, heads   dq workgroups
//   1 x 500, 12/2                     54, 60,  48    44.9 37.7 | 52.3  41.6 |  71.4  57.1
//   1 x 500, 8/8                      40, 40,  32    46.3 36.6 | 51.4  38.7 |  71.2  51.3
//   1 x 1000, 14/2, d = 64           136,156, 128    43.1 39.5 | 53.5  46.8 |  95.0  76.7
//   6 x 384, 12/2                    252,288, 216    51.9 50.8 |(60.5  57.4)|  72.3  65.1
//   4 x 600, 12/2                    240,288, 240    55.6 53.8 |(69.3  61.7)|  90.0  80.4
//   2 x 500, 32/8                    272,304, 256   (51.0 52.7)|(62.4  61.3)|  85.1  79.1
//   8 x 500, 12/2                    432,480, 384   (62.6 64.0)|(78.2  81.6)| (95.2  94.6)
//   1 x 4000, 12/2 (two pairs)       402,468, 378     110  102 |  174   167 |   453   404
//   2 x 2000, 12/2 (four)            408,468, 384    84.2 77.8 |  127   128 |   248   220
inline bool in_one_launch(int B, int npairs, const HeadTiling& tiling, int64_t total_rows) {
  const int64_t rows = kTileRows * tiling.row_blocks * (int64_t)B;
  const int64_t blocks = (total_rows + rows - 1) / rows * npairs * tiling.splits;
  return blocks <= (npairs <= 4 ? 512 : 256);
}

}  // namespace bc

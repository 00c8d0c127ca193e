// Which workgroup of the masked attention's kernels works on what, and where the hardware puts it.  Plain arithmetic without
// memory, shared by the kernels, the calls that launch them and a host test that plays a grid through.
#pragma once
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
// changing places from row to row; 16 equal trajectories take what they took).  Two pairs an XCD with one head split come to two engines
// either way, for every other even number it is four.  An odd number comes to all four in turn by itself, and changing places
// would undo that (130 trajectories, 129 of some 50 rows and one of 14,046, 5/1 heads, ratio 4: forward 590 us, 469 at the same place, gradients 2503 and
// 2067; 27 of which one has 956 rows, 32/8 heads: forward 31.8 and 27.0).
BC_HOST_DEVICE int pair_in_turn(int at, int pstride, unsigned row) {
  return pstride % 16 == 0 ? (int)((at + 8u * row) % (unsigned)pstride) : at;
}

}  // namespace bc

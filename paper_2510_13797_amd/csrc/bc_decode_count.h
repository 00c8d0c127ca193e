// How the workgroups of a decode step agree that a sequence is done.  Plain arithmetic without memory, shared
// by the kernels and by a host test that plays every order in which the workgroups of a sequence can start.
//
// A launch has max_chunks workgroups for every (sequence, KV head) pair, a step rewrites the sequence's tables
// at its end, and every wave works out from the tables which rows are its own.  So the tables may move only
// when every wave of every workgroup of the sequence has read them, the workgroups without rows among them:
// one that starts late (behind another stream's work, or in the second round of a grid that does not fit the
// chip) would otherwise see a sequence one row longer, find itself a chunk, and count where nobody expects it.
//
//  * A whole sequence (one chunk): whoever has rows takes its tickets as soon as its loads have landed, and
//    a workgroup without rows takes one; the holder of the sequence's last ticket finishes the step.
//  * A sequence cut into chunks: every workgroup of a pair arrives at the pair's counter, with or without a
//    chunk; the last one folds the pair's partial results and takes one ticket for the pair.
// A launch that leaves a sequence's tables alone counts only what it has to fold.
#pragma once

#if defined(__HIPCC__)
#define BC_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define BC_HOST_DEVICE inline
#endif

namespace bc {

struct SequenceCut { int rows_per_chunk, nchunks; };

// L >= 1 resident rows.  forced > 0: rows of a chunk; otherwise the rows are spread evenly over as many of
// the max_chunks workgroups as have chunk_rows rows to read, and a sequence shorter than split_rows stays
// whole (its partial would cost more than the cut saves).
BC_HOST_DEVICE SequenceCut cut_sequence(int L, int forced, int max_chunks, int split_rows, int chunk_rows) {
  int rows = forced;
  if (rows <= 0 && max_chunks == 1) return {(L + 31) & ~31, 1};
  if (rows <= 0) {
    const int by_rows = (L + chunk_rows - 1) / chunk_rows;
    const int n = L < split_rows ? 1 : by_rows < max_chunks ? by_rows : max_chunks;
    rows = (((L + n - 1) / n) + 31) & ~31;
  }
  return {rows, (L + rows - 1) / rows};
}

enum class CloseBy { nothing, ticket, arrival };

// What a workgroup does behind its reads.  update: the launch rewrites the sequence's tables.
BC_HOST_DEVICE CloseBy closing_move(bool update, bool has_chunk, int nchunks) {
  if (nchunks > 1) return update || has_chunk ? CloseBy::arrival : CloseBy::nothing;
  return update ? CloseBy::ticket : CloseBy::nothing;
}
// arrivals of a pair of a cut sequence
BC_HOST_DEVICE int arrivals_due(bool update, int nchunks, int max_chunks) { return update ? max_chunks : nchunks; }
// tickets of a sequence; own: tickets the workgroups with rows of one pair take
BC_HOST_DEVICE int tickets_due(int Hkv, int own, int nchunks, int max_chunks) {
  return nchunks > 1 ? Hkv : Hkv * (own + max_chunks - 1);
}

}  // namespace bc

// bc_decode_attn: single-token grouped-query attention over the ragged compressed cache
// (Sec. 2 and Sec. 3.1 of the paper: standard attention over whatever is resident).
//
// Split-K flash decoding.  Work item = (sequence, KV head) pair x chunk of rows; grid =
// (KV heads, sequences, chunks).  From 128 pairs on (fp32: 129, but see f32_split_rows) a pair is one chunk and its workgroup
// finishes it.  With fewer pairs the resident rows of a sequence are spread evenly over up to 64
// workgroups (short sequences stay whole, see make_plan); every chunk
// writes an (m, l, o) partial and the workgroup that arrives last folds the partials of its pair in
// chunk order.  No float atomics and no fences: results are bit-reproducible.  Large ragged batches
// (more pairs than compute units) can dispatch the longest sequences first (bc_sort_by_length).
// Batches of at most 128 pairs with short caches use two workgroups per pair, each with all K rows and
// one half of the V columns, so that all compute units pull data and nothing has to be merged.
//
// Two main kernels:
//  * decode_lds_kernel (bf16, d = 128 or 64; decode_lds_cut_kernel where sequences are cut): every
//    wave streams 32-row K and V tiles from HBM straight into its own LDS region with 16-byte LDS-DMA
//    loads (1 KB of consecutive bytes per instruction, 16 KB in flight per wave at d = 128), then forms
//    the q.K products and the p.V sums of all query heads of the group with 16x16x32 bf16 MFMA tiles
//    fed from LDS (K by 128-bit reads, V by the 16-bit transposing reads), softmax in registers.
//  * decode_valu_kernel (fp32): rows held in registers, 16 bytes per lane, fed to the fp32 matrix
//    instructions; for bf16 rows, where the plan asks for it, plain FMA dot products completed by a
//    DPP all-reduce.
// Both carry the fused step (append before, eviction after the attention) in the same launch: the
// appended row is read from the caller's tensors, everyone who has read a sequence's tables is counted
// (bc_decode_count.h), and the holder of the sequence's last ticket moves the beacon and the tables.
#include <algorithm>
#include <atomic>
#include <climits>
#include <cstdint>
#include <cstdio>
#include <type_traits>
#include "bc_common.h"
#include "bc_decode_count.h"

namespace bc {

// Every sequence's ticket counter has a 128-byte line to itself: the workgroups of a launch finish
// close together, and their atomics on a shared line would queue up behind each other.
constexpr int kTicketStride = 32;

struct DecodeParams {
  const char* k_slab;
  const char* v_slab;
  const int64_t* base;
  const int32_t* cap;
  const int32_t* P;
  const int32_t* nb;
  const int32_t* w;
  int32_t* err;
  const char* q;
  float* out;
  const uint8_t* active;
  float* part;         // [pairs][max_chunks][Gp*D + kPartTail]: o, then (running max in log2 units, denominator) of every head
  int32_t* arrivals;   // chunks of a pair whose partial is written; zero between launches
  int64_t arrival_stride;     // from sequence to sequence (the pairs of a sequence are neighbours)
  // fused step (all nullable): append this token row first, evict with this beacon afterwards
  const int32_t* c;
  int32_t* nb_rw;
  int32_t* w_rw;
  const char* new_k;
  const char* new_v;
  const char* bk;
  const char* bv;
  int32_t* tickets;    // [B] counters kTicketStride ints apart, zero between launches
  const int32_t* order;     // [B] dispatch order (workgroup i serves sequence order[i]) or null
  const int32_t* budget;   // [B] cap on nb + w (nullable), with
  uint8_t* live;           // [B] cleared when the cap is reached
  int32_t beacon_row;  // the fused row is the beacon closing a full window (bk = new_k, bv = new_v)
  int32_t B;
  int32_t spec_P, spec_cap;   // bc_cache::uniform_P, uniform_cap (0 = no promise)
  int32_t Hq, Hkv, g;  // g = real group size
  int32_t Gp;          // padded group size of the partial layout
  int32_t rows_per_wg; // R: rows per workgroup when a chunk size is forced; otherwise (0) the
                       // resident rows of a sequence are spread evenly over its chunks
  int32_t max_chunks;
  int32_t chunk_rows;  // rows a chunk is cut down to, as long as there are chunks left
  int32_t split_rows;  // shorter sequences stay whole
  float qscale;        // softmax scale * log2(e)
};

// Kernels that wait for one round trip after the other take the addresses of the tables as arguments of their own in front of the others, the
// number of which (FILE_FLAGS) the hardware leaves in scalar registers: the tables are asked for by the first instructions (cut sequences: a step 0.1 us
// shorter).  Where the first tiles are asked for before the tables are back it is no gain: they wait for the other arguments, and one counter serves both.
#define BC_TABLE_ARGUMENTS const int32_t *tP, const int32_t *tnb, const int32_t *tw, const int32_t *tcap, const int32_t *tc, const int64_t *tbase
constexpr int kTableArguments = 6 * 8;      // bytes

struct PairInfo {
  int s, kvh, L, nchunks, chunk, row0, row_end;
  int P, nb, w_att, cap, c;   // tables as the attention of this launch sees them
  int64_t base;               // first entry of the sequence in the slabs
  int new_row;                // slot of the row appended by this launch, or -1
  bool evict_due;             // this launch ends with beacon append + eviction
  bool store_new_row;         // the appended row outlives this launch: write it to the slab
  bool update;                // tables change at the end of this launch
  bool live;
};

// Common prologue: which rows does this workgroup own?  Uniform across the workgroup.  All
// table loads are issued together.  With a fused append the state rules of bc_append_kv are
// applied here, identically in every workgroup of the sequence.
constexpr int kLptMaxB = 4096;       // sort key: length * 4096 + index
constexpr int kLptMaxLen = 1 << 19;
constexpr int kLptMinPairs = 256;    // compute units of the chip: below this every workgroup starts at once

// Longest sequence first: with more workgroups than the chip holds at once and ragged lengths,
// the dispatch order decides the tail.  bc_sort_by_length ranks the B sequences by resident
// length (keys made unique by the index, so the ranks are a permutation) into an array the
// caller owns; with that array in bc_cache::order, workgroup number i of a decode launch (in
// dispatch order) serves sequence order[i].  The array is only read by the decode launches, so
// every workgroup sees the same permutation even while a fused step updates the tables, and it
// may be as old as the caller likes.
struct SortParams {
  const uint8_t* active;
  const int32_t *P, *nb, *w;
  int32_t* order;
  int32_t B;
};

__global__ __launch_bounds__(256) void sort_by_length_kernel(SortParams p) {
  __shared__ int s_key[kLptMaxB];
  for (int t = threadIdx.x; t < p.B; t += blockDim.x) {
    const int act = p.active ? p.active[t] : 1;
    int len = act ? p.P[t] + p.nb[t] + p.w[t] + 1 : 0;         // inactive sequences rank last
    len = min(max(len, 0), kLptMaxLen - 1);
    s_key[t] = (len << 12) | (kLptMaxB - 1 - t);
  }
  for (int t = p.B + threadIdx.x; t < ((p.B + 3) & ~3); t += blockDim.x) s_key[t] = -1;
  __syncthreads();
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= p.B) return;
  const int mine = s_key[t];
  int rank = 0;                                               // number of larger keys
  for (int u = 0; u < p.B; u += 4) {
    const int4 o = *reinterpret_cast<const int4*>(s_key + u);
    rank += (o.x > mine) + (o.y > mine) + (o.z > mine) + (o.w > mine);
  }
  p.order[rank] = t;
}

// The kernel arguments span four 64-byte lines, five with AT bytes of table addresses in front, that the code below would touch one
// after the other, each a miss of the scalar cache on the way to the first tile request: ask for all of them at once.
// LAST: the last line too (kernels that begin with the query's address ask for what it holds anyway; asked for twice, a step is 0.4 % longer).
template <int AT, bool LAST = true>
__device__ __forceinline__ void touch_kernel_arguments() {
  typedef __attribute__((address_space(4))) const int const_int_t;
  const_int_t* ka = (const_int_t*)__builtin_amdgcn_kernarg_segment_ptr();
  constexpr int kLines = (AT + (int)sizeof(DecodeParams) + 63) / 64;
  static_assert(AT < 64 && (kLines == 4 || kLines == 5), "a load for every line of the arguments");
  const int a = ka[AT / 4], b = ka[16], c = ka[32], d = ka[kLines == 5 || LAST ? 48 : 32], e = ka[LAST ? 16 * (kLines - 1) : 32];
  asm volatile("" : : "s"(a), "s"(b), "s"(c), "s"(d), "s"(e));
}

// The kernel arguments, to be read afresh: what only the end of a kernel needs holds no scalar registers before
// (kept from the start, 38 of them went through vector lanes in front of the first tile requests: one sequence of
// 1551 rows, 8 KV heads, 11.8 us a step instead of 10.8).
template <int AT>
__device__ __forceinline__ DecodeParams arguments_again() {
  typedef __attribute__((address_space(4))) const char const_char_t;
  typedef __attribute__((address_space(4))) const DecodeParams const_params_t;
  const_params_t* at = (const_params_t*)((const_char_t*)__builtin_amdgcn_kernarg_segment_ptr() + AT);
  asm volatile("" : "+s"(at));
  return *(const DecodeParams*)at;
}

// slot: the sequence's index, or its rank in the dispatch order when there is one.  The grid
// carries (KV head, slot, chunk) in its three dimensions, so that nothing has to be divided
// before the tables can be requested; all of them are requested together.
struct NoEarlyWork { __device__ __forceinline__ void operator()() const {} };
// The six table entries travel through the scalar cache, requested by hand: their counter is not the vector loads' one, so work started in
// the meantime (the first tile, when the caller has promised the slab geometry) does not have to be back before they are.
struct TableEntries { int32_t P, nb, w, cap, c; int64_t base; };
__device__ __forceinline__ void request_tables(const DecodeParams& p, int s, TableEntries& t) {
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(t.P) : "s"(p.P + s) : "memory");
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(t.nb) : "s"(p.nb + s) : "memory");
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(t.w) : "s"(p.w + s) : "memory");
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(t.cap) : "s"(p.cap + s) : "memory");
  asm volatile("s_load_dwordx2 %0, %1, 0x0" : "=s"(t.base) : "s"(p.base + s) : "memory");
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(t.c) : "s"(p.c + s) : "memory");
}
// early: the entries of sequence `slot`, requested before.
template <typename F = NoEarlyWork>
__device__ __forceinline__ PairInfo pair_info(const DecodeParams& p, int slot, int kvh, int chunk,
                                              const F& while_tables_travel = F(), const TableEntries* early = nullptr) {
  PairInfo pi;
  TableEntries t;
  int act, w;
  int s = slot;
  bool bad_order = false;
  // (values that are the same for the whole workgroup are moved to scalar registers where the
  // compiler cannot see that itself - anything it loads through the vector path - so that the
  // conditions on them become real branches instead of lane masks)
  if (p.order) {
    s = __builtin_amdgcn_readfirstlane(p.order[slot]);
    bad_order = (unsigned)s >= (unsigned)p.B;        // not written by bc_sort_by_length
    if (bad_order) s = 0;
  }
  pi.s = s;
  pi.kvh = kvh;
  {
    if (early == nullptr) {
      request_tables(p, pi.s, t);
    } else if (p.order) {
      // the sequence is another than the early request took it for, whose entries are on their way all the same: scalar loads return in any
      // order, and their registers are not free before they have
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : : "s"(early->P), "s"(early->nb), "s"(early->w), "s"(early->cap), "s"(early->base), "s"(early->c) : "memory");
      request_tables(p, pi.s, t);
    } else {
      t = *early;
    }
    while_tables_travel();
    asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(t.P), "+s"(t.nb), "+s"(t.w), "+s"(t.cap), "+s"(t.base), "+s"(t.c) : : "memory");
    pi.P = t.P; pi.nb = t.nb; w = t.w; pi.cap = t.cap; pi.base = t.base; pi.c = t.c;
    // (the address of the kernel arguments keeps its registers up to here: the check of the generated code
    // tells these loads from the arguments' by them)
    asm volatile("" : : "s"(__builtin_amdgcn_kernarg_segment_ptr()));
  }
  act = p.active ? __builtin_amdgcn_readfirstlane((int)p.active[pi.s]) : 1;
  if (bad_order) {
    if (chunk == 0 && threadIdx.x == 0) atomicOr(p.err, BC_ERRBIT_STATE);
    act = 0;
  }
  const bool herald = chunk == 0 && pi.kvh == 0 && threadIdx.x == 0;   // reports errors
  pi.live = false;
  pi.update = false; pi.evict_due = false; pi.new_row = -1; pi.store_new_row = false;
  pi.L = 0; pi.nchunks = 0; pi.chunk = chunk; pi.row0 = 0; pi.row_end = 0; pi.w_att = w;
  // beacon step: only sequences whose window is full take part; one that has no room for the
  // beacon at the tail is reported and left alone
  bool take = act != 0;
  if (take && p.beacon_row) {
    take = pi.c > 0 && w == pi.c;
    if (take && pi.P + pi.nb + w >= pi.cap) {
      if (herald) atomicOr(p.err, BC_ERRBIT_CAPACITY);
      take = false;
    }
  }
  if (take) {
    const int L_old = pi.P + pi.nb + w;
    bool append_ok = false;
    if (p.beacon_row) {
      append_ok = true;
    } else if (p.new_k) {
      if (pi.c > 0 && w >= pi.c) { if (herald) atomicOr(p.err, BC_ERRBIT_STATE); }
      else if (L_old >= pi.cap)  { if (herald) atomicOr(p.err, BC_ERRBIT_CAPACITY); }
      else append_ok = true;
    }
    pi.L = L_old + (append_ok ? 1 : 0);
    pi.w_att = w + (append_ok ? 1 : 0);
    if (append_ok) pi.new_row = L_old;
    if (p.beacon_row) {
      pi.evict_due = true;          // the row just attended to moves behind the earlier beacons
    } else if (p.bk && pi.c > 0) {
      if (pi.w_att == pi.c + 1) { if (herald) atomicOr(p.err, BC_ERRBIT_STATE); }
      else if (pi.w_att == pi.c) pi.evict_due = true;
    }
    // a row that this step's eviction drops at once (c = 1, or the beacon itself, which goes
    // straight to its slot behind the earlier beacons) is never written at the tail
    pi.store_new_row = append_ok && !(pi.evict_due && (pi.w_att == 1 || p.beacon_row));
    if (pi.L <= 0) {
      if (herald) atomicOr(p.err, BC_ERRBIT_STATE);
    } else {
      const SequenceCut cut = cut_sequence(pi.L, p.rows_per_wg, p.max_chunks, p.split_rows, p.chunk_rows);
      const int rpc = cut.rows_per_chunk;
      pi.nchunks = cut.nchunks;
      // the evaluation cap is tested on what this step's attention sees, whether or not the
      // append went through
      pi.update = append_ok || pi.evict_due ||
                  (p.budget && pi.nb + pi.w_att >= __builtin_amdgcn_readfirstlane(p.budget[pi.s]));
      if (pi.chunk < pi.nchunks) {
        pi.row0 = pi.chunk * rpc;
        pi.row_end = min(pi.L, pi.row0 + rpc);
        pi.live = true;
      }
    }
  }
  // (uniform by construction; said explicitly for what went through vector arithmetic)
  pi.L = __builtin_amdgcn_readfirstlane(pi.L);
  pi.nchunks = __builtin_amdgcn_readfirstlane(pi.nchunks);
  pi.row0 = __builtin_amdgcn_readfirstlane(pi.row0);
  pi.row_end = __builtin_amdgcn_readfirstlane(pi.row_end);
  pi.new_row = __builtin_amdgcn_readfirstlane(pi.new_row);
  pi.live = __builtin_amdgcn_readfirstlane((int)pi.live) != 0;
  pi.update = __builtin_amdgcn_readfirstlane((int)pi.update) != 0;
  pi.evict_due = __builtin_amdgcn_readfirstlane((int)pi.evict_due) != 0;
  pi.store_new_row = __builtin_amdgcn_readfirstlane((int)pi.store_new_row) != 0;
  return pi;
}

// The beacon entry of KV heads head0 .. head0 + heads - 1 goes to its slot behind the earlier beacons (the evicted
// window's first row): by threads 0 .. threads - 1, once every reader of these heads' rows is done with them.  Four units
// a thread are asked for before the first is stored.  FROM_LDS: from the heads' K and V rows as request_beacon left them, one of each at a time (in a loop of its
// own, which is shorter code; steps that evict differ by less than their runs do).
constexpr int kBeaconBytes = 4096;
template <int ROWB, bool FROM_LDS>
__device__ __forceinline__ void store_beacon(const DecodeParams& p, const PairInfo& pi, int head0, int heads, int thread,
                                             int threads, const char* lds_k = nullptr, const char* lds_v = nullptr) {
  constexpr int UPR = ROWB / 16;                   // 16-byte units per row
  const int n16 = heads * UPR;                     // 16-byte units of K (or of V)
  const int64_t slot = (pi.base * p.Hkv + (int64_t)head0 * pi.cap + pi.P + pi.nb) * ROWB, head_bytes = (int64_t)pi.cap * ROWB;
  auto place = [&](int i) { return slot + (int64_t)(i / UPR) * head_bytes + ((i & (UPR - 1)) << 4); };
  if constexpr (FROM_LDS) {
#pragma clang loop unroll(disable)
    for (int i = thread; i < n16; i += threads) {
      const u32x4_t k = *reinterpret_cast<const u32x4_t*>(lds_k + (i << 4)), v = *reinterpret_cast<const u32x4_t*>(lds_v + (i << 4));
      *reinterpret_cast<u32x4_t*>(const_cast<char*>(p.k_slab) + place(i)) = k;
      *reinterpret_cast<u32x4_t*>(const_cast<char*>(p.v_slab) + place(i)) = v;
    }
  } else {
    const int64_t src0 = (int64_t)(pi.s * p.Hkv + head0) * ROWB;
    auto unit = [&](int i) { return *reinterpret_cast<const u32x4_t*>((i >= n16 ? p.bv - n16 * 16 : p.bk) + src0 + (i << 4)); };
    auto put = [&](int i, u32x4_t x) {
      const int which = i >= n16;
      if (i < 2 * n16) *reinterpret_cast<u32x4_t*>(const_cast<char*>(which ? p.v_slab : p.k_slab) + place(which ? i - n16 : i)) = x;
    };
    for (int i = thread; i < 2 * n16; i += 4 * threads) {
      const int end = 2 * n16 - 1;
      const u32x4_t a = unit(i), b = unit(min(i + threads, end)), c = unit(min(i + 2 * threads, end)), d = unit(min(i + 3 * threads, end));
      put(i, a); put(i + threads, b); put(i + 2 * threads, c); put(i + 3 * threads, d);
    }
  }
}
// The beacon rows of all KV heads into LDS (by one wave, uncounted loads), where they fit, for whoever turns out to
// draw the sequence's last ticket.  Asked for then, they were round trips to pages that nothing had touched yet, at the very
// end of the step (a step that evicts: 32/8 heads, one sequence of 599 rows 8.3 -> 7.4 us, 64 of 400 23.6 -> 22.9; 12/2 heads, 64 of
// 527 9.7 before and after).
template <int ROWB>
__device__ __forceinline__ bool beacon_fits(const DecodeParams& p) { return 2 * p.Hkv * ROWB <= kBeaconBytes; }
template <int ROWB>
__device__ __forceinline__ void request_beacon(const DecodeParams& p, int s, int lane, const char* lds_dst) {
  const int n = p.Hkv * ROWB;
  const int64_t at = (int64_t)s * n;
  for (int i0 = 0; i0 < 2 * n; i0 += 1024) {
    const int i = min(i0 + 16 * lane, 2 * n - 16);
    lds_dma16<false>((i >= n ? p.bv - n : p.bk) + at + i, lds_dst + i0);
  }
}
// What the holder of a sequence's last ticket does, as one wave, once every reader of the sequence's tables is done with
// them: the tables move on, the ticket counter returns to zero.
__device__ __forceinline__ void move_tables(const DecodeParams& p, const PairInfo& pi, int lane) {
  if (lane == 0) {
    // (past the L2: other words of the line are counted on by workgroups of other XCDs)
    __hip_atomic_store(p.tickets + pi.s * kTicketStride, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    p.nb_rw[pi.s] = pi.nb + (pi.evict_due ? 1 : 0);
    p.w_rw[pi.s] = pi.evict_due ? 0 : pi.w_att;
    if (p.budget && pi.nb + pi.w_att >= p.budget[pi.s]) p.live[pi.s] = 0;   // generation interrupted
  }
}
// Both, for a sequence that is not cut.
template <int ROWB>
__device__ __forceinline__ void finish_step(const DecodeParams& p, const PairInfo& pi, int lane, const char* beacon = nullptr) {
  if (pi.evict_due) {
    if (beacon != nullptr) store_beacon<ROWB, true>(p, pi, 0, p.Hkv, lane, 64, beacon, beacon + p.Hkv * ROWB);
    else store_beacon<ROWB, false>(p, pi, 0, p.Hkv, lane, 64);
  }
  move_tables(p, pi, lane);
}

// ---------------------------------------------------------------------------
// partial results of a sequence cut into chunks
// ---------------------------------------------------------------------------
// The chunks of a pair run on different XCDs, whose L2s do not see each other's dirty lines.  Partials
// therefore go past the caches in both directions (system scope: stores through to memory, loads from
// it) and no cache has to be written back or invalidated: an agent-scope release in their place took 50 us.
// A chunk's partial has its 128-byte lines to itself.
constexpr int kPartTail = 32;        // floats behind the o rows: [Gp] (maximum, denominator), padding

__device__ __forceinline__ float* chunk_partial(const DecodeParams& p, const PairInfo& pi, int D, int chunk) {
  return p.part + ((int64_t)(pi.s * p.Hkv + pi.kvh) * p.max_chunks + chunk) * (p.Gp * D + kPartTail);
}
__device__ __forceinline__ void store_part(float* a, float x) {
  __hip_atomic_store(reinterpret_cast<uint32_t*>(a), __float_as_uint(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void store_part2(float* a, float x, float y) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(a), (uint64_t)__float_as_uint(y) << 32 | __float_as_uint(x),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ uint64_t load_part2(const float* a) {
  return __hip_atomic_load(reinterpret_cast<const uint64_t*>(a), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Counts this workgroup at its pair (called by all of its threads, once it has stored its partial and done all
// its reads of the tables and the slab, or without a chunk).  True for the one that finds all others there: every
// partial of the pair is then written, and every wave of the pair's workgroups has read the tables.
__device__ __forceinline__ bool last_arrival(const DecodeParams& p, const PairInfo& pi, int* s_arrived) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wave's part of the partial is in memory
  __syncthreads();                                       // ... and everyone's
  int32_t* arrivals = p.arrivals + pi.s * p.arrival_stride + pi.kvh;
  if (threadIdx.x == 0) *s_arrived = __hip_atomic_fetch_add(arrivals, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(*s_arrived) != arrivals_due(pi.update, pi.nchunks, p.max_chunks) - 1) return false;
  if (threadIdx.x == 0) __hip_atomic_store(arrivals, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// The fold, in chunk order (so results do not depend on which workgroup it is).  A second launch for it cost
// 4.5 us and the gap between two dependent launches.  What bounds it is one round trip to memory, and what the compiler puts in front: offsets
// of 64 bits for all chunks, worked out before the first load and kept in vector lanes, with three loads and an exponential a chunk and lane and the
// beacon's round trip ahead of it took 1.9 us from the last arrival to the end of the launch, 1.15 now (one sequence of 1551 rows, 32/8 heads, a step that evicts
// 10.1 -> 8.7 us; 16 layers of 45 ragged sequences, 14/2 heads, d = 64, 169 -> 149).  A lane of each sixteen has the maximum and the denominator of one
// chunk, and its weight goes round by DPP.  behind_loads: called when the first chunks' loads are out.
template <int NT, int D, typename F>
__device__ __forceinline__ void merge_chunks(const DecodeParams& p, const PairInfo& pi, const F& behind_loads) {
  // sixteen chunks at a time, their loads in flight together (eight where the kernel would need more registers for it)
  constexpr int kBatch = NT > 256 ? 16 : 8;
  const char* part = reinterpret_cast<const char*>(chunk_partial(p, pi, D, 0));      // (scalar, with an offset per lane)
  const uint32_t step = (uint32_t)(p.Gp * D + kPartTail) * 4u;
  auto load = [&](uint32_t at) __attribute__((always_inline)) { return load_part2(reinterpret_cast<const float*>(part + at)); };
  float* outp = p.out + (int64_t)(pi.s * p.Hq + pi.kvh * p.g) * D;
  const int mine = threadIdx.x & (kBatch - 1);
#pragma clang loop unroll(disable)
  for (int i0 = 0; i0 < p.g * D; i0 += 2 * NT) {
    const int i = i0 + 2 * threadIdx.x;
    if (i >= p.g * D) continue;
    uint32_t ml = (uint32_t)(p.Gp * D + 2 * (i / D)) * 4u, at = 4u * i;
    float mx = kNegBig, lsum = 0.f, o0 = 0.f, o1 = 0.f;
#pragma clang loop unroll(disable)
    for (int n = pi.nchunks; n > 0; n -= kBatch) {       // chunks left
      const uint64_t mlv = load(ml + (uint32_t)min(mine, n - 1) * step);
      uint64_t ov[kBatch];
#pragma unroll
      for (int k0 = 0; k0 < kBatch; k0 += 4) {
        if (k0 < n) {                                    // (a branch of the whole wave; behind the last chunk it repeats, with a weight of zero)
#pragma unroll
          for (int k = k0; k < k0 + 4; ++k) ov[k] = load(at + (uint32_t)min(k, n - 1) * step);
        } else {
#pragma unroll
          for (int k = k0; k < k0 + 4; ++k) ov[k] = 0;
        }
      }
      if (i0 == 0 && n == pi.nchunks) behind_loads();
      const float m = mine < n ? __uint_as_float((uint32_t)mlv) : kNegBig;
      const float mn = fmaxf(mx, group_allreduce_max<kBatch>(m));
      const float keep = fast_exp2(mx - mn), a = mine < n ? fast_exp2(m - mn) : 0.f;
      mx = mn;
      lsum = lsum * keep + group_allreduce_sum<kBatch>(a * __uint_as_float((uint32_t)(mlv >> 32)));
      o0 *= keep; o1 *= keep;
      each_of<kBatch>([&](auto k) __attribute__((always_inline)) {
        const float ak = lane_of_row<k>(a);
        o0 = fmaf(__uint_as_float((uint32_t)ov[k]), ak, o0);
        o1 = fmaf(__uint_as_float((uint32_t)(ov[k] >> 32)), ak, o1);
      });
      ml += kBatch * step; at += kBatch * step;
      asm volatile("" : "+v"(ml), "+v"(at));             // (no addresses worked out for all passes in front of the first load)
    }
    *reinterpret_cast<float2*>(outp + i) = make_float2(o0 / lsum, o1 / lsum);
  }
}

// The end of a workgroup of a cut sequence, in one place of its kernel for those with and without rows (the first of them brings the code into the
// instruction cache).  beacon: the beacon rows of all heads in LDS, or null.
struct Closing { PairInfo pi; const char* beacon; };
template <int NT, int D, int ROWB>
__device__ __forceinline__ void close_pair(const Closing& end, int* s_arrived) {
  const PairInfo& pi = end.pi;
  const char* beacon = end.beacon;
  if (!last_arrival(arguments_again<kTableArguments>(), pi, s_arrived)) return;
  // The pair's ticket goes out behind the loads of the partials, whose answers the wave would otherwise wait for it with.  (Its place as
  // one of the lane's own: of what it takes for the wave's, the compiler makes a sum over lanes and looks at the answer at once.)
  int drawn = -1;
  {
    const DecodeParams p = arguments_again<kTableArguments>();
    merge_chunks<NT, D>(p, pi, [&]() __attribute__((always_inline)) {
      if (!pi.update || threadIdx.x != 0) return;
      int at = pi.s * kTicketStride;
      asm volatile("" : "+v"(at));
      drawn = __hip_atomic_fetch_add(p.tickets + at, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
  }
  if (!pi.update) return;
  const DecodeParams p = arguments_again<kTableArguments>();
  // everyone who reads this KV head's rows has arrived: its beacon row need not wait for the sequence's last ticket
  if (pi.evict_due) {
    if (beacon != nullptr) store_beacon<ROWB, true>(p, pi, pi.kvh, 1, threadIdx.x, NT, beacon + pi.kvh * ROWB, beacon + (p.Hkv + pi.kvh) * ROWB);
    else store_beacon<ROWB, false>(p, pi, pi.kvh, 1, threadIdx.x, NT);
  }
  if (threadIdx.x >= 64) return;
  if (__builtin_amdgcn_readfirstlane(drawn) == tickets_due(p.Hkv, 0, pi.nchunks, p.max_chunks) - 1)
    move_tables(p, pi, threadIdx.x);
}
// The end of a workgroup without rows, but for what it does for a pair that is cut: true where close_pair() is its end.  own: see tickets_due().
template <int ROWB>
__device__ __forceinline__ bool close_without_chunk(const PairInfo& pi, int own) {
  const CloseBy move = closing_move(pi.update, false, pi.nchunks);
  if (move != CloseBy::ticket) return move == CloseBy::arrival;
  __syncthreads();                 // every wave has read the tables
  if (threadIdx.x >= 64) return false;
  const DecodeParams p = arguments_again<kTableArguments>();
  int drawn = -1;
  if (threadIdx.x == 0) drawn = atomicAdd(p.tickets + pi.s * kTicketStride, 1);
  if (__builtin_amdgcn_readfirstlane(drawn) == tickets_due(p.Hkv, own, pi.nchunks, p.max_chunks) - 1)
    finish_step<ROWB>(p, pi, threadIdx.x);
  return false;
}

// Epilogue of the plain-ALU kernel: s_m/s_l/s_acc hold one (m, l, o) per wave in LDS; merge them in wave order
// and write the result or the chunk partial.  CHUNKS: the sequence may be cut into chunks.
template <int NW, int D, bool CHUNKS>
__device__ __forceinline__ void merge_waves_and_store(const DecodeParams& p, const PairInfo& pi,
                                                      const float* s_m, const float* s_l,
                                                      const float* s_acc, int ml_stride,
                                                      int acc_stride) {
  // ml_stride, acc_stride: floats between the entries of two waves in s_m / s_l and in s_acc
  const int nout = p.g * D;
  float* outp = p.out + (int64_t)(pi.s * p.Hq + pi.kvh * p.g) * D;
  // (NW * 64 threads: the block size read from the launch descriptor would be one more scalar-cache miss)
  for (int i = threadIdx.x; i < nout; i += NW * 64) {
    const int h = i / D, x = i - h * D;
    float mx = s_m[h];
#pragma unroll
    for (int wv = 1; wv < NW; ++wv) mx = fmaxf(mx, s_m[wv * ml_stride + h]);
    float lsum = 0.f, o = 0.f;
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
      const float a = fast_exp2(s_m[wv * ml_stride + h] - mx);
      lsum += s_l[wv * ml_stride + h] * a;
      o += s_acc[wv * acc_stride + h * D + x] * a;
    }
    if (!CHUNKS || pi.nchunks == 1) {
      __builtin_nontemporal_store(o / lsum, outp + i);   // streamed out: nothing left dirty in L2
    } else {
      float* po = chunk_partial(p, pi, D, pi.chunk);
      float* pml = po + p.Gp * D;
      store_part(po + i, o);
      if (x == 0) {
        store_part2(pml + 2 * h, mx, lsum);
      }
    }
  }
}

// The same merge, four output columns per thread (128-bit LDS reads and stores): fewer waves
// take part, which shortens this serial tail of the matrix-core kernel.
// DIVIDE: a correctly rounded quotient, for fp32 rows.
template <int NW, int D, int DOUT, int APITCH, bool CHUNKS, bool DIVIDE = false>
__device__ __forceinline__ void merge_waves_and_store4(const DecodeParams& p, const PairInfo& pi,
                                                       const float* s_m, const float* s_l,
                                                       const float* s_acc, int wave_stride, int col0) {
  constexpr int Q = D / 4;                       // column quads per head
  const int nitems = p.g * Q;
  float* outp = p.out + (int64_t)(pi.s * p.Hq + pi.kvh * p.g) * DOUT + col0;
  for (int i = threadIdx.x; i < nitems; i += NW * 64) {
    const int h = i / Q, x = (i - h * Q) * 4;
    // all reads first: the merge is one LDS round trip, not one per wave
    float mw[NW], lw[NW];
    f32x4_t ow[NW];
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
      mw[wv] = s_m[wv * wave_stride + h];
      lw[wv] = s_l[wv * wave_stride + h];
      ow[wv] = *reinterpret_cast<const f32x4_t*>(s_acc + wv * wave_stride + h * APITCH + x);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    float mx = mw[0];
#pragma unroll
    for (int wv = 1; wv < NW; ++wv) mx = fmaxf(mx, mw[wv]);
    float lsum = 0.f;
    f32x4_t o = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
      const float a = fast_exp2(mw[wv] - mx);
      lsum += lw[wv] * a;
      o += ow[wv] * a;
    }
    if (!CHUNKS || pi.nchunks == 1) {
      if constexpr (DIVIDE) o = f32x4_t{o[0] / lsum, o[1] / lsum, o[2] / lsum, o[3] / lsum};
      else o *= __builtin_amdgcn_rcpf(lsum);      // (one rounding error of the hardware reciprocal)
      __builtin_nontemporal_store(o, reinterpret_cast<f32x4_t*>(outp + h * DOUT + x));
    } else {
      float* po = chunk_partial(p, pi, D, pi.chunk);
      float* pml = po + p.Gp * D;
      store_part2(po + h * D + x, o[0], o[1]);
      store_part2(po + h * D + x + 2, o[2], o[3]);
      if (x == 0) {
        store_part2(pml + 2 * h, mx, lsum);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// bf16, d = 128 or 64: LDS-DMA tiles + MFMA
// ---------------------------------------------------------------------------
constexpr int kLdsWaves = 8;           // waves per workgroup
constexpr int kLdsWavesSplit = 12;     // ... of the two-workgroups-per-pair form on short caches (12 KB of LDS per wave)
constexpr int kSplitWaves12MaxCap = 1100;   // rows: beyond this eight waves are as fast or faster (measured)
constexpr int kTileRows = 32;          // rows per wave tile
constexpr int kLdsBytes = kLdsWaves * 2 * kTileRows * 256;   // d = 128: 128 KB (half of it for d = 64)
constexpr int kLdsBytesSplit = kLdsWavesSplit * 3 * kTileRows * 128;   // K tile + half a V tile per wave: 144 KB
constexpr int kLdsBytesMax = (kLdsBytesSplit > kLdsBytes ? kLdsBytesSplit : kLdsBytes) + kBeaconBytes;

typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

// K/V rows are read exactly once per launch: they are loaded with the non-temporal cache policy
// (the `nt` bit of the load instructions), which measured 5 % faster per step than the default
// policy at config 2.
constexpr int kStreamMinWorkgroups = 48;

template <bool STREAM> __device__ __forceinline__ uint4 load16(const char* p);
template <> __device__ __forceinline__ uint4 load16<false>(const char* p) {
  return *reinterpret_cast<const uint4*>(p);
}
__device__ __forceinline__ uint4 load16_stream(const char* p) {
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
  const u32x4_t r = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(r.x, r.y, r.z, r.w);
}

template <> __device__ __forceinline__ uint4 load16<true>(const char* p) { return load16_stream(p); }

// STREAM: 1 = load K and V with the non-temporal policy (large launches; small ones are
// latency-bound and about a microsecond faster with the default policy, 0); 2 = V only: with two
// workgroups per pair and long caches the K lines, which the partner reads a little later, are
// better kept cacheable.
// VS: workgroups per (sequence, KV head) pair.  With VS = 2 (batches of at most 128 pairs, which
// would leave half of the compute units idle) two workgroups serve a pair: both read all K rows
// and compute the same scores and weights, each reads one half of every V row and produces that
// half of the output columns - no partial results to merge.  The partner's workgroup index is
// larger by the number of pairs, which is the same XCD (same L2) when that number is a
// multiple of 8: the K rows then come from HBM once.
// NW: waves per workgroup, 8 or (two workgroups per pair, short caches: every wave then has one or
// two tiles, and twelve waves finish a sequence of up to 384 rows in one pass) 12.
// SHORT: every wave has at most two tiles (the caller's max_cap is at most 2 * NW * 32 rows, one
// chunk per pair, no dispatch order).  The code is then a straight line: query and appended row
// are requested first (their addresses do not need the tables), then the K part of the first
// tile, its V part, and the second tile's K and V parts into registers - everything in flight
// from the start, in the order it is needed - and every stage waits only for what it is about to
// read: scores and softmax of a tile run while its V rows are still on their way, so that behind
// the last byte only one value product is left.
// CHUNKS: the plan cuts sequences into chunks.  A kernel of its own: with the fold compiled into the kernel of
// whole sequences, 34 scalar registers of that spilled (200 pairs of 1000 rows: 20.6 us a step without, 21.2 with;
// 320 of 1200: 45.2, 46.6).
// True where close_pair() is still to come, with what it wants in `end`.
template <int STREAM, int D, int VS, int NW, bool SHORT, bool CHUNKS>
__device__ __forceinline__ bool decode_lds(const DecodeParams& p, Closing* end) {
  static_assert(!CHUNKS || (VS == 1 && !SHORT), "the straight-line form and the V halves have whole sequences");
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  constexpr bool KSTREAM = STREAM == 1, VSTREAM = STREAM >= 1;
  constexpr int DV = D / VS;               // V (and output) columns of this workgroup
  constexpr int VROWB = DV * 2;            // bytes of its part of a V row, = row pitch of the V tile in LDS
  constexpr int VUPR = VROWB / 16;
  constexpr int VRPI = 1024 / VROWB;
  constexpr int VNDMA = kTileRows / VRPI;
  constexpr int VTILEB = kTileRows * VROWB;
  constexpr int ROWB = D * 2;              // bytes of one row of one KV head: 256 or 128
  constexpr int UPR = ROWB / 16;           // 16-byte units per row: 16 or 8
  constexpr int RPI = 1024 / ROWB;         // rows one 1 KB LDS-DMA instruction brings: 4 or 8
  constexpr int NDMA = kTileRows / RPI;    // such instructions per K (or V) tile: 8 or 4
  constexpr int NI = D / 32;               // MFMAs (k = 32) along the head dimension: 4 or 2
  constexpr int NJ = DV / 16;              // 16-column blocks of the output held here: 8 or 4
  constexpr int TILEB = kTileRows * ROWB;  // one K (or V) tile: 8 or 4 KB
  constexpr int ARGS = CHUNKS ? kTableArguments : 0;      // where they lie
  TableEntries tables;
  if constexpr (CHUNKS) request_tables(p, (int)blockIdx.y, tables);
  touch_kernel_arguments<ARGS, !CHUNKS>();
  // grid: (KV head, slot, chunk from the last or V half), see decode_grid().  VS = 2: the slots are padded so that a pair's two
  // workgroups are 8k apart in dispatch order (workgroups go to the XCDs in turn).
  const int vhalf = VS == 1 ? 0 : (int)blockIdx.z;
  const int slot = (int)blockIdx.y, kvh0 = (int)blockIdx.x;
  if (VS != 1 && slot >= p.B) return false;
  // (the wave's number as a scalar: conditions on it become real branches, not lane masks)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r4 = lane / UPR, pos = lane & (UPR - 1);   // row within a 1 KB load, unit within the row
  const int r4v = lane / VUPR, posv = lane & (VUPR - 1);   // the same for this workgroup's part of V
  const int n = lane & 15, kb = lane >> 4;       // MFMA column / k-block of this lane
  char* wk = lds + wave * (TILEB + VTILEB);
  char* wv = wk + TILEB;

  // B operand of the score product: Q^T, column n = query head, k = head-dim index.
  // The loads are written out by hand so that the compiler does not count them: it cannot tell
  // the order in which they and the LDS-DMA loads complete, and would put a wait for ALL
  // outstanding loads - the next tile's among them - in front of the first use in every pass of
  // the tile loop.  They are older than any tile load the wave waits for.
  bf16x8_t qb[NI];
  auto request_query = [&](int s_) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      u32x4_t r;
      if constexpr (CHUNKS) {
        // (the columns behind the group's heads repeat the last one and are not looked at: shorter code than leaving their lanes out)
        const char* src = p.q + ((int64_t)(s_ * p.Hq + kvh0 * p.g + min(n, p.g - 1)) * D + 32 * i + 8 * kb) * 2;
        asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(r) : "v"(src) : "memory");
      } else {
        r = u32x4_t{0u, 0u, 0u, 0u};
        if (n < p.g) {
          const char* src = p.q + ((int64_t)(s_ * p.Hq + kvh0 * p.g + n) * D + 32 * i + 8 * kb) * 2;
          asm volatile("global_load_dwordx4 %0, %1, off" : "+v"(r) : "v"(src) : "memory");
        }
      }
      qb[i] = __builtin_bit_cast(bf16x8_t, r);
    }
  };
  // Fused append: lanes 0..UPR-1 carry the new K row, the next VUPR lanes this workgroup's part of
  // the new V row (16 bytes each); loaded by hand like the query, for the same reason.  The
  // instruction is issued whether or not a row is appended (the other lanes, and all lanes of a
  // plain attention call, read the head of the query tensor instead): the waits below count it.
  u32x4_t newrow_v;
  auto request_new_row = [&](int s_) {
    const char* src = p.q + ((lane & 7) << 4);      // (128 bytes: inside the smallest query tensor)
    if (p.new_k != nullptr && lane < UPR + VUPR) {
      if constexpr (VS == 1)
        src = (lane < UPR ? p.new_k : p.new_v) + (int64_t)(s_ * p.Hkv + kvh0) * ROWB + ((lane & (UPR - 1)) << 4);
      else
        src = lane < UPR
            ? p.new_k + (int64_t)(s_ * p.Hkv + kvh0) * ROWB + (lane << 4)
            : p.new_v + (int64_t)(s_ * p.Hkv + kvh0) * ROWB + vhalf * VROWB + ((lane - UPR) << 4);
    }
    asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(newrow_v) : "v"(src) : "memory");
  };
  // HBM -> LDS: the K part of a tile (NDMA instructions, each RPI whole rows = 1 KB), then this
  // workgroup's V part, 16-byte units XOR-swizzled by the row.  Addresses are a base in scalar
  // registers plus a 32-bit offset per lane.  CLAMP: rows beyond `last_row` are read from
  // `last_row` instead (they are masked later; the loads stay inside the resident rows); without
  // it the tile's rows must all exist, and the lane offsets do not depend on the tile.
  const uint32_t wk_lds = lds_address(lds) + wave * (TILEB + VTILEB), wv_lds = wk_lds + TILEB;
  auto request_tile_dma = [&](auto clamp, uint64_t kb_, uint64_t vb_, int trow0, int last_row) {
    constexpr bool CLAMP = decltype(clamp)::value;
#pragma unroll
    for (int j = 0; j < NDMA; ++j) {
      const int row = RPI * j + r4;
      const uint32_t unit = (uint32_t)(pos ^ tile_swz<D>(row)) << 4;
      if constexpr (CLAMP)
        lds_dma16_s<KSTREAM>((uint32_t)min(trow0 + row, last_row) * ROWB + unit, kb_, wk_lds + j * 1024);
      else
        lds_dma16_s<KSTREAM>((uint32_t)r4 * ROWB + unit, kb_ + (uint64_t)(trow0 + RPI * j) * ROWB, wk_lds + j * 1024);
    }
#pragma unroll
    for (int j = 0; j < VNDMA; ++j) {
      const int vrow = VRPI * j + r4v;
      const uint32_t unit = (uint32_t)(posv ^ tile_swz<DV>(vrow)) << 4;
      if constexpr (CLAMP)
        lds_dma16_s<VSTREAM>((uint32_t)min(trow0 + vrow, last_row) * ROWB + unit, vb_, wv_lds + j * 1024);
      else
        lds_dma16_s<VSTREAM>((uint32_t)r4v * ROWB + unit, vb_ + (uint64_t)(trow0 + VRPI * j) * ROWB, wv_lds + j * 1024);
    }
  };
  // (not initialised, and written by request_tile_regs only: the loads are invisible to the
  // compiler, so a register-to-register copy between a load and its wait would copy what is not
  // there yet; the check of the generated code looks for exactly that)
  u32x4_t kreg[NDMA], vreg[VNDMA];
  auto request_tile_regs = [&](uint64_t kb_, uint64_t vb_, int trow0, int last_row) {
#pragma unroll
    for (int j = 0; j < NDMA; ++j)
      load16_uncounted_s<KSTREAM>(kreg[j], (uint32_t)min(trow0 + RPI * j + r4, last_row) * ROWB + (pos << 4), kb_);
#pragma unroll
    for (int j = 0; j < VNDMA; ++j)
      load16_uncounted_s<VSTREAM>(vreg[j], (uint32_t)min(trow0 + VRPI * j + r4v, last_row) * ROWB + (posv << 4), vb_);
  };
  if constexpr (SHORT || CHUNKS) {      // no dispatch order, the sequence is the slot: nothing here needs the tables
    request_query(slot);
    request_new_row(slot);
  }
  // Prompt rows never change and are always resident.  When the caller has promised the slab
  // geometry (every sequence: P = spec_P, cap = spec_cap, base = index * spec_cap), a wave whose
  // first tile lies inside the prompt requests it before the tables are back; whatever the
  // tables say afterwards decides: if the geometry is another, the tile is requested again.
  // (Requesting the tiles behind the prompt early as well, under a promised number of resident
  // rows, was measured: with everything asked for at once the step is 2 % slower.)
  bool early_tile = false;
  auto request_early_tiles = [&]() {
    if (p.spec_P > 0 && p.order == nullptr && p.max_chunks == 1 && (wave + 1) * kTileRows <= p.spec_P) {
      const int64_t off_ = ((int64_t)slot * p.spec_cap * p.Hkv + (int64_t)kvh0 * p.spec_cap) * ROWB;
      request_tile_dma(std::false_type{}, (uint64_t)(p.k_slab + off_), (uint64_t)(p.v_slab + off_ + vhalf * VROWB),
                       wave * kTileRows, 0);
      early_tile = true;
    }
  };
  const PairInfo pi = VS == 1 && !SHORT ? pair_info(p, slot, kvh0, CHUNKS ? p.max_chunks - 1 - (int)blockIdx.z : 0, NoEarlyWork(),
                                                            CHUNKS ? &tables : nullptr)
                                        : pair_info(p, slot, kvh0, 0, request_early_tiles);
  // Tiles wave, wave + NW, ... of the chunk belong to this wave.
  const int ntiles = (pi.row_end - pi.row0 + kTileRows - 1) / kTileRows;
  bool nothing_to_do = !pi.live;
  if constexpr (SHORT) {
    // more rows than the caller's max_cap allows: no wave of the sequence goes on (none takes
    // a ticket, so its tables and the counters stay as they were)
    if (ntiles > 2 * NW) {
      if (pi.kvh == 0 && vhalf == 0 && tid == 0) atomicOr(p.err, BC_ERRBIT_STATE);
      nothing_to_do = true;
    }
  }
  auto query_landed = [&]() {
#pragma unroll
    for (int i = 0; i < NI; ++i) landed(qb[i]);
    landed(newrow_v);
  };
  if (nothing_to_do) {
    wait_vmcnt<0>();
    if constexpr (CHUNKS) {
      query_landed();          // (what is asked for before it is known to be wanted keeps its registers until it is there)
      *end = Closing{pi, nullptr};
      return close_without_chunk<ROWB>(pi, NW);
    }
    return false;
  }
  // rows the tile loads may touch: the resident rows that are already in the slab
  const int last_slab_row = max((pi.new_row >= 0 ? pi.new_row : pi.L) - 1, 0);
  if (early_tile && (pi.P != p.spec_P || pi.cap != p.spec_cap || pi.base != (int64_t)pi.s * p.spec_cap))
    early_tile = false;      // the promise does not hold here: the tile is requested again below

  const HalfSelectors sel = half_selectors();
  const int64_t stream_off = (pi.base * p.Hkv + (int64_t)pi.kvh * pi.cap) * ROWB;
  const char* kbase = p.k_slab + stream_off;
  const char* vbase = p.v_slab + stream_off + vhalf * VROWB;
  const uint64_t kbase_s = (uint64_t)kbase, vbase_s = (uint64_t)vbase;      // (uniform: scalar registers)
  if constexpr (!SHORT && !CHUNKS) {           // the sequence may come from the dispatch order: after the tables
    request_query(pi.s);
    request_new_row(pi.s);
  }

  f32x4_t O[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) O[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = kNegBig, l_run = 0.f;

  // A wave's first tile goes from HBM to LDS by LDS-DMA; the second is requested at the same
  // time into registers, so both are in flight from the start.  Afterwards: copy the register
  // tile to LDS, request the next tile into the freed registers, compute - one tile always in
  // flight behind the one in use.
  auto k_regs_to_lds = [&]() {
#pragma unroll
    for (int j = 0; j < NDMA; ++j) {
      const int row = RPI * j + r4;
      *reinterpret_cast<u32x4_t*>(wk + row * ROWB + ((pos ^ tile_swz<D>(row)) << 4)) = kreg[j];
    }
  };
  auto v_regs_to_lds = [&]() {
#pragma unroll
    for (int j = 0; j < VNDMA; ++j) {
      const int vrow = VRPI * j + r4v;
      *reinterpret_cast<u32x4_t*>(wv + vrow * VROWB + ((posv ^ tile_swz<DV>(vrow)) << 4)) = vreg[j];
    }
  };
  auto k_regs_landed = [&]() {
#pragma unroll
    for (int j = 0; j < NDMA; ++j) landed(kreg[j]);
  };
  auto v_regs_landed = [&]() {
#pragma unroll
    for (int j = 0; j < VNDMA; ++j) landed(vreg[j]);
  };
  if (wave < ntiles && !early_tile) {
    const int trow0 = pi.row0 + wave * kTileRows;
    if (trow0 + kTileRows <= last_slab_row + 1) request_tile_dma(std::false_type{}, kbase_s, vbase_s, trow0, 0);
    else request_tile_dma(std::true_type{}, kbase_s, vbase_s, trow0, last_slab_row);
  }
  // (the last wave has the fewest tiles; its loads have landed by the barrier in front of the merge)
  char* beacon = lds + NW * (TILEB + VTILEB);
  if (pi.evict_due && wave == NW - 1) {
    const DecodeParams again = arguments_again<ARGS>();
    if (beacon_fits<ROWB>(again)) request_beacon<ROWB>(again, pi.s, lane, beacon);
  }

  // Fused step, whole sequence: every wave with rows takes a ticket as soon as its last load from the
  // slab has landed (the tables were read at the start), a workgroup without rows takes one; whoever
  // draws the last one may write the beacon row and update the tables.  The answer is only looked at
  // after the wave merge, so the atomic's round trip (about a microsecond) hides behind the remaining
  // compute.  (Of a sequence cut into chunks the workgroup that folds a pair's takes one for the pair: a ticket for
  // every wave of every chunk were 1472 atomics on one counter for 3000 rows of 8 KV heads, 23.7 us a step instead of 12.2.)
  int ticket = -1;
  auto take_ticket = [&]() {
    if (pi.update && lane == 0 && (!CHUNKS || pi.nchunks == 1)) {
      const int one_ = 1;
      asm volatile("global_atomic_add %0, %1, %2, off sc0"
                   : "=v"(ticket) : "v"(p.tickets + pi.s * kTicketStride), "v"(one_) : "memory");
    }
  };
  // The appended row is not in the slab yet: place it in the tile (K part before the scores, V
  // part before the value product), clear the V rows behind it, store it for later steps (unless
  // this step's eviction drops it at once).  Only the sequence's last tile can hold it.
  auto patch_k_row = [&](int trow0) {
    const int ra = pi.new_row - trow0;
    if (ra >= 0 && ra < kTileRows && lane < UPR)
      *reinterpret_cast<u32x4_t*>(wk + ra * ROWB + ((lane ^ tile_swz<D>(ra)) << 4)) = newrow_v;
  };
  auto patch_v_row_and_store = [&](int trow0) {
    const int ra = pi.new_row - trow0;
    if (ra < 0 || ra >= kTileRows) return;
    int lane_ = lane;
    asm volatile("" : "+v"(lane_));       // addresses worked out here and not kept from before the tile loop (cut
                                          // sequences, 48 pairs of 1100 rows: 19.9 us a step with, 14.1 without)
    if (lane >= UPR && lane < UPR + VUPR) {
      const int u = lane_ - UPR;
      *reinterpret_cast<u32x4_t*>(wv + ra * VROWB + ((u ^ tile_swz<DV>(ra)) << 4)) = newrow_v;
      if (pi.store_new_row)
        *reinterpret_cast<u32x4_t*>(const_cast<char*>(vbase) + (int64_t)pi.new_row * ROWB + (u << 4)) = newrow_v;
    } else if (lane < UPR) {
      if (pi.store_new_row && vhalf == 0)
        *reinterpret_cast<u32x4_t*>(const_cast<char*>(kbase) + (int64_t)pi.new_row * ROWB + (lane_ << 4)) = newrow_v;
    }
    for (int rr = ra + 1 + r4v; rr < kTileRows; rr += VRPI)
      *reinterpret_cast<uint4*>(wv + rr * VROWB + (posv << 4)) = make_uint4(0u, 0u, 0u, 0u);
  };

  // ---- scores, transposed: S^T[key][head] = K . Q^T.  Row m of sub-tile t is key
  //      8*(m/4) + 4*t + m%4, so that a lane ends up with 8 consecutive keys of one head:
  //      lane (n, kb) holds head n, keys trow0 + 8*kb + e, e = 4*t + r.
  // ---- softmax: the scores stay unscaled; the softmax scale (>= 0) enters through one fused
  //      multiply-add per key, p = 2^(s*qs - m).  Only a sequence's last tile has rows beyond its
  //      end; the tests for them sit behind a branch that is uniform over the wave.  The weights
  //      leave as p = hi + lo with both parts bf16: the p.V product keeps ~16 bits of p.
  bf16x8_t phi, plo;
  auto scores_and_softmax = [&](int trow0, bool first) {
    f32x4_t S[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      S[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      const int row = ((n >> 2) << 3) + 4 * t + (n & 3);
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int u = 4 * i + kb;
        const bf16x8_t a =
            *reinterpret_cast<const bf16x8_t*>(wk + row * ROWB + ((u ^ tile_swz<D>(row)) << 4));
        S[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qb[i], S[t], 0, 0, 0);
      }
    }
    const bool partial = trow0 + kTileRows > pi.row_end;
    const int nvalid = pi.row_end - trow0 - 8 * kb;        // keys e < nvalid of this lane exist
    float sv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) sv[e] = S[e >> 2][e & 3];
    if (partial) {
#pragma unroll
      for (int e = 0; e < 8; ++e) sv[e] = e < nvalid ? sv[e] : kNegBig;
    }
    float tmax = fmaxf(fmaxf(fmaxf(fmaxf(sv[0], sv[1]), sv[2]), fmaxf(fmaxf(sv[3], sv[4]), sv[5])),
                       fmaxf(sv[6], sv[7]));
    tmax = rows_allreduce_max(tmax);
    const float m_new = fmaxf(m_run, tmax * p.qscale);
    float pe[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) pe[e] = fast_exp2(fmaf(sv[e], p.qscale, -m_new));
    if (partial) {      // (with a scale of zero the fused form gives 1 for the missing keys, not 0)
#pragma unroll
      for (int e = 0; e < 8; ++e) pe[e] = e < nvalid ? pe[e] : 0.f;
    }
    const float psum = ((pe[0] + pe[1]) + (pe[2] + pe[3])) + ((pe[4] + pe[5]) + (pe[6] + pe[7]));
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const uint32_t hp = pack2_bf16(pe[e], pe[e + 1]);
      hi[e >> 1] = hp;
      lo[e >> 1] = pack2_bf16(minus_half(pe[e], hp, sel.low), minus_half(pe[e + 1], hp, sel.high));
    }
    // a wave's first tile finds empty accumulators: nothing to rescale
    if (!first) {
      const float alpha = fast_exp2(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int j = 0; j < NJ; ++j) O[j] *= alpha;
    }
    m_run = m_new;
    l_run += psum;
    phi = __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
    plo = __builtin_bit_cast(bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
  };
  // ---- O^T[dcol][head] += V^T . P^T ; V^T comes from the transposing LDS read: lane r of a
  //      16-lane block points at 4 consecutive dcols of key 8*kb + r/4 (+4 for the 2nd read)
  auto value_product = [&]() {
    const int r = lane & 15;
    const int key0 = 8 * kb + (r >> 2);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int u = 2 * j + ((r & 3) >> 1);
      const int sub = (r & 1) << 3;
      const int rowa = key0, rowb = key0 + 4;
      const s16x4_t a0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_s16x4_t*)(wv + rowa * VROWB + ((u ^ tile_swz<DV>(rowa)) << 4) + sub));
      const s16x4_t a1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_s16x4_t*)(wv + rowb * VROWB + ((u ^ tile_swz<DV>(rowb)) << 4) + sub));
      typedef __attribute__((ext_vector_type(8))) short s16x8_t;
      const s16x8_t a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
      const bf16x8_t av = __builtin_bit_cast(bf16x8_t, a);
      O[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, phi, O[j], 0, 0, 0);
      O[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, plo, O[j], 0, 0, 0);
    }
  };

  if constexpr (SHORT) {
    // Loads in flight, oldest first: query (NI), appended row (1), K of the first tile (NDMA),
    // its V part (VNDMA) and, with a second tile, its K (NDMA) and V (VNDMA) into registers.
    const int trowA = wave * kTileRows, trowB = trowA + NW * kTileRows;
    if (wave >= ntiles) {
      wait_vmcnt<0>();          // query and row loads, before their registers are reused
      query_landed();
      take_ticket();
    } else if (wave + NW < ntiles) {
      request_tile_regs(kbase_s, vbase_s, trowB, last_slab_row);
      wait_vmcnt<VNDMA + NDMA + VNDMA>();          // K of the first tile is in LDS
      query_landed();
      scores_and_softmax(trowA, true);
      wait_vmcnt<NDMA + VNDMA>();                  // ... and its V part
      value_product();
      wait_vmcnt<VNDMA>();                         // K of the second tile is in registers
      k_regs_landed();
      k_regs_to_lds();
      patch_k_row(trowB);
      scores_and_softmax(trowB, false);
      wait_vmcnt<0>();
      v_regs_landed();
      v_regs_to_lds();
      patch_v_row_and_store(trowB);
      take_ticket();
      value_product();
    } else {
      wait_vmcnt<VNDMA>();
      query_landed();
      patch_k_row(trowA);
      scores_and_softmax(trowA, true);
      wait_vmcnt<0>();
      patch_v_row_and_store(trowA);
      take_ticket();
      value_product();
    }
  } else {
    if (wave >= ntiles) {
      wait_vmcnt<0>();          // the query loads, before their registers are reused
      query_landed();
      if (CHUNKS && pi.nchunks == 1) {         // (those of a cut sequence take none)
        // One more round trip: where the query was asked for in front of the tables, the tickets of these waves came together with those of the
        // workgroups without rows, and the waves with rows queued up behind them on the counter (steps of one sequence under a capacity of 1100 rows, with
        // the query behind the tables, in front of them, and so: 130 rows, 32/8 heads, d = 64, 6.0, 6.9, 6.0 us; 100 rows, 64/16 heads, d = 128,
        // 8.0, 9.1, 8.2; 60 rows, 32/8 heads, d = 128, 7.0, 6.25, 6.35; 1551 rows, cut, 9.3, 9.2, 9.3).
        request_new_row(slot);
        wait_vmcnt<0>();
        landed(newrow_v);
      }
      take_ticket();
    } else {
      for (int tile = wave;; tile += NW) {
        const int trow0 = pi.row0 + tile * kTileRows;
        if (tile + NW < ntiles) {
          // the next tile of this wave goes to registers while this one is in use; the tile in
          // use has landed once at most those loads are pending
          request_tile_regs(kbase_s, vbase_s, trow0 + NW * kTileRows, last_slab_row);
          wait_vmcnt<NDMA + VNDMA>();
          query_landed();
          scores_and_softmax(trow0, tile == wave);
          value_product();
          wait_vmcnt<0>();
          k_regs_landed();
          v_regs_landed();
          k_regs_to_lds();
          v_regs_to_lds();
        } else {
          // this wave's last tile: nothing between here and the end of the kernel waits for
          // memory, so the ticket's answer can stay out
          wait_vmcnt<0>();
          query_landed();
          patch_k_row(trow0);
          patch_v_row_and_store(trow0);
          take_ticket();
          scores_and_softmax(trow0, tile == wave);
          value_product();
          break;
        }
      }
    }
  }

  // denominators: sum the four k-blocks of each head
  l_run = rows_allreduce_sum(l_run);

  // ---- merge the waves through LDS.  Every wave leaves its (m, l, o) at the start of its own
  // tile region, which nobody else touches, as soon as it is done: one barrier, and the early
  // waves' writes do not wait for the late ones.
  // (rows of DV floats would all start on the same LDS bank: a pitch of DV + 4 floats spreads the
  // 128-bit writes of the up to eight heads over the banks)
  constexpr int APITCH = DV + 4;
  constexpr int WSTRIDE = (TILEB + VTILEB) / 4;                   // floats between two waves' regions
  static_assert((8 * APITCH + 16 + 1) * 4 <= TILEB + VTILEB, "the partial fits the wave's region");
  float* s_acc = reinterpret_cast<float*>(lds);                    // wave w: [8][APITCH] at w * WSTRIDE
  float* s_m = s_acc + 8 * APITCH;                                 //         [8] behind it
  float* s_l = s_m + 8;
  if (n < p.g) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      *reinterpret_cast<f32x4_t*>(s_acc + wave * WSTRIDE + n * APITCH + 16 * j + 4 * kb) = O[j];
    if (kb == 0) { s_m[wave * WSTRIDE + n] = m_run; s_l[wave * WSTRIDE + n] = l_run; }
  }
  __syncthreads();
  merge_waves_and_store4<NW, DV, D, APITCH, CHUNKS>(p, pi, s_m, s_l, s_acc, WSTRIDE, vhalf * DV);
  if constexpr (CHUNKS) {
    if (pi.nchunks > 1) {
      *end = Closing{pi, beacon_fits<ROWB>(arguments_again<ARGS>()) ? beacon : nullptr};
      return true;
    }
  }

  // ---- the wave that drew the sequence's last ticket writes the beacon row and updates the tables
  if (!pi.update) return false;
  wait_vmcnt<0>();     // the ticket has arrived
  landed(ticket);
  if (__builtin_amdgcn_readfirstlane(ticket) != tickets_due(p.Hkv, VS * NW, 1, CHUNKS ? p.max_chunks : 1) - 1) return false;
  finish_step<ROWB>(p, pi, lane, beacon_fits<ROWB>(p) ? beacon : nullptr);
  return false;
}

template <int STREAM, int D, int VS, int NW, bool SHORT = false>
__global__ __launch_bounds__(NW * 64) void decode_lds_kernel(DecodeParams p) {
  decode_lds<STREAM, D, VS, NW, SHORT, false>(p, nullptr);
}
template <int STREAM, int D, int NW>
__global__ __launch_bounds__(NW * 64) void decode_lds_cut_kernel(BC_TABLE_ARGUMENTS, DecodeParams p) {
  p.P = tP; p.nb = tnb; p.w = tw; p.cap = tcap; p.c = tc; p.base = tbase;
  p.order = nullptr;            // (see follows_order())
  Closing end;
  if (!decode_lds<STREAM, D, 1, NW, false, true>(p, &end)) return;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  close_pair<NW * 64, D, D * 2>(end, reinterpret_cast<int*>(lds));
}

// ---------------------------------------------------------------------------
// rows in registers: fp32, and bf16 where the plan asks for it
// ---------------------------------------------------------------------------
constexpr int kValuWaves = 4;

// fp32 rows on the fp32 matrix instructions (products and sums in 32 bits).  A wave's tile is 16 rows (d = 128) or 32
// (d = 64), 8 KB of K and of V, from HBM into registers:
//  * S^T[row][head] = K.Q^T in steps of four head-dim indices, one for each 16-lane row of the wave.  Which four does
//    not matter as long as both operands agree: lane (m, b) takes row m, elements 16*i + 4*b .. +3, and the c-th of
//    each four form a step.  K comes in as whole 256-byte pieces of four rows and goes through LDS into that order (loaded
//    in it, neighbouring lanes are different rows and the load path serves 16 bytes a clock: 64 rows 1.75 us instead of 1.44).
//  * A lane ends with rows 4*b + e of one head, which is the operand of O^T[column][head] += V^T.P^T when step e takes
//    these rows; lane (m, b) takes columns 64*j + 4*m .. +3 of row 4*b + e as they are loaded, and the c-th of each four
//    form a block of 16 result columns.  The weights never leave their lane.
// Half or more of the 16 head columns are padding (groups have up to eight heads); 64 rows of d = 128 on four waves are
// 0.87 us of matrix issue all the same.
// What bounds it: launch gap, tables, first bytes and the merge for short sequences (50 rows: 5.0 to 7.7 us a step, 7.5 to
// 16.4 on FMA instructions with sums over lanes, the form before), 45 GB/s a compute unit for long ones of few pairs, HBM for
// large batches (12/2 heads, d = 128: 120 sequences of 760 rows 60.1 -> 33.7 us; 16/2 heads, 64 of 1500 rows 110 -> 38.4; 8/1
// heads, 4 of 508 rows 17.5 -> 10.2).  Eight waves a workgroup: no difference, the load path is the same one.
template <int D, int G, bool CHUNKS>
__device__ __forceinline__ bool decode_f32_rows(const DecodeParams& p, Closing* end) {
  constexpr int RB = D * 4;
  constexpr int SUB = 128 / D, ROWS = 16 * SUB;    // 16-row blocks of a tile, its rows
  constexpr int KI = D / 16, VJ = D / 64;          // 16-byte units per lane: of a K block's operand, of a row
  constexpr int NW = kValuWaves;
  typedef __attribute__((ext_vector_type(4))) float row16_t;

  TableEntries tables;
  request_tables(p, (int)blockIdx.y, tables);
  touch_kernel_arguments<kTableArguments>();
  constexpr int APITCH = D + 4, WSTRIDE = G * APITCH + 2 * G + (2 * G) % 4;      // of the merge at the end, in floats
  constexpr int LDS = NW * (16 * SUB * RB > 4 * WSTRIDE ? 16 * SUB * RB : 4 * WSTRIDE);
  __shared__ __attribute__((aligned(1024))) char tiles[LDS];
  const PairInfo pi = pair_info(p, (int)blockIdx.y, (int)blockIdx.x, CHUNKS ? p.max_chunks - 1 - (int)blockIdx.z : 0,
                                NoEarlyWork(), &tables);
  if (!pi.live) {
    if constexpr (CHUNKS) {
      *end = Closing{pi, nullptr};
      return close_without_chunk<RB>(pi, NW);
    }
    return false;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, kb = lane >> 4;
  const int ntiles = (pi.row_end - pi.row0 + ROWS - 1) / ROWS;
  const int64_t stream_off = (pi.base * p.Hkv + (int64_t)pi.kvh * pi.cap) * RB;
  const char* kbase = p.k_slab + stream_off;
  const char* vbase = p.v_slab + stream_off;
  // Fused step: the appended row (always the sequence's last) is not in the slab yet and comes from the caller's
  // tensors; rows behind the chunk's end repeat its last one (masked).
  const int64_t new_off = (int64_t)(pi.s * p.Hkv + pi.kvh) * RB;
  auto row_of = [&](const char* base, const char* appended, int r) {
    r = min(r, pi.row_end - 1);
    return r == pi.new_row ? appended + new_off : base + (int64_t)r * RB;
  };

  // lane (n, kb) brings 16 bytes of rows 4*kb + e: 256 consecutive bytes of four rows an instruction
  row16_t kk[2][SUB][4][VJ], vv[2][SUB][4][VJ];
  auto load = [&](int stage, int tile) __attribute__((always_inline)) {
    const int r0 = pi.row0 + tile * ROWS + 4 * kb;
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const char* kr = row_of(kbase, p.new_k, r0 + 16 * u + e) + 16 * n;
#pragma unroll
        for (int j = 0; j < VJ; ++j)
          kk[stage][u][e][j] = __builtin_nontemporal_load(reinterpret_cast<const row16_t*>(kr + 256 * j));
      }
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const char* vr = row_of(vbase, p.new_v, r0 + 16 * u + e) + 16 * n;
#pragma unroll
        for (int j = 0; j < VJ; ++j)
          vv[stage][u][e][j] = __builtin_nontemporal_load(reinterpret_cast<const row16_t*>(vr + 256 * j));
      }
  };
  // K goes through the wave's part of LDS into operand order, 16-byte unit x of row y at unit x ^ y of each 256 bytes: neither
  // the writes (16 units of a row) nor the reads (one unit of 16 rows) meet in a bank.
  char* wk = tiles + wave * (16 * SUB * RB);
  const int ksrc = n * RB + ((kb ^ n) << 4);      // operand i: ^ 64 * (i % 4), + 256 * (i / 4)
  auto k_to_lds = [&](int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < VJ; ++j)
          *reinterpret_cast<row16_t*>(wk + (16 * u + 4 * kb + e) * RB + 256 * j + ((n ^ (4 * kb + e)) << 4)) = kk[stage][u][e][j];
  };

  // Q^T: column n = query head, the steps' elements as for K (the columns behind the group repeat its last head and are
  // not looked at)
  row16_t q[KI];
  const char* qrow = p.q + (int64_t)(pi.s * p.Hq + pi.kvh * p.g + min(n, p.g - 1)) * RB + 16 * kb;
#pragma unroll
  for (int i = 0; i < KI; ++i) q[i] = *reinterpret_cast<const row16_t*>(qrow + 64 * i);

  f32x4_t O[4 * VJ];
#pragma unroll
  for (int j = 0; j < 4 * VJ; ++j) O[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = kNegBig, l_run = 0.f;
  auto work = [&](int stage, int tile, bool last) __attribute__((always_inline)) {
    const int r0 = pi.row0 + tile * ROWS;
    float s[SUB][4];
    float tmax = kNegBig;
    k_to_lds(stage);
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
      // Eight sums side by side, of 8 (d = 64) or 16 products, then a tree.  (As two sums, and all rows of a wave in one sum below, results were
      // 1.2 to 2 times as far from 64 bits as the FMA form's, which sums four products and then over lanes.  Relative error of FMA, two sums, as
      // here, 1e-7: 64 sequences, d = 64, 40 rows 1.3, 1.9, 1.3, 120 rows 1.5, 2.0, 1.6, 600 rows with scores twice as wide 2.7, 4.4, 2.7; d = 128 1.3, 2.1, 1.4,
      // then 1.5, 2.6, 1.6 and 2.6, 4.9, 2.9; 200 of 1500 rows 2.4, 4.3, 2.0; 1.01 of FMA's on the average of what was measured.  It costs 1.2 % of a
      // step; sums of eight products at d = 128 too, 0.99, spill a register.)
      f32x4_t score[8];
#pragma unroll
      for (int i = 0; i < KI; ++i) {
        const row16_t k = *reinterpret_cast<const row16_t*>(wk + 16 * u * RB + (ksrc ^ (64 * (i & 3))) + 256 * (i >> 2));
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          f32x4_t& sum = score[4 * (i & 1) + c];
          sum = __builtin_amdgcn_mfma_f32_16x16x4f32(k[c], q[i][c], i < 2 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : sum, 0, 0, 0);
        }
      }
      score[0] = ((score[0] + score[1]) + (score[2] + score[3])) + ((score[4] + score[5]) + (score[6] + score[7]));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool there = r0 + 16 * u + 4 * kb + e < pi.row_end;
        s[u][e] = there ? score[0][e] : kNegBig;
        tmax = fmaxf(tmax, s[u][e]);
      }
    }
    tmax = rows_allreduce_max(tmax);
    const float m_new = fmaxf(m_run, tmax * p.qscale);
    const float alpha = fast_exp2(m_run - m_new);
    m_run = m_new;
    float psum = 0.f;
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool there = r0 + 16 * u + 4 * kb + e < pi.row_end;
        s[u][e] = there ? fast_exp2(fmaf(s[u][e], p.qscale, -m_new)) : 0.f;
        psum += s[u][e];
      }
    l_run = l_run * alpha + psum;
    // the appended row (the last of the sequence's last tile) outlives the step: stored for later ones (no reader
    // touches the slab there in this launch)
    if (last && pi.store_new_row && r0 + ROWS > pi.new_row) {
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (r0 + 16 * u + 4 * kb + e == pi.new_row)
#pragma unroll
            for (int j = 0; j < VJ; ++j) {
              const int64_t at = (int64_t)pi.new_row * RB + 256 * j + 16 * n;
              *reinterpret_cast<row16_t*>(const_cast<char*>(kbase) + at) = kk[stage][u][e][j];
              *reinterpret_cast<row16_t*>(const_cast<char*>(vbase) + at) = vv[stage][u][e][j];
            }
      }
    }
    // sixteen rows by themselves, then to the rest
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
      f32x4_t T[4 * VJ];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < VJ; ++j)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            f32x4_t& sum = T[4 * j + c];
            sum = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[stage][u][e][j][c], s[u][e], e == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : sum, 0, 0, 0);
          }
#pragma unroll
      for (int j = 0; j < 4 * VJ; ++j) O[j] = u == 0 ? O[j] * alpha + T[j] : O[j] + T[j];
    }
  };
  // The next tile's loads go out one after every other matrix instruction of the scores: all at once they keep the wave
  // from its work until the memory pipeline has accepted them.
  auto spread_loads = []() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Tiles wave, wave + NW, ... of the chunk are this wave's; one is on its way while another is worked on.  (Written out
  // so that each place knows which loads are out: behind a join the compiler would wait for all of them.)
  int tile = wave, mine = (ntiles - wave + NW - 1) / NW;
  if (mine > 0) {
    load(0, tile);
    for (; mine > 2; mine -= 2, tile += 2 * NW) {
      load(1, tile + NW);
      work(0, tile, false);
      spread_loads();
      load(0, tile + 2 * NW);
      work(1, tile + NW, false);
      spread_loads();
    }
    if (mine == 2) {
      load(1, tile + NW);
      work(0, tile, false);
      spread_loads();
      work(1, tile + NW, true);
    } else {
      work(0, tile, true);
    }
  }
  // Whole sequence: every wave takes a ticket when its reads of the slab are done, and looks at the answer behind the
  // merge (by hand, as in decode_lds: the compiler would wait for it here).
  __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0), said so that the compiler knows
  int ticket = -1;
  if (pi.update && lane == 0 && (!CHUNKS || pi.nchunks == 1)) {
    const int one = 1;
    asm volatile("global_atomic_add %0, %1, %2, off sc0" : "=v"(ticket) : "v"(p.tickets + pi.s * kTicketStride), "v"(one) : "memory");
  }
  l_run = rows_allreduce_sum(l_run);

  // merge the waves through LDS: lane (n, kb) holds columns 64*j + 16*kb + 4*e .. +3 of head n
  // (each wave's part of LDS is its own up to the barrier)
  constexpr int PITCH = LDS / NW / 4;
  float* s_part = reinterpret_cast<float*>(tiles);
  float* s_m = s_part + G * APITCH;
  float* s_l = s_m + G;
  if (n < G) {
#pragma unroll
    for (int j = 0; j < VJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        *reinterpret_cast<f32x4_t*>(s_part + wave * PITCH + n * APITCH + 64 * j + 16 * kb + 4 * e) =
            f32x4_t{O[4 * j][e], O[4 * j + 1][e], O[4 * j + 2][e], O[4 * j + 3][e]};
    if (kb == 0) { s_m[wave * PITCH + n] = m_run; s_l[wave * PITCH + n] = l_run; }
  }
  __syncthreads();
  merge_waves_and_store4<NW, D, D, APITCH, CHUNKS, true>(p, pi, s_m, s_l, s_part, PITCH, 0);
  if constexpr (CHUNKS) {
    if (pi.nchunks > 1) {
      *end = Closing{pi, nullptr};
      return true;
    }
  }
  if (!pi.update) return false;
  wait_vmcnt<0>();
  landed(ticket);
  if (__builtin_amdgcn_readfirstlane(ticket) != tickets_due(p.Hkv, NW, 1, CHUNKS ? p.max_chunks : 1) - 1) return false;
  finish_step<RB>(p, pi, lane);
  return false;
}

// The same on FMA instructions, for bf16 rows (BC_PLAN_PLAIN_ALU) and small fp32 groups (fma_is_faster).
// CHUNKS: as for the matrix kernel.
template <typename T, int D, int G, int U, bool CHUNKS>
__device__ __forceinline__ bool decode_alu_rows(const DecodeParams& p, Closing* end) {
  constexpr int ES = Elem<T>::size;
  constexpr int EPL = Elem<T>::per16;   // elements per lane per row
  constexpr int LPR = D / EPL;          // lanes per row
  constexpr int RPI = 64 / LPR;         // rows per wave load instruction
  constexpr int RB = D * ES;            // row bytes
  constexpr int ROWS_PER_PASS = kValuWaves * RPI * U;

  TableEntries tables;
  request_tables(p, (int)blockIdx.y, tables);
  touch_kernel_arguments<kTableArguments>();
  const PairInfo pi = pair_info(p, (int)blockIdx.y, (int)blockIdx.x, CHUNKS ? p.max_chunks - 1 - (int)blockIdx.z : 0,
                                NoEarlyWork(), &tables);
  if (!pi.live) {
    if constexpr (CHUNKS) {
      *end = Closing{pi, nullptr};
      return close_without_chunk<RB>(pi, 1);
    }
    return false;
  }
  const int row_end = pi.row_end;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane / LPR, ls = lane - lr * LPR;
  const int64_t stream_off = (pi.base * p.Hkv + (int64_t)pi.kvh * pi.cap) * RB + ls * 16;
  const char* kbase = p.k_slab + stream_off;
  const char* vbase = p.v_slab + stream_off;

  // q slice of every head of the group, pre-scaled so that exp() becomes exp2()
  float qf[G][EPL];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    if (h < p.g) {
      const uint4 r = *reinterpret_cast<const uint4*>(
          p.q + ((int64_t)(pi.s * p.Hq + pi.kvh * p.g + h) * D) * ES + ls * 16);
      unpack16(r, qf[h], T{});
#pragma unroll
      for (int e = 0; e < EPL; ++e) qf[h][e] *= p.qscale;
    } else {
#pragma unroll
      for (int e = 0; e < EPL; ++e) qf[h][e] = 0.f;
    }
  }

  float m[G], l[G], acc[G][EPL];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    m[h] = kNegBig; l[h] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[h][e] = 0.f;
  }

  // Fused step: the appended row (always the sequence's last) is not in the slab yet.  The loop
  // below covers the rows that are; the workgroup whose chunk holds the appended row takes it
  // from the caller's tensors in a pass of its own behind the loop and stores it for later steps
  // (unless this step's eviction drops it at once).  No reader touches the slab at that row in
  // this launch, so the store races with nothing.
  const bool new_row_here = pi.new_row >= pi.row0 && pi.new_row < row_end;      // (uniform)
  const int slab_end = new_row_here ? pi.new_row : row_end;

  for (int pr = pi.row0 + wave * (RPI * U); pr < slab_end; pr += ROWS_PER_PASS) {
    uint4 kk[U], vv[U];
    bool valid[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = pr + u * RPI + lr;
      valid[u] = r < slab_end;
      const int rc = valid[u] ? r : (slab_end - 1);  // stay inside the resident rows
      kk[u] = load16_stream(kbase + (int64_t)rc * RB);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = pr + u * RPI + lr;
      const int rc = valid[u] ? r : (slab_end - 1);
      vv[u] = load16_stream(vbase + (int64_t)rc * RB);
    }
    float sc[U][G];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float kf[EPL];
      unpack16(kk[u], kf, T{});
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float a = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) a = fmaf(qf[h][e], kf[e], a);
        a = group_allreduce_sum<LPR>(a);
        sc[u][h] = valid[u] ? a : kNegBig;
      }
    }
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float mn = m[h];
#pragma unroll
      for (int u = 0; u < U; ++u) mn = fmaxf(mn, sc[u][h]);
      const float alpha = fast_exp2(m[h] - mn);
      m[h] = mn;
      l[h] *= alpha;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[h][e] *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float pw = valid[u] ? fast_exp2(sc[u][h] - mn) : 0.f;
        sc[u][h] = pw;
        l[h] += pw;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float vf[EPL];
      unpack16(vv[u], vf, T{});
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[h][e] = fmaf(sc[u][h], vf[e], acc[h][e]);
    }
  }

  if (new_row_here && wave == 0) {
    // the appended row: one more row for the first lane group of the first wave
    const int64_t at = (int64_t)(pi.s * p.Hkv + pi.kvh) * RB + ls * 16;
    const uint4 kq = *reinterpret_cast<const uint4*>(p.new_k + at);
    const uint4 vq = *reinterpret_cast<const uint4*>(p.new_v + at);
    if (pi.store_new_row && lr == 0) {
      *reinterpret_cast<uint4*>(const_cast<char*>(kbase) + (int64_t)pi.new_row * RB) = kq;
      *reinterpret_cast<uint4*>(const_cast<char*>(vbase) + (int64_t)pi.new_row * RB) = vq;
    }
    float kf[EPL], vf[EPL];
    unpack16(kq, kf, T{});
    unpack16(vq, vf, T{});
    const bool mine = lr == 0;
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float a = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) a = fmaf(qf[h][e], kf[e], a);
      a = group_allreduce_sum<LPR>(a);
      const float sc1 = mine ? a : kNegBig;
      const float mn = fmaxf(m[h], sc1);
      const float alpha = fast_exp2(m[h] - mn);
      const float pw = mine ? fast_exp2(sc1 - mn) : 0.f;
      m[h] = mn;
      l[h] = l[h] * alpha + pw;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[h][e] = fmaf(pw, vf[e], acc[h][e] * alpha);
    }
  }

  // merge the RPI lane groups of a wave (fixed butterfly order)
#pragma unroll
  for (int off = LPR; off < 64; off <<= 1) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float mo = __shfl_xor(m[h], off, 64);
      const float lo = __shfl_xor(l[h], off, 64);
      const float mn = fmaxf(m[h], mo);
      const float a = fast_exp2(m[h] - mn), b = fast_exp2(mo - mn);
      m[h] = mn;
      l[h] = l[h] * a + lo * b;
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        const float ao = __shfl_xor(acc[h][e], off, 64);
        acc[h][e] = acc[h][e] * a + ao * b;
      }
    }
  }

  __shared__ float s_acc[kValuWaves * G * D];
  __shared__ float s_m[kValuWaves * G], s_l[kValuWaves * G];
  if (lr == 0) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) s_acc[(wave * G + h) * D + ls * EPL + e] = acc[h][e];
      if (ls == 0) { s_m[wave * G + h] = m[h]; s_l[wave * G + h] = l[h]; }
    }
  }
  __syncthreads();
  // Fused step, whole sequence: one ticket per workgroup, taken once all its waves have used the rows
  // they read (the barrier above); the answer comes back under the merge.  The workgroup that draws the
  // sequence's last one finishes the step.
  int ticket = -1;
  if ((!CHUNKS || pi.nchunks == 1) && pi.update && tid == 0) ticket = atomicAdd(p.tickets + pi.s * kTicketStride, 1);
  merge_waves_and_store<kValuWaves, D, CHUNKS>(p, pi, s_m, s_l, s_acc, G, G * D);
  if constexpr (CHUNKS) {
    if (pi.nchunks > 1) {
      *end = Closing{pi, nullptr};
      return true;
    }
  }
  if (!pi.update || wave != 0) return false;
  if (__builtin_amdgcn_readfirstlane(ticket) != tickets_due(p.Hkv, 1, 1, CHUNKS ? p.max_chunks : 1) - 1) return false;
  finish_step<RB>(p, pi, lane);
  return false;
}

// Two workgroups of the matrix form share a compute unit.  (Groups of seven and eight used to be compiled for one, which only their FMA form
// needs: see kLonePairs for what is left of that.)
template <typename T, int D, int G, int U, bool CHUNKS, bool FMA = !std::is_same<T, float>::value>
__global__ __launch_bounds__(256, FMA ? 1 : 2)
void decode_valu_kernel(BC_TABLE_ARGUMENTS, DecodeParams p) {
  p.P = tP; p.nb = tnb; p.w = tw; p.cap = tcap; p.c = tc; p.base = tbase;
  if constexpr (CHUNKS) p.order = nullptr;            // (see follows_order())
  Closing end;
  bool closing;
  if constexpr (!FMA) closing = decode_f32_rows<D, G, CHUNKS>(p, &end);
  else closing = decode_alu_rows<T, D, G, U, CHUNKS>(p, &end);
  if constexpr (CHUNKS) {
    __shared__ int s_arrived;
    if (closing) close_pair<256, D, D * Elem<T>::size>(end, &s_arrived);
  }
}

static size_t align256(size_t x) { return (x + 255) / 256 * 256; }

struct DecodePlan {
  bool lds;           // LDS/MFMA kernel (bf16, d = 128) or the VALU kernel
  bool eight_waves;   // cut plans of the LDS kernel: one workgroup of eight waves a compute unit (d = 64: two fit), or two of four (see pick_lds_kernel)
  bool fma;           // the latter on FMA instructions (bf16 always, fp32 by fma_is_faster())
  int lone_bytes;     // LDS that keeps its workgroups from sharing a compute unit, or none (see kLonePairs)
  int Gp;             // padded group size
  int rows_per_pass;  // rows one pass of a workgroup covers
  int R;              // rows per workgroup
  int max_chunks;
  int chunk_rows, split_rows;         // see DecodeParams
  size_t tickets_bytes, arrivals_bytes, part_bytes;
  size_t total() const { return tickets_bytes + arrivals_bytes + part_bytes; }
  void size_for(const bc_shape* sh) {
    const size_t pairs = (size_t)sh->B * sh->Hkv;
    tickets_bytes = align256((size_t)sh->B * kTicketStride * 4);
    arrivals_bytes = sh->Hkv < kTicketStride ? 0 : align256(pairs * 4);
    part_bytes = pairs * max_chunks * (Gp * sh->d + kPartTail) * 4;
  }
};

static int padded_group(int g) { return g <= 1 ? 1 : g <= 2 ? 2 : g <= 4 ? 4 : g <= 6 ? 6 : 8; }

// see make_plan
constexpr int kSplitMinCap = 960, kSplitMinCapSome = 2 * kLdsWavesSplit * kTileRows + 1, kSplitMinCapSome64 = 912;
constexpr int kSplitMinRows = 320, kSplitMinRows64 = 384, kSplitMinRowsMany = 512;
constexpr int kSplitAlone = 512, kSplitAlone64 = 832;
constexpr int kFewPairs = 32, kFewPairsLong = 64;
static int few_pairs(int d, int max_cap) { return d == 128 && max_cap >= 1024 ? kFewPairsLong : kFewPairs; }
// Capacity from which on a step's plan has chunks.  us a step, whole / cut, of sequences as long as the capacity lets them be ("r": ragged, from 60 rows on).
// Fewer than 16 pairs, d = 128: 8 pairs (32/8 heads) of 600 rows 7.4 / 8.2, 750 8.1 / 8.5, 900 9.1 / 8.9, 14 (12/2) 8.0 / 8.1, 8.9 / 8.4, 10.1 / 8.6; d = 64: 6.6 / 7.5, 7.4 / 7.7,
// 8.1 / 8.1 and 6.8 / 7.4, 7.5 / 7.5, 8.5 / 7.6.  (Few KV heads a sequence would be better off cut from 750 or 900 rows on.)
// More than 48, d = 128: 64 of 700 11.1 / 11.4, of 930 13.2 / 12.6, r 12.2 / 10.8, 120 12.1 / 14.5, 15.5 / 17.0, r 13.3 / 14.0; d = 64: 64 8.9 / 8.6, 10.1 / 9.3, r 9.5 / 8.4, 120 9.4 /
// 10.1, 10.7 / 11.0, r 9.9 / 9.4.  (Up to 64 pairs would be better off cut from 930 rows on, with d = 64 from 700.)
// In between, d = 128: up to the rows that two tiles of each of twelve waves hold (24 of 780 11.0 / 8.9, of 930 12.3 / 9.2, r 11.8 / 8.5; 48 11.5 / 11.6, 12.8 / 12.0, r 12.0 / 10.9; 16 as
// two sequences of eight heads 9.4 / 9.05, 10.0 / 9.4, as one of 16 9.98 / 10.10, 10.76 / 10.51).
// d = 64: there up to 32 pairs of few KV heads a sequence (16 of 790 7.6 / 7.4, 24 7.9 / 7.6, 32 of four heads 7.9 / 7.8; three sequences of six 7.7 / 7.8, of eight 7.9 / 8.0, two of
// eight 7.55 / 8.0: all chunks of a sequence are counted on one line of memory), and 48 (9.4 / 8.4: whole, they read past the caches, see kStreamMinWorkgroups).  The others up to the 28 tiles
// with which a wave's fourth begins (40 of 790 8.05 / 8.25, 890 8.0 / 8.25, 905 8.8 / 8.3; two sequences of eight heads 7.6 / 8.1, 8.45 / 8.2 at 905), and 960 where a sequence has more KV
// heads than twelve (16 in one sequence 7.6 / 9.3, at 935 8.5 / 9.5, in two 7.9 / 8.9 and 8.8 / 9.0; 32 in one 8.8 / 10.2, 9.9 / 10.4).
static int split_capacity(const bc_shape* sh) {
  const long npairs = (long)sh->B * sh->Hkv;
  if (npairs < 16 || npairs > 48) return kSplitMinCap;
  if (sh->d == 128 || npairs >= kStreamMinWorkgroups || (npairs <= 32 && sh->Hkv <= 5)) return kSplitMinCapSome;
  return sh->Hkv <= 12 ? kSplitMinCapSome64 : kSplitMinCap;
}
constexpr long kMostChunks = 64;
constexpr int kChunkRowsMax = 512;    // rows a chunk of the matrix kernel need not go beyond: two passes of eight waves
constexpr int kPlanForSizing = -1;    // rows_override value: size the workspace (see below)

// fp32 groups of one or two on FMA instructions: they need so few registers there that four (groups of two), six (d = 128) or seven
// workgroups share a compute unit, two on the matrix instructions, which waste 14 or 15 columns of 16 besides.  Where all
// workgroups run at once on FMA but not on the matrix instructions, FMA is faster for short sequences of equal length (FMA,
// matrix, us a step of 50 / 130 rows; groups of one, d = 128: 512 pairs 10.7, 10.0 / 19.2, 17.0; 880 13.2, 15.5 /
// 26.1, 28.5; 1200 15.4, 19.4 / 31.9, 37.9; 2000 25.6, 27.7 / 58.2, 54.7; d = 64: 880 14.0, 12.7 / 18.8, 18.9; 1200 15.4, 15.8 / 21.0, 24.5;
// 2000 23.9, 22.1 / 37.6, 34.0; groups of two, d = 64: 512 10.4, 8.4 / 13.6, 11.9; 880 12.5, 12.7 / 17.2, 19.5; 1200 18.2, 16.2 / 26.6,
// 25.1; ragged, 2040 pairs of 17 to 104 rows, groups of one, d = 128: 27 and 30, 1584 of 10 to 55, d = 64:
// 16 and 19).  From some 200 rows on both take what HBM takes (520 pairs of 600 rows, groups of one, d = 128: 63, 68; 1000 104, 104), and
// where few workgroups are left for a second round of the matrix form they fill in behind the short ones of a ragged batch, while FMA is slow on the
// long ones (matrix / FMA time, lengths spread evenly up to 130, 200, 400, 600 rows; groups of one, d = 128: 520 pairs 0.87, 0.81, 0.77, 0.73;
// 660 1.03, 0.95, 0.87, 0.85; 800 1.07, 1.02, 0.92, 0.93; d = 64: 1060 0.98, 0.89, 0.80, 0.77; 1250 1.07, 0.97, 0.87, 0.83; groups of two, d = 64: 520
// 0.89, 0.86, 0.83, 0.78; 720 1.01, 0.98, 0.98, 0.97; d = 128: 520 0.81, 0.74, 0.71, 0.67; 720 0.96, 0.92, 0.84, 0.84): so only
// for capacities of up to 256 rows, and for those beyond 136 with 128 pairs more (groups of two of d = 128: 160 and 64).  What that
// costs are batches of equal length and some 50 % more workgroups than run at once (800 pairs of 400 rows, groups of one, d = 128: FMA 59, matrix 64).
static bool fma_is_faster(long npairs, int Gp, int d, int max_cap) {
  const bool wide_pair = Gp == 2 && d == 128;
  if (Gp > 2 || max_cap > (wide_pair ? 160 : 256)) return false;
  const long above = (Gp == 1 && d == 64 ? 1024 : 512) + (max_cap <= (wide_pair ? 64 : 136) ? 0 : 128);
  const long most = Gp == 2 ? 1024 : d == 64 ? 1792 : max_cap <= 128 ? LONG_MAX : 1536;
  return npairs > above && npairs <= most;
}

// Rows from which on an fp32 sequence is cut (the plan of a capacity below that has one chunk).  A workgroup goes through 64 (d =
// 128) or 128 rows a pass; whole and cut meet in the third pass, with more than 64 pairs of d = 128 in the fourth or fifth (us a step,
// whole / cut.  d = 64 at 300, 350, 400 rows: 8 pairs 8.8 / 7.7, 8.9 / 7.7, 10.7 / 7.8; 64 pairs 9.5 / 8.5, 9.6 / 8.7, 11.3 / 8.9; 100 pairs
// 10.4 / 9.8, 10.2 / 10.3, 12.0 / 10.8; 127 pairs 10.7 / 10.3, 10.6 / 10.7, 12.3 / 11.2.  d = 128 at 150, 200, 260 rows: 8 pairs 8.9 / 8.1, 10.6 /
// 8.1, 12.1 / 8.1; 64 pairs 9.3 / 8.7, 11.1 / 9.0, 12.7 / 10.7; 96 pairs 10.1 / 10.3, 11.7 / 10.7, 13.0 / 12.4; 127 pairs 10.3 / 10.8, 12.3 / 11.6,
// 14.1 / 13.2).  The lines are lower than batches of equal length call for: the
// longest sequences of a ragged one set its time (100 pairs of 37 to 1000 rows, d = 64: 18.9 cut from 898 rows on, 13.3 from 258 on; 64 pairs of 37
// to 500: 11.0 from 450, 8.6).  Attention alone has a launch in front to clear its counters, 1 to 2 us where there are many, and is cut
// later (33 pairs, d = 64, 400 rows: 10.2 / 9.1; 64 pairs, d = 128, groups of six, 230 rows: 10.3 / 11.2; 100 pairs, d = 128, 300 and 350 rows: 13.2
// / 13.6, 15.0 / 13.8; 128 pairs of 500: 18.8 / 18.0, of groups of six 18.7 / 19.7).
// More than 128 pairs: whole, without the fold and its workgroups (200 pairs in two chunks, d = 64: 29.2 / 33.2 at 1500 rows, 37.1 / 42.5
// at 2000; 150 pairs of 500 rows in plans of one and three chunks that cut none of them: 11.7, 12.3, attention alone on 130 of 300 rows 13.5, 15.4).  Only groups of one and two with d = 64,
// which one workgroup a pair draws the least for, are cut where they are long and three chunks run at once (150 pairs: 26.6 / 24.6 at 1500 rows, 32.7 /
// 32.7 at 2000; three sequences of 1500 rows among those of 50 to 300 23.8 / 15.4, of 4400 59.7 / 28.4; 170 pairs of 37 to 2000 31.4 / 32.5).
constexpr long kF32MostPairs = 512 / 3;
constexpr int kF32SplitRowsMany = 1408;
static int f32_split_rows(long npairs, int Gp, int d, int rows_per_pass, bool alone) {
  if (npairs > 128) return npairs <= kF32MostPairs && d == 64 && Gp <= 2 ? kF32SplitRowsMany + (alone ? 128 : 0) : INT_MAX;
  const bool early = npairs <= 32 || (d == 64 && npairs <= 64);
  const int passes = alone ? (early ? 3 : npairs <= 96 ? 4 : 8) : d == 64 || npairs <= 64 ? 2 : npairs <= 96 ? 3 : 4;
  return passes * rows_per_pass + 2;
}

// Groups of seven and eight, few more pairs than compute units: one workgroup each, by LDS that nobody uses, so that the pairs
// left over start behind short sequences and not beside long ones, whose time doubles.  us a step, two a compute unit / one: 260 pairs of 100 to
// 1000 rows, d = 64, 27.8 / 23.9, d = 128 48.3 / 37.8, 272 28.4 / 24.6 and 48.8 / 38.3, 288 31.2 / 33.9 and 51.6 / 54.3, 304 31.5 / 33.9 and 52.0 / 54.1;
// 272 of 20 to 200 11.5 / 12.0 and 15.7 / 14.5; of equal length two are always better (260 of 300 rows 16.5 / 18.7, 25.3 / 26.9).
// Compiled for one workgroup, as these groups were, 300 of 200 rows 15.6, and 12.7 with two, d = 128
// 23.3 and 20.0; 800 of 500 50.5 and 43.0, 85.9 and 79.3; 100 of 100 to 1000, d = 64, 15.5 and 14.3; 8 of 200 7.7 and 7.5.
constexpr int kLonePairs = 280;
constexpr int kLoneBytes = 52 << 10;      // with the tiles' 32 KB more than half of a compute unit's

// alone: attention without a step.
static DecodePlan make_plan(const bc_shape* sh, int max_cap, int rows_override, int plan_bits, bool alone = false) {
  DecodePlan pl;
  pl.eight_waves = true;
  const long npairs = (long)sh->B * sh->Hkv;
  pl.lds = sh->kv_dtype == BC_BF16 && !(plan_bits & BC_PLAN_PLAIN_ALU);
  if (pl.lds) {
    pl.Gp = 8;
    pl.rows_per_pass = kLdsWaves * kTileRows;
  } else {
    pl.Gp = padded_group(sh->Hq / sh->Hkv);
    const int epl = 16 / elem_size(sh->kv_dtype);
    const int lpr = sh->d / epl, rpi = 64 / lpr;
    pl.rows_per_pass = kValuWaves * rpi * 8;
  }
  pl.chunk_rows = pl.lds ? std::min(kChunkRowsMax, std::max(2 * kTileRows, (max_cap + 15) / 16)) : pl.rows_per_pass;
  pl.split_rows = kSplitMinRows;
  // capacity from which on the plan has chunks at all
  int split_cap = alone ? kSplitMinCap : split_capacity(sh);
  if (!pl.lds) {
    // (a step reads its appended row behind the passes over the slab's)
    const int whole_passes = (npairs > kFewPairs || pl.Gp * sh->d >= 512 ? 1 : 2) + (alone ? 1 : 0);
    pl.split_rows = whole_passes * pl.rows_per_pass + 2;
    split_cap = (alone ? 4 : whole_passes) * pl.rows_per_pass + 1;
    // fp32: a plan has chunks only where its capacity lets a sequence be cut
    if (sh->kv_dtype == BC_F32) pl.split_rows = split_cap = f32_split_rows(npairs, pl.Gp, sh->d, pl.rows_per_pass, alone);
  }
  if (rows_override > 0) {
    // forced chunk size (experiments, tests): fixed rows per workgroup
    int R = ((rows_override + pl.rows_per_pass - 1) / pl.rows_per_pass) * pl.rows_per_pass;
    while ((max_cap + R - 1) / R > 64) R += pl.rows_per_pass;   // bound the partials per pair
    pl.R = R;
    pl.max_chunks = (max_cap + R - 1) / R;
  } else {
    // One workgroup per (sequence, KV head) pair when there are enough pairs.  With fewer, the rows of a
    // sequence are spread over as many workgroups as run at once, of at least two tiles or one pass of rows, and at
    // most sixteen, whose partials are folded in one round of loads, or one for every 512 rows (one sequence of
    // 150,256 rows, one KV head: sixteen 94 us, 64 38; 16,900 rows: 17.1, 15.5; 6000 rows, 8 KV heads: a chunk for
    // every 256 rows 15.7, every 512 14.8).  That many are 256 of the matrix kernel
    // at d = 128 (128 KB of LDS each; a second round of workgroups takes more than the cut saves), and 512 at d = 64 or with four waves (see
    // pick_lds_kernel).  At d = 128 eight waves and 256 are faster with up to 64 pairs (us a step, four waves / eight; 48 pairs of 1500 rows 13.3 / 12.2,
    // of 60 to 1500 11.3 / 10.5; 64 of 1500 14.0 / 12.6, of 60 to 1100 10.4 / 9.2, of 60 to 3000 16.8 / 16.0; 64 of 100 to 2000, eight pairs of each length, 11.9 / 12.0),
    // beyond that a sequence has three chunks or two, of which a ragged batch's longest are too long (72 pairs of 100 to 2000 12.4 / 14.2; 96 15.5 / 17.2;
    // of equal length, 1700 rows, 15.8 / 15.1 and 20.9 / 19.7).  Attention alone the same (34 pairs of 1100 rows 12.8 / 11.0, 48 of 60 to 1500 13.6 / 11.8, 64 of 60 to
    // 3000 19.3 / 18.6).  With less than 1024 rows of capacity the line is still at 32 pairs, where it was for all: nothing measured speaks for that (34 pairs of 780 rows 11.3 / 9.4, 40 of 1000
    // 11.8 / 10.25, 64 of 60 to 1000 11.0 / 10.2, attention alone on 40 of 1000 12.7 / 11.2), but plans there are known by their number of chunks.  At d = 64 512 is the line from 33 pairs on (90 of up to 1900 rows 10.2, with 256 10.7).
    // Up to split_capacity() rows of capacity all sequences stay whole.  Where the batch may have longer sequences the shorter ones run in the tile loop, and are cut from 320 rows on (whole, cut: 48 pairs of 400 rows,
    // capacity 1600, 9.8 / 7.9; 64 of 400, capacity 1150, 9.1 / 7.8), with d = 64 from 384 (32 pairs of 340 6.1 / 6.2, 40 of 60 to 700 from 512, 384 and 320 rows on 6.9, 6.8
    // and 6.9; 450 rows, four pairs 7.5 / 7.2, eight in one sequence 7.7 / 7.3) and one and two pairs from 512 (450 rows 6.4 / 6.8, 6.5 / 6.8), with more than 64 pairs from 512 where d is 64 (from 512, from 384: 126 pairs
    // of 400 to 505 rows 8.9 / 9.3, 110 8.8 / 9.1, 90 8.5 / 8.65, but 126 of 60 to 600 8.9 / 8.7, 80 of 60 to 600 8.55 / 8.05; 90 ragged ones, 16 layers, 149 / 152) or there are four
    // chunks at most (120 pairs of 60 to 1500 rows, from 512 15.9, from 320 16.3); attention alone, which pays for its counters besides, cuts them later.
    // The plain-ALU kernel is bound by its arithmetic, 64 or 128 rows a pass of 1 to 7 us (by group and d), against
    // some 2 us that a fold takes: cut from the second pass on, or from the third where a pass is short and the
    // batch is small, with up to 256 pairs.  256 workgroups run at once with groups of three or more (over 256
    // registers), otherwise 512; beyond that a second round takes more than the cut saves.  Attention alone has a launch in
    // front to clear its counters, some 1.5 us: its sequences are cut one pass later, and by capacities beyond four passes.
    // fp32: lines in f32_split_rows().  More workgroups than 256 do not help there (40 pairs of 760 rows: 480 15.3, 240 13.5; 120 ragged
    // ones of 200 to 1200, d = 128, 29.2, 26.5; 128 pairs of 350, in four chunks and in two 16.3, 14.2) but for many pairs with
    // the shorter rows of d = 64 (100 pairs of up to 4400 rows: 26.4, and 34.0 with 256).
    pl.eight_waves = npairs <= few_pairs(sh->d, max_cap) ||
                     (sh->d == 128 && (plan_bits & (BC_PLAN_NO_SMALL_WORKGROUPS | BC_PLAN_CACHEABLE_LOADS)));
    const bool one_per_cu = pl.lds ? pl.eight_waves
                            : sh->kv_dtype == BC_F32 ? npairs <= (sh->d == 64 ? 64 : 128) : pl.Gp >= 4;
    const long at_once = one_per_cu ? 256 : 512, most_pairs = pl.lds ? 127 : sh->kv_dtype == BC_F32 ? kF32MostPairs : 256;
    long chunks = 1;
    if (npairs <= most_pairs && max_cap >= split_cap) {
      chunks = at_once / npairs;
      const long by_rows = (max_cap + pl.chunk_rows - 1) / pl.chunk_rows, most = npairs < 128 ? kMostChunks : 4;
      if (chunks > by_rows) chunks = by_rows;
      if (chunks > most) chunks = most;
      if (pl.lds && !alone)
        pl.split_rows = npairs > 64 && (sh->d == 64 || chunks <= 4) ? kSplitMinRowsMany : sh->d == 128 ? kSplitMinRows : npairs <= 2 ? kSplitMinRowsMany : kSplitMinRows64;
      if (pl.lds && alone) pl.split_rows = chunks <= 4 && npairs > 64 ? 2 * kSplitAlone : sh->d == 64 ? kSplitAlone64 : kSplitAlone;
    }
    pl.R = 0;                                        // spread evenly, decided per sequence
    pl.max_chunks = (int)chunks;
  }
  pl.fma = !pl.lds && (sh->kv_dtype == BC_BF16 || (pl.max_chunks == 1 && fma_is_faster(npairs, pl.Gp, sh->d, max_cap)));
  pl.lone_bytes = !pl.lds && !pl.fma && pl.Gp == 8 && pl.max_chunks == 1 && npairs > 256 && npairs <= kLonePairs ? kLoneBytes : 0;
  // Workspace sizing: the most chunks the automatic plan can choose, 64 with few pairs and four otherwise (a
  // forced chunk size on a large batch may use as many).
  if (rows_override == kPlanForSizing) pl.max_chunks = npairs < 128 ? 64 : 4;
  pl.size_for(sh);
  return pl;
}

// (KV head, sequence, chunk): the same chunk of all pairs lies side by side and spreads over the XCDs, to which
// workgroups go in turn.  With the chunk in front, a plan of eight chunks had all rows of sequences that stay whole on
// one XCD (64 pairs of 505 rows, 12/2 heads: 19.4 us a step, 12.1 now).  The last chunks come first: only the longest
// sequences have them (16 layers of 45 ragged sequences, 14/2 heads, d = 64: 192 us from the first, 172 from the last).
static dim3 decode_grid(const bc_shape* shape, const DecodePlan& pl) { return dim3(shape->Hkv, shape->B, pl.max_chunks); }

template <typename T, int D, int G>
static void launch_valu_group(const DecodeParams& p, const DecodePlan& pl, dim3 grid, hipStream_t st) {
  if constexpr (std::is_same<T, float>::value && G <= 2) {
    if (pl.fma) {
      decode_valu_kernel<T, D, G, 8, false, true><<<grid, 256, 0, st>>>(p.P, p.nb, p.w, p.cap, p.c, p.base, p);
      return;
    }
  }
  if (p.max_chunks > 1) decode_valu_kernel<T, D, G, 8, true><<<grid, 256, 0, st>>>(p.P, p.nb, p.w, p.cap, p.c, p.base, p);
  else decode_valu_kernel<T, D, G, 8, false><<<grid, 256, pl.lone_bytes, st>>>(p.P, p.nb, p.w, p.cap, p.c, p.base, p);
}
template <typename T, int D>
static void launch_valu(const DecodeParams& p, const DecodePlan& pl, dim3 grid, hipStream_t st) {
  switch (pl.Gp) {
    case 1: launch_valu_group<T, D, 1>(p, pl, grid, st); break;
    case 2: launch_valu_group<T, D, 2>(p, pl, grid, st); break;
    case 4: launch_valu_group<T, D, 4>(p, pl, grid, st); break;
    case 6: launch_valu_group<T, D, 6>(p, pl, grid, st); break;
    default: launch_valu_group<T, D, 8>(p, pl, grid, st); break;
  }
}

// Which instantiation of the LDS/MFMA kernel serves a call, with its launch shape.  `name` is the
// kernel's name as profilers print it.
struct LdsLaunch {
  void (*fn)(DecodeParams);
  void (*cut)(BC_TABLE_ARGUMENTS, DecodeParams);
  const char* name;
  dim3 grid;
  int threads;
  int lds_bytes;
};
#define BC_LDS_KERNEL(...) decode_lds_kernel<__VA_ARGS__>, nullptr, "bc::decode_lds_kernel<" #__VA_ARGS__ ">"
#define BC_LDS_CUT_KERNEL(...) nullptr, decode_lds_cut_kernel<__VA_ARGS__>, "bc::decode_lds_cut_kernel<" #__VA_ARGS__ ">"

static LdsLaunch pick_lds_kernel(const bc_shape* shape, const bc_cache* cache, const DecodePlan& pl,
                                 bool ordered) {
  const int pairs = shape->B * shape->Hkv;
  const dim3 grid = decode_grid(shape, pl);
  const int lds_full = kLdsBytes + kBeaconBytes, lds_half = kLdsBytes / 2 + kBeaconBytes;      // tiles, beacon rows
  // launches that cannot saturate the memory system are latency-bound: default cache policy
  const bool cacheable = (cache->plan & BC_PLAN_CACHEABLE_LOADS) != 0;
  const bool general = (cache->plan & BC_PLAN_GENERAL_LOOP) != 0;
  const bool stream = (long)pairs * pl.max_chunks >= kStreamMinWorkgroups && !cacheable;
  // at most two tiles per wave of an eight-wave workgroup: the straight-line form of the kernel
  const bool two8 = pl.max_chunks == 1 && !ordered && !general && cache->max_cap <= 2 * kLdsWaves * kTileRows;
  // two workgroups per pair (each one half of the V columns) while that still fits the chip
  int slots = shape->B;                   // padded until the pairs are a multiple of 8
  while ((slots * shape->Hkv) & 7) ++slots;
  const bool vsplit = shape->d == 128 && pl.max_chunks == 1 && 2 * slots * shape->Hkv <= kLptMinPairs &&
                      !(cache->plan & BC_PLAN_ONE_WORKGROUP_PER_PAIR);
  if (vsplit) {
    // K lines are read by both workgroups of a pair: streamed while the batch's K is small
    // enough for the partner's request to find the line still on its way or in the L2
    // (measured up to about 48 MB), cacheable beyond
    const bool stream2 = 2L * pairs >= kStreamMinWorkgroups && !cacheable;
    const bool small_k = (int64_t)pairs * cache->max_cap * 256 <= (48LL << 20);
    // short caches: twelve waves (most sequences then need one pass); long ones: eight
    const bool w12 = cache->max_cap <= kSplitWaves12MaxCap;
    const bool two12 = w12 && cache->max_cap <= 2 * kLdsWavesSplit * kTileRows && !general;
    const dim3 g2(shape->Hkv, slots, 2);
    const int t12 = kLdsWavesSplit * 64, l12 = kLdsBytesSplit + kBeaconBytes, t8 = kLdsWaves * 64;
    const int l8 = kLdsWaves * 3 * kTileRows * 128 + kBeaconBytes;
    if (two12) return stream2 ? LdsLaunch{BC_LDS_KERNEL(1, 128, 2, 12, true), g2, t12, l12}
                              : LdsLaunch{BC_LDS_KERNEL(0, 128, 2, 12, true), g2, t12, l12};
    if (!stream2) return w12 ? LdsLaunch{BC_LDS_KERNEL(0, 128, 2, 12), g2, t12, l12}
                             : LdsLaunch{BC_LDS_KERNEL(0, 128, 2, 8), g2, t8, l8};
    if (small_k) return w12 ? LdsLaunch{BC_LDS_KERNEL(1, 128, 2, 12), g2, t12, l12}
                            : LdsLaunch{BC_LDS_KERNEL(1, 128, 2, 8), g2, t8, l8};
    return LdsLaunch{BC_LDS_KERNEL(2, 128, 2, 8), g2, t8, l8};
  }
  // Workgroups of four waves, two per compute unit (64 KB of LDS each at d = 128), so that one's start
  // and end phases - tables, first bytes, merge, store - overlap with the other's streaming: for
  // sequences cut into chunks of more pairs than eight-wave workgroups serve well (see make_plan), and
  // with more pairs than the chip holds workgroups and short caches.  Measured at 512 pairs of 512
  // rows: 28.2 -> 25.4 us; with long ragged sequences (512 pairs of up to 2700 rows) the longest
  // streams set the pace and eight waves are faster (54.5 against 62.5 us).
  const bool small = stream && !(cache->plan & BC_PLAN_NO_SMALL_WORKGROUPS);
  if (pl.max_chunks > 1) {
    if (shape->d == 128) {
      if (small && pl.R == 0 && !pl.eight_waves)
        return LdsLaunch{BC_LDS_CUT_KERNEL(1, 128, 4), grid, 4 * 64, lds_half};
      return stream ? LdsLaunch{BC_LDS_CUT_KERNEL(1, 128, 8), grid, kLdsWaves * 64, lds_full}
                    : LdsLaunch{BC_LDS_CUT_KERNEL(0, 128, 8), grid, kLdsWaves * 64, lds_full};
    }
    return stream ? LdsLaunch{BC_LDS_CUT_KERNEL(1, 64, 8), grid, kLdsWaves * 64, lds_half}
                  : LdsLaunch{BC_LDS_CUT_KERNEL(0, 64, 8), grid, kLdsWaves * 64, lds_half};
  }
  if (shape->d == 128) {
    if (small && pairs > kLptMinPairs && cache->max_cap <= kSplitWaves12MaxCap)
      return LdsLaunch{BC_LDS_KERNEL(1, 128, 1, 4), grid, 4 * 64, lds_half};
    if (two8) return stream ? LdsLaunch{BC_LDS_KERNEL(1, 128, 1, 8, true), grid, kLdsWaves * 64, lds_full}
                            : LdsLaunch{BC_LDS_KERNEL(0, 128, 1, 8, true), grid, kLdsWaves * 64, lds_full};
    return stream ? LdsLaunch{BC_LDS_KERNEL(1, 128, 1, 8), grid, kLdsWaves * 64, lds_full}
                  : LdsLaunch{BC_LDS_KERNEL(0, 128, 1, 8), grid, kLdsWaves * 64, lds_full};
  }
  if (two8) return stream ? LdsLaunch{BC_LDS_KERNEL(1, 64, 1, 8, true), grid, kLdsWaves * 64, lds_half}
                          : LdsLaunch{BC_LDS_KERNEL(0, 64, 1, 8, true), grid, kLdsWaves * 64, lds_half};
  return stream ? LdsLaunch{BC_LDS_KERNEL(1, 64, 1, 8), grid, kLdsWaves * 64, lds_half}
                : LdsLaunch{BC_LDS_KERNEL(0, 64, 1, 8), grid, kLdsWaves * 64, lds_half};
}

// The LDS kernel needs 128 KB of dynamic LDS: opt in once per device.  Two host threads that get
// here together both set the (same) attributes; the flag only saves the later calls.
static int32_t enable_big_lds() {
  static std::atomic<bool> done[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return BC_ERR_HIP;
  if (done[dev].load(std::memory_order_acquire)) return BC_OK;
  const void* kernels[] = {reinterpret_cast<const void*>(decode_lds_kernel<1, 128, 1, 4>),
                           reinterpret_cast<const void*>(decode_lds_cut_kernel<1, 128, 4>),
                           reinterpret_cast<const void*>(decode_lds_cut_kernel<0, 128, 8>),
                           reinterpret_cast<const void*>(decode_lds_cut_kernel<1, 128, 8>),
                           reinterpret_cast<const void*>(decode_lds_cut_kernel<0, 64, 8>),
                           reinterpret_cast<const void*>(decode_lds_cut_kernel<1, 64, 8>),
                           reinterpret_cast<const void*>(decode_lds_kernel<0, 128, 1, 8>),
                           reinterpret_cast<const void*>(decode_lds_kernel<1, 128, 1, 8>),
                           reinterpret_cast<const void*>(decode_lds_kernel<0, 128, 1, 8, true>),
                           reinterpret_cast<const void*>(decode_lds_kernel<1, 128, 1, 8, true>),
                           reinterpret_cast<const void*>(decode_lds_kernel<0, 64, 1, 8>),
                           reinterpret_cast<const void*>(decode_lds_kernel<1, 64, 1, 8>),
                           reinterpret_cast<const void*>(decode_lds_kernel<0, 64, 1, 8, true>),
                           reinterpret_cast<const void*>(decode_lds_kernel<1, 64, 1, 8, true>),
                           reinterpret_cast<const void*>(decode_lds_kernel<0, 128, 2, 8>),
                           reinterpret_cast<const void*>(decode_lds_kernel<1, 128, 2, 8>),
                           reinterpret_cast<const void*>(decode_lds_kernel<2, 128, 2, 8>),
                           reinterpret_cast<const void*>(decode_lds_kernel<0, 128, 2, 12>),
                           reinterpret_cast<const void*>(decode_lds_kernel<1, 128, 2, 12>),
                           reinterpret_cast<const void*>(decode_lds_kernel<0, 128, 2, 12, true>),
                           reinterpret_cast<const void*>(decode_lds_kernel<1, 128, 2, 12, true>)};
  bool ok = true;
  for (const void* kfn : kernels)
    ok = ok && hipFuncSetAttribute(kfn, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytesMax) ==
                   hipSuccess;
  if (!ok)
    return BC_ERR_HIP;
  done[dev].store(true, std::memory_order_release);
  return BC_OK;
}

__global__ void fill_zero_kernel(uint32_t* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// Batches that need more than one round of workgroups follow the caller's dispatch order
// (bc_sort_by_length), if there is one; with fewer workgroups everything starts at once.
static bool follows_order(const bc_shape* shape, const bc_cache* cache, const DecodePlan& pl) {
  return cache->order && pl.max_chunks == 1 && shape->B * shape->Hkv > kLptMinPairs &&
         !(cache->plan & BC_PLAN_IGNORE_ORDER);
}

// Attention launch shared by bc_decode_attn (k = beacon_k = NULL) and the fused bc_decode_step.
static int32_t launch_attention(const bc_shape* shape, const bc_cache* cache, const DecodePlan& pl,
                                const void* q, float* out, const uint8_t* active, void* workspace,
                                size_t workspace_bytes, const void* k, const void* v, const void* bk,
                                const void* bv, hipStream_t hs, const int32_t* budget = nullptr,
                                uint8_t* live = nullptr, bool beacon_row = false) {
  DecodeParams p;
  p.k_slab = static_cast<const char*>(cache->k_slab);
  p.v_slab = static_cast<const char*>(cache->v_slab);
  p.base = cache->base; p.cap = cache->cap; p.P = cache->P; p.nb = cache->nb; p.w = cache->w;
  p.err = cache->err;
  p.q = static_cast<const char*>(q);
  p.out = out;
  p.active = active;
  char* ws = static_cast<char*>(workspace);
  p.tickets = reinterpret_cast<int32_t*>(ws);
  // Counters from the front, partial results at the back: calls of another batch size that share the
  // workspace find their counters as they left them.
  p.part = pl.max_chunks > 1 ? reinterpret_cast<float*>(ws + (workspace_bytes - pl.part_bytes) / 256 * 256) : nullptr;
  // a pair's chunks are counted on the line of its sequence's ticket counter; where that has not got a
  // place for every KV head they have an array, cleared in front of the launch.  Attention alone takes no
  // tickets and asks nothing of the workspace it is given: its counters are cleared in front of the launch too
  // (a second launch, as the fold used to be; the steps, whose tickets start at zero anyway, do without).
  p.arrivals = p.tickets + 1;
  p.arrival_stride = kTicketStride;
  size_t clear_bytes = !k ? pl.tickets_bytes : 0;
  if (pl.arrivals_bytes) {
    p.arrivals = reinterpret_cast<int32_t*>(ws + pl.tickets_bytes);
    p.arrival_stride = shape->Hkv;
    clear_bytes = pl.arrivals_bytes;
  }
  if (pl.max_chunks > 1 && clear_bytes)
    fill_zero_kernel<<<(int)std::min<size_t>(1024, (clear_bytes + 1023) / 1024), 256, 0, hs>>>(
        reinterpret_cast<uint32_t*>(pl.arrivals_bytes ? p.arrivals : p.tickets), (int64_t)(clear_bytes / 4));
  p.c = cache->c; p.nb_rw = cache->nb; p.w_rw = cache->w;
  p.new_k = static_cast<const char*>(k); p.new_v = static_cast<const char*>(v);
  p.bk = static_cast<const char*>(bk); p.bv = static_cast<const char*>(bv);
  p.budget = budget; p.live = live;
  p.beacon_row = beacon_row ? 1 : 0;
  p.B = shape->B;
  p.order = follows_order(shape, cache, pl) ? cache->order : nullptr;
  p.Hq = shape->Hq; p.Hkv = shape->Hkv; p.g = shape->Hq / shape->Hkv;
  p.Gp = pl.Gp;
  p.rows_per_wg = pl.R;
  p.max_chunks = pl.max_chunks;
  p.chunk_rows = pl.chunk_rows; p.split_rows = pl.split_rows;
  p.qscale = shape->scale * kLog2e;
  p.spec_P = (cache->plan & BC_PLAN_IGNORE_PROMISE) ? 0 : cache->uniform_P;
  p.spec_cap = cache->uniform_cap;

  const dim3 grid = decode_grid(shape, pl);
  if (pl.lds) {
    const int32_t st = enable_big_lds();
    if (st != BC_OK) return st;
    const LdsLaunch k = pick_lds_kernel(shape, cache, pl, p.order != nullptr);
    if (k.cut) k.cut<<<k.grid, k.threads, k.lds_bytes, hs>>>(p.P, p.nb, p.w, p.cap, p.c, p.base, p);
    else k.fn<<<k.grid, k.threads, k.lds_bytes, hs>>>(p);
  } else if (shape->kv_dtype == BC_BF16) {
    if (shape->d == 128) launch_valu<bf16_t, 128>(p, pl, grid, hs);
    else launch_valu<bf16_t, 64>(p, pl, grid, hs);
  } else {
    if (shape->d == 128) launch_valu<float, 128>(p, pl, grid, hs);
    else launch_valu<float, 64>(p, pl, grid, hs);
  }
  return launch_status();
}

static int32_t check_attention_args(const bc_shape* shape, const bc_cache* cache, const void* q,
                                    const float* out, const void* workspace, size_t workspace_bytes,
                                    DecodePlan* pl, bool alone = false) {
  int32_t st = check_shape(shape);
  if (st != BC_OK) return st;
  st = check_cache(cache);
  if (st != BC_OK) return st;
  if (!q || !out || !aligned16(q) || !aligned16(out)) return BC_ERR_ARG;
  if (shape->B > 65535 || shape->Hkv > 65535) return BC_ERR_SHAPE;      // grid dimensions
  if (!nonnegative_finite(shape->scale)) return BC_ERR_ARG;   // the kernels take maxima of unscaled scores
  if (cache->rows_per_workgroup < 0 || (cache->plan & ~BC_PLAN_ALL_BITS)) return BC_ERR_ARG;
  *pl = make_plan(shape, cache->max_cap, cache->rows_per_workgroup, cache->plan, alone);
  if ((cache->plan & BC_PLAN_NEED_MATRIX_KERNEL) && !pl->lds) return BC_ERR_SHAPE;
  if (!workspace || !aligned16(workspace) || workspace_bytes < pl->total()) return BC_ERR_WORKSPACE;
  return BC_OK;
}

}  // namespace bc

using namespace bc;

extern "C" int32_t bc_sort_by_length(const bc_shape* shape, const bc_cache* cache,
                                     const uint8_t* active, int32_t* order, void* stream) {
  int32_t st = check_shape(shape);
  if (st != BC_OK) return st;
  st = check_cache(cache);
  if (st != BC_OK) return st;
  if (!order) return BC_ERR_ARG;
  if (shape->B > kLptMaxB) return BC_ERR_SHAPE;
  SortParams p;
  p.active = active; p.P = cache->P; p.nb = cache->nb; p.w = cache->w;
  p.order = order; p.B = shape->B;
  sort_by_length_kernel<<<(shape->B + 255) / 256, 256, 0, as_stream(stream)>>>(p);
  return launch_status();
}

extern "C" size_t bc_decode_workspace_bytes(const bc_shape* shape, int32_t max_cap) {
  if (check_shape(shape) != BC_OK || max_cap < 1) return 0;
  // sized for the largest number of chunks the automatic plan can select, for either kernel
  const DecodePlan a = make_plan(shape, max_cap, kPlanForSizing, 0),
                   b = make_plan(shape, max_cap, kPlanForSizing, BC_PLAN_PLAIN_ALU);
  return a.total() > b.total() ? a.total() : b.total();
}

extern "C" int32_t bc_workspace_init(void* workspace, size_t workspace_bytes, void* stream) {
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 3u)) return BC_ERR_ARG;
  const int64_t n = (int64_t)(workspace_bytes / 4);
  if (n == 0) return BC_OK;
  const int64_t blocks = (n + 255) / 256;
  fill_zero_kernel<<<(int)(blocks < 4096 ? blocks : 4096), 256, 0, as_stream(stream)>>>(
      static_cast<uint32_t*>(workspace), n);
  return launch_status();
}

extern "C" int32_t bc_decode_plan_describe(const bc_shape* shape, const bc_cache* cache, char* text,
                                           size_t text_bytes) {
  if (!text || text_bytes == 0) return BC_ERR_ARG;
  text[0] = 0;
  int32_t st = check_shape(shape);
  if (st != BC_OK) return st;
  st = check_cache(cache);
  if (st != BC_OK) return st;
  if (cache->rows_per_workgroup < 0 || (cache->plan & ~BC_PLAN_ALL_BITS)) return BC_ERR_ARG;
  const DecodePlan pl = make_plan(shape, cache->max_cap, cache->rows_per_workgroup, cache->plan);
  if ((cache->plan & BC_PLAN_NEED_MATRIX_KERNEL) && !pl.lds) return BC_ERR_SHAPE;
  const char* merged = pl.max_chunks > 1 ? " + merge by a pair's last workgroup" : "";
  if (pl.lds) {
    const LdsLaunch k = pick_lds_kernel(shape, cache, pl, follows_order(shape, cache, pl));
    snprintf(text, text_bytes, "%s grid=(%u,%u,%u) threads=%d lds=%d chunks=%d%s", k.name, k.grid.x,
             k.grid.y, k.grid.z, k.threads, k.lds_bytes, pl.max_chunks, merged);
  } else {
    const dim3 grid = decode_grid(shape, pl);
    snprintf(text, text_bytes, "bc::decode_valu_kernel<%s, %d, %d, 8, %s, %s> grid=(%u,%u,%u) threads=256 chunks=%d%s",
             shape->kv_dtype == BC_BF16 ? "bc::bf16_t" : "float", shape->d, pl.Gp, pl.max_chunks > 1 ? "true" : "false",
             pl.fma ? "true" : "false", grid.x, grid.y, grid.z, pl.max_chunks, merged);
  }
  return BC_OK;
}

extern "C" int32_t bc_decode_attn(const bc_shape* shape, const bc_cache* cache, const void* q,
                                  float* out, const uint8_t* active, void* workspace,
                                  size_t workspace_bytes, void* stream) {
  DecodePlan pl;
  const int32_t st = check_attention_args(shape, cache, q, out, workspace, workspace_bytes, &pl, true);
  if (st != BC_OK) return st;
  return launch_attention(shape, cache, pl, q, out, active, workspace, workspace_bytes, nullptr, nullptr, nullptr,
                          nullptr, as_stream(stream));
}

// bc_decode_step behind its argument checks (shared with the allocation-free form)
static int32_t decode_step_checked(const bc_shape* shape, const bc_cache* cache, const DecodePlan& pl,
                                   const void* k, const void* v, const void* q, float* out,
                                   const void* beacon_k, const void* beacon_v, const uint8_t* active,
                                   void* workspace, size_t workspace_bytes, void* stream) {
  if (!k || !v || !aligned16(k) || !aligned16(v)) return BC_ERR_ARG;
  if ((beacon_k == nullptr) != (beacon_v == nullptr)) return BC_ERR_ARG;
  if (beacon_k && (!aligned16(beacon_k) || !aligned16(beacon_v))) return BC_ERR_ARG;
  // one launch, whichever kernel serves the shape: append, attention and eviction fused
  return launch_attention(shape, cache, pl, q, out, active, workspace, workspace_bytes, k, v, beacon_k, beacon_v,
                          as_stream(stream));
}

extern "C" int32_t bc_decode_step(const bc_shape* shape, const bc_cache* cache, const void* k,
                                  const void* v, const void* q, float* out, const void* beacon_k,
                                  const void* beacon_v, const uint8_t* active, void* workspace,
                                  size_t workspace_bytes, void* stream) {
  DecodePlan pl;
  const int32_t st = check_attention_args(shape, cache, q, out, workspace, workspace_bytes, &pl);
  if (st != BC_OK) return st;
  return decode_step_checked(shape, cache, pl, k, v, q, out, beacon_k, beacon_v, active, workspace, workspace_bytes,
                             stream);
}

// ---------------------------------------------------------------------------
// bc_decode_step for callers that cannot allocate: the workspace is a fixed array in device memory
// ---------------------------------------------------------------------------
namespace bc {
// BC_NOALLOC_SCRATCH_BYTES of counters and results, and what the padding of the partials to whole lines adds.
constexpr size_t kScratchBytes = BC_NOALLOC_SCRATCH_BYTES / 2 * 3;
static_assert(2 * (64 + kPartTail) <= 3 * (64 + 2), "the padding of a partial, at most that of one head with d = 64");
// One copy per GPU the library runs on, at an address of its own, held until the process ends.
// (In host code the array's name is only a handle: its device address comes from
// hipGetSymbolAddress, once per device, below.)
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

static int32_t scratch_of_current_device(unsigned char** ptr) {
  static unsigned char* address[64];
  static std::atomic<bool> known[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return BC_ERR_HIP;
  if (!known[dev].load(std::memory_order_acquire)) {
    void* a = nullptr;
    if (hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)) != hipSuccess || a == nullptr) return BC_ERR_HIP;
    address[dev] = static_cast<unsigned char*>(a);      // (two threads racing here store the same value)
    known[dev].store(true, std::memory_order_release);
  }
  *ptr = address[dev];
  return BC_OK;
}
}  // namespace bc

extern "C" int32_t bc_decode_step_noalloc(const bc_shape* shape, const bc_cache* cache, const void* k,
                                          const void* v, const void* q, float* out, const void* beacon_k,
                                          const void* beacon_v, const uint8_t* active, void* stream) {
  // the checks of bc_decode_step (the workspace is checked below, against the scratch array)
  DecodePlan pl;
  int32_t st = check_attention_args(shape, cache, q, out, reinterpret_cast<void*>(uintptr_t(256)), SIZE_MAX, &pl);
  if (st != BC_OK) return st;
  if (!k || !v || !aligned16(k) || !aligned16(v)) return BC_ERR_ARG;
  if ((beacon_k == nullptr) != (beacon_v == nullptr)) return BC_ERR_ARG;
  if (beacon_k && (!aligned16(beacon_k) || !aligned16(beacon_v))) return BC_ERR_ARG;
  // What this call's plan may touch: the per-sequence counters and, when sequences are cut into chunks, a counter
  // and the results (o, maximum, denominator) of every pair, without the padding the array has its other half
  // for.  (The automatic plan cuts at most 256 pairs into 512 chunks together: some 2 MB.)
  size_t need = pl.tickets_bytes;
  if (pl.max_chunks > 1) {
    const size_t pairs = (size_t)shape->B * shape->Hkv, heads = pairs * pl.max_chunks * pl.Gp;
    need += align256(pairs * 4) + align256(heads * shape->d * 4) + align256(heads * 2 * 4);
  }
  if (need > BC_NOALLOC_SCRATCH_BYTES) return BC_ERR_WORKSPACE;
  unsigned char* ws = nullptr;
  st = scratch_of_current_device(&ws);
  if (st != BC_OK) return st;
  // Every call on this GPU shares the array and finds what the last one left: the counters must
  // start at zero (a fill kernel, not a memset node: callers may be capturing a graph).
  const int64_t n = (int64_t)(pl.tickets_bytes / 4);
  const int64_t blocks = (n + 255) / 256;
  fill_zero_kernel<<<(int)(blocks < 1024 ? blocks : 1024), 256, 0, as_stream(stream)>>>(
      reinterpret_cast<uint32_t*>(ws), n);
  st = launch_status();
  if (st != BC_OK) return st;
  return decode_step_checked(shape, cache, pl, k, v, q, out, beacon_k, beacon_v, active, ws, kScratchBytes, stream);
}

extern "C" int32_t bc_beacon_step(const bc_shape* shape, const bc_cache* cache, const void* k,
                                  const void* v, const void* q, float* out, const uint8_t* active,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  DecodePlan pl;
  int32_t st = check_attention_args(shape, cache, q, out, workspace, workspace_bytes, &pl);
  if (st != BC_OK) return st;
  if (!k || !v || !aligned16(k) || !aligned16(v)) return BC_ERR_ARG;
  // one launch: beacon row at the tail, its attention, compaction
  return launch_attention(shape, cache, pl, q, out, active, workspace, workspace_bytes, k, v, k, v,
                          as_stream(stream), nullptr, nullptr, true);
}

extern "C" int32_t bc_decode_step_budget(const bc_shape* shape, const bc_cache* cache, const void* k,
                                         const void* v, const void* q, float* out,
                                         const void* beacon_k, const void* beacon_v,
                                         const int32_t* budget, uint8_t* live, void* workspace,
                                         size_t workspace_bytes, void* stream) {
  DecodePlan pl;
  int32_t st = check_attention_args(shape, cache, q, out, workspace, workspace_bytes, &pl);
  if (st != BC_OK) return st;
  if (!k || !v || !aligned16(k) || !aligned16(v) || !budget || !live) return BC_ERR_ARG;
  if ((beacon_k == nullptr) != (beacon_v == nullptr)) return BC_ERR_ARG;
  if (beacon_k && (!aligned16(beacon_k) || !aligned16(beacon_v))) return BC_ERR_ARG;
  // The cap is tested on the state the attention saw (before the eviction); the holder of the
  // sequence's last ticket clears the mask after the eviction has used it.
  return launch_attention(shape, cache, pl, q, out, live, workspace, workspace_bytes, k, v, beacon_k, beacon_v,
                          as_stream(stream), budget, live);
}

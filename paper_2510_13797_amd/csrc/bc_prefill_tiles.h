// What the kernels of the masked attention share: the compacted key list of a query tile, the
// visibility of a tile's keys as bits, tiles of 32 rows staged in LDS in the order the matrix
// operands are read, and the operand and result helpers of the 32x32x16 matrix instructions.
#pragma once
#include <cstddef>
#include <type_traits>

#include "bc_common.h"
#include "bc_prefill_grid.h"

namespace bc {

constexpr int kTileStages = 3;        // tiles in LDS: one in use, two on their way

typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(8))) short s16x8_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

// ---------------------------------------------------------------------------
// tables of the trajectories
// ---------------------------------------------------------------------------
// In device memory or, from the calls that take them as host arrays, for up to BC_INLINE_TRAJECTORIES trajectories in the kernel
// arguments (a launch in front that stored them took 3 us a call, 10 % of a small forward and backward pass).  Sixteen are 400 bytes of
// them; 4 KB would hold some 240.  (128 inline, trajectories of some 200 rows, 4/1 heads, forward and gradients: 3 and 16 trajectories 43.0 and
// 45.5 us with either, 17 52.2 through memory and 48.1 inline, 40 61.3 and 56.6, 100 102.5 and 98.8.)
struct InlineTables {
  int64_t row_off[BC_INLINE_TRAJECTORIES + 1];
  int32_t P[BC_INLINE_TRAJECTORIES], c[BC_INLINE_TRAJECTORIES];
};
struct Trajectory { int64_t off0; int rows, P, c; };
// Params: the only argument of the kernel, with row_off (null: inline), P, c and tab.
template <typename Params>
__device__ __forceinline__ Trajectory trajectory(const Params& p, int b) {
  Trajectory t;
  int64_t end;
  if (p.row_off != nullptr) {
    t.off0 = p.row_off[b]; end = p.row_off[b + 1]; t.P = p.P[b]; t.c = p.c[b];
  } else {
    typedef __attribute__((address_space(4))) const char const_char_t;
    typedef __attribute__((address_space(4))) const InlineTables const_tables_t;
    const_tables_t* in = (const_tables_t*)((const_char_t*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(Params, tab));
    t.off0 = in->row_off[b]; end = in->row_off[b + 1]; t.P = in->P[b]; t.c = in->c[b];
  }
  t.rows = (int)(end - t.off0);
  return t;
}
// Host arrays -> p; tables: device memory for more trajectories than fit.
template <typename Params>
int32_t host_tables(Params& p, const int64_t* row_offsets, const int32_t* P, const int32_t* c, int32_t B, void* tables,
                    void* stream) {
  if (B <= BC_INLINE_TRAJECTORIES) {
    p.row_off = nullptr; p.P = nullptr; p.c = nullptr;
    for (int b = 0; b < B; ++b) { p.tab.row_off[b] = row_offsets[b]; p.tab.P[b] = P[b]; p.tab.c[b] = c[b]; }
    p.tab.row_off[B] = row_offsets[B];
    return BC_OK;
  }
  const int32_t st = bc_trajectory_tables(row_offsets, P, c, B, tables, stream);
  p.row_off = static_cast<const int64_t*>(tables);
  p.P = reinterpret_cast<const int32_t*>(p.row_off + B + 1);
  p.c = p.P + B;
  return st;
}

// ---------------------------------------------------------------------------
// key list of a query tile
// ---------------------------------------------------------------------------
// The keys of a query tile as a list of entries in tiles of 32: the full tiles of run A and of run B
// (nothing masked: tiles 0 .. dense-1), then the tail: what is left of A, what is left of B and the
// band, back to back (each padded to whole tiles on its own: 7 % more matrix instructions on
// trajectories of 8688 rows).
struct KeyRuns {
  WindowStride ws;
  int P, band_start, FA, dense, tA, tAB, nT, NT;
  __device__ __forceinline__ KeyRuns(const WindowStride& w, int prompt, int r0, int r1) : ws(w), P(prompt) {
    int nA = 0, nB = 0;
    band_start = 0;
    if (ws.c > 0 && r0 >= P) {
      const int m0 = (int)window_of(ws, (uint32_t)(r0 - P));
      nA = P; nB = m0; band_start = P + m0 * ws.stride;
    }
    FA = nA / kTileRows;
    dense = FA + nB / kTileRows;
    tA = nA % kTileRows;
    tAB = tA + nB % kTileRows;
    nT = tAB + r1 - band_start + 1;
    NT = dense + (nT + kTileRows - 1) / kTileRows;
  }
  // row of entry y of the tail
  __device__ __forceinline__ int tail_row(int y) const {
    if (y >= tAB) return band_start + y - tAB;
    return y < tA ? FA * kTileRows + y : P + ((dense - FA) * kTileRows + y - tA) * ws.stride + ws.c;
  }
  // tiles that hold anything row `last` or an earlier one may see
  __device__ __forceinline__ int tiles_up_to(int last) const {
    return dense + (last - band_start + tAB) / kTileRows + 1;
  }
  // first row of the window row r lies in (prompt rows: of no use, every key they see is below P)
  __device__ __forceinline__ int window_start(int r) const {
    return ws.c > 0 && r >= P ? P + (int)window_of(ws, (uint32_t)(r - P)) * ws.stride : 0x7fffffff;
  }
  // Bit x: row r may see entry y0 + x of the tail (y0 a multiple of 32).  A key of the band is seen by
  // every later row if it is a prompt row or a beacon (a property of the key alone: lane x works out
  // key x, one vote gives the tile's word) and otherwise from its own window on, i.e. if it is not
  // before r's window.  `own`: window_start(r).
  __device__ __forceinline__ uint32_t visible(int y0, int r, int own, int lane) const {
    const int y = y0 + (lane & 31), j = band_start + y - tAB;
    bool everyone = y < tAB || j < P || ws.c <= 0;
    if (!everyone) {
      const uint32_t u = (uint32_t)(j - P);
      everyone = (int)(u - window_of(ws, u) * (uint32_t)ws.stride) == ws.c;
    }
    const uint32_t dense_bits = (uint32_t)__builtin_amdgcn_ballot_w64(everyone);
    const int base = band_start - tAB + y0;             // row of entry y0, were it of the band
    const int from = own - base, upto = r - base;
    const uint32_t mine = from >= 32 ? 0u : ~0u << max(from, 0);
    const uint32_t past = upto < 0 ? 0u : upto >= 31 ? ~0u : (2u << upto) - 1u;
    return (dense_bits | mine) & past;                  // (entries that do not exist lie behind r)
  }
};

// What the loads of a tile need: byte offset of entry 0 from the (trajectory, KV head) base, bytes
// from entry to entry, entries that exist (32 or more: all); or mixed >= 0: the tile holds the tail's
// entries from that one on, rows of different runs, and off is 0 (they may lie before the band).
struct TileLoad { int64_t off; int64_t step; int nvalid, mixed; };

// The tiles of KeyRuns in order, as loads.  Kept as a cursor with constant increments inside a run:
// working the offsets out anew from the tile number took some 70 scalar instructions and ten
// branches per tile, which a wave issues one after the other between its matrix instructions.
struct TileCursor {
  int64_t row_bytes, off, step;
  int left, seg, y;
  __device__ __forceinline__ TileCursor(const KeyRuns& r, int64_t rb) : row_bytes(rb), seg(-1) { left = 1; next_segment(r); }
  __device__ __forceinline__ void next_segment(const KeyRuns& r) {
    do {
      ++seg;
      y = 0;
      if (seg == 0) { left = r.FA; off = 0; step = row_bytes; }
      else if (seg == 1) { left = r.dense - r.FA; off = (int64_t)(r.P + r.ws.c) * row_bytes; step = r.ws.stride * row_bytes; }
      else { left = 0x7fffffff; off = ((int64_t)r.band_start - r.tAB) * row_bytes; step = row_bytes; }
    } while (left == 0);
  }
  __device__ __forceinline__ TileLoad next(const KeyRuns& r) {
    const bool mixed = seg == 2 && y < r.tAB;
    const TileLoad t{mixed ? 0 : off, step, seg == 2 ? r.nT - y : kTileRows, mixed ? y : -1};
    off += step * kTileRows;
    y += kTileRows;
    if (__builtin_expect(--left == 0, 0)) next_segment(r);
    return t;
  }
};

// Element e of a lane's 16 results of a 32x32 product is row 8*(e/4) + 4*(lane/32) + e%4 of the tile;
// `see` is the visibility word shifted right by 4*(lane/32).
__device__ __forceinline__ bool visible_bit(uint32_t see, int e) { return (see >> (8 * (e >> 2) + (e & 3))) & 1u; }
__device__ __forceinline__ float keep_if_visible(float x, uint32_t see, int e) {
  const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)see, 8 * (e >> 2) + (e & 3), 1);
  return __uint_as_float(__float_as_uint(x) & m);
}

// ---------------------------------------------------------------------------
// tiles in LDS
// ---------------------------------------------------------------------------
// A tile of 32 rows of D bf16 is staged as blocks of 8 rows x 8 units (16 bytes each): 1 KB, one
// LDS-DMA instruction that reads 128 consecutive bytes of each of 8 rows.  Block (rg, uh) holds rows
// 8*rg.. and units 8*uh..; it lies at (4*uh + rg) KB.  Inside a block the units stand in one of two
// orders, chosen so that the addresses of all operands of a tile are one register per lane plus
// constants, and that no read has a bank conflict (a 128-bit read is served in groups of 16 lanes -
// {0-3, 12-15, 20-27} and {4-11, 16-19, 28-31} of each half wave - that must cover the 64 banks; a
// transposing 64-bit read in half waves).
//
// Row order (operand "rows of the tile": lane l takes row l%32, head-dim elements 16*i + 8*(l/32)..):
// unit u of row y at 16-byte slot (u%8/2)*16 + ((y%8)*2 + u%2 ^ rg/2).
// Measured: 245 bytes per clock and CU, what linear addresses reach; the XOR swizzle of 256-byte rows
// used before (rows {a + 8b} of one unit apart) ran at 126: its lanes 0-3, 12-15, 20-27 met in pairs.
//
// Column order (operand "tile transposed": lane l takes head-dim column 32*j + l%32 and the tile
// rows its results e = 8*s.. of a product over the tile stand for): unit u of row y at slot
// (u%8/4)*32 + (y%8)*4 + u%4.
// What a lane of wave rg moves: the wave brings the blocks of row group rg, one instruction for each
// 128 bytes of the row.
struct TileLane { int row; uint32_t in_row; };       // row of the tile, byte offset inside the 128

__device__ __forceinline__ TileLane rows_tile_lane(int lane, int rg) {
  return TileLane{8 * rg + ((lane & 15) >> 1), (uint32_t)(2 * (lane >> 4) + ((lane & 1) ^ (rg >> 1))) << 4};
}
__device__ __forceinline__ TileLane cols_tile_lane(int lane, int rg) {
  return TileLane{8 * rg + ((lane & 31) >> 2), (uint32_t)(4 * (lane >> 5) + (lane & 3)) << 4};
}
__device__ __forceinline__ int rows_read_offset(int lane) {
  const int y = lane & 31, rg = y >> 3;
  return rg * 1024 + ((((y & 7) * 2 + (lane >> 5)) ^ (rg >> 1)) << 4);
}
template <int D> constexpr int rows_read_imm(int i) { return (i >> 2) * 4096 + (i & 3) * 256; }
__device__ __forceinline__ int cols_read_offset(int lane) {
  const int rl = lane & 15;
  return (((4 * (lane >> 5) + (rl >> 2)) * 4 + 2 * ((lane >> 4) & 1) + ((rl & 3) >> 1)) << 4) + ((rl & 1) << 3);
}
// base: tile + cols_read_offset(lane)
template <int D>
__device__ __forceinline__ bf16x8_t cols_operand(const char* base, int j, int s) {
  const char* a = base + (j >> 1) * 4096 + (j & 1) * 512 + 2 * s * 1024;
  const s16x4_t a0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)a);
  const s16x4_t a1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(a + 1024));
  return __builtin_bit_cast(bf16x8_t, (s16x8_t)__builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Either order (a tile read both ways, the backward's): unit u of row y at slot
// (u%8/2)*16 + ((y%8)*2 + u%2 ^ rg/2 ^ 8*(u/2%2)): the row order with bit 3 flipped for every second pair of
// units, so that the transposing reads of a half wave, 16 lanes in each of two neighbouring pairs, cover the
// 64 banks once.
__device__ __forceinline__ TileLane either_tile_lane(int lane, int rg) {
  const int t = (lane & 15) ^ ((lane >> 1) & 8);
  return TileLane{8 * rg + (t >> 1), (uint32_t)(2 * (lane >> 4) + ((t & 1) ^ (rg >> 1))) << 4};
}
// row operand i: tile + either_rows_offset(lane) ^ 128 * (i % 2), + rows_read_imm<D>(i)
__device__ __forceinline__ int either_rows_offset(int lane) { return rows_read_offset(lane); }
// column operand (j, s): tile + either_cols_offset(lane, s), as cols_operand takes it
__device__ __forceinline__ int either_cols_offset(int lane, int s) {
  const int rl = lane & 15, odd = (lane >> 4) & 1;
  return odd * 256 + (((8 * (lane >> 5) + 2 * (rl >> 2) + ((rl & 3) >> 1)) ^ s ^ (8 * odd)) << 4) + ((rl & 1) << 3);
}

// The lane's byte offset from the tile's base; entries that do not exist repeat the first one (what is
// computed from them is masked).  WIDE: a trajectory's rows may span 4 GB or more.
template <bool WIDE>
__device__ __forceinline__ std::conditional_t<WIDE, int64_t, uint32_t> tile_lane_offset(const KeyRuns& runs, const TileLoad& t,
                                                                                        const TileLane& ln, int64_t row_bytes) {
  using OFF = std::conditional_t<WIDE, int64_t, uint32_t>;
  const int e = ln.row < t.nvalid ? ln.row : 0;
  if (t.mixed >= 0) return (OFF)runs.tail_row(t.mixed + e) * (OFF)row_bytes + ln.in_row;      // (t.off is 0)
  return (OFF)e * (OFF)t.step + ln.in_row;
}
// HBM -> LDS: one block, 1 KB
template <bool WIDE, typename OFF>
__device__ __forceinline__ void issue_block(const char* tile_base, OFF lane_offset, uint32_t lds_addr) {
  if constexpr (!WIDE) {       // scalar base, 32-bit offset per lane
    lds_dma16_s<false>(lane_offset, (uint64_t)tile_base, lds_addr);
  } else {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 : : "s"(lds_addr), "v"(tile_base + lane_offset) : "memory");
  }
}

// A wave's own 32 rows (row `last` repeated behind it) into a tile of its own in LDS, from where they are read as operands.
// Loaded straight into the operands' registers, 16 bytes of 32 rows at a time, they took most of a workgroup's time
// before its first product: with dO and the output 16,000 cycles of an idle chip, 12,000 with whole rows.
template <int D>
__device__ __forceinline__ void issue_wave_rows(const char* first, uint32_t row_bytes, int last, int lane, uint32_t lds_addr) {
#pragma unroll
  for (int rg = 0; rg < kTileRows / 8; ++rg) {
    const TileLane t = rows_tile_lane(lane, rg);
    const uint32_t o = (uint32_t)min(t.row, last) * row_bytes + t.in_row;
#pragma unroll
    for (int n = 0; n < D / 64; ++n) issue_block<false>(first + 128 * n, o, lds_addr + n * 4096 + rg * 1024);
  }
}
template <int D>
__device__ __forceinline__ void read_wave_rows(const char* tile, int lane, bf16x8_t (&x)[D / 16]) {
  const char* a = tile + rows_read_offset(lane);
#pragma unroll
  for (int i = 0; i < D / 16; ++i) x[i] = *reinterpret_cast<const bf16x8_t*>(a + rows_read_imm<D>(i));
}

// The point by which operands loaded before a tile loop have landed: the compiler waits here and not
// in front of their first use inside the loop, where the wait would cover the tiles' loads too.
template <int N>
__device__ __forceinline__ void landed_operands(bf16x8_t (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
}
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
// Workgroup barrier for LDS traffic whose loads the compiler does not count: no implied wait.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---------------------------------------------------------------------------
// values
// ---------------------------------------------------------------------------
// all-reduce over the two halves of a wave (lane l with l ^ 32)
__device__ __forceinline__ float halves_max(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float halves_sum(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// A lane's 16 values of a 32x32 product as the two bf16 parts (to 16 bits together) of the operands of the next one, pair by pair, so
// that the work spreads over other instructions.  The remainder x - h is exact.  (By the bf16 dot product, one instruction instead of two,
// the decode kernels' way, each of the sixteen of a tile held up the matrix pipe by some eight cycles: a loop of 32x32x16 products with one
// beside each ran at 78 % of the pipe, with four FMA at 90 %.  16 trajectories of 8688 rows: dkv 22.5 -> 20.4 million cycles,
// dq 15.8 -> 15.2, forward 10.0 -> 9.6.)
struct Parts {
  uint32_t h[8], l[8];
  __device__ __forceinline__ void split(int n, float a, float b) {
    h[n] = pack2_bf16(a, b);
    l[n] = pack2_bf16(a - __uint_as_float(h[n] << 16), b - __uint_as_float(h[n] & 0xffff0000u));
    asm volatile("" : "+v"(h[n]), "+v"(l[n]));        // (worked out here and not where they are used)
  }
  __device__ __forceinline__ bf16x8_t operand(int part, int k) const {       // values 8 * k ..
    const uint32_t* w = (part ? l : h) + 4 * k;
    return __builtin_bit_cast(bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
  }
};
// Between two steps of code whose order is written out.
__device__ __forceinline__ void step_fence() { __builtin_amdgcn_sched_barrier(0); }

// Half the columns (pass 0 or 1) of a wave's 32 x D results (accumulator layout: lane l holds
// columns 32*j + 8*i + 4*(l/32) .. +3 of row l%32) -> LDS -> bursts of D/2 floats per row.
// row(t): which row of `base` row t goes to, or -1.  Written once, not read again by the launch: streaming.
template <int D, typename F>
__device__ __forceinline__ void store_rows(float* my, const f32x16_t (&acc)[D / 32], float mul, int pass, int lane,
                                           float* base, int row_stride, F row) {
  constexpr int OW = D / 2, UW = OW / 4, RPP = 64 / UW;      // columns and units of a pass, rows per instruction
  const int y = lane & 31, half = lane >> 5;
#pragma unroll
  for (int jb = 0; jb < D / 64; ++jb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x16_t& a = acc[(D / 64) * pass + jb];
      *reinterpret_cast<f32x4_t*>(my + y * OW + (((8 * jb + 2 * i + half) ^ (y & (UW - 1))) << 2)) =
          f32x4_t{a[4 * i] * mul, a[4 * i + 1] * mul, a[4 * i + 2] * mul, a[4 * i + 3] * mul};
    }
  // All reads, then all stores: each read stood behind a store that it might alias and a branch, and a workgroup's end took
  // 5,000 to 6,000 cycles (three short trajectories 72.8 -> 71.1 us a pass; 16 of 8688 rows 3293 -> 3281, little more than two runs differ by).
  f32x4_t val[32 / RPP];
  int to[32 / RPP];
#pragma unroll
  for (int n = 0; n < 32 / RPP; ++n) {
    const int t = RPP * n + lane / UW, unit = lane & (UW - 1);
    val[n] = *reinterpret_cast<const f32x4_t*>(my + t * OW + ((unit ^ (t & (UW - 1))) << 2));
    to[n] = row(t);
  }
  float* at = base + OW * pass + (lane & (UW - 1)) * 4;
#pragma unroll
  for (int n = 0; n < 32 / RPP; ++n)
    if (to[n] >= 0) __builtin_nontemporal_store(val[n], reinterpret_cast<f32x4_t*>(at + (int64_t)to[n] * row_stride));
}

// Whether byte offsets inside a trajectory's K or V rows may need more than 32 bits.
inline bool rows_span_4gb(int32_t max_rows, const bc_shape* sh) {
  return (uint64_t)max_rows * (uint64_t)sh->Hkv * (uint64_t)(sh->d * 2) >= 0x100000000ull;
}

}  // namespace bc

// bc_prefill_attn_bwd: gradients of the beacon-masked prefill attention (Fig. 2, Sec. 3.2 of the
// paper: training runs the masked forward in parallel and differentiates through it).
//
// With S = scale*Q.K^T on the visible pairs, A = softmax(S), O = A.V and upstream dO:
//   Delta_r = sum_x dO[r,x]*O[r,x]        dV = A^T.dO        dA = dO.V^T
//   dS = A*(dA - Delta)                   dQ = scale*dS.K    dK = scale*dS^T.Q
// A is recomputed from the saved log-sum-exp.  Two kernels, both on the compacted structure of
// the mask, no atomics (results are reproducible), plus a small fixed-order reduction:
//
//  dq kernel   the forward's walk with the forward's workgroups: four waves, each 32 query rows of
//              one head, over prompt run, gathered beacon run and masked band.  Also writes
//              (lse*log2e, Delta) per row, head-major, for the second kernel.
//              (Small launches: a kernel of its own does that, and the workgroups of both kernels are one launch.)
//  dkv kernel  one workgroup = 64 keys of one KV head; three kinds of key block:
//                prompt keys      -> stream every later row of every head of the group (dense)
//                gathered beacons -> the same, from the first beacon's row on (dense)
//                response tokens  -> only the rows up to the end of their window (masked band)
//              so the dense part of the work is spent on the ~P + S/(c+1) keys every row sees.
//              A dense block is long (every later row x every head); it is cut into parts (see
//              dense_parts()), which write partial dK/dV to the workspace, and a third kernel adds
//              them in a fixed order.  Response blocks are cut only where the chip is not full (band_splits)
//              and store their result directly otherwise.
//
// All contractions are 32x32x16 bf16 MFMA; A and dS are split into two bf16 parts before they
// enter a product (their rounding would otherwise dominate the error); tiles of 32 rows are gathered
// into LDS by 16-byte LDS-DMA loads, in the order that serves row and column operands alike
// (bc_prefill_tiles.h).
//
// What bounds both: the card's power limit on large launches, the chain of a tile's steps on small ones.  On 16 trajectories of 8688
// rows (12/2 heads, d = 128) the dkv kernel issues 1458 GFLOP of MFMA work in 1.52 ms, the dq kernel 947 in 1.06 (averages under the profiler; both with the
// matrix pipe 55 to 58 % busy at 1.75 to 1.8 GHz; a loop of such products alone runs at 1.75 PFLOP/s and 1.75 GHz, with the operand reads and
// vector work of the dq kernel at 1.3): fewer cycles give a lower clock and half of what they should.  The forms before, 16x16x32
// MFMA with 16 rows of two heads or 16 keys per wave and tiles read at half rate by bank conflicts, took 1.24 and 1.83 ms.
// A forward and backward pass of that batch takes 3100 to 3210 us (cards differ by 3 %), of three trajectories of 336 to 795 rows 52.
#include "bc_prefill_tiles.h"

namespace bc {

struct BwdParams {
  const char* q;
  const char* k;
  const char* v;
  const float* out;
  const float* lse;
  const char* dout;
  const int64_t* row_off;
  const int32_t* P;
  const int32_t* c;
  float* dq;
  float* dk;
  float* dv;
  float* stat;          // [Hq][total_rows][2]: lse*log2(e), -Delta
  float* part;          // splits * 2 * total_rows rows [Hkv][D]: partial dk, dv (see KeyParts)
  int32_t D;            // head dimension (the reduction kernel reads it; the others are templates)
  int32_t splits;       // rows of partial sums there is room for, per row, of dk and of dv
  int32_t most;         // most workgroups that share a dense key block
  int32_t band;         // workgroups that share a response block (see band_splits), at most `splits`
  int32_t least;        // tiles of one of more than `splits` parts
  int64_t total_rows;
  int32_t Hq, Hkv, g;
  HeadTiling tiling;    // dq kernel
  int32_t dq_rows;      // rows of its grid
  int32_t npairs;       // (trajectory, KV head) pairs
  int32_t pstride;      // see pair_stride()
  int32_t turn;         // see pair_turn()
  float scale;
  float qscale;         // scale * log2(e)
  InlineTables tab;
};

#define BC_INLINE __attribute__((always_inline))      // lambdas: their captures stay in registers

// ---------------------------------------------------------------------------
// dq kernel
// ---------------------------------------------------------------------------
// The forward's walk with the same workgroups: four waves, 32 query rows of one head each.  Its registers let two
// workgroups share a compute unit, so there is LDS for five tiles - one by columns, the next by rows, two on their way and one
// that is asked for - (the forward loses its third workgroup to a fourth: 0.70 -> 0.81 ms) and, before
// the walk, for the rows of all waves: with those through LDS and Delta from whole rows a pass of three short
// trajectories takes 72.8 us instead of 75.4.  What is left in front of the first product, some 10,000 cycles, is
// mostly the first touch of the output's rows.
// A third workgroup fits at d = 64 (16 trajectories of 7200 to 8700 rows, 14/2 heads: 623 -> 605 us with the passes below).
constexpr int kDqStages = 5;

// Delta of a row: sixteen lanes with four of every 64 columns each, the same in all of them.
template <int D>
__device__ __forceinline__ float row_dot(const float4 (&o)[D / 64], const uint2 (&y)[D / 64]) {
  float sum = 0.f;
#pragma unroll
  for (int t = 0; t < D / 64; ++t)
    sum += __uint_as_float(y[t].x << 16) * o[t].x + __uint_as_float(y[t].x & 0xffff0000u) * o[t].y +
           __uint_as_float(y[t].y << 16) * o[t].z + __uint_as_float(y[t].y & 0xffff0000u) * o[t].w;
  return group_allreduce_sum<16>(sum);
}
template <int D> constexpr int dq_lds() {
  constexpr int TILE = kTileRows * D * 2, RING = kDqStages * 2 * TILE, ROWS = (2 + 2 * kTileWaves) * TILE;
  return RING > ROWS ? RING : ROWS;
}
// Rows of a workgroup by, heads hh of the group; at_x and the launch's row of the grid give the pair.  JOINED: log-sum-exp and
// Delta are in the workspace.
template <int D, bool WIDE, bool JOINED>
__device__ __forceinline__ void dq_block(const BwdParams& p, char* lds, int at_x, int hh, int by, int ny) {
  constexpr int ROWB = D * 2, KS = D / 16, NJ = D / 32, TILE = kTileRows * ROWB;
  constexpr int NLD = TILE / 1024 / kTileWaves;     // LDS-DMA instructions per wave, tile and tensor
  constexpr int LOOK = kDqStages - 2;
  static_assert(LOOK == 3, "the counts of begin_pass");
  static_assert(dq_lds<D>() >= kTileWaves * 32 * (D / 2) * 4, "the gradient tiles fit the ring's LDS");

  const int pair = pair_in_turn(at_x, p.pstride, p.turn, blockIdx.y);
  if (pair >= p.npairs) return;
  const int kvh = pair % p.Hkv, b = pair / p.Hkv;
  const Trajectory traj = trajectory(p, b);
  const int64_t off0 = traj.off0;
  const int S = traj.rows;
  const int rows_wg = kTileRows * p.tiling.row_blocks;
  const int r0 = (ny - 1 - by) * rows_wg;        // long tiles first
  if (r0 >= S) return;
  const int r1 = min(r0 + rows_wg - 1, S - 1);
  const WindowStride ws = window_stride(traj.c, S);
  const KeyRuns runs(ws, traj.P, r0, r1);
  const int NT = runs.NT;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int wb = wave / p.tiling.heads;                         // row block and head of this wave
  const int head = hh * p.tiling.heads + (wave - wb * p.tiling.heads);
  const int rw0 = r0 + kTileRows * wb;
  const int rw1 = min(rw0 + kTileRows - 1, r1);
  const int ntw = head < p.g && rw0 <= r1 ? runs.tiles_up_to(rw1) : 0;

  const int64_t kv_row_bytes = (int64_t)p.Hkv * ROWB;
  const char* kbase = p.k + (off0 * p.Hkv + kvh) * ROWB;
  const char* vbase = p.v + (off0 * p.Hkv + kvh) * ROWB;
  const uint32_t lds0 = lds_address(lds) + wave * 1024;
  const TileLane tlane = either_tile_lane(lane, wave);
  TileCursor cursor(runs, kv_row_bytes);
  auto issue_tile = [&](int stage) BC_INLINE {
    const TileLoad t = cursor.next(runs);
    const auto o = tile_lane_offset<WIDE>(runs, t, tlane, kv_row_bytes);
#pragma unroll
    for (int n = 0; n < NLD; ++n) {           // (128 bytes further on in each row)
      issue_block<WIDE>(kbase + t.off + 128 * n, o, lds0 + stage * (2 * TILE) + n * 4096);
      issue_block<WIDE>(vbase + t.off + 128 * n, o, lds0 + stage * (2 * TILE) + TILE + n * 4096);
    }
  };
  issue_tile(0);

  // Q and dO of the wave's rows, into the LDS behind the first tile
  const int r = min(rw0 + col, r1), rw = min(rw0, r1);
  const int64_t first = (off0 + rw) * p.Hq + kvh * p.g + min(head, p.g - 1);
  issue_wave_rows<D>(p.q + first * ROWB, (uint32_t)p.Hq * ROWB, r1 - rw, lane, lds_address(lds) + (2 + 2 * wave) * TILE);
  issue_wave_rows<D>(p.dout + first * ROWB, (uint32_t)p.Hq * ROWB, r1 - rw, lane, lds_address(lds) + (3 + 2 * wave) * TILE);
  // Delta: sixteen lanes a row, four rows at a time
  float part[8];
  if constexpr (!JOINED) {
    float4 o[8][D / 64];
    uint2 y[8][D / 64];
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const uint32_t e = (uint32_t)min(4 * n + (lane >> 4), r1 - rw) * (uint32_t)(p.Hq * D) + 4 * (lane & 15);
#pragma unroll
      for (int t = 0; t < D / 64; ++t) {
        o[n][t] = *reinterpret_cast<const float4*>(p.out + first * D + e + 64 * t);
        y[n][t] = *reinterpret_cast<const uint2*>(p.dout + first * ROWB + 2 * (uint64_t)(e + 64 * t));
      }
    }
#pragma unroll
    for (int n = 0; n < 8; ++n) part[n] = row_dot<D>(o[n], y[n]);
  }
  float lse2, delta;
  if constexpr (JOINED) {
    const float* stat = p.stat + ((int64_t)(kvh * p.g + min(head, p.g - 1)) * p.total_rows + off0 + r) * 2;
    lse2 = stat[0];
    delta = -stat[1];
  } else {
    lse2 = p.lse[(off0 + r) * p.Hq + kvh * p.g + min(head, p.g - 1)] * kLog2e;
  }
  // this lane's query row: Q^T and dO^T as B operands, log-sum-exp and Delta of the row
  char* mine = lds + (2 + 2 * wave) * TILE;
  bf16x8_t qb[KS], dob[KS];
  wait_vmcnt<0>();
  read_wave_rows<D>(mine, lane, qb);
  read_wave_rows<D>(mine + TILE, lane, dob);
  landed_operands(qb);
  landed_operands(dob);
  if constexpr (!JOINED) {
    asm volatile("" : : : "memory");      // (Delta's floats replace the operands' rows)
    float row_delta = part[0];
#pragma unroll
    for (int n = 1; n < 8; ++n) row_delta = (lane & 7) == n ? part[n] : row_delta;
    if ((lane & 8) == 0) reinterpret_cast<float*>(mine)[4 * (lane & 7) + (lane >> 4)] = row_delta;
    delta = reinterpret_cast<const float*>(mine)[col];
  }
  asm volatile("" : "+v"(delta), "+v"(lse2));
  lds_barrier();            // every wave has its rows
#pragma unroll
  for (int t = 1; t < LOOK; ++t)
    if (t < NT) issue_tile(t);
  const int own = runs.window_start(r);

  f32x16_t dQ[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) dQ[j] = f32x16_t{0.f};
  const int roff[2] = {either_rows_offset(lane), either_rows_offset(lane) ^ 128};
  const int coff[2] = {either_cols_offset(lane, 0), either_cols_offset(lane, 1)};

  // A pass forms dS of tile kt and adds the tile before it to dQ.  Its order is written out (step_fence(): nothing is moved across):
  // the split of the tile before stands beside the scores' matrix instructions, exponentials and dS beside dQ's, and LDS operands
  // are asked for several instructions ahead.  In one chain a tile - scores, dS, dQ - a wave left the matrix pipe idle for half of
  // its time, and the compiler, left to itself, asks for an operand in front of the instruction that takes it and puts all vector
  // work in one place (the same passes without the order: 1072 us as before).  16 trajectories of 8688 rows, 12/2 heads 1072 -> 1027 us
  // under the profiler, at the power limit 15.2 -> 14.1 million cycles; three short ones 18.4 -> 17.4.
  constexpr int SLOTS = 4 * NJ, PRE = 3;         // matrix instructions of a tile's dQ; steps that row operands are ahead
  float ds[16];
  Parts y;
  auto col_of = [&](const char* tile, int n) BC_INLINE { return cols_operand<D>(tile + coff[n / NJ], n % NJ, n / NJ); };
  auto step_dq = [&](const bf16x8_t& c, int m) BC_INLINE {        // dQ^T += K^T . dS^T: operand m / 2, part m % 2
    const int n = m / 2;
    dQ[n % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c, y.operand(m & 1, n / NJ), dQ[n % NJ], 0, 0, 0);
  };
  auto split = [&](int g) BC_INLINE { y.split(g, ds[2 * g], ds[2 * g + 1]); };
  int stage = 0;
  auto next_stage = [&]() BC_INLINE { stage = stage + 1 == kDqStages ? 0 : stage + 1; };
  auto begin_pass = [&](int kt) BC_INLINE {
    if (kt + 2 < NT) wait_vmcnt<4 * NLD>();         // (the loads of the next two tiles may stay out)
    else if (kt + 1 < NT) wait_vmcnt<2 * NLD>();
    else wait_vmcnt<0>();
    lds_barrier();
    // tile kt has landed, and everyone has finished tile kt - 2, whose stage is the one tile kt + LOOK goes into
    if (kt + LOOK < NT) issue_tile(stage >= 2 ? stage - 2 : stage + kDqStages - 2);
  };
  auto form_ds = [&](int kt, const char* tile, auto more, const char* before, auto masked) BC_INLINE {
    constexpr bool MORE = decltype(more)::value, MASKED = decltype(masked)::value;      // MORE: there is a tile before
    uint32_t see = ~0u;
    if constexpr (MASKED) see = runs.visible((kt - runs.dense) * kTileRows, r, own, lane) >> (4 * half);
    bf16x8_t rk[KS], rv[KS], c[2 * NJ];
    f32x16_t s = f32x16_t{0.f}, dp = f32x16_t{0.f};
    auto rows = [&](int i) BC_INLINE {
      const char* a = tile + roff[i & 1] + rows_read_imm<D>(i);
      rk[i] = *reinterpret_cast<const bf16x8_t*>(a);
      rv[i] = *reinterpret_cast<const bf16x8_t*>(a + TILE);
    };
#pragma unroll
    for (int i = 0; i < PRE; ++i) rows(i);
    step_fence();
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rk[i], qb[i], s, 0, 0, 0);
      if (i + PRE < KS) rows(i + PRE);
      if constexpr (MORE) {
#pragma unroll
        for (int g = i * 8 / KS; g < (i + 1) * 8 / KS; ++g) split(g);
      }
      step_fence();
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rv[i], dob[i], dp, 0, 0, 0);
      if (MORE && i >= KS - NJ) c[i - KS + NJ] = col_of(before, i - KS + NJ);
      step_fence();
    }
#pragma unroll
    for (int m = 0; m < SLOTS; ++m) {
      if constexpr (MORE) {
        step_dq(c[m / 2], m);
        if (m % 2 == 0 && m / 2 + NJ < 2 * NJ) c[m / 2 + NJ] = col_of(before, m / 2 + NJ);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e)               // (the scores are there behind the second instruction)
        if (m == 2 + e * (SLOTS - 3) / 15) {
          ds[e] = fast_exp2(fmaf(s[e], p.qscale, -lse2)) * (dp[e] - delta);
          if constexpr (MASKED) ds[e] = keep_if_visible(ds[e], see, e);
          asm volatile("" : "+v"(ds[e]));        // (worked out here and not behind the next barrier)
        }
      step_fence();
    }
  };

  begin_pass(0);
  int kt = 1;
  if (ntw > 0) {
    form_ds(0, lds, std::false_type{}, lds, std::true_type{});       // (the words of a dense tile have all bits set)
    auto pass = [&](auto masked) BC_INLINE {
      const char* before = lds + stage * (2 * TILE);
      next_stage();
      begin_pass(kt);
      form_ds(kt, lds + stage * (2 * TILE), std::true_type{}, before, masked);
    };
    for (const int nd = min(runs.dense, ntw); kt < nd; ++kt) pass(std::false_type{});
    for (; kt < ntw; ++kt) pass(std::true_type{});
#pragma unroll
    for (int g = 0; g < 8; ++g) split(g);
#pragma unroll
    for (int m = 0; m < SLOTS; ++m) step_dq(col_of(lds + stage * (2 * TILE), m / 2), m);
  }
  for (; kt < NT; ++kt) {
    next_stage();
    begin_pass(kt);
  }
  lds_barrier();          // the tile stages are free: the epilogue reuses LDS
  if (ntw == 0) return;

  float* my = reinterpret_cast<float*>(lds + wave * (32 * (D / 2) * 4));
#pragma unroll
  for (int pass = 0; pass < 2; ++pass)
    store_rows<D>(my, dQ, p.scale, pass, lane, p.dq + ((off0 + rw0) * p.Hq + kvh * p.g + head) * D, p.Hq * D,
                  [&](int t) { return rw0 + t <= rw1 ? t : -1; });
  if (!JOINED && rw0 + col <= rw1)
    p.stat[((int64_t)(kvh * p.g + head) * p.total_rows + off0 + r) * 2 + half] = half ? -delta : lse2;
}

template <int D, bool WIDE>
__global__ __launch_bounds__(kTileWaves * 64, D == 64 ? 3 : 2) void prefill_bwd_dq_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) char lds[dq_lds<D>()];
  const int hh = blockIdx.x / p.pstride;
  dq_block<D, WIDE, false>(p, lds, blockIdx.x - hh * p.pstride, hh, blockIdx.y, gridDim.y);
}

// ---------------------------------------------------------------------------
// dkv kernel
// ---------------------------------------------------------------------------
constexpr int kDkvStages = 2;

// 4 bytes per lane from HBM into LDS
__device__ __forceinline__ void lds_dma4_s(uint32_t lane_offset, uint64_t base, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               : : "s"(lds_addr), "v"(lane_offset), "s"(base) : "memory");
}

// The key blocks of a trajectory and what they are cut into (dense_parts()).  The partial sums lie by key, not by row: part for part the
// dense keys' dk, then their dv, behind them the same of the response tokens where their blocks are cut.
struct KeyParts {
  int prompt, beacons, tokens;       // keys: treated as dense-causal, complete windows' beacons, response rows that are no beacons
  int prompt_blocks, dense_blocks;
  int parts;                         // of a dense block
  __device__ __forceinline__ KeyParts(const BwdParams& p, const Trajectory& t, const WindowStride& ws) {
    prompt = ws.c > 0 ? min(t.P, t.rows) : t.rows;               // without compression every row behaves like a prompt row
    beacons = ws.c > 0 ? (int)window_of(ws, (uint32_t)(t.rows - prompt)) : 0;
    tokens = t.rows - prompt - beacons;
    prompt_blocks = (prompt + kDkvKeys - 1) / kDkvKeys;
    dense_blocks = prompt_blocks + (beacons + kDkvKeys - 1) / kDkvKeys;
    parts = dense_parts(p.splits, p.most, p.band, p.least, p.npairs, p.g, p.D, t.rows, prompt + beacons, dense_blocks);
  }
  // first row of sum `of` of the dense keys (the tokens) of a trajectory; of: 2 * part + (0 for dk, 1 for dv)
  __device__ __forceinline__ int64_t dense_row(const BwdParams& p, int64_t off0, int of) const {
    return 2 * p.splits * off0 + (int64_t)of * (prompt + beacons);
  }
  __device__ __forceinline__ int64_t token_row(const BwdParams& p, int64_t off0, int of) const {
    return dense_row(p, off0, 2 * parts) + (int64_t)of * tokens;
  }
};

// The two waves of a pair share 32 keys.  One forms the scores and A and adds dO^T.A to dV, the other
// forms dA, takes A through LDS, and adds Q^T.dS to dK: three of the six products each, and half of the
// accumulators and key operands, so that three waves fit a SIMD where one wave per 32 keys (two times 64
// accumulators and 64 operand registers) would leave room for one.
// JOINED: two workgroups a compute unit, whose registers and LDS let a pass work on two tiles.
template <bool JOINED> constexpr int dkv_stages() { return JOINED ? kDkvStages + 1 : kDkvStages; }
template <bool JOINED> constexpr int dkv_exchange() { return JOINED ? 2 * 8192 : 8192; }       // bytes in which A changes hands
template <int D, bool JOINED> constexpr int dkv_lds() {
  return dkv_stages<JOINED>() * (4 * kTileRows * D + 256) + dkv_exchange<JOINED>() + kTileWaves * 768;
}
template <int D, bool JOINED>
__device__ __forceinline__ void dkv_block(const BwdParams& p, char* lds, int by) {
  constexpr int ROWB = D * 2, KS = D / 16, NJ = D / 32, TILE = kTileRows * ROWB, STAGES = dkv_stages<JOINED>();
  constexpr int RING = STAGES * 2 * TILE, STAT = RING, XCH = RING + STAGES * 256;
  constexpr int OUT = kTileWaves * 32 * (D / 2) * 4;
  constexpr int KEYS_AT = XCH + dkv_exchange<JOINED>();
  static_assert(KEYS_AT >= OUT && KEYS_AT + kTileWaves * 768 == dkv_lds<D, JOINED>(), "the gradient tiles fit");
  // grid: x = (trajectory, KV head), y = key block; the long dense blocks of every trajectory
  // are dispatched before any short one
  const int pair = pair_in_turn(blockIdx.x, p.pstride, p.turn, blockIdx.y);
  if (pair >= p.npairs) return;
  const int kvh = pair % p.Hkv, b = pair / p.Hkv;
  const Trajectory traj = trajectory(p, b);
  const int64_t off0 = traj.off0;
  const int S = traj.rows;
  const WindowStride ws = window_stride(traj.c, S);
  const int c = ws.c, cp1 = ws.stride;
  // key blocks of this (trajectory, KV head): prompt keys | gathered beacons | response rows
  const KeyParts cut(p, traj, ws);
  const int Pk = cut.prompt, nresp = S - Pk, nbeac = cut.beacons;
  const int NPB = cut.prompt_blocks, nd = cut.dense_blocks, NLB = (nresp + kDkvKeys - 1) / kDkvKeys;
  // The dense blocks (prompt keys, beacons) stream every later row of every head; the tiles of each
  // are dealt to `parts` workgroups, whose partial sums another kernel adds in a fixed order.
  // The short response blocks are cut where the chip is not full; a block of one part stores its result directly.
  const int dense = cut.parts;
  const int at = (int)by - nd * dense;                  // place among the response blocks' parts
  const int parts = at < 0 ? dense : p.band;
  const int of = at < 0 ? (int)by : at;
  const int blk = of / parts + (at < 0 ? 0 : nd), split = parts > 1 ? of % parts : -1;
  if (blk >= nd + NLB) return;
  const int kind = blk < NPB ? 0 : blk < nd ? 1 : 2;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int kg = wave >> 1;                                     // the pair's 32 keys of the block
  const bool keys_role = ((wave ^ blockIdx.x ^ by) & 1) != 0;   // dA, dS, dK; otherwise scores, A, dV

  // this lane's key, the rows the block streams, and the rows the key is seen from: [jkey, last]
  int jkey, last;
  int sum_at;          // the key's place among the partial sums of its kind
  bool key_ok;
  int rs, re;          // first and last streamed row
  if (kind == 0) {
    const int j0 = blk * kDkvKeys;
    jkey = j0 + 32 * kg + col; key_ok = jkey < Pk;
    sum_at = jkey;
    rs = j0; re = S - 1; last = re;
  } else if (kind == 1) {
    const int m0 = (blk - NPB) * kDkvKeys, m = m0 + 32 * kg + col;
    key_ok = m < nbeac; jkey = Pk + m * cp1 + c;
    sum_at = Pk + m;
    rs = Pk + m0 * cp1 + c; re = S - 1; last = re;
  } else {
    const int j0 = Pk + (blk - nd) * kDkvKeys;
    jkey = j0 + 32 * kg + col; key_ok = jkey < S;
    const int jl = min(j0 + kDkvKeys - 1, S - 1);
    const int wl = (int)window_of(ws, (uint32_t)(jl - Pk));
    rs = j0; re = min(S - 1, Pk + (wl + 1) * cp1 - 1);      // through the closing beacon
    const uint32_t u = (uint32_t)(min(jkey, S - 1) - Pk), w = window_of(ws, u);
    if ((int)(u - w * (uint32_t)cp1) == c) key_ok = false;  // beacon rows belong to the beacon blocks
    sum_at = (int)(u - w);
    last = min(re, Pk + ((int)w + 1) * cp1 - 1);            // a response token: inside its own window
  }
  if (!key_ok) { jkey = rs; last = -1; }       // loads stay in range; seen from no row
  // what the pair's keys are seen from together, and what all of them are seen from
  int any_first = key_ok ? jkey : 0x7fffffff, all_first = jkey, any_last = last, all_last = last;
#pragma unroll
  for (int off = 1; off < 32; off <<= 1) {
    any_first = min(any_first, __shfl_xor(any_first, off, 64));
    all_first = max(all_first, __shfl_xor(all_first, off, 64));
    any_last = max(any_last, __shfl_xor(any_last, off, 64));
    all_last = min(all_last, __shfl_xor(all_last, off, 64));
  }
  any_first = __builtin_amdgcn_readfirstlane(any_first); all_first = __builtin_amdgcn_readfirstlane(all_first);
  any_last = __builtin_amdgcn_readfirstlane(any_last); all_last = __builtin_amdgcn_readfirstlane(all_last);

  // K^T or V^T of the keys as B operand (column = key, k = head-dim index)
  bf16x8_t op[KS];
  {
    const char* krow = (keys_role ? p.v : p.k) + ((off0 + jkey) * p.Hkv + kvh) * ROWB + 16 * half;
#pragma unroll
    for (int i = 0; i < KS; ++i)
      op[i] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(krow + 32 * i));
  }
  landed_operands(op);

  // Row tiles are streamed from the last row of the range backwards, all heads of a row tile one behind the other, and the parts of
  // a block take them in turn.  All dense key blocks and parts of a (trajectory, KV head) pair need the rows from the end of
  // the trajectory back to their own keys, start together (they are neighbours in dispatch order, on the same XCD) and so walk
  // the same rows at the same time: the later readers of a tile find it in the L2.  (Head by head and part behind part, blocks of different
  // length were soon at different heads: 16 trajectories of 8688 rows read 5.4 GB past the L2 and take 3218 us a
  // pass, 3.7 GB and 3190 now.)
  const int ntile = (re - rs) / kTileRows + 1;       // row tiles per head
  const int stride = split >= 0 ? parts : 1, first = split >= 0 ? split : 0;
  const int count = (ntile * p.g - first + stride - 1) / stride;       // tiles of this workgroup
  const int step_h = stride % p.g, step_rt = stride / p.g;
  struct Place { int h, rt; };
  auto advance = [&](Place& x) BC_INLINE {
    x.h += step_h; x.rt -= step_rt;
    if (x.h >= p.g) { x.h -= p.g; --x.rt; }
  };
  const int64_t q_row_bytes = (int64_t)p.Hq * ROWB;
  const TileLane tlane = either_tile_lane(lane, 2 * kg);       // (the next eight rows at the same place)
  const uint32_t lds0 = lds_address(lds);
  Place next{first % p.g, ntile - 1 - first / p.g};
  // By the keys' waves alone, half a tile each, while the others form A.  (By all four waves it was 460 of the 3,700
  // cycles of a tile's chain: 16 trajectories of 8688 rows 3331 -> 3293 us a pass, three short ones 74.8 -> 72.8.)
  auto issue_tile = [&](int stage) BC_INLINE {
    const int h = kvh * p.g + next.h, row0 = rs + next.rt * kTileRows;
    advance(next);
    const int left = S - 1 - row0;                   // (rows that do not exist repeat the last one)
    const int64_t at = (off0 + row0) * q_row_bytes + (int64_t)h * ROWB;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const uint32_t o = (uint32_t)min(tlane.row + 8 * u, left) * (uint32_t)q_row_bytes + tlane.in_row;
      const uint32_t dst = lds0 + stage * (2 * TILE) + (2 * kg + u) * 1024;
#pragma unroll
      for (int n = 0; n < D / 64; ++n) {
        lds_dma16_s<false>(o, (uint64_t)(p.q + at + 128 * n), dst + n * 4096);
        lds_dma16_s<false>(o, (uint64_t)(p.dout + at + 128 * n), dst + TILE + n * 4096);
      }
    }
    if (kg == 0) {         // 32 rows' log-sum-exp, then their Delta
      const float* st = p.stat + ((int64_t)h * p.total_rows + off0 + row0) * 2;
      lds_dma4_s((uint32_t)min(col, left) * 8u + half * 4u, (uint64_t)st, lds0 + STAT + stage * 256);
    }
  };
  f32x16_t acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = f32x16_t{0.f};
  const int rows_tile = keys_role ? TILE : 0, cols_tile = TILE - rows_tile;     // Q or dO by rows, the other by columns
  const int roff[2] = {rows_tile + either_rows_offset(lane), rows_tile + (either_rows_offset(lane) ^ 128)};
  const int coff[2] = {cols_tile + either_cols_offset(lane, 0), cols_tile + either_cols_offset(lane, 1)};
  const int soff = STAT + (keys_role ? 128 : 0) + 16 * half;
  f32x4_t* xch = reinterpret_cast<f32x4_t*>(lds + XCH + kg * 4096) + lane;      // JOINED: 8 KB further on for every other tile
  // the lane's key, the last row it is seen from and where its sums go: in LDS, every register of the loop is in use
  int* kept_key = reinterpret_cast<int*>(lds + KEYS_AT + wave * 768) + lane;
  kept_key[0] = jkey;
  kept_key[64] = last;
  kept_key[128] = !key_ok ? -1 : split >= 0 ? sum_at : jkey;
  constexpr int EARLY = D == 64 ? NJ : 0;       // column operands the keys' waves ask for in front of the second barrier
  constexpr int SLOTS = 4 * NJ;                 // matrix instructions of a column product

  // The order of a pass is written out (step_fence(): nothing is moved across): LDS operands are asked for several instructions
  // ahead, and both kinds of wave have a loop of their own.  Forward and gradients, us a pass: one trajectory of 2100 rows 80.1 -> 77.2, one of
  // 300, 4/1 heads, 41.5 -> 40.0, three of 336 to 795 60.1 -> 59.3, eight of 1100 to 3300 778 -> 771; 16 of 8688, at the power limit, 3172
  // and 3165.  All 168 registers are in use: one spilled into the loop waits for the tile's loads with its own (3200 -> 3330), and two
  // workgroups a compute unit with one barrier a pass and tiles worked on two at a time took 1486 us in place of 1467 on the
  // large batch.
  auto passes = [&](auto keys) BC_INLINE {
    constexpr bool KEYS = decltype(keys)::value;
    Place now = next;
    int stage = 1;
    if (KEYS && count > 0) issue_tile(0);
    for (int it = 0; it < count; ++it) {
      stage ^= 1;
      const char* tile = lds + stage * (2 * TILE);
      const int row0 = rs + now.rt * kTileRows;
      advance(now);
      // tile `it` has landed, and everyone has finished tile it-1
      if constexpr (KEYS) wait_vmcnt<0>();
      lds_barrier();
      // a row tile that ends in front of the pair's first key, or starts behind the last row any of its
      // keys is seen from, adds nothing here
      const bool busy = row0 + kTileRows - 1 >= any_first && row0 <= any_last;
      f32x16_t x;              // scores, or dA - Delta: the sums of dA start at -Delta
      bf16x8_t c[2 * NJ];
      float val[16];           // A, or dS
      auto col_of = [&](int n) BC_INLINE { return cols_operand<D>(tile + coff[n / NJ], n % NJ, n / NJ); };
      if (busy) {
        f32x4_t stat[4];       // log-sum-exp or -Delta of the lane's rows
        auto stats = [&](int q) BC_INLINE { stat[q] = *reinterpret_cast<const f32x4_t*>(lds + soff + stage * 256 + 32 * q); };
        bf16x8_t r[KS];
        auto row_of = [&](int i) BC_INLINE { r[i] = *reinterpret_cast<const bf16x8_t*>(tile + roff[i & 1] + rows_read_imm<D>(i)); };
        if constexpr (KEYS) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            stats(q);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * q + e] = stat[q][e];
          }
        } else {
          x = f32x16_t{0.f};
        }
#pragma unroll
        for (int i = 0; i < KS; ++i) row_of(i);         // (all of them in front of the first product)
        step_fence();
#pragma unroll
        for (int i = 0; i < KS; ++i) {
          x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r[i], op[i], x, 0, 0, 0);
          if (!KEYS && i >= KS - 4) stats(i - KS + 4);
          if (KEYS && i >= KS - EARLY) c[i - KS + EARLY] = col_of(i - KS + EARLY);
          step_fence();
        }
        if constexpr (!KEYS) {
#pragma unroll
          for (int e = 0; e < 16; ++e) val[e] = fast_exp2(fmaf(x[e], p.qscale, -stat[e / 4][e % 4]));
          if (row0 < all_first || row0 + kTileRows - 1 > all_last) {
            const int from = kept_key[0] - row0, upto = kept_key[64] - row0;
            const uint32_t mine = from >= 32 ? 0u : ~0u << max(from, 0);
            const uint32_t past = upto < 0 ? 0u : upto >= 31 ? ~0u : (2u << upto) - 1u;
            const uint32_t see = (mine & past) >> (4 * half);
#pragma unroll
            for (int e = 0; e < 16; ++e) val[e] = keep_if_visible(val[e], see, e);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
            xch[64 * q] = f32x4_t{val[4 * q], val[4 * q + 1], val[4 * q + 2], val[4 * q + 3]};
        }
      }
      if (KEYS && it + 1 < count) issue_tile(stage ^ 1);
      lds_barrier();       // A of tile `it` is there
      if (!busy) continue;
      if constexpr (KEYS) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4_t a = xch[64 * q];
#pragma unroll
          for (int e = 0; e < 4; ++e) val[4 * q + e] = a[e] * x[4 * q + e];
        }
      }
      // dV^T += dO^T.A or dK^T += Q^T.dS
#pragma unroll
      for (int n = KEYS ? EARLY : 0; n < NJ; ++n) c[n] = col_of(n);
      Parts y;
#pragma unroll
      for (int g = 0; g < 4; ++g) y.split(g, val[2 * g], val[2 * g + 1]);
      step_fence();
#pragma unroll
      for (int m = 0; m < SLOTS; ++m) {
        const int n = m / 2;
        acc[n % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[n], y.operand(m & 1, n / NJ), acc[n % NJ], 0, 0, 0);
        if (m % 2 == 0 && n + NJ < 2 * NJ) c[n + NJ] = col_of(n + NJ);
#pragma unroll
        for (int g = 4; g < 8; ++g)
          if (m == (g - 4) * NJ / 2) y.split(g, val[2 * g], val[2 * g + 1]);
        step_fence();
      }
    }
  };
  // JOINED: a pass forms A or dA of tile `it` beside the column product of the tile before, with one barrier: A of a tile is taken in the pass
  // behind the one that forms it.  What bounds a launch that leaves the chip idle is the chain of its longest parts: a pass of the keys' waves is some 2,000 cycles,
  // 770 of them matrix instructions, the rest the operands' way through LDS, the split and the loads' issue.  Forward and gradients, in two steps with a
  // barrier each (`passes`) and so: three trajectories of 336 to 795 rows 52.2 -> 50.9 us, one of 3100, 5/1 heads, 78.3 -> 74.9, two of 2128, 12/2 heads, 101.1 ->
  // 98.9.  (In launches that fill the chip three workgroups a compute unit are better: 8 trajectories of 3200 rows, 8/8 heads, 383 and 404, 16 of 8688 3231 and 3313.)
  struct TileAt { int64_t at; const float* stat; uint32_t row[2], stat_row; };
  auto next_tile = [&]() BC_INLINE {                 // (behind the last place: one of the first row tile again)
    const int h = kvh * p.g + next.h, row0 = rs + max(next.rt, 0) * kTileRows;
    advance(next);
    const int left = S - 1 - row0;                   // (rows that do not exist repeat the last one)
    TileAt t;
    t.at = (off0 + row0) * q_row_bytes + (int64_t)h * ROWB;
    t.stat = p.stat + ((int64_t)h * p.total_rows + off0 + row0) * 2;
#pragma unroll
    for (int u = 0; u < 2; ++u) t.row[u] = (uint32_t)min(tlane.row + 8 * u, left) * (uint32_t)q_row_bytes + tlane.in_row;
    t.stat_row = (uint32_t)min(col, left) * 8u + half * 4u;
    return t;
  };
  // By the keys' waves beside their column products.  (In front of the pass 51.3 us for the three trajectories, by all four waves 51.9.)
  auto load_part = [&](const TileAt& t, int stage, int part) BC_INLINE {       // one of D / 16: 1 KB of Q or dO
    const int which = part % 2, u = part / 2 % 2, n = part / 4;
    lds_dma16_s<false>(t.row[u], (uint64_t)((which ? p.dout : p.q) + t.at + 128 * n),
                       lds0 + stage * (2 * TILE) + (2 * kg + u) * 1024 + which * TILE + n * 4096);
  };
  auto load_stat = [&](const TileAt& t, int stage) BC_INLINE {
    if (kg == 0) lds_dma4_s(t.stat_row, (uint64_t)t.stat, lds0 + STAT + stage * 256);
  };
  auto load_tile = [&](int stage) BC_INLINE {
    const TileAt t = next_tile();
#pragma unroll
    for (int part = 0; part < D / 16; ++part) load_part(t, stage, part);
    load_stat(t, stage);
  };
  auto joined_passes = [&](auto keys) BC_INLINE {
    constexpr bool KEYS = decltype(keys)::value;
    constexpr int PRE = 4;         // products that row operands are asked for ahead
    Place now = next;
    int stage = STAGES - 1;
    if (KEYS && count > 0) load_tile(0);
    bool busy_before = false;
    float val[16];                 // A, or dA - Delta, of the tile before
    const char* before = lds;
    for (int it = 0; it <= count; ++it) {
      stage = stage + 1 == STAGES ? 0 : stage + 1;
      const char* tile = lds + stage * (2 * TILE);
      const int row0 = rs + now.rt * kTileRows;
      advance(now);
      // tile `it` has landed, and everyone has finished pass it - 1, which was the last to look at tile it - 2
      if constexpr (KEYS) wait_vmcnt<0>();
      lds_barrier();
      const int into = stage + 1 == STAGES ? 0 : stage + 1;      // of the next tile
      const bool busy = it < count && row0 + kTileRows - 1 >= any_first && row0 <= any_last;
      f32x4_t* put = xch + (it & 1) * 512;
      const f32x4_t* got = xch + (~it & 1) * 512;
      auto pass = [&](auto cur, auto prev) BC_INLINE {
        constexpr bool CUR = decltype(cur)::value, PREV = decltype(prev)::value;
        f32x16_t x;                // scores, or dA - Delta: the sums of dA start at -Delta
        f32x4_t stat[4], a[4];     // log-sum-exp or -Delta of the lane's rows; A of the tile before
        bf16x8_t r[KS], c[2 * NJ];
        Parts y;
        auto row_of = [&](int i) BC_INLINE { r[i] = *reinterpret_cast<const bf16x8_t*>(tile + roff[i & 1] + rows_read_imm<D>(i)); };
        auto col_of = [&](int n) BC_INLINE { c[n] = cols_operand<D>(before + coff[n / NJ], n % NJ, n / NJ); };
        TileAt to;
        auto split = [&](int g) BC_INLINE {
          if constexpr (KEYS) y.split(g, a[g / 2][2 * g % 4] * val[2 * g], a[g / 2][2 * g % 4 + 1] * val[2 * g + 1]);      // dS
          else y.split(g, val[2 * g], val[2 * g + 1]);
        };
        if constexpr (CUR) {
#pragma unroll
          for (int q = 0; q < 4; ++q) stat[q] = *reinterpret_cast<const f32x4_t*>(lds + soff + stage * 256 + 32 * q);
#pragma unroll
          for (int i = 0; i < PRE; ++i) row_of(i);
        }
        if constexpr (KEYS && PREV) {
#pragma unroll
          for (int q = 0; q < 4; ++q) a[q] = got[64 * q];
        }
        if constexpr (CUR) {
          if constexpr (KEYS) {
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] = stat[e / 4][e % 4];
          } else {
            x = f32x16_t{0.f};
          }
        }
        step_fence();
#pragma unroll
        for (int i = 0; i < KS; ++i) {
          if constexpr (CUR) {
            x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r[i], op[i], x, 0, 0, 0);
            if (i + PRE < KS) row_of(i + PRE);
            if (KEYS && i == 0) to = next_tile();
          }
          if constexpr (PREV) {
            if (i >= KS - NJ) col_of(i - KS + NJ);
            // (what is asked for in front of the first product is there behind the second)
#pragma unroll
            for (int g = 0; g < 8; ++g)
              if (i == KS / 4 + g * (KS - KS / 4) / 8) split(g);
          }
          step_fence();
        }
#pragma unroll
        for (int m = 0; m < SLOTS; ++m) {
          if constexpr (PREV) {
            const int n = m / 2;
            acc[n % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[n], y.operand(m & 1, n / NJ), acc[n % NJ], 0, 0, 0);
            if (m % 2 == 0 && n + NJ < 2 * NJ) col_of(n + NJ);
          }
          if constexpr (CUR && KEYS) {
            if (m % 2 == 1) load_part(to, into, m / 2);
            if (m == SLOTS - 1) load_stat(to, into);
          }
          if constexpr (CUR && !KEYS) {            // (the scores are there behind the second product)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if (m == 2 + e * (SLOTS - 3) / 15) {
                val[e] = fast_exp2(fmaf(x[e], p.qscale, -stat[e / 4][e % 4]));
                asm volatile("" : "+v"(val[e]));   // (worked out here and not behind the next barrier)
              }
          }
          step_fence();
        }
        if constexpr (CUR && KEYS) {
#pragma unroll
          for (int e = 0; e < 16; ++e) val[e] = x[e];
        }
        if constexpr (CUR && !KEYS) {
          if (row0 < all_first || row0 + kTileRows - 1 > all_last) {
            const int from = kept_key[0] - row0, upto = kept_key[64] - row0;
            const uint32_t mine = from >= 32 ? 0u : ~0u << max(from, 0);
            const uint32_t past = upto < 0 ? 0u : upto >= 31 ? ~0u : (2u << upto) - 1u;
            const uint32_t see = (mine & past) >> (4 * half);
#pragma unroll
            for (int e = 0; e < 16; ++e) val[e] = keep_if_visible(val[e], see, e);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) put[64 * q] = f32x4_t{val[4 * q], val[4 * q + 1], val[4 * q + 2], val[4 * q + 3]};
        }
      };
      if (busy) {
        if (busy_before) pass(std::true_type{}, std::true_type{});
        else pass(std::true_type{}, std::false_type{});
      } else {
        if (KEYS && it + 1 < count) load_tile(into);
        if (busy_before) pass(std::false_type{}, std::true_type{});
      }
      busy_before = busy;
      before = tile;
    }
  };
  if constexpr (JOINED) {
    if (keys_role) joined_passes(std::true_type{});
    else joined_passes(std::false_type{});
  } else {
    if (keys_role) passes(std::true_type{});
    else passes(std::false_type{});
  }
  lds_barrier();

  // every key row is owned by exactly one lane column of one block: plain stores
  using global_float = __attribute__((address_space(1))) float;
  global_float *dk = (global_float*)p.dk, *dv = (global_float*)p.dv;
  asm("" : "+s"(dk), "+s"(dv));        // (chosen by address, they went through scratch memory)
  float* base = (float*)(keys_role ? dk : dv) + off0 * p.Hkv * D;
  if (split >= 0) {
    const int of = 2 * split + (keys_role ? 0 : 1);
    base = p.part + (kind == 2 ? cut.token_row(p, off0, of) : cut.dense_row(p, off0, of)) * p.Hkv * D;
  }
  float* my = reinterpret_cast<float*>(lds + wave * (32 * (D / 2) * 4));
  const int key_row = kept_key[128];
#pragma unroll
  for (int pass = 0; pass < 2; ++pass)
    store_rows<D>(my, acc, keys_role ? p.scale : 1.0f, pass, lane, base + kvh * D, p.Hkv * D,
                  [&](int t) { return __shfl(key_row, t, 64); });
}

template <int D>
__global__ __launch_bounds__(kTileWaves * 64, 3) void prefill_bwd_dkv_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) char lds[dkv_lds<D, false>()];
  dkv_block<D, false>(p, lds, blockIdx.y);
}

// Launches that leave the chip idle are a chain of kernels that each wait for the one before, and the dkv kernel waits for nothing but
// Delta.  So Delta has a kernel of its own there, and the workgroups of both kernels go out together, dq first: three trajectories of 336 to
// 795 rows, 12/2 heads, dq 18 and dkv 18 us become 6 and 27 under the profiler, a pass of forward and gradients 58.9 -> 54.0.  Delta's kernel is
// the first touch of `out`: with 64 rows a workgroup, four loads of a thread out at once, it takes 6.4 us, with 16 rows 6.2.
constexpr int kDeltaRows = 16;        // rows of one head that a workgroup takes at a time: sixteen lanes a row
template <int D>
__global__ __launch_bounds__(256) void prefill_bwd_delta_kernel(BwdParams p) {
  const Trajectory traj = trajectory(p, blockIdx.x);
  // (in 32 bits: a joined launch has at most 65,536 rows of a head, see in_one_launch())
  const uint32_t units = (uint32_t)traj.rows * (uint32_t)p.Hq, Hq = (uint32_t)p.Hq;
  const int lane = threadIdx.x & 15;
  for (uint32_t i = blockIdx.y * kDeltaRows + (threadIdx.x >> 4); i < units; i += gridDim.y * kDeltaRows) {
    const int64_t at = traj.off0 * p.Hq + i;
    float4 o[D / 64];
    uint2 y[D / 64];
    float lse2 = p.lse[at];
#pragma unroll
    for (int t = 0; t < D / 64; ++t) {
      o[t] = *reinterpret_cast<const float4*>(p.out + at * D + 4 * lane + 64 * t);
      y[t] = *reinterpret_cast<const uint2*>(p.dout + (at * D + 4 * lane + 64 * t) * 2);
    }
    const float delta = row_dot<D>(o, y);
    // (asked for with the rest: used by two lanes of sixteen, it had been taken behind the sum and the branch, one more round trip)
    asm volatile("" : "+v"(lse2));
    lse2 *= kLog2e;
    const uint32_t row = i / Hq, head = i - row * Hq;
    if (lane < 2) p.stat[((int64_t)head * p.total_rows + traj.off0 + row) * 2 + lane] = lane ? -delta : lse2;
  }
}
template <int D>
__global__ __launch_bounds__(kTileWaves * 64, 2) void prefill_bwd_joined_kernel(BwdParams p) {
  __shared__ __attribute__((aligned(1024))) char lds[dq_lds<D>() > dkv_lds<D, true>() ? dq_lds<D>() : dkv_lds<D, true>()];
  if ((int)blockIdx.y < p.dq_rows * p.tiling.splits) {
    const int by = blockIdx.y / p.tiling.splits;
    dq_block<D, false, true>(p, lds, blockIdx.x, blockIdx.y - by * p.tiling.splits, by, p.dq_rows);
  } else {
    dkv_block<D, true>(p, lds, blockIdx.y - p.dq_rows * p.tiling.splits);
  }
}

// Sum of the partials of the dense keys (prompt rows and beacons) and, where the response blocks were cut too, of the
// response tokens, in split order.  Rows of blocks in one part were written directly.  grid: x = trajectory, y = blocks that share its
// keys (a thread for every 16 bytes of every row, which had to find the row's trajectory and whether it is dense, took 47 us instead
// of 16 for 16 trajectories of 8688 rows: one row in twelve is dense).
// What bounds it: HBM on large launches, the way to a wave's first load on small ones.  A wave takes 64 units of 16 bytes of a key, or as many keys as make
// 64 units, so that a key's place is worked out once and without a division, and all parts of a unit are on their way together.  (A unit a thread, two
// divisions of 64 bits each, the parts one by one, 128 workgroups a trajectory: three trajectories of 336 to 795 rows 7.0 us of an idle chip; forward and gradients
// 50.9 -> 49.6, two of 504 rows, 32/8 heads, uncompressed 79.3 -> 73.4, one of 3100, 5/1 heads, 74.9 -> 69.3, two of 6300, 16/2 heads, 374 -> 368.)
__global__ __launch_bounds__(256) void prefill_bwd_reduce_kernel(BwdParams p) {
  const int b = blockIdx.x;
  const Trajectory traj = trajectory(p, b);
  const int64_t off0 = traj.off0;
  if (traj.rows <= 0) return;
  const WindowStride ws = window_stride(traj.c, traj.rows);
  const KeyParts cut(p, traj, ws);
  const int ndense = cut.prompt + cut.beacons;
  const int first = cut.parts > 1 ? 0 : ndense, end = ndense + (p.band > 1 ? traj.rows - cut.prompt : 0);      // dense keys, then response rows
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int per_row = p.Hkv * (p.D / 4);         // 16-byte units
  const int keys = reduce_keys(per_row), slices = reduce_slices(per_row);
  const int mine = keys > 1 ? lane / per_row : 0, step = (int)gridDim.y * 4;      // (the lane's key among them)
  const int64_t row_floats = (int64_t)p.Hkv * p.D;
  int item = (int)blockIdx.y * 4 + wave;
  int slice = item % slices;
  const int slice_step = step % slices;
  for (int at0 = first + item / slices * keys; at0 < end;) {
    const int n = at0 + mine, unit = (keys > 1 ? lane - mine * per_row : 64 * slice + lane);      // key, place in its row
    bool there = n < end && mine < keys && unit < per_row;
    int row, sum, plane;
    int64_t at;
    if (n < ndense) {
      row = n < cut.prompt ? n : cut.prompt + (n - cut.prompt) * ws.stride + ws.c;
      sum = cut.parts; plane = ndense; at = cut.dense_row(p, off0, 0) + n;
    } else {
      const uint32_t u = (uint32_t)(n - ndense), w = window_of(ws, u);      // (response rows: there are none without compression)
      if ((int)(u - w * (uint32_t)ws.stride) == ws.c) there = false;        // a beacon
      row = cut.prompt + (int)u;
      sum = p.band; plane = cut.tokens; at = cut.token_row(p, off0, 0) + (int)(u - w);
    }
    if (there) {
      const float* from = p.part + at * row_floats + 4 * unit;
      const int64_t next = (int64_t)plane * row_floats;
      f32x4_t sk = f32x4_t{0.f, 0.f, 0.f, 0.f}, sv = sk;
      // two parts (large launches), or up to eight on their way at a time, also of the last seven
      auto add = [&](int s0, auto count) BC_INLINE {
        constexpr int N = decltype(count)::value;
        f32x4_t xk[N], xv[N];
#pragma unroll
        for (int e = 0; e < N; ++e) {
          const float* x = from + 2 * min(s0 + e, sum - 1) * next;
          xk[e] = *reinterpret_cast<const f32x4_t*>(x);
          xv[e] = *reinterpret_cast<const f32x4_t*>(x + next);
        }
        step_fence();
        // (a branch around an addition took the load behind it along: the parts came one by one)
        const f32x4_t zero = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < N; ++e) {
          sk += s0 + e < sum ? xk[e] : zero;
          sv += s0 + e < sum ? xv[e] : zero;
        }
      };
      if (sum <= 2) {
        add(0, std::integral_constant<int, 2>{});
      } else {
        for (int s0 = 0; s0 < sum; s0 += 8) add(s0, std::integral_constant<int, 8>{});
      }
      const int64_t to = (off0 + row) * row_floats + 4 * unit;
      *reinterpret_cast<f32x4_t*>(p.dk + to) = sk;
      *reinterpret_cast<f32x4_t*>(p.dv + to) = sv;
    }
    // the wave's next item: `step` items further on
    slice += slice_step;
    at0 += step / slices * keys;
    if (slice >= slices) { slice -= slices; at0 += keys; }
  }
}

template <int D>
static void launch_bwd(const BwdParams& p, bool joined, bool wide, dim3 dq_grid, dim3 dkv_grid, int32_t max_rows, hipStream_t hs) {
  if (joined) {          // (never wide: all rows together are at most 128 for each of the joined kernel's dq workgroups)
    const int64_t n = ((int64_t)max_rows * p.Hq + kDeltaRows - 1) / kDeltaRows;
    prefill_bwd_delta_kernel<D><<<dim3(p.npairs / p.Hkv, (int)(n < 1024 ? n : 1024)), 256, 0, hs>>>(p);
    const dim3 grid(p.pstride, dq_grid.y * p.tiling.splits + dkv_grid.y);
    prefill_bwd_joined_kernel<D><<<grid, kTileWaves * 64, 0, hs>>>(p);
    return;
  }
  if (wide) prefill_bwd_dq_kernel<D, true><<<dq_grid, kTileWaves * 64, 0, hs>>>(p);
  else prefill_bwd_dq_kernel<D, false><<<dq_grid, kTileWaves * 64, 0, hs>>>(p);
  prefill_bwd_dkv_kernel<D><<<dkv_grid, kTileWaves * 64, 0, hs>>>(p);
}

// Floats of the workspace's first part (stat), rounded up so that the partials behind it start at 256 bytes:
// they are stored and summed 16 bytes at a time, and an odd number of rows times heads would put them 8 off.
static size_t stat_floats(const bc_shape* shape, int64_t total_rows) {
  return ((size_t)total_rows * shape->Hq * 2 + 63) / 64 * 64;
}

}  // namespace bc

using namespace bc;

extern "C" size_t bc_prefill_bwd_workspace_bytes(const bc_shape* shape, int64_t total_rows) {
  if (check_shape(shape) != BC_OK || total_rows < 1) return 0;
  const int hs = dense_splits(shape->B, shape->Hq, shape->Hkv, total_rows);
  size_t bytes = stat_floats(shape, total_rows) * sizeof(float);
  if (hs > 1) bytes += (size_t)hs * 2 * total_rows * shape->Hkv * shape->d * sizeof(float);
  return bytes;
}

// p has its tables.
static int32_t prefill_backward(BwdParams& p, const bc_shape* shape, const void* q, const void* k, const void* v,
                                const float* out, const float* lse, const void* dout, int32_t max_rows,
                                int64_t total_rows, float* dq, float* dk, float* dv, void* workspace, void* stream) {
  p.q = static_cast<const char*>(q); p.k = static_cast<const char*>(k);
  p.v = static_cast<const char*>(v); p.out = out; p.lse = lse;
  p.dout = static_cast<const char*>(dout);
  p.dq = dq; p.dk = dk; p.dv = dv;
  p.stat = static_cast<float*>(workspace);
  p.part = p.stat + stat_floats(shape, total_rows);
  p.splits = dense_splits(shape->B, shape->Hq, shape->Hkv, total_rows);
  p.most = most_parts(p.splits);
  p.total_rows = total_rows;
  p.D = shape->d;
  p.Hq = shape->Hq; p.Hkv = shape->Hkv; p.g = shape->Hq / shape->Hkv;
  p.scale = shape->scale;
  p.qscale = shape->scale * kLog2e;
  hipStream_t hs = as_stream(stream);
  p.npairs = shape->B * shape->Hkv;
  p.pstride = pair_stride(p.npairs);
  p.turn = pair_turn(p.pstride);
  p.tiling = head_tiling(p.g);
  const int rows_wg = kTileRows * p.tiling.row_blocks;
  const dim3 dq_grid(p.tiling.splits * p.pstride, (max_rows + rows_wg - 1) / rows_wg);
  p.dq_rows = dq_grid.y;
  p.band = band_splits(shape->B, shape->Hq, shape->Hkv, total_rows, p.splits);
  p.least = least_tiles(p.g, p.band);
  const int key_blocks = (max_rows + kDkvKeys - 1) / kDkvKeys;
  const dim3 dkv_grid(p.pstride, (int)dkv_grid_rows(p.npairs, p.most, p.band, key_blocks));
  const bool wide = rows_span_4gb(max_rows, shape), joined = in_one_launch(shape->B, p.npairs, p.tiling, total_rows);
  if (shape->d == 128) launch_bwd<128>(p, joined, wide, dq_grid, dkv_grid, max_rows, hs);
  else launch_bwd<64>(p, joined, wide, dq_grid, dkv_grid, max_rows, hs);
  if (p.splits > 1) {
    const int per_row = shape->Hkv * (shape->d / 4), keys = reduce_keys(per_row);
    const int64_t blocks = ((int64_t)(max_rows + keys - 1) / keys * reduce_slices(per_row) + 3) / 4, most = reduce_blocks(shape->B);
    prefill_bwd_reduce_kernel<<<dim3(shape->B, (int)(blocks < most ? blocks : most)), 256, 0, hs>>>(p);
  }
  return launch_status();
}

static int32_t check_backward(const bc_shape* shape, const void* q, const void* k, const void* v, const float* out,
                              const float* lse, const void* dout, const void* row_offsets, const void* P, const void* c,
                              int32_t max_rows, int64_t total_rows, const float* dq, const float* dk, const float* dv,
                              const void* workspace, size_t workspace_bytes) {
  const int32_t st = check_shape(shape);
  if (st != BC_OK) return st;
  if (shape->kv_dtype != BC_BF16) return BC_ERR_SHAPE;
  if (!q || !k || !v || !out || !lse || !dout || !row_offsets || !P || !c || !dq || !dk || !dv)
    return BC_ERR_ARG;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out) || !aligned16(dout) ||
      !aligned16(dq) || !aligned16(dk) || !aligned16(dv))
    return BC_ERR_ARG;
  if (max_rows < 1 || max_rows >= (1 << 26) || total_rows < max_rows) return BC_ERR_ARG;
  if (!positive_finite(shape->scale)) return BC_ERR_ARG;
  if (!workspace || !aligned16(workspace) ||
      workspace_bytes < bc_prefill_bwd_workspace_bytes(shape, total_rows))
    return BC_ERR_WORKSPACE;
  return BC_OK;
}

extern "C" int32_t bc_prefill_attn_bwd(const bc_shape* shape, const void* q, const void* k,
                                       const void* v, const float* out, const float* lse,
                                       const void* dout, const int64_t* row_offsets,
                                       const int32_t* P, const int32_t* c, int32_t max_rows,
                                       int64_t total_rows, float* dq, float* dk, float* dv,
                                       void* workspace, size_t workspace_bytes, void* stream) {
  const int32_t st = check_backward(shape, q, k, v, out, lse, dout, row_offsets, P, c, max_rows, total_rows, dq, dk, dv,
                                    workspace, workspace_bytes);
  if (st != BC_OK) return st;
  BwdParams p;
  p.row_off = row_offsets; p.P = P; p.c = c;
  return prefill_backward(p, shape, q, k, v, out, lse, dout, max_rows, total_rows, dq, dk, dv, workspace, stream);
}

extern "C" int32_t bc_prefill_attn_bwd_host(const bc_shape* shape, const void* q, const void* k, const void* v,
                                            const float* out, const float* lse, const void* dout,
                                            const int64_t* row_offsets, const int32_t* P, const int32_t* c,
                                            int32_t max_rows, int64_t total_rows, float* dq, float* dk, float* dv,
                                            void* tables, void* workspace, size_t workspace_bytes, void* stream) {
  int32_t st = check_backward(shape, q, k, v, out, lse, dout, row_offsets, P, c, max_rows, total_rows, dq, dk, dv,
                              workspace, workspace_bytes);
  if (st != BC_OK) return st;
  BwdParams p;
  st = host_tables(p, row_offsets, P, c, shape->B, tables, stream);
  if (st != BC_OK) return st;
  return prefill_backward(p, shape, q, k, v, out, lse, dout, max_rows, total_rows, dq, dk, dv, workspace, stream);
}

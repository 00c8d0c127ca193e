// bc_prefill_attn: beacon-masked prefill attention, forward (Fig. 2, Sec. 3.2 of the paper).
//
// Training keeps every row and hides what eviction would have removed.  Seen from a tile of
// query rows that lies in the response, the visible keys are three runs:
//   A  the prompt rows                                   (dense, nothing masked)
//   B  the beacons of every window that ended before the tile's first window
//      (one row every c+1 rows: a strided gather,         dense, nothing masked)
//   C  the band from the start of the tile's first window to the tile's last row
//      (block-diagonal windows plus the beacons inside:   masked by integer arithmetic)
// so the kernel walks a compacted key list of about P + r/(c+1) + 32 + c rows per tile
// instead of the r rows of causal attention, and never materialises a mask.  Tiles that
// touch the prompt use run C alone with the same predicate (which is then plain causal).
//
// One workgroup = four waves that share the K/V tiles; one wave = 32 query rows of one head.  Tiles of
// 32 keys are gathered from HBM into a 3-stage LDS ring by 16-byte LDS-DMA loads (one barrier per
// tile) and fed to 32x32x16 MFMA: S^T = K.Q^T in bf16, O^T += V^T.P^T with P split into two bf16 parts
// so that the softmax weights keep about 16 bits (or, in the workspace form, as one half-precision
// part against a half-precision copy of V).  Softmax runs online in registers in the accumulator
// layout, whose keys are the value product's operand as they stand.  The output tile goes through LDS
// so that every row is written to HBM in bursts.  Head dimension 128 or 64 (a template parameter).
//
// What bounds it: the matrix cores under the card's power limit.  16 trajectories of 8688 rows, 12/2
// heads, d = 128: 724 GFLOP of MFMA work are issued in 0.76 ms in a training pass, 0.81 in calls behind one
// another and 0.68 in the fastest (0.96, 0.89 and 1.06 PFLOP/s; matrix pipe busy 61 % of the cycles at the 1.7 GHz the
// clock falls to; a library product of 16384^3 runs at 1.34 PFLOP/s here).  The form
// before this one, 16x16x32 MFMA with 16 rows of three heads per wave and two waves per SIMD, took
// 0.80-0.85 ms.  Measured on the way, each against its neighbour in one session:
//  - 32x32x16 instead of 16x16x32: half the operand reads per product, and vector work of other waves
//    fits beside it (a loop of MFMA and FMA bursts, two waves per SIMD, six FMA per 32x32x16 or three per
//    16x16x32: 1.01 against 1.29 times the MFMA time alone);
//  - at most 168 registers, three waves per SIMD: with work of neighbouring tiles interleaved by hand inside a
//    wave and two waves per SIMD the same loop took 0.80 ms (higher matrix load, lower clock);
//  - operands of a tile at one register plus constants, no bank conflicts (bc_prefill_tiles.h);
//  - loads asked for behind the scores' MFMAs, their addresses from a cursor, and prompt and beacon
//    remainders packed with the band (7 % fewer MFMAs, bc_prefill_tiles.h): together 0.77 -> 0.70 ms.
#include <cstddef>
#include <cstring>
#include <type_traits>

#include "bc_prefill_tiles.h"

namespace bc {

typedef __attribute__((ext_vector_type(2))) float pf_f32x2_t;
typedef __attribute__((ext_vector_type(2))) _Float16 pf_f16x2_t;
typedef __attribute__((ext_vector_type(8))) _Float16 pf_f16x8_t;

struct PrefillParams {
  const char* q;
  const char* k;
  const char* v;
  const char* v16;         // V rounded to half precision, same layout (workspace form only)
  const uint32_t* flags;   // workspace form: kPfFlagBytes verdicts of the conversion pass, 0 = every V entry fits; else NULL
  const int64_t* row_off;
  const int32_t* P;
  const int32_t* c;
  float* out;
  float* lse;
  int32_t Hq, Hkv, g;
  HeadTiling tiling;
  int32_t npairs;     // (trajectory, KV head) pairs
  int32_t pstride;    // pairs per head split in the grid, see pair_stride()
  int32_t turn;       // see pair_turn()
  float qscale;       // softmax scale * log2(e)
  InlineTables tab;
};

constexpr size_t kPfFlagBytes = 256;

#define BC_INLINE __attribute__((always_inline))      // lambdas: their captures stay in registers

constexpr float kPfRedo = 256.f;      // a lane's 16 weights may sum to this before the reference moves
constexpr float kPfLazy = 2.0f;       // ... and then it moves where a row's maximum is this much (log2) above it

template <int D> constexpr int prefill_lds() { return kTileStages * 2 * kTileRows * D * 2; }

// One wave = 32 query rows of one head, four waves per workgroup (heads of one KV head or row blocks).
// HALF: the weights enter the value product as one half-precision part (11 bits) against V in half
// precision, instead of two bf16 parts against V in bf16: a third fewer matrix instructions and no
// split.  V's copy in half precision is exact for entries between 2^-14 and 65504 in magnitude (bf16
// has fewer mantissa bits), which a conversion pass checks; its verdict chooses the form.
template <int D, bool HALF, bool WIDE>
__device__ __forceinline__ void prefill_rows(const PrefillParams& p, char* lds) {
  constexpr int ROWB = D * 2;                 // bytes of a K or V row
  constexpr int KS = D / 16;                  // k-steps of the score product
  constexpr int NJ = D / 32;                  // 32-column blocks of the output
  constexpr int TILE = kTileRows * ROWB;      // bytes of one K (or V) tile
  constexpr int NLD = TILE / 1024 / kTileWaves;     // LDS-DMA instructions per wave, tile and tensor
  constexpr int LDS = prefill_lds<D>();
  constexpr int OW = D / 2;                   // output columns that go through LDS at a time
  static_assert(LDS >= kTileWaves * 32 * OW * 4, "the output tiles fit the ring's LDS");

  const int hh = blockIdx.x / p.pstride, pair = pair_in_turn(blockIdx.x - hh * p.pstride, p.pstride, p.turn, blockIdx.y);
  if (pair >= p.npairs) return;
  const int kvh = pair % p.Hkv, b = pair / p.Hkv;
  const Trajectory traj = trajectory(p, b);
  const int64_t off0 = traj.off0;
  const int S = traj.rows;
  const int rows_wg = kTileRows * p.tiling.row_blocks;
  const int r0 = (gridDim.y - 1 - blockIdx.y) * rows_wg;        // long tiles first
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
  // tiles this wave works on (none without a head or without rows); the workgroup's NT >= ntw are
  // loaded and passed by all waves together
  const int ntw = head < p.g && rw0 <= r1 ? runs.tiles_up_to(rw1) : 0;

  const int64_t kv_row_bytes = (int64_t)p.Hkv * ROWB;
  const char* kbase = p.k + (off0 * p.Hkv + kvh) * ROWB;
  const char* vbase = (HALF ? p.v16 : p.v) + (off0 * p.Hkv + kvh) * ROWB;
  const uint32_t lds0 = lds_address(lds) + wave * 1024;
  const TileLane klane = rows_tile_lane(lane, wave), vlane = cols_tile_lane(lane, wave);
  TileCursor cursor(runs, kv_row_bytes);
  auto issue_tile = [&](int stage) BC_INLINE {
    const TileLoad t = cursor.next(runs);
    const auto ko = tile_lane_offset<WIDE>(runs, t, klane, kv_row_bytes);
    const auto vo = tile_lane_offset<WIDE>(runs, t, vlane, kv_row_bytes);
#pragma unroll
    for (int n = 0; n < NLD; ++n) {           // (128 bytes further on in each row)
      issue_block<WIDE>(kbase + t.off + 128 * n, ko, lds0 + stage * (2 * TILE) + n * 4096);
      issue_block<WIDE>(vbase + t.off + 128 * n, vo, lds0 + stage * (2 * TILE) + TILE + n * 4096);
    }
  };
  issue_tile(0);

  // this lane's query row; Q^T as the B operand (column = row, k = head-dim index).  The wave's rows come through the
  // stages behind the first tile's.
  const int r = min(rw0 + col, r1), rw = min(rw0, r1);
  bf16x8_t qb[KS];
  static_assert(LDS >= (2 + kTileWaves) * TILE, "the waves' rows fit behind the first tile");
  issue_wave_rows<D>(p.q + ((off0 + rw) * p.Hq + kvh * p.g + min(head, p.g - 1)) * ROWB, (uint32_t)p.Hq * ROWB, r1 - rw,
                     lane, lds_address(lds) + (2 + wave) * TILE);
  wait_vmcnt<0>();
  read_wave_rows<D>(lds + (2 + wave) * TILE, lane, qb);
  landed_operands(qb);
  lds_barrier();            // every wave has its rows
  if (NT > 1) issue_tile(1);
  const int own = runs.window_start(r);

  f32x16_t O[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) O[j] = f32x16_t{0.f};
  // The reference m of the running softmax is lazy: weights are formed against it as it is and only
  // where their sum over a lane's 16 keys passes kPfRedo (fp32 sums and the two-part weights carry
  // such weights without loss) is the tile's maximum taken, the reference moved and the tile's
  // weights formed again - from scores computed a second time, so that the ordinary path keeps no
  // copy of them and takes no maximum at all.  A row's first tile always goes that way (reference
  // -1e30: the weights overflow).
  float m_run = kNegBig, l_run = 0.f;
  const int koff = rows_read_offset(lane), voff = TILE + cols_read_offset(lane);

  int stage = 0;
  auto scores = [&](const char* ka) BC_INLINE {
    f32x16_t s = f32x16_t{0.f};
#pragma unroll
    for (int i = 0; i < KS; ++i)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          *reinterpret_cast<const bf16x8_t*>(ka + rows_read_imm<D>(i)), qb[i], s, 0, 0, 0);
    return s;
  };
  auto work = [&](int kt, auto masked) BC_INLINE {
    constexpr bool MASKED = decltype(masked)::value;
    const char* tile = lds + stage * (2 * TILE);
    uint32_t see = ~0u;
    if constexpr (MASKED) see = runs.visible((kt - runs.dense) * kTileRows, r, own, lane) >> (4 * half);
    float pe[16];
    uint32_t h16[8];
    float psum;
    auto weights = [&](const f32x16_t& s) BC_INLINE {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        pe[e] = fast_exp2(fmaf(s[e], p.qscale, -m_run));
        if constexpr (MASKED) pe[e] = keep_if_visible(pe[e], see, e);
      }
      if constexpr (HALF) {
        // the denominators are summed from the rounded weights that enter the value product, so that
        // numerator and denominator carry the same rounding: what is left of it in o is second order
        psum = 0.f;
        const pf_f16x2_t one2 = {(_Float16)1.f, (_Float16)1.f};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const pf_f16x2_t h2 = __builtin_convertvector(pf_f32x2_t{pe[2 * e], pe[2 * e + 1]}, pf_f16x2_t);
          psum = __builtin_amdgcn_fdot2(h2, one2, psum, false);
          h16[e] = __builtin_bit_cast(uint32_t, h2);
        }
      } else {
        psum = (((pe[0] + pe[1]) + (pe[2] + pe[3])) + ((pe[4] + pe[5]) + (pe[6] + pe[7]))) +
               (((pe[8] + pe[9]) + (pe[10] + pe[11])) + ((pe[12] + pe[13]) + (pe[14] + pe[15])));
      }
    };
    // The order of a pass is written out (step_fence(): nothing is moved across), LDS operands are asked for several instructions
    // ahead and not, as the compiler has it, in front of the instruction that takes them (three short trajectories 14.8 -> 14.2 us;
    // 27,109 rows of 32/8 heads with the half-precision form 389 -> 385; 16 trajectories of 8688 rows, at the power limit, take what
    // they took).
    bf16x8_t r[KS], c[2 * NJ];
    auto col_of = [&](int n) BC_INLINE { return cols_operand<D>(tile + voff, n % NJ, n / NJ); };
#pragma unroll
    for (int i = 0; i < KS; ++i) r[i] = *reinterpret_cast<const bf16x8_t*>(tile + koff + rows_read_imm<D>(i));
    step_fence();
    {
      f32x16_t s = f32x16_t{0.f};
#pragma unroll
      for (int i = 0; i < KS; ++i) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(r[i], qb[i], s, 0, 0, 0);
        if (i >= KS - NJ) c[i - KS + NJ] = col_of(i - KS + NJ);
        step_fence();
      }
      // the next loads, behind the scores' matrix instructions: at the head of the pass the four
      // waves' sixteen instructions stood in front of all matrix work
      if (kt + 2 < NT) issue_tile(stage >= 1 ? stage - 1 : kTileStages - 1);
      weights(s);
    }
    if (__builtin_expect(__any(psum > kPfRedo), 0)) {
      const f32x16_t s = scores(tile + opaque(koff));     // (reads the operands again)
      float tmax = kNegBig;
#pragma unroll
      for (int e = 0; e < 16; ++e) tmax = fmaxf(tmax, visible_bit(see, e) ? s[e] : kNegBig);
      tmax = halves_max(tmax);
      const float m_cand = tmax * p.qscale;
      const float m_new = m_cand > m_run + kPfLazy ? m_cand : m_run;
      const float alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int j = 0; j < NJ; ++j) O[j] *= alpha;
      weights(s);
    }
    l_run += psum;
    // O^T += V^T . P^T ; V^T through the transposing LDS read
    if constexpr (HALF) {
      step_fence();
#pragma unroll
      for (int n = 0; n < 2 * NJ; ++n) {
        const uint32_t* w = h16 + 4 * (n / NJ);
        O[n % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(pf_f16x8_t, c[n]),
                                                           __builtin_bit_cast(pf_f16x8_t, make_uint4(w[0], w[1], w[2], w[3])),
                                                           O[n % NJ], 0, 0, 0);
        if (n + NJ < 2 * NJ) c[n + NJ] = col_of(n + NJ);
        step_fence();
      }
    } else {
      Parts y;
#pragma unroll
      for (int g = 0; g < 4; ++g) y.split(g, pe[2 * g], pe[2 * g + 1]);
      step_fence();
#pragma unroll
      for (int m = 0; m < 4 * NJ; ++m) {
        const int n = m / 2;
        O[n % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(c[n], y.operand(m & 1, n / NJ), O[n % NJ], 0, 0, 0);
        if (m % 2 == 0 && n + NJ < 2 * NJ) c[n + NJ] = col_of(n + NJ);
#pragma unroll
        for (int g = 4; g < 8; ++g)
          if (m == (g - 4) * NJ / 2) y.split(g, pe[2 * g], pe[2 * g + 1]);
        step_fence();
      }
    }
  };
  // tile kt has landed (this wave's part); after the barrier everyone's part has, and everyone has
  // finished tile kt-1, whose stage is the one tile kt+2 goes into
  auto begin_pass = [&](int kt) BC_INLINE {
    if (kt + 1 < NT) wait_vmcnt<2 * NLD>();         // (the next tile's loads may stay out)
    else wait_vmcnt<0>();
    lds_barrier();
  };
  auto end_pass = [&]() BC_INLINE { stage = stage + 1 == kTileStages ? 0 : stage + 1; };

  int kt = 0;
  for (const int nd = min(runs.dense, ntw); kt < nd; ++kt) {
    begin_pass(kt);
    work(kt, std::false_type{});
    end_pass();
  }
  for (; kt < ntw; ++kt) {
    begin_pass(kt);
    work(kt, std::true_type{});
    end_pass();
  }
  for (; kt < NT; ++kt) {
    begin_pass(kt);
    if (kt + 2 < NT) issue_tile(stage >= 1 ? stage - 1 : kTileStages - 1);
    end_pass();
  }
  lds_barrier();          // the tile stages are free: the epilogue reuses LDS
  if (ntw == 0) return;

  // ---- epilogue: normalise, transpose through LDS, write the rows in bursts of OW floats
  const float l = halves_sum(l_run);
  const float inv = 1.0f / l;
  float* my = reinterpret_cast<float*>(lds + wave * (32 * OW * 4));
#pragma unroll
  for (int pass = 0; pass < 2; ++pass)
    store_rows<D>(my, O, inv, pass, lane, p.out + ((off0 + rw0) * p.Hq + kvh * p.g + head) * D, p.Hq * D,
                  [&](int t) { return rw0 + t <= rw1 ? t : -1; });
  if (p.lse && half == 0 && rw0 + col <= rw1)
    p.lse[(off0 + r) * p.Hq + kvh * p.g + head] = (m_run + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
}

// EITHER: the form the conversion pass found V to fit, one of the two by a branch that is uniform over the launch.  (As two
// launches, of which one left at its first instruction, with a third that cleared the verdict and a fourth that stored the tables, a
// call took 30 us where its kernels' work is 10 to 15; now 19.  Large launches run at the power limit: 27,109 rows 489 us, both.
// Both forms in one kernel keep 24 to 30 scalar registers in vector lanes, and at d = 64 four waves a SIMD where the half-precision form alone had five.  That
// costs nothing that shows: read afresh in each form, without spills, 16 trajectories of 8688 rows, d = 64, 367 us and 363, 27,109 rows of 32/8 heads 287 and 287,
// d = 128 484 and 486, three short ones 19.4 to 20.8 and 19.9.)
template <int D, bool EITHER, bool WIDE>
__global__ __launch_bounds__(kTileWaves * 64, 3) void prefill_kernel(PrefillParams p) {
  __shared__ __attribute__((aligned(1024))) char lds[prefill_lds<D>()];
  if constexpr (EITHER) {
    static_assert(kPfFlagBytes == 64 * 4, "a word of verdicts per lane");
    if (!__any(p.flags[threadIdx.x & 63] != 0)) {
      prefill_rows<D, true, WIDE>(p, lds);
      return;
    }
  }
  prefill_rows<D, false, WIDE>(p, lds);
}

// V in half precision for the workspace form, 8 entries per unit.  Each workgroup leaves a verdict byte: whether a
// finite entry of its does not fit (65520 and beyond rounds to infinity).  One workgroup of sixteen waves per compute
// unit, four units of a thread on their way together: 27,109 rows of 8 heads, 55 MB read and 55 written, 21 us.
__global__ __launch_bounds__(1024) void prefill_v16_kernel(const uint4* __restrict__ v, uint4* __restrict__ v16,
                                                           int64_t units, uint8_t* flags) {
  __shared__ int s_over;
  if (threadIdx.x == 0) s_over = 0;
  __syncthreads();
  bool over = false;
  const int64_t step = (int64_t)gridDim.x * 1024;
  for (int64_t i0 = (int64_t)blockIdx.x * 1024 + threadIdx.x; i0 < units; i0 += 4 * step) {
    u32x4_t x[4];
#pragma unroll
    for (int n = 0; n < 4; ++n)
      x[n] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(v + (i0 + n * step < units ? i0 + n * step : i0)));
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      float f[8];
      unpack16(make_uint4(x[n].x, x[n].y, x[n].z, x[n].w), f, bf16_t{});
      uint32_t h[4];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        over = over || (fabsf(f[e]) >= 65520.f && fabsf(f[e]) < __builtin_inff()) ||
               (fabsf(f[e + 1]) >= 65520.f && fabsf(f[e + 1]) < __builtin_inff());
        h[e >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pf_f32x2_t{f[e], f[e + 1]}, pf_f16x2_t));
      }
      if (i0 + n * step < units) v16[i0 + n * step] = make_uint4(h[0], h[1], h[2], h[3]);
    }
  }
  if (__any(over) && (threadIdx.x & 63) == 0) atomicOr(&s_over, 1);
  __syncthreads();
  // (workgroups that are not there are answered for by the first)
  if (threadIdx.x == 0) flags[blockIdx.x] = (uint8_t)s_over;
  if (blockIdx.x == 0 && threadIdx.x >= gridDim.x && threadIdx.x < kPfFlagBytes) flags[threadIdx.x] = 0;
}

// Words that travel in the kernel arguments.  Two sizes: the small one is what 31 trajectories take; the large
// one keeps the arguments under 4 KB, and more trajectories take more launches.
template <int N> struct ArgumentWords {
  uint32_t* dst;
  int32_t n;
  uint32_t w[N];
};
template <int N>
__global__ __launch_bounds__(256) void store_words_kernel(ArgumentWords<N> a) {
  typedef __attribute__((address_space(4))) const uint32_t const_word_t;      // (a.w[i] would go through scratch)
  const_word_t* w = (const_word_t*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(ArgumentWords<N>, w) / 4;
  for (int i = threadIdx.x; i < a.n; i += blockDim.x) a.dst[i] = w[i];
}
template <int N>
static void store_words(uint32_t* dst, const uint32_t* src, int n, hipStream_t hs) {
  ArgumentWords<N> a;
  a.dst = dst;
  a.n = n;
  memcpy(a.w, src, (size_t)n * 4);
  store_words_kernel<N><<<1, 256, 0, hs>>>(a);
}
static void store_words(uint32_t* dst, const void* src, int64_t n, hipStream_t hs) {
  constexpr int kFew = 126, kMany = 1000;
  const uint32_t* from = static_cast<const uint32_t*>(src);
  for (int64_t at = 0; at < n; at += kMany) {
    const int m = (int)(n - at < kMany ? n - at : kMany);
    if (m <= kFew) store_words<kFew>(dst + at, from + at, m, hs);
    else store_words<kMany>(dst + at, from + at, m, hs);
  }
}

template <int D, bool EITHER>
static void launch_prefill_d(const PrefillParams& p, bool wide, dim3 grid, hipStream_t hs) {
  if (wide) prefill_kernel<D, EITHER, true><<<grid, kTileWaves * 64, 0, hs>>>(p);
  else prefill_kernel<D, EITHER, false><<<grid, kTileWaves * 64, 0, hs>>>(p);
}
template <bool EITHER>
static void launch_prefill(const PrefillParams& p, int d, bool wide, dim3 grid, hipStream_t hs) {
  if (d == 128) launch_prefill_d<128, EITHER>(p, wide, grid, hs);
  else launch_prefill_d<64, EITHER>(p, wide, grid, hs);
}

// Shared by the entry points; p has its tables.  workspace == nullptr: the two-part form alone.
static int32_t prefill_forward(PrefillParams& p, const bc_shape* shape, const void* q, const void* k, const void* v,
                               int32_t max_rows, int64_t total_rows, float* out, float* lse, void* workspace,
                               void* stream) {
  p.q = static_cast<const char*>(q);
  p.k = static_cast<const char*>(k);
  p.v = static_cast<const char*>(v);
  p.v16 = nullptr; p.flags = nullptr;
  p.out = out; p.lse = lse;
  p.Hq = shape->Hq; p.Hkv = shape->Hkv; p.g = shape->Hq / shape->Hkv;
  p.qscale = shape->scale * kLog2e;
  p.tiling = head_tiling(p.g);
  p.npairs = shape->Hkv * shape->B;
  p.pstride = pair_stride(p.npairs);
  p.turn = pair_turn(p.pstride);
  const int rows_wg = kTileRows * p.tiling.row_blocks;
  const dim3 grid(p.tiling.splits * p.pstride, (max_rows + rows_wg - 1) / rows_wg);
  const bool wide = rows_span_4gb(max_rows, shape);
  hipStream_t hs = as_stream(stream);
  if (workspace) {
    char* v16 = static_cast<char*>(workspace) + kPfFlagBytes;
    const int64_t units = total_rows * shape->Hkv * shape->d / 8;
    const int64_t blocks = (units + 1023) / 1024;
    prefill_v16_kernel<<<(int)(blocks < (int64_t)kPfFlagBytes ? blocks : (int64_t)kPfFlagBytes), 1024, 0, hs>>>(
        static_cast<const uint4*>(v), reinterpret_cast<uint4*>(v16), units, static_cast<uint8_t*>(workspace));
    p.v16 = v16; p.flags = static_cast<const uint32_t*>(workspace);
    launch_prefill<true>(p, shape->d, wide, grid, hs);
  } else {
    launch_prefill<false>(p, shape->d, wide, grid, hs);
  }
  return launch_status();
}

// What every form checks; the tables are device or host arrays.
static int32_t check_prefill(const bc_shape* shape, const void* q, const void* k, const void* v, const void* row_offsets,
                             const void* P, const void* c, int32_t max_rows, const float* out) {
  const int32_t st = check_shape(shape);
  if (st != BC_OK) return st;
  if (shape->kv_dtype != BC_BF16) return BC_ERR_SHAPE;
  if (!q || !k || !v || !row_offsets || !P || !c || !out) return BC_ERR_ARG;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out)) return BC_ERR_ARG;
  if (max_rows < 1 || max_rows >= (1 << 26)) return BC_ERR_ARG;
  if (!positive_finite(shape->scale)) return BC_ERR_ARG;       // the kernel takes maxima of unscaled scores
  return BC_OK;
}
static int32_t check_prefill_workspace(const bc_shape* shape, int32_t max_rows, int64_t total_rows, const void* workspace,
                                       size_t workspace_bytes) {
  if (total_rows < max_rows) return BC_ERR_ARG;
  if (!workspace || !aligned16(workspace) || workspace_bytes < bc_prefill_workspace_bytes(shape, total_rows))
    return BC_ERR_WORKSPACE;
  return BC_OK;
}

}  // namespace bc

using namespace bc;

extern "C" int32_t bc_trajectory_tables(const int64_t* row_offsets, const int32_t* P, const int32_t* c, int32_t B,
                                        void* tables, void* stream) {
  if (!row_offsets || !P || !c || !tables || (reinterpret_cast<uintptr_t>(tables) & 7u)) return BC_ERR_ARG;
  if (B < 1) return BC_ERR_SHAPE;
  hipStream_t hs = as_stream(stream);
  uint32_t* dst = static_cast<uint32_t*>(tables);
  const int64_t offset_words = 2 * ((int64_t)B + 1);
  if (P == reinterpret_cast<const int32_t*>(row_offsets + B + 1) && c == P + B) {      // one array already
    store_words(dst, row_offsets, offset_words + 2 * (int64_t)B, hs);
  } else {
    store_words(dst, row_offsets, offset_words, hs);
    store_words(dst + offset_words, P, B, hs);
    store_words(dst + offset_words + B, c, B, hs);
  }
  return launch_status();
}

extern "C" size_t bc_prefill_workspace_bytes(const bc_shape* shape, int64_t total_rows) {
  if (check_shape(shape) != BC_OK || total_rows < 1) return 0;
  return kPfFlagBytes + (size_t)total_rows * shape->Hkv * shape->d * 2;
}

extern "C" int32_t bc_prefill_attn_ws(const bc_shape* shape, const void* q, const void* k,
                                      const void* v, const int64_t* row_offsets, const int32_t* P,
                                      const int32_t* c, int32_t max_rows, int64_t total_rows,
                                      float* out, float* lse, void* workspace,
                                      size_t workspace_bytes, void* stream) {
  int32_t st = check_prefill(shape, q, k, v, row_offsets, P, c, max_rows, out);
  if (st != BC_OK) return st;
  st = check_prefill_workspace(shape, max_rows, total_rows, workspace, workspace_bytes);
  if (st != BC_OK) return st;
  PrefillParams p;
  p.row_off = row_offsets; p.P = P; p.c = c;
  return prefill_forward(p, shape, q, k, v, max_rows, total_rows, out, lse, workspace, stream);
}

extern "C" int32_t bc_prefill_attn(const bc_shape* shape, const void* q, const void* k,
                                   const void* v, const int64_t* row_offsets, const int32_t* P,
                                   const int32_t* c, int32_t max_rows, float* out, float* lse,
                                   void* stream) {
  const int32_t st = check_prefill(shape, q, k, v, row_offsets, P, c, max_rows, out);
  if (st != BC_OK) return st;
  PrefillParams p;
  p.row_off = row_offsets; p.P = P; p.c = c;
  return prefill_forward(p, shape, q, k, v, max_rows, 0, out, lse, nullptr, stream);
}

extern "C" int32_t bc_prefill_attn_host(const bc_shape* shape, const void* q, const void* k, const void* v,
                                        const int64_t* row_offsets, const int32_t* P, const int32_t* c,
                                        int32_t max_rows, int64_t total_rows, float* out, float* lse, void* tables,
                                        void* workspace, size_t workspace_bytes, void* stream) {
  int32_t st = check_prefill(shape, q, k, v, row_offsets, P, c, max_rows, out);
  if (st != BC_OK) return st;
  if (workspace) {
    st = check_prefill_workspace(shape, max_rows, total_rows, workspace, workspace_bytes);
    if (st != BC_OK) return st;
  }
  PrefillParams p;
  st = host_tables(p, row_offsets, P, c, shape->B, tables, stream);
  if (st != BC_OK) return st;
  return prefill_forward(p, shape, q, k, v, max_rows, total_rows, out, lse, workspace, stream);
}

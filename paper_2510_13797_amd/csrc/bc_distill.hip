// Token-level distillation loss (Eq. 1, Sec. 3.2) against a teacher stored as its top-k logits
// per token (App. A): forward (per-token KL, student log-sum-exp, mean) and the gradient with
// respect to the student's logits.  Both are one streaming pass over the [T, V] logits: one
// workgroup per token, 16-byte loads, a running (max, sum) per thread that is rescaled once per
// batch of loads, and a workgroup reduction at the end.  HBM-bound by construction.
//
// A row may start at any element (V odd in bf16: every second row is 2 bytes off): the elements in
// front of its first 16-byte boundary and behind its last one are taken one by one by the first
// threads, everything between by 16-byte units (509 rows of 50,257 bf16, loss and gradient pass: 63 -> 13 and
// 73 -> 20 us against one element per load).
#include "bc_common.h"

namespace bc {
namespace {

constexpr int kDistillThreads = 256;       // threads of a workgroup: ordinary,
constexpr int kDistillThreadsMany = 1024;  // and for few, long rows (many_threads())
constexpr int kMaxTeacher = 1024;          // largest k
constexpr float kLn2 = 0.6931471805599453f;

struct DistillParams {
  const void* z;            // [T, V] student logits
  const float* tl;          // [T, k] teacher top-k logits
  const int32_t* tidx;      // [T, k] their token ids
  float* loss;              // [T]
  float* lse;               // [T]   (forward: nullable output; backward: input)
  void* dz;                 // [T, V] backward output, dtype of z
  int64_t T;
  int32_t V, k;
  float grad_scale;
};

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
// every thread gets the result; red: NW floats of LDS, reusable after the call
template <int NW>
__device__ __forceinline__ float block_max(float x, float* red) {
  x = wave_max(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) r = fmaxf(r, red[i]);
  return r;
}
template <int NW>
__device__ __forceinline__ float block_sum(float x, float* red) {
  x = wave_sum(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) r += red[i];   // fixed order: reproducible
  return r;
}

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
// 16 bytes of the logits.  KEEP: leave them in the Infinity Cache, where the gradient pass finds what the loss
// pass read; otherwise out of the way of the caches (see logits_kept()).
template <bool KEEP>
__device__ __forceinline__ uint4 load16_logits(const uint4* p) {
  if constexpr (KEEP) return *p;
  const u32x4_t r = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(r.x, r.y, r.z, r.w);
}

// one element as its bits, and what the bits mean
template <typename T> __device__ __forceinline__ uint32_t load_bits(const void* p, int64_t i);
template <> __device__ __forceinline__ uint32_t load_bits<float>(const void* p, int64_t i) {
  return static_cast<const uint32_t*>(p)[i];
}
template <> __device__ __forceinline__ uint32_t load_bits<bf16_t>(const void* p, int64_t i) {
  return static_cast<const uint16_t*>(p)[i];
}
template <typename T> __device__ __forceinline__ float bits_value(uint32_t u) {
  return __uint_as_float(Elem<T>::size == 4 ? u : u << 16);
}
template <typename T> __device__ __forceinline__ float load_elem(const void* p, int64_t i) {
  return bits_value<T>(load_bits<T>(p, i));
}
__device__ __forceinline__ uint32_t bf16_rne(float f) {   // finite or inf/nan preserved
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
typedef __attribute__((ext_vector_type(2))) float ds_f32x2_t;
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {   // RNE, a in the low half
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(ds_f32x2_t{a, b}, bf16x2_t));
}
__device__ __forceinline__ void store16_stream(uint4* p, const uint4& w) {
  __builtin_nontemporal_store(u32x4_t{w.x, w.y, w.z, w.w}, reinterpret_cast<u32x4_t*>(p));
}
template <typename T> __device__ __forceinline__ void store_elem(void* p, int64_t i, float x);
template <> __device__ __forceinline__ void store_elem<float>(void* p, int64_t i, float x) {
  static_cast<float*>(p)[i] = x;
}
template <> __device__ __forceinline__ void store_elem<bf16_t>(void* p, int64_t i, float x) {
  static_cast<uint16_t*>(p)[i] = static_cast<uint16_t>(bf16_rne(x));
}

// A row of V elements as what lies in front of its first 16-byte boundary, whole 16-byte units, and
// the rest.
struct RowSpan {
  int32_t head, units, tail;
  // the element in front of or behind the units that is this thread's, if any (there are at most 14)
  __device__ __forceinline__ bool has_edge() const { return static_cast<int>(threadIdx.x) < head + tail; }
  __device__ __forceinline__ int32_t edge(int32_t V) const {
    const int32_t i = threadIdx.x;
    return i < head ? i : V - tail + (i - head);
  }
};
template <typename T>
__device__ __forceinline__ RowSpan row_span(const void* row, int32_t V) {
  RowSpan r;
  const int32_t off = static_cast<int32_t>(reinterpret_cast<uintptr_t>(row) & 15u);
  r.head = min(((16 - off) & 15) / Elem<T>::size, V);
  r.units = (V - r.head) / Elem<T>::per16;
  r.tail = V - r.head - r.units * Elem<T>::per16;
  return r;
}

// f(b, valid) for the B units base + b * NT + tid of a batch: no tests in a full batch, and in the last one the
// steps that do not exist are left out: each by a test and jump of its own, or (CHAIN) all by one jump.  A row of 1000
// logits has one step and seven to leave out: the loss of 1000 such rows takes 5.1 us with CHAIN, 5.6 without;
// of 4096 x 151,936 logits 190 and 187.  (Clamped loads in place of masked ones: 12.5 us for 1000 rows of 16,000
// logits instead of 9.7.)
template <int NT, int B, int I = 0, typename F>
__device__ __forceinline__ void for_first_steps(int base, int units, const F& f) {
  if (base + I * NT < units) {
    f(I, base + I * NT + static_cast<int>(threadIdx.x) < units);
    if constexpr (I + 1 < B) for_first_steps<NT, B, I + 1>(base, units, f);
  }
}
template <int NT, int B, bool CHAIN, typename F>
__device__ __forceinline__ void for_batch(int base, int units, const F& f) {
  if (base + B * NT <= units) {
#pragma unroll
    for (int b = 0; b < B; ++b) f(b, true);
  } else if constexpr (CHAIN) {
    for_first_steps<NT, B>(base, units, f);
  } else {
#pragma unroll
    for (int b = 0; b < B; ++b)
      if (base + b * NT < units) f(b, base + b * NT + static_cast<int>(threadIdx.x) < units);
  }
}

// Running log-sum-exp of one row in the base-2 domain: returns (max, sum of 2^(x*log2e - max))
// reduced over the workgroup.
template <typename T, int NT, int B, bool KEEP>
__device__ __forceinline__ void row_lse(const void* zrow, int32_t V, float* red, float& m_out,
                                        float& s_out) {
  constexpr int EPU = Elem<T>::per16;
  const RowSpan span = row_span<T>(zrow, V);
  const uint4* row = reinterpret_cast<const uint4*>(static_cast<const char*>(zrow) + span.head * Elem<T>::size);
  float m = kNegBig, s = 0.f;
  uint32_t edge = 0;              // (looked at behind the units: one round trip for both)
  if (span.has_edge()) edge = load_bits<T>(zrow, span.edge(V));
  for (int base = 0; base < span.units; base += NT * B) {
    uint4 r[B];
    for_batch<NT, B, KEEP>(base, span.units, [&](int b, bool valid) {
      if (valid) r[b] = load16_logits<KEEP>(row + base + b * NT + threadIdx.x);
    });
    float bm = kNegBig;
    for_batch<NT, B, KEEP>(base, span.units, [&](int b, bool valid) {
      float x[EPU];
      unpack16(r[b], x, T{});
      float um = kNegBig;
#pragma unroll
      for (int e = 0; e < EPU; ++e) um = fmaxf(um, x[e]);
      if (valid) bm = fmaxf(bm, um);
    });
    const float mn = fmaxf(m, bm * kLog2e);
    s *= fast_exp2(m - mn);
    m = mn;
    for_batch<NT, B, KEEP>(base, span.units, [&](int b, bool valid) {
      float x[EPU];
      unpack16(r[b], x, T{});
      float acc = 0.f;
#pragma unroll
      for (int e = 0; e < EPU; ++e) acc += fast_exp2(fmaf(x[e], kLog2e, -m));
      if (valid) s += acc;
    });
  }
  if (span.has_edge()) {
    const float x = bits_value<T>(edge) * kLog2e, mn = fmaxf(m, x);
    s = s * fast_exp2(m - mn) + fast_exp2(x - mn);
    m = mn;
  }
  const float M = block_max<NT / 64>(m, red);
  s_out = block_sum<NT / 64>(s * fast_exp2(m - M), red);
  m_out = M;
}

// Teacher side of one token: softmax over its k stored logits.  Each thread keeps the entries
// i = tid, tid + NT, ... (at most kMaxTeacher / NT of them).

template <typename T, int NT, int B, bool KEEP>
__global__ void __launch_bounds__(NT)
topk_kl_fwd_kernel(DistillParams p) {
  constexpr int kPerThread = kMaxTeacher / NT;
  __shared__ float red[NT / 64];
  const int64_t t = blockIdx.x;
  const void* zrow = static_cast<const char*>(p.z) + t * p.V * Elem<T>::size;
  // the k gathered student logits and the teacher row first: their latency hides behind the stream
  float zs[kPerThread], tl[kPerThread];
  bool bad = false;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) {
    const int i = threadIdx.x + j * NT;
    zs[j] = 0.f; tl[j] = kNegBig;
    if (i < p.k) {
      int32_t id = p.tidx[t * p.k + i];
      if (id < 0 || id >= p.V) { bad = true; id = 0; }
      zs[j] = load_elem<T>(zrow, id);
      tl[j] = p.tl[t * p.k + i];
    }
  }
  float m2, s2;
  row_lse<T, NT, B, KEEP>(zrow, p.V, red, m2, s2);
  const float lse_s = (m2 + __log2f(s2)) * kLn2;
  float tm = kNegBig;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) tm = fmaxf(tm, tl[j]);
  tm = block_max<NT / 64>(tm, red);
  float ts = 0.f;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) ts += fast_exp2((tl[j] - tm) * kLog2e);
  ts = block_sum<NT / 64>(ts, red);
  const float lse_t = tm + __log2f(ts) * kLn2;
  float kl = 0.f;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) {
    const int i = threadIdx.x + j * NT;
    if (i < p.k) {
      const float lpt = tl[j] - lse_t;
      kl += fast_exp2(lpt * kLog2e) * (lpt - (zs[j] - lse_s));
    }
  }
  if (bad) kl = __builtin_nanf("");
  kl = block_sum<NT / 64>(kl, red);
  if (threadIdx.x == 0) {
    p.loss[t] = kl;
    if (p.lse) p.lse[t] = lse_s;
  }
}

// mean of T floats in double, one workgroup, fixed order
__global__ void __launch_bounds__(1024) mean_kernel(const float* x, int64_t T, float* out) {
  __shared__ double part[1024];
  double a = 0.0;
  for (int64_t i = threadIdx.x; i < T; i += 1024) a += static_cast<double>(x[i]);
  part[threadIdx.x] = a;
  __syncthreads();
  for (int s = 512; s >= 1; s >>= 1) {
    if (static_cast<int>(threadIdx.x) < s) part[threadIdx.x] += part[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = static_cast<float>(part[0] / static_cast<double>(T));
}

template <typename T, bool VEC, int NT, int B, bool KEEP>
__global__ void __launch_bounds__(NT)
topk_kl_bwd_kernel(DistillParams p) {
  constexpr int kPerThread = kMaxTeacher / NT;
  __shared__ float red[NT / 64];
  constexpr int EPU = Elem<T>::per16;
  const int64_t t = blockIdx.x;
  const void* zrow = static_cast<const char*>(p.z) + t * p.V * Elem<T>::size;
  void* drow = static_cast<char*>(p.dz) + t * p.V * Elem<T>::size;
  const float nl = -p.lse[t] * kLog2e;
  const float gs = p.grad_scale;
  // teacher probabilities of this token
  float tl[kPerThread];
  int32_t id[kPerThread];
  float tm = kNegBig;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) {
    const int i = threadIdx.x + j * NT;
    tl[j] = kNegBig; id[j] = -1;
    if (i < p.k) {
      tl[j] = p.tl[t * p.k + i];
      const int32_t x = p.tidx[t * p.k + i];
      id[j] = (x >= 0 && x < p.V) ? x : -1;
    }
    tm = fmaxf(tm, tl[j]);
  }
  tm = block_max<NT / 64>(tm, red);
  float ts = 0.f;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) ts += fast_exp2((tl[j] - tm) * kLog2e);
  ts = block_sum<NT / 64>(ts, red);
  const float inv_ts = 1.f / ts;

  if (VEC) {
    const RowSpan span = row_span<T>(zrow, p.V);
    const int off = span.head * Elem<T>::size;
    const uint4* row = reinterpret_cast<const uint4*>(static_cast<const char*>(zrow) + off);
    uint4* out = reinterpret_cast<uint4*>(static_cast<char*>(drow) + off);
    uint32_t edge = 0;
    if (span.has_edge()) edge = load_bits<T>(zrow, span.edge(p.V));
    for (int base = 0; base < span.units; base += NT * B) {
      uint4 r[B];
      for_batch<NT, B, true>(base, span.units, [&](int b, bool valid) {
        if (valid) r[b] = load16_logits<KEEP>(row + base + b * NT + threadIdx.x);
      });
      for_batch<NT, B, true>(base, span.units, [&](int b, bool valid) {
        float x[EPU];
        unpack16(r[b], x, T{});
#pragma unroll
        for (int e = 0; e < EPU; ++e) x[e] = gs * fast_exp2(fmaf(x[e], kLog2e, nl));
        uint4 w;
        if constexpr (EPU == 4) {
          w = make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]),
                         __float_as_uint(x[3]));
        } else {
          w = make_uint4(pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]),
                         pack_bf16(x[6], x[7]));
        }
        if (valid) store16_stream(out + base + b * NT + threadIdx.x, w);
      });
    }
    if (span.has_edge())
      store_elem<T>(drow, span.edge(p.V), gs * fast_exp2(fmaf(bits_value<T>(edge), kLog2e, nl)));
  } else {
    for (int v = threadIdx.x; v < p.V; v += NT)
      store_elem<T>(drow, v, gs * fast_exp2(fmaf(load_elem<T>(zrow, v), kLog2e, nl)));
  }
  // the k teacher ids: overwrite with softmax minus the teacher probability, computed afresh from
  // the logit (one rounding).  The barrier orders these stores after the streaming stores of the
  // same workgroup.
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) {
    if (id[j] >= 0) {
      const float ps = fast_exp2(fmaf(load_elem<T>(zrow, id[j]), kLog2e, nl));
      const float pt = fast_exp2((tl[j] - tm) * kLog2e) * inv_ts;
      store_elem<T>(drow, id[j], gs * (ps - pt));
    }
  }
}

int32_t check_distill(int64_t T, int32_t V, int32_t k, const void* z, int32_t dtype,
                      const float* tl, const int32_t* tidx) {
  if (!z || !tl || !tidx) return BC_ERR_ARG;
  if (dtype != BC_F32 && dtype != BC_BF16) return BC_ERR_SHAPE;
  if (T < 0 || T > 0x7fffffffLL || V < 1 || k < 1 || k > V ||
      k > kMaxTeacher)
    return BC_ERR_SHAPE;
  return BC_OK;
}

// The gradient's 16-byte units need rows of both tensors at the same place inside 16 bytes.
bool rows_aligned_alike(const void* a, const void* b) {
  return ((reinterpret_cast<uintptr_t>(a) ^ reinterpret_cast<uintptr_t>(b)) & 15u) == 0;
}

// Logits that fit the 256 MB Infinity Cache are loaded with the default policy: the gradient pass, which
// stores past the caches, then reads most of them from there (both passes, 600 x 151,936 in bf16 = 182 MB:
// 110 -> 96 us; 243 MB: 145 -> 126; 304 MB: 164 -> 163).  Beyond that they are streamed (395 MB: 233
// against 252 us, 622 MB: 343 against 376).
bool logits_kept(const DistillParams& p, int32_t dtype) {
  return p.T * p.V * elem_size(dtype) <= (int64_t(256) << 20);
}

// A token has a workgroup to itself, of 256 threads; 1024 where tokens leave compute units idle (256 or fewer) and a
// row keeps them busy, and with up to 1024 tokens where the logits are streamed from memory.  Loss and gradient pass
// in us, 256 against 1024 threads:
//   bf16, 64 x 151,936: 14.3, 12.5 and 14.1, 11.0; x 32,000: 6.45, 6.35 and 6.2, 5.4; x 16,000: 5.6, 5.7 and 4.95,
//   4.5; x 8000: 4.95, 5.35 and 4.15, 4.1; f32, 64 x 12,000: 5.3, 5.45 and 4.8, 4.5; x 50,257: 8.7, 7.6 and 8.7, 7.6
//   bf16, 512 x 8000: 5.5, 7.4 and 4.95, 5.55; 1000 x 1000: 5.1, 11.4 and 4.45, 7.85; 1000 x 50,257: 21.6, 23.1 and
//   34.9, 33.4 (201 MB: kept in the Infinity Cache)
//   bf16, 1000 x 151,936: 52.7, 50.1 and 121, 113; f32, 700 x 100,000: 46.0, 45.0 and 110, 106 (streamed); with
//   2048 tokens there is nothing to gain.
bool many_threads(const DistillParams& p, int32_t dtype) {
  return (p.T <= 256 && static_cast<int64_t>(p.V) * elem_size(dtype) >= (30 << 10)) ||
         (p.T <= 1024 && !logits_kept(p, dtype));
}

template <typename T, bool KEEP>
void launch_fwd(const DistillParams& p, int32_t dtype, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(p.T));
  if (many_threads(p, dtype)) topk_kl_fwd_kernel<T, kDistillThreadsMany, 4, KEEP><<<grid, kDistillThreadsMany, 0, s>>>(p);
  else topk_kl_fwd_kernel<T, kDistillThreads, 8, KEEP><<<grid, kDistillThreads, 0, s>>>(p);
}
template <typename T, bool VEC, bool KEEP>
void launch_bwd(const DistillParams& p, int32_t dtype, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(p.T));
  if (many_threads(p, dtype)) topk_kl_bwd_kernel<T, VEC, kDistillThreadsMany, 4, KEEP><<<grid, kDistillThreadsMany, 0, s>>>(p);
  else topk_kl_bwd_kernel<T, VEC, kDistillThreads, 8, KEEP><<<grid, kDistillThreads, 0, s>>>(p);
}
template <typename T>
void launch_bwd(const DistillParams& p, int32_t dtype, hipStream_t s) {
  if (!rows_aligned_alike(p.z, p.dz)) launch_bwd<T, false, true>(p, dtype, s);
  else if (logits_kept(p, dtype)) launch_bwd<T, true, true>(p, dtype, s);
  else launch_bwd<T, true, false>(p, dtype, s);
}
template <typename T>
void launch_fwd(const DistillParams& p, int32_t dtype, hipStream_t s) {
  if (logits_kept(p, dtype)) launch_fwd<T, true>(p, dtype, s);
  else launch_fwd<T, false>(p, dtype, s);
}

}  // namespace
}  // namespace bc

extern "C" int32_t bc_topk_kl_loss(int64_t T, int32_t V, int32_t k, const void* student_logits,
                                   int32_t logits_dtype, const float* teacher_logits,
                                   const int32_t* teacher_idx, float* loss_per_token,
                                   float* lse, float* loss_mean, void* stream) {
  using namespace bc;
  int32_t st = check_distill(T, V, k, student_logits, logits_dtype, teacher_logits, teacher_idx);
  if (st != BC_OK) return st;
  if (!loss_per_token) return BC_ERR_ARG;
  if (T == 0) return BC_OK;
  DistillParams p{};
  p.z = student_logits; p.tl = teacher_logits; p.tidx = teacher_idx;
  p.loss = loss_per_token; p.lse = lse; p.T = T; p.V = V; p.k = k;
  hipStream_t s = as_stream(stream);
  if (logits_dtype == BC_BF16) launch_fwd<bf16_t>(p, logits_dtype, s);
  else launch_fwd<float>(p, logits_dtype, s);
  if (loss_mean) hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(1024), 0, s, loss_per_token, T, loss_mean);
  return launch_status();
}

extern "C" int32_t bc_topk_kl_loss_bwd(int64_t T, int32_t V, int32_t k,
                                       const void* student_logits, int32_t logits_dtype,
                                       const float* teacher_logits, const int32_t* teacher_idx,
                                       const float* lse, float grad_scale, void* dlogits,
                                       void* stream) {
  using namespace bc;
  int32_t st = check_distill(T, V, k, student_logits, logits_dtype, teacher_logits, teacher_idx);
  if (st != BC_OK) return st;
  if (!lse || !dlogits || dlogits == student_logits) return BC_ERR_ARG;
  if (T == 0) return BC_OK;
  DistillParams p{};
  p.z = student_logits; p.tl = teacher_logits; p.tidx = teacher_idx;
  p.lse = const_cast<float*>(lse); p.dz = dlogits; p.T = T; p.V = V; p.k = k;
  p.grad_scale = grad_scale;
  hipStream_t s = as_stream(stream);
  if (logits_dtype == BC_BF16) launch_bwd<bf16_t>(p, logits_dtype, s);
  else launch_bwd<float>(p, logits_dtype, s);
  return launch_status();
}

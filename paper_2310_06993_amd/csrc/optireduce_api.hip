// C ABI of liboptireduce_hip: argument checks and kernel dispatch.  Semantics are stated in
// include/optireduce.h; nothing here allocates or synchronises.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "../../include/optireduce.h"
#include "launch_table.hpp"

namespace orhost {
extern const KernelTable or_kernel_table_0, or_kernel_table_11, or_kernel_table_12, or_kernel_table_13,
    or_kernel_table_14, or_kernel_table_15, or_kernel_table_16;

TimingEvents& timing_events() {
  static thread_local TimingEvents t = {nullptr, nullptr};
  return t;
}

const KernelTable* table_for_class(int cls) {
  switch (cls) {
    case 0: return &or_kernel_table_0;
    case 11: return &or_kernel_table_11;
    case 12: return &or_kernel_table_12;
    case 13: return &or_kernel_table_13;
    case 14: return &or_kernel_table_14;
    case 15: return &or_kernel_table_15;
    case 16: return &or_kernel_table_16;
    default: return nullptr;
  }
}
}  // namespace orhost

namespace {
using ordev::PathArgs;
using ordev::u64;

thread_local int g_last_hip_error = 0;

// ------------------------------------------------------------------ streaming masked sum + count
// Sec. 3.1.1 aggregation with no transform around it: each lane owns VEC consecutive entries (16
// bytes of one worker's shard), reads the VEC mask bits of every worker and adds under select.
// U workers are asked for at once, those that are left over two at once, PAIR, or one by one (the rules are at launch_masked_reduce and where
// k_masked_reduce_batched is launched).  `keep`: the results stay in the L2 for who reads them next.
template <class Wire, int VEC, int U, bool PAIR>
__device__ __forceinline__ void masked_reduce_at(const Wire* __restrict__ shards, const uint32_t* __restrict__ masks,
                                                 int N, u64 L, float* __restrict__ sum_out,
                                                 uint8_t* __restrict__ count_out, u64 e, bool keep) {
  if (e >= L) return;
  typedef Wire vec_t __attribute__((ext_vector_type(VEC)));
  const u64 words = L >> 5;
  float acc[VEC];
  uint32_t cnt[VEC];
#pragma unroll
  for (int j = 0; j < VEC; ++j) { acc[j] = 0.0f; cnt[j] = 0; }
  const int sh = (int)(e & 31);
  int i = 0;
  auto add = [&](auto at_once) {
    constexpr int W = decltype(at_once)::value;
    vec_t x[W];
    uint32_t m[W];
#pragma unroll
    for (int u = 0; u < W; ++u) {
      x[u] = __builtin_nontemporal_load((const vec_t*)(shards + (u64)(i + u) * L + e));
      m[u] = masks[(u64)(i + u) * words + (e >> 5)] >> sh;
    }
    // bf16: all of them, before the first is added; the compiler mixes them otherwise (fp32: it does not, and its own order is 2 to 4 % better in
    // launches of few entries).  us, with the mean, without -> with, N = 4 / 8 / 24, 20000 entries 4.50 -> 4.13 / 5.30 -> 4.58 / 8.83 -> 6.48
    if (sizeof(Wire) == 2) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < W; ++u)
#pragma unroll
      for (int j = 0; j < VEC; ++j) {
        const bool got = (m[u] >> j) & 1u;
        float f;
        if constexpr (sizeof(Wire) == 4) f = x[u][j]; else f = __builtin_bit_cast(float, (uint32_t)x[u][j] << 16);
        acc[j] += got ? f : 0.0f;
        cnt[j] += got ? 1u : 0u;
      }
    i += W;
  };
  while (i + U <= N) add(std::integral_constant<int, U>{});
  if (U > 4 && i + 4 <= N) add(std::integral_constant<int, 4>{});
  if (U > 2 && PAIR && i + 2 <= N) add(std::integral_constant<int, 2>{});
  if (U > 1) while (i < N) add(std::integral_constant<int, 1>{});
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 s[VEC / 4];
  uint32_t c[VEC / 4];
#pragma unroll
  for (int q = 0; q < VEC / 4; ++q) {
    s[q] = f4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    c[q] = cnt[4 * q] | (cnt[4 * q + 1] << 8) | (cnt[4 * q + 2] << 16) | (cnt[4 * q + 3] << 24);
  }
  const bool words_of_counts = ((uintptr_t)count_out & 3) == 0;
  if (keep) {
    ordev::keep_apart();
#pragma unroll
    for (int q = 0; q < VEC / 4; ++q) *(f4*)(sum_out + e + 4 * q) = s[q];
    if (words_of_counts) {
#pragma unroll
      for (int q = 0; q < VEC / 4; ++q) *(uint32_t*)(count_out + e + 4 * q) = c[q];
    }
    ordev::keep_apart();
  } else {
#pragma unroll
    for (int q = 0; q < VEC / 4; ++q) __builtin_nontemporal_store(s[q], (f4*)(sum_out + e + 4 * q));
    if (words_of_counts) {
#pragma unroll
      for (int q = 0; q < VEC / 4; ++q) __builtin_nontemporal_store(c[q], (uint32_t*)(count_out + e + 4 * q));
    }
  }
  if (!words_of_counts) {   // or_reduce_decode* takes counts at any address
#pragma unroll
    for (int j = 0; j < VEC; ++j) count_out[e + j] = (uint8_t)cnt[j];
  }
}

template <class Wire, int VEC, int U>
__global__ __launch_bounds__(256) void k_masked_reduce(const Wire* __restrict__ shards,
                                                       const uint32_t* __restrict__ masks, int N, u64 L,
                                                       float* __restrict__ sum_out, uint8_t* __restrict__ count_out, bool keep) {
  masked_reduce_at<Wire, VEC, U, true>(shards, masks, N, L, sum_out, count_out, ((u64)blockIdx.x * 256 + threadIdx.x) * VEC, keep);
}

// several buckets in one launch (a 25 MiB bucket is a few hundred workgroups here): descriptors in the kernel
// arguments; workgroup x serves entries of bucket j from (x - start[j]) * 256 * VEC on
struct ReduceBucket {
  const void* shards;
  const uint32_t* masks;
  float* sum;
  uint8_t* count;
  u64 L;
};
struct ReduceBatch {
  int n, N;
  uint32_t start[ordev::kMaxBatch + 1];
  ReduceBucket b[ordev::kMaxBatch];
};
static_assert(sizeof(ReduceBatch) <= 4096, "kernel arguments are limited to 4 KB");
// Four workers at once and results past the caches, whatever the size.  What is left over, pair -> one by one, us, bf16: N = 2 / 3 / 7, 24 buckets of 16384
// entries 3.98 -> 4.22 / 4.65 -> 4.99 / 5.68 -> 6.14, 24 of 819200 34.4 -> 33.5 / 39.3 -> 39.3 / 63.6 -> 63.1, N = 2, two of 26188800 97.2 -> 86.1;  fp32: N = 2 / 6, 24 of 819200
// 42.1 -> 44.1 / 95.5 -> 95.8.
constexpr u64 kBatchPairTo = 2048;   // workgroups
template <class Wire, int VEC, bool PAIR>
__global__ __launch_bounds__(256) void k_masked_reduce_batched(ReduceBatch rb) {
  const uint32_t x = blockIdx.x;
  int j = 0;
  while (j + 1 < rb.n && rb.start[j + 1] <= x) ++j;
  masked_reduce_at<Wire, VEC, 4, PAIR>((const Wire*)rb.b[j].shards, rb.b[j].masks, rb.N, rb.b[j].L, rb.b[j].sum, rb.b[j].count,
                              ((u64)(x - rb.start[j]) * 256 + threadIdx.x) * VEC, false);
}

// Workers asked for at once.  A launch of few workgroups waits for every batch: eight at once.  us, four -> eight, reduce + finalize,
// bf16, 65536 entries, N = 16 / 32 6.7 -> 6.1 / 9.3 -> 8.2, 524288 entries 8.7 -> 8.0 / 12.8 -> 11.2, but 1048576 entries, N = 8 / 32 8.9 -> 9.2 /
// 16.9 -> 17.8.  fp32 launches that fill the chip many times over do best with as few rows of memory open as
// possible: one.  us, four -> one, 3194880 entries, N = 8 / 32 28.4 -> 28.0 / 83.7 -> 80.9, 12345664 entries 99.8 -> 97.0 / 306 -> 293, 8388608
// entries (rows a power of two apart) 72.3 -> 66.6 / 213 -> 202, but 1000000 entries 11.8 -> 12.8 / 28.0 -> 30.9, and a few workgroups more than
// run at once (2048) are a long chain: 2100000 entries, N = 12 25.5 -> 28.3; bf16, of half as many bytes, from 16 workers on
// and later: 8388608 / 12345664 entries, N = 16 71.0 -> 65.6 / 98.2 -> 96.2, N = 32 131 -> 109 / 167 -> 161, but N = 8 44.2 -> 43.1 / 63.3 -> 64.6, 6000000
// entries, N = 16 48.4 -> 50.2; and with two workers where sum and counts go past the caches: us of the reduce by itself, a pair at once -> one,
// 40000000 / 60000000 / 120000000 entries 72.2 -> 66.2 / 108 -> 97.5 / 218 -> 193, but kept, 14000000 entries 24.7 -> 26.0 (N = 3, 6: no difference).
// bf16 launches of 950 to 1300 workgroups (about four to five a CU) in between, from 12 workers on: two.  us, four -> two, 2100000 entries, N = 12 / 13 / 16 /
// 17 / 24 18.4 -> 17.9 / 19.4 -> 18.7 / 21.7 -> 21.1 / 22.8 -> 21.4 / 27.6 -> 26.3, 2300000 entries 19.9 -> 19.3 / 20.5 -> 20.0 / 22.7 -> 22.1 / 24.4 -> 23.2 / 30.2 ->
// 28.7, but 1500000 entries, N = 16 15.1 -> 15.0, 3194880 entries 28.3 -> 29.7.
// Sum and counts stay in the L2 (32 MB) where they fit: k_finalize reads every entry on the XCD that wrote it; and in the last-level cache
// (256 MB) where the workers together are at most 12 bytes an entry, or 16 and sum and counts few enough to live next to them.  us, streamed past ->
// kept, bf16, N = 4, 3194880 / 14000000 / 30000000 / 60000000 entries 16.1 -> 15.0 / 50.8 -> 46.8 / 106 -> 100 / 209 -> 221, N = 2, 18000000 entries
// 56.9 -> 50.4, N = 8, 6000000 / 10000000 / 18000000 entries 32.0 -> 30.8 / 49.4 -> 48.2 / 90.6 -> 92.7; fp32, N = 2 / 3, 14000000 entries 55.4 -> 52.4 / 64.2
// -> 62.1, N = 4, 10000000 entries 52.0 -> 50.9, N = 8, 14000000 entries 112 -> 114.  From 32 bytes read an entry on, where the workers go through the L2 too,
// only up to 10 MB: bf16, N = 16, 2700000 entries 25.6 -> 26.2, N = 24, 4000000 44.9 -> 46.0;  fp32, N = 8 / 24, 3194880 entries 27.1 -> 27.8 / 59.9 -> 62.9, 4600000
// 39.1 -> 39.5 / 91.0 -> 92.9, but 2100000 entries 19.6 -> 19.3 / 42.3 -> 41.6, and with fewer, fp32, N = 5, 2700000 entries 19.2 -> 18.8.
constexpr u64 kReduceFew = 256, kReduceTwoFrom = 950, kReduceTwoTo = 1300, kReduceMany = 3000, kReduceManyBf16 = 4096;
// (Not where the decode of larger blocks comes next, which gains from what it finds in the caches: up to 24 MB there.  us, reduce + decode of 2^16, 45 blocks, fp32,
// N = 8 / 24 40.3 -> 38.6 / 72.5 -> 70.7, bf16, N = 16 / 32 40.4 -> 39.1 / 56.5 -> 54.9.)
inline bool keep_results(u64 bytes, int bytes_read, bool for_decode) {   // sum and counts; of all workers an entry
  return bytes <= (bytes_read <= 12 ? 160u << 20 : bytes_read <= 16 ? 64u << 20 : bytes_read < 32 || for_decode ? 24u << 20 : 10u << 20);
}
template <class Wire, int VEC>
hipError_t launch_masked_reduce(const void* shards, const uint32_t* masks, int N, u64 L, float* sum_out,
                                uint8_t* count_out, hipStream_t s, int pos, bool for_decode) {
  if (L == 0) return hipSuccess;
  const u64 threads = (L + VEC - 1) / VEC;
  const u64 blocks = (threads + 255) / 256;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
  const bool keep = keep_results(L * 5, N * (int)sizeof(Wire), for_decode);
  const bool one = sizeof(Wire) == 4 ? blocks >= kReduceMany : (N >= 16 && blocks >= kReduceManyBf16) || (N == 2 && !keep);
  auto kernel = k_masked_reduce<Wire, VEC, 4>;
  if (blocks <= kReduceFew && N >= 8) kernel = k_masked_reduce<Wire, VEC, 8>;
  else if (one) kernel = k_masked_reduce<Wire, VEC, 1>;
  else if constexpr (sizeof(Wire) == 2) if (N >= 12 && blocks >= kReduceTwoFrom && blocks < kReduceTwoTo) kernel = k_masked_reduce<Wire, VEC, 2>;
  return orhost::launch_kernel(kernel, dim3((unsigned)blocks), dim3(256), s, pos, (const Wire*)shards, masks, N, L, sum_out, count_out, keep);
}

// ------------------------------------------------------------------ small streaming kernels
// mean = sum / count, 0 where count is 0 (Sec. 3.1.1 "averages" over what arrived); VEC entries a lane
template <class Out, int VEC>
__global__ __launch_bounds__(256) void k_finalize(const float* __restrict__ sum, const uint8_t* __restrict__ count, u64 L,
                                                  Out* __restrict__ mean) {
  const u64 e = ((u64)blockIdx.x * 256 + threadIdx.x) * VEC;
  if (e >= L) return;
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 s4[VEC / 4];
  uint32_t c4[VEC / 4];
#pragma unroll
  for (int q = 0; q < VEC / 4; ++q) {
    s4[q] = *(const f4*)(sum + e + 4 * q);
    c4[q] = *(const uint32_t*)(count + e + 4 * q);
  }
  float m[VEC];
#pragma unroll
  for (int j = 0; j < VEC; ++j) {
    const float c = (float)((c4[j / 4] >> (8 * (j % 4))) & 0xFFu);
    m[j] = c > 0.0f ? s4[j / 4][j % 4] / c : 0.0f;
  }
  if constexpr (sizeof(Out) == 4) {
    *(f4*)(mean + e) = f4{m[0], m[1], m[2], m[3]};
  } else {
    typedef uint16_t hv __attribute__((ext_vector_type(VEC)));
    hv h;
#pragma unroll
    for (int j = 0; j < VEC; ++j) h[j] = __builtin_bit_cast(uint16_t, (__bf16)m[j]);
    *(hv*)(mean + e) = h;
  }
}

__global__ void k_zero_u64(unsigned long long* p) { *p = 0; }
__global__ __launch_bounds__(256) void k_zero_u64n(unsigned long long* p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Sec. 3.4 loss monitoring: total of the received counts of a shard (16 counts per lane, byte sums
// with v_sad_u8, one 64-bit atomic per wavefront)
__global__ __launch_bounds__(256) void k_received_total(const uint8_t* __restrict__ count, u64 L,
                                                        unsigned long long* __restrict__ total) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  uint32_t acc = 0;
  const bool wide = ((uintptr_t)count & 15) == 0;   // or_reduce_decode_batched takes counts at any address
  for (u64 e = ((u64)blockIdx.x * 256 + threadIdx.x) * 16; e < L; e += (u64)gridDim.x * 256 * 16) {
    if (wide && e + 16 <= L) {
      const u4 c = *(const u4*)(count + e);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_sad_u8(c[j], 0u, acc);
    } else {
      for (u64 i = e; i < L && i < e + 16; ++i) acc += count[i];
    }
  }
  unsigned long long w = acc;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) w += __shfl_xor(w, o, 64);
  if ((threadIdx.x & 63) == 0 && w) atomicAdd(total, w);
}

// Second level of hierarchical 2D TAR (Sec. 3.1.2, App. A): sums with sums, counts with counts, over
// the groups whose partial aggregate arrived; 4 entries per lane
__global__ __launch_bounds__(256) void k_masked_reduce_pairs(const float* __restrict__ sums,
                                                             const uint8_t* __restrict__ counts,
                                                             const uint32_t* __restrict__ masks, int G, u64 L,
                                                             float* __restrict__ sum_out,
                                                             uint8_t* __restrict__ count_out) {
  const u64 e = ((u64)blockIdx.x * 256 + threadIdx.x) * 4;
  if (e >= L) return;
  typedef float f4 __attribute__((ext_vector_type(4)));
  const u64 words = L >> 5;
  const int sh = (int)(e & 31);
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  uint32_t cnt[4] = {0, 0, 0, 0};
  for (int g = 0; g < G; ++g) {
    // read once: nontemporal, as in k_masked_reduce
    const f4 x = __builtin_nontemporal_load((const f4*)(sums + (u64)g * L + e));
    const uint32_t c4 = __builtin_nontemporal_load((const uint32_t*)(counts + (u64)g * L + e));
    const uint32_t m = masks[(u64)g * words + (e >> 5)] >> sh;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool got = (m >> j) & 1u;
      acc[j] += got ? x[j] : 0.0f;
      cnt[j] += got ? ((c4 >> (8 * j)) & 0xFFu) : 0u;
    }
  }
  __builtin_nontemporal_store(f4{acc[0], acc[1], acc[2], acc[3]}, (f4*)(sum_out + e));
  __builtin_nontemporal_store((cnt[0] & 0xFFu) | ((cnt[1] & 0xFFu) << 8) | ((cnt[2] & 0xFFu) << 16) | (cnt[3] << 24),
                              (uint32_t*)(count_out + e));
}

// ------------------------------------------------------------------ checks
bool aligned(const void* p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; }
bool valid_k(int k) { return k >= OR_MIN_LOG2 && k <= OR_MAX_LOG2; }
int class_of(int k) { return k <= 10 ? 0 : k; }

bool ranges_overlap(const void* a, u64 abytes, const void* b, u64 bbytes) {
  uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
  return a0 < b0 + bbytes && b0 < a0 + abytes;
}

// armed timing events serve exactly one entry-point call, whatever its outcome
struct DisarmOnExit {
  ~DisarmOnExit() { orhost::timing_events() = {nullptr, nullptr}; }
};

or_status finish(hipError_t e) {
  if (e == hipSuccess) return OR_OK;
  g_last_hip_error = (int)e;
  return OR_ERR_HIP;
}

u64 padded(u64 n, int k) {
  const u64 B = (u64)1 << k;
  return (n + B - 1) / B * B;
}

// number of leading tiles that lie, together with every other tile of their transform block, wholly inside
// the first n entries (those need no bounds checks)
u64 full_units(u64 n, int k, int tile_log2) {
  const int group_log2 = k > tile_log2 ? k : tile_log2;   // a block above 2^14 spans 2^(k-14) tiles
  return (n >> group_log2) << (group_log2 - tile_log2);
}

float scale_of(int k) { return (float)(1.0 / sqrt((double)((u64)1 << k))); }

or_status check_base(int k, u64 base) {
  const u64 B = (u64)1 << k;
  const u64 q = B > 128 ? B : 128;
  return (base % q) ? OR_ERR_SHAPE : OR_OK;
}

// vector transforms: `in_es`/`out_es` are element sizes; the side of length n_pad is the encoded one
or_status check_transform(const void* in, u64 in_len, int in_es, void* out, u64 out_len, int out_es, int k, u64 base) {
  if (!valid_k(k)) return OR_ERR_BLOCK;
  if (check_base(k, base)) return OR_ERR_SHAPE;
  if (in_len == 0 && out_len == 0) return OR_OK;
  if (!in || !out) return OR_ERR_NULL;
  if (!aligned(in, 16) || !aligned(out, 16)) return OR_ERR_ALIGN;
  if (in_len > ((u64)1 << 46) || out_len > ((u64)1 << 46)) return OR_ERR_SHAPE;
  if (ranges_overlap(in, in_len * in_es, out, out_len * out_es)) {
    // every workgroup reads the whole of its tile (or block of tiles) before it writes any of it
    const bool exact_in_place = (in == out) && in_len == out_len && in_es == out_es;
    if (!exact_in_place) return OR_ERR_SHAPE;
  }
  return OR_OK;
}

template <class T>
or_status encode_impl(const T* grad, u64 n, int k, u64 seed, u64 base, T* out, void* stream, bool bf16) {
  DisarmOnExit disarm;
  const u64 n_pad = valid_k(k) ? padded(n, k) : 0;
  if (or_status s = check_transform(grad, n, sizeof(T), out, n_pad, sizeof(T), k, base)) return s;
  if (n == 0) return OR_OK;
  const orhost::KernelTable* t = orhost::table_for_class(class_of(k));
  PathArgs a = {};
  a.in = grad; a.out = out; a.n = n; a.n_pad = n_pad; a.seed = seed; a.base = base; a.k = k; a.scale = scale_of(k);
  const u64 units = (n_pad + ((u64)1 << t->tile_log2) - 1) >> t->tile_log2;
  a.unit0 = full_units(n, k, t->tile_log2);   // tiles whose whole block lies inside the n valid entries
  return finish((bf16 ? t->encode_bf16 : t->encode_f32)(a, units, (hipStream_t)stream, orhost::LAUNCH_ONLY));
}

template <class T>
or_status decode_impl(const float* agg, const uint8_t* count, bool finalize, u64 n, int k, u64 seed, u64 base, T* out,
                      void* stream, bool bf16, const uint32_t* stage2_mask = nullptr, bool masked = false) {
  DisarmOnExit disarm;
  const u64 n_pad = valid_k(k) ? padded(n, k) : 0;
  if (or_status s = check_transform(agg, n_pad, 4, out, n, sizeof(T), k, base)) return s;
  if (n == 0) return OR_OK;
  if (finalize) {
    if (!count) return OR_ERR_NULL;
    if (ranges_overlap(count, n_pad, out, n * sizeof(T))) return OR_ERR_SHAPE;
  }
  if (masked) {
    if (!stage2_mask) return OR_ERR_NULL;
    if (!aligned(stage2_mask, 4)) return OR_ERR_ALIGN;
    if (ranges_overlap(stage2_mask, n_pad / 8, out, n * sizeof(T))) return OR_ERR_SHAPE;
  }
  const orhost::KernelTable* t = orhost::table_for_class(class_of(k));
  PathArgs a = {};
  a.in = agg; a.count_in = count; a.masks = stage2_mask; a.out = out; a.n = n; a.n_pad = n_pad; a.seed = seed;
  a.base = base; a.k = k;
  a.scale = scale_of(k);
  const u64 units = (n_pad + ((u64)1 << t->tile_log2) - 1) >> t->tile_log2;
  a.unit0 = full_units(n, k, t->tile_log2);
  orhost::launch_fn f = masked     ? (bf16 ? t->decode_masked_bf16 : t->decode_masked_f32)
                        : finalize ? (bf16 ? t->finalize_decode_bf16 : t->finalize_decode_f32)
                                   : (bf16 ? t->decode_bf16 : t->decode_f32);
  return finish(f(a, units, (hipStream_t)stream, orhost::LAUNCH_ONLY));
}

or_status check_reduce(const void* shards, const uint32_t* masks, int N, u64 L, int es) {
  if (N < 1 || N > OR_MAX_WORKERS) return OR_ERR_WORKERS;
  if (L % 32) return OR_ERR_SHAPE;
  if (L > ((u64)1 << 40)) return OR_ERR_SHAPE;
  if (L == 0) return OR_OK;
  if (!shards || !masks) return OR_ERR_NULL;
  if (!aligned(shards, 16) || !aligned(masks, 4)) return OR_ERR_ALIGN;
  if ((L * es) % 16) return OR_ERR_SHAPE;  // every worker's row must start 16-byte aligned
  return OR_OK;
}

template <class T>
or_status masked_reduce_impl(const T* shards, const uint32_t* masks, int N, u64 L, float* sum_out, uint8_t* count_out,
                             void* stream) {
  DisarmOnExit disarm;
  if (or_status s = check_reduce(shards, masks, N, L, sizeof(T))) return s;
  if (L == 0) return OR_OK;
  if (!sum_out || !count_out) return OR_ERR_NULL;
  if (!aligned(sum_out, 16) || !aligned(count_out, 4)) return OR_ERR_ALIGN;
  const u64 in_bytes = (u64)N * L * sizeof(T), mask_bytes = (u64)N * (L / 8);
  if (ranges_overlap(sum_out, L * 4, shards, in_bytes) || ranges_overlap(count_out, L, shards, in_bytes) ||
      ranges_overlap(sum_out, L * 4, masks, mask_bytes) || ranges_overlap(count_out, L, masks, mask_bytes) ||
      ranges_overlap(sum_out, L * 4, count_out, L))
    return OR_ERR_SHAPE;
  constexpr int VEC = 16 / sizeof(T);
  return finish(launch_masked_reduce<T, VEC>(shards, masks, N, L, sum_out, count_out, (hipStream_t)stream,
                                             orhost::LAUNCH_ONLY, false));
}

size_t workspace_bytes(u64 L, int k) {
  if (!valid_k(k) || k <= 14) return 0;
  const u64 sums = (L * 4 + 255) / 256 * 256;
  const u64 counts = (L + 255) / 256 * 256;
  return (size_t)(sums + counts);
}

// argument checks shared by or_reduce_decode*, or_fused_path* and the batched form (es = element bytes)
or_status check_path(const void* in, const uint32_t* masks, int N, u64 L, int k, u64 base, void* out, uint8_t* count_out,
                     void* ws, size_t ws_bytes, int es) {
  if (!valid_k(k)) return OR_ERR_BLOCK;
  if (or_status s = check_reduce(in, masks, N, L, es)) return s;
  if (L % ((u64)1 << k)) return OR_ERR_SHAPE;
  if (check_base(k, base)) return OR_ERR_SHAPE;
  if (L == 0) return OR_OK;
  if (!out) return OR_ERR_NULL;
  if (!aligned(out, 16)) return OR_ERR_ALIGN;
  const u64 in_bytes = (u64)N * L * es, mask_bytes = (u64)N * (L / 8);
  if (ranges_overlap(out, L * es, in, in_bytes) || ranges_overlap(out, L * es, masks, mask_bytes))
    return OR_ERR_SHAPE;
  if (count_out && (ranges_overlap(count_out, L, in, in_bytes) || ranges_overlap(count_out, L, masks, mask_bytes) ||
                    ranges_overlap(count_out, L, out, L * es)))
    return OR_ERR_SHAPE;
  const size_t need = workspace_bytes(L, k);
  if (need) {
    if (!ws || ws_bytes < need) return OR_ERR_WORKSPACE;
    if (!aligned(ws, 256)) return OR_ERR_ALIGN;
    if (ranges_overlap(ws, need, in, in_bytes) || ranges_overlap(ws, need, masks, mask_bytes) ||
        ranges_overlap(ws, need, out, L * es) || (count_out && ranges_overlap(ws, need, count_out, L)))
      return OR_ERR_SHAPE;
  }
  return OR_OK;
}

// Reduce + decode of blocks above 2^14: one kernel for both, or a reduction and a decode with sum and counts in between?  The same
// additions in the same order, so the same bits.  The one kernel moves less, but a workgroup takes a whole block through all
// workers one after the other, so launches that leave CUs idle pay for every worker.  us, two launches -> one, fp32 2^15 / 2^16,
// bf16 2^15 / 2^16:  N = 1, 2 blocks 12.2 -> 10.5 / 21.5 -> 19.1, 12.1 -> 10.3 / 21.5 -> 18.8;  N = 2, 16 blocks 14.1 -> 14.7 /
// 24.5 -> 26.6, 13.9 -> 12.2 / 24.2 -> 23.1, 48 blocks 17.0 -> 15.4 / 31.4 -> 27.1, 16.4 -> 12.8 / 29.4 -> 24.0;  N = 8, 48
// blocks 22.5 -> 30.6 / 43.1 -> 58.3, 18.5 -> 21.6 / 33.7 -> 41.4, 96 blocks 33.9 -> 33.6 / 64.1 -> 64.2, 25.2 -> 22.6 /
// 47.2 -> 44.7, 256 blocks 74.7 -> 56.5 / 146 -> 113, 48.8 -> 32.9 / 92.0 -> 69.0;  N = 16, 96 blocks 52.1 -> 58.0 / 100 -> 114,
// 33.8 -> 35.7 / 65.0 -> 72.7, 128 blocks 67.0 -> 62.2 / 133 -> 125, 42.0 -> 37.3 / 81.4 -> 79.0;  N = 32, 128 blocks 124 -> 114 /
// 224 -> 229, 67.7 -> 65.8 / 144 -> 141.
bool reduce_in_one_kernel(u64 blocks, int N, bool bf16) {
  if (N <= 2) return N == 1 || bf16 || blocks >= 48;
  return blocks >= (N <= 8 ? 96 : 128);
}

// enqueue one checked shard: T = float or uint16_t (bf16 bits).  `allow` = which of this entry point's first /
// last launches this shard may be (timing events ride on those only); `total`, if not null, is expected to be
// zero already and receives the number of arrivals.
template <class T>
or_status run_path(bool fused, const T* in, const uint32_t* masks, int N, u64 L, int k, u64 seed, u64 base, T* out,
                   uint8_t* count_out, void* ws, void* stream, bool bf16, int allow = orhost::LAUNCH_ONLY,
                   unsigned long long* total = nullptr) {
  if (L == 0) return OR_OK;
  const size_t need = workspace_bytes(L, k);
  const orhost::KernelTable* t = orhost::table_for_class(class_of(k));
  hipStream_t s = (hipStream_t)stream;
  const u64 units = (L + ((u64)1 << t->tile_log2) - 1) >> t->tile_log2;
  const int first = orhost::LAUNCH_FIRST & allow, last = orhost::LAUNCH_LAST & allow;
  PathArgs a = {};
  a.in = in; a.masks = masks; a.out = out; a.count_out = count_out; a.n = L; a.n_pad = L; a.seed = seed; a.base = base;
  a.N = N; a.k = k; a.scale = scale_of(k); a.total_out = total;
  if (!need) {
    orhost::launch_fn f = fused ? (bf16 ? t->fused_bf16 : t->fused_f32) : (bf16 ? t->reduce_decode_bf16 : t->reduce_decode_f32);
    return finish(f(a, units, s, first | last));
  }
  // a block spans several tiles
  float* ws_f32 = (float*)ws;
  uint8_t* ws_cnt = (uint8_t*)ws + (L * 4 + 255) / 256 * 256;
  PathArgs d = {};
  d.out = out; d.n = L; d.n_pad = L; d.seed = seed; d.base = base; d.k = k; d.scale = a.scale;
  d.in = ws_f32;
  d.unit0 = units;   // shards hold whole blocks: no tile of the decode needs bounds checks
  if (fused) {   // no workspace, but for bf16 blocks of 2^16 in launches of few blocks, whose means go through it
    a.mean_out = ws_f32;
    return finish((bf16 ? t->fused_bf16 : t->fused_f32)(a, units, s, first | last));
  }
  if (reduce_in_one_kernel(L >> k, N, bf16))
    return finish((bf16 ? t->reduce_decode_bf16 : t->reduce_decode_f32)(a, units, s, first | last));
  uint8_t* cnt = count_out ? count_out : ws_cnt;
  constexpr int VEC = 16 / sizeof(T);
  if (hipError_t e = launch_masked_reduce<T, VEC>(in, masks, N, L, ws_f32, cnt, s, first, true)) return finish(e);
  d.count_in = cnt;
  if (total) {
    u64 blocks = (L / 16 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (hipError_t e = orhost::launch_kernel(k_received_total, dim3((unsigned)(blocks ? blocks : 1)), dim3(256), s, 0,
                                             (const uint8_t*)cnt, L, total))
      return finish(e);
  }
  return finish((bf16 ? t->finalize_decode_bf16 : t->finalize_decode_f32)(d, units, s, last));
}

template <class T>
or_status path_impl(bool fused, const T* in, const uint32_t* masks, int N, u64 L, int k, u64 seed, u64 base, T* out,
                    uint8_t* count_out, void* ws, size_t ws_bytes, void* stream, bool bf16) {
  DisarmOnExit disarm;
  if (or_status s = check_path(in, masks, N, L, k, base, out, count_out, ws, ws_bytes, sizeof(T))) return s;
  return run_path<T>(fused, in, masks, N, L, k, seed, base, out, count_out, ws, stream, bf16);
}

// Entries a lane.  bf16: eight, 16 bytes of the mean and the entries of a workgroup of k_masked_reduce, whose results are then on the XCD that
// reads them; but four where sum and counts are read from memory (keep_results).  us, reduce + finalize, four -> eight: N = 2, 524288 / 20000000 /
// 30000000 entries 5.8 -> 4.7 / 57.3 -> 56.7 / 82.6 -> 80.8, but 60000000 / 120000000 entries, N = 2 181 -> 184 / 362 -> 370, N = 4 205 -> 208 / 404 -> 412.
constexpr u64 kFinalizeNarrowFrom = 160u << 20;   // bytes of sum and counts
template <class Out>
or_status finalize_impl(const float* sum, const uint8_t* count, u64 L, Out* mean, void* stream) {
  DisarmOnExit disarm;
  if (L % 32 || L > ((u64)1 << 40)) return OR_ERR_SHAPE;
  if (L == 0) return OR_OK;
  if (!sum || !count || !mean) return OR_ERR_NULL;
  if (!aligned(sum, 16) || !aligned(count, 4) || !aligned(mean, 16)) return OR_ERR_ALIGN;
  if (ranges_overlap(mean, L * sizeof(Out), count, L)) return OR_ERR_SHAPE;
  if (ranges_overlap(mean, L * sizeof(Out), sum, L * 4) && !((const void*)mean == (const void*)sum && sizeof(Out) == 4))
    return OR_ERR_SHAPE;
  const bool wide = sizeof(Out) == 2 && L * 5 <= kFinalizeNarrowFrom;
  const u64 blocks = (L / (wide ? 8 : 4) + 255) / 256;
  if (blocks > 0x7FFFFFFFull) return OR_ERR_SHAPE;
  auto kernel = k_finalize<Out, 4>;
  if constexpr (sizeof(Out) == 2) if (wide) kernel = k_finalize<Out, 8>;
  return finish(orhost::launch_kernel(kernel, dim3((unsigned)blocks), dim3(256), (hipStream_t)stream,
                                      orhost::LAUNCH_ONLY, sum, count, L, mean));
}

or_status received_total_impl(const uint8_t* count, u64 L, unsigned long long* total, void* stream) {
  DisarmOnExit disarm;
  if (L > ((u64)1 << 40)) return OR_ERR_SHAPE;
  if (!total) return OR_ERR_NULL;
  if (!aligned(total, 8)) return OR_ERR_ALIGN;
  if (L && !count) return OR_ERR_NULL;
  if (L && !aligned(count, 16)) return OR_ERR_ALIGN;
  if (L && ranges_overlap(total, 8, count, L)) return OR_ERR_SHAPE;
  hipStream_t s = (hipStream_t)stream;
  if (hipError_t e = orhost::launch_kernel(k_zero_u64, dim3(1), dim3(1), s, L ? orhost::LAUNCH_FIRST : orhost::LAUNCH_ONLY,
                                           total))
    return finish(e);
  if (L == 0) return OR_OK;
  u64 blocks = (L / 16 + 255) / 256;
  if (blocks > 4096) blocks = 4096;   // grid-stride: a few atomics per CU are enough
  if (blocks == 0) blocks = 1;
  return finish(orhost::launch_kernel(k_received_total, dim3((unsigned)blocks), dim3(256), s, orhost::LAUNCH_LAST, count, L,
                                      total));
}

or_status pairs_impl(const float* sums, const uint8_t* counts, const uint32_t* masks, int G, u64 L, float* sum_out,
                     uint8_t* count_out, void* stream) {
  DisarmOnExit disarm;
  if (or_status s = check_reduce(sums, masks, G, L, 4)) return s;
  if (L == 0) return OR_OK;
  if (!counts || !sum_out || !count_out) return OR_ERR_NULL;
  if (!aligned(counts, 4) || !aligned(sum_out, 16) || !aligned(count_out, 4)) return OR_ERR_ALIGN;
  const u64 sb = (u64)G * L * 4, cb = (u64)G * L, mb = (u64)G * (L / 8);
  if (ranges_overlap(sum_out, L * 4, sums, sb) || ranges_overlap(sum_out, L * 4, counts, cb) ||
      ranges_overlap(sum_out, L * 4, masks, mb) || ranges_overlap(count_out, L, sums, sb) ||
      ranges_overlap(count_out, L, counts, cb) || ranges_overlap(count_out, L, masks, mb) ||
      ranges_overlap(sum_out, L * 4, count_out, L))
    return OR_ERR_SHAPE;
  const u64 blocks = (L / 4 + 255) / 256;
  if (blocks > 0x7FFFFFFFull) return OR_ERR_SHAPE;
  return finish(orhost::launch_kernel(k_masked_reduce_pairs, dim3((unsigned)blocks), dim3(256), (hipStream_t)stream,
                                      orhost::LAUNCH_ONLY, sums, counts, masks, G, L, sum_out, count_out));
}

// How the non-empty buckets of a batched call are spread over launches: as few launches as the descriptor
// limit allows, the buckets divided evenly among them.
struct BatchPlan {
  int nonempty, launches, per_launch;
};
BatchPlan plan_batches(int nonempty) {
  BatchPlan p = {nonempty, 0, 0};
  if (nonempty > 0) {
    p.launches = (nonempty + ordev::kMaxBatch - 1) / ordev::kMaxBatch;
    p.per_launch = (nonempty + p.launches - 1) / p.launches;
  }
  return p;
}

// No output of one bucket may touch anything of another bucket (the buckets of a launch run concurrently).  `each(f)` calls
// f(pointer, bytes, written, owner) for every span of the call; false: a written span overlaps a span of another owner (what
// overlaps within one bucket is that bucket's check).  Written spans are sorted by address, kChunk at a time in an array on the
// stack (nothing is allocated), and every other span is looked up among them: for the 238 buckets of a GPT-2-XL-sized gradient
// a comparison of all pairs took 0.3 ms of the host's time before the first launch, this takes a few microseconds.
template <class Each>
bool spans_disjoint(const Each& each) {
  struct Span {
    uintptr_t lo, hi;
    int owner;
  };
  constexpr size_t kChunk = 1024;   // 24 KB
  Span w[kChunk];
  for (size_t first = 0;; first += kChunk) {
    size_t at = 0, m = 0;
    each([&](const void* p, u64 bytes, bool written, int owner) {
      if (!p || !bytes || !written) return;
      if (at >= first && m < kChunk) w[m++] = {(uintptr_t)p, (uintptr_t)p + bytes, owner};
      ++at;
    });
    const auto before = [](const Span& a, const Span& b) { return a.lo < b.lo; };
    if (!std::is_sorted(w, w + m, before)) std::sort(w, w + m, before);
    for (size_t i = 1; i < m; ++i)   // written spans of one owner are disjoint already
      if (w[i].lo < w[i - 1].hi) return false;
    bool apart = true;
    at = 0;
    each([&](const void* p, u64 bytes, bool written, int owner) {
      if (!p || !bytes || !apart) return;
      if (written && at++ < first + kChunk) return;   // compared just now, or with an earlier chunk
      const uintptr_t lo = (uintptr_t)p, hi = lo + bytes;
      // the first written span that ends behind the start of this one
      const Span* s = std::upper_bound(w, w + m, lo, [](uintptr_t v, const Span& x) { return v < x.hi; });
      for (; s != w + m && s->lo < hi; ++s)
        if (s->owner != owner) apart = false;
    });
    if (!apart) return false;
    if (m < kChunk) return true;
  }
}

hipError_t zero_totals(unsigned long long* totals, int n, hipStream_t s, int pos) {
  return orhost::launch_kernel(k_zero_u64n, dim3((unsigned)((n + 255) / 256)), dim3(256), s, pos, totals, n);
}

// or_fused_path_batched* (fused = true) and or_reduce_decode_batched (fused = false)
or_status path_batched_impl(bool fused, const or_bucket* buckets, int n, int N, int k, bool bf16,
                            unsigned long long* totals, void* ws, size_t ws_bytes, void* stream) {
  DisarmOnExit disarm;
  if (n < 0) return OR_ERR_SHAPE;
  if (n == 0) return OR_OK;
  if (!buckets) return OR_ERR_NULL;
  if (totals && !aligned(totals, 8)) return OR_ERR_ALIGN;
  const u64 es = bf16 ? 2 : 4;
  // ---- every bucket is checked before anything is enqueued
  int nonempty = 0;
  for (int j = 0; j < n; ++j) {
    const or_bucket& q = buckets[j];
    if (or_status s = check_path(q.grads, q.masks, N, q.shard_len, k, q.base_index, q.out, q.count_out, ws, ws_bytes, (int)es))
      return s;
    if (q.shard_len == 0) continue;
    ++nonempty;
  }
  const bool apart = spans_disjoint([&](auto&& span) {
    span(totals, totals ? (u64)n * 8 : 0, true, -1);
    for (int j = 0; j < n; ++j) {
      const or_bucket& q = buckets[j];
      const u64 L = q.shard_len;
      span(q.grads, (u64)N * L * es, false, j);
      span(q.masks, (u64)N * (L / 8), false, j);
      span(q.out, L * es, true, j);
      span(q.count_out, L, true, j);
    }
  });
  if (!apart) return OR_ERR_SHAPE;
  // The buckets share the workspace one after the other: nothing that is read may lie in it, and a bucket's results not in the
  // part that it or a later one uses.  (What only earlier, longer ones used is free again by then.)
  u64 ws_used = 0, ws_all = 0;
  for (int j = 0; j < n; ++j) ws_all = std::max(ws_all, (u64)workspace_bytes(buckets[j].shard_len, k));
  for (int j = ws_all ? n - 1 : -1; j >= 0; --j) {
    const or_bucket& q = buckets[j];
    const u64 L = q.shard_len;
    if (L == 0) continue;
    ws_used = std::max(ws_used, (u64)workspace_bytes(L, k));
    if (ranges_overlap(ws, ws_all, q.grads, (u64)N * L * es) || ranges_overlap(ws, ws_all, q.masks, (u64)N * (L / 8)) ||
        ranges_overlap(ws, ws_used, q.out, L * es) || (q.count_out && ranges_overlap(ws, ws_used, q.count_out, L)))
      return OR_ERR_SHAPE;
  }
  if (ws_used && totals && ranges_overlap(ws, ws_used, totals, (u64)n * 8)) return OR_ERR_SHAPE;
  const orhost::KernelTable* t = orhost::table_for_class(class_of(k));
  orhost::batch_fn f = fused ? (bf16 ? t->fused_batched_bf16 : t->fused_batched_f32)
                             : (bf16 ? t->reduce_decode_batched_bf16 : t->reduce_decode_batched_f32);
  const BatchPlan plan = plan_batches(nonempty);
  hipStream_t s = (hipStream_t)stream;
  // ---- enqueue: the entry point's very first launch carries the start event, its last one the stop event
  bool first_pending = true;
  if (totals) {
    if (hipError_t e = zero_totals(totals, n, s, nonempty ? orhost::LAUNCH_FIRST : orhost::LAUNCH_ONLY)) return finish(e);
    first_pending = false;
  }
  if (!nonempty) return OR_OK;
  int seen = 0;
  // blocks above 2^14: one bucket after the other, sharing the workspace in stream order.  (A single bucket as if it came alone: few
  // blocks of 2^16 are split over workgroups that meet in the workspace.)
  if (!f || (fused && bf16 && k == 16 && nonempty == 1)) {
    for (int j = 0; j < n; ++j) {
      const or_bucket& q = buckets[j];
      if (q.shard_len == 0) continue;
      ++seen;
      const int allow = (first_pending ? orhost::LAUNCH_FIRST : 0) | (seen == nonempty ? orhost::LAUNCH_LAST : 0);
      first_pending = false;
      unsigned long long* one = totals ? totals + j : nullptr;
      or_status st = bf16 ? run_path<uint16_t>(fused, (const uint16_t*)q.grads, q.masks, N, q.shard_len, k, q.seed,
                                               q.base_index, (uint16_t*)q.out, q.count_out, ws, stream, true, allow, one)
                          : run_path<float>(fused, (const float*)q.grads, q.masks, N, q.shard_len, k, q.seed, q.base_index,
                                            (float*)q.out, q.count_out, ws, stream, false, allow, one);
      if (st) return st;
    }
    return OR_OK;
  }
  for (int j = 0; seen < nonempty;) {
    ordev::BatchArgs ba = {};
    ba.N = N; ba.k = k; ba.scale = scale_of(k); ba.totals = totals;
    u64 tiles = 0;
    int m = 0;
    for (; j < n && m < plan.per_launch; ++j) {
      const or_bucket& q = buckets[j];
      if (q.shard_len == 0) {
        if (totals && m) { ++j; break; }   // totals[first + m] is bucket first + m: a run of buckets without a gap
        continue;
      }
      const u64 units = (q.shard_len + ((u64)1 << t->tile_log2) - 1) >> t->tile_log2;
      if (tiles + units > 0x7FFFFFFFull) {
        if (m == 0) return OR_ERR_SHAPE;   // cannot happen: check_path bounds the shard length
        break;
      }
      if (m == 0) ba.first = j;
      ba.tile_start[m] = (uint32_t)tiles;
      ba.b[m] = {q.grads, q.masks, q.out, q.count_out, q.shard_len, q.seed, q.base_index};
      tiles += units;
      ++m;
    }
    ba.n = m;
    ba.tile_start[m] = (uint32_t)tiles;
    seen += m;
    const int pos = (first_pending ? orhost::LAUNCH_FIRST : 0) | (seen == nonempty ? orhost::LAUNCH_LAST : 0);
    first_pending = false;
    if (hipError_t e = f(ba, tiles, s, pos)) return finish(e);
  }
  return OR_OK;
}

// one bucket of the separate calls on several buckets
or_status check_stage_bucket(const or_stage_bucket& q, bool reduce, int N, int k, u64 es) {
  const u64 L = q.shard_len;
  if (L % 32 || L > ((u64)1 << 40)) return OR_ERR_SHAPE;
  if (L == 0) return OR_OK;
  if (!q.sum || !q.count) return OR_ERR_NULL;
  if (!aligned(q.sum, 16) || !aligned(q.count, 4)) return OR_ERR_ALIGN;
  if (ranges_overlap(q.sum, L * 4, q.count, L)) return OR_ERR_SHAPE;
  if (reduce) {
    if (or_status s = check_reduce(q.shards, q.masks, N, L, (int)es)) return s;
    const u64 in_bytes = (u64)N * L * es, mask_bytes = (u64)N * (L / 8);
    if (ranges_overlap(q.sum, L * 4, q.shards, in_bytes) || ranges_overlap(q.count, L, q.shards, in_bytes) ||
        ranges_overlap(q.sum, L * 4, q.masks, mask_bytes) || ranges_overlap(q.count, L, q.masks, mask_bytes))
      return OR_ERR_SHAPE;
  } else {
    if (L % ((u64)1 << k)) return OR_ERR_SHAPE;   // buckets hold whole blocks
    if (check_base(k, q.base_index)) return OR_ERR_SHAPE;
    if (!q.out) return OR_ERR_NULL;
    if (!aligned(q.out, 16)) return OR_ERR_ALIGN;
    if (ranges_overlap(q.out, L * es, q.count, L)) return OR_ERR_SHAPE;
    if (ranges_overlap(q.out, L * es, q.sum, L * 4) && !((const void*)q.out == (const void*)q.sum && es == 4))
      return OR_ERR_SHAPE;   // in place is allowed for fp32: a workgroup reads its whole tile before it writes
  }
  return OR_OK;
}

// or_masked_reduce_batched (reduce = true) and or_finalize_decode_batched (reduce = false)
or_status stage_batched_impl(bool reduce, const or_stage_bucket* buckets, int n, int N, int k, bool bf16, void* stream) {
  DisarmOnExit disarm;
  if (n < 0) return OR_ERR_SHAPE;
  if (!reduce && !valid_k(k)) return OR_ERR_BLOCK;
  if (reduce && (N < 1 || N > OR_MAX_WORKERS)) return OR_ERR_WORKERS;
  if (n == 0) return OR_OK;
  if (!buckets) return OR_ERR_NULL;
  const u64 es = bf16 ? 2 : 4;
  int nonempty = 0;
  for (int j = 0; j < n; ++j) {
    const or_stage_bucket& q = buckets[j];
    if (or_status s = check_stage_bucket(q, reduce, N, k, es)) return s;
    if (q.shard_len == 0) continue;
    ++nonempty;
  }
  const bool apart = spans_disjoint([&](auto&& span) {
    for (int j = 0; j < n; ++j) {
      const or_stage_bucket& q = buckets[j];
      const u64 L = q.shard_len;
      if (reduce) {
        span(q.shards, (u64)N * L * es, false, j);
        span(q.masks, (u64)N * (L / 8), false, j);
      } else {
        span(q.out, L * es, true, j);
      }
      span(q.sum, L * 4, reduce, j);
      span(q.count, L, reduce, j);
    }
  });
  if (!apart) return OR_ERR_SHAPE;
  if (!nonempty) return OR_OK;
  hipStream_t s = (hipStream_t)stream;
  const BatchPlan plan = plan_batches(nonempty);
  const orhost::KernelTable* t = reduce ? nullptr : orhost::table_for_class(class_of(k));
  orhost::batch_fn f = reduce ? nullptr : (bf16 ? t->finalize_decode_batched_bf16 : t->finalize_decode_batched_f32);
  const u64 per_wg = reduce ? 256 * (16 / es) : ((u64)1 << t->tile_log2);   // entries one workgroup serves
  int seen = 0;
  if (!reduce && !f) {   // blocks above 2^14: one bucket after the other
    for (int j = 0; j < n; ++j) {
      const or_stage_bucket& q = buckets[j];
      if (q.shard_len == 0) continue;
      ++seen;
      PathArgs d = {};
      d.in = q.sum; d.count_in = q.count; d.out = q.out; d.n = d.n_pad = q.shard_len; d.seed = q.seed; d.base = q.base_index;
      d.k = k; d.scale = scale_of(k);
      const u64 units = q.shard_len >> t->tile_log2;
      d.unit0 = units;
      const int pos = (seen == 1 ? orhost::LAUNCH_FIRST : 0) | (seen == nonempty ? orhost::LAUNCH_LAST : 0);
      if (hipError_t e = (bf16 ? t->finalize_decode_bf16 : t->finalize_decode_f32)(d, units, s, pos)) return finish(e);
    }
    return OR_OK;
  }
  for (int j = 0; seen < nonempty;) {
    ReduceBatch rb = {};
    ordev::BatchArgs ba = {};
    rb.N = N;
    ba.k = k; ba.scale = scale_of(k);
    u64 wgs = 0;
    int m = 0;
    for (; j < n && m < plan.per_launch; ++j) {
      const or_stage_bucket& q = buckets[j];
      if (q.shard_len == 0) continue;
      const u64 units = (q.shard_len + per_wg - 1) / per_wg;
      if (wgs + units > 0x7FFFFFFFull) {
        if (m == 0) return OR_ERR_SHAPE;   // cannot happen: the shard length is bounded above
        break;
      }
      rb.start[m] = ba.tile_start[m] = (uint32_t)wgs;
      rb.b[m] = {q.shards, q.masks, q.sum, q.count, q.shard_len};
      ba.b[m] = {q.sum, q.count, q.out, nullptr, q.shard_len, q.seed, q.base_index};
      wgs += units;
      ++m;
    }
    rb.n = ba.n = m;
    rb.start[m] = ba.tile_start[m] = (uint32_t)wgs;
    const int pos = (seen == 0 ? orhost::LAUNCH_FIRST : 0) | (seen + m == nonempty ? orhost::LAUNCH_LAST : 0);
    seen += m;
    hipError_t e;
    if (!reduce) e = f(ba, wgs, s, pos);
    else if (bf16) e = orhost::launch_kernel(wgs <= kBatchPairTo ? k_masked_reduce_batched<uint16_t, 8, true> : k_masked_reduce_batched<uint16_t, 8, false>,
                                             dim3((unsigned)wgs), dim3(256), s, pos, rb);
    else e = orhost::launch_kernel(k_masked_reduce_batched<float, 4, true>, dim3((unsigned)wgs), dim3(256), s, pos, rb);
    if (e) return finish(e);
  }
  return OR_OK;
}

// ------------------------------------------------------------------ scratch for callers that cannot allocate
// or_fused_path_bf16_static: the workspace of the kernels for blocks above 2^14 lives in this array instead of
// caller memory.  Each GPU holds its own copy at its own address; host code never uses the array's name as an
// address, only the pointer that hipGetSymbolAddress returned for the device that is current.
constexpr u64 kStaticMaxShard = OR_STATIC_MAX_SHARD_LEN;
constexpr size_t kScratchBytes = ((kStaticMaxShard * 4 + 255) / 256 * 256) + ((kStaticMaxShard + 255) / 256 * 256);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[kMaxDevices] = {};

// the scratch array's address on the current device (looked up once per device), or null with *err set
void* scratch_of_current_device(hipError_t* err) {
  int dev = -1;
  *err = hipGetDevice(&dev);
  if (*err != hipSuccess) return nullptr;
  if (dev < 0 || dev >= kMaxDevices) {
    *err = hipErrorInvalidDevice;
    return nullptr;
  }
  std::lock_guard<std::mutex> hold(g_scratch_lock);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    *err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (*err != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

// loss > t, exactly: missing / sent is a ratio of integers and t a binary fraction, so both sides are
// compared as integers (no rounded quotient in between)
bool ratio_exceeds(uint64_t missing, uint64_t sent, double t) {
  if (t < 0.0) return true;        // a loss is never negative
  if (t >= 1.0) return false;      // and never above 1
  if (t == 0.0) return missing > 0;
  int e;
  const double fr = frexp(t, &e);                       // t = fr * 2^e, 0.5 <= fr < 1, e <= 0
  const unsigned __int128 mant = (unsigned __int128)(uint64_t)ldexp(fr, 53);   // exact: fr has 53 bits
  const unsigned __int128 prod = mant * sent;           // t * sent = prod / 2^(53 - e); sent < 2^48
  const int sh = 53 - e;                                // >= 53
  if (sh >= 120) return missing > 0;                    // t * sent < 1
  return (unsigned __int128)missing > (prod >> sh);     // missing * 2^sh > prod  <=>  missing > floor(prod / 2^sh)
}

}  // namespace

extern "C" {

uint64_t or_padded_len(uint64_t n, int block_log2) { return valid_k(block_log2) ? padded(n, block_log2) : 0; }
size_t or_workspace_bytes(uint64_t shard_len, int block_log2) { return workspace_bytes(shard_len, block_log2); }
int or_version(void) { return 200; }
int or_last_hip_error(void) { return g_last_hip_error; }

or_status or_time_next_call(void* start_event, void* stop_event) {
  orhost::timing_events() = {(hipEvent_t)start_event, (hipEvent_t)stop_event};
  return OR_OK;
}

const char* or_status_string(or_status s) {
  switch (s) {
    case OR_OK: return "ok";
    case OR_ERR_NULL: return "a required pointer is NULL";
    case OR_ERR_BLOCK: return "block_log2 out of range";
    case OR_ERR_WORKERS: return "worker count out of range";
    case OR_ERR_SHAPE: return "bad length, base_index or overlap";
    case OR_ERR_ALIGN: return "pointer not aligned";
    case OR_ERR_WORKSPACE: return "workspace missing or too small";
    case OR_ERR_HIP: return "HIP launch failed";
    default: return "unknown status";
  }
}

or_status or_rht_encode(const float* grad, uint64_t n, int block_log2, uint64_t seed, float* out, void* stream) {
  return encode_impl<float>(grad, n, block_log2, seed, 0, out, stream, false);
}
or_status or_rht_encode_at(const float* grad, uint64_t n, int block_log2, uint64_t seed, uint64_t base_index,
                           float* out, void* stream) {
  return encode_impl<float>(grad, n, block_log2, seed, base_index, out, stream, false);
}
or_status or_rht_encode_bf16(const uint16_t* grad, uint64_t n, int block_log2, uint64_t seed, uint64_t base_index,
                             uint16_t* out, void* stream) {
  return encode_impl<uint16_t>(grad, n, block_log2, seed, base_index, out, stream, true);
}

or_status or_masked_reduce(const float* shards, const uint32_t* masks, int N, uint64_t shard_len, float* sum_out,
                           uint8_t* count_out, void* stream) {
  return masked_reduce_impl<float>(shards, masks, N, shard_len, sum_out, count_out, stream);
}
or_status or_masked_reduce_bf16(const uint16_t* shards, const uint32_t* masks, int N, uint64_t shard_len,
                                float* sum_out, uint8_t* count_out, void* stream) {
  return masked_reduce_impl<uint16_t>(shards, masks, N, shard_len, sum_out, count_out, stream);
}

or_status or_rht_decode(const float* agg, uint64_t n, int block_log2, uint64_t seed, float* out, void* stream) {
  return decode_impl<float>(agg, nullptr, false, n, block_log2, seed, 0, out, stream, false);
}
or_status or_rht_decode_at(const float* agg, uint64_t n, int block_log2, uint64_t seed, uint64_t base_index,
                           float* out, void* stream) {
  return decode_impl<float>(agg, nullptr, false, n, block_log2, seed, base_index, out, stream, false);
}
or_status or_rht_decode_bf16(const float* agg, uint64_t n, int block_log2, uint64_t seed, uint64_t base_index,
                             uint16_t* out, void* stream) {
  return decode_impl<uint16_t>(agg, nullptr, false, n, block_log2, seed, base_index, out, stream, true);
}

or_status or_finalize_decode(const float* sum, const uint8_t* count, uint64_t n, int block_log2, uint64_t seed,
                             uint64_t base_index, float* out, void* stream) {
  return decode_impl<float>(sum, count, true, n, block_log2, seed, base_index, out, stream, false);
}
or_status or_finalize_decode_bf16(const float* sum, const uint8_t* count, uint64_t n, int block_log2,
                                  uint64_t seed, uint64_t base_index, uint16_t* out, void* stream) {
  return decode_impl<uint16_t>(sum, count, true, n, block_log2, seed, base_index, out, stream, true);
}

or_status or_reduce_decode(const float* shards, const uint32_t* masks, int N, uint64_t shard_len, int block_log2,
                           uint64_t seed, uint64_t base_index, float* out, uint8_t* count_out, void* workspace,
                           size_t workspace_bytes, void* stream) {
  return path_impl<float>(false, shards, masks, N, shard_len, block_log2, seed, base_index, out, count_out, workspace,
                          workspace_bytes, stream, false);
}
or_status or_reduce_decode_bf16(const uint16_t* shards, const uint32_t* masks, int N, uint64_t shard_len,
                                int block_log2, uint64_t seed, uint64_t base_index, uint16_t* out,
                                uint8_t* count_out, void* workspace, size_t workspace_bytes, void* stream) {
  return path_impl<uint16_t>(false, shards, masks, N, shard_len, block_log2, seed, base_index, out, count_out,
                             workspace, workspace_bytes, stream, true);
}
or_status or_fused_path(const float* grads, const uint32_t* masks, int N, uint64_t shard_len, int block_log2,
                        uint64_t seed, uint64_t base_index, float* out, uint8_t* count_out, void* workspace,
                        size_t workspace_bytes, void* stream) {
  return path_impl<float>(true, grads, masks, N, shard_len, block_log2, seed, base_index, out, count_out, workspace,
                          workspace_bytes, stream, false);
}
or_status or_fused_path_bf16(const uint16_t* grads, const uint32_t* masks, int N, uint64_t shard_len,
                             int block_log2, uint64_t seed, uint64_t base_index, uint16_t* out, uint8_t* count_out,
                             void* workspace, size_t workspace_bytes, void* stream) {
  return path_impl<uint16_t>(true, grads, masks, N, shard_len, block_log2, seed, base_index, out, count_out, workspace,
                             workspace_bytes, stream, true);
}

or_status or_fused_path_bf16_static(const uint16_t* grads, const uint32_t* masks, int N, uint64_t shard_len,
                                    int block_log2, uint64_t seed, uint64_t base_index, uint16_t* out,
                                    uint8_t* count_out, void* stream) {
  DisarmOnExit disarm;
  const size_t need = workspace_bytes(shard_len, block_log2);
  if (need && shard_len > kStaticMaxShard) return OR_ERR_WORKSPACE;   // beyond what the static scratch holds
  void* ws = nullptr;
  if (need) {
    hipError_t e;
    ws = scratch_of_current_device(&e);
    if (!ws) return finish(e);
  }
  if (or_status s = check_path(grads, masks, N, shard_len, block_log2, base_index, out, count_out, ws, need, 2)) return s;
  return run_path<uint16_t>(true, grads, masks, N, shard_len, block_log2, seed, base_index, out, count_out, ws, stream, true);
}

or_status or_finalize(const float* sum, const uint8_t* count, uint64_t shard_len, float* mean_out, void* stream) {
  return finalize_impl<float>(sum, count, shard_len, mean_out, stream);
}
or_status or_finalize_bf16(const float* sum, const uint8_t* count, uint64_t shard_len, uint16_t* mean_out,
                           void* stream) {
  return finalize_impl<uint16_t>(sum, count, shard_len, mean_out, stream);
}
or_status or_loss_decision(uint64_t received_total, int N, uint64_t shard_len, const or_loss_policy* policy,
                           int prev_transform_on, int* action_out, int* transform_on_out, double* loss_out) {
  if (!policy || !action_out || !transform_on_out) return OR_ERR_NULL;
  if (N < 1 || N > OR_MAX_WORKERS) return OR_ERR_WORKERS;
  if (policy->transform_on_loss != policy->transform_on_loss || policy->skip_loss != policy->skip_loss ||
      policy->halt_loss != policy->halt_loss)
    return OR_ERR_SHAPE;
  if (shard_len == 0 || shard_len > UINT64_MAX / (uint64_t)N) return OR_ERR_SHAPE;
  const uint64_t sent = (uint64_t)N * shard_len;
  if (received_total > sent) return OR_ERR_SHAPE;
  // the missing arrivals are an exact integer, and every threshold is compared with the exact ratio
  const uint64_t missing = sent - received_total;
  *action_out = ratio_exceeds(missing, sent, policy->halt_loss)
                    ? OR_ACT_HALT
                    : (ratio_exceeds(missing, sent, policy->skip_loss) ? OR_ACT_SKIP : OR_ACT_APPLY);
  *transform_on_out = (prev_transform_on || ratio_exceeds(missing, sent, policy->transform_on_loss)) ? 1 : 0;
  if (loss_out) *loss_out = (double)missing / (double)sent;   // reported value only: one rounding
  return OR_OK;
}

or_status or_received_total(const uint8_t* count, uint64_t shard_len, uint64_t* total_out, void* stream) {
  return received_total_impl(count, shard_len, (unsigned long long*)total_out, stream);
}
or_status or_rht_decode_masked(const float* agg, const uint32_t* mask, uint64_t n, int block_log2, uint64_t seed,
                               uint64_t base_index, float* out, void* stream) {
  return decode_impl<float>(agg, nullptr, false, n, block_log2, seed, base_index, out, stream, false, mask, true);
}
or_status or_rht_decode_masked_bf16(const float* agg, const uint32_t* mask, uint64_t n, int block_log2,
                                    uint64_t seed, uint64_t base_index, uint16_t* out, void* stream) {
  return decode_impl<uint16_t>(agg, nullptr, false, n, block_log2, seed, base_index, out, stream, true, mask, true);
}
or_status or_masked_reduce_pairs(const float* sums, const uint8_t* counts, const uint32_t* masks, int G,
                                 uint64_t shard_len, float* sum_out, uint8_t* count_out, void* stream) {
  return pairs_impl(sums, counts, masks, G, shard_len, sum_out, count_out, stream);
}

or_status or_fused_path_batched(const or_bucket* buckets, int n_buckets, int N, int block_log2, int bf16,
                                void* workspace, size_t workspace_bytes, void* stream) {
  return path_batched_impl(true, buckets, n_buckets, N, block_log2, bf16 != 0, nullptr, workspace, workspace_bytes, stream);
}
or_status or_fused_path_batched_monitored(const or_bucket* buckets, int n_buckets, int N, int block_log2, int bf16,
                                          uint64_t* totals, void* workspace, size_t workspace_bytes, void* stream) {
  return path_batched_impl(true, buckets, n_buckets, N, block_log2, bf16 != 0, (unsigned long long*)totals, workspace,
                           workspace_bytes, stream);
}
or_status or_reduce_decode_batched(const or_bucket* buckets, int n_buckets, int N, int block_log2, int bf16,
                                   uint64_t* totals, void* workspace, size_t workspace_bytes, void* stream) {
  return path_batched_impl(false, buckets, n_buckets, N, block_log2, bf16 != 0, (unsigned long long*)totals, workspace,
                           workspace_bytes, stream);
}
or_status or_masked_reduce_batched(const or_stage_bucket* buckets, int n_buckets, int N, int bf16, void* stream) {
  return stage_batched_impl(true, buckets, n_buckets, N, OR_MIN_LOG2, bf16 != 0, stream);
}
or_status or_finalize_decode_batched(const or_stage_bucket* buckets, int n_buckets, int block_log2, int bf16,
                                     void* stream) {
  return stage_batched_impl(false, buckets, n_buckets, 1, block_log2, bf16 != 0, stream);
}

}  // extern "C"

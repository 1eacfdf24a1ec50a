// The fused path for blocks of 2^12 .. 2^14 entries with every worker encoded by itself, for launches of few tiles (in
// bf16, of few workers too): per worker sign flip (layout A), transposed transform to layout B, addition under the received
// mask; the mean is decoded the same way back.
//
// Latency bounds such launches.  The other form (rht_fused.hpp) looks at all received bits before the first addition and
// encodes the whole workers' sum last; here that start and that last transform cost more than the transforms they save.
// us, that form -> this one, 1 % of the packets lost, data in the cache: fp32, 4 workers: 2^12, 512 tiles 9.8 -> 9.0; 2^13,
// 128 tiles 11.4 -> 9.3, 1024 tiles 34.7 -> 29.6; 2^14, 256 tiles 18.8 -> 16.6; bf16, 4 workers: 2^13, 400 tiles 16.7 ->
// 14.3.  Larger launches are bound by memory (fp32) or by the transforms (bf16: 2^13, 8 workers, 1024 tiles 39 -> 47).
#pragma once
#include "rht_kernels.hpp"

namespace ordev {

template <int K, class In, bool TOTAL>
__device__ __forceinline__ void fused_each_tile(const PathArgs& a, u64 unit) {
  constexpr int T = Geo<K>::T, R = Geo<K>::R;
  constexpr bool FULL = kShardTilesFull<K>;
  static_assert(Geo<K>::PARTS == 1 && R == 16 && Geo<K>::Q >= 1, "tiles that transform_transposed takes");
  __shared__ float xbuf[2][tr_floats<K>];
  __shared__ uint32_t arrived;
  if (TOTAL && threadIdx.x == 0) arrived = 0;   // the transforms' barriers lie before and after the additions
  const int wave = wave_id(), lane = lane_id();
  const u64 L = a.n_pad, e0 = unit * T;
  const In* grads = (const In*)a.in;
  const float sigma = tr_sigma(lane);
  float acc[R], va[R];
  uint32_t cnt[R / 4];
  int full = 0, flip = 0;
  const int moff = mask_word_offset<K>(wave, lane);
  const u64 mrow = L >> 5;
  // the first worker's tile is requested before the signs are computed, so Philox runs under its latency
  load_tile<K, false, FULL, true>(grads, e0, L, wave, lane, va);
  uint32_t ma = load_mask_words<K, FULL>(a.masks, e0, L, moff);
  u64 sg[R];
  sign_masks(a.seed, a.base + e0 + (u64)wave * Geo<K>::WAVE_ENTRIES, sg);
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int r = 0; r < R / 4; ++r) cnt[r] = 0;

  auto encode_and_add = [&](float (&v)[R], uint32_t words) {
    apply_signs(v, sg);
    transform_transposed<K>(v, xbuf[flip], xbuf[flip ^ 1], wave, lane);
    flip ^= 1;
    masked_accumulate(v, words, acc, cnt, full);
  };
  // Two tile buffers: the next worker's tile travels while this one is transformed.  The loads inside
  // the loop are unconditional (the last one or two workers are handled after it), so that the count
  // of loads in flight is the same on every path into a wait and the compiler waits for the older
  // tile only.
  float vb[R];
  uint32_t mb;
  auto request = [&](int i, float (&v)[R], uint32_t& words) {
    load_tile<K, false, FULL, true>(grads + (u64)i * L, e0, L, wave, lane, v);
    words = load_mask_words<K, FULL>(a.masks + (u64)i * mrow, e0, L, moff);
  };
  int i = 0;
  for (; i + 2 < a.N; i += 2) {
    request(i + 1, vb, mb);
    encode_and_add(va, ma);
    request(i + 2, va, ma);
    encode_and_add(vb, mb);
  }
  if (i + 1 < a.N) {
    request(i + 1, vb, mb);
    encode_and_add(va, ma);
    encode_and_add(vb, mb);
  } else {
    encode_and_add(va, ma);
  }
  __builtin_amdgcn_sched_barrier(0);
  store_counts<K, FULL>(a.count_out, e0, L, wave, lane, cnt, full);
  if (TOTAL && a.total_out) {   // Sec. 3.4 loss monitoring: gathered in LDS, one atomic per workgroup
    uint32_t n = 0;
#pragma unroll
    for (int r = 0; r < R / 4; ++r) n = __builtin_amdgcn_sad_u8(cnt[r], 0u, n);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o, 64);
    if (lane == 0) atomicAdd(&arrived, n + (uint32_t)full * (64 * R));
  }
  finalize_mean(acc, cnt, full, sigma * a.scale);
  __builtin_amdgcn_sched_barrier(0);
  transform_transposed<K>(acc, xbuf[flip], xbuf[flip ^ 1], wave, lane);   // the same code takes layout B to A
  if (TOTAL && a.total_out && threadIdx.x == 0) atomicAdd(a.total_out, (unsigned long long)arrived);
  __builtin_amdgcn_sched_barrier(0);
  const float c = a.scale * sigma;
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] *= c;
  apply_signs(acc, sg);
  store_tile<K, false, FULL, true>((In*)a.out, e0, L, wave, lane, acc);
}

template <int K, class In>
__global__ __launch_bounds__(Geo<K>::THREADS) __attribute__((amdgpu_waves_per_eu(1)))
void k_fused_each(PathArgs a) {
  fused_each_tile<K, In, false>(a, blockIdx.x);
}
template <int K, class In>
__global__ __launch_bounds__(Geo<K>::THREADS) __attribute__((amdgpu_waves_per_eu(1)))
void k_fused_each_batched(BatchArgs ba) {
  PathArgs a;
  const u64 unit = bucket_of(ba, a);
  fused_each_tile<K, In, true>(a, unit);
}

}  // namespace ordev

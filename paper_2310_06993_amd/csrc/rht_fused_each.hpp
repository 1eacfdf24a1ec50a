// The fused path for blocks of up to 2^14 entries (bf16: 2^10) with every worker encoded by itself: per worker sign flip (layout A),
// transform to layout B, rounding to the wire type (bf16), addition under the received mask; the mean is decoded the same way
// back.  Tiles of 2, 4, 8 or 16 wavefronts use the transposed transform of rht_tile.hpp, in both directions.
//
// bf16: every worker's encoded value is rounded as if it had been stored and sent, so every worker has to be encoded (above 2^10:
// rht_fused_bf16.hpp).  fp32: blocks of 2^12 .. 2^14, and few workers at 2^11 and below 2^10, where adding up whole workers first costs
// more at the start and the end of a workgroup than the transforms that it saves (figures at the rule, inst.hip).
//
// PREFETCH: a second tile buffer, so that the next worker's tile is in flight during the transform (same arithmetic, same
// results).  It shortens the chain of dependent steps of a workgroup and wins while a launch puts at most three workgroups on
// each of the 256 CUs; without it more of them fit, which wins beyond that.  fp32 2^12, us, without -> with: N = 8, 512 tiles
// 23.4 -> 20.3, 780 tiles 24.5 -> 25.2; N = 32, 780 tiles 75 -> 85, 2560 tiles 231 -> 244.
#pragma once
#include "rht_kernels.hpp"

namespace ordev {

// `arrived`: arrivals of the workgroup's tiles, and how many of its wavefronts have added theirs; `tiles`: of this workgroup.  FULL:
// the tile is not cut short by the end of the shard.
template <int K, class In, bool PREFETCH, bool TOTAL, int SLOTS, bool FULL>
__device__ __forceinline__ void fused_each_tile(const PathArgs& a, u64 unit, int wave, int tiles,
                                                float (*xbuf)[Geo<K>::Q >= 1 ? tr_floats<K> : 1], uint32_t* arrived) {
  constexpr int T = Geo<K>::T, R = Geo<K>::R;
  constexpr bool TRANSP = Geo<K>::Q >= 1;   // tiles of one wavefront: the plain transform, which needs no LDS there
  static_assert(Geo<K>::PARTS == 1 && R == 16, "blocks of up to 2^14, 16 entries a lane");
  const int lane = lane_id(), kt = tile_bits<K>(a.k);
  const u64 L = a.n_pad, e0 = unit * T;
  const In* grads = (const In*)a.in;
  const float sigma = TRANSP ? tr_sigma(lane) : lane_sigma(lane, kt < 6 ? kt : 6);
  // a power-of-two scale commutes with rounding to the wire type; any other scale is applied first
  const bool scale_first = sizeof(In) == 2 && (a.k & 1);
  float acc[R], va[R];
  uint32_t cnt[R / 4];
  int full = 0, flip = 0;
  const int moff = mask_word_offset<K>(wave, lane);
  const u64 mrow = L >> 5;
  static_assert(FULL || Geo<K>::W == 1, "only tiles of one wavefront are cut short");
  [[maybe_unused]] const int left = FULL ? T : (int)(L - e0);
  auto request = [&](int i, float (&v)[R], uint32_t& words) {
    if constexpr (FULL) {
      load_tile<K, false, true, true>(grads + (u64)i * L, e0, L, wave, lane, v);
    } else {   // past the end: the last entry again, as a zero (range-checked loads: their descriptors in vector registers, see below)
      const In* q = grads + (u64)i * L + e0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int e = r * 64 + lane;
        const float x = to_f32(load_one<true>(&q[e < left ? e : left - 1]));
        v[r] = e < left ? x : 0.0f;
      }
    }
    words = load_mask_words<K, FULL>(a.masks + (u64)i * mrow, e0, L, moff);
  };
  // the first worker's tile is requested before the signs are computed, so Philox runs under its latency
  uint32_t ma;
  request(0, va, ma);
  u64 sg[R];
  sign_masks(a.seed, a.base + e0 + (u64)wave * Geo<K>::WAVE_ENTRIES, sg);
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int r = 0; r < R / 4; ++r) cnt[r] = 0;

  auto encode_and_add = [&](float (&v)[R], uint32_t words) {
    apply_signs(v, sg);
    if constexpr (TRANSP) transform_transposed<K>(v, xbuf[flip], xbuf[flip ^ 1], wave, lane);
    else transform<K, true>(v, xbuf[0], wave, lane, kt);
    flip ^= 1;
    if constexpr (sizeof(In) == 2) {
      if (scale_first) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = round_to<In>(v[r] * a.scale);
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = round_to<In>(v[r]);
      }
    }
    masked_accumulate(v, words, acc, cnt, full);
  };
  if constexpr (PREFETCH) {
    // The loads inside the loop are unconditional (the last one or two workers are handled after it), so that the count
    // of loads in flight is the same on every path into a wait and the compiler waits for the older tile only.
    float vb[R];
    uint32_t mb;
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
  } else {
    for (int i = 0; i < a.N; ++i) {
      encode_and_add(va, ma);
      if (i + 1 < a.N) request(i + 1, va, ma);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  store_counts<K, FULL>(a.count_out, e0, L, wave, lane, cnt, full);
  if constexpr (TOTAL) {   // Sec. 3.4 loss monitoring: gathered in LDS, one atomic per workgroup
    if (a.total_out) {
      uint32_t n = 0;
#pragma unroll
      for (int r = 0; r < R / 4; ++r) n = __builtin_amdgcn_sad_u8(cnt[r], 0u, n);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o, 64);
      if (lane == 0) {
        atomicAdd(&arrived[0], n + (uint32_t)full * (64 * R));
        if constexpr (SLOTS > 1) {
          __threadfence_block();   // the arrivals before the sign that they are there
          if (atomicAdd(&arrived[1], 1u) == (uint32_t)tiles - 1) atomicAdd(a.total_out, (unsigned long long)atomicAdd(&arrived[0], 0u));
        }
      }
    }
  }
  finalize_mean(acc, cnt, full, sigma * (scale_first ? 1.0f : a.scale));
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (TRANSP) transform_transposed<K>(acc, xbuf[flip], xbuf[flip ^ 1], wave, lane);   // the same code takes layout B to A
  else transform<K, false>(acc, xbuf[0], wave, lane, kt);
  if (TOTAL && SLOTS == 1 && a.total_out && threadIdx.x == 0) atomicAdd(a.total_out, (unsigned long long)arrived[0]);
  __builtin_amdgcn_sched_barrier(0);
  const float c = a.scale * sigma;
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] *= c;
  apply_signs(acc, sg);
  store_tile<K, false, FULL, true>((In*)a.out, e0, L, wave, lane, acc);
}

// SLOTS > 1 (tiles of one wavefront): the workgroup's wavefronts serve SLOTS tiles of a bucket, one atomic for all their arrivals
// (see fused_tile).  K = 0: whether the tile is cut short is decided once, for all accesses.  (With
// range-checked loads in the loop over the workers the compiler keeps their descriptors in vector registers and makes a loop of
// every load: launches of whole tiles two to three times slower, one cut tile of 32 workers 48 -> 69 us.)
template <int K, class In, bool PREFETCH, bool TOTAL, int SLOTS>
__device__ __forceinline__ void fused_each(const PathArgs& a, u64 first_unit, u64 units) {
  static_assert(SLOTS == 1 || Geo<K>::W == 1, "several tiles per workgroup: tiles of one wavefront");
  __shared__ float xbuf[2][Geo<K>::Q >= 1 ? tr_floats<K> : 1];
  __shared__ uint32_t arrived[2];
  if (TOTAL && threadIdx.x < 2) arrived[threadIdx.x] = 0;   // the transforms' barriers lie before and after the additions
  const int slot = SLOTS > 1 ? wave_id() : 0, wave = SLOTS > 1 ? 0 : wave_id();
  const int tiles = units - first_unit < SLOTS ? (int)(units - first_unit) : SLOTS;
  if constexpr (SLOTS > 1) {
    __syncthreads();   // the only one: from here on every wavefront is on its own
    if (slot >= tiles) return;
  }
  const u64 unit = first_unit + slot;
  if constexpr (kShardTilesFull<K>) {
    fused_each_tile<K, In, PREFETCH, TOTAL, SLOTS, true>(a, unit, wave, tiles, xbuf, arrived);
  } else {
    if ((unit + 1) * Geo<K>::T <= a.n_pad) fused_each_tile<K, In, PREFETCH, TOTAL, SLOTS, true>(a, unit, wave, tiles, xbuf, arrived);
    else fused_each_tile<K, In, PREFETCH, TOTAL, SLOTS, false>(a, unit, wave, tiles, xbuf, arrived);
  }
}

template <int K, class In, bool PREFETCH>
__global__ __launch_bounds__(Geo<K>::THREADS) __attribute__((amdgpu_waves_per_eu(1)))
void k_fused_each(PathArgs a) {
  fused_each<K, In, PREFETCH, false, 1>(a, blockIdx.x, gridDim.x);
}
// K = 0 with arrival totals: a workgroup serves SLOTS = kEachSlots tiles of one bucket, and ba.tile_start counts workgroups.  us, a
// workgroup per tile -> eight: 60 x 400 tiles, N = 8, bf16 2^8 200 -> 145 with totals; without them 4 x 100 tiles 15 -> 17.
template <int K> constexpr int kEachSlots = K == 0 ? 8 : 1;
template <int K, class In, bool PREFETCH, int SLOTS>
__global__ __launch_bounds__(Geo<K>::THREADS * SLOTS) __attribute__((amdgpu_waves_per_eu(1)))
void k_fused_each_batched(BatchArgs ba) {
  constexpr int T = Geo<K>::T;
  PathArgs a;
  const u64 group = bucket_of(ba, a, blockIdx.x);
  fused_each<K, In, PREFETCH, (SLOTS == kEachSlots<K>), SLOTS>(a, group * SLOTS, (a.n_pad + T - 1) / T);
}

}  // namespace ordev

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

// `missing`: what the workgroup's tiles miss, and how many of its wavefronts have added theirs; `tiles`: of this workgroup.  FULL:
// the tile is not cut short by the end of the shard.
template <int K, class In, bool PREFETCH, bool TOTAL, int SLOTS, bool FULL>
__device__ __forceinline__ void fused_each_tile(const PathArgs& a, u64 unit, int wave, int tiles,
                                                float (*xbuf)[Geo<K>::Q >= 1 ? tr_floats<K> : 1], uint32_t* missing) {
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
      // With totals the offsets are formed here and 32 bits wide: kept in registers all along they take 16 more than without totals,
      // and with them a wavefront from every SIMD.  142 registers -> 93, us, bf16 2^9, N = 16, 3500 / 5000 tiles 63.6 -> 51.5 / 71.0 -> 61.4.
      // (Without totals 126 -> 92: 5000 tiles 67.0 -> 60.5, but up to 4096 tiles 2 % slower.)
      int lane_t = lane;
      if constexpr (TOTAL) asm volatile("" : "+v"(lane_t));
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if constexpr (TOTAL) {   // (blocks past the end are not stored, whatever they hold)
          const unsigned e = r * 64 + lane_t, last = left - 1;
          v[r] = to_f32(load_one<true>(&q[e < last ? e : last]));
        } else {
          const int e = r * 64 + lane;
          const float x = to_f32(load_one<true>(&q[e < left ? e : left - 1]));
          v[r] = e < left ? x : 0.0f;
        }
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
  if constexpr (TOTAL) {   // Sec. 3.4 loss monitoring: gathered in LDS, one atomic per workgroup at most
    if (a.total_out) {
      const uint32_t n = missing_of<R>(cnt, full, a.N, FULL ? 64 * R : left);
      if (lane == 0) {
        if (n) atomicAdd(&missing[0], n);
        if constexpr (SLOTS > 1) {
          __threadfence_block();   // what is missing before the sign that it is there
          if (atomicAdd(&missing[1], 1u) == (uint32_t)tiles - 1) add_total(a, unit < SLOTS, atomicAdd(&missing[0], 0u));
        }
      }
    }
  }
  finalize_mean(acc, cnt, full, sigma * (scale_first ? 1.0f : a.scale));
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (TRANSP) transform_transposed<K>(acc, xbuf[flip], xbuf[flip ^ 1], wave, lane);   // the same code takes layout B to A
  else transform<K, false>(acc, xbuf[0], wave, lane, kt);
  if (TOTAL && SLOTS == 1 && a.total_out && threadIdx.x == 0) add_total(a, unit == 0, missing[0]);
  __builtin_amdgcn_sched_barrier(0);
  const float c = a.scale * sigma;
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] *= c;
  apply_signs(acc, sg);
  store_tile<K, false, FULL, true>((In*)a.out, e0, L, wave, lane, acc);
}

// SLOTS > 1 (tiles of one wavefront): the workgroup's wavefronts serve SLOTS tiles of a bucket, one atomic for all that they miss
// (see fused_tile).  K = 0: whether the tile is cut short is decided once, for all accesses.  (With
// range-checked loads in the loop over the workers the compiler keeps their descriptors in vector registers and makes a loop of
// every load: launches of whole tiles two to three times slower, one cut tile of 32 workers 48 -> 69 us.)
template <int K, class In, bool PREFETCH, bool TOTAL, int SLOTS>
__device__ __forceinline__ void fused_each(const PathArgs& a, u64 first_unit, u64 units) {
  static_assert(SLOTS == 1 || Geo<K>::W == 1, "several tiles per workgroup: tiles of one wavefront");
  __shared__ float xbuf[2][Geo<K>::Q >= 1 ? tr_floats<K> : 1];
  __shared__ uint32_t missing[2];
  if (TOTAL && threadIdx.x < 2) missing[threadIdx.x] = 0;   // the transforms' barriers lie before and after the additions
  const int slot = SLOTS > 1 ? wave_id() : 0, wave = SLOTS > 1 ? 0 : wave_id();
  const int tiles = units - first_unit < SLOTS ? (int)(units - first_unit) : SLOTS;
  if constexpr (SLOTS > 1) {
    __syncthreads();   // the only one: from here on every wavefront is on its own
    if (slot >= tiles) return;
  }
  const u64 unit = first_unit + slot;
  if constexpr (kShardTilesFull<K>) {
    fused_each_tile<K, In, PREFETCH, TOTAL, SLOTS, true>(a, unit, wave, tiles, xbuf, missing);
  } else {
    if ((unit + 1) * Geo<K>::T <= a.n_pad)
      with_block_size<K>(a, [&](const PathArgs& b) __attribute__((always_inline)) { fused_each_tile<K, In, PREFETCH, TOTAL, SLOTS, true>(b, unit, wave, tiles, xbuf, missing); });
    else if constexpr (sizeof(In) == 2)   // the tile that is cut short too (figures below); fp32, 2^8, N = 2 / 3, 3146496 entries, for any size -> this 10.8 -> 11.6 / 13.0 -> 14.5
      with_block_size<K, 0, 9>(a, [&](const PathArgs& b) __attribute__((always_inline)) { fused_each_tile<K, In, PREFETCH, TOTAL, SLOTS, false>(b, unit, wave, tiles, xbuf, missing); });
    else fused_each_tile<K, In, PREFETCH, TOTAL, SLOTS, false>(a, unit, wave, tiles, xbuf, missing);
  }
}

// For launches that leave CUs idle: G groups of W wavefronts encode G workers side by side.  The encoded values of a round go
// through LDS, zero where they were lost, and group g adds those of its share of the registers over the workers, in order: the same
// operations in the same order as above.  Group 0 decodes.  Bound by the chain of rounds: with four wavefronts a SIMD a round of 2^12
// takes about 1.5 us of vector instructions and 1.6 us of LDS (figures at the rule, inst.hip).
template <int K, class In, int G, bool TOTAL, bool FULL>
__device__ __forceinline__ void fused_each_groups_tile(const PathArgs& a, u64 unit, int grp, int wave, float (*x)[Geo<K>::Q >= 1 ? tr_floats<K> : 1024],
                                                       float (*y)[Geo<K>::Q >= 1 ? tr_floats<K> : 1], uint32_t* missing, uint32_t* lossy) {
  constexpr int T = Geo<K>::T, R = Geo<K>::R, W = Geo<K>::W, S = R / G;   // S: registers of a share
  constexpr bool TRANSP = Geo<K>::Q >= 1;
  static_assert(Geo<K>::PARTS == 1 && R == 16 && G >= 2 && G <= 16, "blocks of up to 2^14, a share is at least a register");
  static_assert(FULL || W == 1, "only tiles of one wavefront are cut short");
  const int lane = lane_id(), kt = tile_bits<K>(a.k), N = a.N;
  const u64 L = a.n_pad, e0 = unit * T, mrow = L >> 5;
  const float sigma = TRANSP ? tr_sigma(lane) : lane_sigma(lane, kt < 6 ? kt : 6);
  const bool scale_first = sizeof(In) == 2 && (a.k & 1);
  const int moff = mask_word_offset<K>(wave, lane);
  [[maybe_unused]] const int left = FULL ? T : (int)(L - e0);
  auto request = [&](int i, float (&v)[R], uint32_t& words) {   // past the last worker: the last one again, not used
    const int w = i < N ? i : N - 1;
    const In* p = (const In*)a.in + (u64)w * L;
    if constexpr (FULL) {
      load_tile<K, false, true, true>(p, e0, L, wave, lane, v);
    } else {   // past the end: the last entry again, as a zero
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int e = r * 64 + lane;
        const float t = to_f32(load_one<true>(&p[e0 + (e < left ? e : left - 1)]));
        v[r] = e < left ? t : 0.0f;
      }
    }
    words = load_mask_words<K, FULL>(a.masks + (u64)w * mrow, e0, L, moff);
  };
  float va[R];
  uint32_t ma;
  request(grp, va, ma);
  u64 sg[R];
  sign_masks(a.seed, a.base + e0 + (u64)wave * Geo<K>::WAVE_ENTRIES, sg);
  float acc[S];
#pragma unroll
  for (int r = 0; r < S; ++r) acc[r] = 0.0f;
  constexpr int V = S < 4 ? S : 4;   // values of one access to LDS
  typedef float values_t __attribute__((ext_vector_type(V)));
  for (int first = 0; first < N; first += G) {
    const bool works = first + grp < N;
    float v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = va[r];
    const uint32_t words = ma;
    if (first + G < N) request(first + grp + G, va, ma);
    apply_signs(v, sg);
    // (a group without a worker goes through the transform for the sake of its barrier)
    if constexpr (TRANSP) transform_transposed<K>(v, x[grp], y[grp], wave, lane);
    else transform<K, true>(v, x[grp], wave, lane, kt);
    if (works) {
      if constexpr (sizeof(In) == 2) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = round_to<In>(scale_first ? v[r] * a.scale : v[r]);
      }
      if (!all_arrived(words)) {
        if (lane == 0) *lossy = 1;
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = in_mask(mask_of_reg(words, r)) ? v[r] : 0.0f;
      }
      float* to = x[grp] + wave * 1024 + lane * V;   // by access; behind this wavefront's reads of its part of x
      if constexpr (TRANSP) to = x[grp] + wave * tr_wave<K> + lane * V;
#pragma unroll
      for (int j = 0; j < R / V; ++j) {
        values_t t;
#pragma unroll
        for (int d = 0; d < V; ++d) t[d] = v[j * V + d];
        *(values_t*)(to + j * 64 * V) = t;
      }
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (first + g < N) {
        const float* from = x[g] + wave * (TRANSP ? tr_wave<K> : 1024) + grp * (64 * S) + lane * V;
#pragma unroll
        for (int j = 0; j < S / V; ++j) {
          const values_t t = *(const values_t*)(from + j * 64 * V);
#pragma unroll
          for (int d = 0; d < V; ++d) acc[j * V + d] += t[d];
        }
      }
    }
    __syncthreads();
  }
  // ---- counts and mean over what arrived.  The last round ended in a barrier behind which everyone sees `lossy`
  float* flat = x[0];
  float* means = flat + G * W * 256;          // by wavefront, register, lane (layout B)
  static_assert(G * T / 4 + T <= G * (TRANSP ? tr_floats<K> : 1024), "counts and means fit");
  const float post = sigma * (scale_first ? 1.0f : a.scale);
  // received bits of 16 entries: half of word lane >> 1 of the wavefront's 32 words, i.e. register lane >> 2, lanes 16 (lane & 3) ..
  uint32_t c4[4];
  const uint32_t all = (uint32_t)N * 0x01010101u;
  const bool inside = FULL || lane * 16 < left;
  if (*(volatile uint32_t*)lossy == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) c4[q] = inside ? all : 0;
    const float f = post * __builtin_amdgcn_rcpf((float)N);
#pragma unroll
    for (int r = 0; r < S; ++r) means[(wave * R + grp * S + r) * 64 + lane] = acc[r] * f;
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) c4[q] = 0;
    const int off = off_b<K>(wave, lane >> 2) + (lane & 3) * 16;
    for (int i = grp; i < N; i += G) {
      const uint32_t bits = inside ? ((const uint16_t*)(a.masks + (u64)i * mrow + (e0 >> 5)))[off >> 4] : 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) c4[q] += (((bits >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;
    }
    *(uint4*)(flat + ((grp * W + wave) * 64 + lane) * 4) = make_uint4(c4[0], c4[1], c4[2], c4[3]);
    __syncthreads();
    // every wavefront adds up the counts of its part over the groups; group 0 keeps what it stores
    const uint8_t* bytes = (const uint8_t*)flat + wave * 1024;
#pragma unroll
    for (int r = 0; r < S; ++r) {
      uint32_t n = 0;
#pragma unroll
      for (int g = 0; g < G; ++g) n += bytes[g * W * 1024 + (grp * S + r) * 64 + lane];
      means[(wave * R + grp * S + r) * 64 + lane] = n ? acc[r] * (post * __builtin_amdgcn_rcpf((float)n)) : 0.0f;
    }
    if (grp == 0) {
#pragma unroll
      for (int g = 1; g < G; ++g) {
        const uint4 o = *(const uint4*)(flat + ((g * W + wave) * 64 + lane) * 4);
        c4[0] += o.x; c4[1] += o.y; c4[2] += o.z; c4[3] += o.w;
      }
    }
  }
  if (grp == 0 && a.count_out) {
    const int off = off_b<K>(wave, lane >> 2) + (lane & 3) * 16;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)(a.count_out + e0), 0, left, 0x00020000);
#pragma unroll
    for (int q = 0; q < 4; ++q) store_counts4(c4[q], rs, off + q * 4, 0, ((uintptr_t)a.count_out & 3) == 0);
  }
  if (TOTAL && grp == 0 && a.total_out && *(volatile uint32_t*)lossy) {   // Sec. 3.4 loss monitoring: gathered in LDS, one atomic per workgroup at most
    uint32_t n = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) n = __builtin_amdgcn_sad_u8(c4[q], 0u, n);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o, 64);
    if (lane == 0) atomicAdd(missing, (uint32_t)N * (FULL ? 1024u : (uint32_t)left) - n);
  }
  __syncthreads();
  if (TOTAL && a.total_out && threadIdx.x == 0) add_total(a, unit == 0, *missing);
  if (grp > 0) return;   // (a barrier waits for the wavefronts that are left)
  float v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = means[(wave * R + r) * 64 + lane];
  __syncthreads();
  if constexpr (TRANSP) transform_transposed<K>(v, x[0], y[0], wave, lane);
  else transform<K, false>(v, x[0], wave, lane, kt);
  const float c = a.scale * sigma;
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] *= c;
  apply_signs(v, sg);
  store_tile<K, false, FULL, true>((In*)a.out, e0, L, wave, lane, v);
}
template <int K, class In, int G, bool TOTAL>
__device__ __forceinline__ void fused_each_groups(const PathArgs& a, u64 unit) {
  constexpr int W = Geo<K>::W;
  __shared__ __align__(16) float x[G][Geo<K>::Q >= 1 ? tr_floats<K> : 1024];
  __shared__ __align__(16) float y[G][Geo<K>::Q >= 1 ? tr_floats<K> : 1];
  __shared__ uint32_t missing, lossy;
  const int grp = wave_id() / W, wave = wave_id() % W;
  if (threadIdx.x == 0) missing = lossy = 0;
  __syncthreads();
  if constexpr (kShardTilesFull<K>) {
    fused_each_groups_tile<K, In, G, TOTAL, true>(a, unit, grp, wave, x, y, &missing, &lossy);
  } else {
    // The tile that is cut short too, bf16: for any size its chain was the launch's.  us, before whole tiles were compiled for each size -> for any size ->
    // this, 2^8, N = 3 / 12, 27392 entries 5.36 -> 5.60 -> 5.14 / 7.92 -> 8.23 -> 7.31, N = 8, 1 M 19.3 -> 18.8 -> 15.9.
    // fp32 (blocks below 2^10, two to five workers): the fewest code.  As a share of what it took before there were sizes, 2^6 .. 2^9, N = 4, whole tiles of several
    // buckets / of one / cut tiles of several / of one: bf16's way 1.03 / 0.98 / 1.10 / 1.04, a switch and one form for cut tiles 1.03 / 0.98 / 1.03 / 1.02, this 0.99 / 0.96 /
    // 1.03 / 1.01.
    constexpr bool F32 = sizeof(In) == 4;
    if ((unit + 1) * Geo<K>::T <= a.n_pad)
      with_block_size<K, F32 ? 9 : 0>(a, [&](const PathArgs& b) __attribute__((always_inline)) { fused_each_groups_tile<K, In, G, TOTAL, true>(b, unit, grp, wave, x, y, &missing, &lossy); });
    else if constexpr (F32) fused_each_groups_tile<K, In, G, TOTAL, false>(a, unit, grp, wave, x, y, &missing, &lossy);
    else
      with_block_size<K, 0, 9>(a, [&](const PathArgs& b) __attribute__((always_inline)) { fused_each_groups_tile<K, In, G, TOTAL, false>(b, unit, grp, wave, x, y, &missing, &lossy); });
  }
}
template <int K, class In, int G>
__global__ __launch_bounds__(Geo<K>::THREADS * G) void k_fused_each_groups(PathArgs a) {
  fused_each_groups<K, In, G, false>(a, blockIdx.x);
}
template <int K, class In, int G>
__global__ __launch_bounds__(Geo<K>::THREADS * G) void k_fused_each_groups_batched(BatchArgs ba) {
  PathArgs a;
  const u64 unit = bucket_of(ba, a, blockIdx.x);
  fused_each_groups<K, In, G, true>(a, unit);
}

template <int K, class In, bool PREFETCH>
__global__ __launch_bounds__(Geo<K>::THREADS) __attribute__((amdgpu_waves_per_eu(1)))
void k_fused_each(PathArgs a) {
  fused_each<K, In, PREFETCH, false, 1>(a, blockIdx.x, gridDim.x);
}
// K = 0 with arrival totals: a workgroup serves SLOTS tiles of one bucket (rule in inst.hip), and ba.tile_start counts workgroups.
// Without totals a workgroup per tile (4 x 100 tiles, eight a workgroup -> one: 17 -> 15).
template <int K, class In, bool PREFETCH, int SLOTS>
__global__ __launch_bounds__(Geo<K>::THREADS * SLOTS) __attribute__((amdgpu_waves_per_eu(1)))
void k_fused_each_batched(BatchArgs ba) {
  constexpr int T = Geo<K>::T;
  PathArgs a;
  const u64 group = bucket_of(ba, a, blockIdx.x);
  fused_each<K, In, PREFETCH, (K != 0 || SLOTS > 1), SLOTS>(a, group * SLOTS, (a.n_pad + T - 1) / T);
}

}  // namespace ordev

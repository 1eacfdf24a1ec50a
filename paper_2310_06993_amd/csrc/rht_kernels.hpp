// Kernels of the gradient-bucket path (OptiReduce Sec. 3.3 encode/decode, Sec. 3.1.1 aggregation),
// one workgroup per output tile.  See rht_tile.hpp for the tile geometry and the two layouts.
#pragma once
#include "rht_tile.hpp"

namespace ordev {

struct PathArgs {
  const void* in;          // encode: gradient; decode: mean (or sum); reduce/fused: [N][L] shards / raw slices
  const uint8_t* count_in; // finalize+decode: received counts
  const uint32_t* masks;   // [N][L/32]
  void* out;               // result vector
  uint8_t* count_out;      // may be null
  float* mean_out;         // fused bf16 in blocks of 2^16, blocks that several workgroups share: the means on their way to the decode
  unsigned long long* total_out;   // may be null: receives the number of (worker, entry) arrivals (Sec. 3.4 loss monitoring)
  u64 n;                   // valid entries of the input (encode) / output (decode)
  u64 n_pad;               // padded length = vector length on the encoded side; shard_len for reduce/fused
  u64 seed;
  u64 base;                // index of entry 0 in the sign stream
  u64 unit0;               // encode / decode: number of leading tiles that need no bounds checks; fused bf16 in blocks of 2^16: of leading blocks that one workgroup serves each
  int N;                   // workers
  int k;                   // block_log2
  float scale;             // 2^(-k/2) rounded to fp32
};

// In the shard kernels a tile can be cut short only when blocks are smaller than a tile (class 0).
template <int K> constexpr bool kShardTilesFull = (K != 0);

template <int K>
__device__ __forceinline__ int tile_bits(int k) { return K ? Geo<K>::KT : k; }

// Class 0 (tiles of 1024 entries for all blocks up to 2^10): the work of a whole tile compiled for each block size, so that its stages are one run
// of code; a branch ahead of every stage kept the compiler from putting one stage's instructions between another's.  us, branches -> this: bf16
// fused path of 2^10, N = 8 / 24, 3145728 entries 23.9 -> 19.2 / 59.8 -> 46.5, 1 M 13.6 -> 12.8 / 27.9 -> 25.8, 65536 5.95 -> 5.66 / 10.7 -> 9.7, of 2^8, N =
// 8, 16.8 M 91.8 -> 75.7;  fp32, 2^9, N = 1 / 3, 3145728 entries 7.0 -> 6.3 / 12.7 -> 10.9;  encode, decode of 2^10, 65536 entries 2.67 -> 2.58, 2.81 -> 2.66,
// bf16 encode, 16.8 M 16.6 -> 14.3;  bf16 reduce + decode 0 .. -3 %.  (Not the fp32 forms that add up whole workers first, rht_fused.hpp: they lose registers.)
// FIRST = 10: comparisons one after the other, each behind the code of the size before it, for the short kernels of encode and decode; else a switch, where
// that code is long and a small size would miss in the instruction cache at every comparison.  us, comparisons -> switch, bf16 fused path, N = 8 / 24, 2^6, 1 M entries
// 12.2 -> 12.0 / 24.9 -> 24.6, 2^8, 65536 entries 5.73 -> 5.68 / 9.52 -> 9.35, 2^10, 1 M 12.8 -> 12.5 / 26.0 -> 25.9;  with totals, N = 8, eight buckets of 131072 entries, 2^6
// 16.7 -> 16.4 (without sizes 16.2), 2^9 16.6 -> 16.9;  but fp32 encode / decode of 65536 entries, 2^10 2.56 -> 2.62 / 2.66 -> 2.68, 2^8 2.48 -> 2.52 / 2.58 -> 2.62.
template <int K, int FIRST = 0, int LAST = 10, class Tile>
__device__ __forceinline__ void with_block_size(const PathArgs& a, Tile&& tile) {
  if constexpr (K == 0) {
    PathArgs known = a;
    if constexpr (FIRST > 5) {
      if (a.k == FIRST) { known.k = FIRST; return tile(known); }
      with_block_size<K, FIRST - 1>(a, (Tile&&)tile);
    } else if constexpr (FIRST == 5) {
      known.k = 5;
      tile(known);
    } else {
      switch (a.k) {
        case 5: known.k = 5; return tile(known);
        case 6: known.k = 6; return tile(known);
        case 7: known.k = 7; return tile(known);
        case 8: known.k = 8; return tile(known);
        case 9: known.k = 9; return tile(known);
        default: known.k = LAST; return tile(known);
      }
    }
  } else {
    tile(a);
  }
}

// ---- blocks above 2^14: one workgroup per block in encode / decode ----------------------------------
// H_{2^k} = H_{2^(k-14)} (x) H_{2^14}: a workgroup holds the block's PARTS tiles in registers (PARTS*R per
// lane), runs the small factor as add/sub between the tiles and the big one tile by tile.  Every input is
// read once and gets its sign once; one Philox evaluation per wavefront covers its part of all the tiles.

// Sign bits of this wavefront's registers in all PARTS tiles of a block, as two vector registers: lane
// q*16 + r holds the 64-bit lane mask of register r of tile q (lo, hi).  `g` = index, in the padded
// vector, of this wavefront's first entry in tile 0 of the block.
template <int K>
__device__ __forceinline__ void block_sign_words(u64 seed, u64 g, uint32_t& lo, uint32_t& hi) {
  static_assert(Geo<K>::R == 16 && Geo<K>::PARTS <= 4, "lane q*16 + r");
  const int l = lane_id(), q = l >> 4, r = l & 15;
  const u64 ctr = ((g + (u64)q * Geo<K>::T) >> 7) + (u64)(r >> 1);   // a counter covers two registers
  const u32x4 w = philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u, (uint32_t)seed, (uint32_t)(seed >> 32));
  lo = (r & 1) ? w.c : w.a;
  hi = (r & 1) ? w.d : w.b;
}
template <int NR>
__device__ __forceinline__ void apply_block_signs(float (&v)[NR], uint32_t lo, uint32_t hi, int q) {
  asm volatile("" : "+v"(lo), "+v"(hi));   // the lane masks of a tile are formed where the tile is used
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const u64 m = (u64)(uint32_t)__builtin_amdgcn_readlane((int)lo, q * 16 + r) |
                  ((u64)(uint32_t)__builtin_amdgcn_readlane((int)hi, q * 16 + r) << 32);
    v[r] = in_mask(m) ? -v[r] : v[r];
  }
  __builtin_amdgcn_sched_barrier(0);
}
// the factor H_{PARTS} across the tiles, in place
template <int PARTS, int NR>
__device__ __forceinline__ void across_tiles(float (&v)[PARTS][NR]) {
#pragma unroll
  for (int s = 1; s < PARTS; s <<= 1)
#pragma unroll
    for (int q = 0; q < PARTS; ++q)
      if ((q & s) == 0) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const float x = v[q][r], y = v[q + s][r];
          v[q][r] = x + y;
          v[q + s][r] = x - y;
        }
      }
}

// Encode and decode store past the caches: their results are not read again here, and their inputs stay.  us, plain -> nontemporal stores,
// fp32 decode of 2^12, 3145728 / 5242880 / 44040192 / 67108864 entries 7.7 -> 5.8 / 9.9 -> 7.5 / 62.8 -> 59.5 / 92.8 -> 90.0, bf16 6.0 -> 5.4 / 8.3 -> 7.1 /
// 33.5 -> 32.3 / 70.2 -> 65.3;  fp32 encode of 2^10 6.5 -> 5.0 / 8.7 -> 7.7 / 59.9 -> 58.6 / 89.6 -> 87.9.
// Part of that is lost again by who reads the results next; call and reader (p += out) together, fp32 encode / decode of 2^12, 2 sets of buffers
// in turn, 4194304 entries 15.1 -> 14.1 / 16.0 -> 14.5, 44040192 150 -> 135 / 151 -> 139.  Hence not where fp32 in- and output are larger than the L2 and both
// fit the last-level cache (256 MB): together, 7340032 / 10485760 entries 24.6 -> 26.0 / 33.6 -> 35.7 and 24.7 -> 26.1 / 34.5 -> 36.0 (by themselves 11.1 -> 10.4 /
// 15.8 -> 15.4 and 11.5 -> 10.3 / 16.5 -> 15.4, of 16 sets 12.0 -> 12.4 / 16.9 -> 17.0 and 12.1 -> 12.5 / 17.4 -> 17.4);  by themselves, 11534336 / 17825792
// entries, decode 17.5 -> 17.8 / 25.0 -> 26.2, encode 16.8 -> 17.2 / 25.2 -> 26.1;  towards its end the cards differ: 25493504 entries, decode 36.5 -> 35.4 on some,
// 36.6 -> 38.8 on another, encode of 26 M 37.9 -> 36.9 and 40.3 -> 41.5.
// 2^13 gains up to 6 M: together, 6291456 / 7340032 entries 21.8 -> 22.0 / 24.7 -> 26.3 and 22.7 -> 21.6 / 25.6 -> 27.0.  Blocks of 2^14, one a workgroup of 16 waves,
// gain for longer: encode, 12582912 / 17825792 / 20971520 / 23068672 entries 20.2 -> 18.6 / 26.2 -> 26.2 / 31.4 -> 30.6 / 32.5 -> 33.6, together 41.4 -> 42.2 / 60.3 -> 62.2
// (12 and 18 M).  bf16 results: by themselves, decode of 2^12, 12 / 20 / 30 M 15.4 -> 14.7 / 23.5 -> 22.1 / 33.3 -> 32.1, together 26.9 -> 27.4 / 40.9 -> 42.2 / 58.4
// -> 60.2: left past the caches.
template <int K> constexpr u64 kKeepFrom = K == 14 ? 16u << 20 : K == 13 ? 13u << 19 : 6u << 20;
constexpr u64 kKeepTo = 32u << 20;
// Few entries, where nothing is gained: together with the reader, decode of 2^12 / 2^13, 219933 entries 5.28 -> 5.44 / 5.89 -> 6.12, but 1048576 8.4 -> 8.2 / 8.9 -> 8.6
// (2^10: no difference).
template <int K> constexpr u64 kKeepFew = K == 0 ? 0 : 3u << 18;
template <int K> constexpr bool keeps_results(u64 n_pad) { return n_pad <= kKeepFew<K> || (n_pad > kKeepFrom<K> && n_pad <= kKeepTo); }
// Decode from sums and counts, one bucket or all buckets of a launch together: by itself, 2^8 / 2^12, 6144000 entries 12.3 -> 12.5 / 11.7 -> 12.4, 9830400 17.4 -> 18.0 /
// 17.5 -> 18.5, 14745600 23.6 -> 25.0 / 23.8 -> 25.4, 18022400 28.6 -> 29.9 / 29.4 -> 30.1, but 4096000 9.4 -> 9.4 / 9.4 -> 8.2, 21299200 36.6 -> 34.6 / 35.6 -> 34.6, 24576000
// 42.1 -> 39.3 / 41.9 -> 39.2;  2^14, 12288000 / 18874368 23.3 -> 21.8 / 32.7 -> 31.8.
template <int K> constexpr bool keeps_finalized(u64 entries) {
  return entries <= kKeepFew<K> || (K < 14 && entries > 11u << 19 && entries <= 19u << 20);
}

// Sec. 3.3 encode: out = B^(-1/2) H D x, blockwise; pad of the last block is zero.
// FULL: every access of the tile lies inside the vectors (no bounds checks).  The first a.unit0 tiles of a launch are
// such tiles, the ragged end takes the checked form, in the same launch: as a launch of its own it cost 2.5 us of host
// time and a gap on the GPU (25.6 M fp32 entries, 6240 tiles: 40.2 -> 37.5 us; one 4096-entry block: 6.0 -> 3.5 us).
template <int K, class In, class Wire, bool FULL>
__device__ __forceinline__ void encode_tile(const PathArgs& a, u64 unit, float* xbuf) {
  constexpr int T = Geo<K>::T, R = Geo<K>::R;
  const int wave = wave_id(), lane = lane_id(), kt = tile_bits<K>(a.k);
  float v[R];
  load_tile<K, false, FULL, true>((const In*)a.in, unit * T, a.n, wave, lane, v);
  u64 sg[R];
  sign_masks(a.seed, a.base + unit * T + (u64)wave * Geo<K>::WAVE_ENTRIES, sg);
  apply_signs(v, sg);
  transform<K, true>(v, xbuf, wave, lane, kt);
  const float c = a.scale * lane_sigma(lane, kt < 6 ? kt : 6);
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] *= c;
  if (sizeof(Wire) == 4 && keeps_results<K>(a.n_pad)) {   // one kernel for both: encode of 2^14, 487689 entries 5.06, a kernel each 5.18
    keep_apart();
    store_tile<K, true, FULL, false>((Wire*)a.out, unit * T, a.n_pad, wave, lane, v);
    keep_apart();
  } else {
    store_tile<K, true, FULL, true>((Wire*)a.out, unit * T, a.n_pad, wave, lane, v);
  }
}
template <int K, class In, class Wire>
__global__ __launch_bounds__(Geo<K>::THREADS) void k_encode(PathArgs a) {
  static_assert(Geo<K>::PARTS == 1, "larger blocks use k_encode_block");
  __shared__ float xbuf[Geo<K>::Q > 0 ? Geo<K>::T : 1];
  if (blockIdx.x < a.unit0) with_block_size<K, 10>(a, [&](const PathArgs& b) __attribute__((always_inline)) { encode_tile<K, In, Wire, true>(b, blockIdx.x, xbuf); });
  else encode_tile<K, In, Wire, false>(a, blockIdx.x, xbuf);
}

// Blocks above 2^14 load nontemporally too from kStreamFrom entries on: fp32 decode of 2^16, plain loads and stores -> nontemporal stores ->
// both, 4194304 / 25493504 / 209715200 entries 18.0 -> 16.1 -> 17.6 / 54 -> 45 -> 43 / 361 -> 351 -> 335, of 2^15 11.2 -> 9.8 -> 10.7 / 56 -> 49 ->
// 47 / 336 -> 347 -> 336.
constexpr u64 kStreamFrom = 8u << 20;

// The same for blocks above 2^14: workgroup x encodes block x (a.unit0 counts tiles).  FULL = false: the block is cut
// short by the end of the input (its pad reads as zero); the output always holds whole blocks.
template <int K, class In, class Wire, bool FULL>
__device__ __forceinline__ void encode_block(const PathArgs& a, float (*xbuf)[Geo<K>::T]) {
  constexpr int T = Geo<K>::T, R = Geo<K>::R, HB = Geo<K>::HB, PARTS = Geo<K>::PARTS;
  const int wave = wave_id(), lane = lane_id(), kt = Geo<K>::KT;
  const u64 tile0 = (u64)blockIdx.x << HB;
  float v[PARTS][R];
  if (a.n_pad > kStreamFrom) {
#pragma unroll
    for (int q = 0; q < PARTS; ++q) load_tile<K, false, FULL, true>((const In*)a.in, (tile0 + q) * T, a.n, wave, lane, v[q]);
  } else {
    keep_apart();
#pragma unroll
    for (int q = 0; q < PARTS; ++q) load_tile<K, false, FULL, false>((const In*)a.in, (tile0 + q) * T, a.n, wave, lane, v[q]);
    keep_apart();
  }
  uint32_t slo, shi;
  block_sign_words<K>(a.seed, a.base + tile0 * T + (u64)wave * Geo<K>::WAVE_ENTRIES, slo, shi);
#pragma unroll
  for (int q = 0; q < PARTS; ++q) apply_block_signs(v[q], slo, shi, q);
  across_tiles<PARTS, R>(v);
  const float c = a.scale * lane_sigma(lane, 6);
#pragma unroll
  for (int p = 0; p < PARTS; ++p) {
    transform<K, true, false>(v[p], xbuf[p & 1], wave, lane, kt);
#pragma unroll
    for (int r = 0; r < R; ++r) v[p][r] *= c;
    store_tile<K, true, true, true>((Wire*)a.out, (tile0 + p) * T, a.n_pad, wave, lane, v[p]);
  }
}
template <int K, class In, class Wire>
__global__ __launch_bounds__(Geo<K>::THREADS) void k_encode_block(PathArgs a) {
  static_assert(Geo<K>::PARTS > 1, "blocks above 2^14");
  __shared__ float xbuf[2][Geo<K>::T];   // the registers allow one workgroup per CU anyway: alternate, one barrier per exchange
  if ((u64)blockIdx.x << Geo<K>::HB < a.unit0) encode_block<K, In, Wire, true>(a, xbuf);
  else encode_block<K, In, Wire, false>(a, xbuf);
}

// Mean tile (layout B) for decode: either the mean itself, or sum / count with 0 where count is 0
// (the "averages" of Sec. 3.1.1 taken over the entries that arrived).  MASKED: second-stage loss
// (the broadcast of the aggregated shard, Sec. 3.1.1): entries whose bit in a.masks is clear never
// arrived and count as zero.
template <int K, bool FINALIZE, bool FULL, bool MASKED, bool NT>
__device__ __forceinline__ void load_mean_tile(const PathArgs& a, u64 tile, int wave, int lane,
                                               float (&v)[Geo<K>::R]) {
  constexpr int T = Geo<K>::T, R = Geo<K>::R;
  load_tile<K, true, FULL, NT>((const float*)a.in, tile * T, a.n_pad, wave, lane, v);
  if constexpr (FINALIZE) {
    float c[R];
    load_tile<K, true, FULL, NT>(a.count_in, tile * T, a.n_pad, wave, lane, c);
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = c[r] > 0.0f ? v[r] * __builtin_amdgcn_rcpf(c[r]) : 0.0f;   // as finalize_mean
  }
  if constexpr (MASKED) {
    const uint32_t w = load_mask_words<K, FULL>(a.masks, tile * T, a.n_pad, mask_word_offset<K>(wave, lane));
    if (!all_arrived(w)) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = in_mask(mask_of_reg(w, r)) ? v[r] : 0.0f;
    }
  }
}

// Sec. 3.3 / Sec. 4 decode: out = D B^(-1/2) H mean, first n entries kept.  FULL as in encode_tile.
template <int K, class Out, bool FINALIZE, bool FULL, bool MASKED, bool KEEP>
__device__ __forceinline__ void decode_tile(const PathArgs& a, u64 unit, float* xbuf) {
  constexpr int T = Geo<K>::T, R = Geo<K>::R;
  static_assert(Geo<K>::PARTS == 1, "larger blocks use k_decode_block");
  const int wave = wave_id(), lane = lane_id(), kt = tile_bits<K>(a.k);
  float v[R];
  load_mean_tile<K, FINALIZE, FULL, MASKED, true>(a, unit, wave, lane, v);
  transform<K, false>(v, xbuf, wave, lane, kt);
  const float c = a.scale * lane_sigma(lane, kt < 6 ? kt : 6);
  u64 sg[R];
  sign_masks(a.seed, a.base + unit * T + (u64)wave * Geo<K>::WAVE_ENTRIES, sg);
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] *= c;
  apply_signs(v, sg);
  store_tile<K, false, FULL, !KEEP>((Out*)a.out, unit * T, a.n, wave, lane, v);
}
// KEEP is chosen on the host: a kernel for both takes longer, 2^13, 65536 entries 3.83, a kernel each 3.79
template <int K, class Out, bool FINALIZE, bool MASKED, bool KEEP>
__global__ __launch_bounds__(Geo<K>::THREADS) void k_decode(PathArgs a) {
  __shared__ float xbuf[Geo<K>::Q > 0 ? Geo<K>::T : 1];
  if (blockIdx.x < a.unit0) with_block_size<K, 10>(a, [&](const PathArgs& b) __attribute__((always_inline)) { decode_tile<K, Out, FINALIZE, true, MASKED, KEEP>(b, blockIdx.x, xbuf); });
  else decode_tile<K, Out, FINALIZE, false, MASKED, KEEP>(a, blockIdx.x, xbuf);
}

// The same for blocks above 2^14 (see k_encode_block).  The input holds whole blocks; FULL = false: the
// output is cut short inside this block.
template <int K, class Out, bool FINALIZE, bool FULL, bool MASKED, bool STREAM>
__device__ __forceinline__ void decode_block(const PathArgs& a, u64 blk, float (*xbuf)[Geo<K>::T]) {
  constexpr int T = Geo<K>::T, R = Geo<K>::R, HB = Geo<K>::HB, PARTS = Geo<K>::PARTS;
  const int wave = wave_id(), lane = lane_id(), kt = Geo<K>::KT;
  const u64 tile0 = blk << HB;
  float v[PARTS][R];
#pragma unroll
  for (int q = 0; q < PARTS; ++q) load_mean_tile<K, FINALIZE, true, MASKED, STREAM>(a, tile0 + q, wave, lane, v[q]);
  uint32_t slo, shi;
  block_sign_words<K>(a.seed, a.base + tile0 * T + (u64)wave * Geo<K>::WAVE_ENTRIES, slo, shi);
  across_tiles<PARTS, R>(v);
  const float c = a.scale * lane_sigma(lane, 6);
#pragma unroll
  for (int p = 0; p < PARTS; ++p) {
    transform<K, false, false>(v[p], xbuf[p & 1], wave, lane, kt);
#pragma unroll
    for (int r = 0; r < R; ++r) v[p][r] *= c;
    apply_block_signs(v[p], slo, shi, p);
    store_tile<K, false, FULL, true>((Out*)a.out, (tile0 + p) * T, a.n, wave, lane, v[p]);
  }
}
// STREAM is chosen on the host: a kernel for both takes longer, 2^15, one block with sums and counts 9.30, a kernel each 9.16, reduce + decode of 16 blocks of
// three workers 14.3, 14.0
template <int K, class Out, bool FINALIZE, bool MASKED, bool STREAM>
__global__ __launch_bounds__(Geo<K>::THREADS) void k_decode_block(PathArgs a) {
  static_assert(Geo<K>::PARTS > 1, "blocks above 2^14");
  __shared__ float xbuf[2][Geo<K>::T];
  if ((u64)blockIdx.x << Geo<K>::HB < a.unit0) decode_block<K, Out, FINALIZE, true, MASKED, STREAM>(a, blockIdx.x, xbuf);
  else decode_block<K, Out, FINALIZE, false, MASKED, STREAM>(a, blockIdx.x, xbuf);
}

// acc += value where the worker's copy arrived.  Arrivals are counted as `full` (workers whose whole
// tile part arrived) plus a per-register byte in cntp (four registers per word; N <= 255 keeps a byte
// from overflowing).  `words` holds the worker's received bits as loaded by load_mask_words.
template <int NR>
__device__ __forceinline__ void masked_accumulate(const float (&v)[NR], uint32_t words, float (&acc)[NR],
                                                  uint32_t (&cntp)[NR / 4], int& full) {
  if (all_arrived(words)) {
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] += v[r];
    ++full;
  } else {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const bool got = in_mask(mask_of_reg(words, r));
      acc[r] += got ? v[r] : 0.0f;
      cntp[r >> 2] += got ? (1u << (8 * (r & 3))) : 0u;
    }
  }
}

template <int NR>
__device__ __forceinline__ int count_of(const uint32_t (&cntp)[NR / 4], int full, int r) {
  return (int)((cntp[r >> 2] >> (8 * (r & 3))) & 0xFFu) + full;
}

// Sec. 3.4 loss monitoring.  A bucket's arrivals are N times its length less what is missing: whoever serves its start adds the
// former, and only those whose part misses something take that off (one thread of a workgroup or a wavefront calls this).  Atomics
// on one 128-byte line, i.e. on the totals of 16 buckets, are served every 4 to 14 ns, which small tiles that all add their arrivals
// wait for.  Batched call with totals, 200 MiB of two workers, 1 % loss in packets of 256, us, every tile's arrivals -> that:
// bf16 2^11 176 -> 75, 2^12 116 -> 79, 2^14 99 -> 98; fp32 2^11 110 -> 64, 2^12 82 -> 65; 32 MiB: bf16 2^11 60 -> 18, 2^12 36 -> 19,
// fp32 2^12 25 -> 17; sixteen workers, where most tiles miss something: 200 MiB, bf16 2^11 57 -> 57, fp32 2^11 50 -> 48.
__device__ __forceinline__ void add_total(const PathArgs& a, bool start, uint32_t missing) {
  const unsigned long long n = (start ? (unsigned long long)a.N * a.n_pad : 0ull) - missing;   // (modulo 2^64, like the sum)
  if (n) atomicAdd(a.total_out, n);
}
// what is missing from a wavefront's `inside` entries: its `full` workers count for all of them, the rest sit in the packed bytes
template <int NR>
__device__ __forceinline__ uint32_t missing_of(const uint32_t (&cntp)[NR / 4], int full, int N, int inside) {
  if (full == N) return 0;
  uint32_t n = 0;
#pragma unroll
  for (int r = 0; r < NR / 4; ++r) n = __builtin_amdgcn_sad_u8(cntp[r], 0u, n);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o, 64);
  return (uint32_t)(N - full) * (uint32_t)inside - n;
}

template <int K, bool FULL>
__device__ __forceinline__ void store_counts(uint8_t* count_out, u64 e0, u64 limit, int wave, int lane,
                                             const uint32_t (&cntp)[Geo<K>::R / 4], int full) {
  constexpr int R = Geo<K>::R;
  if (!count_out) return;
  float c[R];
#pragma unroll
  for (int r = 0; r < R; ++r) c[r] = (float)count_of<R>(cntp, full, r);
  store_tile<K, true, FULL, true>(count_out, e0, limit, wave, lane, c);
  __builtin_amdgcn_sched_barrier(0);
}

// The counts of a path call may lie at any address: the wide stores below are for those aligned to them, else bytes.
// `aligned`: the same on every lane (it is a property of the call's pointer).
__device__ __forceinline__ void store_counts4(uint32_t c, __amdgpu_buffer_rsrc_t rs, int off, int tile_off, bool aligned) {
  if (aligned) {
    __builtin_amdgcn_raw_buffer_store_b32(c, rs, off, tile_off, kBufNt);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(c >> (8 * j)), rs, off + j, tile_off, kBufNt);
  }
}

// mean over what arrived (0 where nothing arrived), times `post`.  The reciprocal of the count comes
// from v_rcp_f32 (1 ulp), far inside the 1e-6 budget of the path.
template <int NR>
__device__ __forceinline__ void finalize_mean(float (&acc)[NR], const uint32_t (&cntp)[NR / 4], int full, float post) {
  uint32_t any = 0;
#pragma unroll
  for (int r = 0; r < NR / 4; ++r) any |= cntp[r];
  if (__builtin_amdgcn_ballot_w64(any != 0) == 0 && full > 0) {
    const float f = post * __builtin_amdgcn_rcpf((float)full);   // every entry arrived `full` times
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] *= f;
  } else {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int c = count_of<NR>(cntp, full, r);
      acc[r] = c ? acc[r] * (post * __builtin_amdgcn_rcpf((float)c)) : 0.0f;
    }
  }
}

// Aggregation of N encoded shards (Sec. 3.1.1), mean over what arrived, decode (Sec. 3.3).  K <= 14.
// The next worker's tile is in flight while the current one is accumulated.
template <int K, class Wire, class Out>
__device__ __forceinline__ void reduce_decode_tile(const PathArgs& a, u64 unit) {
  constexpr int T = Geo<K>::T, R = Geo<K>::R;
  constexpr bool FULL = kShardTilesFull<K>;
  static_assert(Geo<K>::PARTS == 1, "blocks above 2^14: k_reduce_decode_block, or sum and count in memory");
  __shared__ float xbuf[Geo<K>::Q > 0 ? T : 1];
  const int wave = wave_id(), lane = lane_id(), kt = tile_bits<K>(a.k);
  const u64 L = a.n_pad, e0 = unit * T;
  const Wire* shards = (const Wire*)a.in;
  float acc[R], va[R], vb[R];
  uint32_t ma, mb = 0, cnt[R / 4];
  int full = 0;
  const int moff = mask_word_offset<K>(wave, lane);
  const u64 mrow = L >> 5;
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int r = 0; r < R / 4; ++r) cnt[r] = 0;
  load_tile<K, true, FULL, true>(shards, e0, L, wave, lane, va);
  ma = load_mask_words<K, FULL>(a.masks, e0, L, moff);
  for (int i = 0; i < a.N; i += 2) {
    if (i + 1 < a.N) {
      load_tile<K, true, FULL, true>(shards + (u64)(i + 1) * L, e0, L, wave, lane, vb);
      mb = load_mask_words<K, FULL>(a.masks + (u64)(i + 1) * mrow, e0, L, moff);
    }
    masked_accumulate(va, ma, acc, cnt, full);
    if (i + 1 < a.N) {
      if (i + 2 < a.N) {
        load_tile<K, true, FULL, true>(shards + (u64)(i + 2) * L, e0, L, wave, lane, va);
        ma = load_mask_words<K, FULL>(a.masks + (u64)(i + 2) * mrow, e0, L, moff);
      }
      masked_accumulate(vb, mb, acc, cnt, full);
    }
  }
  store_counts<K, FULL>(a.count_out, e0, L, wave, lane, cnt, full);
  if (a.total_out) {
    const int inside = FULL || L - e0 >= T ? 64 * R : (int)(L - e0);   // tiles of several wavefronts are not cut short
    const uint32_t missing = missing_of<R>(cnt, full, a.N, inside);
    if (lane == 0) add_total(a, e0 == 0 && wave == 0, missing);
  }
  finalize_mean(acc, cnt, full, 1.0f);
  transform<K, false>(acc, xbuf, wave, lane, kt);
  const float c = a.scale * lane_sigma(lane, kt < 6 ? kt : 6);
  u64 sg[R];
  sign_masks(a.seed, a.base + e0 + (u64)wave * Geo<K>::WAVE_ENTRIES, sg);
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] *= c;
  apply_signs(acc, sg);
  store_tile<K, false, FULL, true>((Out*)a.out, e0, L, wave, lane, acc);
}
template <int K, class Wire, class Out>
__global__ __launch_bounds__(Geo<K>::THREADS) void k_reduce_decode(PathArgs a) {
  // fp32 by itself: for any size.  us, that -> compiled for each, 2^10, N = 12 / 24 / 32, 901120 entries 11.0 -> 11.5 / 17.8 -> 19.4 / 22.1 -> 24.6, 1 M 11.9 -> 12.2 / 19.6 -> 21.0
  // / 24.3 -> 26.7, but N = 2, 65536 entries 3.54 -> 3.51, N = 4, 1.2 M 7.3 -> 7.2.  (bf16 and buckets: no such loss.)
  if constexpr (sizeof(Wire) == 4) reduce_decode_tile<K, Wire, Out>(a, blockIdx.x);
  else with_block_size<K>(a, [&](const PathArgs& b) __attribute__((always_inline)) { reduce_decode_tile<K, Wire, Out>(b, blockIdx.x); });
}

// Several buckets of one launch shape class (same N, block size and type) in ONE launch: small buckets
// (a 25 MiB DDP bucket is only ~100 tiles per shard) cannot fill 256 CUs on their own.  Descriptors ride
// in the kernel arguments; workgroup x serves tile x - tile_start[j] of bucket j.
constexpr int kMaxBatch = 64;   // 64 descriptors keep BatchArgs under the 4 KB of kernel arguments
struct BucketArgs {
  const void* in;          // raw slices / encoded shards; finalize+decode: the fp32 sums
  const void* aux;         // received masks [N][L/32]; finalize+decode: the uint8 counts
  void* out;
  uint8_t* count_out;
  u64 shard_len, seed, base;
};
struct BatchArgs {
  int n, N, k;
  float scale;
  unsigned long long* totals;   // may be null: totals[first + j] receives bucket j's number of arrivals (add_total)
  int first;
  uint32_t tile_start[kMaxBatch + 1];
  BucketArgs b[kMaxBatch];
};

static_assert(sizeof(BatchArgs) <= 4096, "kernel arguments are limited to 4 KB");

// bucket j of the launch as the arguments of a single-bucket call
__device__ __forceinline__ void bucket_args(const BatchArgs& ba, PathArgs& a, int j) {
  a = PathArgs{};
  a.in = ba.b[j].in; a.masks = (const uint32_t*)ba.b[j].aux; a.count_in = (const uint8_t*)ba.b[j].aux;
  a.out = ba.b[j].out; a.count_out = ba.b[j].count_out;
  a.n = a.n_pad = ba.b[j].shard_len; a.seed = ba.b[j].seed; a.base = ba.b[j].base;
  a.N = ba.N; a.k = ba.k; a.scale = ba.scale;
  a.total_out = ba.totals ? ba.totals + ba.first + j : nullptr;
}
// the bucket that unit x of the launch lies in
template <bool WALK = false>
__device__ __forceinline__ int bucket_index(const BatchArgs& ba, uint32_t x) {
  // buckets that end at or before tile x: one comparison a lane (a walk over the descriptors was up to 60 dependent
  // scalar loads ahead of a workgroup's first access).  us, walk -> that, 64 buckets: finalize + decode 2^14 19.2 -> 14.7, reduce +
  // decode bf16 2^11 26.2 -> 17.8; but reduce + decode fp32 with its data in the cache 2^14 37.5 -> 42.6, 2^10 16 buckets 14.5 ->
  // 17.1 (in memory: the same), which therefore walks
  int j = 0;
  if constexpr (WALK) {
    while (j + 1 < ba.n && ba.tile_start[j + 1] <= x) ++j;
  } else {
    const int lane = lane_id();
    j = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane + 1 < ba.n && ba.tile_start[lane + 1] <= x));
  }
  return j;
}
// its arguments; returns the tile inside it
template <bool WALK = false>
__device__ __forceinline__ u64 bucket_of(const BatchArgs& ba, PathArgs& a, uint32_t x) {
  const int j = bucket_index<WALK>(ba, x);
  bucket_args(ba, a, j);
  return x - ba.tile_start[j];
}

// The three-call path on several buckets: aggregation + mean + decode of encoded shards, and mean + decode of
// (sum, count) pairs; every bucket holds whole blocks.
template <int K, class Wire>
__global__ __launch_bounds__(Geo<K>::THREADS) void k_reduce_decode_batched(BatchArgs ba) {
  PathArgs a;
  const u64 unit = bucket_of<sizeof(Wire) == 4>(ba, a, blockIdx.x);
  with_block_size<K>(a, [&](const PathArgs& b) __attribute__((always_inline)) { reduce_decode_tile<K, Wire, Wire>(b, unit); });
}
template <int K, class Out, bool KEEP>
__global__ __launch_bounds__(Geo<K>::THREADS) void k_finalize_decode_batched(BatchArgs ba) {
  PathArgs a;
  const u64 unit = bucket_of(ba, a, blockIdx.x);
  __shared__ float xbuf[Geo<K>::Q > 0 ? Geo<K>::T : 1];
  with_block_size<K, 10>(a, [&](const PathArgs& b) __attribute__((always_inline)) { decode_tile<K, Out, true, kShardTilesFull<K>, false, KEEP>(b, unit, xbuf); });
}

}  // namespace ordev

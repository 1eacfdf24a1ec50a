// One block-size class of kernels (compile with -DOR_K=0, 11, 12, ... 16).
#include "launch_table.hpp"
#include "rht_fused.hpp"
#include "rht_fused_each.hpp"
#if OR_K >= 11 && OR_K <= 15
#include "rht_fused_bf16.hpp"
#if OR_K <= 14
#include "rht_encode_bf16.hpp"
#endif
#endif
#if OR_K > 14
#include "rht_encode_block.hpp"
#include "rht_fused_f32_block.hpp"
#if OR_K == 16
#include "rht_fused_bf16_64k.hpp"
#endif
#include "rht_reduce_block.hpp"
#endif

#ifndef OR_K
#error "compile with -DOR_K=<class>"
#endif

namespace orhost {
using namespace ordev;

namespace {
constexpr int K = OR_K;
typedef Geo<K> G;

#define OR_LAUNCHER_T(name, kernel, threads)                                                 \
  /* serves output tiles 0 .. units - 1, one workgroup per tile */                           \
  hipError_t name(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {    \
    if (units == 0) return hipSuccess;                                                       \
    if (units > 0x7FFFFFFFull) return hipErrorInvalidValue;                                  \
    return launch_kernel(kernel, dim3((unsigned)units), dim3(threads), s, pos, a);           \
  }
#define OR_LAUNCHER(name, kernel) OR_LAUNCHER_T(name, kernel, G::THREADS)

// blocks above 2^14: one workgroup per block of G::PARTS tiles; a.unit0 and units count tiles
#define OR_BLOCK_LAUNCHER(name, kernel)                                                      \
  hipError_t name(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {    \
    const unsigned long long blocks = units >> G::HB;                                        \
    if (blocks == 0) return hipSuccess;                                                      \
    if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;                                 \
    return launch_kernel(kernel, dim3((unsigned)blocks), dim3(G::THREADS), s, pos, a);       \
  }

#if OR_K <= 14
#define OR_F32_LAUNCHER(name, Args, keep, kernel, ...)                                         \
  hipError_t name(const Args& a, unsigned long long units, hipStream_t s, int pos) {           \
    if (units == 0) return hipSuccess;                                                         \
    if (units > 0x7FFFFFFFull) return hipErrorInvalidValue;                                    \
    return launch_kernel(keep ? kernel<K, __VA_ARGS__, true> : kernel<K, __VA_ARGS__, false>, dim3((unsigned)units), dim3(G::THREADS), s, pos, a); \
  }
OR_LAUNCHER(enc_f32, (k_encode<K, float, float>))
OR_F32_LAUNCHER(dec_f32, PathArgs, keeps_results<K>(a.n_pad), k_decode, float, false, false)
OR_F32_LAUNCHER(fdec_f32, PathArgs, keeps_finalized<K>(a.n_pad), k_decode, float, true, false)
OR_F32_LAUNCHER(mdec_f32, PathArgs, keeps_results<K>(a.n_pad), k_decode, float, false, true)
#define OR_DEC(Out, FIN, MASKED) (k_decode<K, Out, FIN, MASKED, false>)
#define OR_XFORM_LAUNCHER OR_LAUNCHER
#else
#define OR_DEC(Out, FIN, MASKED) (a.n_pad > kStreamFrom ? k_decode_block<K, Out, FIN, MASKED, true> : k_decode_block<K, Out, FIN, MASKED, false>)
#define OR_XFORM_LAUNCHER OR_BLOCK_LAUNCHER
OR_BLOCK_LAUNCHER(enc_f32, (k_encode_block<K, float, float>))
OR_BLOCK_LAUNCHER(dec_f32, OR_DEC(float, false, false))
OR_BLOCK_LAUNCHER(fdec_f32, OR_DEC(float, true, false))
OR_BLOCK_LAUNCHER(mdec_f32, OR_DEC(float, false, true))
#endif
#if OR_K == 0
OR_LAUNCHER(enc_bf16, (k_encode<K, bf16_t, bf16_t>))
#elif OR_K <= 14
OR_LAUNCHER_T(enc_bf16, k_encode_bf16<K>, MTile<K>::THREADS)
#else
// Few blocks: a workgroup for each of the 2^14 values of a block, which all read the whole of it (the same bits).  Two of them fill a CU, and
// beyond that they only read more.  us, a workgroup a block -> that: 2^15, 128 / 256 / 300 blocks 7.3 -> 5.4 / 8.1 -> 7.3 / 11.0 -> 12;  2^16,
// 65 / 128 blocks 12.5 -> 8.7 / 13 -> 10.3, with two workgroups a block 9.7 / 11.0, 200 blocks with two of them 13.9 -> 19.
// (In place a workgroup has to have read the whole block before anyone writes to it.)
constexpr unsigned long long kEncodeSplit = K == 15 ? 256 : 128;
template <int SPLIT>
hipError_t enc_bf16_split(const PathArgs& a, unsigned long long blocks, hipStream_t s, int pos) {
  const unsigned long long grid = SPLIT == 1 ? blocks : (blocks + 7) / 8 * 8 * SPLIT;
  if (grid > 0x7FFFFFFFull) return hipErrorInvalidValue;
  return launch_kernel(k_encode_block_bf16<K, SPLIT>, dim3((unsigned)grid), dim3(EBlock<K>::THREADS), s, pos, a);
}
hipError_t enc_bf16(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {
  const unsigned long long blocks = units >> G::HB;
  if (blocks == 0) return hipSuccess;
  return blocks <= kEncodeSplit && a.in != a.out ? enc_bf16_split<EBlock<K>::P>(a, blocks, s, pos) : enc_bf16_split<1>(a, blocks, s, pos);
}
#endif
OR_XFORM_LAUNCHER(dec_bf16, OR_DEC(bf16_t, false, false))
OR_XFORM_LAUNCHER(fdec_bf16, OR_DEC(bf16_t, true, false))
OR_XFORM_LAUNCHER(mdec_bf16, OR_DEC(bf16_t, false, true))
#if OR_K <= 14
// reduce+decode of 2^13 and 2^14 blocks keeps 32 entries per lane
constexpr int KR = (K == 13 || K == 14) ? K + kWide : K;
OR_LAUNCHER_T(rdec_f32, (k_reduce_decode<KR, float, float>), Geo<KR>::THREADS)
OR_LAUNCHER_T(rdec_bf16, (k_reduce_decode<KR, bf16_t, bf16_t>), Geo<KR>::THREADS)
// several buckets per launch: `units` = tiles of all the buckets together
#define OR_BATCH_LAUNCHER(name, kernel, threads)                                             \
  hipError_t name(const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {   \
    if (units == 0) return hipSuccess;                                                       \
    if (units > 0x7FFFFFFFull) return hipErrorInvalidValue;                                  \
    return launch_kernel(kernel, dim3((unsigned)units), dim3(threads), s, pos, a);           \
  }
OR_BATCH_LAUNCHER(rdecb_f32, (k_reduce_decode_batched<KR, float>), Geo<KR>::THREADS)
OR_BATCH_LAUNCHER(rdecb_bf16, (k_reduce_decode_batched<KR, bf16_t>), Geo<KR>::THREADS)
OR_F32_LAUNCHER(fdecb_f32, BatchArgs, keeps_finalized<K>(units * G::T), k_finalize_decode_batched, float)
OR_BATCH_LAUNCHER(fdecb_bf16, (k_finalize_decode_batched<K, bf16_t, false>), G::THREADS)
// Which workers are added before they are encoded is a matter of type, block size and number of workers alone: the two ways
// round differently, and a bucket gives the same bits alone, in a batch and as part of a longer shard.
//   bf16: every worker is encoded by itself (its encoded value is rounded); above 2^10 in a kernel of its own (rht_fused_bf16.hpp).
//   fp32 2^10: the whole workers' sum first (rht_fused.hpp).  us, every worker by itself -> sum first: N = 2, 64 tiles 5.8 -> 5.2;
//     N = 8, 780 tiles 16.7 -> 10.1, 12800 tiles 86.8 -> 87.0; a loss in every copy of every tile, N = 8, 2560 tiles 26.0 -> 21.6.
//   fp32 below 2^10, where the blocks of a tile are told apart: from six workers on.  2^8: N = 2, 3120
//     blocks 6.5 -> 6.8; N = 8, 1024 blocks 12.9 -> 7.3, 10240 blocks 22.2 -> 21.7, 51200 blocks 86.6 -> 90.2; N = 32, 3120 blocks
//     52.9 -> 26.9; a loss in every copy of every tile, N = 8, 3120 blocks 17.4 -> 15.4, 51200 blocks 92.5 -> 96.1.
//   fp32 2^11: from six workers on.  N = 2, 64 tiles 4.9 -> 5.5; N = 4, 64 tiles 6.4 -> 6.7, 780 tiles 10.2 -> 9.6; N = 8, 64 tiles
//     9.5 -> 7.2, 780 tiles 16.3 -> 13.8, 12800 tiles 167 -> 171.
//   fp32 2^12 .. 2^14: every worker by itself.  2^12, N = 16: 100 tiles with 5 % loss 19.2 -> 18.2, 780 tiles 41.8 -> 43.3, 6400
//     tiles 301 -> 312; N = 64, 780 tiles 142 -> 157; 2^13, N = 8: 256 tiles 16.6 -> 20.0, 2560 tiles 133 -> 136; 2^14, N = 8: 256
//     tiles 29.4 -> 32.6, 2556 tiles 283 -> 292; a loss in every copy: 2^13, 2560 tiles 139 -> 158.  (The sum first wins where nearly
//     every copy is whole: 2^14, N = 16, 2560 tiles 481 -> 479, N = 32 926 -> 868.)
constexpr bool kMaySumFirst = K == 0 || K == 11;
[[maybe_unused]] bool sum_first_wins(int k, int N) { return k == 10 || (k <= 11 && N >= 6); }
// GROUPS while a launch leaves CUs idle and has the workers for its four groups (same bits as STREAM).  us, without -> with:
// 2^10, 256 tiles, N = 2 5.4 -> 6.7, N = 4 with a loss in every tile 7.4 -> 6.6; 2^11, N = 8, 512 tiles 10.7 -> 9.3, 781 tiles
// 11.9 -> 15.6.
[[maybe_unused]] bool groups_win(unsigned long long tiles, int N) {
  if (N < 6) return N >= 4 && tiles <= 256;
  return tiles <= 512;
}
// The second tile buffer of k_fused_each (same bits with and without) pays up to three workgroups on a CU.  (Tiles of 8 or 16
// wavefronts, at most two workgroups on a CU whatever the grid: always.  K = 0: launches that small encode workers side by side, which
// leaves the case of one worker.  It has no next one, and yet this form is the shorter chain: fp32 2^8, 64 tiles 4.07 -> 3.95.)
[[maybe_unused]] bool prefetch_wins(unsigned long long tiles) { return G::W >= 8 || tiles <= 3 * 256; }
template <bool SPLIT>   // blocks below 2^10, several to a tile
hipError_t sum_first(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if (groups_win(units, a.N))
    return launch_kernel(k_fused<K, GROUPS, SPLIT>, dim3((unsigned)units), dim3(kFusedThreads<K> * kGroups), s, pos, a);
  return launch_kernel(k_fused<K, STREAM, SPLIT>, dim3((unsigned)units), dim3(kFusedThreads<K>), s, pos, a);
}
// k_fused_each_groups: how many groups of wavefronts encode workers side by side (1: none; the same bits)?  Launches that leave CUs idle,
// where the shorter chain is worth the trip of the encoded values through LDS.  us, without -> with:
//   bf16 2^10 and below: 2^10, N = 8, 64 tiles 12.9 -> 6.0, 1024 tiles 16.8 -> 13.3, 2048 tiles 18.8 -> 24.8; N = 32, 1024 tiles 54.9 ->
//     34.2 with eight groups (sixteen: 44.6); 2^9, N = 16, 50 tiles 22.0 -> 7.5 with sixteen (eight: 8.3); N = 2, 1024 tiles 6.2 -> 6.2
//     Five to seven workers in more than 512 tiles: two rounds of four.  Eight -> four: N = 5, 600 / 1024 tiles 10.4 -> 9.1 / 12.5 -> 10.4,
//     N = 7 10.8 -> 9.7 / 13.1 -> 11.0; with totals and 5 % loss N = 5 14.1 -> 13.8 / 17.5 -> 16.9 (eight tiles a workgroup one after the
//     other 15.0 / 16.0: fewer atomics; with 1 % loss 15.8 against 12.8).
//   fp32 below 2^10 (two to five workers): N = 4, 1024 tiles 8.3 -> 6.2, 2048 tiles 10.0 -> 7.8; N = 5, 3000 tiles 12.5 -> 16.9
//   fp32 2^11 (two to five): N = 4, 64 tiles 6.3 -> 5.5, 256 tiles 6.8 -> 6.6; N = 3, 1 / 16 / 64 / 256 tiles, 5 %
//     loss 5.1 -> 4.8 / 5.5 -> 5.6 / 5.6 -> 5.8 / 5.8 -> 6.3, nothing lost 4.9 -> 4.5 / 5.1 -> 5.0 / 5.2 -> 5.2 / 5.5 -> 5.8; N = 2 5.0 -> 5.2; N = 5, 300 tiles 8.2 -> 9.4
//   fp32 2^12: N = 16, 100 tiles 19.4 -> 16.3, 200 tiles 19.5 -> 17.9; N = 32, 8 tiles 34.5 -> 26.3; N = 8, 128 tiles 11.4 -> 10.8, 256 tiles
//     11.6 -> 12.2; N = 6, 100 tiles 9.4 -> 10.1
//   fp32 2^13: N = 32, 2 tiles 41.6 -> 48.9; N = 8, 64 tiles 13.9 -> 16.6
constexpr int kEachGroups = K == 0 ? 16 : K == 11 || K == 12 ? 4 : 1;
[[maybe_unused]] int each_groups(unsigned long long tiles, int N) {
  int most = 1;
  if (K == 0) most = tiles <= 256 ? 16 : tiles <= 512 ? 8 : tiles <= 1024 ? (N <= 7 ? 4 : 8) : 1;
  if (K == 11 && (N == 3 || N == 4) && tiles <= (N == 3 ? 16 : 256)) most = 4;
  if (K == 12 && tiles <= (N >= 12 ? 200 : 128) && N >= 8) most = 4;
  int g = 1;
  while (g < most && g < N) g *= 2;
  return g;
}
// the smallest number of groups that a class launches: no kernels that nothing reaches
constexpr int kFewestGroups = K == 0 ? 2 : 4;
template <class In, int GR>
hipError_t launch_each_groups(int g, const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if (K == 0 && sizeof(In) == 4 && a.k > 9) return hipErrorInvalidValue;   // cannot happen (sum_first_wins): the kernel knows no other sizes
  if constexpr (GR > kFewestGroups) if (g < GR) return launch_each_groups<In, GR / 2>(g, a, units, s, pos);
  return launch_kernel(k_fused_each_groups<K, In, GR>, dim3((unsigned)units), dim3(G::THREADS * GR), s, pos, a);
}
template <class In, int GR>
hipError_t launch_each_groups(int g, const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if (K == 0 && sizeof(In) == 4 && a.k > 9) return hipErrorInvalidValue;   // cannot happen (sum_first_wins): the kernel knows no other sizes
  if constexpr (GR > kFewestGroups) if (g < GR) return launch_each_groups<In, GR / 2>(g, a, units, s, pos);
  return launch_kernel(k_fused_each_groups_batched<K, In, GR>, dim3((unsigned)units), dim3(G::THREADS * GR), s, pos, a);
}
template <class In>
hipError_t fused(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if (units == 0) return hipSuccess;
  if (units > 0x7FFFFFFFull) return hipErrorInvalidValue;
  const dim3 grid((unsigned)units);
  if constexpr (kMaySumFirst && sizeof(In) == 4) {
    if (sum_first_wins(a.k, a.N)) {
      if (K == 0 && a.k < 10) return sum_first<K == 0>(a, units, s, pos);
      return sum_first<false>(a, units, s, pos);
    }
  }
  constexpr int most = K == 0 && sizeof(In) == 4 ? 8 : kEachGroups;   // fp32 below 2^10: up to five workers
  if constexpr (most > 1)
    if (const int g = each_groups(units, a.N); g > 1) return launch_each_groups<In, most>(g, a, units, s, pos);
  if (prefetch_wins(units)) return launch_kernel(k_fused_each<K, In, true>, grid, dim3(G::THREADS), s, pos, a);
  if constexpr (G::W < 8) return launch_kernel(k_fused_each<K, In, false>, grid, dim3(G::THREADS), s, pos, a);
  return hipErrorInvalidValue;   // not reached
}
// workgroups of SLOTS tiles each; tile_start then counts workgroups
template <int SLOTS, class Kernel>
hipError_t launch_slots(Kernel kernel, int tile_threads, const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if constexpr (SLOTS == 1) return launch_kernel(kernel, dim3((unsigned)units), dim3(tile_threads), s, pos, a);
  BatchArgs b = a;
  uint32_t groups = 0;
  for (int j = 0; j < a.n; ++j) {
    b.tile_start[j] = groups;
    groups += (a.tile_start[j + 1] - a.tile_start[j] + SLOTS - 1) / SLOTS;
  }
  b.tile_start[a.n] = groups;
  return launch_kernel(kernel, dim3(groups), dim3(tile_threads * SLOTS), s, pos, b);
}
template <bool SPLIT>
hipError_t sum_first(const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if (groups_win(units, a.N))
    return launch_kernel(k_fused_batched<K, GROUPS, SPLIT>, dim3((unsigned)units), dim3(kFusedThreads<K> * kGroups), s, pos, a);
  return launch_slots<kBatchSlots<K, STREAM>>(k_fused_batched<K, STREAM, SPLIT>, kFusedThreads<K>, a, units, s, pos);
}
template <class In, int SLOTS>
hipError_t launch_each(const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if constexpr (SLOTS != 4)   // launches of more tiles
    if (prefetch_wins(units)) return launch_slots<SLOTS>(k_fused_each_batched<K, In, true, SLOTS>, G::THREADS, a, units, s, pos);
  if constexpr (G::W < 8) return launch_slots<SLOTS>(k_fused_each_batched<K, In, false, SLOTS>, G::THREADS, a, units, s, pos);
  return hipErrorInvalidValue;   // not reached
}
template <class In>
hipError_t fused_batched(const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if (units == 0) return hipSuccess;
  if (units > 0x7FFFFFFFull) return hipErrorInvalidValue;
  if constexpr (kMaySumFirst && sizeof(In) == 4) {
    if (sum_first_wins(a.k, a.N)) {
      if (K == 0 && a.k < 10) return sum_first<K == 0>(a, units, s, pos);
      return sum_first<false>(a, units, s, pos);
    }
  }
  constexpr int most = K == 0 && sizeof(In) == 4 ? 8 : kEachGroups;   // fp32 below 2^10: up to five workers
  if constexpr (most > 1)
    if (const int g = each_groups(units, a.N); g > 1) return launch_each_groups<In, most>(g, a, units, s, pos);
  // K = 0 with totals, tiles a workgroup: eight share an atomic, four come and go more evenly, which is worth more in launches that
  // leave an uneven number of eights on a CU.  us, eight -> four: bf16 2^9, N = 8, 1 % loss, 2048 / 2200 / 6400 / 12800 tiles 22.5 -> 22.7 / 30.6 ->
  // 25.3 / 53.9 -> 48.5 / 88 -> 81, 5 % loss 23.2 -> 24.0 / 31.7 -> 27.6 / 55.7 -> 50.6 / 91 -> 84;  N = 4, 5 % loss, 2048 / 3277 / 12800 tiles
  // 15.7 -> 17.0 / 21.0 -> 23.5 / 55 -> 53;  fp32 2^9, N = 3, 12800 tiles, 1 / 5 % loss 46 -> 44 / 47 -> 52.
  if constexpr (K == 0) {
    if (a.totals && units > 2048) return launch_each<In, 4>(a, units, s, pos);
    if (a.totals) return launch_each<In, 8>(a, units, s, pos);
  }
  return launch_each<In, 1>(a, units, s, pos);
}
constexpr launch_fn fus_f32 = fused<float>;
constexpr batch_fn fusb_f32 = fused_batched<float>;
#if OR_K == 0
constexpr launch_fn fus_bf16 = fused<bf16_t>;
constexpr batch_fn fusb_bf16 = fused_batched<bf16_t>;
#endif
#else
OR_BLOCK_LAUNCHER(rdec_f32, (k_reduce_decode_block<K, float>))
OR_BLOCK_LAUNCHER(rdec_bf16, (k_reduce_decode_block<K, bf16_t>))
// fp32: 2^15 values a workgroup.  2^16: then the means are decoded where they are
unsigned long long half_grid(unsigned long long blocks) { return K == 15 ? blocks : (blocks + 7) / 8 * 8 * 2; }
hipError_t fus_f32(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {
  const unsigned long long blocks = units >> G::HB;
  if (blocks == 0) return hipSuccess;
  if (half_grid(blocks) > 0x7FFFFFFFull) return hipErrorInvalidValue;
  const dim3 grid((unsigned)half_grid(blocks));
  if (K == 15) return launch_kernel(k_fused_f32_half<K>, grid, dim3(1024), s, pos, a);
  if (hipError_t e = launch_kernel(k_fused_f32_half<K>, grid, dim3(1024), s, pos & LAUNCH_FIRST, a)) return e;
  PathArgs d = a;
  d.in = a.out;
  d.unit0 = units;   // shards hold whole blocks
  return dec_f32(d, units, s, pos & LAUNCH_LAST);
}
hipError_t fusb_f32(const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {
  const unsigned long long blocks = units >> G::HB;
  if (blocks == 0) return hipSuccess;
  if (half_grid(blocks) > 0x7FFFFFFFull) return hipErrorInvalidValue;
  BatchArgs b = a;
  for (int j = 0; j <= a.n; ++j) b.tile_start[j] >>= G::HB;
  const dim3 grid((unsigned)half_grid(blocks));
  if (K == 15) return launch_kernel(k_fused_f32_half_batched<K>, grid, dim3(1024), s, pos, b);
  if (hipError_t e = launch_kernel(k_fused_f32_half_batched<K>, grid, dim3(1024), s, pos & LAUNCH_FIRST, b)) return e;
  if constexpr (K == 16)
    return launch_kernel(blocks << K > kStreamFrom ? k_decode_block_batched<K, true> : k_decode_block_batched<K, false>, dim3((unsigned)blocks),
                         dim3(G::THREADS), s, pos & LAUNCH_LAST, b);
  return hipErrorInvalidValue;   // not reached
}
#endif
#if OR_K >= 11 && OR_K <= 15
// a workgroup per block; `units` and tile_start of the call count tiles (of at most 2^14)
#if OR_K <= 14
constexpr int kGroupsBf16 = K == 11 ? 8 : 16 / MTile<K>::W;
// How many groups of wavefronts encode workers side by side (1: none; the same bits)?  As many as there are workers for, in launches
// that leave CUs idle or leave room on them.  us, without -> with: 2^11, N = 8, 64 blocks 11.6 -> 6.9, 512 blocks 12.7 -> 9.6 (1024:
// 13.9 -> 16.6), N = 3, 100 blocks 7.0 -> 6.3;  2^12, N = 8, 64 blocks 13.2 -> 8.9;  2^13, N = 8, 64 blocks 15.9 -> 13.0, 512 blocks 20.1 ->
// 28.7;  2^14, N = 32, 2 blocks 65.5 -> 59.1, N = 8, 64 blocks 21.2 -> 20.5, 256 blocks 22.0 -> 23.2, N = 3, 100 blocks 11.7 -> 13.3.
// Two groups, up to 2^13, have a form of their own (fused_bf16_pair), which is the shorter chain for few workers and leaves room for a third
// workgroup on a CU.  us, 5 % loss: 2^11, N = 2, 65 blocks 5.3 -> 4.8, none -> it 512 blocks 6.5 -> 6.3;  2^12, four groups -> it, N = 3, 65 blocks 6.9 ->
// 6.9 (nothing lost 5.6 -> 5.9), N = 4, 129 / 300 blocks 7.4 -> 7.3 / 9.1 -> 8.5, N = 8, 300 / 512 blocks 13.2 -> 13.1 / 15.1 -> 14.1, N = 16, 300 / 512 blocks 20.4 -> 22.7 / 22.1 -> 23.4, none -> it, N = 3, 513 /
// 768 blocks 10.3 -> 9.4 / 10.9 -> 10.4, N = 16, 513 / 768 blocks 31.6 -> 26.4 / 33.4 -> 30.3;  2^13, four groups -> it, N = 4, 16 / 129 blocks 9.4 ->
// 8.4 / 10.1 -> 8.9, N = 6, 64 / 256 blocks 12.2 -> 11.6 / 14.1 -> 12.2, N = 8, 64 / 256 blocks 13.4 -> 13.7 / 15.5 -> 14.4.
bool pair_wins(unsigned long long blocks, int N) {
  if (K == 11) return N <= 2 && blocks <= (N == 1 ? 256 : 512);
  if (K == 12) return blocks <= 256 ? N <= 2 : blocks <= 512 ? N <= 8 : blocks <= 768 && N > 1;
  return K == 13 && N <= 6 && blocks <= 256;
}
int groups_bf16(unsigned long long blocks, int N) {
  int most = kGroupsBf16;
  if (pair_wins(blocks, N)) return 2;
  if (N < (K <= 12 ? 3 : K == 13 ? 4 : 6)) return 1;
  if (blocks > (K == 14 ? 128 : 256)) most = K == 11 ? 8 : K == 12 && blocks <= 512 ? 4 : 1;
  if (blocks > 512) most = 1;
  int g = 1;
  while (g < most && g < N) g *= 2;
  return g;
}
template <int G>
hipError_t launch_groups(int g, const PathArgs& a, unsigned long long blocks, hipStream_t s, int pos) {
  if constexpr (G > 2) if (g < G) return launch_groups<G / 2>(g, a, blocks, s, pos);
  return launch_kernel(k_fused_bf16_groups<K, G>, dim3((unsigned)blocks), dim3(MTile<K>::THREADS * G), s, pos, a);
}
template <int G>
hipError_t launch_groups(int g, const BatchArgs& a, unsigned long long blocks, hipStream_t s, int pos) {
  if constexpr (G > 2) if (g < G) return launch_groups<G / 2>(g, a, blocks, s, pos);
  return launch_kernel(k_fused_bf16_groups_batched<K, G>, dim3((unsigned)blocks), dim3(MTile<K>::THREADS * G), s, pos, a);
}
#endif
hipError_t fus_bf16(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {
  const unsigned long long blocks = units >> G::HB;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
#if OR_K <= 14
  if (const int g = groups_bf16(blocks, a.N); g > 1) return launch_groups<kGroupsBf16>(g, a, blocks, s, pos);
#endif
  return launch_kernel(k_fused_bf16<K>, dim3((unsigned)blocks), dim3(MTile<K>::THREADS), s, pos, a);
}
hipError_t fusb_bf16(const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {
  const unsigned long long blocks = units >> G::HB;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
#if OR_K <= 14
  if (const int g = groups_bf16(blocks, a.N); g > 1) return launch_groups<kGroupsBf16>(g, a, blocks, s, pos);
#endif
  BatchArgs b = a;
  for (int j = 0; j <= a.n; ++j) b.tile_start[j] >>= G::HB;
  return launch_kernel(k_fused_bf16_batched<K>, dim3((unsigned)blocks), dim3(MTile<K>::THREADS), s, pos, b);
}
#endif
#if OR_K == 16
// A workgroup per block, or two or four that meet in the workspace (the same bits)?  A workgroup takes 7 us a worker, and takes
// 4.5 / 3.3 us for a half / a quarter of the encoded values.  us, four / two / one workgroups a block: N = 8, 16
// blocks 48 / 64 / 91, 64 blocks 52 / 65 / 92, 100 blocks 86 / 67 / 92, 128 blocks 88 / 68 / 92, 160 blocks 122 / 118 / 94;  N = 2, 64
// blocks 30 / 34 / 37, 128 blocks 44 / 36 / 38;  N = 32, 2 blocks 136 / 190 / 297.  (With nothing lost two of them, which both read the whole block,
// take 4.3 us a worker: N = 8, 100 blocks 57.)  That was with bank conflicts in the exchange; without them four take 45 at 16 and 48 at 64 blocks.
// The same for the blocks that a walk has over in its last round, in launches of their own behind it.  us, in the walk -> that: N = 8, 300 / 384
// / 600 / 1100 blocks 181 -> 147 / 181 -> 166 / 272 -> 253 / 440 -> 427;  N = 32, 257 / 300 blocks 600 -> 458 / 622 -> 470;  N = 2, 300 / 384 blocks
// 74.5 -> 69.3 / 75.0 -> 77.6;  N = 1, 300 / 384 blocks 45.4 -> 48.8 / 46.0 -> 56.7.
constexpr unsigned long long kFourSplit = 64, kTwoSplit = 128;
constexpr unsigned long long kWalkers = 256;   // workgroups that walk over the blocks: one fills a CU
hipError_t fus_bf16(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {
  const unsigned long long blocks = units >> G::HB;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
  const unsigned long long over = blocks > kWalkers && a.N > 1 ? blocks % kWalkers : 0;
  const unsigned long long split = blocks <= kTwoSplit ? blocks : over <= (a.N == 2 ? kFourSplit : kTwoSplit) ? over : 0;
  PathArgs w = a;
  w.unit0 = blocks - split;
  if (w.unit0) {
    const dim3 grid((unsigned)(w.unit0 < kWalkers ? w.unit0 : kWalkers));
    if (hipError_t e = launch_kernel(k_fused_bf16_64k, grid, dim3(512), s, split ? pos & LAUNCH_FIRST : pos, w)) return e;
    pos &= LAUNCH_LAST;
  }
  if (split == 0) return hipSuccess;
  const unsigned eights = (unsigned)(split + 7) / 8 * 8;
  if (hipError_t e = split <= kFourSplit ? launch_kernel(k_fused_bf16_split_64k<1>, dim3(eights * 4), dim3(512), s, pos & LAUNCH_FIRST, w)
                                         : launch_kernel(k_fused_bf16_split_64k<2>, dim3(eights * 2), dim3(512), s, pos & LAUNCH_FIRST, w))
    return e;
  return launch_kernel(k_decode_64k, dim3((unsigned)split), dim3(512), s, pos & LAUNCH_LAST, w);
}
hipError_t fusb_bf16(const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {
  const unsigned long long blocks = units >> G::HB;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
  BatchArgs b = a;
  for (int j = 0; j <= a.n; ++j) b.tile_start[j] >>= G::HB;
  return launch_kernel(k_fused_bf16_batched_64k, dim3((unsigned)(blocks < kWalkers ? blocks : kWalkers)), dim3(512), s, pos, b);
}
#endif
}  // namespace

#if !defined(__HIP_DEVICE_COMPILE__)
#define OR_CAT2(a, b) a##b
#define OR_CAT(a, b) OR_CAT2(a, b)
extern const KernelTable OR_CAT(or_kernel_table_, OR_K) = {
    G::TL, enc_f32, enc_bf16, dec_f32, dec_bf16, fdec_f32, fdec_bf16, mdec_f32, mdec_bf16,
    rdec_f32, rdec_bf16, fus_f32, fus_bf16,
#if OR_K <= 14
    fusb_f32, fusb_bf16, rdecb_f32, rdecb_bf16, fdecb_f32, fdecb_bf16
#else
    fusb_f32, fusb_bf16, nullptr, nullptr, nullptr, nullptr
#endif
};
#endif

}  // namespace orhost

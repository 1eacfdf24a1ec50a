// One block-size class of kernels (compile with -DOR_K=0, 11, 12, ... 16).
#include "launch_table.hpp"
#include "rht_fused.hpp"
#include "rht_fused_each.hpp"
#if OR_K > 14
#include "rht_encode_block.hpp"
#include "rht_fused_mx.hpp"
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
#define OR_ENC(In, Wire) (k_encode<K, In, Wire>)
#define OR_DEC(Out, FIN, MASKED) (k_decode<K, Out, FIN, MASKED>)
#define OR_XFORM_LAUNCHER OR_LAUNCHER
#else
#define OR_ENC(In, Wire) (k_encode_block<K, In, Wire>)
#define OR_DEC(Out, FIN, MASKED) (k_decode_block<K, Out, FIN, MASKED>)
#define OR_XFORM_LAUNCHER OR_BLOCK_LAUNCHER
#endif
OR_XFORM_LAUNCHER(enc_f32, OR_ENC(float, float))
#if OR_K <= 14
OR_LAUNCHER(enc_bf16, OR_ENC(bf16_t, bf16_t))
#else
// workgroups that walk over the blocks: as many as 256 CUs hold at a time
hipError_t enc_bf16(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {
  const unsigned long long blocks = units >> G::HB, resident = K == 15 ? 512 : 256;
  if (blocks == 0) return hipSuccess;
  return launch_kernel(k_encode_block_bf16<K>, dim3((unsigned)(blocks < resident ? blocks : resident)), dim3(1024), s, pos, a);
}
#endif
OR_XFORM_LAUNCHER(dec_f32, OR_DEC(float, false, false))
OR_XFORM_LAUNCHER(dec_bf16, OR_DEC(bf16_t, false, false))
OR_XFORM_LAUNCHER(fdec_f32, OR_DEC(float, true, false))
OR_XFORM_LAUNCHER(fdec_bf16, OR_DEC(bf16_t, true, false))
OR_XFORM_LAUNCHER(mdec_f32, OR_DEC(float, false, true))
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
OR_BATCH_LAUNCHER(fdecb_f32, (k_finalize_decode_batched<K, float>), G::THREADS)
OR_BATCH_LAUNCHER(fdecb_bf16, (k_finalize_decode_batched<K, bf16_t>), G::THREADS)
// GROUPS (tiles up to 2^12) while a launch leaves CUs idle and has the workers for its four groups.  us, 256 tiles, without
// -> with: 2^12, N = 6 9.5 -> 10.2, N = 8 12.1 -> 11.3; 2^10, N = 2 5.4 -> 6.7, N = 4 with a loss in every tile 7.4 -> 6.6.
// Smaller tiles leave room for more of them: 2^11, N = 8, 512 tiles 10.7 -> 9.3, 781 tiles 11.9 -> 15.6.
[[maybe_unused]] bool groups_win(unsigned long long tiles, int N) {
  if (K > 12) return false;
  if (K == 12) return N >= 8 && tiles <= 256;
  if (N < 6) return N >= 4 && tiles <= 256;
  return tiles <= 512;
}
// every worker encoded by itself (rht_fused_each.hpp): bf16 always, fp32 while a launch is short (2^14, N = 4, 1024 tiles
// 75 -> 70 us; N = 8, 2556 tiles with bursts of loss 272 -> 282)
template <class In>
[[maybe_unused]] bool each_wins(unsigned long long tiles) {
  if (sizeof(In) == 2) return true;
  return K >= 12 && tiles <= (K == 12 ? 1024 : K == 13 ? 2048 : 1536);
}
// The second tile buffer of those pays up to three workgroups on a CU.  (Tiles of 8 or 16 wavefronts, at most two workgroups
// on a CU whatever the grid: always.)
bool prefetch_wins(unsigned long long tiles) { return G::W >= 8 || tiles <= 3 * 256; }
template <class In>
hipError_t fused(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if (units == 0) return hipSuccess;
  if (units > 0x7FFFFFFFull) return hipErrorInvalidValue;
  if constexpr (sizeof(In) == 4 && K <= 12) {
    if (groups_win(units, a.N))
      return launch_kernel(k_fused<K, GROUPS>, dim3((unsigned)units), dim3(kFusedThreads<K> * kGroups), s, pos, a);
  }
  if constexpr (sizeof(In) == 2 || K >= 12) {
    if (each_wins<In>(units)) {
      if (sizeof(In) == 4 || prefetch_wins(units))
        return launch_kernel(k_fused_each<K, In, true>, dim3((unsigned)units), dim3(G::THREADS), s, pos, a);
      if constexpr (sizeof(In) == 2)
        return launch_kernel(k_fused_each<K, In, false>, dim3((unsigned)units), dim3(G::THREADS), s, pos, a);
    }
  }
  if constexpr (sizeof(In) == 4) {
    return launch_kernel(k_fused<K, STREAM>, dim3((unsigned)units), dim3(kFusedThreads<K>), s, pos, a);
  }
}
template <class In>
hipError_t fused_batched(const BatchArgs& a, unsigned long long units, hipStream_t s, int pos) {
  if (units == 0) return hipSuccess;
  if (units > 0x7FFFFFFFull) return hipErrorInvalidValue;
  if constexpr (sizeof(In) == 4 && K <= 12) {
    if (groups_win(units, a.N))
      return launch_kernel(k_fused_batched<K, GROUPS>, dim3((unsigned)units), dim3(kFusedThreads<K> * kGroups), s, pos, a);
  }
  if constexpr (sizeof(In) == 2 || K >= 12) {
    if (each_wins<In>(units)) {
      if (sizeof(In) == 4 || prefetch_wins(units))
        return launch_kernel(k_fused_each_batched<K, In, true>, dim3((unsigned)units), dim3(G::THREADS), s, pos, a);
      if constexpr (sizeof(In) == 2)
        return launch_kernel(k_fused_each_batched<K, In, false>, dim3((unsigned)units), dim3(G::THREADS), s, pos, a);
    }
  }
  if constexpr (sizeof(In) == 4) {
    constexpr int SLOTS = kBatchSlots<K, STREAM>;
    if constexpr (SLOTS == 1) {
      return launch_kernel(k_fused_batched<K, STREAM>, dim3((unsigned)units), dim3(kFusedThreads<K>), s, pos, a);
    } else {
      BatchArgs b = a;   // tile_start in workgroups of SLOTS tiles
      uint32_t groups = 0;
      for (int j = 0; j < a.n; ++j) {
        b.tile_start[j] = groups;
        groups += (a.tile_start[j + 1] - a.tile_start[j] + SLOTS - 1) / SLOTS;
      }
      b.tile_start[a.n] = groups;
      return launch_kernel(k_fused_batched<K, STREAM>, dim3(groups), dim3(kFusedThreads<K> * SLOTS), s, pos, b);
    }
  }
}
constexpr launch_fn fus_f32 = fused<float>, fus_bf16 = fused<bf16_t>;
constexpr batch_fn fusb_f32 = fused_batched<float>, fusb_bf16 = fused_batched<bf16_t>;
#else
// one workgroup per pair of output tiles; `units` = output tiles of the shard
#define OR_PAIR_LAUNCHER(name, kernel)                                                       \
  hipError_t name(const PathArgs& a, unsigned long long units, hipStream_t s, int pos) {    \
    if (units == 0) return hipSuccess;                                                       \
    const unsigned long long blocks = units >> G::HB, per = G::PARTS / 2;                    \
    unsigned long long grid = per == 1 ? blocks : (blocks + 7) / 8 * 8 * per;                \
    if (grid > 0x7FFFFFFFull) return hipErrorInvalidValue;                                   \
    return launch_kernel(kernel, dim3((unsigned)grid), dim3(G::THREADS), s, pos, a);         \
  }
OR_BLOCK_LAUNCHER(rdec_f32, (k_reduce_decode_block<K, float>))
OR_BLOCK_LAUNCHER(rdec_bf16, (k_reduce_decode_block<K, bf16_t>))
OR_PAIR_LAUNCHER(fus_f32, (k_fused_pairs<K, float>))
OR_PAIR_LAUNCHER(fus_bf16, (k_fused_mx<K>))
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
    nullptr, nullptr, nullptr, nullptr, nullptr, nullptr
#endif
};
#endif

}  // namespace orhost

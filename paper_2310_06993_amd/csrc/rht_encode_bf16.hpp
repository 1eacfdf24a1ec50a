// Encode (OptiReduce Sec. 3.3) of bf16 gradients in blocks of 2^11 .. 2^14 entries: one workgroup per block, positions, products
// and exchange as in rht_fused_bf16.hpp.
//
// Bound by memory: inputs and outputs of 0.8 to 3.2 GB in turn, several times the last-level cache, 6.0 - 6.5 TB/s of both together (a plain
// copy of the same buffers 4.7 - 5.1).  us, stages one by one with 2 bytes a lane per access -> this: 2^11, 210e6 entries 149 -> 131;  2^12, 13.1e6
// 14.4 -> 10.9, 210e6 153 -> 130;  2^13, 210e6 157 -> 130;  2^14, 131e3 4.9 -> 4.1, 13.1e6 15.9 -> 11.5, 210e6 167 -> 136;  one ragged block of 2^11 / 2^12 /
// 2^13 / 2^14 2.60 -> 2.70 / 2.81 -> 2.87 / 3.43 -> 3.20 / 4.6 -> 3.9.
#pragma once
#include "rht_fused_bf16.hpp"

namespace ordev {

template <int K, bool FULL>
__device__ __forceinline__ void encode_bf16_block(const PathArgs& a, u64 blk, float* x) {
  const int wave = wave_id(), lane = lane_id();
  const u64 e0 = blk << K, first = e0 + (u64)wave * 2048;
  u32x4v p[4];
  const u64 left = FULL ? 2048 : a.n > first ? a.n - first : 0;   // of the wavefront's entries; zeros past the end
  if (FULL || left >= 2048) {
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const bf16_t*)a.in + first, 4096);
#pragma unroll
    for (int q = 0; q < 4; ++q) p[q] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, q * 1024, kBufNt));
  } else {   // the end of the input: pairs that lie inside, and the entry without a partner
    const int inside = (int)left & ~1;
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const bf16_t*)a.in + first, inside * 2);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int d = 0; d < 4; ++d) p[q][d] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, lane * 16 + q * 1024 + d * 4, 0, 0);
    if (left & 1) {
      const uint32_t last = ((const uint16_t*)a.in)[first + inside];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int d = 0; d < 4; ++d) p[q][d] = lane * 8 + q * 512 + d * 2 == inside ? last : p[q][d];
    }
  }
  const uint32_t signs = mt_signs(a.seed, a.base + first, (uint8_t*)(x + wave * 2048), lane);
  __builtin_amdgcn_wave_barrier();
  Operand h = mt_operand(lane);
  float v[32];
  mt_encode_s1(p, signs, h, v);
  mt_store_s1(v, x, wave, lane);
  lds_barrier<MTile<K>::W>();
  mt_s2<K, false>(v, x, wave, lane);
  mt_encode_s2<K>(v, a.scale);
  const float c = K & 1 ? 1.0f : a.scale;
  // Registers r and r + 1 are neighbouring runs of 32 entries, the lane halves the next two: packed and exchanged with the
  // neighbour lane, so that a lane stores two consecutive entries of one of them and a store covers 128 consecutive entries.
  const int odd = lane & 1;
  const uint32_t pick = odd ? 0x03020706u : 0x05040100u;   // bytes 0..3: our pair, 4..7: the neighbour's
  const __amdgpu_buffer_rsrc_t out = rsrc_of((const bf16_t*)a.out + e0, MTile<K>::T * 2);
  const int at = (wave * 128 + (lane >> 5) * 64 + odd * 32 + (lane & 30)) * 2;
#pragma unroll
  for (int r = 0; r < 32; r += 2) {
    const uint32_t own = pack_bf16x2(v[r] * c, v[r + 1] * c);
    const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xf, 0xf, true);   // lane ^ 1
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_amdgcn_perm(other, own, pick), out, at, (r >> 1) << (K - 3), kBufNt);
  }
}
// (four wavefronts: with more registers the compiler lets the products end in accumulation registers, and every value is copied from
// there; one block of 2^11 / 2^12 / 2^13 2.52 -> 2.47, 2.74 -> 2.70, 3.20 -> 3.11)
template <int K>
__global__ __launch_bounds__(MTile<K>::THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k_encode_bf16(PathArgs a) {
  __shared__ __align__(16) float x[MTile<K>::T];
  if (blockIdx.x < a.unit0) encode_bf16_block<K, true>(a, blockIdx.x, x);
  else encode_bf16_block<K, false>(a, blockIdx.x, x);
}

}  // namespace ordev

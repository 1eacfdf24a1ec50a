// Encode (OptiReduce Sec. 3.3) of bf16 gradients in blocks of 2^15 / 2^16 entries: the first factor on the matrix cores and one exchange
// through LDS, as in rht_fused_bf16_64k.hpp.
//
// A workgroup of 8 wavefronts makes 2^14 encoded values at a time, so 64 KB of LDS and 128 registers a lane are enough and two
// workgroups share a CU: one's loads and stores run under the other's arithmetic.  The products make these parts: an operand holds the
// columns of one value of the last bits of the first factor, H_32 (e0 e1 e2 e7 e8) of 2^15 and H_64 (e9 too, two accumulated products)
// of 2^16.  Nothing is read twice.  Entry bits of the positions, T = K - 6:
//   L   as loaded            regs e0 e1 e2, (e9) eT e(T+1) e(T+2)   lanes e3 .. e8               waves e(T+3) ..
//   S1  after the products   regs e3 e4 eT e(T+1) e(T+2)            lanes e0 e1 e2 e7 e5 e6      waves e(T+3) ..   parts e8 (e9)
//   S2  encoded              regs e5 e6 e(T+3) ..                   lanes e0 .. e4 e7            waves eT ..       parts e8 (e9)
// (With the block's highest bits in the place of e8 and e9, which puts a part's results in a row: 3 to 5 % slower between 256 and 2000
// blocks, the same above.)
//
// Bound by memory (a large copy: 5.2 TB/s).  us, stages one by one, 2^16 in one workgroup of 16 wavefronts that asks for the next block before
// it transforms this one -> this: 2^16, 800e6 entries 659 -> 561 (5.7 TB/s), 700 / 512 / 256 blocks 44.1 -> 38.7 / 30.0 -> 26.7 / 15.4 -> 15.0;
// 2^15, 800e6 entries 624 -> 536 (6.0 TB/s), 512 / 256 blocks 15.0 -> 13.8 / 9.2 -> 8.0.  One block of 2^15 / 2^16 7.6 -> 4.5 / 11.4 -> 5.6,
// ragged 14.1 -> 4.6 / 23.8 -> 5.8.
#pragma once
#include "rht_fused_bf16.hpp"

namespace ordev {

template <int K>
struct EBlock {
  static constexpr int P = 1 << (K - 14), LOADS = 4 * P, C = LOADS / 8, THREADS = 512;   // C: products for a value
  static_assert(K == 15 || K == 16, "blocks of 2^15 / 2^16");
};

// SPLIT workgroups a block, on one XCD (blockIdx modulo 8) next to each other: they read the same entries
template <int K, int SPLIT, bool FULL>
__device__ __forceinline__ void encode_block_bf16(const PathArgs& a, u64 blk, int part0, float* x, uint8_t* bytes) {
  typedef EBlock<K> E;
  const int wave = wave_id(), lane = lane_id();
  const u64 e0 = blk << K;
  u32x4v p[E::LOADS];   // load q: 8 entries from at + step(q) of the block on
  const int at = wave * 4096 * E::C + lane * 8;
  auto step = [](int q) { return q * 512; };
  const u64 left = FULL ? 1 << K : a.n - e0;   // of the block's entries; zeros past the end
  if (FULL || left >= (u64)(wave * 4096 * E::C + 4096 * E::C)) {
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const bf16_t*)a.in + e0, 2 << K);
#pragma unroll
    for (int q = 0; q < E::LOADS; ++q) p[q] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, at * 2, step(q) * 2, kBufNt));
  } else {   // the end of the input: pairs that lie inside, and the entry without a partner
    const int inside = (int)left & ~1;
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const bf16_t*)a.in + e0, inside * 2);
#pragma unroll
    for (int q = 0; q < E::LOADS; ++q)
#pragma unroll
      for (int d = 0; d < 4; ++d) p[q][d] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (at + step(q) + d * 2) * 2, 0, 0);
    if (left & 1) {
      const uint32_t last = ((const uint16_t*)a.in)[e0 + inside];
#pragma unroll
      for (int q = 0; q < E::LOADS; ++q)
#pragma unroll
        for (int d = 0; d < 4; ++d) p[q][d] = at + step(q) + d * 2 == inside ? last : p[q][d];
    }
  }
  {   // signs: sixteen Philox counters for each of the P runs of 2048 entries, one a lane, spread through the wavefront's 1 KB
    const u64 ctr = ((a.base + e0 + (u64)wave * 4096 * E::C) >> 7) + (u64)(lane & (32 * E::C - 1));
    const u32x4 w = philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
    uint8_t* mine = bytes + wave * 1024;
    *(uint4*)(mine + lane * 16) = make_uint4(w.a, w.b, w.c, w.d);
    __builtin_amdgcn_wave_barrier();
    auto byte = [&](int q) { return (uint32_t)mine[lane + q * 64]; };
#pragma unroll
    for (int q = 0; q < E::LOADS; q += 4) {
      uint32_t word = pair_signs(byte(q) | byte(q + 1) << 8 | byte(q + 2) << 16 | byte(q + 3) << 24);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        flip_pairs(p[q + c], word);
        asm volatile("" : "+v"(p[q + c]));   // here, not again in every part
      }
    }
  }
  const __amdgpu_buffer_rsrc_t out = rsrc_of((const bf16_t*)a.out + e0, 2 << K);
  const int odd = lane & 1;
  const uint32_t pick = odd ? 0x03020706u : 0x05040100u;   // bytes 0..3: our pair, 4..7: the neighbour's
#pragma unroll
  for (int turn = 0; turn < E::P / SPLIT; ++turn) {
    const int s = SPLIT == 1 ? turn ^ (turn >> 1) : part0 + turn;   // 0 1 3 2; bit 0: e8, bit 1: e9
    if (K == 16 && (SPLIT == 1 ? turn == 2 : turn == 0 && (part0 & 2))) {   // e9 changes: minus the entries of the second products
#pragma unroll
      for (int q = 1; q < E::LOADS; q += 2)
#pragma unroll
        for (int d = 0; d < 4; ++d) p[q][d] ^= 0x80008000u;
    }
    // the +-1 operand: lane l holds column n = l & 15, rows 8 (l >> 4) + 0..7; n0 n1 n2 pair with the entry's place in the load, n3
    // with lane bit 4 (e7), e8 of the part with lane bit 5
    int lane_t = lane;
    asm volatile("" : "+v"(lane_t));   // formed here, not kept in registers all along
    const uint32_t n1 = lane_t & 2 ? 0x80008000u : 0u, n2 = lane_t & 4 ? 0x80008000u : 0u;
    uint32_t w = lane_t & 1 ? 0xBF803F80u : 0x3F803F80u;
    w ^= (lane_t & 24) == 24 ? 0x80008000u : 0u;
    if (s & 1) w ^= lane_t & 32 ? 0x80008000u : 0u;
    const u32x4v h = {w, w ^ n1, w ^ n2, w ^ n1 ^ n2};
    float v[32];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      f32x4v d = {0};
#pragma unroll
      for (int c = 0; c < E::C; ++c)
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8v, p[t * E::C + c]), __builtin_bit_cast(bf16x8v, h), d, 0, 0, 0);
      v[4 * t] = d[0]; v[4 * t + 1] = d[1]; v[4 * t + 2] = d[2]; v[4 * t + 3] = d[3];
    }
    reg_stages(v, 0, 5);
    // from the lowest address bit up: e5 e6 e0 e1 e2 e7 e3 e4 e8 ..
    float* to = x + wave * 2048 + (lane_t & 7) * 4 + ((lane_t >> 3) & 1) * 32 + (lane_t >> 4);
#pragma unroll
    for (int r = 0; r < 32; ++r) to[(r & 3) * 64 + (r >> 2) * 256] = v[r];
    lds_barrier<8>();
    const float* from = x + (lane_t & 7) * 4 + ((lane_t >> 3) & 3) * 64 + (lane_t >> 5) * 32 + wave * 256;
#pragma unroll
    for (int r = 0; r < 32; r += 4) {
      const f32x4v t = *(const f32x4v*)(from + (r >> 2) * 2048);
      v[r] = t[0]; v[r + 1] = t[1]; v[r + 2] = t[2]; v[r + 3] = t[3];
    }
    if (turn + 1 < E::P / SPLIT) lds_barrier<8>();   // everyone has read.  Here, where all wavefronts are together anyway
    reg_stages(v, 0, 5);
    // Registers r and r + 1 are neighbouring runs of 32 entries: packed and exchanged with the neighbour lane, so that a lane stores two
    // consecutive entries of one of them
    const int to_entry = s * 256 + (wave << (K - 6)) + (lane_t >> 5) * 128 + odd * 32 + (lane_t & 30);
#pragma unroll
    for (int r = 0; r < 32; r += 2) {
      const uint32_t own = pack_bf16x2(v[r] * a.scale, v[r + 1] * a.scale);
      const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xf, 0xf, true);   // lane ^ 1
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_amdgcn_perm(other, own, pick), out, to_entry * 2, (((r >> 1) & 1) * 64 + ((r >> 2) << (K - 3))) * 2, kBufNt);
    }
  }
}

template <int K, int SPLIT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_encode_block_bf16(PathArgs a) {
  __shared__ __align__(16) float x[1 << 14];
  __shared__ __align__(16) uint8_t bytes[8 * 1024];
  const unsigned slot = blockIdx.x >> 3;
  const u64 blk = SPLIT == 1 ? blockIdx.x : slot / SPLIT * 8 + (blockIdx.x & 7), blocks = a.n_pad >> K;
  if (SPLIT > 1 && blk >= blocks) return;
  const int part0 = (int)(slot % SPLIT) * (EBlock<K>::P / SPLIT);
  if (blk < (a.unit0 >> (K - 14))) encode_block_bf16<K, SPLIT, true>(a, blk, part0, x, bytes);
  else encode_block_bf16<K, SPLIT, false>(a, blk, part0, x, bytes);
}

}  // namespace ordev

// Encode (OptiReduce Sec. 3.3) of bf16 gradients in blocks of 2^15 / 2^16 entries (P = 2 / 4 tiles of 2^14).
//
// A workgroup holds a whole block in registers.  2^16 blocks leave room for one workgroup on a CU, and nothing would run
// under a block's loads and stores.  Hence: a workgroup walks over blocks and asks for the next one before it transforms
// the current one.  (2^15: two workgroups on a CU do that for each other.)  The entries in flight stay packed pairs (8 registers a tile and lane beside 16 of data), 16 bytes a lane
// per load.  Layouts and the 2^14 transform are those of rht_fused.hpp, the factor across tiles is add / subtract.
// Bound by memory (a large copy: 5.2 TB/s): 1.0e9 entries 930 -> 777 us at 2^16 and 932 -> 749 at 2^15 (5.2 and 5.4 TB/s);
// 3e6 entries at 2^16 28.9 -> 22.3, 30e6 at 2^15 46.5 -> 28.0.  Before: 2 bytes a lane per load, one block a workgroup.
#pragma once
#include "rht_fused.hpp"

namespace ordev {

// Sign bits of this lane's 16 entries (in A) of each of the block's P tiles, from one Philox evaluation: lane 8 p + i holds
// counter i of tile p.  `g` = sign-stream index of the wavefront's first entry in tile 0; x as in lane_signs.
template <int P, class In>
__device__ __forceinline__ void block_lane_signs(u64 seed, u64 g, float* x, int wave, int lane, uint32_t (&sg)[P]) {
  typedef FTile<14, In> F;
  const u64 ctr = ((g + (u64)((lane >> 3) & (P - 1)) * F::T) >> 7) + (u64)(lane & 7);
  const u32x4 w = philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u, (uint32_t)seed, (uint32_t)(seed >> 32));
  uint32_t* words = (uint32_t*)(x + wave * F::PART);
  if (lane < 8 * P) *(uint4*)(words + lane * 4) = make_uint4(w.a, w.b, w.c, w.d);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int p = 0; p < P; ++p) {
    uint32_t bits = 0;
#pragma unroll
    for (int c = 0; c < F::C; ++c) {
      const uint32_t t = words[p * 32 + c * 2 * F::V + (lane >> (5 - F::VB))] >> ((lane & ((32 >> F::VB) - 1)) << F::VB);
      bits |= (t & ((1u << F::V) - 1)) << (c * F::V);
    }
    sg[p] = bits;
  }
  __builtin_amdgcn_wave_barrier();
}

// 16 registers of 64 consecutive entries each (register r: from entry `first` + r * STEP on) as bf16.  Two registers are packed
// and exchanged with the neighbour lane, so that a lane stores two consecutive entries of one of them: 4 bytes a lane, not 2.
template <int STEP>
__device__ __forceinline__ void store_pairs_bf16(const float (&v)[16], __amdgpu_buffer_rsrc_t rs, int tile_byte, int first, int lane) {
  const int odd = lane & 1;
  const uint32_t pick = odd ? 0x03020706u : 0x05040100u;   // bytes 0..3: our pair, 4..7: the neighbour's
  const int at = (first + (lane & ~1) + odd * STEP) * 2;
#pragma unroll
  for (int r = 0; r < 16; r += 2) {
    const uint32_t own = pack_bf16x2(v[r], v[r + 1]);
    const uint32_t other = (uint32_t)__builtin_amdgcn_mov_dpp((int)own, 0xB1, 0xf, 0xf, true);   // lane ^ 1
    // even: (own.lo, other.lo); odd: (other.hi, own.hi)
    const uint32_t x = __builtin_amdgcn_perm(other, own, pick);
    __builtin_amdgcn_raw_buffer_store_b32(x, rs, at, tile_byte + r * STEP * 2, kBufNt);
  }
}

template <int K>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(K == 15 ? 8 : 4)))
void k_encode_block_bf16(PathArgs a) {
  typedef FTile<14, bf16_t> F;
  constexpr int P = 1 << (K - 14), T = F::T, W = F::W, BUFS = K == 15 ? 1 : 2;
  constexpr bool AHEAD = K == 16;
  static_assert(F::reg_entry(1) == 1024 && F::reg_entry(8) == 8192, "register bits of B are entry bits 10 .. 13");
  __shared__ __align__(16) float xbuf[BUFS][W * F::PART];
  const int wave = wave_id(), lane = lane_id();
  const u64 full = a.unit0 >> (K - 14), blocks = a.n_pad >> K;   // blocks that lie inside the input; with the cut one
  Raw16<bf16_t> raw[P];
  auto request = [&](u64 blk) {   // past the last block: zeros, without touching memory
    const bool there = blk < blocks;
    const u64 first = ((there ? blk : 0) << K) + (u64)wave * 1024, left = there && a.n > first ? a.n - first : 0;
    const int valid = left < (P - 1) * T + 1024 ? (int)left : (P - 1) * T + 1024;
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const bf16_t*)a.in + first, valid * 2);
    if (!there || blk < full) {
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int c = 0; c < F::C; ++c)
          raw[p].q[c] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, p * (T * 2) + c * 1024, kBufNt));
    } else {   // the block that the end of the input cuts short: entry by entry, zeros past the end
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int c = 0; c < F::C; ++c)
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            const int at = p * (T * 2) + c * 1024 + d * 4;
            const uint32_t lo = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, lane * 16 + at, 0, 0);
            const uint32_t hi = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, lane * 16 + at + 2, 0, 0);
            raw[p].q[c][d] = lo | hi << 16;
          }
    }
  };
  if (AHEAD) request(blockIdx.x);
  int flip = 0;
  for (u64 blk = blockIdx.x; blk < blocks; blk += gridDim.x) {
    const u64 ew = (blk << K) + (u64)wave * 1024;
    if (!AHEAD) request(blk);
    int lane_t = lane;   // addresses formed here, not kept in registers all along
    asm volatile("" : "+v"(lane_t));
    if (BUFS == 1) __syncthreads();   // nobody still reads the last exchange
    uint32_t sg[P];
    block_lane_signs<P, bf16_t>(a.seed, a.base + ew, xbuf[flip], wave, lane_t, sg);
    float v[P][16];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int r = 0; r < 16; ++r) v[p][r] = flip_sign(entry_of<bf16_t>(raw[p], r), sg[p], r);
    __builtin_amdgcn_sched_barrier(0);
    if (AHEAD) request(blk + gridDim.x);
    __builtin_amdgcn_sched_barrier(0);
    across_tiles<P, 16>(v);
    const float c = a.scale * wire_sigma<14, bf16_t>(wave);
    const __amdgpu_buffer_rsrc_t out = rsrc_of((const bf16_t*)a.out + (blk << K), P * T * 2);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      if (BUFS == 1 && p > 0) __syncthreads();
      to_wire<14, bf16_t>(v[p], xbuf[flip], wave, lane_t, 14);
      flip ^= BUFS - 1;
#pragma unroll
      for (int r = 0; r < 16; ++r) v[p][r] *= c;
      store_pairs_bf16<F::reg_entry(1)>(v[p], out, p * (T * 2), wire_wave_entry<14, bf16_t>(wave), lane_t);
    }
  }
}

}  // namespace ordev

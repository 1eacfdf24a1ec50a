// Reduce + decode (OptiReduce Sec. 3.1.1 aggregation, Sec. 3.3 / Sec. 4 decode) of encoded shards in blocks of 2^15 / 2^16
// entries (P = 2 / 4 tiles of 2^14): one workgroup per block, from the N workers' shards to the decoded mean.
//
// Bound by memory: the sum of a block stays in registers (P * 16 a lane) from the first worker to the decode, where a
// reduction of its own writes sum and counts (5 bytes an entry) for a decode that reads them again.  Loads are 16 bytes a
// lane (layout A of rht_fused.hpp) with DEPTH tiles in flight; a wavefront looks at a tile's received bits once and takes
// the plain additions if nothing is missing in its part.  Counts are not carried along: a wavefront that saw a loss reads
// the bits of that tile again at the end.
// N = 8, from reduction + decode: 1024 blocks of 2^16 605 -> 427 us (5.8 TB/s), bf16 368 -> 263; 2048 blocks of 2^15 595 -> 426,
// bf16 360 -> 241.  (With the 2^14 transform of rht_fused.hpp, which has no DPP stages for most bits and stores from its own
// layout, 1 to 10 % less from four workers and 256 blocks on; its order of stages gave other bits than the two launches that small shards take.)
#pragma once
#include "rht_fused.hpp"

namespace ordev {

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

// Received bits of the lane's 16 entries in A (bit r = register r); `word`: lane l holds word l & 31 of the 32 words of the
// wavefront's 1024 entries.
template <class In>
__device__ __forceinline__ uint32_t lane_bits(uint32_t word, int lane) {
  typedef FTile<14, In> F;
  uint32_t bits = 0;
#pragma unroll
  for (int c = 0; c < F::C; ++c) {
    const int from = c * 2 * F::V + (lane >> (5 - F::VB));
    const uint32_t t = (uint32_t)__builtin_amdgcn_ds_bpermute(from * 4, (int)word) >> ((lane & ((32 >> F::VB) - 1)) << F::VB);
    bits |= (t & ((1u << F::V) - 1)) << (c * F::V);
  }
  return bits;
}

template <int K, class In>
__global__ __launch_bounds__(1024) void k_reduce_decode_block(PathArgs a) {
  typedef FTile<14, In> F;
  constexpr int P = 1 << (K - 14), T = F::T, W = F::W, ES = sizeof(In), DEPTH = ES == 4 || P == 2 ? 2 : 4;
  __shared__ __align__(16) float xbuf[2][W * F::PART];
  __shared__ uint32_t arrived;
  const int wave = wave_id(), lane = lane_id();
  const int N = a.N;
  const u64 L = a.n_pad, row_bytes = L >> 3;
  const u64 e0 = (u64)blockIdx.x << K, ew = e0 + (u64)wave * 1024;   // first entry of the block / of this wavefront's part
  if (threadIdx.x == 0) arrived = 0;   // behind the barriers of the transform when it is added to

  auto request = [&](int i, int p, Raw16<In>& r) {   // past the last worker: zeros, without touching memory
    const bool there = i < N;
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const In*)a.in + (u64)(there ? i : 0) * L + ew, there ? ((P - 1) * T + 1024) * ES : 0);
#pragma unroll
    for (int c = 0; c < F::C; ++c)
      r.q[c] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, p * (T * ES) + c * 1024, kBufNt));
  };
  auto request_word = [&](int i, int p) {
    const bool there = i < N;
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const uint8_t*)a.masks + (u64)(there ? i : 0) * row_bytes + (ew >> 3), there ? ((P - 1) * T + 1024) >> 3 : 0);
    return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (lane & 31) * 4, p * (T >> 3), 0);
  };

  float v[P][16];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int r = 0; r < 16; ++r) v[p][r] = 0.0f;
  uint32_t lossy = 0;   // bit p: something of tile p is missing in this wavefront's part
  {
    Raw16<In> ring[DEPTH];
    uint32_t words[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      request(d / P, d % P, ring[d]);
      words[d] = request_word(d / P, d % P);
    }
    for (int i = 0; i < N; ++i) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        Raw16<In>& x = ring[p % DEPTH];
        uint32_t& w = words[p % DEPTH];
        if (all_arrived(w)) {
#pragma unroll
          for (int r = 0; r < 16; ++r) v[p][r] += entry_of<In>(x, r);
        } else {
          lossy |= 1u << p;
          const uint32_t bits = lane_bits<In>(w, lane);
#pragma unroll
          for (int r = 0; r < 16; ++r) {   // what did not arrive may be anything, NaN too
            const int keep = (int)(bits << (31 - r)) >> 31;
            v[p][r] += __builtin_bit_cast(float, (int)__builtin_bit_cast(int, entry_of<In>(x, r)) & keep);
          }
        }
        request(i + (p + DEPTH) / P, (p + DEPTH) % P, x);
        w = request_word(i + (p + DEPTH) / P, (p + DEPTH) % P);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ---- counts, mean over what arrived
  const __amdgpu_buffer_rsrc_t counts = rsrc_of(a.count_out + ew, a.count_out ? (P - 1) * T + 1024 : 0);   // none: stores are dropped
  const bool counts_aligned = ((uintptr_t)a.count_out & 3) == 0;
  uint32_t total = 0;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    uint32_t c4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) c4[q] = (uint32_t)N * 0x01010101u;
    if (!((lossy >> p) & 1)) {
      const float f = __builtin_amdgcn_rcpf((float)N);
#pragma unroll
      for (int r = 0; r < 16; ++r) v[p][r] *= f;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) c4[q] = 0;
      for (int i = 0; i < N; i += 4) {
        uint32_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = request_word(i + u, p);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t bits = lane_bits<In>(w[u], lane);
#pragma unroll
          for (int q = 0; q < 4; ++q) c4[q] += (((bits >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t n = (c4[r >> 2] >> (8 * (r & 3))) & 0xFFu;
        v[p][r] = n ? v[p][r] * __builtin_amdgcn_rcpf((float)n) : 0.0f;
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) total = __builtin_amdgcn_sad_u8(c4[q], 0u, total);
    // registers 4 q .. 4 q + 3 are four consecutive entries
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = (4 * q >> F::VB) * 64 * F::V + (4 * q & (F::V - 1));
      store_counts4(c4[q], counts, lane * F::V, p * T + e, counts_aligned);
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- decode, by the stages of decode_block in their order: the same bits as from a reduction and a decode of their own.  Each
  // tile goes through LDS from A to layout B of rht_tile.hpp; the two buffers alternate, one barrier per exchange.
  uint32_t slo, shi;
  block_sign_words<K>(a.seed, a.base + ew, slo, shi);
  across_tiles<P, 16>(v);
  const float c = a.scale * lane_sigma(lane, 6);
  const __amdgpu_buffer_rsrc_t out = rsrc_of((const In*)a.out + e0, P * T * ES);
#pragma unroll
  for (int p = 0; p < P; ++p) {
    int lane_t = lane;   // addresses formed here, not kept in registers all along
    asm volatile("" : "+v"(lane_t));
    lds_a<14, In, true>(v[p], xbuf[0], wave, lane_t);
    __syncthreads();
    const float* mine = xbuf[0] + F::padded(wave * 64) + lane_t;
#pragma unroll
    for (int r = 0; r < 16; ++r) v[p][r] = mine[F::padded(r << 10)];
    transform<K, false, false>(v[p], xbuf[1], wave, lane_t, 14);
#pragma unroll
    for (int r = 0; r < 16; ++r) v[p][r] *= c;
    apply_block_signs(v[p], slo, shi, p);
    if constexpr (ES == 2) {
      store_pairs_bf16<64>(v[p], out, p * (T * ES), wave * 1024, lane_t);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v[p][r]), out, (wave * 1024 + lane_t) * 4, (p * T + r * 64) * 4, kBufNt);
    }
  }
  if (a.total_out) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) total += (uint32_t)__shfl_xor((int)total, o, 64);
    if (lane == 0) atomicAdd(&arrived, total);   // zeroed ahead of the barriers above
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(a.total_out, (unsigned long long)arrived);
  }
}

}  // namespace ordev

// The fused path (OptiReduce Sec. 3.3 encode, Sec. 3.1.1 aggregation, Sec. 3.3 / Sec. 4 decode) of fp32 slices in blocks of 2^15 /
// 2^16 entries.  A workgroup makes 2^15 encoded values: a whole block of 2^15, from the slices to the decoded mean; or one half of a
// block of 2^16 (index bit 15 = h; H_{2^16} = H_2 (x) H_{2^15}: the sum or the difference of the two halves of its input), up to the
// mean, which goes to the output and is decoded there in place by a kernel of its own.  No workspace, no table of signs.
//
// The encode is linear and the signs are the same for every worker: the workers whose copy of the workgroup's values arrived WHOLE
// are added up as they come from memory and encoded once, after those that lost something, which are encoded one by one.
//
// 16 wavefronts, 32 values a lane, 2048 consecutive ones a wavefront.  Entry bits of the positions (e0 is the lowest; e0 .. e14):
//   L   as loaded and stored   regs e0 e1 (16 bytes), e8 e9 e10    lanes e2 .. e7               waves e11 ..
//   S1                         regs e2 e3 e4 e6 e7                 lanes e5 e0 e1 e8 e9 e10     waves e11 ..
//   S2  encoded ("wire")       regs e5 e11 e12 e13 e14             lanes e0 .. e4 e6            waves e7 ..    (as MTile<15>)
// All fifteen stages are additions between registers.  L to S1 stays inside the wavefront, S1 to S2 is the exchange between them.  The
// side that goes first stores singly and the other loads 16 bytes a lane, which LDS serves twice as fast as the other way round.
//
// us, tile by tile with a table of signs and every worker by itself -> this: 2^15, N = 8, 1280 blocks, 1 % loss in packets 351 -> 288
// (5.5 TB/s of slices, masks, results and counts), 0.2 % in bursts 341 -> 265;  N = 32, 300 blocks, 5 % 454 -> 377, one block 177 -> 145;  2^16, N = 8, 640 blocks 543 -> 488, 16
// blocks 82 -> 68;  N = 32, 150 blocks, 5 % 614 -> 512;  N = 2, 1000 blocks 352 -> 337.  (One to four blocks of two or three workers that
// lost something: 2^15 18.9 -> 19.5, 2^16 31.6 -> 32.5.)  Bound by memory where nearly every copy is whole, else
// by the encode (fifteen stages and two trips through LDS, on a CU with nothing else on it), 2^16 also by the second reading of the
// slices, which the L2 serves in part: without the nontemporal hint 548 -> 488.
#pragma once
#include "rht_fused_bf16.hpp"

namespace ordev {

typedef MTile<15> Half;
constexpr int kHalf = 1 << 15;

// ---- LDS positions.  Inside the wavefront (its own 2048 floats), from the lowest address bit up: e2 e3 (e4^e0) e5 (e6^e1) e7 e0 e1 e8 e9 e10
template <bool STORE>
__device__ __forceinline__ void half_l(float (&v)[32], float* mine, int lane) {
#pragma unroll
  for (int r = 0; r < 32; ++r) {
    float* p = mine + (lane ^ ((r & 1) * 4 + ((r >> 1) & 1) * 16)) + r * 64;
    if constexpr (STORE) *p = v[r]; else v[r] = *p;
  }
}
template <bool STORE>
__device__ __forceinline__ void half_s1(float (&v)[32], float* mine, int lane) {
  // lanes e5 e0 e1 e8 e9 e10
  const int at = (lane & 1) * 8 + ((lane >> 1) & 1) * (64 + 4) + ((lane >> 2) & 1) * (128 + 16) + (lane >> 3) * 256;
#pragma unroll
  for (int g = 0; g < 8; ++g) {   // registers e2 e3 | e4 e6 e7
    f32x4v* p = (f32x4v*)(mine + (at ^ ((g & 1) * 4 + ((g >> 1) & 1) * 16)) + (g >> 2) * 32);
    if constexpr (STORE) {
      *p = f32x4v{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
    } else {
      const f32x4v t = *p;
      v[4 * g] = t[0]; v[4 * g + 1] = t[1]; v[4 * g + 2] = t[2]; v[4 * g + 3] = t[3];
    }
  }
}
// between the wavefronts: e5 e11 e0 e1 (e2^e8) (e3^e9) e4 e6 e7 e8 e9 e10 e12 e13 e14
template <bool STORE>
__device__ __forceinline__ void half_x1(float (&v)[32], float* x, int wave, int lane) {
  const int at = (lane & 1) + ((lane >> 1) & 3) * 4 + ((lane >> 3) & 1) * (512 + 16) + ((lane >> 4) & 1) * (1024 + 32) + (lane >> 5) * 2048 +
                 (wave & 1) * 2 + (wave >> 1) * 4096;
#pragma unroll
  for (int r = 0; r < 32; ++r) {
    float* p = x + (at ^ ((r & 3) * 16)) + (r >> 2) * 64;
    if constexpr (STORE) *p = v[r]; else v[r] = *p;
  }
}
template <bool STORE>
__device__ __forceinline__ void half_x2(float (&v)[32], float* x, int wave, int lane) {
  const int at = ((lane * 4) ^ (((wave >> 1) & 3) * 16)) + wave * 256;
#pragma unroll
  for (int g = 0; g < 8; ++g) {   // registers e5 e11 | e12 e13 e14
    f32x4v* p = (f32x4v*)(x + at + g * 4096);
    if constexpr (STORE) {
      *p = f32x4v{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
    } else {
      const f32x4v t = *p;
      v[4 * g] = t[0]; v[4 * g + 1] = t[1]; v[4 * g + 2] = t[2]; v[4 * g + 3] = t[3];
    }
  }
}

// Signs of the lane's 32 entries in L: bit 31 - r is that of register r.
__device__ __forceinline__ uint32_t half_signs(u64 seed, u64 first, uint8_t* bytes, int lane) {
  const u64 ctr = (first >> 7) + (u64)(lane & 15);
  const u32x4 w = philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u, (uint32_t)seed, (uint32_t)(seed >> 32));
  if (lane < 16) *(uint4*)(bytes + lane * 16) = make_uint4(w.a, w.b, w.c, w.d);
  __builtin_amdgcn_wave_barrier();
  uint32_t s = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) s |= (((uint32_t)bytes[32 * q + (lane >> 1)] >> (4 * (lane & 1))) & 0xFu) << (4 * q);
  __builtin_amdgcn_wave_barrier();
  return __builtin_bitreverse32(s);
}
__device__ __forceinline__ float flip_next(float v, uint32_t& word) {   // by the top bit of `word`, which moves on
  const float f = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) ^ (word & 0x80000000u));
  asm("v_add_u32 %0, %0, %0" : "+v"(word));
  return f;
}

// `h`: the half of a block of 2^16; `e0`: first entry of the block
template <int K, bool TOTAL>
__device__ __forceinline__ void fused_f32_half(const PathArgs& a, u64 e0, int h) {
  constexpr int PARTS = 1 << (K - 15);
  __shared__ __align__(16) float x[kHalf];
  __shared__ uint32_t marks[8];        // one bit per worker: something is missing
  __shared__ uint8_t order[256];
  __shared__ uint32_t missing;
  const int wave = wave_id(), lane = lane_id(), N = a.N;
  const u64 L = a.n_pad, eo = e0 + (u64)h * kHalf;   // eo: first of the workgroup's encoded values
  float* mine = x + wave * 2048;
  if (threadIdx.x < 8) marks[threadIdx.x] = 0;
  if (TOTAL && threadIdx.x == 0) missing = 0;
  lds_barrier<16>();

  // ---- who lost something
  for (int i = 0; i < N; i += 8) {
    uint32_t w[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) w[u] = mt_words<15>(a, eo, i + u, wave, lane);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i + u < N && !all_arrived(w[u]) && lane == 0) atomicOr(&marks[(i + u) >> 5], 1u << ((i + u) & 31));
  }
  uint32_t signs[PARTS];
#pragma unroll
  for (int p = 0; p < PARTS; ++p) signs[p] = half_signs(a.seed, a.base + e0 + (u64)p * kHalf + (u64)wave * 2048, (uint8_t*)mine, lane);
  if (PARTS == 2 && h) signs[PARTS - 1] = ~signs[PARTS - 1];   // minus the second half
  lds_barrier<16>();
  int lossy = 0;
  for (int i = 0; i < N; i += 32) lossy += __builtin_popcount((uint32_t)__builtin_amdgcn_readfirstlane((int)marks[i >> 5]));
  const uint32_t ord = order_workers(marks, order, N, lossy, lane);
  auto worker = [&](int j) { return (int)(((uint32_t)__builtin_amdgcn_readlane((int)ord, j & 63) >> (j >> 6 << 3)) & 0xFFu); };

  u32x4v q[8];
  auto request = [&](int j, int part) {   // the j-th worker in order; past the last: zeros, without touching memory
    const bool there = j < N;
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const float*)a.in + (u64)(there ? worker(j) : 0) * L + e0 + (u64)part * kHalf + (u64)wave * 2048, there ? 8192 : 0);
#pragma unroll
    for (int c = 0; c < 8; ++c) q[c] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, c * 1024, PARTS == 1 ? kBufNt : 0));
  };
  auto encode = [&](float (&v)[32]) {   // L -> S2; behind a barrier since anyone read x
    int lane_t = lane;   // addresses formed here, not kept in registers all along
    asm volatile("" : "+v"(lane_t));
    reg_stages(v, 0, 5);
    half_l<true>(v, mine, lane_t);
    __builtin_amdgcn_wave_barrier();
    half_s1<false>(v, mine, lane_t);
    reg_stages(v, 0, 5);
    lds_barrier<16>();   // every wavefront has read its part
    half_x1<true>(v, x, wave, lane_t);
    lds_barrier<16>();
    half_x2<false>(v, x, wave, lane_t);
    lds_barrier<16>();   // everyone has read; here, where all are together anyway
    reg_stages(v, 0, 5);
  };

  float acc[32], v[32];
#pragma unroll
  for (int r = 0; r < 32; ++r) acc[r] = 0.0f;
  request(0, 0);
  bool fresh = true;   // v holds nothing yet
  for (int j = 0; j < N; ++j) {
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
      uint32_t word = signs[p];
      asm volatile("" : "+v"(word));
      if (fresh && p == 0) {
#pragma unroll
        for (int r = 0; r < 32; ++r) v[r] = 0.0f;
      }
#pragma unroll
      for (int r = 0; r < 32; ++r) {
        v[r] += flip_next(__builtin_bit_cast(float, (uint32_t)q[r >> 2][r & 3]), word);
        asm volatile("" : "+v"(v[r]));   // here, ahead of the next request, which needs the registers
      }
      request(p + 1 < PARTS ? j : j + 1, (p + 1) % PARTS);
    }
    fresh = j < lossy || j == N - 1;
    if (fresh) {
      const uint32_t words = j < lossy ? mt_words<15>(a, eo, worker(j), wave, lane) : 0xFFFFFFFFu;
      encode(v);
      if (!all_arrived(words)) mt_mask(v, words);
#pragma unroll
      for (int r = 0; r < 32; ++r) {
        acc[r] += v[r];
        asm volatile("" : "+v"(acc[r]));   // here, not where the sum is next used
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- counts, mean over what arrived
  uint32_t c8[8];
  if (lossy == 0) {
#pragma unroll
    for (int c = 0; c < 8; ++c) c8[c] = (uint32_t)N * 0x01010101u;
  } else {
    mt_recount<15>(a, eo, 0, 1, wave, lane, c8);
  }
  mt_store_counts<15>(a, eo, wave, lane, c8);
  if (TOTAL && a.total_out && lossy) mt_add_missing(c8, N, &missing, lane);
  if (lossy == 0) {
    const float f = a.scale * __builtin_amdgcn_rcpf((float)N);
#pragma unroll
    for (int r = 0; r < 32; ++r) acc[r] *= f;
  } else {
    uint8_t* counts = (uint8_t*)mine;
    *(uint4*)(counts + lane * 32) = make_uint4(c8[0], c8[1], c8[2], c8[3]);
    *(uint4*)(counts + lane * 32 + 16) = make_uint4(c8[4], c8[5], c8[6], c8[7]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 32; ++r) acc[r] = mt_mean(acc[r], mt_count(counts, r, lane), a.scale);
  }
  lds_barrier<16>();   // the counts are read, what is missing is there
  if (TOTAL && a.total_out && threadIdx.x == 0) add_total(a, eo == 0, missing);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (PARTS == 2) {   // the mean, where the decoded block will be
    const __amdgpu_buffer_rsrc_t out = rsrc_of((const float*)a.out + eo + wave * 128, (kHalf - wave * 128) * 4);
    const int at = ((lane & 31) + (lane >> 5) * 64) * 4;
#pragma unroll
    for (int r = 0; r < 32; ++r)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, acc[r]), out, at, ((r & 1) * 32 + (r >> 1) * 2048) * 4, 0);
  } else {   // decode: S2, S1, L
    reg_stages(acc, 0, 5);
    half_x2<true>(acc, x, wave, lane);
    lds_barrier<16>();
    half_x1<false>(acc, x, wave, lane);
    lds_barrier<16>();
    reg_stages(acc, 0, 5);
    half_s1<true>(acc, mine, lane);
    __builtin_amdgcn_wave_barrier();
    half_l<false>(acc, mine, lane);
    reg_stages(acc, 0, 5);
    const __amdgpu_buffer_rsrc_t out = rsrc_of((const float*)a.out + e0 + (u64)wave * 2048, 8192);
    uint32_t word = signs[0];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      u32x4v o;
#pragma unroll
      for (int d = 0; d < 4; ++d) o[d] = __builtin_bit_cast(uint32_t, flip_next(acc[4 * c + d] * a.scale, word));
      store16<kBufNt>(o, out, lane * 16 + c * 1024);
    }
  }
}

// workgroup x: block and half.  The two of a block of 2^16 read the same entries: on one XCD (blockIdx modulo 8) next to each other
template <int K>
__device__ __forceinline__ void half_of(unsigned x, u64& blk, int& h) {
  if constexpr (K == 15) {
    blk = x;
    h = 0;
  } else {
    const unsigned slot = x >> 3;
    h = (int)(slot & 1);
    blk = (u64)(slot >> 1) * 8 + (x & 7);
  }
}
template <int K>
__global__ __launch_bounds__(1024) void k_fused_f32_half(PathArgs a) {
  u64 blk;
  int h;
  half_of<K>(blockIdx.x, blk, h);
  if (blk >= a.n_pad >> K) return;
  fused_f32_half<K, false>(a, blk << K, h);
}
template <int K>
__global__ __launch_bounds__(1024) void k_fused_f32_half_batched(BatchArgs ba) {   // ba.tile_start counts blocks
  u64 blk;
  int h;
  half_of<K>(blockIdx.x, blk, h);
  if (blk >= ba.tile_start[ba.n]) return;
  PathArgs a;
  const u64 unit = bucket_of(ba, a, (uint32_t)blk);
  fused_f32_half<K, true>(a, unit << K, h);
}
// the means of 2^16 blocks in the buckets' outputs, decoded in place
template <int K, bool STREAM>
__global__ __launch_bounds__(Geo<K>::THREADS) void k_decode_block_batched(BatchArgs ba) {
  __shared__ float xbuf[2][Geo<K>::T];
  PathArgs a;
  const u64 unit = bucket_of(ba, a, blockIdx.x);
  a.in = a.out;
  decode_block<K, float, false, true, false, STREAM>(a, unit, xbuf);
}

}  // namespace ordev

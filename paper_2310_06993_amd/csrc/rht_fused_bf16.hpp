// The fused path (OptiReduce Sec. 3.3 encode, Sec. 3.1.1 aggregation, Sec. 3.3 / Sec. 4 decode) of bf16 slices in blocks of
// 2^11 .. 2^15 entries: one workgroup per block, every worker encoded by itself (its encoded value is rounded to bf16).
//
// The first five of the K butterfly stages are a product with H_32 on the matrix cores: the raw entries are bf16 and the matrix is
// +-1, so it is exact up to the order of its fp32 additions.  The data is the A operand (32 rows x 16 entries a product, two
// products accumulated), hence the five finished index bits come out on lanes and four of the five others in registers: what
// is left are plain additions between registers before and after ONE exchange through LDS -- no stage across lanes at all.
// Wavefronts hold 2048 entries, 32 a lane.  Entry bits of the positions (e0 is the lowest; waves: the lowest bit first):
//   L   as loaded and stored   regs e0 e1 e2 (16 bytes), e9 e10    lanes e3 .. e8             waves e11 ..
//   S1  after the product      regs e3 e4 e6 e7 e10                lanes e0 e1 e2 e8 e9 e5    waves e11 ..
//   S2  encoded ("wire")       regs e5, the four highest           lanes e0 .. e4 e6          waves e7 ..
//   S3  in the decode          regs e3 e4 e6 e7 e8                 lanes e0 e1 e2 e9 e5 e10   waves e11 ..
// Product: e0 e1 e2 e8 e9; S1: its registers; S2: e5 and e11 and up.  Decode: S2 all registers, S3 and L what is left of theirs.
// In S2 a register covers two runs of 32 entries: two words of received bits, used as the halves of a lane mask.
//
// Per worker and 2048 entries about 360 vector instructions and 8 + 16 accesses to LDS, where the stages one by one (signs, unpacking,
// fourteen stages) took 700 and 128.  Large launches of 2^11 .. 2^14 are bound by memory: without transform and exchange 135 us of
// 159 (2^14, N = 8, 2556 blocks, nothing lost).  A block of 2^15 fills a CU: its exchanges and arithmetic take turns.  us, stages one
// by one -> this: 2^14, N = 8, 2556 blocks, 2 % loss in bursts 230 -> 165 (5.1 TB/s), 5 % in single packets 241 -> 177;  2^15, N = 8,
// 1280 blocks 258 -> 196;  2^13, N = 8, 5000 blocks 209 -> 153;  2^12, N = 16, 10000 blocks 375 -> 271, N = 2 74 -> 54;  2^11, N = 8,
// 20000 blocks 195 -> 142.  Two workers in flight instead of one: 164 -> 170.
// The price is a longer decode, which has half as many wavefronts; in launches of few blocks and workers two groups share it
// (fused_bf16_pair): 2^12, N = 2, 129 blocks 5.7 -> 5.6;  2^13, N = 3, 65 blocks 8.3 -> 8.2.  Those that still lose: 2^12, N = 3, 5 % loss, 512
// blocks 8.7 -> 8.9 .. 9.2;  a single worker, 65 blocks of 2^11 / 2^12 / 2^13 3.9 -> 4.1 / 4.2 -> 4.4 / 5.1 -> 5.3.
#pragma once
#include "rht_fused.hpp"

namespace ordev {

typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
typedef float f32x16v __attribute__((ext_vector_type(16)));

// The signs of four loads of 8 entries a lane, from their four sign bytes, as pairs in the order of the loads: bit 31 - j is the sign
// of the odd entry of pair j, bit 15 - j that of the even one.  Pair j's signs are then (word << j) & 0x80008000, and the next pair's
// word is word + word, which issues at twice the rate of a shift.
__device__ __forceinline__ uint32_t pair_signs(uint32_t bytes) {
  uint32_t w = __builtin_bitreverse32(bytes), t;
  // bit 31 - 2 j: even entry, bit 30 - 2 j: odd one; unshuffle, and put the odd ones on top
  t = (w ^ (w >> 1)) & 0x22222222u; w ^= t ^ (t << 1);
  t = (w ^ (w >> 2)) & 0x0C0C0C0Cu; w ^= t ^ (t << 2);
  t = (w ^ (w >> 4)) & 0x00F000F0u; w ^= t ^ (t << 4);
  t = (w ^ (w >> 8)) & 0x0000FF00u; w ^= t ^ (t << 8);
  return w << 16 | w >> 16;
}
// flips the signs of a load's four pairs and moves `word` on to the next load's
__device__ __forceinline__ void flip_pairs(u32x4v& y, uint32_t& word) {
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    y[d] ^= word & 0x80008000u;
    asm("v_add_u32 %0, %0, %0" : "+v"(word));
  }
}

// Barrier for what goes through LDS: loads from memory stay in flight.  (A tile of one wavefront has its accesses to LDS in order.)
template <int W>
__device__ __forceinline__ void lds_barrier() {
  if constexpr (W > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  else __builtin_amdgcn_wave_barrier();
}

template <int K>
struct MTile {
  static constexpr int Q = K - 11, W = 1 << Q, T = 1 << K, R = 32, THREADS = 64 * W;
  static_assert(K >= 11 && K <= 15, "blocks of 2^11 .. 2^15");
  // floats; entry bits e3 e4 e0 e1 e2 e6 e5 e7 .. from the lowest address bit up: 16-byte accesses from S1 and S3, 32 different
  // banks for every half of a wavefront in S2
  static constexpr int s2_reg(int r) { return (r & 1) * 64 + ((r >> 1) << (K - 4)); }
};

template <int K, bool STORE>
__device__ __forceinline__ void mt_s2(float (&v)[32], float* x, int wave, int lane) {
  float* p = x + (lane & 7) * 4 + ((lane >> 3) & 3) + (lane >> 5) * 32 + wave * 128;
#pragma unroll
  for (int r = 0; r < 32; ++r) {
    if constexpr (STORE) p[MTile<K>::s2_reg(r)] = v[r]; else v[r] = p[MTile<K>::s2_reg(r)];
  }
}

// ---- a worker's entries and received bits on their way to one wavefront: part `wave` of the block that starts at entry e0
struct InFlight {
  u32x4v q[4];
  uint32_t words;
};
// Received bits in S2: lane l holds run l & 3 (32 entries) of the wavefront's 128 entries in sixteenth l >> 2 of the block.
template <int K>
__device__ __forceinline__ uint32_t mt_words(const PathArgs& a, u64 e0, int i, int wave, int lane) {
  const bool there = i < a.N;   // no such worker: zeros, without touching memory
  const __amdgpu_buffer_rsrc_t rs = rsrc_of((const uint8_t*)a.masks + (u64)(there ? i : 0) * (a.n_pad >> 3) + (e0 >> 3) + wave * 16,
                                            there ? (MTile<K>::T >> 3) - wave * 16 : 0);
  return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, ((lane >> 2) << (K - 7)) + (lane & 3) * 4, 0, 0);
}
template <int K>
__device__ __forceinline__ void mt_request(const PathArgs& a, u64 e0, int i, int wave, int lane, InFlight& f) {
  const bool there = i < a.N;
  const __amdgpu_buffer_rsrc_t rs = rsrc_of((const bf16_t*)a.in + (u64)(there ? i : 0) * a.n_pad + e0 + (u64)wave * 2048, there ? 4096 : 0);
#pragma unroll
  for (int q = 0; q < 4; ++q) f.q[q] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, q * 1024, kBufNt));
  f.words = mt_words<K>(a, e0, i, wave, lane);
}

// Signs of the lane's four loads (pair_signs): 16 Philox counters a wavefront, spread through its own 256 bytes at `bytes`.
__device__ __forceinline__ uint32_t mt_signs(u64 seed, u64 first, uint8_t* bytes, int lane) {
  const u64 ctr = (first >> 7) + (u64)(lane & 15);
  const u32x4 w = philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u, (uint32_t)seed, (uint32_t)(seed >> 32));
  if (lane < 16) *(uint4*)(bytes + lane * 16) = make_uint4(w.a, w.b, w.c, w.d);
  __builtin_amdgcn_wave_barrier();
  return pair_signs((uint32_t)bytes[lane] | (uint32_t)bytes[lane + 64] << 8 | (uint32_t)bytes[lane + 128] << 16 | (uint32_t)bytes[lane + 192] << 24);
}

// The +-1 operand: lane l holds column n = l & 31, rows 8 (l >> 5) + 0..7; n0 n1 n2 pair with the entry's place in the load (e0 e1
// e2), n3 with l >> 5 (e8), n4 with the load's number (e9): the second product's operand is the first's with the sign of n4.
struct Operand {
  u32x4v first;
  uint32_t second;
};
__device__ __forceinline__ Operand mt_operand(int lane) {
  const uint32_t n1 = lane & 2 ? 0x80008000u : 0u, n2 = lane & 4 ? 0x80008000u : 0u;
  const uint32_t w = (lane & 1 ? 0xBF803F80u : 0x3F803F80u) ^ ((lane & 40) == 40 ? 0x80008000u : 0u);
  return {u32x4v{w, w ^ n1, w ^ n2, w ^ n1 ^ n2}, lane & 16 ? 0x80008000u : 0u};
}

// signs, products and the register stages of S1
__device__ __forceinline__ void mt_encode_s1(const u32x4v (&p)[4], uint32_t signs, Operand& h, float (&v)[32]) {
  asm volatile("" : "+v"(signs), "+v"(h.second));   // the masks of the signs and the second operand are formed here, not kept in registers
  u32x4v second = h.first;
#pragma unroll
  for (int d = 0; d < 4; ++d) second[d] ^= h.second;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    f32x16v d = {0};
#pragma unroll
    for (int q = 2 * c; q < 2 * c + 2; ++q) {
      u32x4v y = p[q];
      flip_pairs(y, signs);
      d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8v, y), __builtin_bit_cast(bf16x8v, q & 1 ? second : h.first), d, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) v[16 * c + r] = d[r];
  }
  reg_stages(v, 0, 5);
}
__device__ __forceinline__ void mt_store_s1(const float (&v)[32], float* x, int wave, int lane) {
  float* to = x + wave * 2048 + (lane & 7) * 4 + ((lane >> 3) & 3) * 256 + (lane >> 5) * 64;
#pragma unroll
  for (int g = 0; g < 8; ++g)   // registers e3 e4 | e6 e7 e10
    *(f32x4v*)(to + (g & 1) * 32 + ((g >> 1) & 1) * 128 + (g >> 2) * 1024) = f32x4v{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
}
// the register stages that are left in S2 (e5 and e11 and up), and the scale where it does not commute with the rounding
template <int K>
__device__ __forceinline__ void mt_encode_s2(float (&v)[32], float scale) {
  reg_stage<0>(v);
  reg_stages(v, K >= 15 ? 1 : 16 - K, 5);
  if constexpr (K & 1) {
#pragma unroll
    for (int r = 0; r < 32; ++r) v[r] *= scale;
  }
}
__device__ __forceinline__ void mt_mask(float (&v)[32], uint32_t words) {   // zero where something was lost
#pragma unroll
  for (int r = 0; r < 32; ++r) {
    const int from = 4 * (r >> 1) + (r & 1);
    const u64 m = (u64)(uint32_t)__builtin_amdgcn_readlane((int)words, from) | (u64)(uint32_t)__builtin_amdgcn_readlane((int)words, from + 2) << 32;
    v[r] = in_mask(m) ? v[r] : 0.0f;
  }
}
// counts of the lane's 32 entries, a byte each, from the received bits of four workers
__device__ __forceinline__ void mt_add_counts(const uint32_t (&w)[4], uint32_t (&c8)[8]) {
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int q = 0; q < 8; ++q) c8[q] += (((w[u] >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;
}
// .. over the workers first, first + step ..
template <int K>
__device__ __forceinline__ void mt_recount(const PathArgs& a, u64 e0, int first, int step, int wave, int lane, uint32_t (&c8)[8]) {
#pragma unroll
  for (int q = 0; q < 8; ++q) c8[q] = 0;
  for (int i = first; i < a.N; i += 4 * step) {
    uint32_t w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) w[u] = mt_words<K>(a, e0, i + u * step, wave, lane);
    mt_add_counts(w, c8);
  }
}
// .. over all of them, where the received bits of the last four are at hand: with no more of them a chain without another trip to memory
template <int K>
__device__ __forceinline__ void mt_recount(const PathArgs& a, u64 e0, int wave, int lane, const uint32_t (&kept)[4], uint32_t (&c8)[8]) {
  if (a.N > 4) {
    mt_recount<K>(a, e0, 0, 1, wave, lane, c8);
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) c8[q] = 0;
    mt_add_counts(kept, c8);
  }
}
__device__ __forceinline__ void mt_keep(uint32_t (&kept)[4], uint32_t words) {
#pragma unroll
  for (int u = 3; u > 0; --u) kept[u] = kept[u - 1];
  kept[0] = words;
}
template <int K>
__device__ __forceinline__ void mt_store_counts(const PathArgs& a, u64 e0, int wave, int lane, const uint32_t (&c8)[8]) {
  if (!a.count_out) return;
  const int at = ((lane >> 2) << (K - 4)) + (lane & 3) * 32;
  const __amdgpu_buffer_rsrc_t rs = rsrc_of(a.count_out + e0 + wave * 128, MTile<K>::T - wave * 128);
  if (((uintptr_t)a.count_out & 15) == 0) {
    store16<kBufNt>(u32x4v{c8[0], c8[1], c8[2], c8[3]}, rs, at);
    store16<kBufNt>(u32x4v{c8[4], c8[5], c8[6], c8[7]}, rs, at + 16);
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) store_counts4(c8[q], rs, at + q * 4, 0, false);
  }
}
// Sec. 3.4 loss monitoring: what the wavefront's 2048 entries miss, gathered in LDS
__device__ __forceinline__ void mt_add_missing(const uint32_t (&c8)[8], int N, uint32_t* missing, int lane) {
  uint32_t n = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) n = __builtin_amdgcn_sad_u8(c8[q], 0u, n);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o, 64);
  if (lane == 0) atomicAdd(missing, (uint32_t)N * 2048u - n);
}
// the counts of the lane's register r in S2, from the wavefront's counts by word (32 bytes a lane) at `counts`
__device__ __forceinline__ uint32_t mt_count(const uint8_t* counts, int r, int lane) {
  return counts[(4 * (r >> 1) + (r & 1) + 2 * (lane >> 5)) * 32 + (lane & 31)];
}
__device__ __forceinline__ float mt_mean(float sum, uint32_t n, float post) {
  return n ? sum * (post * __builtin_amdgcn_rcpf((float)n)) : 0.0f;
}

// the decode of one block, S2 -> L; nobody reads x any more
template <int K>
__device__ __forceinline__ void mt_decode(float (&v)[32], float* x, int wave, int lane) {
  constexpr int W = MTile<K>::W, TOP = K - 4;   // S2's registers: e5 and e TOP ..
  reg_stages(v, 0, 5);
  mt_s2<K, true>(v, x, wave, lane);
  lds_barrier<W>();
  float* mine = x + wave * 2048;
  {
    const float* p = mine + (lane & 7) * 4 + ((lane >> 3) & 1) * 512 + ((lane >> 4) & 1) * 64 + (lane >> 5) * 1024;
#pragma unroll
    for (int g = 0; g < 8; ++g) {   // registers e3 e4 | e6 e7 e8
      const f32x4v t = *(const f32x4v*)(p + (g & 1) * 32 + (g >> 1) * 128);
      v[4 * g] = t[0]; v[4 * g + 1] = t[1]; v[4 * g + 2] = t[2]; v[4 * g + 3] = t[3];
    }
  }
  reg_stages(v, 0, TOP <= 7 ? 3 : TOP == 8 ? 4 : 5);
  __builtin_amdgcn_wave_barrier();
  // inside the wavefront, from the lowest address bit up: e0 e1 (e2^e3) (e4^e9) e5 e2 e6 e7 e8 e9 e10
  {
    const int at = (lane & 3) + ((lane >> 2) & 1) * (4 + 32) + ((lane >> 3) & 1) * (8 + 512) + ((lane >> 4) & 1) * 16 + (lane >> 5) * 1024;
#pragma unroll
    for (int r = 0; r < 32; ++r) mine[(at ^ ((r & 3) << 2)) + (r >> 2) * 64] = v[r];
  }
  __builtin_amdgcn_wave_barrier();
  {
    const int at = (lane & 7) * 4 + (lane >> 3) * 64;
#pragma unroll
    for (int g = 0; g < 8; ++g) {   // registers e0 e1 | e2 e9 e10
      const f32x4v t = *(const f32x4v*)(mine + (at ^ ((g & 3) << 2)) + (g & 1) * 32 + (g >> 1) * 512);
      v[4 * g] = t[0]; v[4 * g + 1] = t[1]; v[4 * g + 2] = t[2]; v[4 * g + 3] = t[3];
    }
  }
  reg_stages(v, 0, TOP <= 9 ? 3 : TOP == 10 ? 4 : 5);
}


// from the decode's registers to memory: scale, rounding, signs
__device__ __forceinline__ void mt_store(const float (&v)[32], uint32_t signs, const PathArgs& a, u64 first, int lane) {
  const __amdgpu_buffer_rsrc_t out = rsrc_of((const bf16_t*)a.out + first, 4096);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    u32x4v o;
#pragma unroll
    for (int d = 0; d < 4; ++d) o[d] = pack_bf16x2(v[8 * q + 2 * d] * a.scale, v[8 * q + 2 * d + 1] * a.scale);
    flip_pairs(o, signs);
    store16<kBufNt>(o, out, lane * 16 + q * 1024);
  }
}

// The decode of one block by two groups of wavefronts, 16 values a lane: the same stages in the same order, so the same bits.  For
// launches of few blocks and workers, where it is a third of the time: half of the values, and no trip of the means to group 0.
// Entry bits of the positions (E = K - 1; waves of both groups: e9 .. eK-2 from S3 on):
//   S2  as encoded    regs e5, eK-4 .. eK-2   lanes e0 .. e4 e6          group eE, waves e7 ..
//   S3                regs e3 e4 e6 eE        lanes e0 e1 e2 e5 e7 e8
//   L                 regs e0 e1 e2 e7        lanes e3 e4 e5 e6 e8 eE    (2^13: e8 is left there, the one stage across lanes)
// x: 2^K floats for S2 -> S3, then 2^K for S3 -> L, inside the wavefront; nobody reads the former any more, and the latter only ahead of
// the barrier.  `bytes`: the block's signs.
template <int K>
__device__ __forceinline__ void mt_decode_shared(float (&v)[16], float* x, const uint8_t* bytes, const PathArgs& a, u64 e0, int grp, int wave,
                                                 int lane) {
  static_assert(K >= 11 && K <= 13, "at most one stage more than the registers take");
  constexpr int E = K - 1, TOP = K - 4;
  const int all = grp * MTile<K>::W + wave;
  reg_stages(v, 0, 4);
  {
    float* p = x + (lane & 7) * 4 + ((lane >> 3) & 3) + (lane >> 5) * 32 + wave * 128 + (grp << E);
#pragma unroll
    for (int r = 0; r < 16; ++r) p[MTile<K>::s2_reg(r)] = v[r];
  }
  lds_barrier<2>();
  {
    const float* p = x + (lane & 7) * 4 + ((lane >> 3) & 1) * 64 + ((lane >> 4) & 1) * 128 + (lane >> 5) * 256 + all * 512;
#pragma unroll
    for (int g = 0; g < 4; ++g) {   // registers e3 e4 | e6 eE
      const f32x4v t = *(const f32x4v*)(p + (g & 1) * 32 + ((g >> 1) << E));
      v[4 * g] = t[0]; v[4 * g + 1] = t[1]; v[4 * g + 2] = t[2]; v[4 * g + 3] = t[3];
    }
  }
  reg_stage<3>(v);
  reg_stages(v, 0, 3);
  // from the lowest address bit up: e0 e1 (e2^e3) e5 (e7^e4) (e8^e6) e3 e4 e6 eE
  float* mine = x + MTile<K>::T + all * 1024;
#pragma unroll
  for (int r = 0; r < 16; ++r) mine[(lane ^ ((r & 1) * 4 + ((r >> 1) & 1) * 16 + ((r >> 2) & 1) * 32)) + r * 64] = v[r];
  __builtin_amdgcn_wave_barrier();
  {
    const int at = (lane & 1) * (4 + 64) + ((lane >> 1) & 1) * (16 + 128) + ((lane >> 2) & 1) * 8 + ((((lane >> 3) ^ (lane >> 4)) & 1) * 32) +
                   ((lane >> 3) & 1) * 256 + (lane >> 5) * 512;
#pragma unroll
    for (int g = 0; g < 4; ++g) {   // registers e0 e1 | e2 e7
      const f32x4v t = *(const f32x4v*)(mine + (at ^ ((g & 1) * 4 + (g >> 1) * 16)));
      v[4 * g] = t[0]; v[4 * g + 1] = t[1]; v[4 * g + 2] = t[2]; v[4 * g + 3] = t[3];
    }
  }
  if constexpr (TOP > 7) reg_stage<3>(v);
  if constexpr (TOP > 8) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float o = __shfl_xor(v[r], 16, 64);
      v[r] = lane & 16 ? o - v[r] : v[r] + o;
    }
  }
  reg_stages(v, 0, 3);
  const int at = (lane & 15) + ((lane >> 4) & 1) * 32 + all * 64 + ((lane >> 5) << (E - 3));   // of 8 entries
  uint32_t signs = pair_signs((uint32_t)bytes[at] | (uint32_t)bytes[at + 16] << 8);
  const __amdgpu_buffer_rsrc_t out = rsrc_of((const bf16_t*)a.out + e0, MTile<K>::T * 2);
#pragma unroll
  for (int q = 0; q < 2; ++q) {   // e7
    u32x4v o;
#pragma unroll
    for (int d = 0; d < 4; ++d) o[d] = pack_bf16x2(v[8 * q + 2 * d] * a.scale, v[8 * q + 2 * d + 1] * a.scale);
    flip_pairs(o, signs);
    store16<kBufNt>(o, out, at * 16 + q * 256);
  }
}

template <int K, bool TOTAL>
__device__ __forceinline__ void fused_bf16_tile(const PathArgs& a, u64 unit) {
  typedef MTile<K> M;
  constexpr int W = M::W, T = M::T, R = M::R;
  __shared__ __align__(16) float x[T];
  __shared__ uint32_t missing;
  const int wave = wave_id(), lane = lane_id(), N = a.N;
  const u64 e0 = unit * T, ew = e0 + (u64)wave * 2048;
  InFlight f;
  mt_request<K>(a, e0, 0, wave, lane, f);
  const uint32_t signs = mt_signs(a.seed, a.base + ew, (uint8_t*)(x + wave * 2048), lane);
  Operand h = mt_operand(lane);
  if (TOTAL && threadIdx.x == 0) missing = 0;   // behind barriers when it is added to

  float acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0f;
  bool clean = true;   // nothing of this wavefront's S2 part was lost so far
  for (int i = 0; i < N; ++i) {
    float v[R];
    int lane_t = lane;   // addresses formed here, not kept in registers all along
    asm volatile("" : "+v"(lane_t));
    mt_encode_s1(f.q, signs, h, v);
    const uint32_t words = f.words;
    mt_request<K>(a, e0, i + 1, wave, lane, f);
    mt_store_s1(v, x, wave, lane_t);
    lds_barrier<W>();
    mt_s2<K, false>(v, x, wave, lane_t);
    // Everyone has read.  Here, where all wavefronts are together anyway: from here to the next stores they may drift apart
    lds_barrier<W>();
    mt_encode_s2<K>(v, a.scale);
    if (!all_arrived(words)) {
      clean = false;
      mt_mask(v, words);
    }
    // one conversion per value with the result in the HIGH half (the low half converts a zero): that is the fp32 pattern of the
    // rounded value, no unpacking
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] += __builtin_bit_cast(float, pack_bf16x2(0.0f, v[r]));
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- counts: the loop above carries none, a wavefront that saw a loss reads its words again
  uint32_t c8[8];
  if (clean) {
#pragma unroll
    for (int q = 0; q < 8; ++q) c8[q] = (uint32_t)N * 0x01010101u;
  } else {
    mt_recount<K>(a, e0, 0, 1, wave, lane, c8);
  }
  mt_store_counts<K>(a, e0, wave, lane, c8);
  if (TOTAL && a.total_out && !clean) mt_add_missing(c8, N, &missing, lane);
  // ---- mean over what arrived
  const float post = K & 1 ? 1.0f : a.scale;
  if (clean) {
    const float f = post * __builtin_amdgcn_rcpf((float)N);
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] *= f;
  } else {
    uint8_t* mine = (uint8_t*)(x + wave * 2048);
    *(uint4*)(mine + lane * 32) = make_uint4(c8[0], c8[1], c8[2], c8[3]);
    *(uint4*)(mine + lane * 32 + 16) = make_uint4(c8[4], c8[5], c8[6], c8[7]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = mt_mean(acc[r], mt_count(mine, r, lane), post);
  }
  lds_barrier<W>();   // the counts are read, what is missing is there
  if (TOTAL && a.total_out && threadIdx.x == 0) add_total(a, unit == 0, missing);
  __builtin_amdgcn_sched_barrier(0);
  mt_decode<K>(acc, x, wave, lane);
  mt_store(acc, signs, a, ew, lane);
}

// For launches that leave CUs idle: G groups of W wavefronts encode G workers side by side.  The encoded values go through LDS as
// the bf16 pairs that they are, and group g adds those of its share of the registers over the workers, in order: the same
// operations in the same order as above.  Group 0 decodes.  (Two groups up to 2^13: fused_bf16_pair.)
template <int K, int G, bool TOTAL>
__device__ __forceinline__ void fused_bf16_groups(const PathArgs& a, u64 unit) {
  typedef MTile<K> M;
  constexpr int W = M::W, T = M::T, R = M::R, D = 16 / G;   // D: pairs of a lane and a share
  static_assert(G >= 2 && G <= 16, "a share is at least a pair");
  __shared__ __align__(16) float x[G][T];
  __shared__ uint32_t missing, lossy;   // lossy: something was lost somewhere in the block
  const int wave_all = wave_id(), lane = lane_id(), N = a.N, grp = wave_all / W, wave = wave_all % W;
  const u64 e0 = unit * T, ew = e0 + (u64)wave * 2048;
  InFlight f;
  mt_request<K>(a, e0, grp, wave, lane, f);
  const uint32_t signs = mt_signs(a.seed, a.base + ew, (uint8_t*)(x[grp] + wave * 2048), lane);
  Operand h = mt_operand(lane);
  if (TOTAL && threadIdx.x == 0) missing = 0;   // behind barriers when it is added to
  float acc[2 * D];
#pragma unroll
  for (int r = 0; r < 2 * D; ++r) acc[r] = 0.0f;
  if (threadIdx.x == 0) lossy = 0;
  typedef uint32_t pairs_t __attribute__((ext_vector_type(D < 4 ? D : 4)));
  constexpr int V = D < 4 ? D : 4;   // pairs of one access to LDS
  uint32_t words = 0;   // received bits of the group's worker in work
  for (int first = 0; first < N; first += G) {
    const bool works = first + grp < N;
    float v[R];
    if (works) {
      mt_encode_s1(f.q, signs, h, v);
      words = f.words;
      mt_request<K>(a, e0, first + grp + G, wave, lane, f);
      mt_store_s1(v, x[grp], wave, lane);
    }
    lds_barrier<2>();
    if (works) mt_s2<K, false>(v, x[grp], wave, lane);
    lds_barrier<2>();
    if (works) {
      mt_encode_s2<K>(v, a.scale);
      if (!all_arrived(words)) {
        if (lane == 0) lossy = 1;   // (zeroed ahead of the barriers above)
        mt_mask(v, words);
      }
      uint32_t* to = (uint32_t*)x[grp] + wave * (16 * 64) + lane * V;   // by access
#pragma unroll
      for (int j = 0; j < 16 / V; ++j) {
        pairs_t t;
#pragma unroll
        for (int d = 0; d < V; ++d) t[d] = pack_bf16x2(v[2 * (j * V + d)], v[2 * (j * V + d) + 1]);
        *(pairs_t*)(to + j * 64 * V) = t;
      }
    }
    lds_barrier<2>();
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (first + g < N) {
        const uint32_t* from = (const uint32_t*)x[g] + wave * (16 * 64) + grp * (64 * D) + lane * V;
#pragma unroll
        for (int j = 0; j < D / V; ++j) {
          const pairs_t t = *(const pairs_t*)(from + j * 64 * V);
#pragma unroll
          for (int d = 0; d < V; ++d) {
            acc[2 * (j * V + d)] += bf16_lo(t[d]);
            acc[2 * (j * V + d) + 1] += bf16_hi(t[d]);
          }
        }
      }
    }
    lds_barrier<2>();
  }
  // ---- counts, mean over what arrived.  The last round ended in a barrier behind which everyone sees `lossy`
  float* means = &x[0][0] + G * W * 512;   // in S2, by register
  const float post = K & 1 ? 1.0f : a.scale;
  if (lossy == 0) {
    const float f = post * __builtin_amdgcn_rcpf((float)N);
#pragma unroll
    for (int r = 0; r < 2 * D; ++r) means[(wave * R + grp * 2 * D + r) * 64 + lane] = acc[r] * f;
    if (grp == 0) {
      uint32_t c8[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) c8[q] = (uint32_t)N * 0x01010101u;
      mt_store_counts<K>(a, e0, wave, lane, c8);
    }
    if (TOTAL && a.total_out && threadIdx.x == 0) add_total(a, unit == 0, 0);
  } else {   // the group's workers, then all of them
    uint32_t* counts = (uint32_t*)&x[0][0];   // [group][wavefront][lane][8]
    static_assert(G * W * 512 + T <= G * T, "counts and means fit");
    uint32_t c8[8] = {};
    if (N <= G) {   // one round: they are at hand
      const uint32_t one[4] = {words, 0, 0, 0};
      mt_add_counts(one, c8);
    } else {
      mt_recount<K>(a, e0, grp, G, wave, lane, c8);
    }
    *(uint4*)(counts + (wave_all * 64 + lane) * 8) = make_uint4(c8[0], c8[1], c8[2], c8[3]);
    *(uint4*)(counts + (wave_all * 64 + lane) * 8 + 4) = make_uint4(c8[4], c8[5], c8[6], c8[7]);
    lds_barrier<2>();
    if (grp == 0) {
#pragma unroll
      for (int g = 1; g < G; ++g) {
        const uint32_t* from = counts + ((g * W + wave) * 64 + lane) * 8;
        const uint4 lo = *(const uint4*)from, hi = *(const uint4*)(from + 4);
        c8[0] += lo.x; c8[1] += lo.y; c8[2] += lo.z; c8[3] += lo.w;
        c8[4] += hi.x; c8[5] += hi.y; c8[6] += hi.z; c8[7] += hi.w;
      }
      *(uint4*)(counts + (wave * 64 + lane) * 8) = make_uint4(c8[0], c8[1], c8[2], c8[3]);
      *(uint4*)(counts + (wave * 64 + lane) * 8 + 4) = make_uint4(c8[4], c8[5], c8[6], c8[7]);
      mt_store_counts<K>(a, e0, wave, lane, c8);
      if (TOTAL && a.total_out) mt_add_missing(c8, N, &missing, lane);
    }
    lds_barrier<2>();
    if (TOTAL && a.total_out && threadIdx.x == 0) add_total(a, unit == 0, missing);
#pragma unroll
    for (int r = 0; r < 2 * D; ++r) {
      const int reg = grp * 2 * D + r;
      means[(wave * R + reg) * 64 + lane] = mt_mean(acc[r], mt_count((const uint8_t*)(counts + wave * 512), reg, lane), post);
    }
  }
  lds_barrier<2>();
  if (grp > 0) return;   // (a barrier waits for the wavefronts that are left)
  float v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = means[(wave * R + r) * 64 + lane];
  lds_barrier<2>();
  mt_decode<K>(v, &x[0][0], wave, lane);
  mt_store(v, signs, a, ew, lane);
}

// Two groups of W wavefronts, for few workers (up to 2^13): a worker each at a time, half of the registers each in the sum and in the
// decode, the same bits again.  A launch of few blocks is one chain from the first load to the last store, so every trip counts:
// the pairs have a place in LDS of their own, which leaves two barriers a round, and every wavefront has the received bits of both
// workers, so that counts and means need neither a barrier nor (up to four workers) another trip to memory.  us, four barriers a round and
// the received bits read again -> this, 1 % loss: N = 2, 65 blocks, 2^11 5.3 -> 4.9, 2^12 5.9 -> 5.5, 2^13 7.2 -> 6.6.
template <int K, bool TOTAL>
__device__ __forceinline__ void fused_bf16_pair(const PathArgs& a, u64 unit) {
  typedef MTile<K> M;
  constexpr int W = M::W, T = M::T, R = M::R;
  __shared__ __align__(16) float x[2][T];
  __shared__ __align__(16) u32x4v pairs[2][W][4][64];
  __shared__ __align__(16) uint8_t sign_bytes[T / 8];
  __shared__ uint32_t missing;
  const int wave_all = wave_id(), lane = lane_id(), N = a.N, grp = wave_all / W, wave = wave_all % W;
  const u64 e0 = unit * T, ew = e0 + (u64)wave * 2048;
  InFlight f;
  mt_request<K>(a, e0, grp, wave, lane, f);
  uint32_t other = mt_words<K>(a, e0, grp ^ 1, wave, lane);
  // (both groups write the same bytes to the same place)
  const uint32_t signs = mt_signs(a.seed, a.base + ew, sign_bytes + wave * 256, lane);
  Operand h = mt_operand(lane);
  if (TOTAL && threadIdx.x == 0) missing = 0;   // behind barriers when it is added to
  float acc[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  bool clean = true;   // nothing of this wavefront's S2 part was lost so far, from either group's workers
  uint32_t kept[4] = {0, 0, 0, 0};
  for (int first = 0; first < N; first += 2) {
    const bool works = first + grp < N, whole = !works || all_arrived(f.words);
    float v[R];
    const uint32_t words = f.words;
    clean = clean && whole && (first + (grp ^ 1) >= N || all_arrived(other));
    mt_keep(kept, words);
    mt_keep(kept, other);
    if (works) mt_encode_s1(f.q, signs, h, v);
    mt_request<K>(a, e0, first + 2 + grp, wave, lane, f);
    other = mt_words<K>(a, e0, first + 2 + (grp ^ 1), wave, lane);
    if (works) mt_store_s1(v, x[grp], wave, lane);
    lds_barrier<2>();
    if (works) {
      mt_s2<K, false>(v, x[grp], wave, lane);
      mt_encode_s2<K>(v, a.scale);
      if (!whole) mt_mask(v, words);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        u32x4v t;
#pragma unroll
        for (int d = 0; d < 4; ++d) t[d] = pack_bf16x2(v[8 * j + 2 * d], v[8 * j + 2 * d + 1]);
        pairs[grp][wave][j][lane] = t;
      }
    }
    lds_barrier<2>();   // the pairs are there; and everyone has read x
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      if (first + g < N) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const u32x4v t = pairs[g][wave][2 * grp + j][lane];
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            acc[8 * j + 2 * d] += bf16_lo(t[d]);
            acc[8 * j + 2 * d + 1] += bf16_hi(t[d]);
          }
        }
      }
    }
  }
  // ---- counts, mean over what arrived
  uint32_t c8[8];
  const float post = K & 1 ? 1.0f : a.scale;
  if (clean) {
#pragma unroll
    for (int q = 0; q < 8; ++q) c8[q] = (uint32_t)N * 0x01010101u;
    const float f = post * __builtin_amdgcn_rcpf((float)N);
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] *= f;
  } else {
    mt_recount<K>(a, e0, wave, lane, kept, c8);
    uint8_t* mine = (uint8_t*)x[1] + wave_all * 2048;
    *(uint4*)(mine + lane * 32) = make_uint4(c8[0], c8[1], c8[2], c8[3]);
    *(uint4*)(mine + lane * 32 + 16) = make_uint4(c8[4], c8[5], c8[6], c8[7]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = mt_mean(acc[r], mt_count(mine, grp * 16 + r, lane), post);
    __builtin_amdgcn_wave_barrier();
  }
  if (grp == 0) {
    mt_store_counts<K>(a, e0, wave, lane, c8);
    if (TOTAL && a.total_out && !clean) mt_add_missing(c8, N, &missing, lane);
  }
  mt_decode_shared<K>(acc, &x[0][0], sign_bytes, a, e0, grp, wave, lane);
  if (TOTAL && a.total_out && threadIdx.x == 0) add_total(a, unit == 0, missing);   // (complete since the decode's barrier)
}

template <int K>
__global__ __launch_bounds__(MTile<K>::THREADS) __attribute__((amdgpu_waves_per_eu(4)))
void k_fused_bf16(PathArgs a) {
  fused_bf16_tile<K, false>(a, blockIdx.x);
}
template <int K>
__global__ __launch_bounds__(MTile<K>::THREADS) __attribute__((amdgpu_waves_per_eu(4)))
void k_fused_bf16_batched(BatchArgs ba) {
  PathArgs a;
  const u64 unit = bucket_of(ba, a, blockIdx.x);
  fused_bf16_tile<K, true>(a, unit);
}
// 128 registers: with more the compiler lets the products end in accumulation registers, and every value is copied from there
template <int K, int G>
__global__ __launch_bounds__(MTile<K>::THREADS * G) __attribute__((amdgpu_num_vgpr(128))) void k_fused_bf16_groups(PathArgs a) {
  if constexpr (G == 2 && K <= 13) fused_bf16_pair<K, false>(a, blockIdx.x);
  else fused_bf16_groups<K, G, false>(a, blockIdx.x);
}
template <int K, int G>
__global__ __launch_bounds__(MTile<K>::THREADS * G) __attribute__((amdgpu_num_vgpr(128))) void k_fused_bf16_groups_batched(BatchArgs ba) {
  PathArgs a;
  const u64 unit = bucket_of(ba, a, blockIdx.x);
  if constexpr (G == 2 && K <= 13) fused_bf16_pair<K, true>(a, unit);
  else fused_bf16_groups<K, G, true>(a, unit);
}

}  // namespace ordev

// The fused path (OptiReduce Sec. 3.3 encode, Sec. 3.1.1 aggregation, Sec. 3.3 / Sec. 4 decode) of fp32 slices for blocks of
// up to 2^11 entries: one workgroup per tile of T = 2^max(10, k) entries, from N raw slices to the decoded mean.  (bf16, whose
// encoded values are rounded worker by worker, few workers at 2^11 and below 2^10, and 2^12 .. 2^14: rht_fused_each.hpp.)
//
// The encode is linear and the signs are the same for every worker, so the workers whose copy of the block arrived
// WHOLE are added up first, as they come from memory, and encoded once.  A worker that lost something in the tile is
// encoded by itself and added under its received bits.  With packet loss that leaves 1 + (workers with a loss in this
// tile) transforms where there were N, and the bulk of the work is a plain streaming sum: 16 bytes a lane per load, no
// barrier in between.  The value of an entry is (sum over whole workers, in increasing order, encoded) + (each of the
// others, in increasing order) in both modes below.  Blocks that share a tile (K = 0) are looked at one by one: a worker that lost
// something in the tile is encoded with zeros in the blocks that it has whole, so no block's value depends on its neighbours'.
//
// Positions (A also of the reduce + decode of larger blocks; V entries per 16 bytes: 4 fp32, 8 bf16; VB = log2 V; 16 entries a lane, 1024 a wavefront)
//   A  as loaded and stored: register bits = entry bits 0 .. VB-1 and VB+6 .. 9, lane = VB .. VB+5, wavefront = 10 ..
//   M  register bits = entry bits VB .. VB+3, lane bits (from 0) = VB+4, VB+5, 0 .. VB-1, VB+6 .. 9, wavefront = 10 ..
//   B  ("wire") lane = entry bits 0 .. 5: a register is 64 consecutive entries, its received bits one lane mask;
//      register bits = the entry bits not transformed in A and M (U0 = VB+4, U1 = VB+5 and the wavefront bits).
// Every stage runs as a plain add / subtract between registers.  Going from A to M stays inside the
// wavefront (no barrier), M to B is the exchange between wavefronts.  Entry e sits in LDS at e + (e >> (VB+4) << VB):
// the 32 lanes of either half of a wavefront then fall into 32 different banks in M and B.
#pragma once
#include "rht_kernels.hpp"

namespace ordev {

template <int K, class In>
struct FTile {
  static constexpr int VB = sizeof(In) == 4 ? 2 : 3, V = 1 << VB, C = 16 / V;   // C loads of 16 bytes a lane
  static constexpr int KT = K ? K : 10, T = 1 << KT, Q = KT - 10, W = 1 << Q;
  static_assert(Q == 0 || Q == 1 || Q == 4, "tiles of 2^10, 2^11 and 2^14 entries; the last ones only in A");
  static constexpr int U0 = VB + 4, U1 = VB + 5;
  static constexpr int O0 = VB == 2 ? 8 : 6, O1 = 9;     // the bits of 6..9 other than U0, U1
  static constexpr int PART = 1024 + 64;                 // floats of a wavefront's entries in LDS
  static constexpr int ROW = (1 << U0) + V;              // floats from one value of entry bit U0 to the next
  static constexpr int reg_bit(int i) {                  // entry bit that register bit i stands for in B
    return Q == 0 ? (i == 0 ? U0 : i == 1 ? U1 : i == 2 ? O0 : O1) : (i == 0 ? U0 : i == 1 ? U1 : i == 2 ? 10 : O0);
  }
  static constexpr int wave_bit(int) {                 // and bit i of the wavefront number
    return O1;
  }
  static constexpr int kLast = Q == 0 ? 2 : 3;   // register bits that are left to transform in B
  static constexpr int reg_entry(int r) {
    int e = 0;
    for (int i = 0; i < 4; ++i) e |= ((r >> i) & 1) << reg_bit(i);
    return e;
  }
  static constexpr int padded(int e) { return e + (e >> U0 << VB); }
};
template <int K, class In>
__device__ __forceinline__ int wire_wave_entry(int wave) {
  int e = 0;
#pragma unroll
  for (int i = 0; i < FTile<K, In>::Q; ++i) e |= ((wave >> i) & 1) << FTile<K, In>::wave_bit(i);
  return e;
}
template <int W>
__device__ __forceinline__ void tile_barrier() {   // tiles of one wavefront need none: its LDS accesses are in order
  if constexpr (W > 1) __syncthreads();
  else __builtin_amdgcn_wave_barrier();
}

// ---- the register stages of the three layouts (K = 0: only the entry bits below k)
template <int K, class In>
__device__ __forceinline__ void stages_a(float (&v)[16], int k) {
  constexpr int VB = FTile<K, In>::VB;
  reg_stage<0>(v);
  reg_stage<1>(v);
  if (VB == 3 || K || k > 8) reg_stage<2>(v);
  if (K || k > 9) reg_stage<3>(v);
}
template <int K, class In>
__device__ __forceinline__ void stages_m(float (&v)[16], int k) {
  constexpr int VB = FTile<K, In>::VB;
  reg_stage<0>(v);
  reg_stage<1>(v);
  if (VB == 2 || K || k > VB + 2) reg_stage<2>(v);
  if (K || k > VB + 3) reg_stage<3>(v);
}
template <int K, class In>
__device__ __forceinline__ void stages_b(float (&v)[16], int k) {
  typedef FTile<K, In> F;
  if (K || k > F::U0) reg_stage<0>(v);
  if (K || k > F::U1) reg_stage<1>(v);
  if constexpr (F::kLast > 2) reg_stage<2>(v);
}

// ---- LDS accesses of the three layouts; x = the tile's buffer of W * PART floats
typedef float f32x4v __attribute__((ext_vector_type(4)));
template <int K, class In, bool STORE>
__device__ __forceinline__ void lds_a(float (&v)[16], float* x, int wave, int lane) {
  typedef FTile<K, In> F;
  float* p = x + wave * F::PART + F::padded(lane * F::V);
#pragma unroll
  for (int r = 0; r < 16; r += 4) {
    f32x4v* q = (f32x4v*)(p + F::padded((r >> F::VB) * 64 * F::V) + (r & (F::V - 1)));
    if constexpr (STORE) {
      *q = f32x4v{v[r], v[r + 1], v[r + 2], v[r + 3]};
    } else {
      const f32x4v t = *q;
      v[r] = t[0]; v[r + 1] = t[1]; v[r + 2] = t[2]; v[r + 3] = t[3];
    }
  }
}
template <int K, class In, bool STORE>
__device__ __forceinline__ void lds_m(float (&v)[16], float* x, int wave, int lane) {
  static_assert(FTile<K, In>::Q <= 1, "tiles of 2^14 entries have no layouts but A");
  typedef FTile<K, In> F;
  float* p = x + wave * F::PART + (lane & 3) * F::ROW + ((lane >> 2) & (F::V - 1)) + (lane >> (2 + F::VB)) * (4 * F::ROW);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if constexpr (STORE) p[r << F::VB] = v[r]; else v[r] = p[r << F::VB];
  }
}
template <int K, class In, bool STORE>
__device__ __forceinline__ void lds_b(float (&v)[16], float* x, int wave, int lane) {
  static_assert(FTile<K, In>::Q <= 1, "tiles of 2^14 entries have no layouts but A");
  typedef FTile<K, In> F;
  float* p = x + F::padded(wire_wave_entry<K, In>(wave)) + lane;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if constexpr (STORE) p[F::padded(F::reg_entry(r))] = v[r]; else v[r] = p[F::padded(F::reg_entry(r))];
  }
}

// Unscaled transform, A -> B.  The caller has made sure that nobody still reads `x`; one barrier inside.
template <int K, class In>
__device__ __forceinline__ void to_wire(float (&v)[16], float* x, int wave, int lane, int k) {
  stages_a<K, In>(v, k);
  lds_a<K, In, true>(v, x, wave, lane);
  __builtin_amdgcn_wave_barrier();
  lds_m<K, In, false>(v, x, wave, lane);
  stages_m<K, In>(v, k);
  lds_m<K, In, true>(v, x, wave, lane);
  tile_barrier<FTile<K, In>::W>();
  lds_b<K, In, false>(v, x, wave, lane);
  stages_b<K, In>(v, k);
}
// B -> A, likewise
template <int K, class In>
__device__ __forceinline__ void from_wire(float (&v)[16], float* x, int wave, int lane, int k) {
  stages_b<K, In>(v, k);
  lds_b<K, In, true>(v, x, wave, lane);
  tile_barrier<FTile<K, In>::W>();
  lds_m<K, In, false>(v, x, wave, lane);
  stages_m<K, In>(v, k);
  lds_m<K, In, true>(v, x, wave, lane);
  __builtin_amdgcn_wave_barrier();
  lds_a<K, In, false>(v, x, wave, lane);
  stages_a<K, In>(v, k);
}

// Sign bits of this lane's 16 entries in A (bit r = register r); `g` = sign-stream index of the wavefront's first
// entry.  Lanes 0..7 hold one Philox counter each; 128 bytes of LDS of the wavefront's own spread the words.
template <int K, class In>
__device__ __forceinline__ uint32_t lane_signs(u64 seed, u64 g, float* x, int wave, int lane) {
  typedef FTile<K, In> F;
  const u64 ctr = (g >> 7) + (u64)(lane & 7);
  const u32x4 w = philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u, (uint32_t)seed, (uint32_t)(seed >> 32));
  uint32_t* words = (uint32_t*)(x + wave * F::PART);
  if (lane < 8) *(uint4*)(words + lane * 4) = make_uint4(w.a, w.b, w.c, w.d);
  __builtin_amdgcn_wave_barrier();
  uint32_t bits = 0;
#pragma unroll
  for (int c = 0; c < F::C; ++c) {
    const uint32_t t = words[c * 2 * F::V + (lane >> (5 - F::VB))] >> ((lane & ((32 >> F::VB) - 1)) << F::VB);
    bits |= (t & ((1u << F::V) - 1)) << (c * F::V);
  }
  __builtin_amdgcn_wave_barrier();
  return bits;
}
__device__ __forceinline__ float flip_sign(float v, uint32_t bits, int r) {   // bit r of `bits` set: -v
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) ^ ((bits << (31 - r)) & 0x80000000u));
}

// ---- entries as loaded: 16 (C loads of 16 bytes)
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float bf16_lo(uint32_t p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t p) { return __builtin_bit_cast(float, p & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {   // round to nearest even, lo in bits 0..15
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, b2));
}
template <class In> struct Raw16 { u32x4v q[sizeof(In) == 4 ? 4 : 2]; };

template <class In> __device__ __forceinline__ float entry_of(const Raw16<In>& x, int r) {
  if constexpr (sizeof(In) == 4) return __builtin_bit_cast(float, (uint32_t)x.q[r >> 2][r & 3]);
  else return r & 1 ? bf16_hi(x.q[r >> 3][(r >> 1) & 3]) : bf16_lo(x.q[r >> 3][(r >> 1) & 3]);
}
// descriptor of `bytes` bytes at p; 0 bytes: loads return zero without touching memory
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, bytes, 0x00020000);
}

// 16 bytes a lane, `off` bytes past the descriptor's base.  The offset is never handed over in a scalar register: hipcc 7.2
// puts no wait between such a 16-byte store and a vector instruction that writes its data registers again, and on this
// chip the new value then reached memory now and then (counts of 8 read back as 8.0f).  Without one it does wait.
template <int AUX>
__device__ __forceinline__ void store16(u32x4v x, __amdgpu_buffer_rsrc_t rs, int off) {
  __builtin_amdgcn_raw_buffer_store_b128(x, rs, off, 0, AUX);
}

// One bit per run of 2^log entries (up to 32 of them): the runs of the block of 2^k that run `at` lies in.
__device__ __forceinline__ uint32_t block_runs(int at, int k, int log) {
  const int g = 1 << (k - log);
  return (0xFFFFFFFFu >> (32 - g)) << (at & ~(g - 1));
}

// The workers in the order they are taken: first those that lost something in the tile, then the others, each kind in
// increasing order.  `marks`: one bit per worker in LDS, set where something is missing; `order`: 256 bytes of LDS (every
// wavefront writes the same values and reads back its own).  The result holds entry j in byte j / 64 of lane j % 64.
__device__ __forceinline__ uint32_t order_workers(const uint32_t* marks, uint8_t* order, int N, int lossy, int lane) {
  for (int i = lane; i < N; i += 64) {
    int below = 0;   // workers with a loss before i
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int bits = i - 32 * q;
      if (bits > 0) below += __builtin_popcount(bits >= 32 ? marks[q] : marks[q] & ((1u << bits) - 1));
    }
    const bool lost = (marks[i >> 5] >> (i & 31)) & 1;
    order[lost ? below : lossy + i - below] = (uint8_t)i;
  }
  __builtin_amdgcn_wave_barrier();
  return (uint32_t)order[lane] | ((uint32_t)order[64 + lane] << 8) | ((uint32_t)order[128 + lane] << 16) | ((uint32_t)order[192 + lane] << 24);
}

// Two ways to go through the workers; the value of every entry comes from the same operations in the same order.
//   STREAM  in increasing order, two workers' loads in flight ahead of the one in work, whatever their kind.
//   GROUPS  for launches too small to fill the chip: four times the wavefronts.  The sum over the whole workers is spread
//           four entries a lane (eight workers' loads in flight at once), then the four groups of W wavefronts encode four
//           workers side by side (that sum is the last one) and group 0 adds the results in order and decodes.
enum FusedMode { STREAM, GROUPS };
constexpr int kGroups = 4;

// SLOTS > 1 (tiles of one wavefront): the workgroup's wavefronts serve SLOTS tiles, for the sake of the arrival totals: one
// atomic per workgroup (add_total).
// SPLIT: blocks below 2^10, several to a tile.
template <int K, int MODE, bool SPLIT, int SLOTS = 1>
__device__ __forceinline__ void fused_tile(const PathArgs& a, u64 first_unit, u64 units) {
  typedef float In;
  typedef FTile<K, In> F;
  constexpr int W = F::W, T = F::T, ES = sizeof(In), G = MODE == GROUPS ? kGroups : 1;
  static_assert(!SPLIT || K == 0, "larger blocks are whole tiles");
  static_assert(F::Q <= 1, "tiles of one or two wavefronts: no sign from DPP stages");
  static_assert(SLOTS == 1 || (W == 1 && G == 1), "several tiles per workgroup: tiles of one wavefront");
  constexpr int BUFS = MODE == GROUPS ? G : SLOTS;
  __shared__ __align__(16) float xbuf[BUFS][W * F::PART];
  __shared__ __align__(16) float ybuf[G > 1 ? G - 1 : 1][G > 1 ? 1024 * W : 4];   // GROUPS: what groups 1.. hand to group 0
  __shared__ __align__(16) uint8_t counts[G * SLOTS][T];
  __shared__ uint32_t marks_all[SLOTS][8];
  __shared__ uint8_t order_all[SLOTS][MODE == STREAM ? 1 : 256];
  __shared__ uint2 missing16[MODE == GROUPS && SPLIT ? 256 : 1];   // per worker with a loss: the runs of 16 entries that miss something
  __shared__ uint32_t missing[2];   // what the workgroup's tiles miss; how many of its wavefronts have added theirs
  const int wave_all = wave_id(), lane = lane_id();
  const int slot = SLOTS > 1 ? wave_all : 0;
  const int grp = G == 1 ? 0 : wave_all / W, wave = SLOTS > 1 ? 0 : G == 1 ? wave_all : wave_all % W;
  if constexpr (SLOTS > 1) {
    if (threadIdx.x < 2) missing[threadIdx.x] = 0;
    __syncthreads();   // the only one: from here on every wavefront is on its own
  }
  const u64 unit = first_unit + slot;
  const int tiles = units - first_unit < SLOTS ? (int)(units - first_unit) : SLOTS;   // of this workgroup
  if (SLOTS > 1 && slot >= tiles) return;
  uint32_t* marks = marks_all[slot];
  uint8_t* order = order_all[slot];
  const int N = a.N, k = a.k;
  const u64 L = a.n_pad, e0 = unit * T, ew = e0 + (u64)wave * 1024;   // first entry of the tile / of the wavefront's part
  // K = 0: the last tile may be cut short (by whole blocks of at least 32 entries)
  const int left = K ? 1024 : (L - e0 < 1024 ? (int)(L - e0) : 1024);
  const u64 row_bytes = L >> 3;
  float* x = xbuf[SLOTS > 1 ? slot : grp];
  if (SLOTS > 1 ? lane < 8 : threadIdx.x < 8) marks[lane & 7] = 0;
  if (SLOTS == 1 && threadIdx.x == 0) missing[0] = 0;

  // ---- loads; no such worker (i < 0 or >= N): zeros, without touching memory.  The whole offset is in the vector operand, which the
  // range check covers by any reading of it: what lies past a tile that is cut short (K = 0) is not read
  auto request = [&](int i, Raw16<In>& r) {   // the lane's entries in A
    const bool there = i >= 0 && i < N;
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const In*)a.in + (u64)(there ? i : 0) * L + ew, there ? left * ES : 0);
#pragma unroll
    for (int c = 0; c < F::C; ++c) r.q[c] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16 + c * 1024, 0, kBufNt));
  };
  const u64 e4 = ew + (u64)(grp * 256);   // (as a runtime part of the offset: 2 % slower)
  const int bytes4 = left > grp * 256 ? (left - grp * 256) * ES : 0;
  auto request4 = [&](int i, u32x4v& r) {   // four entries from 256 grp + 4 lane of the wavefront's part
    const bool there = i >= 0 && i < N;
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const In*)a.in + (u64)(there ? i : 0) * L + e4, there ? bytes4 : 0);
    r = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, 0, 0));
  };
  auto request_bits = [&](int i) {   // received bits of the lane's 16 entries from 16 lane of the wavefront's part on
    const bool there = i >= 0 && i < N;
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const uint8_t*)a.masks + (u64)(there ? i : 0) * row_bytes + (ew >> 3), there ? left >> 3 : 0);
    return (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, lane * 2, 0, 0);
  };
  int word_off;   // byte offset of mask word (lane & 1) of register (lane >> 1) & 15 in B
  {
    int e = wire_wave_entry<K, In>(wave) + (lane & 1) * 32;
#pragma unroll
    for (int i = 0; i < 4; ++i) e |= ((lane >> (i + 1)) & 1) << F::reg_bit(i);
    word_off = e >> 3;
  }
  auto request_words = [&](int i) {
    const bool there = i >= 0 && i < N;
    const __amdgpu_buffer_rsrc_t rs =
        rsrc_of((const uint8_t*)a.masks + (u64)(there ? i : 0) * row_bytes + (e0 >> 3), there ? (K ? T : left) >> 3 : 0);
    return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, word_off, 0, 0);
  };

  // the received bits are asked for first (answers come in order), then the first workers' entries
  constexpr int U = 8;
  Raw16<In> ra, rb;
  u32x4v q4[MODE == GROUPS ? U : 1];
  uint32_t ma = 0, mb = 0, bits[U];
#pragma unroll
  for (int u = 0; u < U; ++u) bits[u] = request_bits(grp + u * G);
  if constexpr (MODE == STREAM) {
    request(0, ra);
    ma = request_words(0);
    request(1, rb);
    mb = request_words(1);
  }
  if constexpr (MODE == GROUPS) {
#pragma unroll
    for (int u = 0; u < U; ++u) request4(u, q4[u]);
  }
  // ---- who lost something, and the counts of the lane's 16 entries, a byte each
  uint32_t c4[4] = {0, 0, 0, 0};
  auto count_bits = [&](uint32_t p) {
#pragma unroll
    for (int q = 0; q < 4; ++q) c4[q] += (((p >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;
  };
  const uint32_t sg = lane_signs<K, In>(a.seed, a.base + ew, x, wave, lane);
  tile_barrier<G * W>();
  bool lossy_here = false;   // a worker of the group lost something in the wavefront's part
  {
    const bool inside = K || lane * 16 < left;
    int full = 0;   // workers that lost nothing in the wavefront's part
    for (int i = grp; i < N; i += U * G) {
      if (i > grp) {
#pragma unroll
        for (int u = 0; u < U; ++u) bits[u] = request_bits(i + u * G);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int w = i + u * G;
        if (w >= N) break;
        if (const u64 lost = __builtin_amdgcn_ballot_w64(inside && bits[u] != 0xFFFFu)) {
          lossy_here = true;
          if (lane == 0) atomicOr(&marks[w >> 5], 1u << (w & 31));
          if (MODE == GROUPS && SPLIT && lane == 0) missing16[w] = make_uint2((uint32_t)lost, (uint32_t)(lost >> 32));
          count_bits(bits[u]);
        } else {
          ++full;
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) c4[q] = inside ? c4[q] + (uint32_t)full * 0x01010101u : 0;
  }
  const int own16 = (wave * 64 + lane) * 16;
  *(uint4*)&counts[SLOTS > 1 ? slot : grp][own16] = make_uint4(c4[0], c4[1], c4[2], c4[3]);
  // Sec. 3.4 loss monitoring: what this wavefront's lanes miss, gathered in LDS; one atomic per workgroup at most
  if (a.total_out) {
    const uint32_t entries = K || left >= 1024 ? 1024u : (uint32_t)left;
    if (lossy_here) {
      uint32_t n = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) n = __builtin_amdgcn_sad_u8(c4[q], 0u, n);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o, 64);
      if (lane == 0) atomicAdd(&missing[0], (uint32_t)((N - grp + G - 1) / G) * entries - n);   // the group's workers
    }
    if constexpr (SLOTS > 1) {
      if (lane == 0) {
        __threadfence_block();   // what is missing before the sign that it is there
        if (atomicAdd(&missing[1], 1u) == (uint32_t)tiles - 1) add_total(a, first_unit == 0, atomicAdd(&missing[0], 0u));
      }
    }
  }
  tile_barrier<G * W>();
  if (SLOTS == 1 && a.total_out && threadIdx.x == 0) add_total(a, unit == 0, missing[0]);

  float acc[16], raw[16], v[16];   // sum over the workers with a loss (B), over the whole ones (A); the one in work
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  auto clear_raw = [&]() {
#pragma unroll
    for (int r = 0; r < 16; ++r) raw[r] = 0.0f;
  };
  int lossy = 0;   // workers with a loss
  auto marks_of = [&](int i) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)marks[i >> 5]); };   // the 32 around worker i
  for (int i = 0; i < N; i += 32) lossy += __builtin_popcount(marks_of(i));
  const int whole = N - lossy;
  const bool has_sum = whole > 0 || SPLIT;
  const uint32_t ord = MODE == STREAM ? 0 : order_workers(marks, order, N, lossy, lane);
  auto worker = [&](int j) -> int {   // the j-th in order, -1 past the end
    return j < N ? (int)(((uint32_t)__builtin_amdgcn_readlane((int)ord, j & 63) >> (j >> 6 << 3)) & 0xFFu) : -1;
  };
  auto add_masked = [&](const float (&y)[16], uint32_t words) {
    if (all_arrived(words)) {   // nothing lost in what this wavefront holds
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] += y[r];
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] += in_mask(mask_of_reg(words, r)) ? y[r] : 0.0f;
    }
  };
  // the signed entries of a worker with a loss.  The shifted copies of the sign bits are formed anew for every worker:
  // kept over the loop they would cost sixteen registers
  auto sign_all = [&](float (&y)[16]) {
    uint32_t s = sg;
    asm volatile("" : "+v"(s));
#pragma unroll
    for (int r = 0; r < 16; ++r) y[r] = flip_sign(y[r], s, r);
  };
  // SPLIT: all ones where the block of the lane's entries 256 c + 4 lane .. + 3 has a run of 32 entries with its bit in `missing`
  auto lost_chunk = [&](uint32_t missing, int c) -> int {
    int at = lane >> 3;   // the masks of runs are formed here, not kept in registers all along
    asm volatile("" : "+v"(at));
    return (missing & block_runs(8 * c + at, k, 5)) != 0 ? -1 : 0;
  };
  // (lane l of the first 32 of `words`: the received bits of entries 32 l ..)
  auto runs_missing = [&](uint32_t words) { return (uint32_t)__builtin_amdgcn_ballot_w64(words != 0xFFFFFFFFu); };
  auto take_signed = [&](const Raw16<In>& y, uint32_t missing) {   // SPLIT: without the blocks that are whole
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int lost = SPLIT ? lost_chunk(missing, c) : -1;
#pragma unroll
      for (int r = 4 * c; r < 4 * c + 4; ++r) v[r] = __builtin_bit_cast(float, __builtin_bit_cast(int, entry_of<In>(y, r)) & lost);
    }
    sign_all(v);
  };
  auto add_whole = [&](const Raw16<In>& y, uint32_t missing) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int lost = SPLIT ? lost_chunk(missing, c) : 0;
#pragma unroll
      for (int r = 4 * c; r < 4 * c + 4; ++r) raw[r] += __builtin_bit_cast(float, __builtin_bit_cast(int, entry_of<In>(y, r)) & ~lost);
    }
  };

  if constexpr (MODE == STREAM) {
    uint32_t lost32 = 0;
    auto consume = [&](int i, Raw16<In>& r16, uint32_t& m) {
      if ((i & 31) == 0) lost32 = marks_of(i);
      const bool lost = (lost32 >> (i & 31)) & 1;
      const uint32_t words = m;
      const uint32_t missing = SPLIT && lost ? runs_missing(words) : 0;
      if (SPLIT || !lost) add_whole(r16, missing);
      if (lost) take_signed(r16, missing);
      request(i + 2, r16);
      m = request_words(i + 2);
      if (lost) {
        int lane_t = lane;   // LDS addresses formed here, not kept in registers all along
        asm volatile("" : "+v"(lane_t));
        tile_barrier<W>();
        to_wire<K, In>(v, x, wave, lane_t, k);
        add_masked(v, words);
      }
    };
    clear_raw();
    for (int i = 0; i < N; i += 2) {
      consume(i, ra, ma);
      if (i + 1 < N) consume(i + 1, rb, mb);
    }
    if (has_sum) {
      sign_all(raw);
      tile_barrier<W>();
      to_wire<K, In>(raw, x, wave, lane, k);
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] += raw[r];
    }
  } else {
    // Items 0 .. lossy - 1 are the workers with a loss, item lossy the sum over what is whole; round t: items 4 t ..
    // 4 t + 3.  The rounds before the last run while the whole workers' entries are on their way.
    request(grp < lossy ? worker(grp) : -1, ra);
    ma = request_words(grp < lossy ? worker(grp) : -1);
    const int items = lossy + has_sum, own4 = (wave * 64 + lane) * 4;
    auto round = [&](int t) {
      const int item = t * G + grp;
      const bool works = item < items, is_sum = item == lossy;
      const uint32_t words = is_sum ? 0xFFFFFFFFu : ma;
      if (works) {
        if (is_sum) {
          lds_a<K, In, false>(v, x, wave, lane);
          sign_all(v);
        } else {
          take_signed(ra, SPLIT ? runs_missing(words) : 0);
        }
      }
      request(item + G < lossy ? worker(item + G) : -1, ra);
      ma = request_words(item + G < lossy ? worker(item + G) : -1);
      if (works) {
        stages_a<K, In>(v, k);
        lds_a<K, In, true>(v, x, wave, lane);
        __builtin_amdgcn_wave_barrier();
        lds_m<K, In, false>(v, x, wave, lane);
        stages_m<K, In>(v, k);
        lds_m<K, In, true>(v, x, wave, lane);
      }
      __syncthreads();
      if (works) {
        lds_b<K, In, false>(v, x, wave, lane);
        stages_b<K, In>(v, k);
        if (grp == 0) {
          add_masked(v, words);
        } else {   // the masked values: registers 4 j .. 4 j + 3 at 256 W j + own4
#pragma unroll
          for (int r = 0; r < 16; ++r) v[r] = in_mask(mask_of_reg(words, r)) ? v[r] : 0.0f;
#pragma unroll
          for (int r = 0; r < 16; r += 4) *(f32x4v*)(ybuf[grp - 1] + r * 64 * W + own4) = f32x4v{v[r], v[r + 1], v[r + 2], v[r + 3]};
        }
      }
      __syncthreads();   // and everyone has read its B positions
      if (grp == 0) {
#pragma unroll
        for (int g = 1; g < G; ++g)
          if (t * G + g < items) {
#pragma unroll
            for (int r = 0; r < 16; r += 4) {
              const f32x4v y = *(const f32x4v*)(ybuf[g - 1] + r * 64 * W + own4);
              acc[r] += y[0]; acc[r + 1] += y[1]; acc[r + 2] += y[2]; acc[r + 3] += y[3];
            }
          }
      }
    };
    float s4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    const uint32_t runs16 = SPLIT ? block_runs((grp & 1) * 16 + (lane >> 2), k, 4) : 0;   // of this lane's four entries, in their half of the tile
    int t = 0;
    for (int b = 0; b < N; b += U) {
      const uint32_t lost = marks_of(b) >> (b & 31);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (!((lost >> u) & 1)) {
#pragma unroll
          for (int r = 0; r < 4; ++r) s4[r] += __builtin_bit_cast(float, (uint32_t)q4[u][r]);
        } else if (SPLIT) {   // its blocks that are whole
          const bool lost_here = ((grp < 2 ? missing16[b + u].x : missing16[b + u].y) & runs16) != 0;
#pragma unroll
          for (int r = 0; r < 4; ++r) s4[r] += lost_here ? 0.0f : __builtin_bit_cast(float, (uint32_t)q4[u][r]);
        }
      if (b + U < N) {
        const uint32_t next = marks_of(b + U) >> ((b + U) & 31);
#pragma unroll
        for (int u = 0; u < U; ++u) request4(!SPLIT && ((next >> u) & 1) ? -1 : b + U + u, q4[u]);
      }
      if (t < lossy / G) round(t++);
    }
    while (t < lossy / G) round(t++);
    if (items > t * G) {
      if (has_sum)   // the sum goes to the group that encodes it (behind a barrier since that buffer was last read)
        *(f32x4v*)(xbuf[lossy % G] + wave * F::PART + F::padded(grp * 256) + F::padded(lane * 4)) = f32x4v{s4[0], s4[1], s4[2], s4[3]};
      __syncthreads();
      round(t);
    }
    if (grp > 0) return;   // (a barrier waits for the wavefronts that are left)
  }

  // ---- counts
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint4 o = *(const uint4*)&counts[SLOTS > 1 ? slot : g][own16];
    if (g == 0) { c4[0] = o.x; c4[1] = o.y; c4[2] = o.z; c4[3] = o.w; }
    else { c4[0] += o.x; c4[1] += o.y; c4[2] += o.z; c4[3] += o.w; }
  }
  if constexpr (G > 1) *(uint4*)&counts[0][own16] = make_uint4(c4[0], c4[1], c4[2], c4[3]);

  // ---- mean over what arrived, decode
  const float post = a.scale;
  tile_barrier<W>();   // every wavefront has read the last exchange
  if (lossy == 0) {
    const float f = post * __builtin_amdgcn_rcpf((float)N);
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] *= f;
  } else {
    // the counts, one byte an entry, through LDS into B
    const uint8_t* mine = counts[slot] + wire_wave_entry<K, In>(wave) + lane;
    uint32_t n[16], least = 255;
#pragma unroll
    for (int r = 0; r < 16; ++r) n[r] = mine[F::reg_entry(r)];
#pragma unroll
    for (int r = 0; r < 16; ++r) least = n[r] < least ? n[r] : least;
    if (__builtin_amdgcn_ballot_w64(least != (uint32_t)N) == 0) {
      const float f = post * __builtin_amdgcn_rcpf((float)N);
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] *= f;
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = n[r] ? acc[r] * (post * __builtin_amdgcn_rcpf((float)n[r])) : 0.0f;
    }
  }
  from_wire<K, In>(acc, x, wave, lane, k);
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = flip_sign(acc[r] * a.scale, sg, r);
  {
    const __amdgpu_buffer_rsrc_t rs = rsrc_of((const In*)a.out + ew, left * ES);
#pragma unroll
    for (int q = 0; q < F::C; ++q) {
      u32x4v o;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = __builtin_bit_cast(uint32_t, acc[4 * q + j]);
      store16<kBufNt>(o, rs, lane * 16 + q * 1024);
    }
  }
  if (a.count_out) {
    const __amdgpu_buffer_rsrc_t rs = rsrc_of(a.count_out + ew, left);
    if (((uintptr_t)a.count_out & 15) == 0) {
      store16<kBufNt>(u32x4v{c4[0], c4[1], c4[2], c4[3]}, rs, lane * 16);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) store_counts4(c4[q], rs, lane * 16 + q * 4, 0, false);
    }
  }
}

template <int K> constexpr int kFusedThreads = 64 << (K ? K - 10 : 0);
// VGPRs are capped so that several workgroups fit on a CU: the loads in flight are those of its neighbours too
template <int K, int MODE, bool SPLIT>
__global__ __launch_bounds__(kFusedThreads<K> * (MODE == GROUPS ? kGroups : 1)) __attribute__((amdgpu_waves_per_eu(4)))
void k_fused(PathArgs a) {
  fused_tile<K, MODE, SPLIT>(a, blockIdx.x, gridDim.x);
}
// K = 0: a workgroup of the plain form serves kBatchSlots tiles of one bucket; ba.tile_start counts workgroups.  With totals fewer tiles
// mean more atomics: us, four / eight tiles a workgroup, 2^10, 5 % loss, N = 4, 4096 / 12800 tiles 26.0 / 22.3, 59.5 / 55.4, N = 16 60.6 / 55.9, 177 / 173;  1 %
// loss, N = 2, 12800 tiles 35.1 / 37.7.  (Without totals, one / eight: N = 8, 1200 / 2048 / 12800 tiles 12.3 / 13.0, 16.6 / 16.3, 85.4 / 88.0, N = 2, 12800 tiles 33.1 /
// 35.9.)
template <int K, int MODE> constexpr int kBatchSlots = K == 0 && MODE != GROUPS ? 8 : 1;
template <int K, int MODE, bool SPLIT>
__global__ __launch_bounds__(kFusedThreads<K> * (MODE == GROUPS ? kGroups : kBatchSlots<K, MODE>)) __attribute__((amdgpu_waves_per_eu(4)))
void k_fused_batched(BatchArgs ba) {
  constexpr int SLOTS = kBatchSlots<K, MODE>, T = FTile<K, float>::T;
  PathArgs a;
  const u64 group = bucket_of(ba, a, blockIdx.x);
  fused_tile<K, MODE, SPLIT, SLOTS>(a, group * SLOTS, (a.n_pad + T - 1) / T);
}

}  // namespace ordev

// The fused path (OptiReduce Sec. 3.3 encode, Sec. 3.1.1 aggregation, Sec. 3.3 / Sec. 4 decode) of bf16 slices in blocks of 2^16
// entries: one workgroup per block, in the manner of rht_fused_bf16.hpp.
//
// The sum of a block over the workers takes 128 registers of each of the 512 lanes (8 wavefronts of 8192 entries, 256 registers a
// lane), the packed entries of the worker in work 64.  That leaves room for a quarter of its encoded values at a time.  The
// products make the quarters: two accumulated products of 16 x 32 entries apply H_64 (e0 e1 e2 e7 e8 e9), and an operand holds the
// columns of one quarter, i.e. of one value of the output bits e8 and e9.  Nothing is read twice and nothing is added up across quarters.
// Entry bits of the positions (as in rht_fused_bf16.hpp; a quarter: e8, e9 fixed):
//   L   as loaded and stored   regs e0 e1 e2, e9 .. e12         lanes e3 .. e8               waves e13 ..
//   S1  after the products     regs e3 e4 e10 e11 e12           lanes e0 e1 e2 e7 e5 e6      waves e13 ..   quarters e8 e9
//   S2  encoded                regs e5 e6 e13 e14 e15           lanes e0 .. e4 e7            waves e10 ..   quarters e8 e9
//   S3  in the decode          regs e3 e4 e7 e10 e11            lanes e0 e1 e2 e5 e6 e12     waves e13 ..   quarters e8 e9
// Decode: S2 all its registers and both bits of the quarters, S3 its registers, L e0 e1 e2 and e12.
//
// Bound by a wavefront's own chain: per worker 1400 additions, 330 other vector instructions and 64 products in each of two
// wavefronts a SIMD, 4.5 us, and 2 us of exchange through LDS, which only partly run at the same time (7 us).  us, two
// workgroups a block that read everything twice and met in memory -> this: N = 8, 15317 blocks 5980 - 6400 -> 4600 - 4760 (4.2 - 4.4 TB/s), 2560
// blocks 970 -> 743, N = 2, 1000 blocks 240 -> 144.
//
// One workgroup is all that fits on a CU, so nothing but the kernel itself runs under its waits for memory.  Three quarters of the
// next worker's entries are written to LDS by the loads themselves (no registers) from the start of a worker on, the last quarter
// is asked for once the entries in registers have been used for the last time; and a workgroup walks over blocks, so that this
// goes on through the decode of a block into the next one.  It does so only while nothing is spilled: the reload of a spilled register
// waits for everything that was asked for before it.  Hence addresses and constants are formed where they are used (`lane_t`).  us,
// 44 bytes of scratch a lane -> none, with the exchange as it was then: N = 1, 129 blocks 25.0 -> 22.9;  N = 2, 1000 blocks 151 -> 144;  N = 8, 2560 blocks 891 -> 879, nothing
// lost 766 -> 738;  N = 32, 300 blocks 626 -> 624.
#pragma once
#include "rht_fused_bf16.hpp"

namespace ordev {

constexpr int kQuarterEntries = 1 << 14;
constexpr int kStaged = 10;   // of a lane's 16 loads of a worker: through LDS

// A quarter in LDS.  S1 stores singly, S2 loads 16 bytes a lane: LDS is read faster than it is written that way.  Each half of a wavefront
// stores to 32 banks of 4 bytes; a 16-byte load goes by 16 lanes, those of a half whose lane bits 2, 3, 4 have the same parity, which have to
// cover 64 banks.  Entry bits from the lowest address bit up: e5 (e6^e7) e0 e1 e2 e3 e4 e7 e10 .. e15, with neither conflicts of the stores
// (lanes e0 e1 e2 e7 e5 in a half) nor of the loads.  e7 is a lane bit of S2, where the XOR swaps two registers of the stage of e6: their sum is
// the same, and their difference changes its sign, the same one for all workers, which the mean takes back (s2_sign).  us, 64 KB, with two
// lanes on every bank 0.45 + 0.23 -> 0.36 + 0.14.
__device__ __forceinline__ int quarter_s1(int wave, int lane) {   // + 32 e3 + 64 e4 + 256 (r >> 2)
  return wave * 2048 + (lane & 7) * 4 + ((lane >> 4) & 1) + (((lane >> 5) ^ (lane >> 3)) & 1) * 2 + ((lane >> 3) & 1) * 128;
}
__device__ __forceinline__ int quarter_s2(int wave, int lane) {   // + 2048 (r >> 2), registers e5 (e6^e7) together
  return (lane & 7) * 4 + ((lane >> 3) & 3) * 32 + (lane >> 5) * 128 + wave * 256;
}
__device__ __forceinline__ float s2_sign(float f, int r, int lane) { return (r & 2) && (lane & 32) ? -f : f; }
// The same positions on the way into the decode, where registers e5 e6 are stored together: e5 e6 e0 e1 e2 e7 e3 e4 e10 .. e15
__device__ __forceinline__ int decode_s2(int wave, int lane) {   // + 2048 (r >> 2)
  return (lane & 7) * 4 + ((lane >> 3) & 3) * 64 + (lane >> 5) * 32 + wave * 256;
}

// Signs of the lane's 16 loads (pair_signs of four loads each): a Philox counter a lane, spread through 1 KB at `bytes`.
__device__ __forceinline__ u32x4v signs_64k(u64 seed, u64 first, uint8_t* bytes, int lane) {
  const u64 ctr = (first >> 7) + (u64)lane;
  const u32x4 w = philox4x32_10((uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u, (uint32_t)seed, (uint32_t)(seed >> 32));
  *(uint4*)(bytes + lane * 16) = make_uint4(w.a, w.b, w.c, w.d);
  __builtin_amdgcn_wave_barrier();
  u32x4v t;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    t[q] = pair_signs((uint32_t)bytes[lane + 256 * q] | (uint32_t)bytes[lane + 256 * q + 64] << 8 | (uint32_t)bytes[lane + 256 * q + 128] << 16 |
                      (uint32_t)bytes[lane + 256 * q + 192] << 24);
  return t;
}

// The decode of one block, from the means in S2 (`acc`, by quarter).  x: nobody reads it any more.
__device__ __forceinline__ void decode_64k(float (&acc)[4][32], float* x, u32x4v sg, const PathArgs& a, u64 e0, int wave, int lane) {
#pragma unroll
  for (int s = 0; s < 4; ++s) reg_stages(acc[s], 0, 5);
  across_tiles<4, 32>(acc);   // e8, e9
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    int lane_t = lane;
    asm volatile("" : "+v"(lane_t));
    if (s > 0) lds_barrier<8>();   // everyone has read the quarter before
    float* to = x + decode_s2(wave, lane_t);
#pragma unroll
    for (int r = 0; r < 32; r += 4) *(f32x4v*)(to + (r >> 2) * 2048) = f32x4v{acc[s][r], acc[s][r + 1], acc[s][r + 2], acc[s][r + 3]};
    lds_barrier<8>();
    const float* from = x + wave * 2048 + (lane_t & 7) * 4 + ((lane_t >> 3) & 3) + (lane_t >> 5) * 1024;
#pragma unroll
    for (int r = 0; r < 32; ++r) acc[s][r] = from[(r & 3) * 64 + ((r >> 2) & 1) * 32 + (r >> 3) * 256];   // registers e3 e4 e7 e10 e11
    reg_stages(acc[s], 0, 5);
  }
  lds_barrier<8>();
  // inside the wavefront, 2048 entries of one (e10, e11) at a time.  From the lowest address bit up: e0 e1 (e2^e3) (e4^e6) e5 (e2^e7) e6
  // e7 e8 e9 e12
  float* mine = x + wave * 2048;
  const __amdgpu_buffer_rsrc_t out = rsrc_of((const bf16_t*)a.out + e0 + (u64)wave * 8192, 16384);
#pragma unroll
  for (int f = 0; f < 4; ++f) {   // e10, e11
    int lane_t = lane;
    asm volatile("" : "+v"(lane_t));
    float v[32];
    {
      const int to = (lane_t & 3) + ((lane_t >> 2) & 1) * (4 + 32) + ((lane_t >> 3) & 1) * 16 + ((lane_t >> 4) & 1) * (8 + 64) + (lane_t >> 5) * 1024;
#pragma unroll
      for (int s = 0; s < 4; ++s)   // e8, e9
#pragma unroll
        for (int r = 0; r < 8; ++r) mine[(to ^ ((r & 3) << 2 | (r >> 2) << 5)) + (r >> 2) * 128 + s * 256] = acc[s][f * 8 + r];
    }
    __builtin_amdgcn_wave_barrier();
    {
      const int from = ((lane_t & 7) * 4 + ((lane_t >> 3) & 1) * 64 + ((lane_t >> 4) & 3) * 128) ^ (((lane_t >> 3) & 1) << 3 | ((lane_t >> 4) & 1) << 5);
#pragma unroll
      for (int g = 0; g < 8; ++g) {   // registers e0 e1 | e2 e9 e12
        const f32x4v t = *(const f32x4v*)(mine + (from ^ ((g & 1) * (4 + 32))) + (g >> 1) * 512);
        v[4 * g] = t[0]; v[4 * g + 1] = t[1]; v[4 * g + 2] = t[2]; v[4 * g + 3] = t[3];
      }
    }
    __builtin_amdgcn_wave_barrier();
    reg_stage<0>(v);
    reg_stage<1>(v);
    reg_stage<2>(v);
    reg_stage<4>(v);
#pragma unroll
    for (int g = 0; g < 4; ++g) {   // e9, e12
      const int q = (g & 1) + 2 * f + 8 * (g >> 1);
      uint32_t word = sg[q >> 2] << (4 * (q & 3));
      u32x4v o;
#pragma unroll
      for (int d = 0; d < 4; ++d) o[d] = pack_bf16x2(v[8 * g + 2 * d] * a.scale, v[8 * g + 2 * d + 1] * a.scale);
      flip_pairs(o, word);
      store16<kBufNt>(o, out, lane * 16 + q * 1024);
    }
  }
}

// next(x, a): the arguments of the x-th block's bucket; returns the block inside it.  NQ = 4: the whole path, workgroups walk over the
// blocks first, first + step ..  NQ = 1, 2: for few blocks (alone or behind a walk), one block's quarters quarter0 .. quarter0 + NQ - 1 (a quarter
// or a half of them), up to the mean, which goes to a.mean_out for k_decode_64k: by quarter, wavefront, four registers, lane.
template <int NQ, class Next>
__device__ __forceinline__ void fused_bf16_walk_64k(uint32_t first, uint32_t blocks, uint32_t step, int quarter0, bool totals, const Next& next) {
  constexpr int B = 1 << 16;
  __shared__ __align__(16) float x[1 << 14];
  __shared__ __align__(16) u32x4v stage[8 * kStaged * 64];
  __shared__ __align__(16) u32x4v lost[512];    // received bits of the worker in work, where something is missing
  __shared__ __align__(16) u32x4v signs[512];   // of the lane's 16 loads: pair_signs of four loads each
  const int wave = wave_id(), lane = lane_id();

  u32x4v p[16];   // load q: 8 entries from 512 q + 8 lane of the wavefront's part
  auto part_of = [&](const PathArgs& a, u64 blk, int i) { return (const bf16_t*)a.in + (u64)i * a.n_pad + (blk << 16) + (u64)wave * 8192; };
  // The loads that write LDS are out of the compiler's sight, which would
  // wait for them ahead of every other access to LDS; landed() is the only wait for them, whatever was asked for after them
  auto request_staged = [&](const bf16_t* part, int from, int to_q) {
    const u32x4v rs = {(uint32_t)(uintptr_t)part, (uint32_t)((uintptr_t)part >> 32), 16384u, 0x00020000u};
    const uint32_t to = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(stage + wave * kStaged * 64);
#pragma unroll
    for (int q = from; q < to_q; ++q)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                   :: "s"(to + q * 1024), "v"(lane * 16), "s"(rs), "s"(q * 1024) : "memory", "m0");
  };
  u32x4v mw;   // received bits of the worker whose entries are on their way
  auto landed = [&]() {   // names what the compiler knows to be in flight: it waits for that here and not behind the loads that follow
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("" : "+v"(p[10]), "+v"(p[11]), "+v"(p[12]), "+v"(p[13]), "+v"(p[14]), "+v"(p[15]), "+v"(mw));
  };
  auto request_rest = [&](const bf16_t* part, int from, int to_q) {   // null: zeros, without touching memory
    const __amdgpu_buffer_rsrc_t rs = rsrc_of(part, part ? 16384 : 0);
#pragma unroll
    for (int q = from; q < to_q; ++q) p[q] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, q * 1024, kBufNt));
  };
  // received bits in S2: the wavefront's 1024 entries of each eighth of the block; lane l holds 128 entries (four words, e5 e6) of
  // eighth l >> 3, from 128 (l & 7) on
  auto words_of = [&](const PathArgs& a, u64 blk, int i) {
    const bool there = i < a.N;
    return rsrc_of((const uint8_t*)a.masks + (u64)(there ? i : 0) * (a.n_pad >> 3) + (blk << 13) + wave * 128, there ? (B >> 3) - wave * 128 : 0);
  };
  const int word_at = (lane >> 3) * 1024 + (lane & 7) * 16;
  auto request_words = [&](__amdgpu_buffer_rsrc_t rs) { mw = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(rs, word_at, 0, 0)); };
  // ---- the +-1 operand of quarter 0: lane l holds column n = l & 15, rows 8 (l >> 4) + 0..7; n0 n1 n2 pair with the entry's place
  // in the load, n3 with lane bit 4 (e7); quarters with e8 set: times the sign of lane bit 5; with e9 set: minus the second product
  auto operand = [](int lane, int quarter) {
    const uint32_t n1 = lane & 2 ? 0x80008000u : 0u, n2 = lane & 4 ? 0x80008000u : 0u;
    uint32_t first = lane & 1 ? 0xBF803F80u : 0x3F803F80u;
    first ^= (lane & 24) == 24 ? 0x80008000u : 0u;
    if (quarter & 1) first ^= lane & 32 ? 0x80008000u : 0u;
    return u32x4v{first, first ^ n1, first ^ n2, first ^ n1 ^ n2};
  };

  for (uint32_t at = first;; at += step) {
    PathArgs a;
    const u64 blk = next(at, a);
    if (at == first) {
      request_staged(part_of(a, blk, 0), 0, kStaged);
      request_rest(part_of(a, blk, 0), kStaged, 16);
      request_words(words_of(a, blk, 0));
    }
    const int N = a.N;
    const u64 e0 = blk << 16;
    {
      int lane_t = lane;   // addresses formed here, not kept in registers all along
      asm volatile("" : "+v"(lane_t));
      signs[wave * 64 + lane_t] = signs_64k(a.seed, a.base + e0 + (u64)wave * 8192, (uint8_t*)(x + wave * 2048), lane_t);
    }
    float acc[NQ][32];
#pragma unroll
    for (int s = 0; s < NQ; ++s)
#pragma unroll
      for (int r = 0; r < 32; ++r) acc[s][r] = 0.0f;
    const bool more = NQ == 4 && at + step < blocks;
    bool clean = true;   // nothing of this wavefront's S2 part was lost so far
    int i = 0;
    do {   // (N >= 1)
      int lane_t = lane;   // as above
      asm volatile("" : "+v"(lane_t));
      landed();
      const bool whole = __builtin_amdgcn_ballot_w64((mw[0] & mw[1] & mw[2] & mw[3]) != 0xFFFFFFFFu) == 0;
      if (!whole) {
        lost[wave * 64 + lane_t] = mw;
        clean = false;
      }
#pragma unroll
      for (int q = 0; q < kStaged; ++q) p[q] = stage[(wave * kStaged + q) * 64 + lane_t];
      const u32x4v sg = signs[wave * 64 + lane_t];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t word = sg[q];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          flip_pairs(p[4 * q + c], word);
          asm volatile("" : "+v"(p[4 * q + c]));   // here, not where they are next used
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wavefront has read its part of the stage
      // the next worker's, or the next block's first one's
      const bf16_t* after = part_of(a, blk, i + 1);
      __amdgpu_buffer_rsrc_t words_after = words_of(a, blk, i + 1);
      if (i + 1 == N) {
        after = nullptr;
        if (more) {
          PathArgs b;
          const u64 blk_b = next(at + step, b);
          after = part_of(b, blk_b, 0);
          words_after = words_of(b, blk_b, 0);
        }
      }
#pragma unroll
      for (int turn = 0; turn < NQ; ++turn) {
        const int at_s = NQ == 4 ? turn ^ (turn >> 1) : turn;   // 0 1 3 2
        const int s = NQ == 4 ? at_s : quarter0 + turn;
        float v[32];
        {
          if (NQ == 4 ? turn == 2 : turn == 0 && (quarter0 & 2)) {   // e9 changes: minus the entries of the second products
#pragma unroll
            for (int q = 1; q < 16; q += 2)
#pragma unroll
              for (int d = 0; d < 4; ++d) p[q][d] ^= 0x80008000u;
          }
          int lane_h = lane;
          asm volatile("" : "+v"(lane_h));   // the operand and the products of this quarter here, not before
          const u32x4v h = operand(lane_h, s);
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            f32x4v d = {0};
            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8v, p[2 * t]), __builtin_bit_cast(bf16x8v, h), d, 0, 0, 0);
            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8v, p[2 * t + 1]), __builtin_bit_cast(bf16x8v, h), d, 0, 0, 0);
            v[4 * t] = d[0]; v[4 * t + 1] = d[1]; v[4 * t + 2] = d[2]; v[4 * t + 3] = d[3];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        // A few loads at a time where the launch fills the chip: a CU takes one of them (1 KB) in 16 cycles, and all wavefronts would wait for the
        // last one's.  (All that are left at once, 15317 blocks of 8 workers 4694 -> 4790.)  Few blocks, whose reads the L2 serves for the most
        // part, take as many as early as they can: us, 3 and 3 later -> 5, the rest at once, NQ = 1, 16 blocks, N = 8 / 32 47.4 -> 45.1 / 133.5 -> 123.4;  4 -> 10,
        // NQ = 2, 128 blocks, N = 32 196 -> 192.
        constexpr int per = NQ <= 2 ? kStaged : 5, at_once = NQ == 1 ? 5 : NQ == 2 ? kStaged : 3, rest_at_once = NQ <= 2 ? 16 : kStaged + 3;
        if (per * turn < kStaged && after) request_staged(after, per * turn, per * turn + at_once);   // (none on their way when the workgroup ends)
        if (turn == NQ - 1) {   // the entries have been used for the last time
          request_rest(after, kStaged, rest_at_once);
          if (rest_at_once == 16) request_words(words_after);
        }
        // a half of the registers at a time after the stage between the halves, and eight of them once the stage between the eights has
        // made them: the other half's stages run under their stores, and only the last stores are waited for.  (That stage before the other
        // three, and four times eight registers by themselves: 2560 blocks of 8 workers, nothing lost, 743 -> 723 us, but other bits.)
        reg_stage<4>(v);
        float* to = x + quarter_s1(wave, lane_t);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          auto& vh = *(float (*)[16])&v[16 * h];
          reg_stages(vh, 0, 3);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int g = 0; g < 2; ++g) {
#pragma unroll
            for (int r = 4 * g; r < 4 * g + 4; ++r) {
              const float t = vh[r];
              vh[r] = t + vh[r + 8];
              vh[r + 8] = t - vh[r + 8];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float* at_r = to + (r & 1) * 32 + (r >> 1) * 64 + g * 256 + h * 1024;
              at_r[0] = vh[4 * g + r];
              at_r[512] = vh[4 * g + r + 8];
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        lds_barrier<8>();
        {
          const float* from = x + quarter_s2(wave, lane_t);
#pragma unroll
          for (int r = 0; r < 32; r += 4) {
            const f32x4v t = *(const f32x4v*)(from + (r >> 2) * 2048);
            v[r] = t[0]; v[r + 1] = t[1]; v[r + 2] = t[2]; v[r + 3] = t[3];
          }
        }
        // Everyone has read the quarter.  Here, where all wavefronts are together anyway: from here to the next stores they may drift
        // apart, so that one's accesses to LDS run under another's arithmetic.
        lds_barrier<8>();
        if (per * turn < kStaged && after) request_staged(after, per * turn + at_once, per * turn + per);
        if (rest_at_once < 16 && turn == NQ - 1) {
          request_rest(after, rest_at_once, 16);
          request_words(words_after);
        }
        reg_stages(v, 0, 5);
        // the result in the HIGH half: the fp32 pattern of the rounded value, no unpacking
#pragma unroll
        for (int r = 0; r < 32; ++r) v[r] = __builtin_bit_cast(float, pack_bf16x2(0.0f, v[r]));
        if (!whole) {
          const u32x4v words = lost[wave * 64 + lane_t];
#pragma unroll
          for (int r = 0; r < 32; ++r) {
            const int from = (r >> 2) * 8 + 2 * s;
            const u64 m = (u64)(uint32_t)__builtin_amdgcn_readlane((int)words[r & 3], from) |
                          (u64)(uint32_t)__builtin_amdgcn_readlane((int)words[r & 3], from + 1) << 32;
            v[r] = in_mask(m) ? v[r] : 0.0f;
          }
        }
#pragma unroll
        for (int r = 0; r < 32; ++r) {
          acc[at_s][r] += v[r];
          asm volatile("" : "+v"(acc[at_s][r]));   // here, not where the sum is next used: v's registers are needed
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } while (++i < N);

    // ---- counts (a byte for each of the 128 entries of the lane's words) and the mean over what arrived
    int lane_m = lane;   // as above
    asm volatile("" : "+v"(lane_m));
    const float post = a.scale;
    const __amdgpu_buffer_rsrc_t counts = rsrc_of(a.count_out + e0 + wave * 1024, a.count_out && quarter0 == 0 ? B - wave * 1024 : 0);   // none, or another workgroup's: stores are dropped
    const bool counts_aligned = ((uintptr_t)a.count_out & 15) == 0;
    // sixteen counts a lane: those from 16 lane on of the wavefront's 1024 entries of eighth q
    auto store_counts = [&](auto&& of) {
      if (counts_aligned) {
#pragma unroll
        for (int q = 0; q < 8; ++q) store16<kBufNt>(of(q), counts, q * 8192 + lane * 16);
      } else {
#pragma unroll 1
        for (int q = 0; q < 8; ++q) {
          const u32x4v c = of(q);
#pragma unroll
          for (int d = 0; d < 4; ++d) store_counts4(c[d], counts, q * 8192 + lane * 16 + d * 4, 0, false);
        }
      }
    };
    uint32_t total = 0;
    if (clean) {
      uint32_t c = (uint32_t)N * 0x01010101u;
      asm volatile("" : "+v"(c));   // here, not ahead of the blocks
      store_counts([&](int) { return u32x4v{c, c, c, c}; });
      total = (uint32_t)N * 128u;
      const float f = post * __builtin_amdgcn_rcpf((float)N);
#pragma unroll
      for (int s = 0; s < NQ; ++s)
#pragma unroll
        for (int r = 0; r < 32; ++r) acc[s][r] *= s2_sign(f, r, lane_m);
    }
    if (!clean) {
      uint8_t* mine = (uint8_t*)x + wave * 8192;   // the wavefront's counts, by word
      uint32_t c8[4][8];   // of a lane's four words
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < 8; ++q) c8[j][q] = 0;
#pragma unroll 1
      for (int i = 0; i < N; i += 4) {
        u32x4v w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = __builtin_bit_cast(u32x4v, __builtin_amdgcn_raw_buffer_load_b128(words_of(a, blk, i + u), word_at, 0, 0));
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < 8; ++q) c8[j][q] += (((w[u][j] >> (4 * q)) & 0xFu) * 0x00204081u) & 0x01010101u;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int q = 0; q < 8; ++q) total = __builtin_amdgcn_sad_u8(c8[j][q], 0u, total);
        *(uint4*)(mine + lane_m * 128 + j * 32) = make_uint4(c8[j][0], c8[j][1], c8[j][2], c8[j][3]);
        *(uint4*)(mine + lane_m * 128 + j * 32 + 16) = make_uint4(c8[j][4], c8[j][5], c8[j][6], c8[j][7]);
      }
      __builtin_amdgcn_wave_barrier();
      store_counts([&](int q) { return *(const u32x4v*)(mine + q * 1024 + lane * 16); });
      const uint8_t* from = mine + (lane_m >> 5) * 128 + (lane_m & 31);
#pragma unroll
      for (int s = 0; s < NQ; ++s)
#pragma unroll
        for (int r = 0; r < 32; ++r) {
          const uint32_t n = from[((r >> 2) * 8 + 2 * (quarter0 + s)) * 128 + (r & 3) * 32];
          acc[s][r] = n ? acc[s][r] * (s2_sign(post, r, lane_m) * __builtin_amdgcn_rcpf((float)n)) : 0.0f;
        }
    }
    if (totals && quarter0 == 0) {   // Sec. 3.4 loss monitoring: gathered in LDS, one atomic per workgroup
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) total += (uint32_t)__builtin_amdgcn_ds_bpermute((lane_m ^ o) << 2, (int)total);   // (__shfl_xor keeps a lane number of its own)
      lds_barrier<8>();
      if (lane == 0) ((uint32_t*)x)[wave] = total;
      lds_barrier<8>();
      if (threadIdx.x == 0) {
        uint32_t n = 0;
        for (int w = 0; w < 8; ++w) n += ((const uint32_t*)x)[w];
        atomicAdd(a.total_out, (unsigned long long)n);
      }
    }
    __builtin_amdgcn_sched_barrier(0);

    if constexpr (NQ == 4) {
      lds_barrier<8>();   // everyone has read what was there
      int lane_t = lane;
      asm volatile("" : "+v"(lane_t));
      decode_64k(acc, x, signs[wave * 64 + lane_t], a, e0, wave, lane_t);
    } else {
      float* to = a.mean_out + e0 + (u64)quarter0 * kQuarterEntries + wave * 2048 + lane * 4;
#pragma unroll
      for (int s = 0; s < NQ; ++s)
#pragma unroll
        for (int r = 0; r < 32; r += 4)
          *(f32x4v*)(to + s * kQuarterEntries + r * 64) = f32x4v{acc[s][r], acc[s][r + 1], acc[s][r + 2], acc[s][r + 3]};
    }
    if (!more) return;
  }
}

static __global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_fused_bf16_64k(PathArgs args) {
  fused_bf16_walk_64k<4>(blockIdx.x, (uint32_t)args.unit0, gridDim.x, 0, args.total_out != nullptr, [&](uint32_t at, PathArgs& a) {
    a = args;
    return (u64)at;
  });
}
static __global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_fused_bf16_batched_64k(BatchArgs ba) {
  int j = bucket_index(ba, blockIdx.x);   // onwards from there by scalar loads
  fused_bf16_walk_64k<4>(blockIdx.x, ba.tile_start[ba.n], gridDim.x, 0, ba.totals != nullptr, [&](uint32_t at, PathArgs& a) {
    while (j + 1 < ba.n && ba.tile_start[j + 1] <= at) ++j;
    bucket_args(ba, a, j);
    return (u64)(at - ba.tile_start[j]);
  });
}
// The blocks from args.unit0 on; 4 / NQ workgroups a block, on one XCD (blockIdx modulo 8) next to each other: they read the same entries
template <int NQ>
static __global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_fused_bf16_split_64k(PathArgs args) {
  const unsigned slot = blockIdx.x >> 3;
  const uint32_t blocks = (uint32_t)(args.n_pad >> 16), blk = (uint32_t)args.unit0 + slot / (4 / NQ) * 8 + (blockIdx.x & 7);
  if (blk >= blocks) return;
  fused_bf16_walk_64k<NQ>(blk, blocks, 0, (int)(slot % (4 / NQ)) * NQ, args.total_out != nullptr, [&](uint32_t at, PathArgs& a) {
    a = args;
    return (u64)at;
  });
}
static __global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_decode_64k(PathArgs a) {
  __shared__ __align__(16) float x[1 << 14];
  const int wave = wave_id(), lane = lane_id();
  const u64 e0 = (a.unit0 + blockIdx.x) << 16;
  float acc[4][32];
  const float* from = a.mean_out + e0 + wave * 2048 + lane * 4;
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int r = 0; r < 32; r += 4) {
      const f32x4v t = *(const f32x4v*)(from + s * kQuarterEntries + r * 64);
      acc[s][r] = t[0]; acc[s][r + 1] = t[1]; acc[s][r + 2] = t[2]; acc[s][r + 3] = t[3];
    }
  const u32x4v sg = signs_64k(a.seed, a.base + e0 + (u64)wave * 8192, (uint8_t*)(x + wave * 2048), lane);
  lds_barrier<8>();
  decode_64k(acc, x, sg, a, e0, wave, lane);
}

}  // namespace ordev

// Prefill path (and large decode batches): the experts of Eq. 1 as an MFMA
// grouped GEMM with the quantised copies (int4 / int2 low copies, the int8
// high copy of an int8 model) dequantised in registers, then the weighted
// combine.
//
//   up:    H[j, r] = silu(X_g W1^T)[j, r] * (X_g W3^T)[j, r]     (fp16 out)
//   down:  E[j, r] = (H_g W2^T)[j, r]                             (fp32 out)
//   combine: y[t] = sum_k w[t,k] * E[pos(t,k)]                    (Eq. 1)
//
// X_g is the group's tokens: the router's stable counting sort lists every
// (token, slot) pair of a work group contiguously (perm[]); the up kernel
// gathers those token rows while staging them in LDS (the permute step),
// and H / E are kept in that group order (row j of the group at position
// offset + j), so the down kernel reads contiguous rows and the combine
// finds each pair through pos[].
//
// What bounds it.  With hundreds of tokens per expert the products do, and
// what feeds them: the LDS port, and the cycles in which a wave issues loads
// instead of products.  With few tokens the HBM stream of the weights does.
// A block is 4 waves, one per SIMD and with the whole unit's registers and
// LDS, and owns 128 RT weight rows (in the up-projection half of them W1, the
// other half the same rows of W3) x up to 256 tokens as
// v_mfma_f32_32x32x16_f16 tiles (weights are the A operand: lane l holds
// A[l%32][8(l/32)+i], B[8(l/32)+i][l%32] and C[8(i/4)+4(l/32)+i%4][l%32]).  A
// wave owns RT tiles of 32 rows and all of the tokens, MT tiles of 32: each
// code is dequantised by one wave, and a block computes no more than 31
// tokens too many.  With the waves 2 x 2 over rows and tokens instead, codes
// were dequantised twice and tokens came in steps of 64: a Mixtral-shaped
// layer took 11 % less time at 512 tokens, 14 % at 64, 3 % at 8192 (all fp16:
// no change, although a step now reads 10 fragments for 16 products, not 8).
//
// Staging.  Both operands go to LDS by direct global-to-LDS loads of 16
// bytes per lane: activations (gathered through the permutation) in stages
// of 64 columns, 8 rows x one full 128-byte line per load; fp16 weights the
// same; codes as they are stored, in units of 64 bytes per row (16 rows per
// load) = 1, 2 or 4 stages of int8, int4 or int2; group scales in units of
// 16 bytes per row = 4 stages.  Each sits in a ring of 3 to 8 slots, the
// weights of the largest fp16 blocks in one of 2 (see Ring).  A code row whose last unit is partial reads its first chunk
// instead, and scales past the row its last dword, which no product uses;
// rows past the matrix or the group repeat the last one and are not stored.
// Nothing outside a row is read.
//
// Bank conflicts.  The 16-byte chunk c of row r sits at position c ^ ((r/2)
// % 8) of a 128-byte LDS row, c ^ ((r/4) % 4) of a 64-byte one (the loads
// permute the source chunks inside the line), so that 16 consecutive rows of
// a fragment read cover the 64 banks: the counters show none, and with the
// swizzle made for 32 banks half of the LDS cycles were conflicts.
//
// Products.  The reduction order inside an MFMA is free as long as both
// operands agree: lane (row = l % 32, half = l / 32) takes columns 32 half +
// 8 s .. + 7 of the stage in step s = 0..3.  A lane's columns of a stage are
// then one quantisation group: 32 int4 codes are one 16-byte read, and the
// lane needs one scale.  Codes become fp16(q * s) in registers after the
// read, in column order.
//
// Pipeline.  Fragments of step s + 1 are read (and converted) between the
// products of step s, two quarters of a step before their use; the barrier
// between stages stands before the last step's products, so that the next
// stage's first fragments are read under those.  A stage's loads are spread
// over the quarters of a stage, one or two each: a load that finds the
// memory pipe full holds up the wave's products.  The loads are inline
// assembly without register results (the compiler would otherwise wait for
// all of them before every LDS read); the waits are explicit counts.
//
// Measured (one layer, up / down-projection, us, sustained, both sides in one
// session; before: 16x16x32 products, 16 or 32 weight rows per wave, 160
// tokens per pass, weights in register rings, activations through LDS):
//   Mixtral shape, 4:3:1 fp16:int4:int2, 8192 tokens 5747 / 3448 -> 3405 /
//   1791 (1.13 and 1.07 PFLOP/s; a large fp16 library GEMM reaches 1.34 -
//   1.48), 512 tokens 406 / 232 -> 363 / 183; half fp16 half int4, 64 tokens
//   336 / 173 -> 278 / 133 (4.3 and 4.5 TB/s); Phi shape, 1337 tokens 664 /
//   354 -> 384 / 161; d 320, f 448, 6 experts, 1337 tokens 53 / 40 -> 16 / 17.
// On the way, at 8192 tokens and fp16 only (up, with a SwiGLU on the
// exponential and reciprocal units from the third figure on): 8 waves of 64
// rows x 128 tokens 3.85 ms; 4 waves 3.70; fragment reads two quarters early
// 3.60; remainders last 3.55; three activation stages instead of two 3.38.
// Blocks in the order of copy widths, or fp16 and narrow ones alternating,
// moved nothing at 512 tokens.
#include <cstddef>

#include "moe_internal.h"

namespace moe {

namespace {

constexpr int kThreads = 256;
constexpr int kStageK = 64;                       // columns per stage, 4 steps of 16
constexpr int kTileTok = 256;                     // tokens per block (MT = 8)
constexpr int kScaleStages = 4;                   // stages per unit of scales
constexpr uint32_t kLdsBytes = 160 * 1024;
constexpr int kMaxSlots = 8;

// Geometry of a block of 128 RT weight rows (a wave: RT tiles of 32) and 32
// MT tokens (every wave: all MT tiles of 32), and its LDS rings: kASlots stages of
// activations (128 bytes of each row), kWSlots units of weights (fp16: 128
// bytes of each row = one stage, codes: 64 bytes = kUnit stages) and of
// scales (16 bytes of each row).  All rings are as deep as the LDS allows;
// the largest fp16 blocks have room for two units of weights, whose loads
// go first in a stage and arrive within it, while the activations have two
// stages.
template <int BITS, int RT, int MT> struct Ring {
  static constexpr int kRows = 128 * RT;
  static constexpr int kSubRows = kRows / 2;       // rows of each of the two sub-blocks
  static constexpr int kRowBytes = BITS == 16 ? 128 : 64;
  static constexpr int kUnit = BITS == 16 ? 1 : 8 / BITS;
  static constexpr uint32_t kASlot = MT * 32 * 128;
  static constexpr uint32_t kWSlot = kRows * kRowBytes;
  static constexpr uint32_t kSSlot = BITS == 16 ? 0 : kRows * 16;
  static constexpr int kFit = (int)(kLdsBytes / (kASlot + kWSlot + kSSlot));
  static constexpr int kASlots = kFit < 3 ? 3 : kFit < kMaxSlots ? kFit : kMaxSlots;
  static constexpr int kWSlots = kFit < 3 ? 2 : kASlots;
  static constexpr uint32_t kWBase = kASlots * kASlot;
  static constexpr uint32_t kSBase = kWBase + kWSlots * kWSlot;
  static_assert(kSBase + kWSlots * kSSlot <= kLdsBytes, "LDS");
  // loads per wave: activations per stage, weights and scales per unit, and
  // the fewest of those that a stage issues
  static constexpr int kALoads = MT;
  static constexpr int kWUnitLoads = RT * kRowBytes / 32;
  static constexpr int kSUnitLoads = BITS == 16 ? 0 : 2 * RT;
  static constexpr int kWLoads = kWUnitLoads / kUnit, kSLoads = kSUnitLoads / kScaleStages;
  static constexpr int kLoads = kWLoads + kSLoads + kALoads;
  // loads that may be in flight when a stage ends: those of the stages
  // after the next one
  static constexpr int kPending = kWSlots == 2 ? kALoads : (kASlots - 2) * kLoads;
};

typedef __attribute__((address_space(3))) uint8_t lds_u8;

// 16 (4) bytes per lane from base + off to LDS at lds + 16 (4) * lane.
// lds and base are wave-uniform.  m0 holds the LDS address; one wait state
// is required between its write and the load.
__device__ inline void lds_load16(uint32_t lds, const uint8_t* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
__device__ inline void lds_load4(uint32_t lds, const uint8_t* base, uint32_t off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :: "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}
// All but the N newest loads of this wave are in LDS and every LDS read of
// it has returned, then the block's barrier.
template <int N>
__device__ inline void stage_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

__device__ inline f16x2 as_h2(uint32_t v) { return __builtin_bit_cast(f16x2, v); }
__device__ inline uint32_t as_u32(f16x2 v) { return __builtin_bit_cast(uint32_t, v); }

constexpr uint32_t kAndOr = 0xEA;  // v_bitop3 truth table of (a & b) | c
__device__ inline uint32_t scaled(uint32_t v, uint32_t bias, f16x2 s2) {
  return as_u32((as_h2(v) - as_h2(bias)) * s2);
}

// A code u whose lowest bit sits at bit p of a 16-bit half, or-ed with the
// exponent of 2^(10-p), is the fp16 number 2^(10-p) + u; a packed subtract
// of 2^(10-p) + 2^(bits-1) and a packed multiply by the scale give fp16(q s).
// frag(q, s): the 8 codes of step s of a lane's 32 (its half of a stage), in
// column order.
template <int BITS> struct Codes;

template <> struct Codes<8> {
  static constexpr int kRaw = 2;  // 16-byte chunks of a lane's 32 codes
  // bytes e0 e1 (e2 e3) of a word with 0x64 above each: 1024 + u
  static __device__ inline f16x8 frag(const u32x4 (&q)[2], int s, f16x2 s2) {
    u32x4 o;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint32_t w = q[s >> 1][(s & 1) * 2 + k];
      o[2 * k] = scaled(__builtin_amdgcn_perm(0x64646464u, w, 0x04010400u), 0x64806480u, s2);
      o[2 * k + 1] = scaled(__builtin_amdgcn_perm(0x64646464u, w, 0x04030402u), 0x64806480u, s2);
    }
    return __builtin_bit_cast(f16x8, o);
  }
};

template <> struct Codes<4> {
  static constexpr int kRaw = 1;
  // byte b of the word (e2b, e2b+1) into bits 0..7 of both halves: u at
  // bit 0 of the low half (1024 + 8), at bit 4 of the high half (64 + 8)
  static __device__ inline f16x8 frag(const u32x4 (&q)[1], int s, f16x2 s2) {
    const uint32_t w = q[0][s];
    u32x4 o;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t t = __builtin_amdgcn_perm(w, w, 0x0C000C00u + (uint32_t)b * 0x00010001u);
      o[b] = scaled(__builtin_amdgcn_bitop3_b32(t, 0x00F0000Fu, 0x54006400u, kAndOr), 0x54806408u, s2);
    }
    return __builtin_bit_cast(f16x8, o);
  }
};

template <> struct Codes<2> {
  static constexpr int kRaw = 1;  // the lane's 8 bytes in the first half
  // half-word s holds e0..e7; byte b (e4b .. e4b+3) into both halves: bits
  // 0 / 2 (1024 + 2, 256 + 2), then bits 4 / 6 (64 + 2, 16 + 2)
  static __device__ inline f16x8 frag(const u32x4 (&q)[1], int s, f16x2 s2) {
    const uint32_t w = q[0][s >> 1];
    u32x4 o;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t t = __builtin_amdgcn_perm(w, w, 0x0C000C00u + (uint32_t)(2 * (s & 1) + b) * 0x00010001u);
      o[2 * b] = scaled(__builtin_amdgcn_bitop3_b32(t, 0x000C0003u, 0x5C006400u, kAndOr), 0x5C086402u, s2);
      o[2 * b + 1] = scaled(__builtin_amdgcn_bitop3_b32(t, 0x00C00030u, 0x4C005400u, kAndOr), 0x4C805420u, s2);
    }
    return __builtin_bit_cast(f16x8, o);
  }
};
template <> struct Codes<16> { static constexpr int kRaw = 1; };

// A wave-uniform pointer in scalar registers.
__device__ inline const uint8_t* uniform(const void* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const uint8_t*>(((uint64_t)hi << 32) | lo);
}

template <class T>
__device__ inline T lds_read(const lds_u8* lds, uint32_t at) {
  return *reinterpret_cast<const __attribute__((address_space(3))) T*>(lds + at);
}

// The two 128-row sub-blocks of a tile: W1 and W3 at the same rows, or two
// consecutive 128-row blocks of W2; rows past `rows` repeat the last one.
struct Sub {
  const uint8_t *w0, *w1;
  const uint8_t *s0, *s1;
  int rows0, rows1;  // rows left in the matrix from the sub-block's first
};

// acc[i][t] (C tile: 32 weight rows x 32 tokens) of the wave's weight tile i
// and token tile t, over all of the ld columns; RT = 2: tile i is 32 rows of
// sub-block i, RT = 1: 16 rows of either.  act: row 0 of the block's activations (gather: x,
// whose rows are perm[...] / K); n tokens.
template <int BITS, int RT, int MT, bool GATHER>
__device__ __forceinline__ void tile_gemm(const Sub& sub, int ld, const f16* act,
                                          const int32_t* perm, int n, int K, lds_u8* lds,
                                          f32x16 (&acc)[RT][MT]) {
  using R = Ring<BITS, RT, MT>;
  const int l = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  const int nst = ld / kStageK;
  const uint32_t row_bytes = (uint32_t)(ld * BITS / 8);
  // load q of a slot covers rows 8 q + l / 8, and position l % 8 of a row
  // holds chunk (l % 8) ^ ((row / 2) % 8); a wave's loads are q = wave + 4 i,
  // so that row / 2 % 8 is 4 (wave % 2) + l / 16
  const uint32_t chunk = 16 * ((l & 7) ^ (4 * (wave & 1) + (l >> 4)));
  // rows of 64 bytes: row 16 q + l / 4, chunk (l % 4) ^ ((row / 4) % 4)
  const uint32_t chunk64 = 16 * ((l & 3) ^ ((l >> 4) & 3));

  uint32_t aoff[R::kALoads];
#pragma unroll
  for (int i = 0; i < R::kALoads; ++i) {
    const int r = min(8 * (wave + 4 * i) + (l >> 3), n - 1);
    const uint32_t src = GATHER ? (uint32_t)(perm[r] / K) : (uint32_t)r;
    aoff[i] = src * (uint32_t)(2 * ld) + chunk;
  }
  const uint8_t* abase = uniform(act);
  // load i of the activations of stage k
  auto load_a = [&](int k, int i, uint32_t slot) {
    lds_load16(lds0 + slot * R::kASlot + (wave + 4 * i) * 1024, abase + (size_t)min(k, nst - 1) * 128,
               aoff[i]);
  };
  // load i of unit u of the weights, the first half of them sub-block 0.  A
  // code row whose last unit is partial reads its first chunk instead.
  auto load_w = [&](int u, int i, uint32_t slot) {
    constexpr int kPer = R::kRowBytes == 128 ? 8 : 16;  // rows per load
    const bool second = i >= R::kWUnitLoads / 2;
    const int r0 = kPer * (wave + 4 * (i % (R::kWUnitLoads / 2))) + (l * kPer >> 6);
    const int r = min(r0, (second ? sub.rows1 : sub.rows0) - 1);
    const uint32_t c0 = (uint32_t)u * R::kRowBytes + (BITS == 16 ? chunk : chunk64);
    const uint32_t c = c0 < row_bytes ? c0 : 0;
    lds_load16(lds0 + R::kWBase + slot * R::kWSlot + (wave + 4 * i) * 1024, second ? sub.w1 : sub.w0,
               (uint32_t)r * row_bytes + c);
  };
  // load p of scale unit v: dword 4 v + l % 4 (two groups each) of rows
  // 64 p + 16 wave + l / 4
  auto load_s = [&](int v, int p, uint32_t slot) {
    const bool second = p >= RT;
    const int r = min(64 * (p % RT) + 16 * wave + (l >> 2), (second ? sub.rows1 : sub.rows0) - 1);
    const int dw = min(4 * v + (l & 3), ld / 64 - 1);
    lds_load4(lds0 + R::kSBase + slot * R::kSSlot + p * 1024 + wave * 256, second ? sub.s1 : sub.s0,
              (uint32_t)r * (uint32_t)(ld / 16) + 4 * dw);
  };

  // the rings' first stages; the loads that the first stage needs come first
#pragma unroll
  for (int v = 0; v < R::kWSlots - 1; ++v) {
#pragma unroll
    for (int p = 0; p < R::kSUnitLoads; ++p) load_s(v, p, v);
#pragma unroll
    for (int i = 0; i < R::kWUnitLoads; ++i) load_w(BITS == 16 ? min(v, nst - 1) : v, i, v);
  }
#pragma unroll
  for (int v = 0; v < R::kASlots - 1; ++v)
#pragma unroll
    for (int i = 0; i < R::kALoads; ++i) load_a(v, i, v);

#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][t][v] = 0.0f;

  const int half = l >> 5;
  const int sw = (l >> 1) & 7, sw64 = (l >> 2) & 3;              // chunk swizzles of this lane's rows
  const uint32_t arow = (uint32_t)(l & 31) * 128;                // token tile 0
  // weight tile 0: RT = 2, 32 rows of sub-block 0 (tile 1: the same rows of
  // sub-block 1); RT = 1, 16 rows of each sub-block
  const uint32_t wrow = RT == 2 ? (uint32_t)(wave * 32 + (l & 31))
                                : (uint32_t)(wave * 16 + (l & 15) + (l & 16 ? R::kSubRows : 0));
  uint32_t cat[4];  // position of the lane's chunk of each step
#pragma unroll
  for (int s = 0; s < 4; ++s) cat[s] = 16 * ((4 * half + s) ^ sw);
  auto tile_row = [](int i) { return (uint32_t)(i * R::kSubRows); };  // tile i, relative to tile 0

  f16x8 a[2][MT], b[2][RT];
  u32x4 q[RT][Codes<BITS>::kRaw];
  f16x2 s2[RT];
  // Fragments of step s of the stage whose slots (and place j in its unit)
  // are given; raw codes and scales are read with step 0.
  auto read_a = [&](int s, int t, uint32_t as) {
    a[s & 1][t] = lds_read<f16x8>(lds, as * R::kASlot + arow + cat[s] + t * 32 * 128);
  };
  auto read_q = [&](int i, int k, uint32_t ws, uint32_t ss) {
    const uint32_t at = R::kWBase + ws * R::kWSlot + (wrow + tile_row(i)) * R::kRowBytes;
    const uint32_t j = (uint32_t)k % R::kUnit;
    if constexpr (BITS == 8) {
#pragma unroll
      for (int h = 0; h < 2; ++h) q[i][h] = lds_read<u32x4>(lds, at + 16 * ((2 * half + h) ^ sw64));
    } else if constexpr (BITS == 4) {
      q[i][0] = lds_read<u32x4>(lds, at + 16 * ((2 * j + half) ^ sw64));
    } else if constexpr (BITS == 2) {
      const u32x2 v = lds_read<u32x2>(lds, at + 16 * (j ^ sw64) + 8 * half);
      q[i][0] = u32x4{v.x, v.y, 0, 0};
    }
    if constexpr (BITS != 16) {
      const uint32_t sc = lds_read<uint16_t>(lds, R::kSBase + ss * R::kSSlot + (wrow + tile_row(i)) * 16 +
                                                      2 * (2 * ((uint32_t)k % kScaleStages) + half));
      s2[i] = as_h2(__builtin_amdgcn_perm(sc, sc, 0x01000100u));
    }
  };
  auto read_w = [&](int s, int i, uint32_t ws) {
    if constexpr (BITS == 16)
      b[s & 1][i] = lds_read<f16x8>(lds, R::kWBase + ws * R::kWSlot + (wrow + tile_row(i)) * 128 + cat[s]);
    else
      b[s & 1][i] = Codes<BITS>::frag(q[i], s, s2[i]);
  };
  auto next = [](uint32_t slot, int slots) { return slot + 1 == (uint32_t)slots ? 0u : slot + 1; };
  // quarter c of the products of step s
  auto products = [&](int s, int c) {
#pragma unroll
    for (int m = c * RT * MT / 4; m < (c + 1) * RT * MT / 4; ++m)
      acc[m % RT][m / RT] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b[s & 1][m % RT], a[s & 1][m / RT],
                                                                   acc[m % RT][m / RT], 0, 0, 0);
  };
  // keeps a quarter's reads and conversions between its products
  auto pin = [&](int c) {
#pragma unroll
    for (int m = c * RT * MT / 4; m < (c + 1) * RT * MT / 4; ++m) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // LDS reads
      __builtin_amdgcn_sched_group_barrier(0x002, BITS == 16 ? 2 : 6, 0);  // VALU
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  uint32_t as = 0, ws = 0, ss = 0;                                         // slots of stage k
  uint32_t al = R::kASlots - 1, wl = R::kWSlots - 1, sl = R::kWSlots - 1;  // slots loaded next
  // Quarter c's share of the loads of one stage, issued between the barrier
  // before stage k and the one in it: weights and scales first.  Past the
  // last stage they repeat it, so that the counts hold.
  auto loads = [&](int k, int c) {
    const int u = BITS == 16 ? min(k + R::kWSlots - 1, nst - 1) : k / R::kUnit + R::kWSlots - 1;
    const int v = k / kScaleStages + R::kWSlots - 1;
    const int j = k % R::kUnit, js = k % kScaleStages;
    constexpr int kSpread = R::kWSlots == 2 ? 16 : 12;
    // slots of a stage for weights and scales; where a unit has fewer loads
    // than stages, every second stage has one
    constexpr int kW = R::kWLoads > 0 ? R::kWLoads : 1;
    constexpr int kS = BITS == 16 ? 0 : 1;
    constexpr int kAll = kW + kS + R::kALoads;
#pragma unroll
    for (int i = c * kAll / kSpread; i < min((c + 1) * kAll / kSpread, kAll); ++i) {
      if (i < kW) {
        if (R::kWLoads > 0) load_w(u, j * R::kWLoads + i, wl);
        else if (j & 1) load_w(u, j >> 1, wl);
      } else if (i < kW + kS) {
        if (R::kSLoads > 0) load_s(v, js, sl);
        else if (js & 1) load_s(v, js >> 1, sl);
      } else {
        load_a(k + R::kASlots - 1, i - kW - kS, al);
      }
    }
  };

  // (deeper rings wait for all: their counts hold from the loop's loads on)
  stage_barrier<R::kASlots == 3 ? R::kALoads : 0>();
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    read_q(i, 0, ws, ss);
    read_w(0, i, ws);
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) read_a(0, t, as);
#pragma unroll
  for (int c = 0; c < 4; ++c) loads(0, c);
  for (int k = 0; k < nst; ++k) {
#pragma unroll
    for (int s = 0; s < 3; ++s) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        loads(k, 4 + 4 * s + c);
        // activation fragments in the first three quarters, each at least two
        // quarters before its use; codes one tile per quarter
#pragma unroll
        for (int t = 0; t < MT; ++t)
          if (3 * t / MT == c) read_a(s + 1, t, as);
#pragma unroll
        for (int i = 0; i < RT; ++i)
          if (c == (BITS == 16 ? 0 : i + 1)) read_w(s + 1, i, ws);
        products(s, c);
        pin(c);
      }
    }
    // every load of stage k + 1 has arrived; the slots of stage k are free
    stage_barrier<R::kPending>();
    as = next(as, R::kASlots);
    al = next(al, R::kASlots);
    if ((k + 1) % R::kUnit == 0) {
      ws = next(ws, R::kWSlots);
      wl = next(wl, R::kWSlots);
    }
    if ((k + 1) % kScaleStages == 0) {
      ss = next(ss, R::kWSlots);
      sl = next(sl, R::kWSlots);
    }
    // (after the last stage: reads that are not multiplied)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      loads(k + 1, c);
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        if (c == 0 && BITS != 16) read_q(i, k + 1, ws, ss);
        if (c == (BITS == 16 ? 0 : i + 2)) read_w(0, i, ws);
      }
#pragma unroll
      for (int t = 0; t < MT; ++t)
        if (3 * t / MT == c) read_a(0, t, as);
      products(3, c);
      pin(c);
    }
  }
  // the LDS must not be handed on with loads in flight
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The SwiGLU's gate, as in the decode kernels: 4e-8 rms and 1.8e-7 at most
// from 64 bits.  On the exponential and reciprocal units alone the rounding of
// the exponent's product adds |a| 2^-24: 1.7e-7 rms and 1.8e-6 at most for
// a ~ N(0, 8^2).  That loses precision, although it takes 1 to 4 % less time
// (a call of the Mixtral shape, 8192 tokens 5.24 / 5.33 ms, 512 tokens 551 /
// 561 us; d 320, f 448, 1337 tokens 47.5 / 49.6 us).  expf with the quotient
// by a corrected reciprocal is as exact and gains up to 1 %, but infinities
// and quotients below 2^-126 then need a select each, which takes that back.
__device__ inline float silu(float a) { return a / (1.0f + expf(-a)); }

// Work item of a block: a group's token tile and a row tile.  Items are
// listed in two runs: first the tiles of all groups that take the largest
// block (more than 192 tokens), then the smaller remainders, so that the
// small ones fill the last round.  Inside a group, up to kSuper token tiles
// alternate fastest: the blocks that run together on an XCD share weight
// rows and token rows.  The hardware hands block b to XCD b % 8: whole sets
// of 256 items (one per compute unit) go to the XCDs in runs of 32, what is
// left in eighths, so that every XCD gets the same mix of copies.
struct Item {
  Group g;
  int tok0, tile;
};
constexpr int kSuper = 8;

// Inclusive sum over the lanes up to this one (DPP row shifts, then the row
// ends broadcast to the rows above).
template <int CTRL, int ROWS>
__device__ inline int dpp_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false);
}
__device__ inline int wave_scan(int v) {
  v = dpp_add<0x111, 0xF>(v);  // row_shr:1
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  v = dpp_add<0x118, 0xF>(v);
  v = dpp_add<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
}

// Slots per XCD for n items, and the item of an XCD's slot (-1: none).
__device__ inline int xcd_slots(int n) { return (n >> 8) * 32 + (((n & 255) + 7) >> 3); }
__device__ inline int xcd_item(int n, int xcd, int slot) {
  const int sets = n >> 8, left = n & 255, per = (left + 7) >> 3;
  if (slot < 32 * sets) return (slot >> 5) * 256 + xcd * 32 + (slot & 31);
  const int q = slot - 32 * sets, item = xcd * per + q;
  return q < per && item < left ? 256 * sets + item : -1;
}

__device__ inline bool take_item(const WorkList* wl, int n_tiles, Item& it) {
  // Lane l takes groups 2 l and 2 l + 1; entries past the list hold stale
  // groups and count nothing.  One memory round trip: the block's group is
  // read from the lane that holds it.
  const int lane = threadIdx.x & 63;
  const u32x4 g0 = reinterpret_cast<const u32x4*>(wl->groups)[2 * lane];
  const u32x4 g1 = reinterpret_cast<const u32x4*>(wl->groups)[2 * lane + 1];
  const int ng = wl->n_groups;
  const int cnt0 = 2 * lane < ng ? (int)g0.w : 0, cnt1 = 2 * lane + 1 < ng ? (int)g1.w : 0;
  const int rem0 = cnt0 % kTileTok, rem1 = cnt1 % kTileTok;
  const int big0 = cnt0 / kTileTok + (rem0 > 192), big1 = cnt1 / kTileTok + (rem1 > 192);
  const int rest0 = rem0 > 0 && rem0 <= 192, rest1 = rem1 > 0 && rem1 <= 192;
  // token tiles of both runs in one scan (at most 2^16 / 256 and 128)
  const int scan = wave_scan((big0 + big1) | (rest0 + rest1) << 16);
  const int all = __builtin_amdgcn_readlane(scan, 63);
  const int n_big = (all & 0xFFFF) * n_tiles, n_rest = (all >> 16) * n_tiles;
  const int slot = blockIdx.x >> 3, xcd = blockIdx.x & 7;
  const int per_big = xcd_slots(n_big);
  const bool small = slot >= per_big;
  const int item = small ? xcd_item(n_rest, xcd, slot - per_big) : xcd_item(n_big, xcd, slot);
  if (item < 0) return false;
  const int upto = small ? scan >> 16 : scan & 0xFFFF;  // token tiles up to this lane's groups
  const int own0 = small ? rest0 : big0, own1 = small ? rest1 : big1;
  const int gl = __ffsll((unsigned long long)__ballot(upto * n_tiles > item)) - 1;
  const int o0 = __builtin_amdgcn_readlane(own0, gl), o1 = __builtin_amdgcn_readlane(own1, gl);
  int in = item - (__builtin_amdgcn_readlane(upto, gl) - o0 - o1) * n_tiles;
  const bool odd = in >= o0 * n_tiles;
  if (odd) in -= o0 * n_tiles;
  const u32x4 g = odd ? g1 : g0;
  it.g.expert = __builtin_amdgcn_readlane((int)g.x, gl);
  it.g.bits = __builtin_amdgcn_readlane((int)g.y, gl);
  it.g.offset = __builtin_amdgcn_readlane((int)g.z, gl);
  it.g.count = __builtin_amdgcn_readlane((int)g.w, gl);
  const int tt = odd ? o1 : o0;  // the group's token tiles in this run
  const int sup = in / (kSuper * n_tiles), left = in - sup * (kSuper * n_tiles);
  const int width = min(kSuper, tt - sup * kSuper);
  it.tile = __builtin_amdgcn_readfirstlane(left / width);
  const int t = sup * kSuper + left - it.tile * width;
  it.tok0 = __builtin_amdgcn_readfirstlane((small ? it.g.count / kTileTok : t) * kTileTok);
  return true;
}
static_assert(sizeof(Group) == 16 && offsetof(WorkList, groups) % 16 == 0 && kMaxKeys == 128,
              "two groups per lane");

// First row `row` of matrix M: weights (codes) and scales.
template <int BITS, int M>
__device__ inline const uint8_t* weights_at(const ExpertEntry& ex, int64_t row, int64_t ld) {
  const uint8_t* w = BITS == 16 ? reinterpret_cast<const uint8_t*>(ex.w[M]) : BITS == 8 ? ex.hq[M] : ex.q[M];
  return uniform(w + row * (ld * BITS / 8));
}
template <int BITS, int M>
__device__ inline const uint8_t* scales_at(const ExpertEntry& ex, int64_t row, int64_t ld) {
  if (BITS == 16) return nullptr;
  return uniform((BITS == 8 ? ex.hs[M] : ex.s[M]) + row * (ld / kGroup));
}

template <int BITS, int RT, int MT>
__device__ __forceinline__ void up_tile(const ExpertEntry& ex, const Item& it, const int32_t* perm,
                                        const f16* x, f16* h, int d, int f, int K, lds_u8* lds) {
  const int n = min(kTileTok, it.g.count - it.tok0);
  const int64_t row0 = (int64_t)it.tile * (64 * RT);
  const Sub sub = {weights_at<BITS, 0>(ex, row0, d), weights_at<BITS, 1>(ex, row0, d),
                   scales_at<BITS, 0>(ex, row0, d), scales_at<BITS, 1>(ex, row0, d),
                   f - (int)row0, f - (int)row0};
  f32x16 acc[RT][MT];
  const int off = it.g.offset + it.tok0;
  tile_gemm<BITS, RT, MT, true>(sub, d, x, perm + off, n, K, lds, acc);
  const int l = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = row0 + wave * (16 * RT);
  if (row >= f) return;
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const int j = 32 * t + (l & 31);
    if (j < n) {
      f16* out = h + (int64_t)(off + j) * f + row + 4 * (l >> 5);
#pragma unroll
      for (int q = 0; q < 2 * RT; ++q) {
        f16x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float a = acc[0][t][4 * q + i];
          const float b = RT == 2 ? acc[RT - 1][t][4 * q + i] : acc[0][t][8 + 4 * (q & 1) + i];
          v[i] = (f16)(silu(a) * b);
        }
        *reinterpret_cast<f16x4*>(out + 8 * q) = v;
      }
    }
  }
}

template <int BITS, int RT, int MT>
__device__ __forceinline__ void down_tile(const ExpertEntry& ex, const Item& it, const f16* h,
                                          float* e, int d, int f, lds_u8* lds) {
  const int n = min(kTileTok, it.g.count - it.tok0);
  const int row0 = it.tile * (128 * RT);
  // a tile whose second half lies past the matrix reads the first half's rows
  const int row1 = row0 + 64 * RT < d ? row0 + 64 * RT : row0;
  const Sub sub = {weights_at<BITS, 2>(ex, row0, f), weights_at<BITS, 2>(ex, row1, f),
                   scales_at<BITS, 2>(ex, row0, f), scales_at<BITS, 2>(ex, row1, f),
                   d - row0, d - row1};
  f32x16 acc[RT][MT];
  const int64_t off = it.g.offset + it.tok0;
  tile_gemm<BITS, RT, MT, false>(sub, f, h + off * f, nullptr, n, 1, lds, acc);
  const int l = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int b = 0; b < 2; ++b) {  // the wave's 16 RT rows of each sub-block
    const int row = row0 + b * (64 * RT) + wave * (16 * RT);
    if (row >= d) continue;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int j = 32 * t + (l & 31);
      if (j < n) {
        float* out = e + (off + j) * d + row + 4 * (l >> 5);
#pragma unroll
        for (int q = 0; q < 2 * RT; ++q) {
          const f32x16& c = acc[RT == 2 ? b : 0][t];
          const int v = RT == 2 ? 4 * q : 8 * b + 4 * (q & 1);
          *reinterpret_cast<f32x4*>(out + 8 * q) = f32x4{c[v], c[v + 1], c[v + 2], c[v + 3]};
        }
      }
    }
  }
}

template <int BITS, int RT>
__device__ __forceinline__ void up_item(const ExpertEntry& ex, const Item& it, const int32_t* perm,
                                        const f16* x, f16* h, int d, int f, int K, lds_u8* lds) {
  switch (min((it.g.count - it.tok0 + 31) / 32, 8)) {
    case 1: return up_tile<BITS, RT, 1>(ex, it, perm, x, h, d, f, K, lds);
    case 2: return up_tile<BITS, RT, 2>(ex, it, perm, x, h, d, f, K, lds);
    case 3: return up_tile<BITS, RT, 3>(ex, it, perm, x, h, d, f, K, lds);
    case 4: return up_tile<BITS, RT, 4>(ex, it, perm, x, h, d, f, K, lds);
    case 5: return up_tile<BITS, RT, 5>(ex, it, perm, x, h, d, f, K, lds);
    case 6: return up_tile<BITS, RT, 6>(ex, it, perm, x, h, d, f, K, lds);
    case 7: return up_tile<BITS, RT, 7>(ex, it, perm, x, h, d, f, K, lds);
    default: return up_tile<BITS, RT, 8>(ex, it, perm, x, h, d, f, K, lds);
  }
}

template <int BITS, int RT>
__device__ __forceinline__ void down_item(const ExpertEntry& ex, const Item& it, const f16* h,
                                          float* e, int d, int f, lds_u8* lds) {
  switch (min((it.g.count - it.tok0 + 31) / 32, 8)) {
    case 1: return down_tile<BITS, RT, 1>(ex, it, h, e, d, f, lds);
    case 2: return down_tile<BITS, RT, 2>(ex, it, h, e, d, f, lds);
    case 3: return down_tile<BITS, RT, 3>(ex, it, h, e, d, f, lds);
    case 4: return down_tile<BITS, RT, 4>(ex, it, h, e, d, f, lds);
    case 5: return down_tile<BITS, RT, 5>(ex, it, h, e, d, f, lds);
    case 6: return down_tile<BITS, RT, 6>(ex, it, h, e, d, f, lds);
    case 7: return down_tile<BITS, RT, 7>(ex, it, h, e, d, f, lds);
    default: return down_tile<BITS, RT, 8>(ex, it, h, e, d, f, lds);
  }
}

template <int RT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
void prefill_up_kernel(const ExpertEntry* __restrict__ table, const WorkList* __restrict__ wl,
                            const int32_t* __restrict__ perm, const f16* __restrict__ x,
                            f16* __restrict__ h, int d, int f, int K, int n_tiles) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kLdsBytes];
  lds_u8* lds = (lds_u8*)smem;
  Item it;
  if (!take_item(wl, n_tiles, it)) return;
  const ExpertEntry ex = table[it.g.expert];
  if (it.g.bits == 16) up_item<16, RT>(ex, it, perm, x, h, d, f, K, lds);
  else if (it.g.bits == 8) up_item<8, RT>(ex, it, perm, x, h, d, f, K, lds);
  else if (it.g.bits == 4) up_item<4, RT>(ex, it, perm, x, h, d, f, K, lds);
  else up_item<2, RT>(ex, it, perm, x, h, d, f, K, lds);
}

template <int RT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
void prefill_down_kernel(const ExpertEntry* __restrict__ table, const WorkList* __restrict__ wl,
                              const f16* __restrict__ h, float* __restrict__ e, int d, int f,
                              int n_tiles) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kLdsBytes];
  lds_u8* lds = (lds_u8*)smem;
  Item it;
  if (!take_item(wl, n_tiles, it)) return;
  const ExpertEntry ex = table[it.g.expert];
  if (it.g.bits == 16) down_item<16, RT>(ex, it, h, e, d, f, lds);
  else if (it.g.bits == 8) down_item<8, RT>(ex, it, h, e, d, f, lds);
  else if (it.g.bits == 4) down_item<4, RT>(ex, it, h, e, d, f, lds);
  else down_item<2, RT>(ex, it, h, e, d, f, lds);
}

// One block per token; thread i owns the float4 pieces i, i + 1024, ... of
// the token's row (d is a multiple of 64): y[t] = sum_k w[t,k] *
// E[pos(t,k)] in slot order (skip -> 0); with h_res: h_res[t] += that and,
// with x_next, x_next[t] = fp16(rmsnorm(h_res[t])) by rmsnorm_rows (the
// same piece layout, so each thread reads back the pieces it wrote).
constexpr int kCombineThreads = kNormThreads;

__global__ __launch_bounds__(kCombineThreads) void combine_prefill_kernel(
    const float* __restrict__ e, const int32_t* __restrict__ pos,
    const float* __restrict__ w, const int8_t* __restrict__ prec, int d, int K,
    float* __restrict__ y, float* __restrict__ h_res, f16* __restrict__ x_next,
    float eps) {
  __shared__ float red[kCombineThreads / 64];
  __shared__ int s_pos[kMaxTopK];
  __shared__ float s_w[kMaxTopK];
  const int t = blockIdx.x;
  if (threadIdx.x < K) {
    const int p = t * K + threadIdx.x;
    s_pos[threadIdx.x] = prec[p] == PREC_SKIP ? -1 : pos[p];
    s_w[threadIdx.x] = w[p];
  }
  __syncthreads();
  const int64_t base = (int64_t)t * d;
  const int n4 = d >> 2;
#pragma unroll
  for (int i = 0; i < kNormPieces; ++i) {
    const int q = threadIdx.x + i * kCombineThreads;
    if (q < n4) {
      const int c = 4 * q;
      f32x4 acc = {0, 0, 0, 0};
      for (int k = 0; k < K; ++k)
        if (s_pos[k] >= 0) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(e + (int64_t)s_pos[k] * d + c);
          acc += s_w[k] * v;
        }
      if (h_res) {
        f32x4* hp = reinterpret_cast<f32x4*>(h_res + base + c);
        *hp = *hp + acc;
      } else {
        *reinterpret_cast<f32x4*>(y + base + c) = acc;
      }
    }
  }
  if (!h_res || !x_next) return;  // no norm asked for (the next layer forms it)
  rmsnorm_rows<1, kNormPieces>(h_res + base, d, eps, 0, 1, red,
                               [&](int, int q, uint32_t lo, uint32_t hi) {
                                 *reinterpret_cast<u32x2*>(x_next + base + 4 * q) = u32x2{lo, hi};
                               });
}

// Blocks for any work list: full token tiles of all the pairs and one
// remainder per group, each run rounded up to whole eighths.
int max_blocks(int T, int K, int max_groups, int n_tiles) {
  return (((T * K / kTileTok + max_groups) * n_tiles + 7) / 8 + 1) * 8;
}

// Blocks of 256 weight rows where the step is expected to have enough of
// them, of 128 rows otherwise.  The step's token tiles: one per group of
// fewer than 256 tokens, half a tile more than its tokens fill otherwise.
// The larger blocks read less from L2 and LDS per product, but fewer than
// about 144 of them (9/16 of the 256 compute units) leave too much of the
// chip idle.  Measured with 256 / 128 rows, us, half of the experts fp16 and
// half int4: down-projection of the Mixtral-shaped layer at 64 and 512 tokens
// (128 larger blocks) 183 / 132 and 246 / 181, of the Phi-shaped one at 512
// (256) 129 / 141; up-projection at d 1024, f 2048, 8 experts, 512 tokens
// (128) 28.8 / 22.9, 1024 tokens (192) 36.9 / 38.9, Mixtral-shaped at 512
// tokens (896) 369 / 382, at 8192 (4:3:1) 3280 / 3924.
bool large_blocks(int T, int K, int E, int n_tiles) {
  const int P = T * K, g = P < E ? P : E;
  const int filled = P / kTileTok + g / 2;
  return (int64_t)(filled > g ? filled : g) * n_tiles >= 144;
}

}  // namespace

hipError_t launch_prefill_up(const ExpertEntry* table, const WorkList* wl, const int32_t* perm,
                             const f16* x, f16* h, int T, int d, int f, int E, int K,
                             int max_groups, hipStream_t s) {
  // whole stages and whole 32-row tiles
  if (d % kStageK || f % 32) return hipErrorInvalidValue;
  const int n_large = (f + 127) / 128, n_small = (f + 63) / 64;
  if (large_blocks(T, K, E, n_large))
    prefill_up_kernel<2><<<max_blocks(T, K, max_groups, n_large), kThreads, 0, s>>>(
        table, wl, perm, x, h, d, f, K, n_large);
  else
    prefill_up_kernel<1><<<max_blocks(T, K, max_groups, n_small), kThreads, 0, s>>>(
        table, wl, perm, x, h, d, f, K, n_small);
  return hipGetLastError();
}

hipError_t launch_prefill_down(const ExpertEntry* table, const WorkList* wl, const f16* h,
                               float* e, int T, int d, int f, int E, int K, int max_groups,
                               hipStream_t s) {
  if (f % kStageK || d % 32) return hipErrorInvalidValue;
  const int n_large = (d + 255) / 256, n_small = (d + 127) / 128;
  if (large_blocks(T, K, E, n_large))
    prefill_down_kernel<2><<<max_blocks(T, K, max_groups, n_large), kThreads, 0, s>>>(
        table, wl, h, e, d, f, n_large);
  else
    prefill_down_kernel<1><<<max_blocks(T, K, max_groups, n_small), kThreads, 0, s>>>(
        table, wl, h, e, d, f, n_small);
  return hipGetLastError();
}

hipError_t launch_combine_prefill(const float* e, const int32_t* pos, const float* w,
                                  const int8_t* prec, int T, int d, int K, float* y,
                                  float* h_res, f16* x_next, float eps, hipStream_t s) {
  combine_prefill_kernel<<<T, kCombineThreads, 0, s>>>(e, pos, w, prec, d, K, y, h_res, x_next, eps);
  return hipGetLastError();
}

}  // namespace moe

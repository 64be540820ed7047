// Group-wise symmetric quantiser producing the quantised expert copies
// (Section 2.2 and Section 4.1 "Configurations": int4 replaces fp16, int2
// replaces int8; the int8 copy itself is the high precision of an int8
// model).  Format: group of 32 consecutive weights along a row,
// s = fp16_rne(max|w| / qmax), q = clamp(rne(w / s), -2^(b-1), qmax),
// stored offset-binary and packed little-endian within each byte.
//
// Exactness: w and s are fp16, so w / s is never within 2^-13 of a
// half-integer unless it is one.  max|w| / 7 and max|w| / 127 have binary
// expansions of period 3 and 7 (or are exact), so rounding them to fp32 and
// then to fp16 cannot land on an fp16 midpoint (that needs a run of 12 equal
// bits): the double rounding equals a single rounding, and that division is
// correctly rounded (__fdiv_rn).  The codes' quotients are formed as
// q = w * r, q += (w - q s) * r with r = 1 / s to 1 ulp: quotients are below
// 200 (a subnormal s may be rounded down by a third), so q is within 2^-14
// of w / s after the first product and within an ulp after the second, which
// decides every quotient that is not half-way; where w / s is a half-integer
// it is an fp32 number, w - q s is exact (fma) and the correction lands on it
// exactly, so rintf sees the tie.  A scale of zero (codes 0) or infinity
// takes the plain division.
//
// What bounds it: the bytes, if the arithmetic stays out of the way.  Four
// lanes share a group, 8 weights each, so that loads (16 bytes a lane), codes
// and scales are contiguous over a wave, and a thread has four groups' loads
// in flight.  Weights and codes pass once: both go with the streaming hint.
// A [14336, 4096] matrix to int4 (151 MB): 34.6 -> 26.2 us = 5.75 TB/s (one
// thread per group with 32 plain divisions before); plain loads 30.1, plain
// stores 28.0, eight groups per thread 29.6; int8 37.3 -> 30.9, int2 32.4 ->
// 25.6 us.
#include "moe_internal.h"

namespace moe {

namespace {

constexpr int kThreads = 256;
constexpr int kChunks = 4;                               // groups per thread
constexpr int kBlockGroups = kThreads / 4 * kChunks;     // 256

// max over the four lanes of a quad
__device__ inline float quad_max(float v) {
  v = fmaxf(v, dpp_f<0xB1>(v));  // quad_perm [1,0,3,2]
  return fmaxf(v, dpp_f<0x4E>(v));  // quad_perm [2,3,0,1]
}

}  // namespace

// Wave w of a block takes 64 groups: chunk c of lane l is weights 8 (l % 4)
// .. + 7 of group 16 c + l / 4.
template <int BITS>
__global__ __launch_bounds__(kThreads) void quantize_kernel(
    const f16* __restrict__ w, int64_t n_groups, uint8_t* __restrict__ codes,
    f16* __restrict__ scales) {
  constexpr int kQmax = (1 << (BITS - 1)) - 1;
  constexpr int kQmin = -(1 << (BITS - 1));
  constexpr int kOff = 1 << (BITS - 1);
  const int lane = threadIdx.x & 63;
  const int64_t g0 = (int64_t)blockIdx.x * kBlockGroups + (threadIdx.x >> 6) * 64;
  u32x4 raw[kChunks];
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const int64_t g = g0 + 16 * c + (lane >> 2);
    raw[c] = g < n_groups ? __builtin_nontemporal_load(
                                reinterpret_cast<const u32x4*>(w + g * kGroup) + (lane & 3))
                          : u32x4{0, 0, 0, 0};
  }
  f16 own = (f16)0.0f;
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    const int64_t g = g0 + 16 * c + (lane >> 2);
    const f16x8 h = __builtin_bit_cast(f16x8, raw[c]);
    float m = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) m = fmaxf(m, fabsf((float)h[j]));
    const f16 s16 = (f16)__fdiv_rn(quad_max(m), (float)kQmax);  // RNE to fp16
    const float s = (float)s16;
    if ((lane & 3) == c) own = s16;
    const bool plain = !(s > 0.0f && s < __builtin_inff());
    const float r = __builtin_amdgcn_rcpf(s);
    float q[8];
    if (!plain) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float v = (float)h[j], a = v * r;
        q[j] = rintf(fmaf(fmaf(-a, s, v), r, a));  // ties to even
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) q[j] = s > 0.0f ? rintf(__fdiv_rn((float)h[j], s)) : 0.0f;
    }
    uint32_t out[2] = {0u, 0u};  // 8 codes, packed from bit 0
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float v = fminf(fmaxf(q[j], (float)kQmin), (float)kQmax);
      // v + offset as the low bits of 2^23 + ... (exact)
      const uint32_t u = __builtin_bit_cast(uint32_t, v + (float)(8388608 + kOff));
      out[j * BITS >> 5] |= (u & ((1u << BITS) - 1)) << (j * BITS & 31);
    }
    if (g < n_groups) {
      uint8_t* dst = codes + g * (4 * BITS) + (lane & 3) * BITS;
      if (BITS == 8) __builtin_nontemporal_store(u32x2{out[0], out[1]}, reinterpret_cast<u32x2*>(dst));
      else if (BITS == 4) __builtin_nontemporal_store(out[0], reinterpret_cast<uint32_t*>(dst));
      else __builtin_nontemporal_store((uint16_t)out[0], reinterpret_cast<uint16_t*>(dst));
    }
  }
  // lane l holds the scale of group 16 (l % 4) + l / 4
  const int64_t g = g0 + 16 * (lane & 3) + (lane >> 2);
  if (g < n_groups) scales[g] = own;
}

hipError_t launch_quantize(const f16* w, int64_t rows, int64_t cols, int bits,
                           uint8_t* codes, f16* scales, hipStream_t s) {
  const int64_t n_groups = rows * (cols / kGroup);
  if (n_groups == 0) return hipSuccess;
  const int threads = kThreads;
  const int64_t blocks = (n_groups + kBlockGroups - 1) / kBlockGroups;
  if (bits == 8)
    quantize_kernel<8><<<dim3((unsigned)blocks), dim3(threads), 0, s>>>(
        w, n_groups, codes, scales);
  else if (bits == 4)
    quantize_kernel<4><<<dim3((unsigned)blocks), dim3(threads), 0, s>>>(
        w, n_groups, codes, scales);
  else
    quantize_kernel<2><<<dim3((unsigned)blocks), dim3(threads), 0, s>>>(
        w, n_groups, codes, scales);
  return hipGetLastError();
}

// Stream-ordered update of one expert table entry (value passed by kernel
// argument, so no host buffer has to outlive the call).
__global__ void set_entry_kernel(ExpertEntry* table, int e, ExpertEntry v) {
  if (threadIdx.x == 0) table[e] = v;
}

hipError_t launch_set_entry(ExpertEntry* table, int e, ExpertEntry v,
                            hipStream_t s) {
  set_entry_kernel<<<1, 64, 0, s>>>(table, e, v);
  return hipGetLastError();
}

}  // namespace moe

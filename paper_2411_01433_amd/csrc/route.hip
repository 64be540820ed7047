// Gating and the token-level precision decision.
//
//   logits l[t, e] = sum_d x[t, d] Wg[e, d]           (Eq. 1 gate, fp32 acc)
//   top-k by (l desc, index asc); w = softmax over the K selected logits
//   (Section 3.2: the gate values are normalised)
//   Eq. 2: with slots already in descending gate order, s_0 = 0 and
//   s_j = sum_{i<j} w_i; miss-tagged experts run high if s <= t1, low if
//   t1 < s <= t2, are skipped if s > t2; slot 0 is always high.
//
// Then a work list groups the (token, slot) pairs by (expert, precision):
// a stable counting sort over pair ids p = t*K + k, so pair order inside a
// group follows token order and the result is deterministic.
#include "moe_internal.h"

namespace moe {

namespace {

constexpr int kRouteThreads = 1024;
// Most tokens of a step that one block routes.  With more, a block per token
// and a second kernel for the work list: from 9 tokens on that is faster but
// for a few tokens of few experts.  Whole steps by one block / by both, us, at
// 9 and 16 tokens: d 256, 8 experts 18.0 / 18.9, 20.4 / 19.2; d 1024, 8
// experts 29.3 / 28.8, 33.0 / 30.2; d 4096, 16 experts (f 6400) 228 / 218, 275
// / 258; d 512, 64 experts 45.9 / 36.6, 60.2 / 42.7.  With the norm formed by
// the router block (one launch instead of three): d 256 22.6 / 21.6, 27.3 /
// 22.0; d 2048, 8 experts (f 4096) 73.0 / 69.7, 83.3 / 74.7.
constexpr int kRouteSmallTokens = 8;
static_assert(kMaxExperts <= kRouteThreads, "one thread per expert stages the table");
constexpr int kRouteWaves = kRouteThreads / 64;
constexpr int kRowChunks = 8;     // 512-column chunks of a row held in registers at once

// fp16-pair dot product with fp32 accumulation.  The operands are taken
// as scalars on purpose: clang's __builtin_bit_cast applied directly to a
// vector component expression (v.y) reads component 0.
__device__ inline float dot2(uint32_t a, uint32_t b, float acc) {
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, a),
                                __builtin_bit_cast(f16x2, b), acc, false);
}

// Wave sums use wave_sum_dpp (moe_internal.h): the decode and prefill
// routers sum their logits with it, so their logits stay bit-identical.

// Dot products of tokens [t0, t1) against all E gate rows.  One wave per
// (expert, batch of up to TB tokens): the gate row chunk is loaded once and
// used for every token of the batch; KB chunks of 512 columns (8 fp16 per
// lane) of the gate row and of each token are loaded before any arithmetic
// so that the loads overlap (one memory latency per KB chunks).  Results go
// to lg[t-t0][e].
template <int TB, int KB>
__device__ void gate_logits(const RouteParams& p, int t0, int t1, float* lg) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int n_waves = blockDim.x >> 6;
  const int n_tb = (t1 - t0 + TB - 1) / TB;
  const int n_items = n_tb * p.E;
  for (int q = wave; q < n_items; q += n_waves) {
    const int e = q % p.E;
    const int tb0 = t0 + (q / p.E) * TB;
    const int nt = min(TB, t1 - tb0);
    const f16* gr = p.wg + (int64_t)e * p.d;
    float acc[TB];
#pragma unroll
    for (int i = 0; i < TB; ++i) acc[i] = 0.0f;
    for (int c0 = 0; c0 < p.d; c0 += KB * 512) {
      u32x4 b[KB], a[TB][KB];
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        const int c = c0 + j * 512 + lane * 8;
        b[j] = c < p.d ? *reinterpret_cast<const u32x4*>(gr + c) : u32x4{0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < TB; ++i)
          a[i][j] = (i < nt && c < p.d)
                        ? *reinterpret_cast<const u32x4*>(p.x + (int64_t)(tb0 + i) * p.d + c)
                        : u32x4{0, 0, 0, 0};
      }
#pragma unroll
      for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int j = 0; j < KB; ++j) {
          acc[i] = dot2(a[i][j].x, b[j].x, acc[i]);
          acc[i] = dot2(a[i][j].y, b[j].y, acc[i]);
          acc[i] = dot2(a[i][j].z, b[j].z, acc[i]);
          acc[i] = dot2(a[i][j].w, b[j].w, acc[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < TB; ++i) {
      const float v = wave_sum_dpp(acc[i]);
      if (lane == 0 && i < nt) lg[(tb0 - t0 + i) * p.E + e] = v;
    }
  }
}

// Copy widths of one expert packed in one int: low copy (4, 2 or 0) in
// bits 0-7, high copy (16 or 8) in bits 8-15.
__device__ inline int pack_widths(const ExpertEntry& x) { return x.low_bits | (x.hi_bits << 8); }
__device__ inline int copy_bits(int widths, int low) { return low ? (widths & 0xFF) : (widths >> 8); }

// One expert's tag and copy widths per thread (E is at most 64, below the
// block size): the loads are issued before the gate loads and the LDS stores
// come after them, so the two memory round trips overlap.
struct TableRow {
  int tag, widths;
  __device__ inline void load(const RouteParams& p) {
    const int e = threadIdx.x;
    tag = e < p.E ? p.table[e].tag : 0;
    widths = e < p.E ? pack_widths(p.table[e]) : 0;
  }
  __device__ inline void store(const RouteParams& p, int* tags, int* wd) const {
    if ((int)threadIdx.x < p.E) {
      tags[threadIdx.x] = tag;
      wd[threadIdx.x] = widths;
    }
  }
};

// ---- decode fast path ------------------------------------------------------
// When the step's activations fit in LDS (T*d*2 <= 64 KiB) and d <= 4096
// (8 chunks of 512 columns per lane in registers), the gate takes
// one memory round trip: each wave issues the loads of its expert row (lane
// l holds columns 512j + 8l .. +7 of chunk j), the block stages x in LDS,
// and every token's logit is summed over the chunks in the same order as
// gate_logits, so the logits are bit-identical to the other routers'.
constexpr int kFastXBytes = 64 * 1024;
constexpr int kFastChunks = 8;  // 512-column chunks held in registers at once
constexpr int kNormBatch = 4;   // tokens per round of the fused RMSNorm
static_assert(kRouteThreads == kNormThreads, "the fused RMSNorm runs on the whole router block");

__host__ __device__ inline bool fast_gate(int T, int d) { return (int64_t)T * d * 2 <= kFastXBytes && d <= kFastChunks * 512; }

__device__ void gate_fast(const RouteParams& p, f16* xs, float* lg) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int kW = kRouteThreads / 64;
  const int nch = (p.d + 511) / 512;
  const int e0 = wave;
  // first group of chunks of this wave's first expert row, before staging
  u32x4 b[kFastChunks];
#pragma unroll
  for (int j = 0; j < kFastChunks; ++j) {
    const int c = j * 512 + lane * 8;
    b[j] = (e0 < p.E && j < nch && c < p.d)
               ? *reinterpret_cast<const u32x4*>(p.wg + (int64_t)e0 * p.d + c)
               : u32x4{0, 0, 0, 0};
  }
  if (p.h_res) {
    // x = fp16(rmsnorm(h_res)), formed here as the residual glue's norm
    // kernel forms it (same sums, same order: bit-identical), written to
    // x_out for the expert kernels and staged in LDS for the gate
    __shared__ float red[kNormBatch * (kNormThreads / 64)];
    for (int t0 = 0; t0 < p.T; t0 += kNormBatch)
      rmsnorm_rows<kNormBatch, 1>(p.h_res, p.d, p.eps, t0, min(kNormBatch, p.T - t0), red,
                                  [&](int t, int q, uint32_t lo, uint32_t hi) {
                                    const int64_t o = (int64_t)t * p.d + 4 * q;
                                    *reinterpret_cast<u32x2*>(p.x_out + o) = u32x2{lo, hi};
                                    *reinterpret_cast<u32x2*>(xs + o) = u32x2{lo, hi};
                                  });
  } else {
    // stage x [T, d] in LDS
    const int nvec = p.T * p.d / 8;
    for (int v = threadIdx.x; v < nvec; v += kRouteThreads)
      reinterpret_cast<u32x4*>(xs)[v] = reinterpret_cast<const u32x4*>(p.x)[v];
  }
  __syncthreads();
  for (int e = e0; e < p.E; e += kW) {
    if (e != e0) {
#pragma unroll
      for (int j = 0; j < kFastChunks; ++j) {
        const int c = j * 512 + lane * 8;
        b[j] = (j < nch && c < p.d) ? *reinterpret_cast<const u32x4*>(p.wg + (int64_t)e * p.d + c)
                                    : u32x4{0, 0, 0, 0};
      }
    }
    for (int t = 0; t < p.T; ++t) {
      float acc = 0.0f;
#pragma unroll
      for (int j = 0; j < kFastChunks; ++j) {
        const int c = j * 512 + lane * 8;
        if (j < nch && c < p.d) {
          const u32x4 xv = *reinterpret_cast<const u32x4*>(xs + (int64_t)t * p.d + c);
          acc = dot2(xv.x, b[j].x, acc);
          acc = dot2(xv.y, b[j].y, acc);
          acc = dot2(xv.z, b[j].z, acc);
          acc = dot2(xv.w, b[j].w, acc);
        }
      }
      const float v = wave_sum_dpp(acc);
      if (lane == 0) lg[t * p.E + e] = v;
    }
  }
}

// top-k, softmax over the selected logits and the Eq. 2 rule for token t by
// one wave: lanes are experts; slot k is the lowest lane with the wave maximum
// of the logits' keys over the experts not yet taken, so exact ties keep the
// lower index.  lrow:
// the token's E logits in LDS; s_idx / s_prec: the pairs in LDS, or null.
// A NaN logit: a decode step's router (FIRST = false) takes it as larger than
// any number (smaller with the sign bit), a prefill's as one that is only
// selected if no expert of a lower index is left.
template <bool FIRST>
__device__ void decide_wave(const RouteParams& p, int t, const float* lrow, const int* tags,
                            RouteOut o, int32_t* s_idx, int8_t* s_prec) {
  const int lane = threadIdx.x & 63;
  float v = lane < p.E ? lrow[lane] : -__builtin_inff();
  int sel[kMaxTopK];
  float ls[kMaxTopK];
  uint64_t taken = 0;
#pragma unroll
  for (int k = 0; k < kMaxTopK; ++k) {
    if (k >= p.K) break;
    uint32_t key = float_key(v);
    if (FIRST) {
      const int first = __ffsll((unsigned long long)~taken) - 1;
      if (v != v) key = lane == first ? 0xFFFFFFFFu : 1u;
      if (taken >> lane & 1) key = 0;
    }
    if (lane >= p.E) key = 0;  // (ties go to lower lanes, and E >= K)
    const uint32_t top = wave_max_u32(key);
    const int e = __ffsll((unsigned long long)__ballot(key == top)) - 1;
    sel[k] = e;
    ls[k] = __builtin_bit_cast(
        float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), __builtin_amdgcn_readfirstlane(e)));
    if (FIRST) taken |= 1ull << e;
    else if (lane == e) v = -__builtin_inff();
  }
  float ex[kMaxTopK];
  float z = 0.0f;
#pragma unroll
  for (int k = 0; k < kMaxTopK; ++k) {
    if (k < p.K) {
      ex[k] = expf(ls[k] - ls[0]);
      z += ex[k];
    }
  }
  float above = 0.0f;  // Eq. 2 running score
#pragma unroll
  for (int k = 0; k < kMaxTopK; ++k) {
    if (k >= p.K) break;
    const float w = ex[k] / z;
    const int e = sel[k];
    const int tag = tags[e];
    int prec;
    if (tag == TAG_FP16 || tag == TAG_INT8) {
      prec = PREC_HIGH;
    } else if (tag == TAG_INT4 || tag == TAG_INT2) {
      prec = PREC_LOW;
    } else {
      const float sc = (k == 0) ? 0.0f : above;
      prec = (k == 0 || sc <= p.t1) ? PREC_HIGH : (sc <= p.t2 ? PREC_LOW : PREC_SKIP);
    }
    above += w;
    if (lane == k) {
      const int pi = t * p.K + k;
      o.idx[pi] = e;
      o.w[pi] = w;
      o.prec[pi] = (int8_t)prec;
      if (s_idx) {
        s_idx[pi] = e;
        s_prec[pi] = (int8_t)prec;
      }
      if (o.user_idx) o.user_idx[pi] = e;
      if (o.user_w) o.user_w[pi] = w;
      if (o.user_prec) o.user_prec[pi] = (int8_t)prec;
    }
  }
}

// Work list of at most 64 pairs by one wave: a stable counting sort over the
// keys (expert, precision), keys in increasing order, one ballot each; a
// pair's rank is the number of lower lanes with the same key, so pair order
// inside a group is the pair index order.  Skipped pairs get no key.
__device__ void worklist_wave(const RouteParams& p, const int32_t* idx, const int8_t* prec,
                              const int* widths, WorkList* wl, int32_t* perm, int32_t* pos) {
  const int lane = threadIdx.x & 63;
  const int N = p.T * p.K;
  int key = -1;
  if (lane < N) {
    const int pr = prec[lane];
    if (pr != PREC_SKIP) key = idx[lane] * 2 + (pr == PREC_LOW);
    else pos[lane] = -1;
  }
  const uint64_t lower = (1ull << lane) - 1ull;
  int off = 0, ng = 0;
  for (int k = 0; k < 2 * p.E; ++k) {
    const uint64_t m = __ballot(key == k);
    if (m == 0) continue;
    const int c = __popcll(m);
    if (key == k) {
      const int at = off + __popcll(m & lower);
      perm[at] = lane;
      pos[lane] = at;
    }
    if (lane == 0) {
      Group g;
      g.expert = k >> 1;
      g.bits = copy_bits(widths[k >> 1], k & 1);
      g.offset = off;
      g.count = c;
      wl->groups[ng] = g;
    }
    ++ng;
    off += c;
  }
  if (lane == 0) wl->n_groups = ng;
}

// Steps of up to kRouteSmallTokens tokens: one block routes every token and
// builds the work list.
__global__ __launch_bounds__(kRouteThreads) void route_decode_kernel(
    RouteParams p, RouteOut o, WorkList* wl, int32_t* perm, int32_t* pos) {
  __shared__ float lg[kRouteSmallTokens * kMaxExperts];
  __shared__ int tags[kMaxExperts], widths[kMaxExperts];
  __shared__ int32_t s_idx[kRouteSmallTokens * kMaxTopK];
  __shared__ int8_t s_prec[kRouteSmallTokens * kMaxTopK];
  __shared__ __attribute__((aligned(16))) f16 xs[kFastXBytes / 2];
  TableRow tr;
  tr.load(p);
  const bool fast = fast_gate(p.T, p.d);
  if (fast) gate_fast(p, xs, lg);
  else if (p.T == 1) gate_logits<1, 8>(p, 0, p.T, lg);
  else if (p.T == 2) gate_logits<2, 8>(p, 0, p.T, lg);
  else gate_logits<4, 4>(p, 0, p.T, lg);
  tr.store(p, tags, widths);
  __syncthreads();
  for (int t = threadIdx.x >> 6; t < p.T; t += kRouteWaves)
    decide_wave<false>(p, t, lg + t * p.E, tags, o, s_idx, s_prec);
  __syncthreads();
  static_assert(kRouteSmallTokens * kMaxTopK <= 64, "one pair per lane");
  if (threadIdx.x < 64) worklist_wave(p, s_idx, s_prec, widths, wl, perm, pos);
}

// More tokens: blocks of TPB tokens each; a second kernel builds the list.
// What bounds it is latency up to some hundred tokens (the single block took
// 20 us at 16 tokens and 57 at 64, both kernels together take 12), then the
// L2 reads of the gate, once per block: 8192 tokens, 16 experts 169 -> 97 us
// for both kernels against one token per block.
// With E <= 16 and d <= 4096 a wave keeps its expert's gate row in registers
// for all of its tokens (the waves beyond the experts take other tokens);
// the token rows are read by every expert's wave and hit L1.  One token per
// block while that leaves compute units free: the call is then two memory
// round trips and a launch.  Logits are summed over the chunks in the same
// order as in the other routers.
template <bool FIRST, int TPB>
__global__ __launch_bounds__(kRouteThreads) void route_tokens_kernel(RouteParams p, RouteOut o) {
  __shared__ float lg[TPB * kMaxExperts];
  __shared__ int tags[kMaxExperts], widths[kMaxExperts];
  const int t0 = blockIdx.x * TPB;
  const int nt = min(TPB, p.T - t0);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  TableRow tr;
  tr.load(p);
  if (p.E <= kRouteWaves && p.d <= kRowChunks * 512) {
    const int per = kRouteWaves / p.E, e = wave % p.E, g = wave / p.E;
    if (g < per) {
      u32x4 b[kRowChunks];
#pragma unroll
      for (int j = 0; j < kRowChunks; ++j) {
        const int c = j * 512 + lane * 8;
        b[j] = c < p.d ? *reinterpret_cast<const u32x4*>(p.wg + (int64_t)e * p.d + c)
                       : u32x4{0, 0, 0, 0};
      }
      for (int t = g; t < nt; t += per) {
        u32x4 a[kRowChunks];
#pragma unroll
        for (int j = 0; j < kRowChunks; ++j) {
          const int c = j * 512 + lane * 8;
          a[j] = c < p.d ? *reinterpret_cast<const u32x4*>(p.x + (int64_t)(t0 + t) * p.d + c)
                         : u32x4{0, 0, 0, 0};
        }
        float acc = 0.0f;
#pragma unroll
        for (int j = 0; j < kRowChunks; ++j) {
          acc = dot2(a[j].x, b[j].x, acc);
          acc = dot2(a[j].y, b[j].y, acc);
          acc = dot2(a[j].z, b[j].z, acc);
          acc = dot2(a[j].w, b[j].w, acc);
        }
        const float v = wave_sum_dpp(acc);
        if (lane == 0) lg[t * p.E + e] = v;
      }
    }
  } else {
    gate_logits<1, 8>(p, t0, t0 + nt, lg);
  }
  tr.store(p, tags, widths);
  __syncthreads();
  for (int t = wave; t < nt; t += kRouteWaves)
    decide_wave<FIRST>(p, t0 + t, lg + t * p.E, tags, o, nullptr, nullptr);
}

// Lanes of this wave with the same key as this lane (key >= 0, below 2^BITS).
template <int BITS>
__device__ inline uint64_t same_key(int key) {
  uint64_t m = __ballot(key >= 0);
#pragma unroll
  for (int b = 0; b < BITS; ++b) {
    const uint64_t on = __ballot(key >> b & 1);
    m &= (key >> b & 1) ? on : ~on;
  }
  return m;
}

// Work list of any number of pairs: a stable counting sort by key = expert *
// 2 + (low ? 1 : 0) in one block.  Wave w owns the pairs [w S, (w + 1) S);
// it counts their keys (a pair's rank among equal keys of 64 pairs is the
// number of lower lanes with that key, found with one ballot per key bit),
// the counts are scanned over keys and waves, and the wave walks its pairs
// again to place them.  Three block barriers whatever the number of pairs;
// with a barrier between every 1024 pairs instead, 8192 tokens took 39 us.
__global__ __launch_bounds__(kRouteThreads) void worklist_kernel(
    RouteParams p, RouteOut o, WorkList* wl, int32_t* perm, int32_t* pos) {
  constexpr int kKeyBits = 7;
  static_assert(kMaxKeys == 1 << kKeyBits && kMaxKeys == 2 * 64, "two keys per lane of one wave");
  __shared__ int widths[kMaxExperts], tags[kMaxExperts];
  __shared__ int at[kRouteWaves][kMaxKeys];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int N = p.T * p.K;
  const int S = ((N + kRouteThreads - 1) / kRouteThreads) * 64;
  const int i0 = wave * S, i1 = min(i0 + S, N);
  const uint64_t lower = (1ull << lane) - 1ull;
  TableRow tr;
  tr.load(p);
  for (int v = tid; v < kRouteWaves * kMaxKeys; v += kRouteThreads) at[v / kMaxKeys][v % kMaxKeys] = 0;
  tr.store(p, tags, widths);
  __syncthreads();
  auto key_of = [&](int i) {
    int key = -1;
    if (i < i1) {
      const int pr = o.prec[i];
      if (pr != PREC_SKIP) key = o.idx[i] * 2 + (pr == PREC_LOW);
    }
    return key;
  };
  for (int c = i0; c < i1; c += 64) {
    const int key = key_of(c + lane);
    const uint64_t m = same_key<kKeyBits>(key);
    if (key >= 0 && (m & lower) == 0) atomicAdd(&at[wave][key], __popcll(m));
  }
  __syncthreads();
  if (wave == 0) {
    // lane l: keys 2 l and 2 l + 1
    int cnt[2], run = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      cnt[h] = 0;
#pragma unroll
      for (int w = 0; w < kRouteWaves; ++w) cnt[h] += at[w][2 * lane + h];
    }
    const int mine = cnt[0] + cnt[1], mine_g = (cnt[0] > 0) + (cnt[1] > 0);
    int off = mine, ng = mine_g;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
      const int a = __shfl_up(off, s, 64), b = __shfl_up(ng, s, 64);
      if (lane >= s) {
        off += a;
        ng += b;
      }
    }
    if (lane == 63) wl->n_groups = ng;
    off -= mine;
    ng -= mine_g;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      run = off;
      if (cnt[h] > 0) {
        Group g;
        g.expert = lane;
        g.bits = copy_bits(widths[lane], h);
        g.offset = off;
        g.count = cnt[h];
        wl->groups[ng++] = g;
      }
      off += cnt[h];
      // first place of every wave's pairs of this key
#pragma unroll
      for (int w = 0; w < kRouteWaves; ++w) {
        const int n = at[w][2 * lane + h];
        at[w][2 * lane + h] = run;
        run += n;
      }
    }
  }
  __syncthreads();
  for (int c = i0; c < i1; c += 64) {
    const int i = c + lane;
    const int key = key_of(i);
    const uint64_t m = same_key<kKeyBits>(key);
    int first = 0;
    if (key >= 0 && (m & lower) == 0) first = atomicAdd(&at[wave][key], __popcll(m));
    first = __shfl(first, m ? __ffsll((unsigned long long)m) - 1 : 0, 64);
    if (key >= 0) {
      const int to = first + __popcll(m & lower);
      perm[to] = i;
      pos[i] = to;
    } else if (i < i1) {
      pos[i] = -1;
    }
  }
}

template <bool FIRST, int TPB>
hipError_t launch_route_tokens(const RouteParams& p, RouteOut o, WorkList* wl, int32_t* perm,
                               int32_t* pos, hipStream_t s) {
  route_tokens_kernel<FIRST, TPB><<<(p.T + TPB - 1) / TPB, kRouteThreads, 0, s>>>(p, o);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  worklist_kernel<<<1, kRouteThreads, 0, s>>>(p, o, wl, perm, pos);
  return hipGetLastError();
}

}  // namespace

bool route_decode_fuses_norm(int T, int d) { return T <= kRouteSmallTokens && fast_gate(T, d); }

hipError_t launch_route_decode(const RouteParams& p, RouteOut o, WorkList* wl,
                               int32_t* perm, int32_t* pos, hipStream_t s) {
  // the fused RMSNorm exists on the LDS-staged gate path only
  if (p.h_res && !route_decode_fuses_norm(p.T, p.d)) return hipErrorInvalidValue;
  if (p.T > kRouteSmallTokens) return launch_route_tokens<false, 1>(p, o, wl, perm, pos, s);
  route_decode_kernel<<<1, kRouteThreads, 0, s>>>(p, o, wl, perm, pos);
  return hipGetLastError();
}

hipError_t launch_route_prefill(const RouteParams& p, RouteOut o, WorkList* wl,
                                int32_t* perm, int32_t* pos, hipStream_t s) {
  // One token per block up to two blocks per compute unit; 4 up to 2048
  // tokens, where blocks of 16 leave half of the units or more without one
  // (whole call at d 4096, f 64, blocks of 16 / 4: 16 experts, 513 tokens 68.3
  // / 56.9 us, 1337 tokens 92.4 / 86.2, 2000 tokens 109.7 / 103.8; 24 experts,
  // 1337 tokens 122.3 / 99.0); then 16, as blocks of 8 were slower at 2500 to
  // 4096 tokens (16 experts 153.4 us, 155.7 by 8).
  if (p.T <= 512) return launch_route_tokens<true, 1>(p, o, wl, perm, pos, s);
  if (p.T <= 2048) return launch_route_tokens<true, 4>(p, o, wl, perm, pos, s);
  return launch_route_tokens<true, 16>(p, o, wl, perm, pos, s);
}

}  // namespace moe

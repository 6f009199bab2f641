// Device functions shared by the score, select and fused score+select kernels: the arithmetic of a score and the
// selection of a row's kept positions exist once, so the fused kernel reproduces the two-call path bit for bit.
#pragma once
#include "common.hpp"

namespace samkv {

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// Sum over aligned groups of W lanes (W in {8, 16, 32}); every lane of a group ends with the total.
// After the quad steps the mirrors pair lanes that already hold equal partial sums.
template <int W>
__device__ __forceinline__ float group_sum(float v) {
  v += dpp_move<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_move<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_move<0x141>(v);  // row_half_mirror: lane i <-> 7 - i
  if (W >= 16) v += dpp_move<0x140>(v);  // row_mirror: lane i <-> 15 - i
  if (W >= 32) v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));  // lane ^ 16
  return v;
}

template <bool BF16>
__device__ __forceinline__ void unpack16(const u32x4& x, float* f) {
  if (BF16) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f[2 * e] = bf16_lo(x[e]);
      f[2 * e + 1] = bf16_hi(x[e]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(x[e]);
  }
}

// The largest bf16 magnitude (bit pattern) of the halves of x so far, in both halves of `mx`.
__device__ __forceinline__ uint32_t bf16_max(uint32_t mx, const u32x4& x) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  u16x2 m = __builtin_bit_cast(u16x2, mx);
#pragma unroll
  for (int e = 0; e < 4; ++e) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, x[e] & 0x7FFF7FFFu));
  return __builtin_bit_cast(uint32_t, m);
}
// The wave's largest into *at, a word of its own (atomics of all waves on one word per head took longer than a pass over V: 5600
// of them 45 us).
__device__ __forceinline__ void write_max(uint32_t* at, uint32_t mx) {
  mx = max(mx & 0xFFFFu, mx >> 16);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
  if ((threadIdx.x & 63) == 0) *at = mx;
}

// The vector a KV head scores its document's keys with: the mean of `group` consecutive head vectors of D floats
// (1 when the fold over the KV group has already been done, G when src holds Eq. 1 per query head).  The lane
// takes its EPL channels.
template <int EPL>
__device__ __forceinline__ void fold_query(const float* src, int d, int group, float* q) {
#pragma unroll
  for (int e = 0; e < EPL; ++e) q[e] = 0.f;
  for (int hh = 0; hh < group; ++hh)
#pragma unroll
    for (int e = 0; e < EPL; ++e) q[e] += src[hh * d + e];
#pragma unroll
  for (int e = 0; e < EPL; ++e) q[e] /= (float)group;
}

// One wave scores RPL * NB * 2 consecutive key rows starting at row0 (rows >= L are skipped): 16 x 16 bytes per
// lane are loaded up front, LPR lanes share one key row, their partial dot products are combined with DPP moves,
// and lane (row group rg, sub < NB) emits row sub * RPL + rg of a batch.  `base` already points at the lane's
// 16-byte column of row 0.
template <bool BF16, int D, class Emit>
__device__ __forceinline__ void score_rows(const char* base, int row0, int L, const float* q, Emit emit) {
  constexpr int EPL = BF16 ? 8 : 4;
  constexpr int LPR = D / EPL;
  constexpr int RPL = 64 / LPR;
  constexpr int NB = 8;
  constexpr size_t ROW_BYTES = (size_t)D * (BF16 ? 2 : 4);
  static_assert(LPR >= NB, "store mapping needs at least NB lanes per row");
  const int lane = threadIdx.x & 63, sub = lane % LPR, rg = lane / LPR;
  u32x4 x[2][NB];
#pragma unroll
  for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      int row = row0 + (b2 * NB + b) * RPL + rg;
      row = row < L ? row : L - 1;
      x[b2][b] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + (size_t)row * ROW_BYTES));
    }
#pragma unroll
  for (int b2 = 0; b2 < 2; ++b2) {
    float keep = 0.f;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float f[EPL];
      unpack16<BF16>(x[b2][b], f);
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < EPL; ++e) s = fmaf(f[e], q[e], s);
      s = group_sum<LPR>(s);
      keep = (sub % NB == b) ? s : keep;
    }
    const int row = row0 + (b2 * NB + (sub % NB)) * RPL + rg;
    if (sub < NB && row < L) emit(row, keep);
  }
}

__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u << 1) == 0u) u = 0u;  // -0 and +0 are one value: ties go by position, not by sign bit
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Which position of its row a thread's e-th key is: a wave owns 64 * E consecutive positions and takes them 64 at a time,
// so that a wave-wide access touches consecutive words (global memory or LDS) and the order of positions is the order of
// (e, lane).
template <int E>
__device__ __forceinline__ int key_position(int e) {
  return (int)(threadIdx.x >> 6) * (64 * E) + e * 64 + (int)(threadIdx.x & 63);
}

// Forced positions (the first n_sink and last n_local of the row) get the largest key.
template <int E>
__device__ __forceinline__ void force_keys(uint32_t (&key)[E], int L, int n_sink, int n_local) {
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = key_position<E>(e);
    if (p < L && (p < n_sink || p >= L - n_local)) key[e] = 0xFFFFFFFFu;
  }
}

// The k-th largest key of a row, as far as the selection needs it: keys > T are kept and, of those == T, the first `need`.
struct Threshold {
  uint32_t T, need;
};

// One bit per pass from the top: ballot + popcount per key, the waves' counts meet in LDS (double-buffered, one barrier
// per pass).  `bucket` = positions < L whose keys agree with the bits decided so far; kk of them are still to be kept.
// Once bucket == kk every one of them is kept whatever the remaining bits say, so the walk stops there (distinct keys:
// after about log2(L) bits below the ones all keys share; rows of equal keys walk all 32).
template <int E, int NT>
__device__ __forceinline__ Threshold threshold_by_bits(const uint32_t (&key)[E], int L, int k, uint32_t (*cnt)[NT / 64]) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t prefix = 0, kk = (uint32_t)k, bucket = (uint32_t)L;
  for (int b = 31; b >= 0 && bucket != kk; --b) {
    // candidate: agrees with the decided bits above b and has bit b set (padding keys are 0: never)
    const uint32_t want = (prefix >> b) | 1u;
    uint32_t c = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) c += __popcll(__ballot((key[e] >> b) == want));
    if (lane == 0) cnt[b & 1][wave] = c;
    __syncthreads();
    uint32_t tot = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) tot += cnt[b & 1][w];
    if (tot >= kk) {
      prefix |= (1u << b);
      bucket = tot;
    } else {
      kk -= tot;
      bucket -= tot;
    }
  }
  // stopped early: every key >= prefix (zeros below the decided bits) is kept; walked to the end: the first kk equal ones
  return {prefix, bucket == kk ? 0xFFFFFFFFu : kk};
}

// The same threshold by 11 + 11 + 10 bits: a histogram in LDS per pass, in which only the keys of the bucket take part.
// A pass costs one LDS atomic per key of the bucket and four barriers instead of 11 passes over all keys.  Scores crowd
// into few values of the top bits, so the histogram exists four times (a lane uses copy lane % 4, 16 banks apart).
constexpr int kHistBits = 11, kHistBins = 1 << kHistBits, kHistCopies = 4, kHistStride = kHistBins + 16;
template <int NT>
struct HistScratch {
  uint32_t hist[kHistCopies * kHistStride];
  uint32_t wave_sum[NT / 64];
  uint32_t pick[3];  // chosen bin, keys of it still to be kept, keys in it
};
template <int E, int NT>
__device__ __forceinline__ Threshold threshold_by_histogram(const uint32_t (&key)[E], int L, int k, HistScratch<NT>& sc) {
  constexpr int NW = NT / 64, BPT = kHistBins / NT;
  static_assert(kHistBins % NT == 0, "bins per thread");
  if (k == 0) return {0xFFFFFFFFu, 0u};  // a document that keeps nothing
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  uint32_t prefix = 0, kk = (uint32_t)k, bucket = (uint32_t)L;
  for (int top = 32; top > 0 && bucket != kk;) {
    const int bits = top < kHistBits ? top : kHistBits, sh = top - bits;
    for (int i = t; i < kHistCopies * kHistStride; i += NT) sc.hist[i] = 0;
    __syncthreads();
    uint32_t* own = sc.hist + (lane & (kHistCopies - 1)) * kHistStride;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool in = key_position<E>(e) < L && (top == 32 || (key[e] >> (top & 31)) == prefix >> (top & 31));
      if (in) atomicAdd(own + ((key[e] >> sh) & ((1u << bits) - 1u)), 1u);
    }
    __syncthreads();
    // thread t holds bins (from the highest down) t * BPT ...: exclusive count of the keys above its bins
    uint32_t n[BPT], sum = 0;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      const int bin = kHistBins - 1 - (t * BPT + j);
      n[j] = 0;
#pragma unroll
      for (int c = 0; c < kHistCopies; ++c) n[j] += sc.hist[c * kHistStride + bin];
      sum += n[j];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    if (lane == 63) sc.wave_sum[wave] = incl;
    __syncthreads();
    uint32_t above = incl - sum;
#pragma unroll
    for (int w = 0; w < NW; ++w) above += w < wave ? sc.wave_sum[w] : 0u;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      if (above < kk && kk <= above + n[j]) {  // exactly one bin
        sc.pick[0] = (uint32_t)(kHistBins - 1 - (t * BPT + j));
        sc.pick[1] = kk - above;
        sc.pick[2] = n[j];
      }
      above += n[j];
    }
    __syncthreads();
    prefix |= sc.pick[0] << sh;
    kk = sc.pick[1];
    bucket = sc.pick[2];
    top = sh;
  }
  return {prefix, bucket == kk ? 0xFFFFFFFFu : kk};
}

// n plus the number of lower lanes in `mask`
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask, uint32_t n) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, n));
}

// Emits the kept positions of a row whose order keys sit in registers (keys of positions >= L are 0): emit(place, position),
// places 0 .. k - 1 in ascending order of the positions.  wsum is LDS scratch of the workgroup.
template <int E, int NT, class Emit>
__device__ __forceinline__ void write_kept(const uint32_t (&key)[E], int L, Threshold th, Emit emit, uint2* wsum) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t n_gt = 0, n_eq = 0, T = th.T;  // counts of the wave
  if constexpr (E <= 8) {
    // by ballots, whose masks stay in scalar registers for the second use below
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool ok = key_position<E>(e) < L;
      n_gt += __popcll(__ballot(ok && key[e] > T));
      n_eq += __popcll(__ballot(ok && key[e] == T));
    }
  } else {
    // per lane, both counts in one word (at most 64 each), summed over the wave; the comparisons below are made anew: 2 E
    // masks kept from above would not fit the registers
    uint32_t n = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool ok = key_position<E>(e) < L;
      n += (ok && key[e] > T ? 1u : 0u) + (ok && key[e] == T ? 0x10000u : 0u);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off);
    n_gt = n & 0xFFFFu;
    n_eq = n >> 16;
    asm volatile("" : "+v"(T));
  }
  if (lane == 0) wsum[wave] = make_uint2(n_gt, n_eq);
  __syncthreads();
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    gt += w < wave ? wsum[w].x : 0u;
    eq += w < wave ? wsum[w].y : 0u;
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = key_position<E>(e);
    const bool is_gt = p < L && key[e] > T, is_eq = p < L && key[e] == T;
    const uint64_t m_gt = __ballot(is_gt), m_eq = __ballot(is_eq);
    const uint32_t g = lanes_below(m_gt, gt), q = lanes_below(m_eq, eq);
    if (is_gt || (is_eq && q < th.need)) emit((int)(g + (q < th.need ? q : th.need)), p);
    gt += __popcll(m_gt);
    eq += __popcll(m_eq);
  }
}

// Rows of up to 64 E keys by ONE wave that holds all of them, its e-th the position 64 e + lane: no barrier, no LDS.  Key `cand`
// is kept if k keys reach it; a bit of the threshold takes a comparison and a popcount per key of the lane.
template <int E>
__device__ __forceinline__ Threshold threshold_in_wave(const uint32_t (&key)[E], int L, int k) {
  if (k == 0) return {0xFFFFFFFFu, 0u};
  uint32_t T = 0, n = (uint32_t)L;  // keys that reach T (padding keys are 0 and reach no candidate)
#pragma unroll 1
  for (uint32_t bit = 0x80000000u; bit != 0 && n != (uint32_t)k; bit >>= 1) {
    const uint32_t cand = T | bit;
    uint32_t c = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) c += __popcll(__ballot(key[e] >= cand));
    if (c >= (uint32_t)k) {
      T = cand;
      n = c;
    }
  }
  if (n == (uint32_t)k) return {T, 0xFFFFFFFFu};
  uint32_t above = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) above += __popcll(__ballot(key[e] > T));
  return {T, (uint32_t)k - above};
}

// The kept positions of such a row in ascending order: emit(place, position) for the keys e with own(e).
template <int E, class Own, class Emit>
__device__ __forceinline__ void emit_kept(const uint32_t (&key)[E], int L, Threshold th, Own own, Emit emit) {
  const int lane = threadIdx.x & 63;
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = e * 64 + lane;
    const bool is_gt = p < L && key[e] > th.T, is_eq = p < L && key[e] == th.T;
    const uint64_t m_gt = __ballot(is_gt), m_eq = __ballot(is_eq);
    if (own(e)) {
      const uint32_t g = lanes_below(m_gt, gt), q = lanes_below(m_eq, eq);
      if (is_gt || (is_eq && q < th.need)) emit((int)(g + (q < th.need ? q : th.need)), p);
    }
    gt += __popcll(m_gt);
    eq += __popcll(m_eq);
  }
}

}  // namespace samkv

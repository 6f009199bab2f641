// Pieces shared by the attention kernels (attn.hip: bf16, attn_f32.hip: float32): kernel arguments, the mapping from
// workgroups to (KV head, batch, row tile), the exchange between half-waves and the store of a wave's output rows.
#pragma once
#include <math.h>

#include "common.hpp"

namespace samkv {

struct AttnArgs {
  const void* q;
  const void* k;
  const void* v;           // V, or its half-precision copy for the bf16 kernels that read one (every one but SPLIT)
  const float* v_unscale;  // per KV head: undoes the copy's scale
  float* out;
  float* lse;
  float* part_o;
  float* part_lse;
  int rows, m, batch_per_kv, n_batch, n_split, chunk;
  int n_self;          // > 0: the last part is the query tokens' own n_self keys, k_self and v_self (k_attn_bf16)
  const void* k_self;
  const void* v_self;
  int kv_groups;  // > 0: KV heads are walked in groups of 8 (one per XCD), see map_block
  float scale;
};

// Exchange between lane l and lane l ^ 32 on the vector ALU (v_permlane32_swap; with both operands equal the first
// result holds the lower half's values in both halves and the second the upper half's): no trip through LDS as a
// 64-wide shuffle would take, which matters because the row maximum sits at the head of every step's dependence chain.
__device__ __forceinline__ float max_across_halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_across_halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Writes a wave's 32 x D block of normalised output rows.  In the accumulator layout a lane holds 4-float pieces of
// ONE row (row = lane % 32), so a direct store instruction scatters 32-byte pieces over 32 rows; issuing the 4 D / 32
// of them takes a few microseconds, which a short workgroup feels.  The block is therefore turned through LDS (the
// wave's own `lds` area; rows of D * 4 + 16 bytes, the pad keeps the 16 lanes of a write phase on distinct banks)
// and leaves as whole rows, 1 KB per instruction.  PARTS = 1 turns the 32 rows at once (area of 32 rows), PARTS = 2
// in two passes of 16 rows (area of 16 rows).  Only this wave touches the area, and a wave's LDS operations execute
// in order, so no workgroup barrier is needed.  dst points at the wave's first row; rows >= n_valid are not written.
template <int D, int PARTS = 1>
__device__ __forceinline__ void store_rows_via_lds(const f32x16 (&o)[D / 32], float inv, float* dst, int n_valid, char* lds,
                                                   int lane) {
  constexpr int RS = D * 4 + 16, LPR = D / 4, RPI = 64 / LPR, ROWS = 32 / PARTS;
  const int rw = lane & 31, h = lane >> 5;
#pragma unroll
  for (int part = 0; part < PARTS; ++part) {
    if (PARTS == 1 || rw / ROWS == part) {
#pragma unroll
      for (int dvb = 0; dvb < D / 32; ++dvb)
#pragma unroll
        for (int j4 = 0; j4 < 4; ++j4) {
          f32x4 x;
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = o[dvb][4 * j4 + e] * inv;
          *reinterpret_cast<f32x4*>(lds + (rw % ROWS) * RS + (dvb * 32 + 8 * j4 + 4 * h) * 4) = x;
        }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < ROWS / RPI; ++i) {
      const int lrow = i * RPI + lane / LPR, row = part * ROWS + lrow;
      const f32x4 x = *reinterpret_cast<const f32x4*>(lds + lrow * RS + (lane % LPR) * 16);
      if (row < n_valid) *reinterpret_cast<f32x4*>(dst + (size_t)row * D + (lane % LPR) * 4) = x;
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// (blockIdx.x, blockIdx.y) -> (KV head, batch, row tile).  Workgroups are handed out x-fastest and round-robin over
// the 8 XCDs, each with its own L2.  The batches (query heads x row blocks) that read one KV head's K/V stream
// should run on one XCD and close in time, and an XCD should not hold more streams at once than its L2 can serve.
// So KV heads are taken in groups of 8, one head per XCD: x = 8 * member + XCD slot runs over the batches of the
// group's heads, y = group * tiles + tile, and a group's row tiles (longest first when causal) are all handed out
// before the next group starts.  With 8 KV heads there is one group and this is "KV head = x % 8, all row tiles in
// longest-first order"; with many KV heads (several layers stacked as heads) an XCD still streams one head at a
// time instead of dozens.  kv_groups == 0 (head count not a multiple of 8): plain x = batch, y = tile.
// A workgroup's coordinates in the (batch, row tile, key chunk) grid of its problem: a plain launch takes them from
// the hardware, the pair launch below hands out two problems' grids from one linear index
// (x, y, z of grid_y rows): plain ints, so that nothing of it ever lives in memory.
__device__ __forceinline__ void map_block(const AttnArgs& a, bool causal, int x, int y, int grid_y, int* kvh, int* batch,
                                          int* tile) {
  int ty;
  if (a.kv_groups > 0) {
    const int tiles = grid_y / a.kv_groups;
    const int grp = y / tiles;
    ty = y - grp * tiles;
    *kvh = grp * 8 + (x & 7);
    *batch = *kvh * a.batch_per_kv + (x >> 3);
    *tile = causal ? tiles - 1 - ty : ty;
  } else {
    const int n_kv = a.n_batch / a.batch_per_kv;
    *kvh = x % n_kv;
    *batch = *kvh * a.batch_per_kv + x / n_kv;
    *tile = causal ? grid_y - 1 - y : y;
  }
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Grids of a pair launch (both attentions of the path in one launch), as linear workgroup indices.
struct PairGrid {
  int n_q, n_q_pad, q_gx, q_gy, c_gx, c_gy;
};

inline AttnArgs make_args(const AttnLaunch& l) {
  AttnArgs a;
  a.q = l.q; a.k = l.k; a.v = l.v; a.v_unscale = l.v_unscale; a.out = l.out; a.lse = l.lse;
  a.part_o = l.part_o; a.part_lse = l.part_lse;
  a.rows = l.rows; a.m = l.m; a.batch_per_kv = l.batch_per_kv; a.n_batch = l.n_batch;
  a.n_split = l.causal ? 1 : l.n_split;
  a.chunk = l.chunk; a.scale = l.scale;
  a.n_self = l.n_self; a.k_self = l.k_self; a.v_self = l.v_self;
  a.kv_groups = 0;
  return a;
}

// Grid of an attention launch over `tiles` row tiles, and the matching kv_groups of the arguments.
inline dim3 attn_grid(AttnArgs* a, int tiles) {
  const int n_kv = a->n_batch / a->batch_per_kv;
  if (n_kv % 8 == 0 && (long long)tiles * (n_kv / 8) <= 65535) {
    a->kv_groups = n_kv / 8;
    return dim3(8 * a->batch_per_kv, tiles * a->kv_groups, a->n_split);
  }
  a->kv_groups = 0;
  return dim3(a->n_batch, tiles, a->n_split);
}

}  // namespace samkv

// Attention over the compacted multi-document cache (Sec. 3.3):
//   causal     - recomputation of the kept tokens: row p sees compacted positions 0..p
//   not causal - the user query's final incremental prefill over the whole compacted cache
// Both are softmax(scale * q k^T) v with float32 statistics; they differ in the mask and in how the
// rows are cut into workgroups.
//
// Two bf16 kernels share the arithmetic and operand layouts.  A wave holds 32 query rows and takes 64 keys per step:
//   S^T = K Q^T   v_mfma_f32_32x32x16_bf16, A = K rows from LDS, B = the wave's 32 query rows (registers,
//                 loaded once).  Computing the transpose puts one query row in one lane column, so the
//                 softmax weights come out of the accumulator already in the B-operand layout of the
//                 next product and never travel through LDS.
//   O^T += V^T P^T  A = V^T read from the row-major V tile in LDS with the transposing LDS read
//                 (ds_read_b64_tr_b16), B = P^T from registers.  bf16 weights would cost 2^-9 of the spread of V per
//                 output; the kernels get more out of 16-bit operands in different ways:
// Half-precision products (k_attn_bf16_dma, k_attn_bf16 for causal problems and both problems in one launch): the weights
//   keep an 11-bit significand, and V arrives as the scaled half-precision copy of vprep.hip, whose power-of-two scale the
//   final normalisation undoes.
// Two-term products (k_attn_bf16 for problems that are not causal): V as stored and every weight as the sum of TWO bf16
//   terms (p = hi + lo, 16 significant bits), which doubles the second product's instructions and needs no copy.  That pays
//   where the products are not what the kernel waits for and the launches that prepare V would cost more: the query
//   attention of short and mid-size caches (bound by latency or by HBM; 34 -> 26 us at M = 1540, 54 -> 45 us at
//   M = 6160 as calls).
// Float32 caches: attn_f32.hip.
// Keys can be cut into chunks (not causal only); k_attn_merge combines the per-chunk results with
// their log-sum-exp.
#include <math.h>

#include <mutex>

#include "attn_common.hpp"

namespace samkv {
namespace {

// ------------------------------------------------------------------ bf16, short problems
// One workgroup = four waves of 32 query rows each; one (row tile, part) per workgroup, a part being all keys of a causal
// problem, a chunk of the cache's keys or, behind them, the query tokens' own keys with their causal mask.  K/V tiles are
// double-buffered in LDS; the next tile's global loads are issued before the current tile's math and land in LDS after it,
// one barrier per tile.  SPLIT: two-term products.
template <int D>
struct Bf16Cfg {
  static constexpr int NW = 4, NT = 64 * NW;
  static constexpr int BQ = 32 * NW, BK = 64;
  static constexpr int KSTR = D * 2 + 16;  // bytes per K row in LDS (pad: 16 rows hit 64 distinct banks)
  static constexpr int VSTR = D * 2 + 64;  // bytes per V row in LDS: the 4 rows x 32 B of a transposing read fall in disjoint bank ranges
  static constexpr int TILE_BYTES = BK * (KSTR + VSTR);
  static constexpr int LDS_BYTES = 2 * TILE_BYTES;
  static constexpr int CHUNKS = (BK * D * 2 / 16) / NT;  // 16-byte chunks per thread per tile and tensor
};

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int D, bool CAUSAL, bool SPLIT>
__device__ __forceinline__ void attn_bf16_body(const AttnArgs a, int bx, int by, int bz, int grid_y) {
  using C = Bf16Cfg<D>;
  static_assert(!(CAUSAL && SPLIT), "causal problems read the half-precision copy of V");
  constexpr int ND = D / 16;   // k-steps of the S^T product
  constexpr int NV = D / 32;   // 32-row blocks of O^T
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int rw = lane & 31, h = lane >> 5;
  // grid = (batch, row tile, key chunk)
  int kvh, batch, qt;
  map_block(a, CAUSAL, bx, by, grid_y, &kvh, &batch, &qt);
  const int q0 = qt * C::BQ;
  const int split = bz;
  const bool own = SPLIT && a.n_self > 0 && split == a.n_split - 1;  // the query tokens' own keys, causally
  const int m = own ? a.n_self : a.m;
  // own keys: row r belongs to token r % n_self of its head and sees the keys up to it, so nothing past the largest token of
  // the row tile is walked, and of that a wave skips what lies past its own
  auto last_token = [&](int first, int n) {  // of the rows first .. first + n - 1
    const int t0 = first % a.n_self;
    return min(t0 + n, a.n_self) - 1;  // rows that go on into the next head include that head's largest token
  };
  const int kv_begin = CAUSAL || own ? 0 : split * a.chunk;
  const int kv_end = CAUSAL ? min(m, q0 + C::BQ)
                     : own  ? last_token(q0, min(C::BQ, a.rows - q0)) + 1
                            : min(m, kv_begin + a.chunk);
  const int n_tiles = (kv_end - kv_begin + C::BK - 1) / C::BK;

  const int r = q0 + wave * 32 + rw;
  const int r_c = min(r, a.rows - 1);
  const int wave_first = q0 + wave * 32;
  const int wave_end = CAUSAL ? wave_first + 32 : own ? last_token(wave_first, 32) + 1 : kv_end;  // no row of the wave sees more

  bf16x8 bq[ND];
  {
    const char* qp = static_cast<const char*>(a.q) + ((size_t)batch * a.rows + r_c) * D * 2 + h * 16;
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) bq[dc] = *reinterpret_cast<const bf16x8*>(qp + dc * 32);
  }
  const char* kbase = static_cast<const char*>(own ? a.k_self : a.k) + (size_t)kvh * m * D * 2;
  const char* vbase = static_cast<const char*>(own ? a.v_self : a.v) + (size_t)kvh * m * D * 2;

  // Tile loads: thread t fetches chunk (row t/CPR + i*RSTEP, 16-byte column t%CPR) of K and of V.  The
  // byte offsets inside a tile are per-thread constants; the tile base is uniform, so a full tile
  // costs no address arithmetic.  Only the last, ragged tile clamps its rows to the final key.
  constexpr int CPR = D / 8, RSTEP = C::NT / CPR;
  uint32_t voff[C::CHUNKS];
#pragma unroll
  for (int i = 0; i < C::CHUNKS; ++i) voff[i] = (uint32_t)((t / CPR + i * RSTEP) * (D * 2) + (t % CPR) * 16);
  u32x4 rk[C::CHUNKS], rv[C::CHUNKS];
  auto load_tile = [&](int tile) {
    const int k0 = kv_begin + tile * C::BK;
    const char* kt = kbase + (size_t)k0 * (D * 2);
    const char* vt = vbase + (size_t)k0 * (D * 2);
    if (k0 + C::BK <= m) {
#pragma unroll
      for (int i = 0; i < C::CHUNKS; ++i) {
        rk[i] = *reinterpret_cast<const u32x4*>(kt + voff[i]);
        rv[i] = *reinterpret_cast<const u32x4*>(vt + voff[i]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < C::CHUNKS; ++i) {
        const int row = min(t / CPR + i * RSTEP, m - 1 - k0);
        const uint32_t off = (uint32_t)(row * (D * 2) + (t % CPR) * 16);
        rk[i] = *reinterpret_cast<const u32x4*>(kt + off);
        rv[i] = *reinterpret_cast<const u32x4*>(vt + off);
      }
    }
  };
  auto store_tile = [&](int buf) {
    char* sk = smem + buf * C::TILE_BYTES;
    char* sv = sk + C::BK * C::KSTR;
#pragma unroll
    for (int i = 0; i < C::CHUNKS; ++i) {
      const int c = t + C::NT * i;
      const int row = c / (D / 8), col = c % (D / 8);
      *reinterpret_cast<u32x4*>(sk + row * C::KSTR + col * 16) = rk[i];
      *reinterpret_cast<u32x4*>(sv + row * C::VSTR + col * 16) = rv[i];
    }
  };

  // one past the last key that counts for this lane's row
  const int key_end = CAUSAL ? min(kv_end, r + 1) : own ? r % a.n_self + 1 : kv_end;

  f32x16 o[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[i][j] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c2 = a.scale * kLog2e;

  load_tile(0);
  store_tile(0);
  // Drain every outstanding load (the query fragment included) before the loop: otherwise the loop's
  // first use of the query registers has to be guarded by waits that also cover the next tile's prefetch.
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  for (int tile = 0; tile < n_tiles; ++tile) {
    const int k0 = kv_begin + tile * C::BK;
    const bool more = tile + 1 < n_tiles;
    if (more) load_tile(tile + 1);

    // a wave whose rows all lie past the last row (ragged last row tile) or before the tile's keys only helps with the
    // tile traffic
    const bool active = wave_first < a.rows && k0 < wave_end;
    if (active) {
      const char* sk = smem + (tile & 1) * C::TILE_BYTES;
      const char* sv = smem + (tile & 1) * C::TILE_BYTES + C::BK * C::KSTR;
      f32x16 s[2];
      {
        // all K fragments of the tile are requested before the first product, so the LDS latency is
        // paid once per tile instead of once per instruction
        bf16x8 ak[2][ND];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int dc = 0; dc < ND; ++dc)
            ak[kb][dc] = *reinterpret_cast<const bf16x8*>(sk + (kb * 32 + rw) * C::KSTR + dc * 32 + h * 16);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
          for (int j = 0; j < 16; ++j) s[kb][j] = 0.f;
#pragma unroll
          for (int dc = 0; dc < ND; ++dc)
            s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak[kb][dc], bq[dc], s[kb], 0, 0, 0);
        }
      }
      // accumulator register j of block kb holds key k0 + kb*32 + 8*(j/4) + 4*h + (j%4) for row r
      if (own || (CAUSAL && k0 + C::BK - 1 > wave_first) || k0 + C::BK > kv_end) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int key = k0 + kb * 32 + 8 * (j >> 2) + 4 * h + (j & 3);
            if (key >= key_end) s[kb][j] = -INFINITY;
          }
      }
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int j = 0; j < 16; ++j) mx = fmaxf(mx, s[kb][j]);
      mx = max_across_halves(mx);
      const float m_new = fmaxf(m_run, mx * c2);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
      m_run = m_new;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int j = 0; j < 16; ++j) s[kb][j] = __builtin_amdgcn_exp2f(fmaf(s[kb][j], c2, -m_use));
      // Two-term weights: hi = bf16(p), lo = bf16(p - hi); hi + lo is p to 2^-17, and the row sum is the plain float32 sum
      // of p.  Half-precision weights: the row sum is taken over the rounded weights (pair . (1, 1) accumulated in
      // float32), so numerator and denominator see the same ones.
      f16x8 bp[2][2];
      bf16x8 bhi[2][2], blo[2][2];
      float psum = 0.f;
      const f16x2 ones = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            const float p0 = s[kb][8 * s2 + e], p1 = s[kb][8 * s2 + e + 1];
            if constexpr (SPLIT) {
              const bf16x2 hi = {(__bf16)p0, (__bf16)p1};
              const bf16x2 lo = {(__bf16)(p0 - (float)hi[0]), (__bf16)(p1 - (float)hi[1])};
              bhi[kb][s2][e] = hi[0];
              bhi[kb][s2][e + 1] = hi[1];
              blo[kb][s2][e] = lo[0];
              blo[kb][s2][e + 1] = lo[1];
              psum += p0 + p1;
            } else {
              const f16x2 pr = {(_Float16)p0, (_Float16)p1};
              bp[kb][s2][e] = pr[0];
              bp[kb][s2][e + 1] = pr[1];
              psum = __builtin_amdgcn_fdot2(pr, ones, psum, false);
            }
          }
      l_run = fmaf(l_run, alpha, psum);
      if (__any(alpha != 1.f)) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
          for (int j = 0; j < 16; ++j) o[i][j] *= alpha;
      }
      const int i16 = lane & 15, q2 = (lane >> 4) & 1;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const int key1 = kb * 32 + 16 * s2 + 4 * h + (i16 >> 2);
#pragma unroll
          for (int dvb = 0; dvb < NV; ++dvb) {
            const char* vp = sv + key1 * C::VSTR + (dvb * 32 + q2 * 16 + 4 * (i16 & 3)) * 2;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp + 8 * C::VSTR));
            union { struct { s16x4 lo, hi; } s; f16x8 v; bf16x8 b; } av;
            av.s.lo = lo;
            av.s.hi = hi;
            if constexpr (SPLIT) {
              o[dvb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av.b, bhi[kb][s2], o[dvb], 0, 0, 0);
              o[dvb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av.b, blo[kb][s2], o[dvb], 0, 0, 0);
            } else {
              o[dvb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av.v, bp[kb][s2], o[dvb], 0, 0, 0);
            }
          }
        }
    }
    if (more) store_tile((tile + 1) & 1);
    __syncthreads();
  }

  const float l_tot = sum_across_halves(l_run);
  const float inv = (SPLIT ? 1.f : a.v_unscale[kvh]) / l_tot;
  const size_t row0 = (size_t)batch * a.rows + wave_first;
  float* op0;
  float* lp0;
  if (a.n_split > 1) {
    const size_t prow = (size_t)split * a.n_batch * a.rows + row0;
    op0 = a.part_o + prow * D;
    lp0 = a.part_lse + prow;
  } else {
    op0 = a.out + row0 * D;
    lp0 = a.lse + row0;
  }
  // The wave's rows leave as whole rows through an LDS area of its own (every read of the tiles lies behind the loop's
  // last barrier).
  constexpr int TURN = 32 * (D * 4 + 16);
  static_assert(C::NW * TURN <= C::LDS_BYTES, "the rows are turned in the tile buffers");
  store_rows_via_lds<D>(o, inv, op0, a.rows - wave_first, smem + wave * TURN, lane);
  if (r < a.rows && h == 0) lp0[rw] = (m_run + __log2f(l_tot)) * kLn2;
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void k_attn_bf16(AttnArgs a) {
  attn_bf16_body<D, CAUSAL, !CAUSAL>(a, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.y);
}

// Both attentions in one launch, see k_attn_bf16_dma_pair; the query attention reads the copy of V as well.
template <int D>
__global__ __launch_bounds__(256, 2) void k_attn_bf16_pair(AttnArgs ac, AttnArgs aq, PairGrid g) {
  const int bid = blockIdx.x;
  if (bid < g.n_q_pad) {
    if (bid >= g.n_q) return;
    attn_bf16_body<D, false, false>(aq, bid % g.q_gx, bid / g.q_gx, 0, g.q_gy);
  } else {
    const int l = bid - g.n_q_pad;
    attn_bf16_body<D, true, false>(ac, l % g.c_gx, l / g.c_gx, 0, g.c_gy);
  }
}

// --------------------------------------------------------------- bf16, asynchronous tile loads (LDS DMA)
// Eight waves, one workgroup per compute unit; two things shape a step.
//
// (1) Software pipeline.  The products of the NEXT tile's scores are issued in the same straight-line
//     block as the softmax of the CURRENT tile, so the matrix pipe and the vector ALU of a SIMD work at
//     the same time without relying on a second wave being in the other phase:
//         step t:   S(t+1) = K(t+1) Q^T      (MFMA)   |   P(t) = exp2(S(t) c - m)      (VALU)
//                   O^T   += V(t)^T P(t)^T   (MFMA)
//     To keep that block free of branches a wave splits its tiles into `n_full` unmasked tiles (this
//     path) and at most one tail tile (the causal diagonal or the ragged end; plain path with masks),
//     and the running maximum is only raised when a row outgrows it by more than 2^8 ("lazy rescale"):
//     weights then stay below 256, which float32 sums and half-precision weights hold without loss, and the
//     rescale of O becomes a rare side branch ahead of the block.
// (2) Asynchronous tile loads.  K/V tiles travel from global memory straight into LDS
//     (global_load_lds_dwordx4: no staging registers, no LDS store instructions) into a ring of three K
//     slots and three V slots, two tiles ahead of their use, so a load has two full steps to land
//     (KG = 2: two slots of each, one tile ahead).
//
// KG = 1: the eight waves hold 256 rows.  KG = 2, for short problems, whose longest row tile's chain of steps and not the
// total work sets the duration: four row groups (128 rows) x two key groups.  A step stages 128 keys, each key group
// takes 64, and the two partial results meet through LDS at the end.  The tiles are twice as large, so the ring has two
// slots and a load one step to land.  Against register-staged, not pipelined kernels with two key groups (pair calls): 32
// heads x 1540 rows 49.8 -> 44.9 us, x 500 rows 21.0 -> 19.5, 16 heads x 3900 rows 92 -> 81; d = 64, 24 heads x 2600 rows
// 52 -> 46, x 3900 rows 93 -> 77.  Which problems take which kernel: attn_bf16_shape.
//
// A wave-wide DMA instruction fills 1 KB of LDS contiguously (lane i -> base + 16 i), i.e. four 256-byte
// rows (eight 128-byte rows at d = 64) with no room for padding, so the tiles are stored unpadded and XOR-swizzled instead: the 16-byte
// chunk c of row r sits at chunk position c ^ (r & 15) for K (16 consecutive rows of one fragment read
// land in 16 different bank groups) and at c ^ 4 (r & 3) for V: a transposing read takes, from each of 8 rows,
// the 64 bytes of one 4-chunk group, and LDS serves 32 lanes (4 of those rows) per cycle over its 64 banks, so the
// 4 rows have to sit in the 4 different groups.  (c ^ 2 (r & 7) spreads 16 lanes' 32-byte pieces instead; the
// counters showed every such read paying two extra cycles of bank conflicts.)  Which global chunk a lane fetches
// is free, so the swizzle costs nothing on the load side; on the read side it is folded into per-lane address
// registers.
//
// d = 64: two rows share the 256 bytes that one access cycle covers, so the swizzle goes by the row pair: K chunk c at
// c ^ ((r >> 1) & 7), V chunk c at c ^ 4 ((r >> 1) & 1).  A wave needs about half the registers and LDS, so two
// workgroups share a compute unit and overlap each other's products and weights: no software pipeline, whose second
// set of scores would cost that (128 registers per wave).  Problems of few workgroups with two key groups take one per
// compute unit and the pipeline instead (32 heads x 1200 rows: 24.7 -> 22.4 us).  The vector ALU is its busiest unit: nine
// vector instructions per product, issued in 55 % of the SIMD cycles, against 36 % for the matrix unit (24 heads over 8 x
// 6450 rows).  Against a register-staged eight-wave kernel, whole pair calls: 24 heads x 6450 rows 185 -> 180 us, 32 x 4120
// 113 -> 105, 56 x 9000 689 -> 651, 32 x 20000 (causal call alone) 1768 -> 1695 (0.97 PFLOP/s).
template <int D, int KG, int WGS>  // WGS: workgroups per compute unit
struct DmaCfg {
  static constexpr int NW = 8, RG = NW / KG, BQ = 32 * RG;   // waves, row groups, rows per workgroup
  static constexpr int BK = 64, BKT = BK * KG;               // keys per wave and per workgroup in a step
  static constexpr int NSLOT = KG == 1 ? 3 : 2;              // tiles in the ring, and how far ahead K and V are requested
  static constexpr int ROWB = D * 2, CPR = ROWB / 16;        // bytes and 16-byte chunks per row
  static constexpr int TILE = BKT * ROWB;                    // unpadded
  static constexpr int MERGE = 64 * (D / 2 + 2) * 4;         // one wave's outputs, maxima and sums
  static constexpr bool QLDS = KG == 2 && WGS == 1;                // the query rows come through LDS (dma_query)
  static constexpr int QROWS = 2 * NSLOT * TILE, LDS_BYTES = QROWS + (QLDS ? BQ * ROWB : 0);  // they lie behind the ring
  static constexpr int NI = TILE / 1024 / NW, RPI = 1024 / ROWB;  // requests per wave and tile, rows per request
  static constexpr int NQ = BQ * ROWB / 1024 / NW;                // requests per wave for the query rows
  static constexpr bool PIPE = WGS == 1;                          // software pipeline inside a wave (1)
  static __device__ __forceinline__ int kswz(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
  static __device__ __forceinline__ int vswz(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }
};

template <int D, int KG, int WGS, bool CAUSAL>
__device__ __forceinline__ void attn_bf16_dma_body(const AttnArgs a, int bx, int by, int bz, int grid_y) {
  using C = DmaCfg<D, KG, WGS>;
  constexpr int NW = C::NW, BQ = C::BQ, BK = C::BK, BKT = C::BKT, ROWB = C::ROWB, CPR = C::CPR, NI = C::NI;
  constexpr int ND = D / 16, NV = D / 32;
  constexpr int TILE = C::TILE, NSLOT = C::NSLOT;
  constexpr float TAU = 8.f;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  // K(j) in slot j % NSLOT at smem + slot * TILE; V(j) in slot j % NSLOT at smem + (NSLOT + slot) * TILE

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int rw = lane & 31, h = lane >> 5;
  int kvh, batch, qt;
  map_block(a, CAUSAL, bx, by, grid_y, &kvh, &batch, &qt);
  // Row tiles of a causal problem start so that the first one, which walks the fewest keys, is the one with few rows:
  // its rows are the remainder, rounded up to whole key tiles (d = 128, 32 heads x 4120 rows: 171 -> 166 us as a pair
  // call, x 8200: 532 -> 522; multiples of 256 unchanged).
  const int q0 = qt * BQ - (CAUSAL ? (BQ - (a.rows % BQ + BK - 1) / BK * BK) % BQ : 0);
  const int split = bz;
  const int kv_begin = CAUSAL ? 0 : split * a.chunk;
  const int kv_end = CAUSAL ? min(a.m, q0 + BQ) : min(a.m, kv_begin + a.chunk);
  const int span = kv_end - kv_begin;
  const int n_tiles = (span + BKT - 1) / BKT;

  const int rg = KG == 1 ? wave : wave % C::RG, kg = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave / C::RG);
  const int r = q0 + rg * 32 + rw;
  const int wave_first = q0 + rg * 32;
  // A wave all of whose rows lie before the first or past the last one (the ragged row tile of a problem: the first of a
  // causal one, the last of another) computes nothing: no full tiles, no tail.  It still sends its share of the tile
  // requests and meets the barriers; its SIMD is left to the waves that have rows.
  const bool has_rows = wave_first >= 0 && wave_first < a.rows;
  // Of the tiles' keys a wave takes 64: unmasked ones in its first n_full tiles, and at most one masked tile after them.
  const int lim = !has_rows ? 0 : CAUSAL ? min(wave_first + 1, span) : span;
  const int n_full = lim >= kg * BK + BK ? (lim - kg * BK - BK) / BKT + 1 : 0;
  const int tail_key = n_full * BKT + kg * BK;
  const bool has_tail = has_rows && tail_key < span && (!CAUSAL || tail_key <= wave_first + 31);

  bf16x8 bq[ND];
  if constexpr (!C::QLDS) {
    const char* qp = static_cast<const char*>(a.q) + ((size_t)batch * a.rows + max(0, min(r, a.rows - 1))) * ROWB + h * 16;
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) bq[dc] = *reinterpret_cast<const bf16x8*>(qp + dc * 32);
  }
  const char* kbase = static_cast<const char*>(a.k) + ((size_t)kvh * a.m + kv_begin) * D * 2;
  const char* vbase = static_cast<const char*>(a.v) + ((size_t)kvh * a.m + kv_begin) * D * 2;

  // ---- DMA side: wave w, instruction i fills rows RPI (NI w + i) .. + RPI - 1 of a tile; lane L lands at chunk
  //      position L % CPR of row RPI (NI w + i) + L / CPR and therefore fetches the chunk that belongs there
  uint32_t goff_k[NI], goff_v[NI];
  int grow[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int row = C::RPI * (NI * wave + i) + lane / CPR, pos = lane % CPR;
    grow[i] = row;
    goff_k[i] = (uint32_t)(row * ROWB + ((pos ^ C::kswz(row)) * 16));
    goff_v[i] = (uint32_t)(row * ROWB + ((pos ^ C::vswz(row)) * 16));
  }
  // The DMA is issued through inline assembly on purpose: the compiler then neither orders later LDS
  // reads behind it (it would drain every outstanding load before each fragment read) nor counts it in
  // its own vmcnt bookkeeping; arrival is awaited by hand (s_waitcnt vmcnt) ahead of the barriers.
  // LDS destinations are handled as integers (LDS address of smem + byte offset, all scalar): a generic pointer
  // would drag a null check and 64-bit arithmetic into every request.  wave_rows: where this wave's rows start
  // inside a tile, as a scalar of its own; the row and mask arithmetic above keeps the per-lane `wave`.
  const uint32_t smem_at = (uint32_t)(size_t)(const __attribute__((address_space(3))) char*)smem;
  const uint32_t wave_rows = __builtin_amdgcn_readfirstlane((uint32_t)(NI * wave * 1024));
  auto dma16 = [&](const char* tile_base, uint32_t byte_off, uint32_t lds_off) {  // lds_off: byte offset into smem
    const uint32_t m0v = __builtin_amdgcn_readfirstlane(smem_at + lds_off);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(m0v), "v"(byte_off), "s"(tile_base)
                 : "memory", "m0");
  };
  auto dma_tile = [&](const char* base, int j, uint32_t slot, const uint32_t (&goff)[NI], bool is_v) {
    const int k0 = j * BKT;
    const char* tp = base + (size_t)k0 * (D * 2);
    if (kv_begin + k0 + BKT <= a.m) {
#pragma unroll
      for (int i = 0; i < NI; ++i) dma16(tp, goff[i], slot + wave_rows + i * 1024);
    } else {
      // last tile of the cache: rows past the final key re-read that key (their scores are masked)
      const int last = a.m - 1 - kv_begin - k0;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int row = grow[i], pos = lane % CPR;
        const int src_chunk = pos ^ (is_v ? C::vswz(row) : C::kswz(row));
        const uint32_t off = (uint32_t)(min(row, last) * (D * 2) + src_chunk * 16);
        dma16(tp, off, slot + wave_rows + i * 1024);
      }
    }
  };
  // The query rows come the same way with two key groups and one workgroup per compute unit, as whole rows with the swizzle
  // of K, and are read as fragments once they have landed.  Loaded as fragments from memory, 16 bytes from each of 32 rows
  // per instruction and by both key groups, every line is requested eight times, and short workgroups wait for that
  // (32 heads x 1540 rows, pair calls: 45.2 -> 42.8 us, x 700 22.8 -> 21.5, 64 x 1000 44.2 -> 40.7; d = 64, 24 x 1200 21.7 ->
  // 21.3).  The other shapes keep the fragment loads, which are in flight beside the tiles: 256 rows, d = 128, 32 heads x 4120
  // 1 % faster, x 2500 1.3 % slower, 64 x 20480 0.8 % slower; two workgroups per compute unit, d = 64, 24 x 2600 1 % faster,
  // 32 x 4120 1.7 % slower.
  auto dma_query = [&]() {
    const int first = max(q0, 0);
    const char* qp = static_cast<const char*>(a.q) + ((size_t)batch * a.rows + first) * ROWB;
    const uint32_t to = __builtin_amdgcn_readfirstlane((uint32_t)(C::QROWS + C::NQ * wave * 1024));
#pragma unroll
    for (int i = 0; i < C::NQ; ++i) {
      const int row = C::RPI * (C::NQ * wave + i) + lane / CPR;
      const int src = max(q0 + row, 0) - first;  // rows before the first or past the last one re-read that one
      dma16(qp, (uint32_t)(min(src, a.rows - 1 - first) * ROWB + ((lane % CPR) ^ C::kswz(row)) * 16), to + i * 1024);
    }
  };
  // where this wave's keys of a tile start
  auto kslot = [&](int j) { return smem + (j % NSLOT) * TILE + kg * BK * ROWB; };
  auto vslot = [&](int j) { return smem + (NSLOT + j % NSLOT) * TILE + kg * BK * ROWB; };
  auto kslot_off = [&](int j) { return (uint32_t)((j % NSLOT) * TILE); };  // the same as byte offsets, for the requests
  auto vslot_off = [&](int j) { return (uint32_t)((NSLOT + j % NSLOT) * TILE); };

  // ---- read side: per-lane swizzled byte offsets inside a slot
  uint32_t kaddr[ND], vaddr[NV];
  {
    const int x = C::kswz(rw);
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) kaddr[dc] = (uint32_t)(rw * ROWB + (((2 * dc + h) ^ x) * 16));
    const int i16 = lane & 15, q2 = (lane >> 4) & 1;
    const int vrow = 4 * h + (i16 >> 2);       // + kb*32 + s2*16 (+8): multiples of 8, do not change the swizzle
    const int xv = C::vswz(vrow);
#pragma unroll
    for (int dvb = 0; dvb < NV; ++dvb) {
      const int c = 4 * dvb + 2 * q2 + ((i16 & 3) >> 1);
      vaddr[dvb] = (uint32_t)(vrow * ROWB + ((c ^ xv) * 16) + 8 * (i16 & 1));
    }
  }

  f32x16 o[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[i][j] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;
  const float c2 = a.scale * kLog2e;

  auto lift = [&](float mx) {
    if (__any(mx > m_ref + TAU)) {
      const float m_new = fmaxf(m_ref, mx);
      const float al = __builtin_amdgcn_exp2f(m_ref - (m_new == -INFINITY ? 0.f : m_new));  // a row still without mass: 0, not NaN
      l_run *= al;
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[i][j] *= al;
      m_ref = m_new;
    }
  };
  auto row_max = [&](const f32x16 (&s)[2]) {
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int j = 0; j < 16; ++j) mx = fmaxf(mx, s[kb][j]);
    mx = max_across_halves(mx);
    return mx * c2;
  };
  auto kfrags = [&](const char* ks, int kb, bf16x8 (&ak)[ND]) {
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) ak[dc] = *reinterpret_cast<const bf16x8*>(ks + kaddr[dc] + kb * 32 * ROWB);
  };
  auto qfrags = [&]() {
    const char* qs = smem + C::QROWS + rg * 32 * ROWB;
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) bq[dc] = *reinterpret_cast<const bf16x8*>(qs + kaddr[dc]);
  };
  // V^T fragments of key group g (16 keys) for the NV blocks of O^T: two transposing reads each
  auto vfrags = [&](const char* vs, int g, f16x8 (&av)[NV]) {
#pragma unroll
    for (int dvb = 0; dvb < NV; ++dvb) {
      const char* vp = vs + vaddr[dvb] + g * 16 * ROWB;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp + 8 * ROWB));
      union { struct { s16x4 lo, hi; } s; f16x8 v; } u;
      u.s.lo = lo;
      u.s.hi = hi;
      av[dvb] = u.v;
    }
  };
  // LDS reads may not be moved across this point (everything else may): keeps a fragment load where it was written,
  // i.e. one group of products ahead of its use, instead of right in front of it
  constexpr int kHoldLds = 0x47F;
  auto weights_pv = [&](f32x16 (&s)[2], const char* vs, float m_use) {
    f16x8 bp[2][2];
    f16x8 va[2][NV];
    vfrags(vs, 0, va[0]);  // lands while the weights are computed
    __builtin_amdgcn_sched_barrier(kHoldLds);
    float psum = 0.f;
    const f16x2 ones = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const float p0 = __builtin_amdgcn_exp2f(fmaf(s[kb][8 * s2 + e], c2, -m_use));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(s[kb][8 * s2 + e + 1], c2, -m_use));
          f16x2 pr = {(_Float16)p0, (_Float16)p1};
          bp[kb][s2][e] = pr[0];
          bp[kb][s2][e + 1] = pr[1];
          psum = __builtin_amdgcn_fdot2(pr, ones, psum, false);
        }
    l_run += psum;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (g + 1 < 4) {
        vfrags(vs, g + 1, va[(g + 1) & 1]);
        __builtin_amdgcn_sched_barrier(kHoldLds);
      }
#pragma unroll
      for (int dvb = 0; dvb < NV; ++dvb)
        o[dvb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[g & 1][dvb], bp[g >> 1][g & 1], o[dvb], 0, 0, 0);
    }
  };

  // the masked tile: scores of keys past the row (causal) or past the last key do not count
  auto mask = [&](int tile, f32x16 (&sc)[2]) {
    // number of keys of the tile that count for this lane's row, less the lane's first key: made here, not ahead of the loop
    int n_ok = (CAUSAL ? min(kv_end, r + 1) : kv_end) - (kv_begin + tile * BKT + kg * BK) - 4 * h;
    asm volatile("" : "+v"(n_ok));
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (kb * 32 + 8 * (j >> 2) + (j & 3) >= n_ok) sc[kb][j] = -INFINITY;
  };
  auto scores = [&](const char* ks, f32x16 (&s)[2]) {
    bf16x8 ak0[ND], ak1[ND];
    kfrags(ks, 0, ak0);
    kfrags(ks, 1, ak1);
#pragma unroll
    for (int j = 0; j < 16; ++j) { s[0][j] = 0.f; s[1][j] = 0.f; }
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) {
      s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak0[dc], bq[dc], s[0], 0, 0, 0);
      s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak1[dc], bq[dc], s[1], 0, 0, 0);
    }
  };
  if constexpr (!C::PIPE) {
    // K(0), V(0) must have landed; with three slots K(1), V(1) stay in flight
    constexpr int AHEAD = NSLOT - 1;
    dma_tile(kbase, 0, kslot_off(0), goff_k, false);
    dma_tile(vbase, 0, vslot_off(0), goff_v, true);
    if (AHEAD > 1 && n_tiles > 1) {
      dma_tile(kbase, 1, kslot_off(1), goff_k, false);
      dma_tile(vbase, 1, vslot_off(1), goff_v, true);
      __builtin_amdgcn_s_waitcnt(0x0F70 | 2 * NI);
    } else {
      __builtin_amdgcn_s_waitcnt(0x0F70);
    }
    __builtin_amdgcn_s_barrier();
    for (int tile = 0; tile < n_tiles; ++tile) {
      const bool more = tile + AHEAD < n_tiles;  // into the slots that step tile - 1 has left
      if (more) {
        dma_tile(kbase, tile + AHEAD, kslot_off(tile + AHEAD), goff_k, false);
        dma_tile(vbase, tile + AHEAD, vslot_off(tile + AHEAD), goff_v, true);
      }
      const uint32_t at = __builtin_amdgcn_readfirstlane(kslot_off(tile) + kg * BK * ROWB);
      const char* ks = smem + at;
      const char* vs = smem + NSLOT * TILE + at;
      if (tile < n_full) {
        f32x16 s[2];
        scores(ks, s);
        lift(row_max(s));
        weights_pv(s, vs, m_ref == -INFINITY ? 0.f : m_ref);
      } else if (tile == n_full && has_tail) {
        f32x16 s[2];
        scores(ks, s);
        mask(tile, s);
        lift(row_max(s));
        weights_pv(s, vs, m_ref == -INFINITY ? 0.f : m_ref);
      }
      if (AHEAD > 1 && more) __builtin_amdgcn_s_waitcnt(0x0F70 | 2 * NI);
      else __builtin_amdgcn_s_waitcnt(0x0F70);
      __builtin_amdgcn_s_barrier();
    }
  } else {
    // ---- prologue: Q and K(0) must have landed before the first scores, V(0) and K(1) before step 0
    constexpr int AHEAD_K = NSLOT, AHEAD_V = NSLOT - 1;  // step t requests K(t + AHEAD_K), V(t + AHEAD_V)
    if constexpr (C::QLDS) dma_query();
    dma_tile(kbase, 0, kslot_off(0), goff_k, false);
    dma_tile(vbase, 0, vslot_off(0), goff_v, true);
    if (n_tiles > 1) dma_tile(kbase, 1, kslot_off(1), goff_k, false);
    if constexpr (NSLOT == 3) {
      if (n_tiles > 1) dma_tile(vbase, 1, vslot_off(1), goff_v, true);
      if (n_tiles > 2) dma_tile(kbase, 2, kslot_off(2), goff_k, false);
    }
    if (NSLOT == 3 && n_tiles > 2) __builtin_amdgcn_s_waitcnt(0x0F70 | 4 * NI);
    else if (NSLOT == 3 && n_tiles > 1) __builtin_amdgcn_s_waitcnt(0x0F70 | 3 * NI);
    else if (n_tiles > 1) __builtin_amdgcn_s_waitcnt(0x0F70 | 2 * NI);
    else __builtin_amdgcn_s_waitcnt(0x0F70 | NI);
    __builtin_amdgcn_s_barrier();
    if constexpr (C::QLDS) qfrags();
    f32x16 sA[2], sB[2];
    scores(kslot(0), sA);
    // K(0) has been read by every wave before step 0 refills its slot: the reads' arrival is waited for here (lgkmcnt(0)),
    // because the products that use them may be scheduled behind the barrier
    if (NSLOT == 3 && n_tiles > 2) __builtin_amdgcn_s_waitcnt(0x0070 | 2 * NI);
    else if (NSLOT == 3 && n_tiles > 1) __builtin_amdgcn_s_waitcnt(0x0070 | NI);
    else __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();

    // step `tile`: S(tile) is in sc; computes S(tile + 1) into sn and adds tile's V contribution
    auto step = [&](int tile, f32x16 (&sc)[2], f32x16 (&sn)[2]) {
      const bool more_k = tile + AHEAD_K < n_tiles, more_v = tile + AHEAD_V < n_tiles;
      if (more_k) dma_tile(kbase, tile + AHEAD_K, kslot_off(tile + AHEAD_K), goff_k, false);
      if (more_v) dma_tile(vbase, tile + AHEAD_V, vslot_off(tile + AHEAD_V), goff_v, true);
      const char* k_next = kslot(tile + 1);
      const char* v_cur = vslot(tile);
      if (tile < n_full) {
        bf16x8 ak0[ND], ak1[ND];
        kfrags(k_next, 0, ak0);
        lift(row_max(sc));
        kfrags(k_next, 1, ak1);
#pragma unroll
        for (int j = 0; j < 16; ++j) { sn[0][j] = 0.f; sn[1][j] = 0.f; }
#pragma unroll
        for (int dc = 0; dc < ND; ++dc) sn[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak0[dc], bq[dc], sn[0], 0, 0, 0);
#pragma unroll
        for (int dc = 0; dc < ND; ++dc) sn[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak1[dc], bq[dc], sn[1], 0, 0, 0);
        weights_pv(sc, v_cur, m_ref == -INFINITY ? 0.f : m_ref);
      } else if (tile == n_full && has_tail) {
        mask(tile, sc);
        lift(row_max(sc));
        weights_pv(sc, v_cur, m_ref == -INFINITY ? 0.f : m_ref);
      }
      // three slots: the tiles needed by the next step were requested one step ago, wait for all but this step's loads
      if (NSLOT == 2) __builtin_amdgcn_s_waitcnt(0x0F70);
      else if (more_k) __builtin_amdgcn_s_waitcnt(0x0F70 | 2 * NI);
      else if (more_v) __builtin_amdgcn_s_waitcnt(0x0F70 | NI);
      else __builtin_amdgcn_s_waitcnt(0x0F70);
      __builtin_amdgcn_s_barrier();
    };
    for (int tile = 0; tile < n_tiles; tile += 2) {
      step(tile, sA, sB);
      if (tile + 1 < n_tiles) step(tile + 1, sB, sA);
    }
  }

  if constexpr (KG == 2) {
    // the second key group hands its running maximum, row sum and accumulator to the first through LDS
    // (element e of lane l at word e * 64 + l: conflict-free), which rescales both to the common maximum
    float* mg = reinterpret_cast<float*>(smem + rg * C::MERGE) + lane;
    if (kg == 1) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) mg[(i * 16 + j) * 64] = o[i][j];
      mg[(NV * 16) * 64] = m_ref;
      mg[(NV * 16 + 1) * 64] = l_run;
    }
    __syncthreads();
    if (kg == 1) return;
    const float m1 = mg[(NV * 16) * 64], l1 = mg[(NV * 16 + 1) * 64];
    const float m_new = fmaxf(m_ref, m1);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float a0 = __builtin_amdgcn_exp2f(m_ref - m_use), a1 = __builtin_amdgcn_exp2f(m1 - m_use);
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[i][j] = o[i][j] * a0 + mg[(i * 16 + j) * 64] * a1;
    l_run = l_run * a0 + l1 * a1;
    m_ref = m_new;
  }
  const float l_tot = sum_across_halves(l_run);
  const float inv = a.v_unscale[kvh] / l_tot;
  if (!has_rows) return;
  const size_t row0 = (size_t)batch * a.rows + wave_first;
  float* op0;
  float* lp0;
  if (a.n_split > 1) {
    const size_t prow = (size_t)split * a.n_batch * a.rows + row0;
    op0 = a.part_o + prow * D;
    lp0 = a.part_lse + prow;
  } else {
    op0 = a.out + row0 * D;
    lp0 = a.lse + row0;
  }
  // whole rows through the wave's share (12 KB; 6 KB at d = 64) of the tile slots (free: the last step ended with every
  // request landed and a barrier), 16 rows at a time; with two key groups through the row group's merge area, which only
  // this wave still touches
  if constexpr (KG == 1)
    store_rows_via_lds<D, 2>(o, inv, op0, a.rows - wave_first, smem + wave * (C::LDS_BYTES / NW), lane);
  else
    store_rows_via_lds<D>(o, inv, op0, a.rows - wave_first, smem + rg * C::MERGE, lane);
  if (r < a.rows && h == 0) lp0[rw] = (m_ref + __log2f(l_tot)) * kLn2;
}

template <int D, int KG, int WGS, bool CAUSAL>
__global__ __launch_bounds__(512, 2 * WGS) void k_attn_bf16_dma(AttnArgs a) {
  attn_bf16_dma_body<D, KG, WGS, CAUSAL>(a, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.y);
}

// Both attentions of the path in ONE launch (same head dimension, same workgroup shape).  The query attention's
// workgroups come first in the linear order and each walks ALL keys for its rows (no key chunks, no partial results,
// no merge): such a workgroup lasts as long as the causal problem's longest row tile, which is handed out right
// behind it, so the query attention hides inside the causal one instead of waiting for it.  n_q_pad, the query
// workgroups rounded up to a multiple of 8, keeps the causal workgroups on the XCD slots map_block assumes.
template <int D, int KG, int WGS>
__global__ __launch_bounds__(512, 2 * WGS) void k_attn_bf16_dma_pair(AttnArgs ac, AttnArgs aq, PairGrid g) {
  const int bid = blockIdx.x;
  if (bid < g.n_q_pad) {
    if (bid >= g.n_q) return;
    attn_bf16_dma_body<D, KG, WGS, false>(aq, bid % g.q_gx, bid / g.q_gx, 0, g.q_gy);
  } else {
    const int l = bid - g.n_q_pad;
    attn_bf16_dma_body<D, KG, WGS, true>(ac, l % g.c_gx, l / g.c_gx, 0, g.c_gy);
  }
}

// out = sum_s w_s * part_o[s] with w_s = exp(lse_s - lse), lse = log sum_s exp(lse_s).  d/4 threads per row, four
// channels each; with many chunks, S groups of them share a row: group g takes the chunks g, g + S, ..., all U of them
// requested at once (S * U chunks at most), and the groups meet in LDS.  Every order is fixed, so the result is
// deterministic.  A chunk without mass (lse = -inf: every score -inf, outputs 0 / 0) and a request past the last chunk are
// left out and not multiplied by a weight of zero, which would turn infinite or undefined outputs into NaN.
// One thread walking all chunks of its channels spends a memory round trip on each: 35 us for 64 rows x 64 chunks, 6 us
// with S = 8.  Few chunks take fewer groups and requests: eight groups for 9 chunks request mostly the same words (8128
// rows x 9 chunks, whole query call with its own keys: 86 us with S = 8, 72 with S = 2), and so do eight requests for two
// chunks.
template <int S, int U>
__global__ __launch_bounds__(256) void k_attn_merge(AttnArgs a, int d) {
  __shared__ f32x4 s_acc[256];
  __shared__ float s_mx[256], s_den[256];
  const int tpr = d / 4, c4 = threadIdx.x % tpr;
  const int slot = threadIdx.x / tpr, sg = slot % S;
  const size_t n_rows = (size_t)a.n_batch * a.rows;
  const size_t row = (size_t)blockIdx.x * (256 / tpr / S) + slot / S;
  const size_t row_c = row < n_rows ? row : n_rows - 1;
  float l[U];
  f32x4 x[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const size_t at = (size_t)min(sg + u * S, a.n_split - 1) * n_rows + row_c;
    l[u] = a.part_lse[at];
    x[u] = *reinterpret_cast<const f32x4*>(a.part_o + at * d + c4 * 4);
  }
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (sg + u * S >= a.n_split) l[u] = -INFINITY;
    mx = fmaxf(mx, l[u]);
  }
  const float m_use = mx == -INFINITY ? 0.f : mx;
  float den = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const bool counts = l[u] != -INFINITY;
    const float w = counts ? expf(l[u] - m_use) : 0.f;
    den += w;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = counts ? fmaf(w, x[u][e], acc[e]) : acc[e];
  }
  if constexpr (S > 1) {
    s_acc[threadIdx.x] = acc;
    s_mx[threadIdx.x] = mx;
    s_den[threadIdx.x] = den;
    __syncthreads();
    if (sg > 0) return;
    float m_all = mx;
#pragma unroll
    for (int g = 1; g < S; ++g) m_all = fmaxf(m_all, s_mx[threadIdx.x + g * tpr]);
    const float m_use = m_all == -INFINITY ? 0.f : m_all;
    const float w0 = expf(mx - m_use);
    den *= w0;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= w0;
#pragma unroll
    for (int g = 1; g < S; ++g) {
      const float w = expf(s_mx[threadIdx.x + g * tpr] - m_use);
      const f32x4 x = s_acc[threadIdx.x + g * tpr];
      den = fmaf(w, s_den[threadIdx.x + g * tpr], den);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(w, x[e], acc[e]);
    }
    mx = m_all;
  }
  if (row >= n_rows) return;
  const float inv = 1.f / den;
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] *= inv;
  *reinterpret_cast<f32x4*>(a.out + row * d + c4 * 4) = acc;
  if (c4 == 0) a.lse[row] = mx + logf(den);
}

template <int D>
hipError_t raise_lds_limit() {
  const void* all[] = {reinterpret_cast<const void*>(&k_attn_bf16<D, true>), reinterpret_cast<const void*>(&k_attn_bf16<D, false>),
                       reinterpret_cast<const void*>(&k_attn_bf16_pair<D>)};
  for (const void* f : all) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, Bf16Cfg<D>::LDS_BYTES);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int D, int KG, int WGS>
hipError_t raise_lds_limit_dma() {
  const void* query = nullptr;
  if constexpr (KG == 1) query = reinterpret_cast<const void*>(&k_attn_bf16_dma<D, 1, WGS, false>);
  const void* all[] = {reinterpret_cast<const void*>(&k_attn_bf16_dma<D, KG, WGS, true>),
                       reinterpret_cast<const void*>(&k_attn_bf16_dma_pair<D, KG, WGS>), query};
  for (const void* f : all) {
    if (f == nullptr) continue;
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, DmaCfg<D, KG, WGS>::LDS_BYTES);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int D, bool CAUSAL>
hipError_t run_bf16(const AttnLaunch& l, hipStream_t s) {
  using C = Bf16Cfg<D>;
  AttnArgs a = make_args(l);
  dim3 grid = attn_grid(&a, (l.rows + C::BQ - 1) / C::BQ);
  hipLaunchKernelGGL((k_attn_bf16<D, CAUSAL>), grid, dim3(C::NT), C::LDS_BYTES, s, a);
  return hipGetLastError();
}

template <int D, int KG, int WGS, bool CAUSAL>
hipError_t run_bf16_dma(const AttnLaunch& l, hipStream_t s) {
  using C = DmaCfg<D, KG, WGS>;
  AttnArgs a = make_args(l);
  dim3 grid = attn_grid(&a, (l.rows + C::BQ - 1) / C::BQ);
  hipLaunchKernelGGL((k_attn_bf16_dma<D, KG, WGS, CAUSAL>), grid, dim3(512), C::LDS_BYTES, s, a);
  return hipGetLastError();
}

AttnShape bf16_shape(const AttnLaunch& l) {
  return l.n_self > 0 ? AttnShape::kStaged : attn_bf16_shape(l.causal, l.n_batch, l.batch_per_kv, l.rows, l.m, l.d);
}

template <int D, bool CAUSAL>
hipError_t run_bf16_d(const AttnLaunch& l, hipStream_t s) {
  if (attn_bf16_reads_v16(l) != (l.v_unscale != nullptr)) return hipErrorInvalidValue;  // V prepared iff the shape reads the copy
  constexpr int WGS = D == 128 ? 1 : 2;
  const AttnShape shape = bf16_shape(l);
  if (shape == AttnShape::kDma) return run_bf16_dma<D, 1, WGS, CAUSAL>(l, s);
  if constexpr (CAUSAL) {
    if (shape == AttnShape::kDmaKeys2) return run_bf16_dma<D, 2, WGS, true>(l, s);
    if (shape == AttnShape::kDmaKeys2One) return run_bf16_dma<D, 2, 1, true>(l, s);
  }
  return run_bf16<D, CAUSAL>(l, s);
}

// Pair launch: the query problem takes the causal problem's kernel shape and walks all keys in one chunk.
bool pair_grid(AttnArgs* ac, AttnArgs* aq, int bq, PairGrid* g, unsigned* total) {
  const dim3 gc = attn_grid(ac, (ac->rows + bq - 1) / bq), gq = attn_grid(aq, (aq->rows + bq - 1) / bq);
  g->c_gx = (int)gc.x; g->c_gy = (int)gc.y; g->q_gx = (int)gq.x; g->q_gy = (int)gq.y;
  const long long n_q = (long long)gq.x * gq.y, n_c = (long long)gc.x * gc.y;
  const long long n_q_pad = (n_q + 7) / 8 * 8;
  if (n_q_pad + n_c > 0x7FFFFFFFll) return false;
  g->n_q = (int)n_q; g->n_q_pad = (int)n_q_pad;
  *total = (unsigned)(n_q_pad + n_c);
  return true;
}

template <int D, int KG, int WGS>
hipError_t run_pair_dma(const AttnLaunch& c, const AttnLaunch& q, hipStream_t s) {
  using C = DmaCfg<D, KG, WGS>;
  AttnArgs ac = make_args(c), aq = make_args(q);
  PairGrid g;
  unsigned total;
  if (!pair_grid(&ac, &aq, C::BQ, &g, &total)) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_attn_bf16_dma_pair<D, KG, WGS>), dim3(total), dim3(512), C::LDS_BYTES, s, ac, aq, g);
  return hipGetLastError();
}

template <int D>
hipError_t run_pair_staged(const AttnLaunch& c, const AttnLaunch& q, hipStream_t s) {
  using C = Bf16Cfg<D>;
  AttnArgs ac = make_args(c), aq = make_args(q);
  PairGrid g;
  unsigned total;
  if (!pair_grid(&ac, &aq, C::BQ, &g, &total)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_attn_bf16_pair<D>, dim3(total), dim3(C::NT), C::LDS_BYTES, s, ac, aq, g);
  return hipGetLastError();
}

template <int D>
hipError_t run_pair_d(const AttnLaunch& c, const AttnLaunch& q, hipStream_t s) {
  constexpr int WGS = D == 128 ? 1 : 2;
  switch (bf16_shape(c)) {
    case AttnShape::kDma: return run_pair_dma<D, 1, WGS>(c, q, s);
    case AttnShape::kDmaKeys2: return run_pair_dma<D, 2, WGS>(c, q, s);
    case AttnShape::kDmaKeys2One: return run_pair_dma<D, 2, 1>(c, q, s);
    default: return run_pair_staged<D>(c, q, s);
  }
}

}  // namespace

// Nearly every attention kernel uses more dynamic LDS than the default limit allows; the limit belongs to the function
// on a device, so it is raised for ALL variants the first time any attention call runs on that device.  After that
// no attention call touches anything but the stream, whatever variant its shape selects (HIP graph capture).
hipError_t attn_prepare_device() {
  constexpr int kMaxDev = 64;
  static std::mutex mu;
  static bool done[kMaxDev] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDev) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (done[dev]) return hipSuccess;
  const hipError_t all[] = {
      raise_lds_limit<128>(), raise_lds_limit<64>(), raise_lds_limit_dma<128, 2, 1>(), raise_lds_limit_dma<64, 2, 2>(),
      raise_lds_limit_dma<64, 2, 1>(), raise_lds_limit_dma<128, 1, 1>(), raise_lds_limit_dma<64, 1, 2>(), attn_f32_raise_limits()};
  for (hipError_t x : all)
    if (x != hipSuccess) return x;
  done[dev] = true;
  return hipSuccess;
}

bool attn_bf16_reads_v16(const AttnLaunch& l) { return l.causal || bf16_shape(l) != AttnShape::kStaged; }

hipError_t launch_attn_bf16(const AttnLaunch& l, hipStream_t s) {
  const hipError_t e = attn_prepare_device();
  if (e != hipSuccess) return e;
  if (l.d == 128) return l.causal ? run_bf16_d<128, true>(l, s) : run_bf16_d<128, false>(l, s);
  return l.causal ? run_bf16_d<64, true>(l, s) : run_bf16_d<64, false>(l, s);
}

hipError_t launch_attn_bf16_pair(const AttnLaunch& causal, const AttnLaunch& query, hipStream_t s) {
  const hipError_t e = attn_prepare_device();
  if (e != hipSuccess) return e;
  if (causal.v_unscale == nullptr || query.v != causal.v) return hipErrorInvalidValue;  // both read the prepared copy
  AttnLaunch q = query;
  q.n_split = 1;
  q.chunk = q.m;
  q.part_o = nullptr;
  q.part_lse = nullptr;
  return causal.d == 128 ? run_pair_d<128>(causal, q, s) : run_pair_d<64>(causal, q, s);
}

template <int S, int U>
static hipError_t run_merge(const AttnLaunch& l, hipStream_t s) {
  const int rpb = 256 / (l.d / 4) / S;
  const size_t n_rows = (size_t)l.n_batch * l.rows;
  hipLaunchKernelGGL((k_attn_merge<S, U>), dim3((unsigned)((n_rows + rpb - 1) / rpb)), dim3(256), 0, s, make_args(l), l.d);
  return hipGetLastError();
}

hipError_t launch_attn_merge(const AttnLaunch& l, hipStream_t s) {
  // all chunks in one batch of requests, spread over no more groups of threads and no more requests than that takes
  if (l.n_split <= 2) return run_merge<1, 2>(l, s);
  if (l.n_split <= 4) return run_merge<1, 4>(l, s);
  if (l.n_split <= 8) return run_merge<1, 8>(l, s);
  if (l.n_split <= 16) return run_merge<2, 8>(l, s);
  if (l.n_split <= 32) return run_merge<4, 8>(l, s);
  if (l.n_split <= kMaxParts) return run_merge<8, 8>(l, s);
  return hipErrorInvalidValue;
}

}  // namespace samkv

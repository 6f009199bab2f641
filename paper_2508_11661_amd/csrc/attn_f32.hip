// Float32 attention over the compacted cache (both problems of attn.hip, same definitions), on the float32 matrix cores.
//
// One workgroup = 4 waves that share 32 query rows; wave w takes the key tiles w, w + 4, ... of 32 keys, and the four
// partial results meet in LDS at the end.
//   S^T = K Q^T     v_mfma_f32_32x32x2_f32, A = K, B = the query rows (registers, loaded once).  A product takes two
//                   channels, one per half-wave; which two is free as long as A and B agree, so a half-wave loads 16
//                   bytes of a row and feeds four products with them.
//   O^T += V^T P^T  the same instruction.  The accumulator of S^T holds, in register j of half-wave h, key
//                   8 (j / 4) + 4 h + j % 4 for the lane's row: exactly a B operand of two keys, so the weights
//                   never leave their registers; A = one V value per lane (a load takes 128 bytes of two rows).
// What bounds it: the matrix unit, 64 cycles per product and 128 products per tile at d = 128.  A product needs so
// little (a K chunk per 256 cycles, a V value per 64) that the operands come straight from L2 into registers, requested
// up to 8 chunks or 32 values ahead (K in groups of four chunks, which together take whole 128-byte lines of their 32
// rows: spread out, the lines left L1 between their four quarters): no LDS tiles, hence no barrier in the loop and no
// lockstep, and the two waves of a SIMD (two workgroups per compute unit) fill each other's softmax, start and merge.
// Measured, 32 heads over 8 KV heads, d = 128: 2307 -> 203 us at M = 1540 (8.4 -> 96 TFLOP/s; the matrix unit is busy 70 %
// of the cycles, the rest is what 6 workgroups per compute unit spend starting and merging), 133 TFLOP/s at M = 6144,
// 137 at M = 12288, of 157 at the matrix unit's rate.  Tiles staged in LDS by asynchronous loads, two barriers per step:
// 228 us and 123 TFLOP/s at the first two sizes.  The kernel before these spent 5 LDS reads per 4 FMA on the vector ALU.
#include "attn_common.hpp"

namespace samkv {
namespace {

constexpr int KG = 4;  // key groups: waves of a workgroup

template <int D>
struct F32Cfg {
  static constexpr int ROW = D * 4 + 16;  // bytes of an output row in LDS (pad: 16 rows hit 64 distinct banks)
  static constexpr int STATS = KG * 32 * ROW;
  static constexpr int LDS_BYTES = STATS + KG * 32 * 8;  // a partial result per wave, then its rows' maxima and sums
};

// 32 query rows from q0 on against the keys [kv_begin, kv_end), part bz of them, by four waves of which this is number kg;
// `smem` is theirs.  Waves that are not `active` only meet the barrier.
template <int D, bool CAUSAL>
__device__ __forceinline__ void attn_f32_unit(const AttnArgs& a, int kvh, int batch, int q0, int kv_begin, int kv_end, int bz,
                                              int kg, char* smem, bool active) {
  using C = F32Cfg<D>;
  constexpr int NV = D / 32, NI = D / 8;  // 32-channel blocks of O^T; 16-byte chunks per lane and row
  constexpr int ROWB = D * 4, NKX = 8, NVX = 32;

  const int lane = threadIdx.x & 63;
  const int rw = lane & 31, h = lane >> 5;
  const int r = q0 + rw;
  if (!active) kv_end = kv_begin;
  const char* kbase = static_cast<const char*>(a.k) + (size_t)kvh * a.m * ROWB;
  const char* vbase = static_cast<const char*>(a.v) + (size_t)kvh * a.m * ROWB;
  const int last = a.m - 1;  // keys past the final one are read as that one (their weights are zero)

  // K chunk i of the tile at k0: 16 bytes of row rw at channel 8 i + 4 h;  V value (j, b): key 8 (j/4) + 4 h + j%4,
  // channel 32 b + rw.  Byte offsets stay below 2^31 (m is limited by the entry points).
  auto kchunk = [&](int k0, int i) {
    return *reinterpret_cast<const f32x4*>(kbase + (uint32_t)(min(k0 + rw, last) * ROWB + h * 16) + i * 32);
  };
  auto vvalue = [&](int k0, int j, int b) {
    return *reinterpret_cast<const float*>(vbase + (uint32_t)(min(k0 + 8 * (j >> 2) + 4 * h + (j & 3), last) * ROWB + rw * 4) + b * 128);
  };

  f32x4 bq[NI], kx[NKX];
  float vx[NVX];
  int k0 = kv_begin + kg * 32;
#pragma unroll
  for (int i = 0; i < NKX; ++i) kx[i] = kchunk(k0, i);
  {
    const char* qp = static_cast<const char*>(a.q) + ((size_t)batch * a.rows + max(0, min(r, a.rows - 1))) * ROWB + h * 16;
#pragma unroll
    for (int i = 0; i < NI; ++i) bq[i] = *reinterpret_cast<const f32x4*>(qp + i * 32);
  }
  f32x16 o[NV];
#pragma unroll
  for (int b = 0; b < NV; ++b)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[b][j] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c2 = (float)((double)a.scale * 1.4426950408889634074);

  for (; k0 < kv_end; k0 += 32 * KG) {
    f32x16 s;
#pragma unroll
    for (int j = 0; j < 16; ++j) s[j] = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kx[i % NKX][e], bq[i][e], s, 0, 0, 0);
      constexpr int F = NI - NKX;
      if (i < F && i % 4 == 3) {
#pragma unroll
        for (int u = 0; u < 4; ++u) kx[(i - 3 + u) % NKX] = kchunk(k0, i - 3 + u + NKX);
      }
      if (i >= F) {  // the last eight chunks: four V values with each, the first NVX of the tile
#pragma unroll
        for (int u = 0; u < 4; ++u) vx[(i - F) * 4 + u] = vvalue(k0, ((i - F) * 4 + u) / NV, ((i - F) * 4 + u) % NV);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if ((CAUSAL && k0 + 31 > q0) || k0 + 32 > kv_end) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int key = k0 + 8 * (j >> 2) + 4 * h + (j & 3);
        if (key >= kv_end || (CAUSAL && key > r)) s[j] = -INFINITY;
      }
    }
    float mx = s[0];
#pragma unroll
    for (int j = 1; j < 16; ++j) mx = fmaxf(mx, s[j]);
    mx = max_across_halves(mx);
    const float m_new = fmaxf(m_run, mx * c2);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
    m_run = m_new;
    float psum = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      s[j] = __builtin_amdgcn_exp2f(fmaf(s[j], c2, -m_use));
      psum += s[j];
    }
    l_run = fmaf(l_run, alpha, psum);
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int b = 0; b < NV; ++b)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[b][j] *= alpha;
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
#pragma unroll
      for (int b = 0; b < NV; ++b)
        o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vx[(j * NV + b) % NVX], s[j], o[b], 0, 0, 0);
      if ((j + 1) * NV + NVX <= 16 * NV) {
#pragma unroll
        for (int b = 0; b < NV; ++b) vx[(j * NV + b) % NVX] = vvalue(k0, (j * NV + b + NVX) / NV, b);
      }
      if (j == 9 || j == 13) {
#pragma unroll
        for (int u = 0; u < 4; ++u) kx[j - 9 + u] = kchunk(k0 + 32 * KG, j - 9 + u);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // The four partial results meet in LDS, as whole rows; each wave then combines and writes eight of them.
  {
    const float l_tot = sum_across_halves(l_run);
    char* own = smem + (kg * 32 + rw) * C::ROW;
#pragma unroll
    for (int b = 0; b < NV; ++b)
#pragma unroll
      for (int j4 = 0; j4 < 4; ++j4) {
        const f32x4 x = {o[b][4 * j4], o[b][4 * j4 + 1], o[b][4 * j4 + 2], o[b][4 * j4 + 3]};
        *reinterpret_cast<f32x4*>(own + (b * 32 + 8 * j4 + 4 * h) * 4) = x;
      }
    float* st = reinterpret_cast<float*>(smem + C::STATS) + (kg * 32 + rw) * 2;
    if (h == 0) { st[0] = m_run; st[1] = l_tot; }
  }
  __syncthreads();
  const size_t row0 = (size_t)batch * a.rows + q0;
  float* op;
  float* lp;
  if (a.n_split > 1) {
    const size_t prow = (size_t)bz * a.n_batch * a.rows + row0;
    op = a.part_o + prow * D;
    lp = a.part_lse + prow;
  } else {
    op = a.out + row0 * D;
    lp = a.lse + row0;
  }
  constexpr int LPR = D / 4, RPI = 64 / LPR;  // lanes per row, rows per step
#pragma unroll
  for (int i = 0; i < 8 / RPI; ++i) {
    const int row = kg * 8 + i * RPI + lane / LPR, c4 = lane % LPR;
    const float* st = reinterpret_cast<const float*>(smem + C::STATS) + row * 2;
    float m_all = st[0];
#pragma unroll
    for (int g = 1; g < KG; ++g) m_all = fmaxf(m_all, st[g * 64]);
    const float m_use = m_all == -INFINITY ? 0.f : m_all;  // no mass in any group: every score is -inf
    float den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      const float w = __builtin_amdgcn_exp2f(st[g * 64] - m_use);
      const f32x4 x = *reinterpret_cast<const f32x4*>(smem + (g * 32 + row) * C::ROW + c4 * 16);
      den = fmaf(st[g * 64 + 1], w, den);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(x[e], w, acc[e]);
    }
    const float inv = 1.f / den;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= inv;
    if (active && q0 + row < a.rows) {
      *reinterpret_cast<f32x4*>(op + (size_t)row * D + c4 * 4) = acc;
      if (c4 == 0) lp[row] = (m_all + __log2f(den)) * kLn2;
    }
  }
}

template <int D, bool CAUSAL>
__device__ __forceinline__ void attn_f32_body(const AttnArgs a, int bx, int by, int bz, int grid_y) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int kvh, batch, qt;
  map_block(a, CAUSAL, bx, by, grid_y, &kvh, &batch, &qt);
  const int q0 = qt * 32, kv_begin = CAUSAL ? 0 : bz * a.chunk;
  // The first key group has the most tiles; which wave, and so which SIMD, that is goes round.
  const int kg = (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + (bx >> 3) + by) & (KG - 1);
  attn_f32_unit<D, CAUSAL>(a, kvh, batch, q0, kv_begin, CAUSAL ? min(a.m, q0 + 32) : min(a.m, kv_begin + a.chunk), bz, kg, smem,
                           true);
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(64 * KG, 2) void k_attn_f32(AttnArgs a) {
  attn_f32_body<D, CAUSAL>(a, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.y);
}

// Both attentions in one launch: the query attention's workgroups (key chunks as in its own launch, so the results are
// the same bits) come first, the causal ones fill the chip behind them.
template <int D>
__global__ __launch_bounds__(64 * KG, 2) void k_attn_f32_pair(AttnArgs ac, AttnArgs aq, PairGrid g) {
  const int bid = blockIdx.x;
  if (bid < g.n_q_pad) {
    if (bid >= g.n_q) return;
    const int per_split = g.q_gx * g.q_gy, split = bid / per_split, l = bid - split * per_split;
    attn_f32_body<D, false>(aq, l % g.q_gx, l / g.q_gx, split, g.q_gy);
  } else {
    const int l = bid - g.n_q_pad;
    attn_f32_body<D, true>(ac, l % g.c_gx, l / g.c_gx, 0, g.c_gy);
  }
}

template <int D, bool CAUSAL>
hipError_t run(const AttnLaunch& l, hipStream_t s) {
  AttnArgs a = make_args(l);
  const dim3 grid = attn_grid(&a, (l.rows + 31) / 32);
  hipLaunchKernelGGL((k_attn_f32<D, CAUSAL>), grid, dim3(64 * KG), F32Cfg<D>::LDS_BYTES, s, a);
  return hipGetLastError();
}

template <int D>
hipError_t run_pair(const AttnLaunch& c, const AttnLaunch& q, hipStream_t s) {
  AttnArgs ac = make_args(c), aq = make_args(q);
  const dim3 gc = attn_grid(&ac, (c.rows + 31) / 32), gq = attn_grid(&aq, (q.rows + 31) / 32);
  const long long n_q = (long long)gq.x * gq.y * gq.z, n_q_pad = (n_q + 7) / 8 * 8, n_c = (long long)gc.x * gc.y;
  if (n_q_pad + n_c > 0x7FFFFFFFll) return hipErrorInvalidValue;
  PairGrid g;
  g.n_q = (int)n_q; g.n_q_pad = (int)n_q_pad;
  g.q_gx = (int)gq.x; g.q_gy = (int)gq.y; g.c_gx = (int)gc.x; g.c_gy = (int)gc.y;
  hipLaunchKernelGGL((k_attn_f32_pair<D>), dim3((unsigned)(n_q_pad + n_c)), dim3(64 * KG), F32Cfg<D>::LDS_BYTES, s, ac, aq, g);
  return hipGetLastError();
}

// ---------------------------------------------------------------- products of half-precision terms
// The half-precision matrix instructions do sixteen times the work of the float32 ones.  A float32 number x, scaled by a power
// of two, is the sum of two half-precision terms, x = hi + lo with lo = half(x - hi), to 2^-23 of x, and a product of two such
// numbers is hi hi' + hi lo' + lo hi' to 2^-22: three products, accumulated in float32, of which a sum takes 24 roundings at
// d = 128 where the float32 instruction takes 64.  Errors against 64 bits over the sizes below: 3.2e-7 to 7.9e-7 of the
// outputs' norm, 5.7e-7 to 1.6e-6 with float32 products; largest difference of a log-sum-exp 2.9e-6 to 6.5e-6, 7.3e-6 to
// 1.2e-5.
//   Eight waves of 32 query rows.  NKG = 1: 256 rows, one stream of keys, 32 a step.  NKG = 2, for short problems: 128 rows,
// whose keys two groups of waves share, 64 a step; their results meet in LDS at the end.
//   Staging: a step's K and V rows come as float32 into registers a step ahead; the next step turns them into two planes of
// terms per tensor in LDS (double-buffered, one barrier per step), between the products of its scores, whose matrix
// instructions leave room for five vector instructions each.  Planes and fragments are laid out and read as in attn.hip.
//   Scales: a wave stages four consecutive rows of a key group (or two such fours) and scales all of them alike, K and V apart,
// by the largest magnitude of the last rows that did not fit the scale in use; a lane whose numbers leave its range, most of
// them only by the rows' first ones, makes the wave look for a new one.  The scales of a step's fours stand beside the planes:
// a register of scores or weights belongs to one four.  A weight is multiplied by its four's V scale over the largest one met
// so far, `unit`, before it is split, and the accumulator is in those units.  Query rows have a scale each.
//   Numbers that the terms would not hold: an infinity or NaN, magnitudes whose scores might pass float32's range, a lane's
// numbers all 2^-12 or more below the scale's magnitude, a four of V rows 2^-8 below `unit`.  The wave that meets one raises a
// flag, and the whole workgroup starts again with float32 products (attn_f32_unit).
//   What bounds it: the matrix unit and the device's power limit (M = 6850, 32 heads: 1100 us, 920 with all inputs zero), for short
// problems the chain of steps.  32 heads over 8 KV heads, d = 128, float32 products -> these: M = 700 53 -> 38 us, 1540 178 -> 80,
// 4120 1077 -> 403, 6850 2913 -> 1100 (350 TFLOP/s); 24 heads, d = 64, M = 1540 75 -> 49, 6450 1019 -> 459.
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int D, int NKG>
struct SplitCfg {
  static constexpr int NW = 8, RG = NW / NKG, BQ = 32 * RG;   // waves, row groups, rows per workgroup
  static constexpr int BK = 32, BKT = BK * NKG;               // keys per wave and per workgroup in a step
  static constexpr int ROWB = D * 2;                          // bytes of a row in a plane
  static constexpr int PLANE = BKT * ROWB, BUF = 4 * PLANE;   // K high, K low, V high, V low
  static constexpr int SCALES = 2 * BUF;                      // [buffer][key group][K, V][half-wave][4] factors that undo the scales
  static constexpr int FLAGS = SCALES + 2 * NKG * 16 * 4;     // [buffer] the tile needs float32 products
  static constexpr int QROWS = NKG == 1 ? 2 * BUF + 1024 : BUF;  // the query rows on their way to registers: not where the first tile goes
  static constexpr int MERGE = 64 * (D / 2 + 4) * 4;          // one wave's outputs, maxima, sums and units
  static constexpr int TURN = (NKG == 1 ? 8 : 32) * (D * 4 + 16);
  static constexpr int END = NKG == 1 ? NW * TURN : RG * (MERGE > TURN ? MERGE : TURN);
  static constexpr int TILES = FLAGS + 16 > END ? FLAGS + 16 : END, PLAIN = 2 * F32Cfg<D>::LDS_BYTES;
  static constexpr int LDS_BYTES = TILES > PLAIN ? TILES : PLAIN;
  static_assert(QROWS + NW * 16 * D * 4 <= (NKG == 1 ? LDS_BYTES : SCALES), "room for 16 query rows of each wave");
  // staging: lanes per row, rows per load, rows and loads per wave
  static constexpr int LPR = D / 4, RPI = 64 / LPR, RW = BKT / NW, NI = RW / RPI;
  static __device__ __forceinline__ int kswz(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
  static __device__ __forceinline__ int vswz(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }
};

// x0 s and x1 s, s a power of two, as the sum of two half-precision terms each
__device__ __forceinline__ void split2(float x0, float x1, float s, uint32_t* hi, uint32_t* lo) {
  const f16x2 h = {(_Float16)(x0 * s), (_Float16)(x1 * s)};
  uint32_t hw = __builtin_bit_cast(uint32_t, h);
  asm("" : "+v"(hw));  // one packed conversion, whose halves the next line reads
  const f16x2 g = __builtin_bit_cast(f16x2, hw);
  const f16x2 l = {(_Float16)fmaf(x0, s, -(float)g[0]), (_Float16)fmaf(x1, s, -(float)g[1])};
  *hi = hw;
  *lo = __builtin_bit_cast(uint32_t, l);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_max(uint32_t v) {
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = dpp_max<0xB1>(v);
  v = dpp_max<0x4E>(v);
  v = dpp_max<0x141>(v);
  v = dpp_max<0x140>(v);
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return __builtin_amdgcn_readfirstlane(max(b[0], b[1]));
}
__device__ __forceinline__ float abs_max(const f32x4& x) {  // NaN wins
  const float m = __builtin_elementwise_maximum(__builtin_fabsf(x[0]), __builtin_fabsf(x[1]));
  return __builtin_fabsf(__builtin_elementwise_maximum(__builtin_elementwise_maximum(m, __builtin_fabsf(x[2])), __builtin_fabsf(x[3])));
}

// Numbers whose largest magnitude has the biased exponent e are multiplied by 2^(kExpScale - 127 - e), which puts that
// magnitude into [2^12, 2^13); a later one may be up to 2^kExpRoom times as large.
constexpr uint32_t kExpScale = 266, kExpUnscale = 12, kExpLow = 13, kExpHigh = 127 + 60, kExpRoom = 3, kExpSpan = 12;
constexpr float kUnitSpan = 0x1p-8f;  // see above: fours of V rows and `unit`
constexpr int kHoldLds = 0x47F;  // LDS accesses may not be moved across such a scheduling barrier
// whether the largest magnitude m of some numbers that are scaled by e is too large, or so small that they lose bits
__device__ __forceinline__ bool outside(float m, uint32_t e) {
  const uint32_t u = __float_as_uint(m);
  return u - 1u < ((e - kExpSpan) << 23) - 1u || u >= min(e + kExpRoom, 255u) << 23;
}

template <int D, int NKG, bool CAUSAL>
__device__ __forceinline__ void attn_split_body(const AttnArgs a, int bx, int by, int bz, int grid_y) {
  using C = SplitCfg<D, NKG>;
  constexpr int BQ = C::BQ, BK = C::BK, BKT = C::BKT, ROWB = C::ROWB, NI = C::NI;
  constexpr int ND = D / 16, NV = D / 32;
  constexpr float TAU = 8.f;
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int rw = lane & 31, h = lane >> 5;
  int kvh, batch, qt;
  map_block(a, CAUSAL, bx, by, grid_y, &kvh, &batch, &qt);
  const int q0 = qt * BQ - (CAUSAL ? (BQ - (a.rows % BQ + BK - 1) / BK * BK) % BQ : 0);
  const int kv_begin = CAUSAL ? 0 : bz * a.chunk;
  const int kv_end = CAUSAL ? min(a.m, q0 + BQ) : min(a.m, kv_begin + a.chunk);
  const int span = kv_end - kv_begin;
  const int n_tiles = (span + BKT - 1) / BKT;

  const int rg = NKG == 1 ? wave : wave % C::RG, kg = NKG == 1 ? 0 : wave / C::RG;
  const int wave_first = q0 + rg * 32;
  const int r = wave_first + rw;
  const bool has_rows = wave_first >= 0 && wave_first < a.rows;
  const int lim = !has_rows ? 0 : CAUSAL ? min(wave_first + 1, span) : span;
  const int n_full = lim >= kg * BK + BK ? (lim - kg * BK - BK) / BKT + 1 : 0;
  const int tail_key = n_full * BKT + kg * BK;
  const bool has_tail = has_rows && tail_key < span && (!CAUSAL || tail_key <= wave_first + 31);

  const char* kbase = static_cast<const char*>(a.k) + ((size_t)kvh * a.m + kv_begin) * D * 4;
  const char* vbase = static_cast<const char*>(a.v) + ((size_t)kvh * a.m + kv_begin) * D * 4;
  const char* qbase = static_cast<const char*>(a.q) + (size_t)batch * a.rows * D * 4;

  // ---- staging
  f32x4 rk[NI], rv[NI];
  const int srow = wave * C::RW + lane / C::LPR, scol = lane % C::LPR;
  auto load_tile = [&](int j) {
    const int k0 = j * BKT;
    const char* kt = kbase + (size_t)k0 * (D * 4);
    const char* vt = vbase + (size_t)k0 * (D * 4);
    const int last = a.m - 1 - kv_begin - k0;
    if (last >= BKT - 1) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t off = (uint32_t)((srow + i * C::RPI) * (D * 4) + scol * 16);
        rk[i] = *reinterpret_cast<const f32x4*>(kt + off);
        rv[i] = *reinterpret_cast<const f32x4*>(vt + off);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const uint32_t off = (uint32_t)(min(srow + i * C::RPI, last) * (D * 4) + scol * 16);
        rk[i] = *reinterpret_cast<const f32x4*>(kt + off);
        rv[i] = *reinterpret_cast<const f32x4*>(vt + off);
      }
    }
  };
  // where the first of its numbers go; the swizzle of the others' rows enters by XOR, as their row bits are its own
  const uint32_t kst = (uint32_t)(srow * ROWB + (((scol >> 1) ^ C::kswz(srow)) * 16) + 8 * (scol & 1));
  const uint32_t vst = (uint32_t)(srow * ROWB + (((scol >> 1) ^ C::vswz(srow)) * 16) + 8 * (scol & 1));
  float* scales = reinterpret_cast<float*>(smem + C::SCALES);
  int* flags = reinterpret_cast<int*>(smem + C::FLAGS);
  uint32_t ek = kExpLow, ev = kExpLow;  // the biased exponents by which this wave scales its rows of K and of V
  bool odd_rows = false;
  float sk, sv;
  auto check_tile = [&]() {
    float mk[NI], mv[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      mk[i] = abs_max(rk[i]);
      mv[i] = abs_max(rv[i]);
    }
    bool off = false;
#pragma unroll
    for (int i = 0; i < NI; ++i) off = off | outside(mk[i], ek) | outside(mv[i], ev);
    odd_rows = false;
    if (__any(off)) {
      uint32_t tk = 0, tv = 0;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        tk = max(tk, __float_as_uint(mk[i]));
        tv = max(tv, __float_as_uint(mv[i]));
      }
      tk = wave_max(tk);
      tv = wave_max(tv);
      if (tk != 0) ek = max(tk >> 23, (uint32_t)kExpLow);
      if (tv != 0) ev = max(tv >> 23, (uint32_t)kExpLow);
      off = false;
#pragma unroll
      for (int i = 0; i < NI; ++i) off = off | outside(mk[i], ek) | outside(mv[i], ev);
      odd_rows = __any(off) || ek >= kExpHigh || ev == 255;
    }
    sk = __uint_as_float((kExpScale - ek) << 23);
    sv = __uint_as_float((kExpScale - ev) << 23);
  };
  // converts and stores the tile in 4 NI pieces of two numbers
  uint2 hi2, lo2;
  auto put_piece = [&](int j, int pc) {
    const int n = pc / 4;
    if (pc % 4 == 0) split2(rk[n][0], rk[n][1], sk, &hi2.x, &lo2.x);
    if (pc % 4 == 1) {
      split2(rk[n][2], rk[n][3], sk, &hi2.y, &lo2.y);
      char* at = smem + ((kst ^ (uint32_t)(C::kswz(n * C::RPI) * 16)) + (j & 1) * C::BUF) + n * C::RPI * ROWB;
      *reinterpret_cast<uint2*>(at) = hi2;
      *reinterpret_cast<uint2*>(at + C::PLANE) = lo2;
    }
    if (pc % 4 == 2) split2(rv[n][0], rv[n][1], sv, &hi2.x, &lo2.x);
    if (pc % 4 == 3) {
      split2(rv[n][2], rv[n][3], sv, &hi2.y, &lo2.y);
      char* at = smem + ((vst ^ (uint32_t)(C::vswz(n * C::RPI) * 16)) + (j & 1) * C::BUF) + n * C::RPI * ROWB;
      *reinterpret_cast<uint2*>(at + 2 * C::PLANE) = hi2;
      *reinterpret_cast<uint2*>(at + 3 * C::PLANE) = lo2;
    }
  };
  auto put_scales = [&](int j) {
    if (lane == 0) {
#pragma unroll
      for (int gi = 0; gi < C::RW / 4; ++gi) {
        const int g8 = wave * (C::RW / 4) + gi, grp = g8 >> 3, gg = g8 & 7;  // group of four rows: key group, place in it
        float* p = scales + (((j & 1) * NKG + grp) * 2) * 8 + (gg & 1) * 4 + (gg >> 1);
        p[0] = __uint_as_float((ek - kExpUnscale) << 23);
        p[8] = __uint_as_float((ev - kExpUnscale) << 23);
      }
      if (odd_rows) flags[j & 1] = 1;
    }
  };
  auto store_tile = [&](int j) {
    check_tile();
#pragma unroll
    for (int pc = 0; pc < 4 * NI; ++pc) put_piece(j, pc);
    put_scales(j);
  };

  load_tile(0);
  if (t < 2) flags[t] = 0;

  // ---- query rows, requested behind the first tile, which is staged and followed by the next while they come
  f16x8 qhi[ND], qlo[ND];
  float cq;
  bool q_slow;
  const float c2 = (float)((double)a.scale * 1.4426950408889634074);
  {
    // They come as whole rows and are turned through LDS (16 rows at a time, swizzled by the row): a load in the layout of the
    // fragments touches 32 lines, 16 of them per wave 4000 cycles ahead of the first tile (32 heads x 700 rows 39.2 -> 37.8 us,
    // 64 x 300 24.2 -> 23.2).
    constexpr int NQ = 16 / C::RPI;
    f32x4 raw[2][NQ], x[ND][2];
    const int ql = lane / C::LPR, qc = lane % C::LPR;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int row = max(0, min(wave_first + 16 * p + i * C::RPI + ql, a.rows - 1));
        raw[p][i] = *reinterpret_cast<const f32x4*>(qbase + (size_t)row * (D * 4) + qc * 16);
      }
    __syncthreads();  // the flags are clear
    store_tile(0);
    if (n_tiles > 1) load_tile(1);
    char* turn = smem + C::QROWS + wave * (16 * D * 4);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int row = i * C::RPI + ql;
        *reinterpret_cast<f32x4*>(turn + row * (D * 4) + (qc ^ row) * 16) = raw[p][i];
      }
      __builtin_amdgcn_wave_barrier();
      if (rw / 16 == p) {
#pragma unroll
        for (int dc = 0; dc < ND; ++dc)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            x[dc][i] = *reinterpret_cast<const f32x4*>(turn + rw % 16 * (D * 4) + ((dc * 4 + h * 2 + i) ^ rw % 16) * 16);
      }
      __builtin_amdgcn_wave_barrier();
    }
    float mq[ND], most = 0.f;
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) {
      mq[dc] = __builtin_elementwise_maximum(abs_max(x[dc][0]), abs_max(x[dc][1]));
      most = __builtin_elementwise_maximum(most, mq[dc]);
    }
    const uint32_t mb = __float_as_uint(most) & 0x7FFFFFFFu;
    const auto sw = __builtin_amdgcn_permlane32_swap(mb, mb, false, false);
    const uint32_t eq = max(max(sw[0], sw[1]) >> 23, (uint32_t)kExpLow);
    bool off = eq >= kExpHigh;
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) off = off || outside(mq[dc], eq);
    q_slow = __any(off);
    const float sq = __uint_as_float((kExpScale - eq) << 23);
    cq = c2 * __uint_as_float((eq - kExpUnscale) << 23);
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) {
      u32x4 hi, lo;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        uint32_t h0, h1, l0, l1;
        split2(x[dc][i][0], x[dc][i][1], sq, &h0, &l0);
        split2(x[dc][i][2], x[dc][i][3], sq, &h1, &l1);
        hi[2 * i] = h0; hi[2 * i + 1] = h1; lo[2 * i] = l0; lo[2 * i + 1] = l1;
      }
      qhi[dc] = __builtin_bit_cast(f16x8, hi);
      qlo[dc] = __builtin_bit_cast(f16x8, lo);
    }
  }

  // ---- read side
  // (the chunk number's other bits enter by XOR: rows and planes are multiples of their size)
  uint32_t kaddr, vaddr;
  {
    kaddr = (uint32_t)((kg * BK + rw) * ROWB + ((h ^ C::kswz(rw)) * 16));
    const int i16 = lane & 15, q2 = (lane >> 4) & 1;
    const int vrow = 4 * h + (i16 >> 2), c = 2 * q2 + ((i16 & 3) >> 1);
    vaddr = (uint32_t)(2 * C::PLANE + (kg * BK + vrow) * ROWB + ((c ^ C::vswz(vrow)) * 16) + 8 * (i16 & 1));
  }

  f32x16 o[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[i][j] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;
  float unit = __uint_as_float(8u << 23);

  auto vfrag = [&](const char* vp) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp + 8 * ROWB));
    union { struct { s16x4 lo, hi; } s; f16x8 v; } u;
    u.s.lo = lo;
    u.s.hi = hi;
    return u.v;
  };

  auto compute = [&](int tile, bool masked) {
    const uint32_t kat = kaddr + (tile & 1) * C::BUF, vat = vaddr + (tile & 1) * C::BUF;
    auto kread = [&](int dc, f16x8* hi, f16x8* lo) {
      const char* at = smem + (kat ^ (uint32_t)(dc * 32));
      *hi = *reinterpret_cast<const f16x8*>(at);
      *lo = *reinterpret_cast<const f16x8*>(at + C::PLANE);
    };
    const float* sc = scales + (((tile & 1) * NKG + kg) * 2) * 8 + h * 4;
    f32x4 fk = *reinterpret_cast<const f32x4*>(sc);
    f32x4 fv = *reinterpret_cast<const f32x4*>(sc + 8);
    const int key0 = kv_begin + tile * BKT + kg * BK;
    f32x16 s, sl;
#pragma unroll
    for (int j = 0; j < 16; ++j) { s[j] = 0.f; sl[j] = 0.f; }
    f32x4 cg;
    {
      constexpr int KA = 3;  // fragments in registers
      f16x8 kh[KA], kl[KA];
#pragma unroll
      for (int dc = 0; dc + 1 < KA; ++dc) kread(dc, &kh[dc], &kl[dc]);
#pragma unroll
      for (int dc = 0; dc < ND; ++dc) {
        if (dc + KA - 1 < ND) kread(dc + KA - 1, &kh[(dc + KA - 1) % KA], &kl[(dc + KA - 1) % KA]);
        __builtin_amdgcn_sched_barrier(kHoldLds);
#pragma unroll
        for (int pc = 0; pc < 4 * NI / ND; ++pc) put_piece(tile + 1, dc * (4 * NI / ND) + pc);
        s = __builtin_amdgcn_mfma_f32_32x32x16_f16(kl[dc % KA], qhi[dc], s, 0, 0, 0);
        sl = __builtin_amdgcn_mfma_f32_32x32x16_f16(kh[dc % KA], qlo[dc], sl, 0, 0, 0);
        f32x16& x = dc & 1 ? s : sl;
        x = __builtin_amdgcn_mfma_f32_32x32x16_f16(kh[dc % KA], qhi[dc], x, 0, 0, 0);
      }
      put_scales(tile + 1);
      if (tile + 2 < n_tiles) load_tile(tile + 2);
#pragma unroll
      for (int j = 0; j < 16; ++j) s[j] += sl[j];
#pragma unroll
      for (int g = 0; g < 4; ++g) cg[g] = fmaxf(cq * fk[g], 0x1p-126f);  // not 0, which would make NaN of a masked score
    }
    if (masked) {
      const int n_ok = (CAUSAL ? min(kv_end, r + 1) : kv_end) - key0 - 4 * h;
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (8 * (j >> 2) + (j & 3) >= n_ok) s[j] = -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int g = 0; g < 4; ++g)
      mx = fmaxf(mx, fmaxf(fmaxf(s[4 * g], s[4 * g + 1]), fmaxf(s[4 * g + 2], s[4 * g + 3])) * cg[g]);
    mx = max_across_halves(mx);
    const float v_most = fmaxf(fmaxf(fv[0], fv[1]), fmaxf(fv[2], fv[3])), v_least = fminf(fminf(fv[0], fv[1]), fminf(fv[2], fv[3]));
    if (__any(mx > m_ref + TAU || v_most > unit || v_least < unit * kUnitSpan)) {
      const float m_new = fmaxf(m_ref, mx), u_new = fmaxf(unit, max_across_halves(v_most));
      const float al = __builtin_amdgcn_exp2f(m_ref - (m_new == -INFINITY ? 0.f : m_new)), alo = al * (unit / u_new);
      l_run *= al;
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[i][j] *= alo;
      m_ref = m_new;
      unit = u_new;
      if (__any(v_least < unit * kUnitSpan) && lane == 0) flags[(tile + 1) & 1] = 1;
    }
    const float per_unit = __uint_as_float((261u << 23) - __float_as_uint(unit));
    const float m_use = m_ref == -INFINITY ? 0.f : m_ref;
    float psum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      s[j] = __builtin_amdgcn_exp2f(fmaf(s[j], cg[j >> 2], -m_use));
      psum[j & 3] += s[j];
    }
    l_run += (psum[0] + psum[1]) + (psum[2] + psum[3]);
    {
      f16x8 ph[2], pl[2];
      auto split_weights = [&](int s2) {
        u32x4 hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          uint32_t hw, lw;
          split2(s[8 * s2 + 2 * e], s[8 * s2 + 2 * e + 1], fv[2 * s2 + (e >> 1)] * per_unit, &hw, &lw);
          hi[e] = hw; lo[e] = lw;
        }
        ph[s2] = __builtin_bit_cast(f16x8, hi);
        pl[s2] = __builtin_bit_cast(f16x8, lo);
      };
      // two 32-channel blocks of 16 keys at a time, their fragments read one such group ahead
      constexpr int NG = NV;
      f16x8 vh[2][2], vl[2][2];
      auto vread = [&](int g) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const char* at = smem + (vat ^ (uint32_t)((g * 2 + b) % NV * 64)) + (g * 2 / NV) * 16 * ROWB;
          vh[g & 1][b] = vfrag(at);
          vl[g & 1][b] = vfrag(at + C::PLANE);
        }
      };
      vread(0);
      split_weights(0);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g + 1 < NG) vread(g + 1);
        __builtin_amdgcn_sched_barrier(kHoldLds);
        const int s2 = g * 2 / NV, b0 = g * 2 % NV;
        if (g == 0) split_weights(1);
#pragma unroll
        for (int b = 0; b < 2; ++b) o[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl[g & 1][b], ph[s2], o[b0 + b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 2; ++b) o[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh[g & 1][b], pl[s2], o[b0 + b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 2; ++b) o[b0 + b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh[g & 1][b], ph[s2], o[b0 + b], 0, 0, 0);
      }
    }
  };

  if (q_slow) flags[0] = 1;
  __syncthreads();
  bool plain = false;
  for (int tile = 0; tile < n_tiles; ++tile) {
    const int odd = flags[tile & 1];
    const bool more = tile + 1 < n_tiles, busy = tile < n_full || (tile == n_full && has_tail);
    if (busy) {
      check_tile();
      compute(tile, tile == n_full);
    } else if (more) {
      store_tile(tile + 1);
      if (tile + 2 < n_tiles) load_tile(tile + 2);
    }
    if (odd) {
      plain = true;
      break;
    }
    __syncthreads();
  }
  if (plain || flags[0] || flags[1]) {
    __syncthreads();
    const int set = wave >> 2;
#pragma unroll 1
    for (int u = set; u < C::BQ / 32; u += 2) {
      const int first = q0 + 32 * u;
      attn_f32_unit<D, CAUSAL>(a, kvh, batch, first, kv_begin, CAUSAL ? min(a.m, first + 32) : kv_end, bz, wave & 3,
                               smem + set * F32Cfg<D>::LDS_BYTES, first >= 0 && first < a.rows);
      __syncthreads();
    }
    return;
  }

  if constexpr (NKG == 2) {
    float* mg = reinterpret_cast<float*>(smem + rg * C::MERGE) + lane;
    if (kg == 1) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) mg[(i * 16 + j) * 64] = o[i][j];
      mg[(NV * 16) * 64] = m_ref;
      mg[(NV * 16 + 1) * 64] = l_run;
      mg[(NV * 16 + 2) * 64] = unit;
    }
    __syncthreads();
    if (kg == 1) return;
    const float m1 = mg[(NV * 16) * 64], l1 = mg[(NV * 16 + 1) * 64], unit1 = mg[(NV * 16 + 2) * 64];
    const float m_new = fmaxf(m_ref, m1), u_new = fmaxf(unit, unit1);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float a0 = __builtin_amdgcn_exp2f(m_ref - m_use), a1 = __builtin_amdgcn_exp2f(m1 - m_use);
    const float s0 = a0 * (unit / u_new), s1 = a1 * (unit1 / u_new);
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[i][j] = o[i][j] * s0 + mg[(i * 16 + j) * 64] * s1;
    l_run = l_run * a0 + l1 * a1;
    m_ref = m_new;
    unit = u_new;
  }
  if (!has_rows) return;
  const float l_tot = sum_across_halves(l_run);
  const float inv = unit * 0.0078125f / l_tot;
  const size_t row0 = (size_t)batch * a.rows + wave_first;
  float* op0;
  float* lp0;
  if (a.n_split > 1) {
    const size_t prow = (size_t)bz * a.n_batch * a.rows + row0;
    op0 = a.part_o + prow * D;
    lp0 = a.part_lse + prow;
  } else {
    op0 = a.out + row0 * D;
    lp0 = a.lse + row0;
  }
  if constexpr (NKG == 1)
    store_rows_via_lds<D, 4>(o, inv, op0, a.rows - wave_first, smem + wave * C::TURN, lane);
  else
    store_rows_via_lds<D>(o, inv, op0, a.rows - wave_first, smem + rg * (C::MERGE > C::TURN ? C::MERGE : C::TURN), lane);
  if (r < a.rows && h == 0) lp0[rw] = (m_ref + __log2f(l_tot)) * kLn2;
}

template <int D, int NKG, bool CAUSAL>
__global__ __launch_bounds__(512, 2) void k_attn_f32_split(AttnArgs a) {
  attn_split_body<D, NKG, CAUSAL>(a, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.y);
}

template <int D, int NKG, bool CAUSAL>
hipError_t run_split(const AttnLaunch& l, hipStream_t s) {
  using C = SplitCfg<D, NKG>;
  AttnArgs a = make_args(l);
  const dim3 grid = attn_grid(&a, (l.rows + C::BQ - 1) / C::BQ);
  hipLaunchKernelGGL((k_attn_f32_split<D, NKG, CAUSAL>), grid, dim3(512), C::LDS_BYTES, s, a);
  return hipGetLastError();
}

template <int NKG>
hipError_t run_split_d(const AttnLaunch& l, hipStream_t s) {
  if (l.d == 128) return l.causal ? run_split<128, NKG, true>(l, s) : run_split<128, NKG, false>(l, s);
  return l.causal ? run_split<64, NKG, true>(l, s) : run_split<64, NKG, false>(l, s);
}

// Both attentions in one launch with the causal one on products of terms (NKG): the query attention's workgroups come first
// and take the shape, the chunks and the order that its own launch would (QKG = 0: float32 products, two units of 32 rows per
// workgroup), so the results are the same bits.  (Behind the causal ones they end last: 32 heads x 1540 rows and 32 tokens,
// with the merge, 112 us in front, 115 behind.)
template <int D, int NKG, int QKG>
__global__ __launch_bounds__(512, 2) void k_attn_f32_split_pair(AttnArgs ac, AttnArgs aq, PairGrid g) {
  const int bid = blockIdx.x;
  if (bid >= g.n_q_pad) {
    const int l = bid - g.n_q_pad;
    attn_split_body<D, NKG, true>(ac, l % g.c_gx, l / g.c_gx, 0, g.c_gy);
    return;
  }
  if (bid >= g.n_q) return;
  const int per_split = g.q_gx * g.q_gy;
  if constexpr (QKG > 0) {
    const int split = bid / per_split, l = bid - split * per_split;
    attn_split_body<D, QKG, false>(aq, l % g.q_gx, l / g.q_gx, split, g.q_gy);
  } else {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), set = wave >> 2;
    const int n = per_split * aq.n_split, u = 2 * bid + set, u_c = min(u, n - 1);
    const int split = u_c / per_split, l = u_c - split * per_split, bx = l % g.q_gx, by = l / g.q_gx;
    int kvh, batch, qt;
    map_block(aq, false, bx, by, g.q_gy, &kvh, &batch, &qt);
    const int kv_begin = split * aq.chunk, kg = (wave + (bx >> 3) + by) & (KG - 1);
    attn_f32_unit<D, false>(aq, kvh, batch, qt * 32, kv_begin, min(aq.m, kv_begin + aq.chunk), split, kg,
                            smem + set * F32Cfg<D>::LDS_BYTES, u < n);
  }
}

template <int D, int NKG, int QKG>
hipError_t run_split_pair(const AttnLaunch& c, const AttnLaunch& q, hipStream_t s) {
  using C = SplitCfg<D, NKG>;
  constexpr int BQ = QKG == 0 ? 32 : SplitCfg<D, QKG == 0 ? 1 : QKG>::BQ, LDS_Q = SplitCfg<D, QKG == 0 ? 1 : QKG>::LDS_BYTES;
  AttnArgs ac = make_args(c), aq = make_args(q);
  const dim3 gc = attn_grid(&ac, (c.rows + C::BQ - 1) / C::BQ), gq = attn_grid(&aq, (q.rows + BQ - 1) / BQ);
  long long n_q = (long long)gq.x * gq.y * gq.z;
  if (QKG == 0) n_q = (n_q + 1) / 2;
  const long long n_q_pad = (n_q + 7) / 8 * 8, n_c = (long long)gc.x * gc.y;
  if (n_q_pad + n_c > 0x7FFFFFFFll) return hipErrorInvalidValue;
  PairGrid g;
  g.n_q = (int)n_q; g.n_q_pad = (int)n_q_pad;
  g.q_gx = (int)gq.x; g.q_gy = (int)gq.y; g.c_gx = (int)gc.x; g.c_gy = (int)gc.y;
  constexpr int LDS = C::LDS_BYTES > LDS_Q ? C::LDS_BYTES : LDS_Q;
  hipLaunchKernelGGL((k_attn_f32_split_pair<D, NKG, QKG>), dim3((unsigned)(n_q_pad + n_c)), dim3(512), LDS, s, ac, aq, g);
  return hipGetLastError();
}

template <int D, int NKG>
hipError_t run_split_pair_q(const AttnLaunch& c, const AttnLaunch& q, AttnF32Shape qs, hipStream_t s) {
  switch (qs) {
    case AttnF32Shape::kPlain: return run_split_pair<D, NKG, 0>(c, q, s);
    case AttnF32Shape::kSplit: return run_split_pair<D, NKG, 1>(c, q, s);
    case AttnF32Shape::kSplitKeys2: return run_split_pair<D, NKG, 2>(c, q, s);
  }
  return hipErrorInvalidValue;
}

template <class F>
hipError_t raise(F* f, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <int D>
hipError_t raise_split() {
  constexpr int L1 = SplitCfg<D, 1>::LDS_BYTES, L2 = SplitCfg<D, 2>::LDS_BYTES, L = L1 > L2 ? L1 : L2;
  const hipError_t all[] = {
      raise(&k_attn_f32_split<D, 1, true>, L), raise(&k_attn_f32_split<D, 1, false>, L), raise(&k_attn_f32_split<D, 2, true>, L),
      raise(&k_attn_f32_split<D, 2, false>, L), raise(&k_attn_f32_split_pair<D, 1, 0>, L), raise(&k_attn_f32_split_pair<D, 1, 1>, L),
      raise(&k_attn_f32_split_pair<D, 1, 2>, L), raise(&k_attn_f32_split_pair<D, 2, 0>, L), raise(&k_attn_f32_split_pair<D, 2, 1>, L),
      raise(&k_attn_f32_split_pair<D, 2, 2>, L)};
  for (hipError_t e : all)
    if (e != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace

hipError_t attn_f32_raise_limits() {
  constexpr int L = F32Cfg<128>::LDS_BYTES;  // d = 64 stays below the default limit
  const hipError_t all[] = {raise(&k_attn_f32<128, true>, L), raise(&k_attn_f32<128, false>, L), raise(&k_attn_f32_pair<128>, L),
                            raise_split<128>(), raise_split<64>()};
  for (hipError_t e : all)
    if (e != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_attn_f32(const AttnLaunch& l, hipStream_t s) {
  const hipError_t e = attn_prepare_device();
  if (e != hipSuccess) return e;
  switch (attn_f32_shape(l.causal, l.n_batch, l.rows, l.m, l.d)) {
    case AttnF32Shape::kSplit: return run_split_d<1>(l, s);
    case AttnF32Shape::kSplitKeys2: return run_split_d<2>(l, s);
    case AttnF32Shape::kPlain: break;
  }
  if (l.d == 128) return l.causal ? run<128, true>(l, s) : run<128, false>(l, s);
  return l.causal ? run<64, true>(l, s) : run<64, false>(l, s);
}

hipError_t launch_attn_f32_pair(const AttnLaunch& causal, const AttnLaunch& query, hipStream_t s) {
  const hipError_t e = attn_prepare_device();
  if (e != hipSuccess) return e;
  const AttnF32Shape cs = attn_f32_shape(1, causal.n_batch, causal.rows, causal.m, causal.d);
  const AttnF32Shape qs = attn_f32_shape(0, query.n_batch, query.rows, query.m, query.d);
  if (cs == AttnF32Shape::kPlain) {
    if (qs != AttnF32Shape::kPlain) {  // few kept tokens, many query rows
      const hipError_t e2 = launch_attn_f32(causal, s);
      return e2 != hipSuccess ? e2 : launch_attn_f32(query, s);
    }
    return causal.d == 128 ? run_pair<128>(causal, query, s) : run_pair<64>(causal, query, s);
  }
  if (causal.d == 128)
    return cs == AttnF32Shape::kSplit ? run_split_pair_q<128, 1>(causal, query, qs, s) : run_split_pair_q<128, 2>(causal, query, qs, s);
  return cs == AttnF32Shape::kSplit ? run_split_pair_q<64, 1>(causal, query, qs, s) : run_split_pair_q<64, 2>(causal, query, qs, s);
}

}  // namespace samkv

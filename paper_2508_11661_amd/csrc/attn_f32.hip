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

// ---------------------------------------------------------------- products of bf16 terms
// The bf16 matrix instructions do sixteen times the work of the float32 ones.  A float32 number x is the sum of three bf16
// terms, x = x1 + x2 + x3 with x1 = bf16(x), x2 = bf16(x - x1), x3 = bf16(x - x1 - x2): each holds eight more bits and bf16 has
// float32's exponents, so the sum is x itself, whatever its neighbours are.  Of the nine products of two such numbers the six
// that can reach 2^-18 of x y are taken, small ones first and the largest in an accumulator of its own where scores are summed;
// the others, x2 y3, x3 y2 and x3 y3, are below 2^-25 of it together.  The sums are float32, with fewer roundings than the
// float32 instruction makes.  Weights and V are multiplied by 2^24 before they are split, so that the last bit of the smallest
// one is still a bf16 number; a term of K or Q that is too small for one moves a score by less than 2^-126 x 2^60 x d.
//   Against 64 bits the errors are below those of float32 products on the inputs tried (72 heads x 700 rows, error over the norm,
// float32 products / these: Gaussian 3.1e-7 / 1.7e-7; channels scaled apart 1.2e-6 / 4.7e-7; a key without V that takes all but
// e^-20 of the weight 2.6e-6 / 1.1e-6; a channel of V 2^-24 of the others, over its own norm, 4.4e-7 / 2.4e-7).  Two
// half-precision terms and three products took 0.6 of the time, but the absolute end of their range showed in the last two:
// 1.4e-3 and 1.9e-4.  An output that one key holds alone is a single product with its normalisation: 3.3e-8 / 5.3e-8, both
// below the unit of rounding.
//   The terms leave out infinities, NaN and magnitudes whose sums might pass float32's range, 2^60 in K and Q and 2^48 in V: the
// wave that meets one raises a flag, and the whole workgroup starts again with float32 products (attn_f32_unit).
//   Eight waves of 32 query rows.  NKG = 1: 256 rows, one stream of keys, 32 a step.  NKG = 2, for short problems: 128 rows,
// whose keys two groups of waves share, 64 a step; their results meet in LDS at the end.
//   Staging: K and V rows come as float32 into registers a step ahead and are turned into three planes of terms per tensor in
// LDS.  There is one buffer of each: V(t) is written between the products of the scores of step t, K(t + 1) between those of
// its outputs, a barrier behind each.  The third term of the query rows stays in LDS, which leaves the registers for the
// fragments.  Planes and fragments are laid out and read as in attn.hip.
//   What bounds it: the matrix unit and the device's power limit (1.2 PFLOP/s of bf16 products at M = 6850), for short problems
// the chain of steps.  32 heads over 8 KV heads, d = 128, float32 products -> these: M = 1540 176 -> 127 us, 4120 1080 -> 661, 6850
// 2913 -> 1870 (206 TFLOP/s); 24 heads, d = 64, M = 6450 1012 -> 733.
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int D, int NKG>
struct SplitCfg {
  static constexpr int NW = 8, RG = NW / NKG, BQ = 32 * RG;   // waves, row groups, rows per workgroup
  static constexpr int BK = 32, BKT = BK * NKG;               // keys per wave and per workgroup in a step
  static constexpr int ROWB = D * 2;                          // bytes of a row in a plane
  static constexpr int PLANE = BKT * ROWB;                    // three planes of K, then three of V
  static constexpr int VAT = 3 * PLANE, Q3 = 6 * PLANE;       // the query rows' third terms: [row group][fragment][lane]
  static constexpr int FLAGS = Q3 + RG * 32 * ROWB;           // [step parity] a step's numbers need float32 products
  // the query rows on their way to registers, eight of each wave: where its third terms will be, or V's first planes
  static constexpr int QTURN = NKG == 1 ? Q3 : VAT, QTURN_WAVE = NKG == 1 ? 32 * ROWB : 8 * D * 4;
  static constexpr int MERGE = 64 * (D / 2 + 2) * 4;          // one wave's outputs, maxima and sums
  static constexpr int TURN = (NKG == 1 ? 8 : 32) * (D * 4 + 16);
  static constexpr int END = NKG == 1 ? NW * TURN : RG * (MERGE > TURN ? MERGE : TURN);
  static constexpr int TILES = FLAGS + 16 > END ? FLAGS + 16 : END, PLAIN = 2 * F32Cfg<D>::LDS_BYTES;
  static constexpr int LDS_BYTES = TILES > PLAIN ? TILES : PLAIN;
  static_assert(QTURN_WAVE >= 8 * D * 4 && NW * QTURN_WAVE <= (NKG == 1 ? FLAGS - Q3 : Q3 - VAT), "room for the query rows");
  // staging: lanes per row, rows per load, rows and loads per wave
  static constexpr int LPR = D / 4, RPI = 64 / LPR, RW = BKT / NW, NI = RW / RPI;
  static __device__ __forceinline__ int kswz(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
  static __device__ __forceinline__ int vswz(int row) { return D == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }
};

// x0 and x1 as the sums of three bf16 terms each, a pair of terms per word
__device__ __forceinline__ void split3(float x0, float x1, uint32_t (&w)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const bf16x2 b = {(__bf16)x0, (__bf16)x1};
    w[i] = __builtin_bit_cast(uint32_t, b);
    asm("" : "+v"(w[i]));  // one packed conversion, whose halves the next lines read
    if (i < 2) {
      x0 -= bf16_lo(w[i]);
      x1 -= bf16_hi(w[i]);
    }
  }
}

constexpr float kTermsEnd = 0x1p60f, kTermsEndV = 0x1p48f, kTermScale = 0x1p24f;  // see above
constexpr int kHoldLds = 0x47F;  // LDS accesses may not be moved across such a scheduling barrier
__device__ __forceinline__ float abs_max(float m, const f32x4& x) {  // NaN wins
#pragma unroll
  for (int e = 0; e < 4; ++e) m = __builtin_elementwise_maximum(m, __builtin_fabsf(x[e]));
  return m;
}

// x, with what is computed from it computed anew: kept across steps, the addresses of all fragments would not fit the registers.
template <class T>
__device__ __forceinline__ T fresh(T x) {
  asm volatile("" : "+v"(x));
  return x;
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
  // (steps and rows past the last are read as that one; without a branch, which would wait for the loads to merge registers)
  const int last_row = a.m - 1 - kv_begin;
  auto load_rows = [&](const char* base, int j, f32x4 (&x)[NI]) {
    const int row = min(j, n_tiles - 1) * BKT + srow;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      x[i] = *reinterpret_cast<const f32x4*>(base + (uint32_t)(min(row + i * C::RPI, last_row) * (D * 4) + scol * 16));
  };
  // where the first of its numbers go; the swizzle of the others' rows enters by XOR, as their row bits are its own
  const uint32_t kst = (uint32_t)(srow * ROWB + (((scol >> 1) ^ C::kswz(srow)) * 16) + 8 * (scol & 1));
  const uint32_t vst = (uint32_t)(C::VAT + srow * ROWB + (((scol >> 1) ^ C::vswz(srow)) * 16) + 8 * (scol & 1));
  int* flags = reinterpret_cast<int*>(smem + C::FLAGS);
  // whether numbers are too large for the terms
  auto check = [&](const f32x4 (&x)[NI], float end) {
    float most = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) most = abs_max(most, x[i]);
    return !(most < end);
  };
  // converts and stores K or V in 2 NI pieces of two numbers
  uint32_t w0[3], w1[3];
  auto put = [&](const f32x4& x, float scale, bool second, char* at) {
    if (!second) {
      split3(x[0] * scale, x[1] * scale, w0);
    } else {
      split3(x[2] * scale, x[3] * scale, w1);
#pragma unroll
      for (int i = 0; i < 3; ++i) *reinterpret_cast<uint2*>(at + i * C::PLANE) = make_uint2(w0[i], w1[i]);
    }
  };
  auto put_k = [&](int pc) {
    const int n = pc / 2;
    put(rk[n], 1.f, pc % 2, smem + (fresh(kst) ^ (uint32_t)(C::kswz(n * C::RPI) * 16)) + n * C::RPI * ROWB);
  };
  auto put_v = [&](int pc) {
    const int n = pc / 2;
    put(rv[n], kTermScale, pc % 2, smem + (fresh(vst) ^ (uint32_t)(C::vswz(n * C::RPI) * 16)) + n * C::RPI * ROWB);
  };

  load_rows(kbase, 0, rk);
  if (t < 2) flags[t] = 0;

  // ---- query rows, requested behind the first keys, which are staged and followed by the next while they come
  bf16x8 q1[ND], q2[ND];
  char* q3 = smem + C::Q3 + rg * 32 * ROWB + lane * 16;
  bool q_odd;
  const float c2 = (float)((double)a.scale * 1.4426950408889634074);
  {
    // They come as whole rows and are turned through LDS (eight rows at a time, swizzled by the row): a load in the layout of
    // the fragments touches 32 lines, 16 of them per wave 4000 cycles ahead of the first tile.
    constexpr int NQ = 8 / C::RPI;
    f32x4 raw[4][NQ], x[ND][2];
    const int ql = lane / C::LPR, qc = lane % C::LPR;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int row = max(0, min(wave_first + 8 * p + i * C::RPI + ql, a.rows - 1));
        raw[p][i] = *reinterpret_cast<const f32x4*>(qbase + (size_t)row * (D * 4) + qc * 16);
      }
    __syncthreads();  // the flags are clear
    if (check(rk, kTermsEnd)) flags[1] = 1;
#pragma unroll
    for (int pc = 0; pc < 2 * NI; ++pc) put_k(pc);
    load_rows(vbase, 0, rv);  // (in the order of the steps, in which the waits for them count)
    load_rows(kbase, 1, rk);
    char* turn = smem + C::QTURN + wave * C::QTURN_WAVE;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int row = i * C::RPI + ql;
        *reinterpret_cast<f32x4*>(turn + row * (D * 4) + (qc ^ row) * 16) = raw[p][i];
      }
      __builtin_amdgcn_wave_barrier();
      if (rw / 8 == p) {
#pragma unroll
        for (int dc = 0; dc < ND; ++dc)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            x[dc][i] = *reinterpret_cast<const f32x4*>(turn + rw % 8 * (D * 4) + ((dc * 4 + h * 2 + i) ^ rw % 8) * 16);
      }
      __builtin_amdgcn_wave_barrier();
    }
    float most = 0.f;
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) {
      most = abs_max(abs_max(most, x[dc][0]), x[dc][1]);
      u32x4 term[3];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        split3(x[dc][i][0], x[dc][i][1], w0);
        split3(x[dc][i][2], x[dc][i][3], w1);
#pragma unroll
        for (int n = 0; n < 3; ++n) {
          term[n][2 * i] = w0[n];
          term[n][2 * i + 1] = w1[n];
        }
      }
      q1[dc] = __builtin_bit_cast(bf16x8, term[0]);
      q2[dc] = __builtin_bit_cast(bf16x8, term[1]);
      if (kg == 0) *reinterpret_cast<u32x4*>(q3 + dc * 1024) = term[2];  // (both key groups hold the same rows)
    }
    q_odd = !(most < kTermsEnd);
  }

  // ---- read side
  // (the chunk number's other bits enter by XOR: rows and planes are multiples of their size)
  uint32_t kaddr, vaddr;
  {
    kaddr = (uint32_t)((kg * BK + rw) * ROWB + ((h ^ C::kswz(rw)) * 16));
    const int i16 = lane & 15, q2 = (lane >> 4) & 1;
    const int vrow = 4 * h + (i16 >> 2), c = 2 * q2 + ((i16 & 3) >> 1);
    vaddr = (uint32_t)(C::VAT + (kg * BK + vrow) * ROWB + ((c ^ C::vswz(vrow)) * 16) + 8 * (i16 & 1));
  }

  f32x16 o[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[i][j] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;

  auto vfrag = [&](const char* vp) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vp + 8 * ROWB));
    union { struct { s16x4 lo, hi; } s; bf16x8 v; } u;
    u.s.lo = lo;
    u.s.hi = hi;
    return u.v;
  };

  f32x16 s;
  // the scores of a step, beside them V's planes
  auto scores = [&]() {
    f32x16 sl;
#pragma unroll
    for (int j = 0; j < 16; ++j) { s[j] = 0.f; sl[j] = 0.f; }
    constexpr int KA = 2;  // fragments in registers
    const uint32_t ka = fresh(kaddr);
    bf16x8 k1[KA], k2[KA], k3[KA];
    auto kread = [&](int dc) {
      const char* at = smem + (ka ^ (uint32_t)(dc * 32));
      k3[dc % KA] = *reinterpret_cast<const bf16x8*>(at + 2 * C::PLANE);
      k2[dc % KA] = *reinterpret_cast<const bf16x8*>(at + C::PLANE);
      k1[dc % KA] = *reinterpret_cast<const bf16x8*>(at);
    };
    kread(0);
#pragma unroll
    for (int dc = 0; dc < ND; ++dc) {
      const bf16x8 x3 = *reinterpret_cast<const bf16x8*>(q3 + dc * 1024);
      if (dc + 1 < ND) kread(dc + 1);
      __builtin_amdgcn_sched_barrier(kHoldLds);
#pragma unroll
      for (int pc = dc * 2 * NI / ND; pc < (dc + 1) * 2 * NI / ND; ++pc) put_v(pc);
      const int n = dc % KA;
      sl = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k3[n], q1[dc], sl, 0, 0, 0);
      sl = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k2[n], q2[dc], sl, 0, 0, 0);
      sl = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k2[n], q1[dc], sl, 0, 0, 0);
      sl = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1[n], q2[dc], sl, 0, 0, 0);
      sl = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1[n], x3, sl, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1[n], q1[dc], s, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) s[j] += sl[j];
  };
  auto weights = [&](int tile, bool masked) {
    if (masked) {
      const int n_ok = (CAUSAL ? min(kv_end, r + 1) : kv_end) - (kv_begin + tile * BKT + kg * BK) - 4 * h;
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (8 * (j >> 2) + (j & 3) >= n_ok) s[j] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int j = 1; j < 16; ++j) mx = fmaxf(mx, s[j]);
    mx = max_across_halves(mx) * c2;
    if (__any(mx > m_ref + TAU)) {
      const float m_new = fmaxf(m_ref, mx);
      const float al = __builtin_amdgcn_exp2f(m_ref - (m_new == -INFINITY ? 0.f : m_new));
      l_run *= al;
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[i][j] *= al;
      m_ref = m_new;
    }
    const float m_use = m_ref == -INFINITY ? 0.f : m_ref;
    float psum[4] = {0.f, 0.f, 0.f, 0.f};  // (a step's own sum, so that small weights beside a large one are not lost one by one)
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      s[j] = __builtin_amdgcn_exp2f(fmaf(s[j], c2, -m_use));
      psum[j & 3] += s[j];
      s[j] *= kTermScale;
    }
    l_run += (psum[0] + psum[1]) + (psum[2] + psum[3]);
  };
  // a step's share of the outputs, beside it K's next planes
  // OWN: its products, 12 to an output, are summed on their own and then added, so that the outputs are rounded once a step.
  // With two key groups the sums are half as long, and at d = 128 the registers are taken.
  constexpr bool OWN = NKG == 1 || D == 64;
  auto outputs = [&]() {
    bf16x8 p[2][3];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      u32x4 term[3];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t w[3];
        split3(s[8 * s2 + 2 * e], s[8 * s2 + 2 * e + 1], w);
#pragma unroll
        for (int n = 0; n < 3; ++n) term[n][e] = w[n];
      }
#pragma unroll
      for (int n = 0; n < 3; ++n) p[s2][n] = __builtin_bit_cast(bf16x8, term[n]);
    }
    constexpr int NG = 2 * NV;  // groups: 16 keys of 32 channels
    bf16x8 v[2][3];
    const uint32_t va = fresh(vaddr);
    auto vread = [&](int g) {
      const char* at = smem + (va ^ (uint32_t)(g / 2 * 64)) + g % 2 * 16 * ROWB;
#pragma unroll
      for (int n = 0; n < 3; ++n) v[g & 1][n] = vfrag(at + n * C::PLANE);
    };
    vread(0);
    f32x16 z;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (g + 1 < NG) vread(g + 1);
      __builtin_amdgcn_sched_barrier(kHoldLds);
#pragma unroll
      for (int pc = g * 2 * NI / NG; pc < (g + 1) * 2 * NI / NG; ++pc) put_k(pc);
      const bf16x8 (&x)[3] = v[g & 1];
      const bf16x8 (&w)[3] = p[g & 1];
      f32x16& y = OWN ? z : o[g / 2];
      if (OWN && g % 2 == 0) {
#pragma unroll
        for (int j = 0; j < 16; ++j) z[j] = 0.f;
      }
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[2], w[0], y, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], w[2], y, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], w[1], y, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], w[0], y, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], w[1], y, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], w[0], y, 0, 0, 0);
      if (OWN && g % 2 == 1) {
#pragma unroll
        for (int j = 0; j < 16; ++j) o[g / 2][j] += z[j];
        __builtin_amdgcn_sched_barrier(0);  // (begun side by side, these sums would not fit the registers)
      }
    }
  };

  if (q_odd) flags[1] = 1;
  __syncthreads();
  bool plain = false;
  for (int tile = 0; tile < n_tiles; ++tile) {
    // what step tile - 1 raised: its slot is written again in step tile + 1 only, behind barriers that follow this read
    if (flags[(tile + 1) & 1]) {
      plain = true;
      break;
    }
    const bool busy = tile < n_full || (tile == n_full && has_tail);
    if (check(rv, kTermsEndV)) flags[tile & 1] = 1;
    if (busy) {
      scores();
    } else {
#pragma unroll
      for (int pc = 0; pc < 2 * NI; ++pc) put_v(pc);
    }
    load_rows(vbase, tile + 1, rv);  // (one load for both cases: the wait for the other's would stand in either)
    if (busy) weights(tile, tile == n_full);
    __syncthreads();  // V(tile) is there, K(tile) has been read
    if (check(rk, kTermsEnd)) flags[tile & 1] = 1;
    if (busy) {
      outputs();
    } else {
#pragma unroll
      for (int pc = 0; pc < 2 * NI; ++pc) put_k(pc);
    }
    load_rows(kbase, tile + 2, rk);
    __syncthreads();  // K(tile + 1) is there, V(tile) has been read
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
  if (!has_rows) return;
  const float l_tot = sum_across_halves(l_run);
  const float inv = 1.f / (l_tot * (kTermScale * kTermScale));
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
// on half-precision terms, 112 us with the merge in front, 115 behind.)
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
  switch (l.f32) {
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
  const AttnF32Shape cs = causal.f32, qs = query.f32;
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

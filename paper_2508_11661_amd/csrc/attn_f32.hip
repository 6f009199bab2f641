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

template <int D, bool CAUSAL>
__device__ __forceinline__ void attn_f32_body(const AttnArgs a, int bx, int by, int bz, int grid_y) {
  using C = F32Cfg<D>;
  constexpr int NV = D / 32, NI = D / 8;  // 32-channel blocks of O^T; 16-byte chunks per lane and row
  constexpr int ROWB = D * 4, NKX = 8, NVX = 32;
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int lane = threadIdx.x & 63;
  // The first key group has the most tiles; which wave, and so which SIMD, that is goes round.
  const int kg = (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + (bx >> 3) + by) & (KG - 1);
  const int rw = lane & 31, h = lane >> 5;
  int kvh, batch, qt;
  map_block(a, CAUSAL, bx, by, grid_y, &kvh, &batch, &qt);
  const int q0 = qt * 32, r = q0 + rw;
  const int kv_begin = CAUSAL ? 0 : bz * a.chunk;
  const int kv_end = CAUSAL ? min(a.m, q0 + 32) : min(a.m, kv_begin + a.chunk);
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
    const char* qp = static_cast<const char*>(a.q) + ((size_t)batch * a.rows + min(r, a.rows - 1)) * ROWB + h * 16;
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
    if (q0 + row < a.rows) {
      *reinterpret_cast<f32x4*>(op + (size_t)row * D + c4 * 4) = acc;
      if (c4 == 0) lp[row] = (m_all + __log2f(den)) * kLn2;
    }
  }
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

template <class F>
hipError_t raise(F* f, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

}  // namespace

hipError_t attn_f32_raise_limits() {
  constexpr int L = F32Cfg<128>::LDS_BYTES;  // d = 64 stays below the default limit
  const hipError_t all[] = {raise(&k_attn_f32<128, true>, L), raise(&k_attn_f32<128, false>, L), raise(&k_attn_f32_pair<128>, L)};
  for (hipError_t e : all)
    if (e != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_attn_f32(const AttnLaunch& l, hipStream_t s) {
  const hipError_t e = attn_prepare_device();
  if (e != hipSuccess) return e;
  if (l.d == 128) return l.causal ? run<128, true>(l, s) : run<128, false>(l, s);
  return l.causal ? run<64, true>(l, s) : run<64, false>(l, s);
}

hipError_t launch_attn_f32_pair(const AttnLaunch& causal, const AttnLaunch& query, hipStream_t s) {
  const hipError_t e = attn_prepare_device();
  if (e != hipSuccess) return e;
  return causal.d == 128 ? run_pair<128>(causal, query, s) : run_pair<64>(causal, query, s);
}

}  // namespace samkv

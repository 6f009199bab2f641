// samkv_score_select: the inner products of a document's keys with its personalized query (Sec. 3.2) and the
// selection of the kept positions in ONE pass: a workgroup owns one (document, KV head) row, streams its K rows
// once, keeps the scores in LDS and selects from there.  The scores never travel to HBM and back (unless the caller
// asks for them), and the selection's barrier-bound passes of one workgroup overlap with the K streaming of its
// neighbours on the compute unit.  Both halves are the device functions the separate kernels use, so the kept
// positions are bit-identical to samkv_score followed by samkv_topk_select.
#include "common.hpp"
#include "kernels_core.hpp"

namespace samkv {
namespace {

// How a row is selected: EA > 0, up to 64 EA keys, by every wave for itself, without a barrier; or by all waves together.
constexpr int kByHistogram = 0, kByBits = -1;

// LDS of a row's scores, or of the histograms that take their place.
__host__ __device__ constexpr int select_lds(int E, int NT, int EA) {
  const int row = E * NT * (int)sizeof(float), hist = EA == kByHistogram && NT == 512 ? (int)sizeof(HistScratch<512>) : 0;
  return ((row > hist ? row : hist) + 15) / 16 * 16;
}

// GATHER: the workgroup also copies the row's kept K and V rows into the compacted cache (samkv_gather's job for this document
// and KV head), by the positions that the selection left in LDS (read back from memory: 320 rows of 400 keys 22.9 us, 21.6
// with the selection below; 40 rows of 2048 59.1 -> 58.6).
template <bool BF16, int D, int E, int NT, int EA, bool GATHER>
__global__ __launch_bounds__(NT) void k_score_select(PtrTable kt, PtrTable vt, IntTable cu_len, IntTable cu_k, const float* qsrc,
                                                     int heads, int group, int total_len, int m_total, int n_ctx, int n_sink,
                                                     int n_local, float* scores, int32_t* idx, int32_t* cu_k_dev, char* k_c,
                                                     char* v_c, uint32_t* v_max) {
  constexpr int EPL = BF16 ? 8 : 4;
  constexpr int LPR = D / EPL;
  constexpr int ROWS_PER_WAVE = (64 / LPR) * 8 * 2;
  constexpr int NW = NT / 64;
  static_assert(NW == kFusedWaves, "waves that write a v_max");
  constexpr size_t ROW_BYTES = (size_t)D * (BF16 ? 2 : 4);
  extern __shared__ __attribute__((aligned(16))) char smem[];
  float* s_sc = reinterpret_cast<float*>(smem);  // the row's scores, then the selection's histograms
  const int i = blockIdx.x, g = blockIdx.y, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (cu_k_dev != nullptr && i == 0 && g == 0)
    for (int n = t; n <= n_ctx; n += NT) cu_k_dev[n] = cu_k.v[n];
  const int L = cu_len.v[i + 1] - cu_len.v[i];
  const int k = cu_k.v[i + 1] - cu_k.v[i];
  const int sub = lane % LPR;

  float q[EPL];
  fold_query<EPL>(qsrc + ((size_t)i * heads + (size_t)g * group) * D + sub * EPL, D, group, q);
  const char* base = static_cast<const char*>(kt.p[i]) + (size_t)g * L * ROW_BYTES + sub * 16;
  for (int row0 = wave * ROWS_PER_WAVE; row0 < L; row0 += NW * ROWS_PER_WAVE)
    score_rows<BF16, D>(base, row0, L, q, [&](int row, float s) { s_sc[row] = s; });
  __syncthreads();
  if (scores != nullptr) {
    float* out = scores + (size_t)g * total_len + cu_len.v[i];
    for (int p = t; p < L; p += NT) out[p] = s_sc[p];
  }

  int32_t* ip = idx + (size_t)g * m_total + cu_k.v[i];
  uint16_t* s_pos = reinterpret_cast<uint16_t*>(smem + select_lds(E, NT, EA));  // the kept positions, for the compaction
  auto keep = [&](int place, int p) {
    ip[place] = p;
    if (GATHER) s_pos[place] = (uint16_t)p;
  };
  if constexpr (EA > 0) {
    // every wave finds the threshold for itself, from the whole row, and writes its share
    uint32_t key[EA];
#pragma unroll
    for (int e = 0; e < EA; ++e) {
      const int p = e * 64 + lane;
      key[e] = p >= L ? 0u : p < n_sink || p >= L - n_local ? 0xFFFFFFFFu : order_key(s_sc[p]);
    }
    emit_kept<EA>(key, L, threshold_in_wave<EA>(key, L, k), [&](int e) { return e % NW == wave; }, keep);
  } else {
    __shared__ uint2 wsum[NW];
    uint32_t key[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int p = key_position<E>(e);
      key[e] = p < L ? order_key(s_sc[p]) : 0u;
    }
    force_keys<E>(key, L, n_sink, n_local);
    if constexpr (EA == kByHistogram) {
      __syncthreads();  // every score has been read
      write_kept<E, NT>(key, L, threshold_by_histogram<E, NT>(key, L, k, *reinterpret_cast<HistScratch<NT>*>(s_sc)), keep, wsum);
    } else {
      __shared__ uint32_t cnt[2][NW];
      write_kept<E, NT>(key, L, threshold_by_bits<E, NT>(key, L, k, cnt), keep, wsum);
    }
  }

  if (GATHER) {
    __syncthreads();
    // LPR lanes copy one K row and one V row; U rows per thread in flight
    constexpr int RPP = NT / LPR, U = 4;
    const int rg = t / LPR;
    uint32_t mx = 0;
    const char* vsrc = static_cast<const char*>(vt.p[i]) + (size_t)g * L * ROW_BYTES + sub * 16;
    const size_t out0 = ((size_t)g * m_total + cu_k.v[i]) * ROW_BYTES + sub * 16;
    for (int r0 = rg; r0 < k; r0 += RPP * U) {
      u32x4 xk[U], xv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * RPP;
        int pos = s_pos[r < k ? r : k - 1];
        pos = pos < 0 ? 0 : (pos >= L ? L - 1 : pos);
        xk[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + (size_t)pos * ROW_BYTES));
        xv[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vsrc + (size_t)pos * ROW_BYTES));
      }
      if (BF16) {
#pragma unroll
        for (int u = 0; u < U; ++u) mx = bf16_max(mx, xv[u]);  // (rows past the last repeat it)
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * RPP;
        if (r < k) {
          __builtin_nontemporal_store(xk[u], reinterpret_cast<u32x4*>(k_c + out0 + (size_t)r * ROW_BYTES));
          __builtin_nontemporal_store(xv[u], reinterpret_cast<u32x4*>(v_c + out0 + (size_t)r * ROW_BYTES));
        }
      }
    }
    if (BF16 && v_max != nullptr) write_max(v_max + ((size_t)g * n_ctx + i) * NW + wave, mx);
  }
}

template <bool BF16, int D, int E, int NT, int EA>
hipError_t run(const ScoreLaunch& a, const SelectLaunch& sl, const QuerySrc& q, const PtrTable& k, const IntTable& cu_len,
               const IntTable& cu_k, const GatherLaunch* ga, const PtrTable* v, hipStream_t s) {
  size_t lds = select_lds(E, NT, EA);
  if (ga != nullptr) lds += (size_t)ga->max_k * sizeof(uint16_t);
  if (ga != nullptr)
    hipLaunchKernelGGL((k_score_select<BF16, D, E, NT, EA, true>), dim3(a.n_ctx, a.hkv), dim3(NT), lds, s, k, *v, cu_len, cu_k, q.q,
                       q.heads, q.group, a.total_len, sl.m_total, a.n_ctx, sl.n_sink, sl.n_local, a.scores, sl.idx,
                       sl.cu_k_dev, static_cast<char*>(ga->k_c), static_cast<char*>(ga->v_c), ga->v_max);
  else
    hipLaunchKernelGGL((k_score_select<BF16, D, E, NT, EA, false>), dim3(a.n_ctx, a.hkv), dim3(NT), lds, s, k, k, cu_len, cu_k, q.q,
                       q.heads, q.group, a.total_len, sl.m_total, a.n_ctx, sl.n_sink, sl.n_local, a.scores, sl.idx,
                       sl.cu_k_dev, nullptr, nullptr, nullptr);
  return hipGetLastError();
}

template <bool BF16, int D>
hipError_t run_len(const ScoreLaunch& a, const SelectLaunch& sl, const QuerySrc& q, const PtrTable& k,
                   const IntTable& cu_len, const IntTable& cu_k, const GatherLaunch* ga, const PtrTable* v, hipStream_t s) {
  // 512 threads a row (256 make twice the passes over its keys, 1024 lose it again in the selection's barriers).  Up to 512 keys
  // every wave holds the row and none waits for another (8 rows of 256 keys with their gather 13.3 -> 10.8 us, 160 of 400
  // 22.9 -> 21.6; 80 of 1024 the other way, 25.3 -> 26.5: 16 comparisons a bit are longer than a barrier).  Above 1024 keys the
  // threshold comes from histograms (320 rows of 2048 keys with their gather: 50 -> 47 us), at every number of rows: here a
  // row's neighbours on the compute unit stream their K meanwhile (1280 rows of 4000 keys 358 -> 361 us, of 2000 185 -> 183,
  // 20 rows of 8000 99 -> 75)
  if (a.max_len <= 256) return run<BF16, D, 2, 512, 4>(a, sl, q, k, cu_len, cu_k, ga, v, s);
  if (a.max_len <= 512) return run<BF16, D, 2, 512, 8>(a, sl, q, k, cu_len, cu_k, ga, v, s);
  if (a.max_len <= 1024) return run<BF16, D, 2, 512, kByBits>(a, sl, q, k, cu_len, cu_k, ga, v, s);
  if (a.max_len <= 2048) return run<BF16, D, 4, 512, kByHistogram>(a, sl, q, k, cu_len, cu_k, ga, v, s);
  if (a.max_len <= 4096) return run<BF16, D, 8, 512, kByHistogram>(a, sl, q, k, cu_len, cu_k, ga, v, s);
  return run<BF16, D, 16, 512, kByHistogram>(a, sl, q, k, cu_len, cu_k, ga, v, s);
}

}  // namespace

hipError_t launch_score_select(const ScoreLaunch& a, const SelectLaunch& sl, const PtrTable& k, const IntTable& cu_len,
                               const IntTable& cu_k, hipStream_t s, const GatherLaunch* ga, const PtrTable* v) {
  if (a.max_len > kFusedMaxLen) {  // rows too long for LDS: the separate kernels, through the caller's score buffer
    if (a.scores == nullptr) return hipErrorInvalidValue;
    hipError_t e = launch_score(a, k, cu_len, s);
    if (e == hipSuccess) e = launch_select(sl, cu_len, cu_k, s);
    if (e == hipSuccess && ga != nullptr) e = launch_gather(*ga, k, *v, cu_len, cu_k, s);
    return e;
  }
  QuerySrc q;
  hipError_t e = launch_score_prologue(a, s, &q);
  if (e != hipSuccess) return e;
  const GatherLaunch* in_kernel = score_select_gathers(a.n_ctx, a.hkv, a.max_len) ? ga : nullptr;
  if (a.dtype == SAMKV_BF16)
    e = a.d == 128 ? run_len<true, 128>(a, sl, q, k, cu_len, cu_k, in_kernel, v, s)
                   : run_len<true, 64>(a, sl, q, k, cu_len, cu_k, in_kernel, v, s);
  else
    e = a.d == 128 ? run_len<false, 128>(a, sl, q, k, cu_len, cu_k, in_kernel, v, s)
                   : run_len<false, 64>(a, sl, q, k, cu_len, cu_k, in_kernel, v, s);
  if (e == hipSuccess && ga != nullptr && in_kernel == nullptr) e = launch_gather(*ga, k, *v, cu_len, cu_k, s);
  return e;
}

}  // namespace samkv

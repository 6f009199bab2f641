// samkv_topk_select: per (document, KV head) row of scores, the positions of the k largest scores
// (Sec. 3.2 with a fixed budget), initial/local positions forced in, output ascending by position.
//
// One workgroup per row, or one wave; the whole row lives in registers (E keys per thread).
//   1. keys: float -> order-preserving uint32; forced positions get the largest key.
//   2. the k-th largest key, by one bit per pass (ballot + popcount: no atomics, so no contention on the few exponent
//      values real scores share) or, for long rows, by 11-bit histograms in LDS.
//   3. kept = key > T, plus the first `need` positions with key == T (ties to the lower position); ballots give every
//      thread its output offset.
#include "common.hpp"
#include "kernels_core.hpp"

namespace samkv {
namespace {

template <int E, int NT, bool HIST>
__global__ __launch_bounds__(NT) void k_select(const float* scores, IntTable cu_len, IntTable cu_k, int total_len,
                                               int m_total, int n_ctx, int n_sink, int n_local, int32_t* idx,
                                               int32_t* cu_k_dev) {
  __shared__ uint2 wsum[NT / 64];
  const int i = blockIdx.x, g = blockIdx.y, t = threadIdx.x;
  if (cu_k_dev != nullptr && i == 0 && g == 0)
    for (int n = t; n <= n_ctx; n += NT) cu_k_dev[n] = cu_k.v[n];
  const int L = cu_len.v[i + 1] - cu_len.v[i];
  const int k = cu_k.v[i + 1] - cu_k.v[i];
  const float* row = scores + (size_t)g * total_len + cu_len.v[i];
  int32_t* out = idx + (size_t)g * m_total + cu_k.v[i];

  uint32_t key[E];
  constexpr int U = E < 16 ? E : 16;  // requests in flight per thread
#pragma unroll
  for (int e0 = 0; e0 < E; e0 += U) {
    float x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = row[min(key_position<E>(e0 + u), L - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) key[e0 + u] = key_position<E>(e0 + u) < L ? order_key(x[u]) : 0u;
    __builtin_amdgcn_sched_barrier(0);
  }
  force_keys<E>(key, L, n_sink, n_local);
  auto keep = [&](int place, int p) { out[place] = p; };
  if constexpr (HIST) {
    __shared__ HistScratch<NT> sc;
    write_kept<E, NT>(key, L, threshold_by_histogram<E, NT>(key, L, k, sc), keep, wsum);
  } else {
    __shared__ uint32_t cnt[2][NT / 64];
    write_kept<E, NT>(key, L, threshold_by_bits<E, NT>(key, L, k, cnt), keep, wsum);
  }
}

// One wave per row of up to 64 E scores.
template <int E>
__global__ __launch_bounds__(64) void k_select_wave(const float* scores, IntTable cu_len, IntTable cu_k, int total_len, int m_total,
                                                    int n_ctx, int n_sink, int n_local, int32_t* idx, int32_t* cu_k_dev) {
  const int i = blockIdx.x, g = blockIdx.y, t = threadIdx.x;
  if (cu_k_dev != nullptr && i == 0 && g == 0)
    for (int n = t; n <= n_ctx; n += 64) cu_k_dev[n] = cu_k.v[n];
  const int L = cu_len.v[i + 1] - cu_len.v[i], k = cu_k.v[i + 1] - cu_k.v[i];
  const float* row = scores + (size_t)g * total_len + cu_len.v[i];
  int32_t* out = idx + (size_t)g * m_total + cu_k.v[i];
  float x[E];
  uint32_t key[E];
#pragma unroll
  for (int e = 0; e < E; ++e) x[e] = row[min(e * 64 + t, L - 1)];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int p = e * 64 + t;
    key[e] = p >= L ? 0u : p < n_sink || p >= L - n_local ? 0xFFFFFFFFu : order_key(x[e]);
  }
  emit_kept<E>(key, L, threshold_in_wave<E>(key, L, k), [](int) { return true; }, [&](int place, int p) { out[place] = p; });
}

template <int E>
hipError_t run_wave(const SelectLaunch& a, const IntTable& cu_len, const IntTable& cu_k, hipStream_t s) {
  hipLaunchKernelGGL(k_select_wave<E>, dim3(a.n_ctx, a.hkv), dim3(64), 0, s, a.scores, cu_len, cu_k, a.total_len, a.m_total,
                     a.n_ctx, a.n_sink, a.n_local, a.idx, a.cu_k_dev);
  return hipGetLastError();
}

template <int E, int NT, bool HIST>
hipError_t run(const SelectLaunch& a, const IntTable& cu_len, const IntTable& cu_k, hipStream_t s) {
  hipLaunchKernelGGL((k_select<E, NT, HIST>), dim3(a.n_ctx, a.hkv), dim3(NT), 0, s, a.scores, cu_len, cu_k, a.total_len,
                     a.m_total, a.n_ctx, a.n_sink, a.n_local, a.idx, a.cu_k_dev);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_select(const SelectLaunch& a, const IntTable& cu_len, const IntTable& cu_k, hipStream_t s) {
  // Up to 512 keys one wave per row, without barriers (8 rows of 256 keys 6.3 -> 3.9 us, 160 of 400 7.0 -> 5.6, 8192 of 300 31
  // -> 12.7; 80 of 1024, whose bit passes take 16 comparisons each, 7.4 -> 9.2).
  // Bit passes for rows of up to 1024 keys: few keys per thread, and four waves keep the barrier rounds short.  Up to
  // 4096 keys the histograms shorten a row (bits / histograms: 40 rows of 1500 keys 8.0 / 6.7 us, 640 of 4096 17.9 /
  // 16.3), but ask for twice the threads, an LDS pass to clear them and, where many scores are equal, atomics on one
  // address.  Bits win where enough rows share a compute unit to hide their barriers: from one row per compute unit on up
  // to 2048 keys (320 rows of 1500 9.6 / 10.4, 2560 of 2048 23.3 / 32.0), from three on up to 4096 (1280 rows of 4096
  // 22.9 / 23.9; all scores equal, 2560 of 4096 51 / 65).  Beyond, histograms at every number of rows measured (40 to
  // 5120): 40 rows of 24000 keys 97 -> 22 us, half of it from loading whole lines.
  const long long rows = (long long)a.n_ctx * a.hkv;
  if (a.max_len <= 128) return run_wave<2>(a, cu_len, cu_k, s);
  if (a.max_len <= 256) return run_wave<4>(a, cu_len, cu_k, s);
  if (a.max_len <= 512) return run_wave<8>(a, cu_len, cu_k, s);
  if (a.max_len <= 1024) return run<4, 256, false>(a, cu_len, cu_k, s);
  if (a.max_len <= 2048) return rows < 256 ? run<4, 512, true>(a, cu_len, cu_k, s) : run<8, 256, false>(a, cu_len, cu_k, s);
  if (a.max_len <= 4096) return rows < 768 ? run<8, 512, true>(a, cu_len, cu_k, s) : run<16, 256, false>(a, cu_len, cu_k, s);
  if (a.max_len <= 8192) return run<16, 512, true>(a, cu_len, cu_k, s);
  if (a.max_len <= 16384) return run<16, 1024, true>(a, cu_len, cu_k, s);
  if (a.max_len <= 32768) return run<32, 1024, true>(a, cu_len, cu_k, s);
  return run<64, 1024, true>(a, cu_len, cu_k, s);
}

}  // namespace samkv

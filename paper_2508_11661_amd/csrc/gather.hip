// samkv_gather: copy the kept K and V rows of every document into one compacted cache (Sec. 3.2:
// the filtered blocks of all documents are concatenated, in document order and original position
// order).  Pure data movement, HBM-bound: 2*d*e bytes read and 2*d*e written per kept token and KV
// head, plus the 4-byte index.
//
// A row is LPR 16-byte chunks; LPR lanes copy one K row and one V row, a wave copies 64/LPR rows per
// step and runs STEPS steps with all of its loads issued before the first store.  The grid is
// (row chunk, document, KV head), so the document's base pointers are uniform over a workgroup.
#include "common.hpp"
#include "kernels_core.hpp"

namespace samkv {
namespace {

// Steps per wave: 64 rows of 256 bytes per workgroup at four, 128 at eight.  The copies are short and each begins with
// a chain of two loads, so four steps, with twice the workgroups, are the rule (eight / four: K and V of 20 documents x
// 8 KV heads, 340 kept rows each, 18.3 / 16.0 us; stored Q rows of 32 heads 25.0 / 23.7 us; 5120 rows' K and V 292 /
// 282 us).  Two exceptions.
//   Where a document's rows fit eight steps and not four, its second workgroup repeats that chain for the few rows left
//   over, which shows once the chip is full of workgroups (eight to four, rows that fill 55 and 75 % of eight steps:
//   256 (document, head) pairs 0.91 to 0.96, 512 0.65 to 0.90, 1024 to 6400 0.71 to 0.93; 128 pairs 0.96 to 1.07).
//   Rows that fill 97 % have nothing left over (1.0 to 1.16, but for the second exception), hence the bound of 7/8 on
//   the average.
//   Where eight steps make two workgroups for every compute unit, evenly long, half as many chains do the same work in
//   one go (512 workgroups, rows that fill 75 to 98 %, one to eight workgroups per document, 0.69 to 0.93; 480 0.91 to
//   1.06; 384 and 640, 94 % and more, 0.95 to 1.22).
constexpr int kStepsFew = 4, kStepsMany = 8;
template <int ROW_BYTES>
int gather_steps(const GatherLaunch& a, const IntTable& cu_k, int heads) {
  constexpr int rows = (64 / (ROW_BYTES / 16)) * kStepsMany * 4;  // of a workgroup
  const int per_doc = (a.max_k + rows - 1) / rows;
  const long long wgs = (long long)per_doc * a.n_ctx * heads;
  if (a.max_k > rows / 2 && per_doc == 1 && 8ll * a.m_total <= 7ll * rows * a.n_ctx) return wgs >= 256 ? kStepsMany : kStepsFew;
  bool even = wgs > 448 && wgs <= 512 && a.max_k > rows / 2;
  for (int i = 0; even && i < a.n_ctx; ++i) even = cu_k.v[i + 1] - cu_k.v[i] > (per_doc - 1) * rows + rows / 2;
  return even ? kStepsMany : kStepsFew;
}

// Where a document's words of the largest V magnitudes start, in workgroups of `rows` rows: room for its workgroups that hold
// rows, and for at most one more, from the prefix sums alone (floor(a / rows) + ceil(n / rows) <= floor((a + n) / rows) + 1).  A
// word per workgroup of the grid would grow with the longest document times the number of documents, and every workgroup of
// launch_v_prep reads a head's words (128 documents, one of 6000 kept rows, the others of 16, 32 heads, whole path: 48128
// words a head 831 us, 1004 words 776, without them 780).
__host__ __device__ __forceinline__ int v_max_begin(const IntTable& cu_k, int i, int rows) { return cu_k.v[i] / rows + i; }

template <int ROW_BYTES, int STEPS>
__global__ __launch_bounds__(256) void k_gather(PtrTable kt, PtrTable vt, IntTable cu_len, IntTable cu_k, int m_total,
                                                const int32_t* idx, char* k_c, char* v_c, uint32_t* v_max) {
  constexpr int LPR = ROW_BYTES / 16;
  constexpr int RPS = 64 / LPR;  // rows per wave step
  constexpr int ROWS_PER_BLOCK = RPS * STEPS * 4;
  const int i = blockIdx.y, g = blockIdx.z;  // document and KV head are uniform over the block
  const int k_i = cu_k.v[i + 1] - cu_k.v[i];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPR, rg = lane / LPR;
  const int r0 = blockIdx.x * ROWS_PER_BLOCK + wave * (RPS * STEPS);
  const int block0 = blockIdx.x * ROWS_PER_BLOCK;
  if (block0 >= k_i && blockIdx.x > 0) return;
  uint32_t* mx_at = nullptr;
  if (v_max != nullptr) {
    const int first = v_max_begin(cu_k, i, ROWS_PER_BLOCK), next = v_max_begin(cu_k, i + 1, ROWS_PER_BLOCK);
    mx_at = v_max + ((size_t)g * v_max_begin(cu_k, gridDim.y, ROWS_PER_BLOCK) + first + blockIdx.x) * 4 + wave;
    // the document's last workgroup clears the room that none has
    if (block0 + ROWS_PER_BLOCK >= k_i && first + (int)blockIdx.x + 1 < next && lane == 0) mx_at[4] = 0;
  }
  if (r0 >= k_i) {
    if (mx_at != nullptr && lane == 0) *mx_at = 0;
    return;
  }
  const int L = cu_len.v[i + 1] - cu_len.v[i];
  const char* ksrc = static_cast<const char*>(kt.p[i]) + (size_t)g * L * ROW_BYTES + sub * 16;
  const char* vsrc = static_cast<const char*>(vt.p[i]) + (size_t)g * L * ROW_BYTES + sub * 16;
  const size_t out0 = ((size_t)g * m_total + cu_k.v[i]) * ROW_BYTES + sub * 16;
  const int32_t* ip = idx + (size_t)g * m_total + cu_k.v[i];

  int p[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int r = r0 + s * RPS + rg;
    p[s] = ip[r < k_i ? r : k_i - 1];
  }
  u32x4 xk[STEPS], xv[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int q = p[s] < 0 ? 0 : (p[s] >= L ? L - 1 : p[s]);
    xk[s] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ksrc + (size_t)q * ROW_BYTES));
    xv[s] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vsrc + (size_t)q * ROW_BYTES));
  }
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int r = r0 + s * RPS + rg;
    if (r < k_i) {
      __builtin_nontemporal_store(xk[s], reinterpret_cast<u32x4*>(k_c + out0 + (size_t)r * ROW_BYTES));
      __builtin_nontemporal_store(xv[s], reinterpret_cast<u32x4*>(v_c + out0 + (size_t)r * ROW_BYTES));
    }
  }
  if (mx_at != nullptr) {  // (rows past the last repeat it)
    uint32_t mx = 0;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) mx = bf16_max(mx, xv[s]);
    write_max(mx_at, mx);
  }
}

// Q-cache variant: one tensor, one row set per QUERY head h, indexed by the kept positions of its KV head
// h / group (the stored per-document Q cache supplies the query states of the kept tokens).
template <int ROW_BYTES, int STEPS>
__global__ __launch_bounds__(256) void k_gather_q(PtrTable qt, IntTable cu_len, IntTable cu_k, int m_total, int group,
                                                  const int32_t* idx, char* q_rec) {
  constexpr int LPR = ROW_BYTES / 16;
  constexpr int RPS = 64 / LPR;
  constexpr int ROWS_PER_BLOCK = RPS * STEPS * 4;
  const int i = blockIdx.y, h = blockIdx.z, g = h / group;
  const int k_i = cu_k.v[i + 1] - cu_k.v[i];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPR, rg = lane / LPR;
  const int r0 = blockIdx.x * ROWS_PER_BLOCK + wave * (RPS * STEPS);
  if (r0 >= k_i) return;
  const int L = cu_len.v[i + 1] - cu_len.v[i];
  const char* src = static_cast<const char*>(qt.p[i]) + (size_t)h * L * ROW_BYTES + sub * 16;
  const size_t out0 = ((size_t)h * m_total + cu_k.v[i]) * ROW_BYTES + sub * 16;
  const int32_t* ip = idx + (size_t)g * m_total + cu_k.v[i];
  int p[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int r = r0 + s * RPS + rg;
    p[s] = ip[r < k_i ? r : k_i - 1];
  }
  u32x4 x[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int q = p[s] < 0 ? 0 : (p[s] >= L ? L - 1 : p[s]);
    x[s] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + (size_t)q * ROW_BYTES));
  }
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int r = r0 + s * RPS + rg;
    if (r < k_i) __builtin_nontemporal_store(x[s], reinterpret_cast<u32x4*>(q_rec + out0 + (size_t)r * ROW_BYTES));
  }
}

// Gather by GLOBAL token positions (position in the concatenation of all documents): used after the cross-document
// block filter, where the number of tokens a document contributes differs from KV head to KV head.  One or two
// tensors per document ([heads][L_i][d] each); head h reads the positions of KV head h / group.  The document of a
// row is found by binary search in the prefix sums, staged in LDS together with the base pointers.
template <int ROW_BYTES, bool TWO>
__global__ __launch_bounds__(256) void k_gather_g(PtrTable at, PtrTable bt, IntTable cu_len, int n_ctx, int m_total,
                                                  int group, const int32_t* gidx, char* a_out, char* b_out) {
  constexpr int LPR = ROW_BYTES / 16;
  constexpr int RPS = 64 / LPR;
  constexpr int STEPS = 4;
  __shared__ int s_cu[SAMKV_MAX_CTX + 1];
  __shared__ const char* s_a[SAMKV_MAX_CTX];
  __shared__ const char* s_b[SAMKV_MAX_CTX];
  for (int n = threadIdx.x; n <= n_ctx; n += 256) s_cu[n] = cu_len.v[n];
  for (int n = threadIdx.x; n < n_ctx; n += 256) {
    s_a[n] = static_cast<const char*>(at.p[n]);
    if (TWO) s_b[n] = static_cast<const char*>(bt.p[n]);
  }
  __syncthreads();
  const int h = blockIdx.y, g = h / group;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPR, rg = lane / LPR;
  const int r0 = blockIdx.x * (RPS * STEPS * 4) + wave * (RPS * STEPS);
  if (r0 >= m_total) return;
  const int total_len = s_cu[n_ctx];
  const int32_t* ip = gidx + (size_t)g * m_total;
  const char* pa[STEPS];
  const char* pb[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int r = r0 + s * RPS + rg;
    int gp = ip[r < m_total ? r : m_total - 1];
    gp = gp < 0 ? 0 : (gp >= total_len ? total_len - 1 : gp);
    int lo = 0, hi = n_ctx;  // document with cu_len[doc] <= gp < cu_len[doc + 1]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_cu[mid] <= gp) lo = mid; else hi = mid;
    }
    const size_t L = s_cu[lo + 1] - s_cu[lo];
    const size_t off = ((size_t)h * L + (gp - s_cu[lo])) * ROW_BYTES + sub * 16;
    pa[s] = s_a[lo] + off;
    if (TWO) pb[s] = s_b[lo] + off;
  }
  u32x4 xa[STEPS], xb[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    xa[s] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(pa[s]));
    if (TWO) xb[s] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(pb[s]));
  }
  const size_t out0 = (size_t)h * m_total * ROW_BYTES + sub * 16;
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int r = r0 + s * RPS + rg;
    if (r < m_total) {
      __builtin_nontemporal_store(xa[s], reinterpret_cast<u32x4*>(a_out + out0 + (size_t)r * ROW_BYTES));
      if (TWO) __builtin_nontemporal_store(xb[s], reinterpret_cast<u32x4*>(b_out + out0 + (size_t)r * ROW_BYTES));
    }
  }
}

template <int ROW_BYTES>
hipError_t run_g(const PtrTable& a, const PtrTable* b, const IntTable& cu_len, int n_ctx, int heads, int group, int m_total,
                 const int32_t* gidx, void* a_out, void* b_out, hipStream_t s) {
  constexpr int ROWS_PER_BLOCK = (64 / (ROW_BYTES / 16)) * 4 * 4;
  dim3 grid((m_total + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK, heads);
  if (b != nullptr)
    hipLaunchKernelGGL((k_gather_g<ROW_BYTES, true>), grid, dim3(256), 0, s, a, *b, cu_len, n_ctx, m_total, group, gidx,
                       static_cast<char*>(a_out), static_cast<char*>(b_out));
  else
    hipLaunchKernelGGL((k_gather_g<ROW_BYTES, false>), grid, dim3(256), 0, s, a, a, cu_len, n_ctx, m_total, group, gidx,
                       static_cast<char*>(a_out), static_cast<char*>(nullptr));
  return hipGetLastError();
}

template <int ROW_BYTES>
dim3 gather_grid(const GatherLaunch& a, int steps, int heads) {
  const int rows = (64 / (ROW_BYTES / 16)) * steps * 4;
  return dim3((a.max_k + rows - 1) / rows, a.n_ctx, heads);
}

template <int ROW_BYTES>
hipError_t run_q(const GatherLaunch& a, const PtrTable& q, const IntTable& cu_len, const IntTable& cu_k, int hq,
                 hipStream_t s) {
  const int steps = gather_steps<ROW_BYTES>(a, cu_k, hq);
  auto kernel = steps == kStepsMany ? k_gather_q<ROW_BYTES, kStepsMany> : k_gather_q<ROW_BYTES, kStepsFew>;
  hipLaunchKernelGGL(kernel, gather_grid<ROW_BYTES>(a, steps, hq), dim3(256), 0, s, q, cu_len, cu_k, a.m_total, hq / a.hkv,
                     a.idx, static_cast<char*>(a.k_c));
  return hipGetLastError();
}

template <int ROW_BYTES>
hipError_t run(const GatherLaunch& a, const PtrTable& k, const PtrTable& v, const IntTable& cu_len,
               const IntTable& cu_k, hipStream_t s) {
  const int steps = gather_steps<ROW_BYTES>(a, cu_k, a.hkv);
  auto kernel = steps == kStepsMany ? k_gather<ROW_BYTES, kStepsMany> : k_gather<ROW_BYTES, kStepsFew>;
  hipLaunchKernelGGL(kernel, gather_grid<ROW_BYTES>(a, steps, a.hkv), dim3(256), 0, s, k, v, cu_len, cu_k, a.m_total, a.idx,
                     static_cast<char*>(a.k_c), static_cast<char*>(a.v_c), a.v_max);
  return hipGetLastError();
}

}  // namespace

int gather_v_parts(const GatherLaunch& a, const IntTable& cu_k, bool fused) {
  if (fused) return a.n_ctx * kFusedWaves;
  const int rows = a.row_bytes == 128 ? 32 * gather_steps<128>(a, cu_k, a.hkv) : 16 * gather_steps<256>(a, cu_k, a.hkv);
  return v_max_begin(cu_k, a.n_ctx, rows) * 4;
}

hipError_t launch_gather(const GatherLaunch& a, const PtrTable& k, const PtrTable& v, const IntTable& cu_len,
                         const IntTable& cu_k, hipStream_t s) {
  switch (a.row_bytes) {
    case 128: return run<128>(a, k, v, cu_len, cu_k, s);
    case 256: return run<256>(a, k, v, cu_len, cu_k, s);
    case 512: return run<512>(a, k, v, cu_len, cu_k, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gather_g(int row_bytes, const PtrTable& a, const PtrTable* b, const IntTable& cu_len, int n_ctx, int heads,
                           int group, int m_total, const int32_t* gidx, void* a_out, void* b_out, hipStream_t s) {
  switch (row_bytes) {
    case 128: return run_g<128>(a, b, cu_len, n_ctx, heads, group, m_total, gidx, a_out, b_out, s);
    case 256: return run_g<256>(a, b, cu_len, n_ctx, heads, group, m_total, gidx, a_out, b_out, s);
    case 512: return run_g<512>(a, b, cu_len, n_ctx, heads, group, m_total, gidx, a_out, b_out, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gather_q(const GatherLaunch& a, const PtrTable& q, const IntTable& cu_len, const IntTable& cu_k,
                           int hq, hipStream_t s) {
  switch (a.row_bytes) {
    case 128: return run_q<128>(a, q, cu_len, cu_k, hq, s);
    case 256: return run_q<256>(a, q, cu_len, cu_k, hq, s);
    case 512: return run_q<512>(a, q, cu_len, cu_k, hq, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace samkv

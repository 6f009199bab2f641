// Shared declarations of the SamKV HIP library (gfx950 only): kernel-argument tables, small device
// helpers and the host-side launch entry points that samkv_api.hip calls.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/samkv.h"

namespace samkv {

// Per-document pointers and prefix sums travel to the kernels by value in the kernel-argument
// segment (no device allocation, no host-to-device copy, nothing for a later call to race with).
struct PtrTable {
  const void* p[SAMKV_MAX_CTX];
};
struct IntTable {
  int32_t v[SAMKV_MAX_CTX + 1];
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// ---- host-side launchers (one per translation unit) -------------------------------------------
struct ScoreLaunch {
  int n_ctx, hq, hkv, d, dtype, n_q_tok, w_loc, max_len, total_len;
  const void* q_tok;
  const void* q_loc;  // may be null
  float* scores;
  float* ws_que;    // [Hq][d]
  float* ws_loc;    // [N][Hq][d]
  float* ws_w;      // [N][Hq]
  float* ws_base;   // [Hq][d]  sum over all documents of |cos| * Q_loc
  float* ws_qt;     // [N][Hkv][d]
};
hipError_t launch_score(const ScoreLaunch& a, const PtrTable& k, const IntTable& cu_len, hipStream_t s);
// Where the per-document vectors of Eq. 1 are after the prologue: [N][heads][d] float32, of which `group`
// consecutive heads are averaged into the vector of one KV head.
struct QuerySrc {
  const float* q;
  int heads, group;
};
hipError_t launch_score_prologue(const ScoreLaunch& a, hipStream_t s, QuerySrc* q);

struct SelectLaunch {
  int n_ctx, hkv, max_len, total_len, m_total, n_sink, n_local;
  const float* scores;
  int32_t* idx;
  int32_t* cu_k_dev;  // may be null
};
hipError_t launch_select(const SelectLaunch& a, const IntTable& cu_len, const IntTable& cu_k, hipStream_t s);

constexpr int kFusedMaxLen = 8192;
constexpr int kFusedWaves = 8;  // of a workgroup of launch_score_select
constexpr int kFusedGatherMaxRows = 2048;  // (document, KV head) rows up to which the fused call also compacts in-kernel

// whether launch_score_select compacts in its own kernel: with thousands of rows (many layers stacked as heads) the streaming
// kernel is faster (0.84 against 0.91 ms at 5120 rows); below that the row's workgroup does it and a launch is saved
inline bool score_select_gathers(int n_ctx, int hkv, int max_len) {
  return max_len <= kFusedMaxLen && (long long)n_ctx * hkv <= kFusedGatherMaxRows;
}

hipError_t launch_block_scores(const float* scores, const IntTable& cu_len, const IntTable& cu_blk, int n_ctx, int hkv,
                               int total_len, int block, float* bscores, hipStream_t s);
hipError_t launch_expand_blocks(const int32_t* bidx, const IntTable& cu_len, const IntTable& cu_kb, const IntTable& cu_k,
                                int n_ctx, int hkv, int block, int32_t* idx, int32_t* cu_k_dev, hipStream_t s);

hipError_t launch_gather_g(int row_bytes, const PtrTable& a, const PtrTable* b, const IntTable& cu_len, int n_ctx, int heads,
                           int group, int m_total, const int32_t* gidx, void* a_out, void* b_out, hipStream_t s);
hipError_t launch_normalize(const float* bscores, const int32_t* bidx, const IntTable& cu_blk, const IntTable& cu_kb,
                            int n_ctx, int hkv, int n_init, int n_local, float* cand, hipStream_t s);
hipError_t launch_filter_expand(const int32_t* sel, const int32_t* bidx, const IntTable& cu_len, const IntTable& cu_kb,
                                int n_ctx, int hkv, int n_sel, int m_total, int block, int32_t* gidx, hipStream_t s);

hipError_t launch_peak_mfma(float* sink, int n_blocks, int iters, int pattern, hipStream_t s);
hipError_t launch_peak_copy(const void* src, void* dst, size_t bytes, hipStream_t s);
hipError_t launch_peak_read(const void* src, size_t bytes, uint32_t* sink, hipStream_t s);

struct GatherLaunch {
  int n_ctx, hkv, row_bytes, m_total, max_k;
  const int32_t* idx;
  void* k_c;
  void* v_c;
  uint32_t* v_max;  // null, or [Hkv][gather_v_parts]: the largest magnitudes of the bf16 V rows that its waves copy, for launch_v_prep
};
// Words of v_max per KV head, by the kernel of launch_gather, or by launch_score_select's own (fused).  At most one per 16 kept
// rows and eight per document.
int gather_v_parts(const GatherLaunch& a, const IntTable& cu_k, bool fused);
hipError_t launch_gather(const GatherLaunch& a, const PtrTable& k, const PtrTable& v, const IntTable& cu_len,
                         const IntTable& cu_k, hipStream_t s);
// Score and selection in one pass over K (rows of at most kFusedMaxLen tokens): a.scores may be null.  With `ga`
// and `v` the same workgroups also compact the kept K and V rows (what launch_gather does).
hipError_t launch_score_select(const ScoreLaunch& a, const SelectLaunch& sl, const PtrTable& k, const IntTable& cu_len,
                               const IntTable& cu_k, hipStream_t s, const GatherLaunch* ga = nullptr,
                               const PtrTable* v = nullptr);
// Q-cache variant: a.k_c receives [Hq][M][d]; q holds per-document [Hq][L_i][d]
hipError_t launch_gather_q(const GatherLaunch& a, const PtrTable& q, const IntTable& cu_len, const IntTable& cu_k,
                           int hq, hipStream_t s);

// Which bf16 attention kernel serves a problem: kDma, asynchronous loads, 256 rows per workgroup (eight waves, one key
// stream for all of them); kDmaKeys2, the same with 128 rows, whose keys two groups of waves share, and kDmaKeys2One, at
// d = 64, its form of one workgroup per compute unit with the score pipeline; kStaged, four waves, 128 rows, register-staged
// loads, two workgroups per compute unit.  All figures: device time of pair calls in us.
// Few rows are start and end of workgroups rather than steps, and most waves of an eight-wave workgroup hold no row: kStaged
// up to 320 rows (kDma / kDmaKeys2 / kStaged: 32 heads x 40 rows 11.1 / 12.0 / 10.1, x 140 15.3 / 14.8 / 13.9, x 300 19.9 /
// 16.8 / 16.9, x 330 21.1 / 17.1 / 18.5; 256 heads x 40 16.9 / 18.3 / 12.3, x 128 22.9 / 23.5 / 17.9; d = 64, 32 heads x 300
// 16.2 / 13.9 / 13.2, x 460 19.7 / 15.5 / 16.1), and further up the more workgroups there are: a third to half of its second
// resident set at 384 and 544 rows, most of it at 640 (96 heads over 12, 512 rows 28.2 / 29.1 / 26.5; 128 over 32, 600 rows
// 44.2 / 41.0 / 38.2; 128 x 520, d = 64, 31.0 / 34.6 / 27.6), where d = 64 wants more of them unless every head reads a K and
// V of its own (128 over 32 x 640: 30.3 / 27.0 / 28.6, 160 over 32 x 640: 33.1 / 30.6 / 29.3).
// Two key groups halve the chain of steps of the longest row tile and make twice as many workgroups, but read each tile for
// half as many rows.  d = 128: up to 512 workgroups of 128 rows (32 heads x 2000 rows 66.2 / 61.2 / 64.2), from 320 of 256
// rows on kDma (64 heads x 1200 47.8 / 54.4 / 52.9, 32 x 2600 82.6 / 84.7 / 86.1), between them kStaged for short rows (96 over
// 12 x 768 40.0 / 42.7 / 36.0) and kDmaKeys2 for long ones (24 x 3000 89.2 / 81.2 / 87.9).
// d = 64: up to 1024 workgroups of 256 rows (24 heads x 6450 174 / 163, 32 x 9000 378 / 382), 384 where no two heads share K
// and V and the head count is no multiple of 8, so that an XCD's L2 does not keep a head's tiles for its second reader (127 x
// 1540 99.1 / 110.9 / 105.7); in the form of one per compute unit while they, and one row tile of query tokens per KV head,
// nearly fit the chip once (kDmaKeys2 -> kDmaKeys2One: 32 heads x 700 18.0 -> 17.0, x 1200 24.7 -> 22.6, x 2000 37.1 -> 39.0;
// 64 heads with their own K and V x 400 18.1 -> 21.6).
// Over 1066 shapes (7 to 512 heads, 330 to 3500 rows) this is 0.9 % from the best of the four on average.
// Not causal: kStaged (V as stored, two-term weights) below 512 rows per KV head, and beyond as long as preparing V would
// cost more than the doubled second product (kStaged / kDma with its preparation, whole calls: 8 KV heads, d = 128, 800 rows
// x 1500 keys 28.6 / 31.2, x 3000 33.8 / 35.6, x 7000 61.1 / 48.8; d = 64, 1024 rows x 3000 26.3 / 32.8, x 7000 39.6 / 40.5, x
// 12000 56.2 / 51.5; 2 KV heads, d = 128, 512 rows x 20000 33.7 / 39.0), at d = 64 somewhat longer where there are workgroups
// enough without chunks (32 KV heads, 2400 rows x 800 38.8 / 48.9; 16, 800 rows x 4500 45.3 / 40.5).
enum class AttnShape { kDma, kDmaKeys2, kDmaKeys2One, kStaged };
inline AttnShape attn_bf16_shape(int causal, int n_batch, int batch_per_kv, int rows, int m, int d) {
  const long long wg256 = (long long)n_batch * ((rows + 255) / 256), wg128 = (long long)n_batch * ((rows + 127) / 128);
  if (!causal) {
    const long long most = d == 128 ? 3000000000ll : wg128 >= 512 ? 4000000000ll : 3400000000ll;
    return rows < 512 || (long long)rows * m * n_batch * d <= most ? AttnShape::kStaged : AttnShape::kDma;
  }
  const int n_kv = n_batch / batch_per_kv;
  if (rows <= 320 || (rows <= 384 && wg128 > 224) || (rows <= 544 && wg128 > 352)) return AttnShape::kStaged;
  if (rows <= 640 && wg128 > 448 && (d == 128 || batch_per_kv == 1 || wg128 >= 800)) return AttnShape::kStaged;
  if (d == 128) {
    if (wg128 <= 512) return AttnShape::kDmaKeys2;
    if (wg256 >= 320) return AttnShape::kDma;
    return rows <= 1536 ? AttnShape::kStaged : AttnShape::kDmaKeys2;
  }
  if (wg128 + 2 * n_kv <= 368) return AttnShape::kDmaKeys2One;
  return wg256 >= (batch_per_kv == 1 && n_kv % 8 != 0 ? 384 : 1024) ? AttnShape::kDma : AttnShape::kDmaKeys2;
}

// Which float32 attention kernel serves a problem: kPlain, float32 products, 32 rows and four groups of keys per workgroup, two
// workgroups per compute unit; kSplit and kSplitKeys2, products of bf16 terms, 256 rows or 128 rows whose keys two groups of
// waves share, one workgroup per compute unit.  Fitted to device times of single calls of all three over 329 causal shapes (1 to
// 512 heads, 64 to 9000 rows) and 997 others (1 to 128 KV heads, 16 to 2048 rows, 150 to 60000 keys): on average 0.4 % and 0.3 %
// behind the best of the three, by more than 5 % on 12 and 15 shapes; against kPlain throughout 21 and 17 % faster, and slower by
// more than 2 % on 1 and 14.  Examples in us, kPlain / kSplit / kSplitKeys2.
// Causal: kPlain has four times the workgroups and a shorter start, so it stays ahead until its workgroups fill the chip, the
// later the more steps the longest row tile takes (d = 128: 8 heads x 3300 rows 226 / 424 / 241, x 6000 599 / 759 / 460; 32 x 700
// 58 / 95 / 59, x 1540 192 / 212 / 137; 64 x 300 32 / 46 / 32, x 400 52 / 59 / 40; d = 64: 16 x 2000 90 / 158 / 93, x 2600 135 /
// 208 / 125; 64 x 400 25 / 35 / 24, x 700 59 / 60 / 39).  kSplit once three rounds of its workgroups exist (d = 128: 64 x 1200
// 228 / 179 / 162, x 2600 917 / 593 / 594, x 4100 2145 / 1316 / 1392; d = 64: 64 x 4100 1139 / 741 / 795), and where heads of one
// row tile fill the chip (d = 128: 200 x 200 48 / 38 / 44).
// Not causal: the same by work, as the keys are cut into chunks; up to 64 rows per KV head, and 256 in all, keep kPlain, whose
// workgroups hold no more (rows x keys x KV heads, d = 128: 32 x 4000 x 128 112 / 175 / 149, 96 x 60000 x 1 47 / 93 / 81, 160 x
// 4000 x 8 40 / 49 / 35), and so do, for longer, problems whose row tiles of 32 fill the chip once without chunks (d = 128: 2048 x
// 300 x 8 36 / 56 / 40; d = 64: 19 / 33 / 24).  kSplit for long ones or where it fills the chip (d = 128: 1024 x 4000 x 16 289 /
// 185 / 187; d = 64: 800 x 1500 x 32 111 / 78 / 84).
enum class AttnF32Shape { kPlain, kSplit, kSplitKeys2 };
inline AttnF32Shape attn_f32_shape(int causal, int n_batch, int rows, int m, int d) {
  const long long wg32 = (long long)n_batch * ((rows + 31) / 32), wg256 = (long long)n_batch * ((rows + 255) / 256);
  if (rows <= 64) return AttnF32Shape::kPlain;
  if (causal) {
    if (wg32 <= (d == 128 ? 500 + (m < 1050 ? m / 3 : 350) : 560 + (m < 1200 ? m / 2 : 600))) return AttnF32Shape::kPlain;
    if (wg256 >= 780 || (rows > 100 && rows <= 256 && n_batch > 128)) return AttnF32Shape::kSplit;
    return AttnF32Shape::kSplitKeys2;
  }
  const long long work = (long long)rows * m * n_batch;
  const bool once = wg32 > 400 && wg32 <= 512;
  if ((long long)n_batch * rows <= 256 || work <= (d == 128 ? (once ? 5000000 : 3500000) : once ? 6000000 : 4500000))
    return AttnF32Shape::kPlain;
  if (rows > 128 && (wg256 >= 160 || (m >= 3000 && work >= 40000000))) return AttnF32Shape::kSplit;
  return AttnF32Shape::kSplitKeys2;
}

// Whether the attention of query tokens over a cache AND their n_self own keys runs as one launch of the short kernel, the
// own keys being one more part beside the key chunks: no copy of V for the cache or for the own values, one merge.
// Problems of 512 rows per KV head and more pay for that with the doubled second product once they are large: one launch
// against preparation, two attentions and merge, 8 KV heads: d = 128, 512 rows x 3000 keys 31 against 53 us, x 20000
// 78 / 99, 1600 rows of 200 tokens x 7000 95 / 109, 1024 of 128 x 25000 178 / 160; d = 64, 2048 of 256 x 4000 45 / 61,
// x 25000 198 / 163.  One workgroup per row tile walks the own keys, without chunks, so they count three times (the rule
// that came closest to the faster side over 600 shapes, within 2.5 % of the slower one where it misses): 8192 rows of 1024
// tokens x 500 keys, d = 64, 66 / 66, d = 128 104 / 88.  Beyond 1024 own keys that chain is longer than what it saves: 8
// heads x 4096 tokens, d = 64, x 1500 keys 113 / 97, 6000 rows of 1500 tokens x 100 58 / 55.
inline bool attn_self_in_kernel(int dtype, int n_kv, int rows, int m, int n_self, int d) {
  if (dtype != SAMKV_BF16) return false;
  if (rows < 512) return true;
  return n_self <= 1024 && (long long)rows * (m + 3ll * n_self) * n_kv * d <= (d == 128 ? 22000000000ll : 12000000000ll);
}

// One attention problem: `n_batch` independent row blocks, batch b reads KV head b / batch_per_kv.
// Row r of a batch attends keys [0, r] (causal) or [0, m) (not causal).
struct AttnLaunch {
  int dtype, d, causal;
  int n_batch, batch_per_kv, rows, m;
  const void* q;   // [n_batch][rows][d]
  const void* k;   // [n_batch / batch_per_kv][m][d]
  const void* v;   // bf16 kernels that read the copy (attn_bf16_reads_v16): what launch_v_prep wrote; otherwise V itself
  const float* v_unscale;  // with the copy: [n_batch / batch_per_kv] factors that undo its power-of-two scale; else null
  float* out;      // [n_batch][rows][d]
  float* lse;      // [n_batch][rows]
  float scale;
  AttnF32Shape f32;    // the kernel of a float32 problem
  int n_split, chunk;  // keys are cut into n_split chunks of `chunk` keys (not causal only)
  float* part_o;       // [n_split][n_batch][rows][d]   workspace when n_split > 1
  float* part_lse;     // [n_split][n_batch][rows]
  // attn_self_in_kernel problems only: the last of the n_split parts is the query tokens' own keys, of which row r of a
  // batch (query head r / n_self, token r % n_self) sees the first r % n_self + 1
  int n_self;
  const void* k_self;  // [n_batch][n_self][d]
  const void* v_self;
};
hipError_t launch_attn_bf16(const AttnLaunch& a, hipStream_t s);
// Whether the bf16 kernel that serves this problem reads the scaled half-precision copy of V (every causal problem, long
// problems that are not causal) or V as stored (short problems that are not causal).  A pair launch always reads the copy.
bool attn_bf16_reads_v16(const AttnLaunch& a);
// Both bf16 attentions of the path in one launch: `causal` and `query` share d, K and the prepared V; the query
// attention runs without key chunks whatever `query` says (its n_split, chunk and partial buffers are ignored).
hipError_t launch_attn_bf16_pair(const AttnLaunch& causal, const AttnLaunch& query, hipStream_t s);
hipError_t launch_attn_f32(const AttnLaunch& a, hipStream_t s);
// Both float32 attentions in one launch (the query attention's key chunks as in its own launch; the merge, where there
// is one, stays a launch of its own).
hipError_t launch_attn_f32_pair(const AttnLaunch& causal, const AttnLaunch& query, hipStream_t s);
hipError_t attn_f32_raise_limits();  // part of attn_prepare_device
constexpr int kMaxParts = 64;  // partial results that one merge takes: key chunks and, for query_attn_self, the own keys
hipError_t launch_attn_merge(const AttnLaunch& a, hipStream_t s);

// Half-precision copy of a bf16 V tensor [n_kv][m][d] for the attention kernels, one power-of-two scale per KV head.
// part: [n_kv][v_prep_chunks(n_kv, m)] scratch words; unscale: [n_kv] factors that undo the scale.
int v_prep_chunks(int n_kv, int m);
// v_max: null, or [n_kv][n_v_max] bf16 magnitudes (bit patterns) whose largest is the head's.
hipError_t launch_v_prep(const void* v, int n_kv, int m, int d, bool causal, void* v16, uint32_t* part, float* unscale,
                         const uint32_t* v_max, int n_v_max, hipStream_t s);

// Raises the dynamic-LDS limit of every attention kernel variant that needs it on the current device (once per device).
hipError_t attn_prepare_device();

// Cache update after recomputation: rows of `cur` (old, updated in place) against rows of `fresh` (new).
struct UpdateLaunch {
  int dtype, d, fusion;
  long long n_rows;   // per tensor (K and V each have n_rows rows of d elements)
  void* k_cur; void* v_cur;
  const void* k_new; const void* v_new;
};
hipError_t launch_kv_update(const UpdateLaunch& a, hipStream_t s);

}  // namespace samkv

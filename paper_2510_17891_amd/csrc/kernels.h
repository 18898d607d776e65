// Launchers of the gfx950 kernels.  Host orchestration (model.hip) calls these; each enqueues on the
// given stream and returns.  Shapes are validated by the caller against what each kernel assumes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_plan.h"
#include "gemm_plan.h"
#include "weight_order.h"

namespace rl {

// Records the message that rl_last_error() returns on this thread and hands back `status` (an rl_status value), so
// that every entry point, whichever source file it lives in, reports failures the same way.
int set_error(int status, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

// One batch row = one (sequence, position) pair being pushed through the decoder.
struct RowMeta {
  int32_t seq;   // sequence id (row of the block table, RNG stream)
  int32_t pos;   // absolute position of the token fed in this row
  int32_t page;  // KV page that holds position pos (what the append and, at a page's first position, the block table need)
  int32_t pad;
};

enum Dtype : int { kF32 = 0, kBF16 = 1 };

// Geometry of the decoder, fixed at init and passed by value to launchers.
struct Geometry {
  int n_layers, hidden, n_q, n_kv, head_dim, ffn, vocab;
  int qk_norm;
  float rms_eps;
  int dtype;
  int max_blocks;   // block-table row length = max_ctx / 16
  int64_t n_pages;  // pages in the pool
  int kv_fp8;       // bf16 models: keys and values are cached as fp8 (e4m3), one byte per element
};

// "Fragment-major" order of a [rows x K] bf16 operand of the MFMA GEMM: 32-row blocks, 64-wide k
// blocks, inside a block [t(4)][hb(2)][row(32)][e(8)] with k = 64 kb + 32 hb + 8 t + e.  A wave reads
// block (rb, kb) as four fully coalesced 1 KiB loads, each already in MFMA 32x32x16 operand order.
__host__ __device__ inline size_t frag_offset(int r, int k, int k_blocks) {
  int rb = r >> 5, row = r & 31, kb = k >> 6, hb = (k >> 5) & 1, t = (k >> 3) & 3, e = k & 7;
  return ((((size_t)(rb * (size_t)k_blocks + kb) * 4 + t) * 2 + hb) * 32 + row) * 8 + e;
}

// Offset of weight element (r, k) in the packed matrix: frag_offset with the k block moved to its slot.
__host__ __device__ inline size_t weight_offset(int r, int k, int k_blocks, int seg) {
  const int kb = k >> 6;
  return frag_offset(r, (weight_kb_slot(kb, seg) << 6) | (k & 63), k_blocks);
}

// ---- elementwise / small kernels (both dtypes) -------------------------------------------------
// What the first kernel of a call moves from the pinned slot of the call to its slot in the workspace, in units of 16
// bytes: the rows from the start of the slot, then up to kSlotRegions more regions.  block_table (may be null): rows at the
// first position of a page are entered there.
constexpr int kSlotRegions = 5;
struct SlotUpload {
  const uint4* src = nullptr;  // host memory, read by the kernel: may be rewritten once the kernel has finished
  uint4* dst = nullptr;
  int n_rows = 0;
  int at[kSlotRegions] = {}, n[kSlotRegions] = {};
  int32_t* block_table = nullptr;
  int max_blocks = 0;
};
// Where the rows of a call come from.  from_table: row r is src[token] (model dtype, V rows of H; ids are clamped to
// [0, V)) with token = tokens[r], or, with tokens == null, last_tok[rows[r].seq] (what the sampler recorded for that
// sequence).  Otherwise src is fp32 [M][H].
struct RowSource {
  const void* src = nullptr;
  int from_table = 0;
  const int32_t* tokens = nullptr;
  const int32_t* last_tok = nullptr;
  const RowMeta* rows = nullptr;  // in host memory: the slot's
  int V = 0;
};
// First kernel of a call: moves the metadata slot, x = the rows of the call, and in bf16 models capture (may be null) = x
// and h_out = the normalised rows.
void launch_entry(hipStream_t s, int dtype, const RowSource& in, const SlotUpload& up, float* x, const void* gain, void* h_out,
                  float* capture, int M, int H, float eps);

// bf16 models: x_out[r] = x_in[r] + sum_{s<S} part[s][r][:] (x_out may be x_in and is not written when S == 0; part may
// then be null);  capture (may be null) gets that row;  if gain != null, h = row * rsqrt(mean(row^2)+eps) * gain written
// as f16 fragment-major.  x_in, x_out 16-byte aligned.
// group > 1: the M rows are the rows r / group of x_in and part (which then hold M / group rows); x_out is another buffer.
void launch_residual_norm(hipStream_t s, const float* x_in, float* x_out, const float* part, int S, const void* gain,
                          void* h_out, float* capture, int M, int H, float eps, int group = 1);

// For the n pairs (row, slot): x_out[slot] = x[row] (H floats), q_out[slot] = q[row] (D floats).
void launch_put_aside(hipStream_t s, const int32_t* pairs, int n, const float* x, float* x_out, int H, const float* q, float* q_out, int D);
// out[r] = in[r / group], M rows of H floats.
void launch_repeat_rows(hipStream_t s, const float* in, float* out, int M, int H, int group);

// Sum the split partials of the QKV projection, apply per-head RMSNorm (q,k) and the rotation (q,k) at
// each row's position, write q as fp32 [M][n_q][d] and append k,v to the row's KV page (rows[r].page).
void launch_qk_rope_append(hipStream_t s, const Geometry& g, const float* qkv_part, int S, const void* q_gain,
                           const void* k_gain, const float2* rope_table, const RowMeta* rows, void* k_pool_layer,
                           void* v_pool_layer, float* q_out, int M);

// Scatter contiguous [n_tokens][n_kv][d] K and V (model dtype) into the pages of one sequence, as its positions
// first_pos .. first_pos + n_tokens - 1 (the block-table row must already name their pages).
void launch_kv_import(hipStream_t s, const Geometry& g, const void* k_src, const void* v_src, int first_pos, int n_tokens,
                      const int32_t* block_table_row, void* k_pool_layer, void* v_pool_layer);

// Sequences that continue others: the first `full` block-table entries of dst become those of src, and with page >= 0 the
// source's next page (partly filled) is copied, in all layers, into `page`, which becomes dst's next entry.  Pool byte
// layout [layer][page][page_bytes].  The descriptors travel as kernel arguments.
constexpr int kForkBatch = 128;
struct ForkBatch {
  struct One { int32_t src, dst, full, page; } f[kForkBatch];
  int n;
};
void launch_fork(hipStream_t s, const ForkBatch& batch, int32_t* block_table, int max_blocks, void* kv_pool, size_t layer_bytes,
                 size_t page_bytes, int n_layers);

// ---- attention -----------------------------------------------------------------------------------
// bf16, head_dim 128: decode attention over paged KV (MFMA), one block per (row, kv head), context cut into
// segments that depend on the context length only and merged in index order; writes f16 fragment-major
// [M x n_q*d].  part: fp32, per (row, head) max_segs rows of d floats followed by max_segs (max, sum) pairs, with
// max_segs = attn_bf16_max_segments(max_ctx).
int attn_bf16_max_segments(int max_ctx);
// skip_segs (per row, may be null): leading segments of the row that a set in `shared` covers; every row with a
// non-zero entry must belong to exactly one set with that n_segs.  max_shared_segs = largest n_segs.
// append (may be null): the kernel forms the rows' queries, new keys and new values from the QKV projection's split
// sums itself and writes the keys and values into the pages (RowMeta::page); `q` is then unused and
// launch_qk_rope_append is not called.  Only for batches with one row per sequence: the block of a row is then the
// only one that needs the row's new key, and it takes it from registers, not from the page.  The arithmetic is the
// one of launch_qk_rope_append, bit for bit.
// window_sets: every row is in a set, and every set in `shared` covers all segments of its rows.
// packs: some entries of `shared` are packs of single segments;  all_packed: they cover all that the sets leave of every row.
// segs_per_block (1..16): segments one block takes of a context of more than 16 segments (> 4096 keys); results do
// not depend on it.
constexpr int kAttnAppendMaxSplits = 4;
struct AttnAppend {
  const float* qkv_part;  // [S][M][(n_q + 2 n_kv) * d]
  int S;                  // <= kAttnAppendMaxSplits
  const void* q_gain;     // per-head RMSNorm gains: both set, or both null
  const void* k_gain;
  const float2* rope_table;
};
// Returns true when the partials of some rows were left in the workspace, i.e. launch_attn_merge_bf16 (same arguments)
// has to follow; the two launches are separate calls so that a caller can time them separately.
bool launch_attn_decode_bf16(hipStream_t s, const Geometry& g, const float* q, const RowMeta* rows,
                             const int32_t* block_table, void* k_pool_layer, void* v_pool_layer,
                             float* part, int max_segs_alloc, int max_ctx_in_batch, void* o_out, int M,
                             const int32_t* skip_segs = nullptr, const AttnShared* shared = nullptr, int n_shared = 0,
                             int max_shared_segs = 0, const AttnAppend* append = nullptr, int segs_per_block = 16,
                             int set_segs = 4, bool window_sets = false, bool packs = false, bool all_packed = false);
void launch_attn_merge_bf16(hipStream_t s, const Geometry& g, const RowMeta* rows, float* part, int max_segs_alloc, int max_ctx_in_batch,
                            void* o_out, int M, const int32_t* skip_segs, int n_shared);
// fp32, even head_dim <= 128: one block per (row, q head), whole context, output fp32 row-major [M][n_q*d].  append (may
// be null; S == 1): as for the bf16 attention, only for batches with one row per sequence.
void launch_attn_f32(hipStream_t s, const Geometry& g, const float* q, const RowMeta* rows,
                     const int32_t* block_table, void* k_pool_layer, void* v_pool_layer,
                     float* o_out, int M, const AttnAppend* append = nullptr);

// ---- projections ---------------------------------------------------------------------------------

// Arguments of the sampling epilogue of the output projection (ignored by the other epilogues).
struct SampleEpilogue {
  const RowMeta* rows = nullptr;  // RNG stream (seq) and position (pos + pos_offset) per row
  int pos_offset = 0;
  float inv_t = 1.f;
  int greedy = 1;
  uint32_t seed_lo = 0, seed_hi = 0;
  const int32_t* forced = nullptr;  // per row, or null
  float* forced_z = nullptr;        // [M] logit of the forced token
  float* part = nullptr;            // [M][N/64][8] per-tile partials for launch_sample_merge
  float* logits_out = nullptr;      // optional [M][N] copy of the logits
};

// Number of K splits the bf16 GEMM uses for (N, K); partial outputs are [S][M][N] fp32.
int gemm_bf16_splits(int N, int K, int epi);
// Partial outputs that a kEpiPartial launch of M rows leaves: the splits, or 1 where the kernel adds them up itself.
int gemm_bf16_partials(int M, int N, int K);
// Whether a product of M rows can be added to the residual stream by the projection itself (kEpiResidual).
bool gemm_bf16_adds_residual(int M, int N, int K);
// Gate/up with the residual sums and the norm before it, for a row or two: x + S split sums [S][M][H], normalised, times W, SwiGLU; x stays as it is.
bool norm_gate_up_takes(int M, int H, int S);
void launch_norm_gate_up(hipStream_t s, const float* x, const float* part, int S, const void* gain, float eps, const void* W, void* out,
                         int M, int F, int H);
// MFMA GEMM of the bf16 models: X f16 fragment-major [M x K], W bf16 fragment-major [N x K] (2N rows for SwiGLU: gate
// and up rows interleaved in groups of 16).
// kEpiPartial: out = fp32 [gemm_bf16_partials(M, N, K)][M][N];  kEpiResidual (only where gemm_bf16_adds_residual): out =
// fp32 [M][N], to which the product's split sums are added in split order;  kEpiSwiGLU: out = f16 fragment-major [M x N] = silu(gate)*up;
// kEpiSample: out unused, results go through *se.  allow_split = false forces S = 1 (finished [M][N] product).
void launch_gemm_bf16(hipStream_t s, const void* X, const void* W, void* out, int M, int N, int K, int epi,
                      bool allow_split = true, const SampleEpilogue* se = nullptr);
// fp32 GEMM on vector ALUs, row-major everything, K even; kEpiPartial writes [M][N] (one split), kEpiResidual adds to
// it.  gain (may be null; not used with kEpiResidual): K gains; the rows of X are RMS-normalised with them first.
void launch_gemm_f32(hipStream_t s, const float* X, const float* W, float* out, int M, int N, int K, int epi,
                     const float* gain = nullptr, float eps = 0.f);

// Row-major [N x K] bf16 -> fragment-major with the k blocks in weight_kb_slot order for segments of `seg` k blocks
// (N % 32 == 0, K % 64 == 0, (K / 64) % (4 seg) == 0).
void launch_pack_weight_bf16(hipStream_t s, const void* src, void* dst, int N, int K, int seg);
// Segment length (k blocks per wave) of the plan that launch_gemm_bf16 uses for an [N x K] weight matrix: split_k says
// whether the product may be split along K over several blocks (QKV, O, down) or never is (gate/up, output projection).
int gemm_bf16_weight_segment(int N, int K, bool split_k);

// ---- sampler ---------------------------------------------------------------------------------------
constexpr int kSampleTile = 2048;  // vocabulary entries per first-stage block of the stand-alone sampler
// Gumbel-max sampling with log-probabilities from fp32 logits [M][V] in memory (two stages).
// part: [M][ceil(V/2048)][8] floats; forced may be null; forced_z: [M] floats.
// The RNG position of row r is rows[r].pos + pos_offset.
// top_k / top_p cut the distribution first (0 / outside (0,1): no cut; ignored when greedy); cut_buf: scratch of
// M * sample_cut_bytes_per_row() bytes (256-byte aligned), needed when sample_is_truncated().  V % 4 == 0, V < 2^22.
size_t sample_cut_bytes_per_row();
inline bool sample_is_truncated(int V, int top_k, float top_p) {
  return (top_k > 0 && top_k < V) || (top_p > 0.0f && top_p < 1.0f);
}
void launch_sample(hipStream_t s, const float* logits, int M, int V, const RowMeta* rows, int pos_offset,
                   const int32_t* forced, float temperature, uint64_t seed, float* part, float* forced_z,
                   int32_t* out_tokens, float* out_logprobs, int top_k = 0, float top_p = 0.f, void* cut_buf = nullptr,
                   int32_t* last_tok = nullptr);
// Second stage alone, over the [M][n_tiles][8] partials the sampling epilogue of the bf16 projection left.
// last_tok (may be null): [max_seqs] table that also receives each row's token at index rows[r].seq (both samplers).
void launch_sample_merge(hipStream_t s, const float* part, int n_tiles, int M, int V, const int32_t* forced,
                         const float* forced_z, float temperature, int32_t* out_tokens, float* out_logprobs,
                         const RowMeta* rows = nullptr, int32_t* last_tok = nullptr);

// out[idx[i]] = src[i] for idx[i] >= 0.
void launch_scatter_f32(hipStream_t s, const float* src, const int32_t* idx, float* out, int n);

}  // namespace rl

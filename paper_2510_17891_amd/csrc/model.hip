// Host side of the rollout library: C boundary, sequence table, per-call metadata, kernel sequencing.
//
// A "row" is one (sequence, position) pair pushed through the decoder.  A decode step is one row per
// sequence; prefill pushes every prompt token as a row, in chunks of max_rows, so both share one code path
// (the KV append of a layer runs for all rows of a chunk before that layer's attention, and a row only
// attends to keys at or before its own position).
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <string>
#include <vector>

#include "../../include/rl.h"
#include "kernels.h"
#include "seq_table.h"

using namespace rl;

namespace rl {

thread_local std::string g_err = "";

int set_error(int st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return st;
}

}  // namespace rl

#define fail(st, ...) ((rl_status)rl::set_error((int)(st), __VA_ARGS__))

namespace {

#define HIP_TRY(expr)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess) return fail(RL_ERR_DEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

constexpr int kRing = 64;  // per-call metadata slots in the workspace
constexpr int kRingCalls = kRing - 2;  // slots that ordinary calls cycle through; the last two belong to a decode graph
// One event covers this many uses of the slots (an event on every call costs the device 2.8 us between two kernels and the
// host 3 us).  Calls of a model are ordered one after another, on whatever streams, because they share the workspace:
// an event behind a later call is behind the earlier ones too.
constexpr int kEpochUses = 12, kEpochs = 8;
static_assert((kEpochs - 1) * kEpochUses > kRingCalls, "the event of a slot's last use is not recorded anew before the slot comes round");
constexpr int kPackMinPairs = 1024;  // (row, kv head) pairs of a decode step from which left-over segments are packed
constexpr int T_MAX_SCORE = 4096;  // sequences per scoring call

size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }

struct Layout {
  size_t block_table, rope, ring, x, x_last, q_last, h, part, q, attn_part, o, a, logits, samp_part, forced_z, tmp_tok, tmp_lp, cuts, last_tok, total;
  size_t slot_bytes, slot_upd, slot_skip, slot_sets, slot_tail, slot_head;
  size_t host_slot_bytes, slot_tok;  // the host side of a slot also holds tokens, which the first kernel reads there
  int max_segs, n_tiles;
};

size_t elem_size(uint32_t dtype) { return dtype == RL_BF16 ? 2 : 4; }
size_t kv_elem_size(const rl_model_config& c) { return c.kv_dtype == RL_KV_FP8 ? 1 : elem_size(c.dtype); }

rl_status check_config(const rl_model_config* c) {
  if (!c) return fail(RL_ERR_INVALID_ARG, "config is NULL");
  if (c->struct_size != sizeof(rl_model_config)) return fail(RL_ERR_INVALID_ARG, "struct_size mismatch");
  if (c->dtype != RL_F32 && c->dtype != RL_BF16) return fail(RL_ERR_INVALID_ARG, "unknown dtype");
  if (c->kv_dtype != RL_KV_SAME && c->kv_dtype != RL_KV_FP8) return fail(RL_ERR_INVALID_ARG, "unknown kv_dtype");
  if (c->kv_dtype == RL_KV_FP8 && c->dtype != RL_BF16) return fail(RL_ERR_UNSUPPORTED, "fp8 keys and values need a bf16 model");
  if (c->reserved != 0) return fail(RL_ERR_INVALID_ARG, "reserved must be 0");
  if (c->kv_block != 16) return fail(RL_ERR_UNSUPPORTED, "kv_block must be 16");
  if (!c->n_layers || !c->hidden || !c->n_q_heads || !c->n_kv_heads || !c->head_dim || !c->ffn)
    return fail(RL_ERR_INVALID_ARG, "zero dimension");
  if (c->n_q_heads % c->n_kv_heads) return fail(RL_ERR_INVALID_ARG, "n_q_heads %% n_kv_heads != 0");
  if (c->max_seqs == 0 || c->max_rows == 0 || c->max_rows > 1024) return fail(RL_ERR_INVALID_ARG, "max_rows must be in [1,1024]");
  if (c->max_ctx == 0 || c->max_ctx % 16) return fail(RL_ERR_INVALID_ARG, "max_ctx must be a positive multiple of 16");
  if (c->hidden % 8 || c->hidden > 8192 || c->head_dim % 2 || c->head_dim > 128 || c->ffn % 8 || c->vocab % 4)
    return fail(RL_ERR_UNSUPPORTED, "need hidden %% 8 == 0, hidden <= 8192, even head_dim <= 128, ffn %% 8 == 0, vocab %% 4 == 0");
  if (c->vocab >= (1u << 22)) return fail(RL_ERR_UNSUPPORTED, "vocab must be below 2^22");
  if (c->dtype == RL_BF16) {
    const uint32_t qd = c->n_q_heads * c->head_dim, nqkv = (c->n_q_heads + 2 * c->n_kv_heads) * c->head_dim;
    if (c->head_dim != 128 || c->n_q_heads / c->n_kv_heads > 8) return fail(RL_ERR_UNSUPPORTED, "bf16 needs head_dim 128 and group <= 8");
    if (c->hidden % 256 || qd % 256 || c->ffn % 256) return fail(RL_ERR_UNSUPPORTED, "bf16 needs hidden, n_q*head_dim, ffn multiples of 256");
    if (nqkv % 64 || c->hidden % 64 || c->ffn % 64 || c->vocab % 64) return fail(RL_ERR_UNSUPPORTED, "bf16 needs projection widths multiples of 64");
    if (c->max_ctx > 65536) return fail(RL_ERR_UNSUPPORTED, "bf16 attention merges at most 256 segments: max_ctx <= 65536");
  }
  return RL_OK;
}

void compute_layout(const rl_model_config& c, Layout* L) {
  const size_t R = c.max_rows, Rp = (R + 31) / 32 * 32, H = c.hidden, d = c.head_dim;
  const size_t nq = c.n_q_heads, nkv = c.n_kv_heads, F = c.ffn, V = c.vocab;
  const size_t act = elem_size(c.dtype);
  const size_t nqkv = (nq + 2 * nkv) * d;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
  L->max_segs = attn_bf16_max_segments((int)c.max_ctx);
  L->n_tiles = (int)((V + kSampleTile - 1) / kSampleTile);
  L->slot_upd = align_up(R * sizeof(RowMeta));
  L->slot_skip = L->slot_upd + align_up(R * 2 * sizeof(int32_t));  // upd: two integers per row
  L->slot_sets = L->slot_skip + align_up(R * sizeof(int32_t));
  L->slot_tail = L->slot_sets + align_up(R * sizeof(AttnShared));  // window sets: up to one per row
  L->slot_head = L->slot_tail + align_up(R * sizeof(RowMeta));
  L->slot_bytes = L->slot_head + align_up(R * sizeof(RowMeta));
  L->slot_tok = L->slot_bytes;
  L->host_slot_bytes = L->slot_tok + align_up(R * sizeof(int32_t));
  L->block_table = take((size_t)c.max_seqs * (c.max_ctx / 16) * 4);
  L->rope = take((size_t)c.max_ctx * (d / 2) * sizeof(float2));
  L->ring = take(kRing * L->slot_bytes);
  L->x = take(R * H * 4);
  L->x_last = take(R * H * 4);
  L->q_last = take(R * nq * d * 4);
  L->h = take(c.dtype == RL_BF16 ? Rp * H * act : 256);  // fp32 projections normalise their rows themselves
  size_t part_elems;
  if (c.dtype == RL_BF16) {
    size_t a1 = (size_t)gemm_bf16_splits((int)nqkv, (int)H, kEpiPartial) * R * nqkv;
    size_t a2 = (size_t)gemm_bf16_splits((int)H, (int)(nq * d), kEpiPartial) * R * H;
    size_t a3 = (size_t)gemm_bf16_splits((int)H, (int)F, kEpiPartial) * R * H;
    part_elems = a1 > a2 ? a1 : a2;
    if (a3 > part_elems) part_elems = a3;
  } else {
    part_elems = R * (nqkv > H ? nqkv : H);
  }
  L->part = take(part_elems * 4);
  L->q = take(R * nq * d * 4);
  L->attn_part = take(c.dtype == RL_BF16 ? R * nq * (size_t)L->max_segs * (d + 2) * 4 : 256);
  L->o = take(Rp * nq * d * act);
  L->a = take(Rp * F * act);
  // bf16: logits never reach memory (sampling happens in the projection's epilogue, 64 entries per partial) unless
  // the distribution is truncated (top-k / top-p need the whole row before any token can be drawn);
  // fp32: logits are written and scanned by the stand-alone sampler (2048 entries per partial).  rl_sample_logits
  // uses the stand-alone sampler in both cases.
  L->logits = take(V ? R * V * 4 : 256);
  const size_t tiles_fused = V / 64 + 1;
  L->samp_part = take(V ? R * (tiles_fused > (size_t)L->n_tiles ? tiles_fused : (size_t)L->n_tiles) * 32 : 256);
  L->forced_z = take(R * 4);
  L->tmp_tok = take(R * 4);
  L->tmp_lp = take(R * 4);
  L->cuts = take(V ? R * sample_cut_bytes_per_row() : 256);
  L->last_tok = take((size_t)c.max_seqs * 4);  // per sequence id: the token its last prefill / decode call returned
  L->total = off;
}

enum Kind { K_EMBED, K_NORM, K_QKV, K_ROPE_APPEND, K_ATTN, K_ATTN_MERGE, K_OPROJ, K_GATEUP, K_DOWN, K_LMHEAD, K_SAMPLE, K_COUNT };
const char* const kKindNames[K_COUNT] = {"embed", "residual_norm", "gemm_qkv", "qk_rope_append", "attn_decode", "attn_merge",
                                        "gemm_o", "gemm_gate_up_swiglu", "gemm_down", "gemm_lm_head", "sample"};

}  // namespace

struct rl_model {
  rl_model_config cfg;
  Geometry geo;
  Layout lay;
  SeqTable* table = nullptr;
  // weights (device pointers)
  const void *embed, *lm_head, *final_norm;
  std::vector<const void*> attn_norm, wqkv, q_norm, k_norm, wo, mlp_norm, w_gate_up, w_down;
  char* kv_pool;
  char* ws;
  size_t layer_kv_bytes, kv_block_bytes;  // one layer of the pool; one K (or V) block of a (page, kv head)
  // pinned host ring for per-call metadata
  char* host_ring = nullptr;
  int ring_next = 0;
  hipEvent_t epoch_ev[kEpochs];
  int64_t epoch = 0, epoch_done = -1;  // the epoch that is filling; the last one the host has seen finished
  int epoch_uses = 0;
  int64_t slot_epoch[kRing];  // epoch of a slot's last use, -1: never used
  float* capture = nullptr;
  bool graph_alive = false;     // a decode graph owns the last two metadata slots
  int attn_segs_per_block = 4;  // segments per attention block of contexts beyond 4096 keys (one per wave)
  int share_attention = 1;  // compute segments inside shared prompt pages once per set of rows where that pays (0: never, 2 / 3: always, in wide / narrow sets)
  bool attention_appends = true;  // decode steps: the attention kernel forms q and appends k, v itself
  // profiling
  bool prof_on = false;
  std::vector<hipEvent_t> ev_pool;
  struct Pending { int kind; hipEvent_t a, b; };
  std::vector<Pending> pending;
  double prof_ms[K_COUNT];
  int64_t prof_n[K_COUNT];
  // host time of rl_decode_step since the last read: admission checks, metadata build + upload, kernel launches
  double host_us[4] = {0.0, 0.0, 0.0, 0.0};  // admission, metadata, enqueue, wait for a metadata slot
  int64_t host_calls = 0;

  template <typename T> T* wsp(size_t off) const { return reinterpret_cast<T*>(ws + off); }
  void* k_pool(int l) const { return kv_pool + (size_t)l * layer_kv_bytes; }
  void* v_pool(int l) const { return kv_pool + (size_t)l * layer_kv_bytes + kv_block_bytes; }
};

namespace {

struct Timer {
  rl_model* m;
  hipStream_t st;
  hipEvent_t b = nullptr;
  int kind;
  Timer(rl_model* m_, hipStream_t st_, int kind_) : m(m_), st(st_), kind(kind_) {
    if (!m->prof_on) return;
    hipEvent_t a = take();
    b = take();
    if (a && b) {
      (void)hipEventRecord(a, st);
      m->pending.push_back({kind, a, b});
    } else {
      b = nullptr;
    }
  }
  ~Timer() {
    if (b) (void)hipEventRecord(b, st);
  }
  hipEvent_t take() {
    if (!m->ev_pool.empty()) { hipEvent_t e = m->ev_pool.back(); m->ev_pool.pop_back(); return e; }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
};

// Reserve a metadata slot: wait (practically never) until its previous upload has been consumed.
rl_status ring_acquire(rl_model* m, int* slot_out) {
  int s = m->ring_next;
  m->ring_next = (s + 1) % kRingCalls;
  const int64_t e = m->slot_epoch[s];
  if (e > m->epoch_done) {  // the device is up to kRingCalls calls behind: the host has nothing better to do than wait
    const auto t0 = std::chrono::steady_clock::now();
    if (e == m->epoch) HIP_TRY(hipDeviceSynchronize());  // only if recording the epoch's event has failed
    else HIP_TRY(hipEventSynchronize(m->epoch_ev[e % kEpochs]));
    if (e < m->epoch) m->epoch_done = e;
    m->host_us[3] += std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count();
  }
  *slot_out = s;
  return RL_OK;
}

// The work that reads the host side of a slot has been enqueued.
rl_status slot_in_use(rl_model* m, hipStream_t st, int slot) {
  m->slot_epoch[slot] = m->epoch;
  if (++m->epoch_uses < kEpochUses) return RL_OK;
  HIP_TRY(hipEventRecord(m->epoch_ev[m->epoch % kEpochs], st));
  m->epoch += 1;
  m->epoch_uses = 0;
  return RL_OK;
}

// Run all decoder layers on the M rows whose residual stream sits in ws.x.  Leaves the last down-projection's
// split partials pending and returns them, so that the caller's final residual_norm adds them.
struct Pending {  // n split sums of M rows that are still to be added to the residual stream, in order
  const float* part = nullptr;
  int n = 0;
};
struct SharedAttn {  // device pointers into the metadata slot of the call (empty: every row on its own)
  const int32_t* skip = nullptr;
  const AttnShared* sets = nullptr;
  int n_sets = 0, max_segs = 0;
  int set_segs = 4;     // segments of a set block
  bool window = false;  // every row is in a set, and the sets cover all segments of their rows
  bool packs = false, all_packed = false;  // some sets are packs of single segments; no row is left to a block of its own
};

// A layer boundary of a capture (may be null) where no norm writes it: the residual stream as it is.
void copy_capture(hipStream_t st, float* cap, const float* x, int M, int H) {
  if (cap) (void)hipMemcpyAsync(cap, x, (size_t)M * H * 4, hipMemcpyDeviceToDevice, st);  // an error stays for hipGetLastError
}

// One layer from the attention on, for M rows with residual stream x.  ap: a decode step, whose attention takes over the
// rotation and the KV append (a row's block is then the only reader of the key it writes); otherwise the queries are in
// q.  Returns the split partials that are left to add to x (none where the projections added them themselves).
Pending finish_layer(rl_model* m, hipStream_t st, int l, int M, const RowMeta* rows, int max_ctx_in_batch, const SharedAttn& sa,
                 const float* q, const AttnAppend* ap, float* x) {
  const Geometry& g = m->geo;
  const bool bf = g.dtype == kBF16;
  const int H = g.hidden, nqd = g.n_q * g.head_dim, F = g.ffn;
  void* h = m->wsp<void>(m->lay.h);
  float* part = m->wsp<float>(m->lay.part);
  float* apart = m->wsp<float>(m->lay.attn_part);
  void* o = m->wsp<void>(m->lay.o);
  void* a = m->wsp<void>(m->lay.a);
  const int32_t* bt = m->wsp<int32_t>(m->lay.block_table);
  if (bf) {
    bool merge;
    { Timer t(m, st, K_ATTN);
      merge = launch_attn_decode_bf16(st, g, q, rows, bt, m->k_pool(l), m->v_pool(l), apart, m->lay.max_segs, max_ctx_in_batch,
                                      o, M, sa.skip, sa.sets, sa.n_sets, sa.max_segs, ap, m->attn_segs_per_block, sa.set_segs, sa.window, sa.packs, sa.all_packed); }
    if (merge) {
      Timer t(m, st, K_ATTN_MERGE);
      launch_attn_merge_bf16(st, g, rows, apart, m->lay.max_segs, max_ctx_in_batch, o, M, sa.skip, sa.n_sets);
    }
  } else {
    Timer t(m, st, K_ATTN);
    launch_attn_f32(st, g, q, rows, bt, m->k_pool(l), m->v_pool(l), (float*)o, M, ap);
  }
  // A row or two: gate/up does the norm before it, and leaves the O projection's split sums pending with those of the down projection behind them;
  // the attention's partials make room for both (a model of one row has no other buffer that long).
  const int s_up = bf ? gemm_bf16_partials(M, H, nqd) : 0, s_down = bf ? gemm_bf16_partials(M, H, F) : 0;
  if (bf && norm_gate_up_takes(M, H, s_up) && !gemm_bf16_adds_residual(M, H, nqd) && !gemm_bf16_adds_residual(M, H, F) &&
      (size_t)(s_up + s_down) * M * H <= (size_t)m->cfg.max_rows * g.n_q * m->lay.max_segs * (g.head_dim + 2)) {
    { Timer t(m, st, K_OPROJ);
      launch_gemm_bf16(st, o, m->wo[l], apart, M, H, nqd, kEpiPartial); }
    { Timer t(m, st, K_GATEUP);
      launch_norm_gate_up(st, x, apart, s_up, m->mlp_norm[l], g.rms_eps, m->w_gate_up[l], a, M, F, H); }
    Timer t(m, st, K_DOWN);
    launch_gemm_bf16(st, a, m->w_down[l], apart + (size_t)s_up * M * H, M, H, F, kEpiPartial);
    return {apart, s_up + s_down};
  }
  int s_o = 1;
  { Timer t(m, st, K_OPROJ);
    if (bf && gemm_bf16_adds_residual(M, H, nqd)) { launch_gemm_bf16(st, o, m->wo[l], x, M, H, nqd, kEpiResidual); s_o = 0; }
    else if (bf) { launch_gemm_bf16(st, o, m->wo[l], part, M, H, nqd, kEpiPartial); s_o = s_up; }
    else { launch_gemm_f32(st, (const float*)o, (const float*)m->wo[l], x, M, H, nqd, kEpiResidual); s_o = 0; } }
  if (bf) {
    Timer t(m, st, K_NORM);
    launch_residual_norm(st, x, x, s_o ? part : nullptr, s_o, m->mlp_norm[l], h, nullptr, M, H, g.rms_eps);
  }
  { Timer t(m, st, K_GATEUP);
    if (bf) launch_gemm_bf16(st, h, m->w_gate_up[l], a, M, F, H, kEpiSwiGLU);
    else launch_gemm_f32(st, x, (const float*)m->w_gate_up[l], (float*)a, M, F, H, kEpiSwiGLU, (const float*)m->mlp_norm[l], g.rms_eps); }
  Timer t(m, st, K_DOWN);
  if (bf && gemm_bf16_adds_residual(M, H, F)) { launch_gemm_bf16(st, a, m->w_down[l], x, M, H, F, kEpiResidual); return {}; }
  if (bf) { launch_gemm_bf16(st, a, m->w_down[l], part, M, H, F, kEpiPartial); return {part, s_down}; }
  launch_gemm_f32(st, (const float*)a, (const float*)m->w_down[l], x, M, H, F, kEpiResidual);
  return {};
}

// Rows of a prefill chunk that end a prompt: device pairs (row of the chunk, prompt).
struct PromptEnds {
  const int32_t* pairs = nullptr;
  int n = 0;
};

// The rows and their first norm (bf16: in h) are there: launch_entry ran.
// one_row_per_seq: the batch is a decode step, which lets the attention kernel take over the rotation and the KV append.
// ends (a prefill chunk; otherwise null): of the last layer, only the keys and values of the chunk's rows are needed by
// anyone, and its output of the rows that end a prompt: the residual stream and the queries of those are put aside (x_last,
// q_last, by prompt) for one pass over the prompts of all chunks, and the layer ends there unless its boundary is captured.
// It saves most of one layer: of four, 4 prompts of 1024 tokens 9.4 -> 7.8 ms and one of 301 1.88 -> 1.72 (with the copies per
// sequence gone); of thirty-six 79.1 -> 77.1 and 12.95 -> 12.75.
Pending run_layers(rl_model* m, hipStream_t st, int M, const RowMeta* rows, int max_ctx_in_batch,
               const SharedAttn& sa = SharedAttn(), bool one_row_per_seq = false, const PromptEnds* ends = nullptr) {
  const Geometry& g = m->geo;
  const bool bf = g.dtype == kBF16;
  const int H = g.hidden, nqkv = (g.n_q + 2 * g.n_kv) * g.head_dim;
  float* x = m->wsp<float>(m->lay.x);
  void* h = m->wsp<void>(m->lay.h);
  float* part = m->wsp<float>(m->lay.part);
  float* q = m->wsp<float>(m->lay.q);
  const float2* rope = m->wsp<float2>(m->lay.rope);
  Pending pend;
  for (int l = 0; l < g.n_layers; ++l) {
    float* cap = m->capture ? m->capture + (size_t)l * m->cfg.max_rows * H : nullptr;
    if (!bf) {
      copy_capture(st, cap, x, M, H);
    } else if (l > 0) {
      Timer t(m, st, K_NORM);
      launch_residual_norm(st, x, x, pend.part, pend.n, m->attn_norm[l], h, cap, M, H, g.rms_eps);
    }
    int s_qkv = 1;
    { Timer t(m, st, K_QKV);
      if (bf) { launch_gemm_bf16(st, h, m->wqkv[l], part, M, nqkv, H, kEpiPartial); s_qkv = gemm_bf16_partials(M, nqkv, H); }
      else launch_gemm_f32(st, x, (const float*)m->wqkv[l], part, M, nqkv, H, kEpiPartial, (const float*)m->attn_norm[l], g.rms_eps); }
    const void* q_gain = g.qk_norm ? m->q_norm[l] : nullptr;
    const void* k_gain = g.qk_norm ? m->k_norm[l] : nullptr;
    const bool fused = one_row_per_seq && m->attention_appends && s_qkv <= kAttnAppendMaxSplits;
    const AttnAppend ap = {part, s_qkv, q_gain, k_gain, rope};
    if (!fused) {
      Timer t(m, st, K_ROPE_APPEND);
      launch_qk_rope_append(st, g, part, s_qkv, q_gain, k_gain, rope, rows, m->k_pool(l), m->v_pool(l), q, M);
    }
    if (ends && l + 1 == g.n_layers) {
      launch_put_aside(st, ends->pairs, ends->n, x, m->wsp<float>(m->lay.x_last), H, q, m->wsp<float>(m->lay.q_last), g.n_q * g.head_dim);
      if (!m->capture) return {};
    }
    pend = finish_layer(m, st, l, M, rows, max_ctx_in_batch, sa, q, fused ? &ap : nullptr, x);
  }
  return pend;
}

// Final norm, output projection and sampling for M rows; row r's residual (pending partials added) is row r / group of `xbuf`,
// which is not the workspace's own x if group > 1.
void run_head(rl_model* m, hipStream_t st, int M, float* xbuf, const Pending& pend, const RowMeta* rows, int pos_offset,
              const int32_t* forced, const rl_sampling* sp, int32_t* out_tokens, float* out_lp, float* debug_logits,
              bool score_only = false, int group = 1) {
  int32_t* last_tok = score_only ? nullptr : m->wsp<int32_t>(m->lay.last_tok);
  const Geometry& g = m->geo;
  void* h = m->wsp<void>(m->lay.h);
  float* logits = m->wsp<float>(m->lay.logits);
  float* cap = m->capture ? m->capture + (size_t)g.n_layers * m->cfg.max_rows * g.hidden : nullptr;
  const bool bf = g.dtype == kBF16;
  if (bf) {
    Timer t(m, st, K_NORM);
    launch_residual_norm(st, xbuf, group > 1 ? m->wsp<float>(m->lay.x) : xbuf, pend.part, pend.n, m->final_norm, h, cap, M, g.hidden, g.rms_eps, group);
  } else {
    if (group > 1) {
      launch_repeat_rows(st, xbuf, m->wsp<float>(m->lay.x), M, g.hidden, group);
      xbuf = m->wsp<float>(m->lay.x);
    }
    copy_capture(st, cap, xbuf, M, g.hidden);
  }
  float* spart = m->wsp<float>(m->lay.samp_part);
  float* fz = m->wsp<float>(m->lay.forced_z);
  const int top_k = sp->top_k > (uint32_t)g.vocab ? 0 : (int)sp->top_k;
  const bool truncated = !score_only && sp->temperature > 0.f && sample_is_truncated(g.vocab, top_k, sp->top_p);
  if (g.dtype == kBF16 && !truncated) {
    SampleEpilogue se;
    se.rows = rows; se.pos_offset = pos_offset;
    se.greedy = !(sp->temperature > 0.f);
    se.inv_t = se.greedy ? 1.0f : 1.0f / sp->temperature;
    if (score_only) se.greedy = 1;  // every row is forced: skip the random numbers, keep the temperature
    se.seed_lo = (uint32_t)(sp->seed & 0xffffffffu); se.seed_hi = (uint32_t)(sp->seed >> 32);
    se.forced = forced; se.forced_z = fz; se.part = spart; se.logits_out = debug_logits;
    { Timer t(m, st, K_LMHEAD);
      launch_gemm_bf16(st, h, m->lm_head, nullptr, M, g.vocab, g.hidden, kEpiSample, false, &se); }
    { Timer t(m, st, K_SAMPLE);
      launch_sample_merge(st, spart, g.vocab >> 6, M, g.vocab, forced, fz, sp->temperature, out_tokens, out_lp, rows, last_tok); }
  } else {
    // logits to memory (a truncated distribution needs the whole row first), then the stand-alone sampler
    { Timer t(m, st, K_LMHEAD);
      if (g.dtype == kBF16) launch_gemm_bf16(st, h, m->lm_head, logits, M, g.vocab, g.hidden, kEpiPartial, false);
      else launch_gemm_f32(st, xbuf, (const float*)m->lm_head, logits, M, g.vocab, g.hidden, kEpiPartial, (const float*)m->final_norm, g.rms_eps); }
    { Timer t(m, st, K_SAMPLE);
      launch_sample(st, logits, M, g.vocab, rows, pos_offset, forced, sp->temperature, sp->seed, spart, fz, out_tokens, out_lp,
                    truncated ? top_k : 0, truncated ? sp->top_p : 0.f, m->wsp<void>(m->lay.cuts), last_tok); }
    if (debug_logits)
      (void)hipMemcpyAsync(debug_logits, logits, (size_t)M * g.vocab * 4, hipMemcpyDeviceToDevice, st);
  }
}

// Checks shared by decode calls; on success the pages are handed out and lens are NOT yet advanced.
rl_status admit_decode(rl_model* m, int32_t n, const int32_t* seq_ids) {
  if (n < 1 || n > (int32_t)m->cfg.max_rows) return fail(RL_ERR_INVALID_ARG, "n_seqs %d outside [1, max_rows=%u]", n, m->cfg.max_rows);
  if (!seq_ids) return fail(RL_ERR_INVALID_ARG, "seq_ids is NULL");
  SeqTable& T = *m->table;
  std::vector<char> seen(T.max_seqs(), 0);
  int64_t need = 0;
  for (int i = 0; i < n; ++i) {
    int32_t s = seq_ids[i];
    if (!T.active(s)) return fail(RL_ERR_BAD_SEQ, "sequence %d is not active", s);
    if (seen[s]) return fail(RL_ERR_INVALID_ARG, "sequence %d appears twice", s);
    seen[s] = 1;
    if (T.len(s) + 1 > T.max_ctx()) return fail(RL_ERR_CTX_OVERFLOW, "sequence %d would exceed max_ctx %d", s, T.max_ctx());
    need += T.pages_missing(s, T.len(s) + 1);
  }
  if (need > T.free_pages()) return fail(RL_ERR_KV_FULL, "need %lld pages, %lld free", (long long)need, (long long)T.free_pages());
  for (int i = 0; i < n; ++i) T.reserve(seq_ids[i], T.len(seq_ids[i]) + 1);
  return RL_OK;
}

// The upload of a call's rows from its host slot hs to its device slot ds; more regions of the slot are added to it.
// table: the rows enter their pages in the block table.
SlotUpload slot_upload(const rl_model* m, const char* hs, char* ds, int n_rows, bool table) {
  static_assert(sizeof(RowMeta) == 16, "one unit per row");
  SlotUpload up;
  up.src = (const uint4*)hs;
  up.dst = (uint4*)ds;
  up.n_rows = n_rows;
  up.block_table = table ? m->wsp<int32_t>(m->lay.block_table) : nullptr;
  up.max_blocks = m->geo.max_blocks;
  return up;
}
void add_region(SlotUpload* up, size_t at, size_t bytes) {  // regions start and are padded at multiples of 256 bytes
  int k = 0;
  while (up->n[k]) ++k;
  up->at[k] = (int)(at / 16);
  up->n[k] = (int)((bytes + 15) / 16);
}

// Copy a plan of shared attention into the host slot, add it to the upload and describe it (device pointers) in *sa.
void place_attn_plan(rl_model* m, char* hs, char* ds, int n, const AttnPlan& plan, SharedAttn* sa, SlotUpload* up) {
  *sa = SharedAttn();
  if (plan.sets.empty()) return;
  memcpy(hs + m->lay.slot_skip, plan.skip.data(), (size_t)n * 4);
  memcpy(hs + m->lay.slot_sets, plan.sets.data(), plan.sets.size() * sizeof(AttnShared));
  add_region(up, m->lay.slot_skip, (size_t)n * 4);
  add_region(up, m->lay.slot_sets, plan.sets.size() * sizeof(AttnShared));
  sa->skip = (const int32_t*)(ds + m->lay.slot_skip);
  sa->sets = (const AttnShared*)(ds + m->lay.slot_sets);
  sa->n_sets = (int)plan.sets.size();
  sa->max_segs = plan.max_shared_segs;
  sa->packs = plan.packs > 0;
  sa->all_packed = plan.all_packed;
}

// First kernel of a call: the upload, the rows into the residual stream, the first norm.  Marks the slot as in use until
// the kernel has read it.
rl_status enter_rows(rl_model* m, hipStream_t st, int slot, const RowSource& in, const SlotUpload& up, int M) {
  float* cap = m->geo.dtype == kBF16 ? m->capture : nullptr;  // layer 0's boundary; fp32: copied in run_layers
  { Timer t(m, st, K_EMBED);
    launch_entry(st, m->geo.dtype, in, up, m->wsp<float>(m->lay.x), m->attn_norm[0], m->wsp<void>(m->lay.h), cap, M, m->geo.hidden, m->geo.rms_eps); }
  return slot_in_use(m, st, slot);
}

RowSource table_rows(const rl_model* m, const char* hs, const int32_t* tokens) {
  RowSource in;
  in.src = m->embed;
  in.from_table = 1;
  in.tokens = tokens;
  in.last_tok = m->wsp<int32_t>(m->lay.last_tok);
  in.rows = (const RowMeta*)hs;
  in.V = m->geo.vocab;
  return in;
}

// Rows per set for a call of n rows (the test switch can ask for the wide sets always or never, whatever the size).
int rows_per_set(const rl_model* m, int n) {
  if (m->share_attention == 2) n = 1 << 20;
  if (m->share_attention == 3) n = 0;
  return attn_rows_per_set(m->geo.n_q / m->geo.n_kv, m->geo.kv_fp8, n, m->geo.n_kv);
}

// Sets of neighbouring rows of one sequence for a chunk of prefill or scoring rows (bf16 only).
void place_window_plan(rl_model* m, char* hs, char* ds, int n, const RowMeta* hr, SharedAttn* sa, SlotUpload* up) {
  *sa = SharedAttn();
  if (m->geo.dtype != kBF16 || !m->share_attention) return;
  std::vector<int32_t> seq(n), pos(n);
  for (int i = 0; i < n; ++i) { seq[i] = hr[i].seq; pos[i] = hr[i].pos; }
  AttnPlan plan;
  plan_window_sets(n, seq.data(), pos.data(), rows_per_set(m, n), &plan);
  if (plan.sets.empty()) return;  // every row on its own
  // The rows left over become sets of one, so that the launch needs no row blocks; the longest contexts come first, so
  // that the blocks still running at its end are short ones.
  for (int i = 0; i < n; ++i) {
    if (plan.skip[i]) continue;
    AttnShared s;
    s.n_rows = 1;
    s.n_segs = attn_num_segments(pos[i] + 1);
    for (int k = 0; k < kAttnSetRows; ++k) s.rows[k] = i;
    plan.skip[i] = s.n_segs;
    plan.sets.push_back(s);
    plan.max_shared_segs = std::max(plan.max_shared_segs, s.n_segs);
  }
  std::stable_sort(plan.sets.begin(), plan.sets.end(), [&](const AttnShared& a, const AttnShared& b) { return pos[a.rows[0]] > pos[b.rows[0]]; });
  place_attn_plan(m, hs, ds, n, plan, sa, up);
  sa->window = sa->n_sets > 0;
}

// Write the rows and the shared-attention plan of one decode call into the host slot hs and describe them (device
// pointers relative to the device slot ds).  Returns the upload that brings them there.
// fixed_shape: the launch shape changes as rarely as it can (decode graphs).
SlotUpload build_decode_meta(rl_model* m, int32_t n, const int32_t* seq_ids, char* hs, char* ds, int* max_ctx_out, SharedAttn* sa,
                             bool fixed_shape = false) {
  RowMeta* hr = (RowMeta*)hs;
  int max_ctx = 0;
  for (int i = 0; i < n; ++i) {
    hr[i].seq = seq_ids[i];
    hr[i].pos = m->table->len(seq_ids[i]);
    hr[i].page = m->table->pages(seq_ids[i])[hr[i].pos >> 4];  // reserved by admit_decode
    hr[i].pad = 0;
    if (hr[i].pos + 1 > max_ctx) max_ctx = hr[i].pos + 1;
  }
  // rows of sequences that hold prompt pages in common and stand at the same position share those segments
  AttnPlan plan;
  // (the test switch's wide and narrow sets: in every call)
  if (m->geo.dtype == kBF16 && m->share_attention && (m->share_attention > 1 || max_ctx > attn_alone_up_to(n, m->geo.n_kv, m->geo.n_q / m->geo.n_kv))) {
    std::vector<int64_t> fam(n);
    std::vector<int32_t> fam_blocks(n), pos(n);
    bool any = false;
    for (int i = 0; i < n; ++i) {
      fam[i] = m->table->prefix_id(seq_ids[i]);
      fam_blocks[i] = m->table->prefix_blocks(seq_ids[i]);
      pos[i] = hr[i].pos;
      any |= fam[i] != 0;
    }
    if (any) {
      plan_shared_attention(n, fam.data(), fam_blocks.data(), pos.data(), rows_per_set(m, n), &plan);
      plan_packs(n, pos.data(), m->geo.n_kv, m->geo.n_q / m->geo.n_kv, m->share_attention == 2 ? 0 : m->share_attention == 3 ? 1 << 30 : kPackMinPairs, n, fixed_shape, &plan);
    }
  }
  SlotUpload up = slot_upload(m, hs, ds, n, true);
  place_attn_plan(m, hs, ds, n, plan, sa, &up);
  if (sa->n_sets) sa->set_segs = attn_set_segments(n, m->geo.n_kv, m->geo.kv_fp8, plan);
  *max_ctx_out = max_ctx;
  return up;
}

// Build the rows of one decode call in a metadata slot of their own; *rows_dev and *sa are device pointers into it, valid once the
// upload has run.
struct DecodeMeta {
  int slot;
  char* hs;
  SlotUpload up;
  const RowMeta* rows_dev;
  int max_ctx;
  SharedAttn sa;
};
rl_status prepare_decode_meta(rl_model* m, int32_t n, const int32_t* seq_ids, DecodeMeta* dm) {
  rl_status rs = ring_acquire(m, &dm->slot);
  if (rs != RL_OK) return rs;
  dm->hs = m->host_ring + (size_t)dm->slot * m->lay.host_slot_bytes;
  char* ds = m->ws + m->lay.ring + (size_t)dm->slot * m->lay.slot_bytes;
  dm->up = build_decode_meta(m, n, seq_ids, dm->hs, ds, &dm->max_ctx, &dm->sa);
  dm->rows_dev = (const RowMeta*)ds;
  return RL_OK;
}

// The kernels of one decode step behind its first: layers and head.
void decode_enqueue(rl_model* m, hipStream_t st, int n, const RowMeta* rows, int max_ctx_in_batch, const SharedAttn& sa,
                    const int32_t* forced_next, const rl_sampling* sp, int32_t* out_tokens, float* out_logprobs, float* debug_logits) {
  const Pending pend = run_layers(m, st, n, rows, max_ctx_in_batch, sa, true);
  run_head(m, st, n, m->wsp<float>(m->lay.x), pend, rows, 1, forced_next, sp, out_tokens, out_logprobs, debug_logits);
}

}  // namespace

// A decode step of a fixed batch as a HIP graph.  What changes from step to step is data (rows and the
// shared-attention plan: one upload from a pinned buffer that the graph's first kernel reads at every launch) except for
// five launch shapes, which form the key of the captured graph: the context that stands for the longest one (block
// counts and shared-memory size of the attention launch; attn_capture_ctx), the number of row sets, the blocks the sets need and the segments of one, and
// whether some or all of what the sets leave of their rows is packed.  When the key changes, the step is captured again.  A batch in
// lock step does so every 1024 steps, once more at 384 keys if its rows leave compute units idle (attn_split), and, where it
// holds samples of one prompt, where they begin to share (attn_alone_up_to) and with each four segments more in the
// prompt's pages.  Two buffers and two graphs alternate, so the host may prepare step k + 1 while step k runs.
struct rl_decode_graph {
  rl_model* m = nullptr;
  std::vector<int32_t> ids;
  rl_sampling sp;
  int32_t* out_tokens = nullptr;
  float* out_logprobs = nullptr;
  char* host[2] = {nullptr, nullptr};  // pinned copies of the metadata slot
  hipEvent_t ev[2] = {nullptr, nullptr};
  bool ev_used[2] = {false, false};
  hipGraphExec_t exec[2] = {nullptr, nullptr};
  struct Key { int ctx, n_sets, set_blocks, set_segs, packs; } key[2] = {{-1, -1, -1, -1, -1}, {-1, -1, -1, -1, -1}};
  int next = 0;
  int64_t captures = 0;
};

extern "C" {

const char* rl_last_error(void) { return g_err.c_str(); }

uint64_t rl_kv_page_bytes(const rl_model_config* c) {
  if (check_config(c) != RL_OK) return 0;
  return (uint64_t)c->n_layers * 2 * c->n_kv_heads * 16 * c->head_dim * kv_elem_size(*c);
}

rl_status rl_query_workspace(const rl_model_config* c, uint64_t* bytes_out) {
  rl_status rs = check_config(c);
  if (rs != RL_OK) return rs;
  if (!bytes_out) return fail(RL_ERR_INVALID_ARG, "bytes_out is NULL");
  Layout L;
  compute_layout(*c, &L);
  *bytes_out = L.total;
  return RL_OK;
}

rl_status rl_init_model(const rl_model_config* c, const rl_weights* w, rl_model** out) {
  rl_status rs = check_config(c);
  if (rs != RL_OK) return rs;
  if (!w || !out) return fail(RL_ERR_INVALID_ARG, "weights or out is NULL");
  if (!w->final_norm || !w->attn_norm || !w->wqkv || !w->wo || !w->mlp_norm || !w->w_gate_up || !w->w_down || !w->kv_pool || !w->workspace)
    return fail(RL_ERR_INVALID_ARG, "a required weight pointer is NULL");
  if (c->vocab && (!w->embed || !w->lm_head)) return fail(RL_ERR_INVALID_ARG, "embed/lm_head is NULL with vocab > 0");
  if (c->qk_norm && (!w->q_norm || !w->k_norm)) return fail(RL_ERR_INVALID_ARG, "q_norm/k_norm is NULL with qk_norm = 1");
  Layout L;
  compute_layout(*c, &L);
  if (c->workspace_bytes < L.total) return fail(RL_ERR_INVALID_ARG, "workspace_bytes %llu < required %llu", (unsigned long long)c->workspace_bytes, (unsigned long long)L.total);
  const uint64_t page_bytes = rl_kv_page_bytes(c);
  const int64_t n_pages = (int64_t)(c->kv_pool_bytes / page_bytes);
  if (n_pages < 1 || n_pages > 0x7fffffff) return fail(RL_ERR_INVALID_ARG, "kv_pool_bytes gives %lld pages", (long long)n_pages);

  rl_model* m = new rl_model();
  m->cfg = *c;
  m->lay = L;
  m->geo = Geometry{(int)c->n_layers, (int)c->hidden, (int)c->n_q_heads, (int)c->n_kv_heads, (int)c->head_dim, (int)c->ffn,
                    (int)c->vocab, (int)c->qk_norm, c->rms_eps, (int)c->dtype, (int)(c->max_ctx / 16), n_pages,
                    c->kv_dtype == RL_KV_FP8 ? 1 : 0};
  m->embed = w->embed; m->lm_head = w->lm_head; m->final_norm = w->final_norm;
  auto copy = [&](std::vector<const void*>& dst, const void* const* src) {
    dst.assign(c->n_layers, nullptr);
    if (src) for (uint32_t l = 0; l < c->n_layers; ++l) dst[l] = src[l];
  };
  copy(m->attn_norm, w->attn_norm); copy(m->wqkv, w->wqkv); copy(m->q_norm, w->q_norm); copy(m->k_norm, w->k_norm);
  copy(m->wo, w->wo); copy(m->mlp_norm, w->mlp_norm); copy(m->w_gate_up, w->w_gate_up); copy(m->w_down, w->w_down);
  for (uint32_t l = 0; l < c->n_layers; ++l)
    if (!m->attn_norm[l] || !m->wqkv[l] || !m->wo[l] || !m->mlp_norm[l] || !m->w_gate_up[l] || !m->w_down[l] ||
        (c->qk_norm && (!m->q_norm[l] || !m->k_norm[l]))) {
      delete m;
      return fail(RL_ERR_INVALID_ARG, "layer %u has a NULL weight pointer", l);
    }
  m->kv_pool = (char*)w->kv_pool;
  m->ws = (char*)w->workspace;
  m->kv_block_bytes = (size_t)16 * c->head_dim * kv_elem_size(*c);
  m->layer_kv_bytes = (size_t)n_pages * c->n_kv_heads * 2 * m->kv_block_bytes;
  m->table = new SeqTable((int)c->max_seqs, (int)c->max_ctx, n_pages);
  for (int i = 0; i < K_COUNT; ++i) { m->prof_ms[i] = 0; m->prof_n[i] = 0; }
  for (int i = 0; i < kRing; ++i) m->slot_epoch[i] = -1;
  for (int i = 0; i < kEpochs; ++i) m->epoch_ev[i] = nullptr;

  auto bail = [&](hipError_t e, const char* what) {
    rl_status r = fail(RL_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
    rl_destroy_model(m);
    return r;
  };
  hipError_t e;
  if ((e = hipHostMalloc((void**)&m->host_ring, kRing * L.host_slot_bytes, hipHostMallocDefault)) != hipSuccess) return bail(e, "hipHostMalloc");
  for (int i = 0; i < kEpochs; ++i)
    if ((e = hipEventCreateWithFlags(&m->epoch_ev[i], hipEventDisableTiming)) != hipSuccess) return bail(e, "hipEventCreate");
  // Stale slots of recycled pages are multiplied by zero weights, so the pool must never hold NaN/Inf patterns.
  if ((e = hipMemset(m->kv_pool, 0, (size_t)n_pages * page_bytes)) != hipSuccess) return bail(e, "hipMemset(kv_pool)");
  if ((e = hipMemset(m->ws + L.block_table, 0, (size_t)c->max_seqs * (c->max_ctx / 16) * 4)) != hipSuccess) return bail(e, "hipMemset(block_table)");
  {
    const int half = (int)c->head_dim / 2;
    std::vector<float2> tab((size_t)c->max_ctx * half);
    for (int i = 0; i < half; ++i) {
      const double freq = std::pow((double)c->rope_base, -2.0 * i / (double)c->head_dim);
      for (uint32_t p = 0; p < c->max_ctx; ++p) {
        const double ang = (double)p * freq;
        tab[(size_t)p * half + i] = make_float2((float)std::cos(ang), (float)std::sin(ang));
      }
    }
    if ((e = hipMemcpy(m->ws + L.rope, tab.data(), tab.size() * sizeof(float2), hipMemcpyHostToDevice)) != hipSuccess) return bail(e, "hipMemcpy(rope)");
  }
  if ((e = hipDeviceSynchronize()) != hipSuccess) return bail(e, "hipDeviceSynchronize");
  *out = m;
  return RL_OK;
}

void rl_destroy_model(rl_model* m) {
  if (!m) return;
  for (auto& p : m->pending) { (void)hipEventDestroy(p.a); (void)hipEventDestroy(p.b); }
  for (auto ev : m->ev_pool) (void)hipEventDestroy(ev);
  for (int i = 0; i < kEpochs; ++i) if (m->epoch_ev[i]) (void)hipEventDestroy(m->epoch_ev[i]);
  if (m->host_ring) (void)hipHostFree(m->host_ring);
  delete m->table;
  delete m;
}

rl_status rl_kv_stats(const rl_model* m, uint64_t* free_pages, uint64_t* total_pages) {
  if (!m) return fail(RL_ERR_INVALID_ARG, "model is NULL");
  if (free_pages) *free_pages = (uint64_t)m->table->free_pages();
  if (total_pages) *total_pages = (uint64_t)m->table->n_pages();
  return RL_OK;
}

rl_status rl_seq_len(const rl_model* m, int32_t seq_id, int32_t* len_out) {
  if (!m || !len_out) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  if (!m->table->active(seq_id)) return fail(RL_ERR_BAD_SEQ, "sequence %d is not active", seq_id);
  *len_out = m->table->len(seq_id);
  return RL_OK;
}

rl_status rl_free_seqs(rl_model* m, int32_t n, const int32_t* seq_ids) {
  if (!m || (n > 0 && !seq_ids) || n < 0) return fail(RL_ERR_INVALID_ARG, "bad arguments");
  SeqTable& T = *m->table;
  std::vector<char> seen(T.max_seqs(), 0);
  for (int i = 0; i < n; ++i) {
    if (!T.active(seq_ids[i])) return fail(RL_ERR_BAD_SEQ, "sequence %d is not active", seq_ids[i]);
    if (seen[seq_ids[i]]) return fail(RL_ERR_INVALID_ARG, "sequence %d appears twice", seq_ids[i]);
    seen[seq_ids[i]] = 1;
  }
  for (int i = 0; i < n; ++i) T.release(seq_ids[i]);
  return RL_OK;
}

rl_status rl_debug_shuffle_free_pages(rl_model* m, uint64_t seed) {
  if (!m) return fail(RL_ERR_INVALID_ARG, "model is NULL");
  m->table->shuffle_free(seed);
  return RL_OK;
}

rl_status rl_debug_share_attention(rl_model* m, int32_t on) {
  if (!m) return fail(RL_ERR_INVALID_ARG, "model is NULL");
  m->share_attention = (on == 2 || on == 3) ? on : on != 0;
  return RL_OK;
}

rl_status rl_debug_attention_split(rl_model* m, int32_t segs_per_block) {
  if (!m) return fail(RL_ERR_INVALID_ARG, "model is NULL");
  if (segs_per_block < 1 || segs_per_block > 16) return fail(RL_ERR_INVALID_ARG, "segs_per_block %d outside [1, 16]", segs_per_block);
  m->attn_segs_per_block = segs_per_block;
  return RL_OK;
}

rl_status rl_debug_attention_appends(rl_model* m, int32_t on) {
  if (!m) return fail(RL_ERR_INVALID_ARG, "model is NULL");
  m->attention_appends = on != 0;
  return RL_OK;
}

rl_status rl_set_capture(rl_model* m, float* buf) {
  if (!m) return fail(RL_ERR_INVALID_ARG, "model is NULL");
  m->capture = buf;
  return RL_OK;
}

rl_status rl_decode_step(rl_model* m, void* stream, int32_t n, const int32_t* seq_ids, const int32_t* in_tokens,
                         const int32_t* forced_next, const rl_sampling* sp, int32_t* out_tokens, float* out_logprobs,
                         float* debug_logits) {
  if (!m || !sp || !out_tokens || !out_logprobs) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  if (m->geo.vocab == 0) return fail(RL_ERR_UNSUPPORTED, "model has no vocabulary");
  hipStream_t st = (hipStream_t)stream;
  const auto t0 = std::chrono::steady_clock::now();
  rl_status rs = admit_decode(m, n, seq_ids);
  if (rs != RL_OK) return rs;
  const auto t1 = std::chrono::steady_clock::now();
  const double waited = m->host_us[3];
  DecodeMeta dm;
  rs = prepare_decode_meta(m, n, seq_ids, &dm);
  if (rs != RL_OK) return rs;
  const auto t2 = std::chrono::steady_clock::now();
  rs = enter_rows(m, st, dm.slot, table_rows(m, dm.hs, in_tokens), dm.up, n);
  if (rs != RL_OK) return rs;
  decode_enqueue(m, st, n, dm.rows_dev, dm.max_ctx, dm.sa, forced_next, sp, out_tokens, out_logprobs, debug_logits);
  HIP_TRY(hipGetLastError());
  for (int i = 0; i < n; ++i) m->table->set_len(seq_ids[i], m->table->len(seq_ids[i]) + 1);
  const auto t3 = std::chrono::steady_clock::now();
  m->host_us[0] += std::chrono::duration<double, std::micro>(t1 - t0).count();
  m->host_us[1] += std::chrono::duration<double, std::micro>(t2 - t1).count() - (m->host_us[3] - waited);
  m->host_us[2] += std::chrono::duration<double, std::micro>(t3 - t2).count();
  m->host_calls += 1;
  return RL_OK;
}

rl_status rl_profile_host_read(rl_model* m, double* admit_us, double* meta_us, double* launch_us, double* wait_us,
                               int64_t* calls) {
  if (!m || !admit_us || !meta_us || !launch_us || !wait_us || !calls) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  *admit_us = m->host_us[0]; *meta_us = m->host_us[1]; *launch_us = m->host_us[2]; *wait_us = m->host_us[3];
  *calls = m->host_calls;
  m->host_us[0] = m->host_us[1] = m->host_us[2] = m->host_us[3] = 0.0;
  m->host_calls = 0;
  return RL_OK;
}

rl_status rl_decode_graph_create(rl_model* m, int32_t n, const int32_t* seq_ids, const rl_sampling* sp,
                                 int32_t* out_tokens, float* out_logprobs, rl_decode_graph** out) {
  if (!m || !seq_ids || !sp || !out_tokens || !out_logprobs || !out) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  if (m->geo.vocab == 0) return fail(RL_ERR_UNSUPPORTED, "model has no vocabulary");
  if (n < 1 || n > (int32_t)m->cfg.max_rows) return fail(RL_ERR_INVALID_ARG, "n_seqs %d outside [1, max_rows=%u]", n, m->cfg.max_rows);
  if (m->graph_alive) return fail(RL_ERR_UNSUPPORTED, "one decode graph per model at a time");
  rl_decode_graph* g = new rl_decode_graph();
  g->m = m;
  g->ids.assign(seq_ids, seq_ids + n);
  g->sp = *sp;
  g->out_tokens = out_tokens;
  g->out_logprobs = out_logprobs;
  for (int b = 0; b < 2; ++b) {
    hipError_t e = hipHostMalloc((void**)&g->host[b], m->lay.slot_bytes, hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&g->ev[b], hipEventDisableTiming);
    if (e != hipSuccess) {
      rl_decode_graph_destroy(g);
      return fail(RL_ERR_DEVICE, "rl_decode_graph_create: %s", hipGetErrorString(e));
    }
    memset(g->host[b], 0, m->lay.slot_bytes);
  }
  m->graph_alive = true;
  *out = g;
  return RL_OK;
}

void rl_decode_graph_destroy(rl_decode_graph* g) {
  if (!g) return;
  for (int b = 0; b < 2; ++b) {
    if (g->ev[b]) { if (g->ev_used[b]) (void)hipEventSynchronize(g->ev[b]); (void)hipEventDestroy(g->ev[b]); }
    if (g->exec[b]) (void)hipGraphExecDestroy(g->exec[b]);
    if (g->host[b]) (void)hipHostFree(g->host[b]);
  }
  if (g->m) g->m->graph_alive = false;
  delete g;
}

rl_status rl_decode_graph_step(rl_decode_graph* g, void* stream, int64_t* captures_out) {
  if (!g) return fail(RL_ERR_INVALID_ARG, "graph is NULL");
  if (!stream) return fail(RL_ERR_INVALID_ARG, "the null stream cannot be captured: pass a stream created by the caller");
  rl_model* m = g->m;
  hipStream_t st = (hipStream_t)stream;
  const int n = (int)g->ids.size();
  rl_status rs = admit_decode(m, n, g->ids.data());
  if (rs != RL_OK) return rs;
  const int b = g->next;
  if (g->ev_used[b]) HIP_TRY(hipEventSynchronize(g->ev[b]));  // the launch that read this buffer last has finished
  char* hs = g->host[b];
  char* ds = m->ws + m->lay.ring + (size_t)(kRingCalls + b) * m->lay.slot_bytes;
  int max_ctx = 0;
  SharedAttn sa;
  const SlotUpload up = build_decode_meta(m, n, g->ids.data(), hs, ds, &max_ctx, &sa, true);
  const rl_decode_graph::Key key = {attn_capture_ctx(n, m->geo.n_kv, m->geo.kv_fp8, max_ctx, sa.n_sets > 0), sa.n_sets, (sa.max_segs + 3) / 4, sa.set_segs, sa.packs + sa.all_packed};
  if (!g->exec[b] || key.ctx != g->key[b].ctx || key.n_sets != g->key[b].n_sets ||
      key.set_blocks != g->key[b].set_blocks || key.set_segs != g->key[b].set_segs || key.packs != g->key[b].packs) {
    if (g->exec[b]) { (void)hipGraphExecDestroy(g->exec[b]); g->exec[b] = nullptr; }
    const bool prof = m->prof_on;
    m->prof_on = false;  // no event pairs inside a captured step
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      SharedAttn sa_cap = sa;
      sa_cap.max_segs = key.set_blocks * 4;  // the attention grid only takes its block count from it
      float* cap = m->geo.dtype == kBF16 ? m->capture : nullptr;
      launch_entry(st, m->geo.dtype, table_rows(m, hs, nullptr), up, m->wsp<float>(m->lay.x), m->attn_norm[0], m->wsp<void>(m->lay.h), cap,
                   n, m->geo.hidden, m->geo.rms_eps);
      decode_enqueue(m, st, n, (const RowMeta*)ds, key.ctx, sa_cap, nullptr, &g->sp, g->out_tokens, g->out_logprobs, nullptr);
      const hipError_t e_end = hipStreamEndCapture(st, &graph);  // always ends the capture
      if (e == hipSuccess) e = e_end;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&g->exec[b], graph, nullptr, nullptr, 0);
    if (graph) (void)hipGraphDestroy(graph);
    m->prof_on = prof;
    if (e != hipSuccess) { g->exec[b] = nullptr; return fail(RL_ERR_DEVICE, "rl_decode_graph_step: capture: %s", hipGetErrorString(e)); }
    g->key[b] = key;
    g->captures += 1;
  }
  HIP_TRY(hipGraphLaunch(g->exec[b], st));
  HIP_TRY(hipEventRecord(g->ev[b], st));
  g->ev_used[b] = true;
  for (int i = 0; i < n; ++i) m->table->set_len(g->ids[i], m->table->len(g->ids[i]) + 1);
  g->next = b ^ 1;
  if (captures_out) *captures_out = g->captures;
  return RL_OK;
}

rl_status rl_decode_hidden(rl_model* m, void* stream, int32_t n, const int32_t* seq_ids, const float* hidden_in,
                           float* hidden_out) {
  if (!m || !hidden_in || !hidden_out) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  hipStream_t st = (hipStream_t)stream;
  rl_status rs = admit_decode(m, n, seq_ids);
  if (rs != RL_OK) return rs;
  DecodeMeta dm;
  rs = prepare_decode_meta(m, n, seq_ids, &dm);
  if (rs != RL_OK) return rs;
  float* x = m->wsp<float>(m->lay.x);
  RowSource in;
  in.src = hidden_in;
  rs = enter_rows(m, st, dm.slot, in, dm.up, n);
  if (rs != RL_OK) return rs;
  const Pending pend = run_layers(m, st, n, dm.rows_dev, dm.max_ctx, dm.sa, true);
  float* cap = m->capture ? m->capture + (size_t)m->geo.n_layers * m->cfg.max_rows * m->geo.hidden : nullptr;
  // the last sums go straight to the caller's buffer, which may be the one the rows came from
  const bool direct = pend.n && (uintptr_t)hidden_out % 16 == 0;
  if (pend.n) {
    Timer t(m, st, K_NORM);
    launch_residual_norm(st, x, direct ? hidden_out : x, pend.part, pend.n, nullptr, nullptr, cap, n, m->geo.hidden, m->geo.rms_eps);
  } else {
    copy_capture(st, cap, x, n, m->geo.hidden);
  }
  if (!direct) HIP_TRY(hipMemcpyAsync(hidden_out, x, (size_t)n * m->geo.hidden * 4, hipMemcpyDeviceToDevice, st));
  HIP_TRY(hipGetLastError());
  for (int i = 0; i < n; ++i) m->table->set_len(seq_ids[i], m->table->len(seq_ids[i]) + 1);
  return RL_OK;
}

// Make each `dst` (valid id, inactive) a continuation of `src` (active) at `len` tokens: the pages that `len`
// tokens fill completely are shared, a partial last page is copied into a page of dst's own.  The caller has
// checked ids and free pages (one per dst when len % 16 != 0) and sets the lengths.  At most max_rows forks.
struct Fork { int32_t src, dst, len; };
static rl_status fork_seqs(rl_model* m, hipStream_t st, const std::vector<Fork>& forks) {
  SeqTable& T = *m->table;
  ForkBatch batch;
  batch.n = 0;
  auto flush = [&]() {
    launch_fork(st, batch, m->wsp<int32_t>(m->lay.block_table), m->geo.max_blocks, m->kv_pool, m->layer_kv_bytes,
                (size_t)m->geo.n_kv * 2 * m->kv_block_bytes, m->geo.n_layers);
    batch.n = 0;
  };
  for (const Fork& f : forks) {
    const int full = f.len / SeqTable::kBlock;
    T.activate(f.dst);
    T.share_prefix(f.dst, f.src, full);
    const bool partial = f.len % SeqTable::kBlock != 0;
    if (partial) T.reserve(f.dst, f.len);
    if (f.len == 0) continue;
    batch.f[batch.n++] = ForkBatch::One{f.src, f.dst, full, partial ? T.pages(f.dst)[full] : -1};
    if (batch.n == kForkBatch) flush();
  }
  if (batch.n) flush();
  return RL_OK;
}

// Prefill of n_prompts prompts, each followed by `group` sequences (seq_ids[i*group + j]).  Member 0 of a group
// runs the prompt; the others share every page the prompt fills completely and get a private copy of the partial
// last page, so the prompt's KV is computed and stored once per group.
static rl_status prefill_impl(rl_model* m, hipStream_t st, int32_t n_prompts, int32_t group, const int32_t* seq_ids,
                              const int32_t* prompt_tokens, const int32_t* prompt_lens, const rl_sampling* sp,
                              int32_t* out_tokens, float* out_logprobs) {
  if (m->geo.vocab == 0) return fail(RL_ERR_UNSUPPORTED, "model has no vocabulary");
  if (n_prompts < 1 || group < 1 || (int64_t)n_prompts * group > (int64_t)m->cfg.max_rows)
    return fail(RL_ERR_INVALID_ARG, "n_prompts %d x group %d outside [1, max_rows=%u]", n_prompts, group, m->cfg.max_rows);
  SeqTable& T = *m->table;
  const int n_all = n_prompts * group;
  const int R = (int)m->cfg.max_rows, H = m->geo.hidden;
  std::vector<char> seen(T.max_seqs(), 0);
  int64_t need = 0, total = 0;
  for (int i = 0; i < n_all; ++i) {
    const int32_t s = seq_ids[i];
    if (!T.valid_id(s)) return fail(RL_ERR_BAD_SEQ, "sequence id %d out of range", s);
    if (T.active(s)) return fail(RL_ERR_BAD_SEQ, "sequence %d is already active", s);
    if (seen[s]) return fail(RL_ERR_INVALID_ARG, "sequence %d appears twice", s);
    seen[s] = 1;
  }
  for (int i = 0; i < n_prompts; ++i) {
    if (prompt_lens[i] < 1) return fail(RL_ERR_INVALID_ARG, "prompt %d is empty", i);
    if (prompt_lens[i] > T.max_ctx() - 1) return fail(RL_ERR_CTX_OVERFLOW, "prompt %d has %d tokens, max_ctx is %d", i, prompt_lens[i], T.max_ctx());
    need += SeqTable::blocks_for(prompt_lens[i]) + (int64_t)(group - 1) * ((prompt_lens[i] % SeqTable::kBlock) ? 1 : 0);
    total += prompt_lens[i];
  }
  for (int64_t i = 0; i < total; ++i)
    if (prompt_tokens[i] < 0 || prompt_tokens[i] >= m->geo.vocab) return fail(RL_ERR_INVALID_ARG, "token %d at %lld outside the vocabulary", prompt_tokens[i], (long long)i);
  if (need > T.free_pages()) return fail(RL_ERR_KV_FULL, "need %lld pages, %lld free", (long long)need, (long long)T.free_pages());

  // Everything below changes sequence state; if a HIP call fails half way, the ids this call activated are released
  // again (their pages return to the pool) before the error is reported.
  auto run = [&]() -> rl_status {
  for (int i = 0; i < n_prompts; ++i) {
    const int32_t s = seq_ids[i * group];
    T.activate(s);
    T.reserve(s, prompt_lens[i]);
  }

  // rows in (prompt, position) order, cut into chunks of R
  int pi = 0, pos = 0;
  int64_t done = 0, tok_off = 0;
  const RowMeta *tail = nullptr, *head = nullptr;  // device rows of the prompts' ends and of all sequences
  int max_len = 0;
  std::vector<int64_t> tok_base(n_prompts);
  for (int i = 0; i < n_prompts; ++i) { tok_base[i] = tok_off; tok_off += prompt_lens[i]; }
  while (done < total) {
    const int M = (int)std::min<int64_t>(R, total - done);
    int slot;
    rl_status rs = ring_acquire(m, &slot);
    if (rs != RL_OK) return rs;
    char* hs = m->host_ring + (size_t)slot * m->lay.host_slot_bytes;
    char* ds = m->ws + m->lay.ring + (size_t)slot * m->lay.slot_bytes;
    RowMeta* hr = (RowMeta*)hs;
    int32_t* ht = (int32_t*)(hs + m->lay.slot_tok);
    int max_ctx = 0;
    int32_t* ends_h = (int32_t*)(hs + m->lay.slot_upd);  // pairs: (row, prompt) of the rows that end a prompt
    PromptEnds ends;
    ends.pairs = (const int32_t*)(ds + m->lay.slot_upd);
    for (int r = 0; r < M; ++r) {
      hr[r].seq = seq_ids[pi * group];
      hr[r].pos = pos;
      hr[r].page = T.pages(hr[r].seq)[pos >> 4];
      hr[r].pad = 0;
      ht[r] = prompt_tokens[tok_base[pi] + pos];
      if (pos + 1 > max_ctx) max_ctx = pos + 1;
      if (pos + 1 == prompt_lens[pi]) { ends_h[2 * ends.n] = r; ends_h[2 * ends.n + 1] = pi; ++ends.n; ++pi; pos = 0; }
      else ++pos;
    }
    SharedAttn sa;
    SlotUpload up = slot_upload(m, hs, ds, M, true);
    place_window_plan(m, hs, ds, M, hr, &sa, &up);
    if (ends.n) add_region(&up, m->lay.slot_upd, (size_t)ends.n * 8);
    done += M;
    if (done == total) {  // the rows of the last passes travel with those of the last chunk
      RowMeta* ht_tail = (RowMeta*)(hs + m->lay.slot_tail);
      RowMeta* ht_head = (RowMeta*)(hs + m->lay.slot_head);
      for (int i = 0; i < n_prompts; ++i) {
        const int32_t s = seq_ids[i * group], last = prompt_lens[i] - 1;
        ht_tail[i] = RowMeta{s, last, T.pages(s)[last >> 4], 0};
        max_len = std::max(max_len, prompt_lens[i]);
      }
      for (int i = 0; i < n_all; ++i) ht_head[i] = RowMeta{seq_ids[i], prompt_lens[i / group], 0, 0};
      add_region(&up, m->lay.slot_tail, (size_t)n_prompts * sizeof(RowMeta));
      add_region(&up, m->lay.slot_head, (size_t)n_all * sizeof(RowMeta));
      tail = (const RowMeta*)(ds + m->lay.slot_tail);
      head = (const RowMeta*)(ds + m->lay.slot_head);
    }
    rs = enter_rows(m, st, slot, table_rows(m, hs, ht), up, M);
    if (rs != RL_OK) return rs;
    const Pending pend = run_layers(m, st, M, (const RowMeta*)ds, max_ctx, sa, false, &ends);
    if (m->capture) {  // the boundary behind the last layer
      float* x = m->wsp<float>(m->lay.x);
      float* cap = m->capture + (size_t)m->geo.n_layers * m->cfg.max_rows * H;
      if (pend.n) launch_residual_norm(st, x, x, pend.part, pend.n, nullptr, nullptr, cap, M, H, m->geo.rms_eps);
      else copy_capture(st, cap, x, M, H);
    }
  }

  // ---- the last rows of all prompts through the rest of the last layer -------------------------------------
  float* x_last = m->wsp<float>(m->lay.x_last);
  const Pending pend = finish_layer(m, st, m->geo.n_layers - 1, n_prompts, tail, max_len, SharedAttn(), m->wsp<float>(m->lay.q_last), nullptr, x_last);

  // ---- the other members of each group: shared full pages, private copy of the partial page ---------------
  if (group > 1) {
    std::vector<Fork> forks;
    for (int i = 0; i < n_prompts; ++i)
      for (int j = 1; j < group; ++j) forks.push_back({seq_ids[i * group], seq_ids[i * group + j], prompt_lens[i]});
    rl_status rs = fork_seqs(m, st, forks);
    if (rs != RL_OK) return rs;
  }

  // logits at the last prompt position of every sequence; the sampled token sits at position prompt_len
  float* keep = m->capture;
  m->capture = nullptr;  // slot n_layers was already written per chunk
  run_head(m, st, n_all, x_last, pend, head, 0, nullptr, sp, out_tokens, out_logprobs, nullptr, false, group);
  m->capture = keep;
  HIP_TRY(hipGetLastError());
  for (int i = 0; i < n_all; ++i) T.set_len(seq_ids[i], prompt_lens[i / group]);
  return RL_OK;
  };
  const rl_status rs = run();
  if (rs != RL_OK)
    for (int i = 0; i < n_all; ++i)
      if (T.active(seq_ids[i])) T.release(seq_ids[i]);  // all were inactive on entry
  return rs;
}

rl_status rl_prefill(rl_model* m, void* stream, int32_t n, const int32_t* seq_ids, const int32_t* prompt_tokens,
                     const int32_t* prompt_lens, const rl_sampling* sp, int32_t* out_tokens, float* out_logprobs) {
  if (!m || !seq_ids || !prompt_tokens || !prompt_lens || !sp || !out_tokens || !out_logprobs)
    return fail(RL_ERR_INVALID_ARG, "NULL argument");
  return prefill_impl(m, (hipStream_t)stream, n, 1, seq_ids, prompt_tokens, prompt_lens, sp, out_tokens, out_logprobs);
}

rl_status rl_prefill_groups(rl_model* m, void* stream, int32_t n_prompts, int32_t group_size, const int32_t* seq_ids,
                            const int32_t* prompt_tokens, const int32_t* prompt_lens, const rl_sampling* sp,
                            int32_t* out_tokens, float* out_logprobs) {
  if (!m || !seq_ids || !prompt_tokens || !prompt_lens || !sp || !out_tokens || !out_logprobs)
    return fail(RL_ERR_INVALID_ARG, "NULL argument");
  return prefill_impl(m, (hipStream_t)stream, n_prompts, group_size, seq_ids, prompt_tokens, prompt_lens, sp, out_tokens,
                      out_logprobs);
}

rl_status rl_seq_fork(rl_model* m, void* stream, int32_t src_seq, int32_t n, const int32_t* new_seq_ids) {
  if (!m || !new_seq_ids) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  if (n < 1 || n > (int32_t)m->cfg.max_rows) return fail(RL_ERR_INVALID_ARG, "n %d outside [1, max_rows=%u]", n, m->cfg.max_rows);
  SeqTable& T = *m->table;
  if (!T.active(src_seq)) return fail(RL_ERR_BAD_SEQ, "sequence %d is not active", src_seq);
  std::vector<char> seen(T.max_seqs(), 0);
  for (int i = 0; i < n; ++i) {
    const int32_t s = new_seq_ids[i];
    if (!T.valid_id(s)) return fail(RL_ERR_BAD_SEQ, "sequence id %d out of range", s);
    if (T.active(s)) return fail(RL_ERR_BAD_SEQ, "sequence %d is already active", s);
    if (seen[s]) return fail(RL_ERR_INVALID_ARG, "sequence %d appears twice", s);
    seen[s] = 1;
  }
  const int32_t len = T.len(src_seq);
  const int64_t need = (len % SeqTable::kBlock) ? n : 0;
  if (need > T.free_pages()) return fail(RL_ERR_KV_FULL, "need %lld pages, %lld free", (long long)need, (long long)T.free_pages());
  std::vector<Fork> forks;
  for (int i = 0; i < n; ++i) forks.push_back({src_seq, new_seq_ids[i], len});
  rl_status rs = fork_seqs(m, (hipStream_t)stream, forks);
  if (rs == RL_OK && hipGetLastError() != hipSuccess) rs = fail(RL_ERR_DEVICE, "rl_seq_fork: kernel launch failed");
  if (rs != RL_OK) {  // release what was activated (all new ids were inactive on entry)
    for (int i = 0; i < n; ++i)
      if (T.active(new_seq_ids[i])) T.release(new_seq_ids[i]);
    return rs;
  }
  for (int i = 0; i < n; ++i) T.set_len(new_seq_ids[i], len);
  return RL_OK;
}

rl_status rl_score(rl_model* m, void* stream, int32_t n, const int32_t* seq_ids, const int32_t* tokens,
                   const int32_t* lens, float temperature, float* out_logprobs) {
  if (!m || !seq_ids || !tokens || !lens || !out_logprobs) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  if (m->geo.vocab == 0) return fail(RL_ERR_UNSUPPORTED, "model has no vocabulary");
  if (n < 1 || n > T_MAX_SCORE) return fail(RL_ERR_INVALID_ARG, "n_seqs %d outside [1, %d]", n, T_MAX_SCORE);
  hipStream_t st = (hipStream_t)stream;
  SeqTable& T = *m->table;
  const int R = (int)m->cfg.max_rows, H = m->geo.hidden;
  std::vector<char> seen(T.max_seqs(), 0);
  int64_t need = 0, total = 0;
  for (int i = 0; i < n; ++i) {
    const int32_t s = seq_ids[i];
    if (!T.valid_id(s)) return fail(RL_ERR_BAD_SEQ, "sequence id %d out of range", s);
    if (T.active(s)) return fail(RL_ERR_BAD_SEQ, "sequence %d is already active", s);
    if (seen[s]) return fail(RL_ERR_INVALID_ARG, "sequence %d appears twice", s);
    seen[s] = 1;
    if (lens[i] < 2) return fail(RL_ERR_INVALID_ARG, "sequence %d has fewer than 2 tokens", i);
    if (lens[i] > T.max_ctx()) return fail(RL_ERR_CTX_OVERFLOW, "sequence %d has %d tokens, max_ctx is %d", i, lens[i], T.max_ctx());
    need += SeqTable::blocks_for(lens[i]);
    total += lens[i];
  }
  for (int64_t i = 0; i < total; ++i)
    if (tokens[i] < 0 || tokens[i] >= m->geo.vocab) return fail(RL_ERR_INVALID_ARG, "token %d at %lld outside the vocabulary", tokens[i], (long long)i);
  if (need > T.free_pages()) return fail(RL_ERR_KV_FULL, "need %lld pages, %lld free", (long long)need, (long long)T.free_pages());

  rl_status result = RL_OK;
  for (int i = 0; i < n; ++i) {
    T.activate(seq_ids[i]);
    T.reserve(seq_ids[i], lens[i]);
  }
  float* x = m->wsp<float>(m->lay.x);
  int32_t* tmp_tok = m->wsp<int32_t>(m->lay.tmp_tok);
  float* tmp_lp = m->wsp<float>(m->lay.tmp_lp);
  rl_sampling sp{temperature, 0u, 0ull, 0.f, 0u};
  int si = 0, pos = 0;
  int64_t done = 0, tok_off = 0, out_off = 0;
  std::vector<int64_t> tok_base(n), out_base(n);
  for (int i = 0; i < n; ++i) { tok_base[i] = tok_off; tok_off += lens[i]; out_base[i] = out_off; out_off += lens[i] - 1; }
  while (done < total && result == RL_OK) {
    const int M = (int)std::min<int64_t>(R, total - done);
    int slot;
    result = ring_acquire(m, &slot);
    if (result != RL_OK) break;
    char* hs = m->host_ring + (size_t)slot * m->lay.host_slot_bytes;
    char* ds = m->ws + m->lay.ring + (size_t)slot * m->lay.slot_bytes;
    RowMeta* hr = (RowMeta*)hs;
    int32_t* ht = (int32_t*)(hs + m->lay.slot_tok);
    int32_t* hf = (int32_t*)(hs + m->lay.slot_upd);  // [0,M): token to score, [M,2M): output index or -1
    int max_ctx = 0;
    for (int r = 0; r < M; ++r) {
      hr[r].seq = seq_ids[si];
      hr[r].pos = pos;
      hr[r].page = T.pages(hr[r].seq)[pos >> 4];
      hr[r].pad = 0;
      ht[r] = tokens[tok_base[si] + pos];
      if (pos + 1 > max_ctx) max_ctx = pos + 1;
      if (pos + 1 == lens[si]) { hf[r] = 0; hf[M + r] = -1; ++si; pos = 0; }
      else { hf[r] = tokens[tok_base[si] + pos + 1]; hf[M + r] = (int32_t)(out_base[si] + pos); ++pos; }
    }
    SharedAttn sa;
    SlotUpload up = slot_upload(m, hs, ds, M, true);
    place_window_plan(m, hs, ds, M, hr, &sa, &up);
    add_region(&up, m->lay.slot_upd, (size_t)2 * M * 4);
    result = enter_rows(m, st, slot, table_rows(m, hs, ht), up, M);
    if (result != RL_OK) break;
    const RowMeta* rows = (const RowMeta*)ds;
    const int32_t* forced = (const int32_t*)(ds + m->lay.slot_upd);
    const Pending pend = run_layers(m, st, M, rows, max_ctx, sa);
    run_head(m, st, M, x, pend, rows, 1, forced, &sp, tmp_tok, tmp_lp, nullptr, true);
    launch_scatter_f32(st, tmp_lp, forced + M, out_logprobs, M);
    done += M;
  }
  if (result == RL_OK && hipGetLastError() != hipSuccess) result = fail(RL_ERR_DEVICE, "kernel launch failed");
  // the sequences were only scratch: later work on this stream is ordered after the kernels above
  for (int i = 0; i < n; ++i) T.release(seq_ids[i]);
  return result;
}

// Append n_tokens positions of given K/V to the active sequence seq_id (length `len` >= 0): pages, block table,
// scatter kernels.  The caller has validated ids, sizes and free pages.
static rl_status append_kv(rl_model* m, hipStream_t st, int32_t seq_id, int32_t n_tokens, const void* const* k_layers,
                           const void* const* v_layers) {
  SeqTable& T = *m->table;
  const int32_t len = T.len(seq_id);
  const size_t have = T.pages(seq_id).size();
  T.reserve(seq_id, len + n_tokens);
  int32_t* bt_row = m->wsp<int32_t>(m->lay.block_table) + (size_t)seq_id * m->geo.max_blocks;
  if (n_tokens > 0) {
    const size_t now = T.pages(seq_id).size();
    // pageable source: the runtime stages it before returning, so the vector may change afterwards
    if (now > have)
      HIP_TRY(hipMemcpyAsync(bt_row + have, T.pages(seq_id).data() + have, (now - have) * 4, hipMemcpyHostToDevice, st));
    for (int l = 0; l < m->geo.n_layers; ++l)
      launch_kv_import(st, m->geo, k_layers[l], v_layers[l], len, n_tokens, bt_row, m->k_pool(l), m->v_pool(l));
  }
  HIP_TRY(hipGetLastError());
  T.set_len(seq_id, len + n_tokens);
  return RL_OK;
}

rl_status rl_seq_import_kv(rl_model* m, void* stream, int32_t seq_id, int32_t n_tokens, const void* const* k_layers,
                           const void* const* v_layers) {
  if (!m || !k_layers || !v_layers) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  SeqTable& T = *m->table;
  if (!T.valid_id(seq_id)) return fail(RL_ERR_BAD_SEQ, "sequence id %d out of range", seq_id);
  if (T.active(seq_id)) return fail(RL_ERR_BAD_SEQ, "sequence %d is already active", seq_id);
  if (n_tokens < 0 || n_tokens > T.max_ctx() - 1) return fail(RL_ERR_CTX_OVERFLOW, "n_tokens %d outside [0, max_ctx)", n_tokens);
  for (int l = 0; l < m->geo.n_layers; ++l)
    if (n_tokens > 0 && (!k_layers[l] || !v_layers[l])) return fail(RL_ERR_INVALID_ARG, "layer %d KV pointer is NULL", l);
  if (SeqTable::blocks_for(n_tokens) > T.free_pages()) return fail(RL_ERR_KV_FULL, "need %d pages, %lld free", SeqTable::blocks_for(n_tokens), (long long)T.free_pages());
  T.activate(seq_id);
  const rl_status rs = append_kv(m, (hipStream_t)stream, seq_id, n_tokens, k_layers, v_layers);
  if (rs != RL_OK) T.release(seq_id);
  return rs;
}

rl_status rl_seq_append_kv(rl_model* m, void* stream, int32_t seq_id, int32_t n_tokens, const void* const* k_layers,
                           const void* const* v_layers) {
  if (!m || !k_layers || !v_layers) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  SeqTable& T = *m->table;
  if (!T.active(seq_id)) return fail(RL_ERR_BAD_SEQ, "sequence %d is not active", seq_id);
  if (n_tokens < 1) return fail(RL_ERR_INVALID_ARG, "n_tokens %d < 1", n_tokens);
  if ((int64_t)T.len(seq_id) + n_tokens > T.max_ctx() - 1)
    return fail(RL_ERR_CTX_OVERFLOW, "sequence %d would hold %lld tokens, max_ctx is %d", seq_id, (long long)T.len(seq_id) + n_tokens, T.max_ctx());
  for (int l = 0; l < m->geo.n_layers; ++l)
    if (!k_layers[l] || !v_layers[l]) return fail(RL_ERR_INVALID_ARG, "layer %d KV pointer is NULL", l);
  const int missing = T.pages_missing(seq_id, T.len(seq_id) + n_tokens);
  if (missing > T.free_pages()) return fail(RL_ERR_KV_FULL, "need %d pages, %lld free", missing, (long long)T.free_pages());
  return append_kv(m, (hipStream_t)stream, seq_id, n_tokens, k_layers, v_layers);
}

rl_status rl_sample_logits(rl_model* m, void* stream, int32_t n, const float* logits, const int32_t* seq_ids,
                           const int32_t* positions, const int32_t* forced, const rl_sampling* sp, int32_t* out_tokens,
                           float* out_logprobs) {
  if (!m || !logits || !seq_ids || !positions || !sp || !out_tokens || !out_logprobs) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  if (m->geo.vocab == 0) return fail(RL_ERR_UNSUPPORTED, "model has no vocabulary");
  if (n < 1 || n > (int32_t)m->cfg.max_rows) return fail(RL_ERR_INVALID_ARG, "n %d outside [1, max_rows]", n);
  hipStream_t st = (hipStream_t)stream;
  int slot;
  rl_status rs = ring_acquire(m, &slot);
  if (rs != RL_OK) return rs;
  char* hs = m->host_ring + (size_t)slot * m->lay.host_slot_bytes;
  char* ds = m->ws + m->lay.ring + (size_t)slot * m->lay.slot_bytes;
  RowMeta* hr = (RowMeta*)hs;
  for (int i = 0; i < n; ++i) { hr[i].seq = seq_ids[i]; hr[i].pos = positions[i]; hr[i].page = 0; hr[i].pad = 0; }
  HIP_TRY(hipMemcpyAsync(ds, hs, (size_t)n * sizeof(RowMeta), hipMemcpyHostToDevice, st));
  if ((rs = slot_in_use(m, st, slot)) != RL_OK) return rs;
  launch_sample(st, logits, n, m->geo.vocab, (const RowMeta*)ds, 0, forced, sp->temperature, sp->seed,
                m->wsp<float>(m->lay.samp_part), m->wsp<float>(m->lay.forced_z), out_tokens, out_logprobs,
                sp->top_k > (uint32_t)m->geo.vocab ? 0 : (int)sp->top_k, sp->top_p, m->wsp<void>(m->lay.cuts));
  HIP_TRY(hipGetLastError());
  return RL_OK;
}

rl_status rl_pack_weight(void* stream, uint32_t dtype, uint32_t kind, const void* src, void* dst, int64_t rows, int64_t cols) {
  if (!src || !dst || rows < 1 || cols < 1) return fail(RL_ERR_INVALID_ARG, "bad arguments");
  if (kind != RL_W_SPLIT_K && kind != RL_W_WHOLE_K) return fail(RL_ERR_INVALID_ARG, "unknown weight kind %u", kind);
  hipStream_t st = (hipStream_t)stream;
  if (dtype == RL_F32) {
    HIP_TRY(hipMemcpyAsync(dst, src, (size_t)rows * cols * 4, hipMemcpyDeviceToDevice, st));
    return RL_OK;
  }
  if (dtype != RL_BF16) return fail(RL_ERR_INVALID_ARG, "unknown dtype");
  if (rows % 64 || cols % 256 || rows > 0x7fffffff || cols > 0x7fffffff) return fail(RL_ERR_UNSUPPORTED, "bf16 packing needs rows %% 64 == 0 and cols %% 256 == 0");
  launch_pack_weight_bf16(st, src, dst, (int)rows, (int)cols, gemm_bf16_weight_segment((int)rows, (int)cols, kind == RL_W_SPLIT_K));
  HIP_TRY(hipGetLastError());
  return RL_OK;
}

rl_status rl_profile_enable(rl_model* m, int32_t on) {
  if (!m) return fail(RL_ERR_INVALID_ARG, "model is NULL");
  m->prof_on = on != 0;
  return RL_OK;
}

rl_status rl_profile_read(rl_model* m, int32_t n_max, const char** names_out, double* ms_out, int64_t* counts_out,
                          int32_t* n_out) {
  if (!m || !names_out || !ms_out || !counts_out || !n_out) return fail(RL_ERR_INVALID_ARG, "NULL argument");
  for (auto& p : m->pending) {
    HIP_TRY(hipEventSynchronize(p.b));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, p.a, p.b));
    m->prof_ms[p.kind] += ms;
    m->prof_n[p.kind] += 1;
    m->ev_pool.push_back(p.a);
    m->ev_pool.push_back(p.b);
  }
  m->pending.clear();
  int k = 0;
  for (int i = 0; i < K_COUNT && k < n_max; ++i) {
    names_out[k] = kKindNames[i];
    ms_out[k] = m->prof_ms[i];
    counts_out[k] = m->prof_n[i];
    m->prof_ms[i] = 0;
    m->prof_n[i] = 0;
    ++k;
  }
  *n_out = k;
  return RL_OK;
}

}  // extern "C"

// C wrappers around the host sequence table so that its logic can be exercised without a GPU.
// Built with g++ into its own small library by the CPU tests; not part of the product library.
#include "attn_plan.h"
#include "cut_plan.h"
#include "gemm_plan.h"
#include "seq_table.h"
#include "weight_order.h"

extern "C" {

void* st_create(int max_seqs, int max_ctx, long long n_pages) { return new rl::SeqTable(max_seqs, max_ctx, n_pages); }
void st_destroy(void* t) { delete (rl::SeqTable*)t; }
long long st_free_pages(void* t) { return ((rl::SeqTable*)t)->free_pages(); }
int st_active(void* t, int s) { return ((rl::SeqTable*)t)->active(s) ? 1 : 0; }
int st_len(void* t, int s) { return ((rl::SeqTable*)t)->len(s); }
int st_pages_missing(void* t, int s, int tokens) { return ((rl::SeqTable*)t)->pages_missing(s, tokens); }
void st_activate(void* t, int s) { ((rl::SeqTable*)t)->activate(s); }
void st_set_len(void* t, int s, int n) { ((rl::SeqTable*)t)->set_len(s, n); }
void st_release(void* t, int s) { ((rl::SeqTable*)t)->release(s); }
void st_shuffle(void* t, unsigned long long seed) { ((rl::SeqTable*)t)->shuffle_free(seed); }
void st_share_prefix(void* t, int dst, int src, int n_blocks) { ((rl::SeqTable*)t)->share_prefix(dst, src, n_blocks); }
int st_refcount(void* t, int page) { return ((rl::SeqTable*)t)->refcount(page); }
int st_n_seq_pages(void* t, int s) { return (int)((rl::SeqTable*)t)->pages(s).size(); }
int st_seq_page(void* t, int s, int i) { return ((rl::SeqTable*)t)->pages(s)[i]; }
// returns the number of pages added; what fits of them as (seq, block, page) triples
int st_reserve(void* t, int s, int tokens, int* added_out, int max_added) {
  auto* T = (rl::SeqTable*)t;
  const int before = (int)T->pages(s).size();
  T->reserve(s, tokens);
  const std::vector<int32_t>& pages = T->pages(s);
  for (int n = 0; n < max_added && before + n < (int)pages.size(); ++n) {
    added_out[3 * n] = s; added_out[3 * n + 1] = before + n; added_out[3 * n + 2] = pages[before + n];
  }
  return (int)pages.size() - before;
}

long long st_prefix_id(void* t, int s) { return ((rl::SeqTable*)t)->prefix_id(s); }
int st_prefix_blocks(void* t, int s) { return ((rl::SeqTable*)t)->prefix_blocks(s); }
int st_weight_kb_slot(int kb, int seg) { return rl::weight_kb_slot(kb, seg); }
int st_attn_alone_up_to(int n_rows, int n_kv, int group) { return rl::attn_alone_up_to(n_rows, n_kv, group); }
int st_attn_rows_per_set(int group, int kv_fp8, int n_rows, int n_kv) {
  return rl::attn_rows_per_set(group, kv_fp8 != 0, n_rows, n_kv);
}
// segments up to which one block takes a row, segments of a block beyond
void st_attn_split(int n_rows, int n_kv, int kv_fp8, int max_ctx, int sets, int segs_per_block, int* out) {
  const rl::AttnSplit r = rl::attn_split(n_rows, n_kv, kv_fp8 != 0, max_ctx, sets != 0, segs_per_block);
  out[0] = r.whole_segs;
  out[1] = r.spb;
}
int st_attn_capture_ctx(int n_rows, int n_kv, int kv_fp8, int max_ctx, int sets) {
  return rl::attn_capture_ctx(n_rows, n_kv, kv_fp8 != 0, max_ctx, sets != 0);
}
int st_attn_num_segments(int ctx) { return rl::attn_num_segments(ctx); }
int st_attn_seg_begin(int sgm, int ctx) { return rl::attn_seg_begin(sgm, (ctx + 31) >> 5, rl::attn_num_segments(ctx)); }
// plan of one decode batch: skip_out[n]; sets_out gets (rows[8], n_rows, n_segs) per set; returns the number of sets
int st_plan_shared(void* t, int n, const int* seq_ids, const int* pos, int rows_per_set, int* skip_out, int* sets_out,
                   int max_sets) {
  auto* T = (rl::SeqTable*)t;
  std::vector<int64_t> fam(n);
  std::vector<int32_t> blocks(n);
  for (int i = 0; i < n; ++i) { fam[i] = T->prefix_id(seq_ids[i]); blocks[i] = T->prefix_blocks(seq_ids[i]); }
  rl::AttnPlan plan;
  rl::plan_shared_attention(n, fam.data(), blocks.data(), pos, rows_per_set, &plan);
  for (int i = 0; i < n; ++i) skip_out[i] = plan.skip[i];
  for (size_t k = 0; k < plan.sets.size() && (int)k < max_sets; ++k) {
    for (int e = 0; e < rl::kAttnSetRows; ++e) sets_out[10 * k + e] = plan.sets[k].rows[e];
    sets_out[10 * k + 8] = plan.sets[k].n_rows;
    sets_out[10 * k + 9] = plan.sets[k].n_segs;
  }
  return (int)plan.sets.size();
}

// segments of a set block of n rows in n_sets sets of up to max_segs segments; alone: some row is in none; packs: packed segments
int st_attn_set_segments(int n, int n_kv, int kv_fp8, int n_sets, int max_segs, int alone, int packs) {
  rl::AttnPlan plan;
  plan.skip.assign(n, max_segs);
  if (alone) plan.skip[n - 1] = 0;
  plan.sets.resize(n_sets);
  plan.max_shared_segs = max_segs;
  plan.packs = packs;
  return rl::attn_set_segments(n, n_kv, kv_fp8 != 0, plan);
}

// what is left behind the shared segments of n rows (skip[r] of them, 0: in no set): skip is updated, sets_out gets the packs
// behind n_sets sets; returns the entries, and in *all whether no row is left
int st_plan_packs(int n, const int* pos, int n_kv, int group, int min_pairs, int max_entries, int padded, int n_sets, int* skip,
                  int* sets_out, int* all) {
  rl::AttnPlan plan;
  plan.skip.assign(skip, skip + n);
  plan.sets.resize(n_sets);
  rl::plan_packs(n, pos, n_kv, group, min_pairs, max_entries, padded != 0, &plan);
  for (int i = 0; i < n; ++i) skip[i] = plan.skip[i];
  for (size_t k = n_sets; k < plan.sets.size(); ++k) {
    int* o = sets_out + 10 * (k - n_sets);
    for (int e = 0; e < rl::kAttnSetRows; ++e) o[e] = plan.sets[k].rows[e];
    o[8] = plan.sets[k].n_rows;
    o[9] = plan.sets[k].n_segs;
  }
  *all = plan.all_packed;
  return plan.packs;
}

// the staged kernel's tile of a projection of more than 64 rows: (row blocks, waves, whether one block walks the whole K range, row blocks
// of the matrix); returns 0 where its K quarters are not rounds of four k blocks, i.e. another kernel takes it
int st_gemm_tile(int M, int N, int K, int epi, int* out) {
  const bool split = epi == rl::kEpiPartial || epi == rl::kEpiResidual;
  const rl::GemmTile t = rl::gemm_tile(M, N, K, epi, split);
  out[0] = t.nb;
  out[1] = t.nw;
  out[2] = rl::gemm_whole_k(M, N, K, epi, split) ? 1 : 0;
  out[3] = epi == rl::kEpiSwiGLU ? N >> 4 : N >> 5;
  return rl::gemm_plan(N, K, split ? rl::kEpiPartial : epi, split).kb_per_wave % 4 == 0;
}

// slices of truncated sampling, units of 256 logits per slice, whether the units' largest logits are kept
int st_cut_slices(int n_rows, int vocab) { return rl::cut_slices(n_rows, vocab); }
int st_cut_units(int vocab, int slices) { return rl::cut_units_per_slice(vocab, slices); }
int st_cut_keeps_units(int vocab, int slices) { return rl::cut_keeps_units(vocab, slices) ? 1 : 0; }

int st_plan_windows(int n, const int* seq, const int* pos, int rows_per_set, int* skip_out, int* sets_out, int max_sets) {
  rl::AttnPlan plan;
  rl::plan_window_sets(n, seq, pos, rows_per_set, &plan);
  for (int i = 0; i < n; ++i) skip_out[i] = plan.skip[i];
  for (size_t k = 0; k < plan.sets.size() && (int)k < max_sets; ++k) {
    for (int e = 0; e < rl::kAttnSetRows; ++e) sets_out[10 * k + e] = plan.sets[k].rows[e];
    sets_out[10 * k + 8] = plan.sets[k].n_rows;
    sets_out[10 * k + 9] = plan.sets[k].n_segs;
  }
  return (int)plan.sets.size();
}

}  // extern "C"

// The rules of csrc/batch_rules.hpp for tests, with the arguments that the library calls them with.
#include "../paper_2505_12658_amd/csrc/batch_rules.hpp"

extern "C" {
int halved_items(int head_dim, int batch, int total_tokens, int n_q_heads, int n_kv_heads, int compute_units) {
  return hydra::rules::halved_items(head_dim, batch, total_tokens, n_q_heads, n_kv_heads, (unsigned)compute_units);
}
int loading_waves(int causal, int batch, int total_tokens, int max_seqlen, int n_q_heads, int n_kv_heads, int compute_units) {
  return hydra::rules::loading_waves(causal != 0, batch, total_tokens, max_seqlen, n_q_heads, n_kv_heads, (unsigned)compute_units);
}
// workgroups of a hybrid batch's wide grid, 0 where it is not taken
int64_t wide_workgroups(int batch, int total_q, int max_q_len, int group, int n_kv_heads, int n_splits, int64_t table_keys) {
  const hydra::rules::WideGrid g = hydra::rules::wide_grid({batch, total_q, max_q_len, group, n_kv_heads, n_splits, table_keys});
  return g.use ? g.workgroups : 0;
}
}

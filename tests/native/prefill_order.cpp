// The prefill attention's workgroup order (csrc/prefill_order.h) for the host
// tests: the order of a call, and every workgroup's (group, block); and the
// workgroups per group of the fp64 re-score (csrc/band_grid.h).
#include "band_grid.h"
#include "prefill_order.h"

extern "C" void prefill_order_of(int n_seq, int n_kv_heads, int G, int d, int max_len, long long* o) {
  const snap::PrefillOrder p = snap::prefill_order(n_seq, n_kv_heads, G, d, max_len);
  o[0] = p.waves;
  o[1] = p.P;
  o[2] = p.n_qblocks;
  o[3] = p.groups;
  o[4] = p.whole;
  o[5] = p.grid;
}

extern "C" int band_workgroups_of(int d_qk, int groups) { return snap::band_workgroups(d_qk, groups); }

extern "C" bool prefill_fits(long long groups, int G, int max_len) { return snap::prefill_grid_fits(groups, G, max_len); }

extern "C" void prefill_blocks_of(int n_seq, int n_kv_heads, int G, int d, int max_len, int* group, int* block) {
  const snap::PrefillOrder p = snap::prefill_order(n_seq, n_kv_heads, G, d, max_len);
  for (int i = 0; i < p.grid; ++i) snap::prefill_block(p, i, group[i], block[i]);
}

// C entries to host rules of libbcd that need no GPU, for test_host_rules.py.
#include <cstring>

#include "../paper_1708_08739_amd/csrc/bcd_host_internal.h"

using namespace bcd;

extern "C" {

// Level-0 slots of sources 0 .. k-1 (internal ids = vertex ids) staged on a
// workspace of G groups and P partitions whose light lists hold capP items
// each; bounds[2 i], bounds[2 i + 1]: the region of source i's list.
void staged_slots(int64_t n, int G, int P, uint64_t capP, uint32_t H, int k, uint64_t *slot, uint64_t *bounds) {
  Graph g;
  g.n = n;
  g.rank.resize((size_t)n);
  for (int64_t v = 0; v < n; ++v) g.rank[(size_t)v] = (int32_t)v;
  Workspace ws;
  ws.graph = &g;
  ws.n = n;
  ws.G = G;
  std::memset(&ws.S, 0, sizeof(ws.S));
  BatchState &S = ws.S;
  S.n = n;
  S.G = G;
  S.P = P;
  S.NL = Workspace::lists(P);
  S.H = H;
  S.capP = capP;
  S.hbase = capP * (uint64_t)P;
  S.capH = (uint64_t)((G + P - 1) / P) * H * kLanes;
  std::vector<uint32_t> items((size_t)k), dest((size_t)k);
  std::vector<unsigned long long> masks((size_t)k);
  std::vector<int32_t> src((size_t)k);
  for (int i = 0; i < k; ++i) src[(size_t)i] = i;
  ws.h_items0 = items.data();
  ws.h_masks0 = masks.data();
  ws.h_dest0 = dest.data();
  ws.stage_sources(src.data(), k);
  BatchState T = S;
  T.P = ws.batch_parts(k);
  T.NL = Workspace::lists(T.P);
  for (int i = 0; i < k; ++i) {
    const int l = list_of(T, (uint32_t)(i / kLanes), (uint32_t)i);
    slot[i] = level0_slot(T, items[(size_t)i], dest[(size_t)i]);
    bounds[2 * i] = list_begin(T, l);
    bounds[2 * i + 1] = list_end(T, l);
  }
  ws.h_items0 = nullptr;
  ws.h_masks0 = nullptr;
  ws.h_dest0 = nullptr;
}

// Sources per batch of a run of ns sources (pipelined_batch).
uint64_t sources_per_batch(int64_t m, int weighted, uint64_t ns, uint64_t width) {
  Graph g;
  g.m = m;
  g.weighted = weighted != 0;
  return pipelined_batch(&g, ns, width);
}

// Groups of a run's second workspace (second_groups).
int second_workspace_groups(int64_t m, int weighted, uint64_t ns, uint64_t sample_of, uint64_t width) {
  Graph g;
  g.m = m;
  g.weighted = weighted != 0;
  return second_groups(&g, ns, sample_of, width);
}

// Width of the pooled workspace a lease takes: pool[0 .. k-1] are the widths of
// the idle ones; 0 = a new one.  lo = 0: a call's own, else a run's second.
int leased_width(const int *pool, int k, int lo, int hi) {
  Graph g;
  for (int i = 0; i < k; ++i) {
    std::unique_ptr<Workspace> w(new Workspace());
    w->batch_ready = true;
    w->G = pool[i];
    g.release(std::move(w));
  }
  std::unique_ptr<Workspace> w = lo == 0 ? g.acquire() : g.acquire(lo, hi);
  return w->batch_ready ? w->G : 0;
}

// Workgroups of 256 threads of a reachability level on a configured shape.
int reach_grid(int block, int grid) {
  Launch L;
  L.block = block;
  L.grid = grid;
  return reach_level_grid(L);
}

// Whether a traversal of at least `levels` levels goes to one workgroup.
int one_workgroup(int64_t n, int64_t m, int64_t levels) {
  Graph g;
  g.n = n;
  g.m = m;
  g.lds_block_bytes = 160 * 1024;
  return reach_one_workgroup(&g, levels);
}

// Bytes of bitmap a traversal of `levels` levels brings to the host, checked
// first after `first` levels, then every eight.
uint64_t bitmap_bytes_copied(int64_t n, int64_t levels, int first) {
  const size_t bytes = ((size_t)n + 31) / 32 * 4;
  uint64_t total = 0;
  bool have = false;
  int chunk = first;
  for (int64_t level = chunk;; level += chunk) {
    have = reach_copies_bitmap(level, chunk, bytes);
    if (have) total += bytes;
    if (level > levels) break;
    chunk = 8;
  }
  return have ? total : total + bytes;
}

// Workgroups of a backward level; *light and *heavy receive those a partition
// deals to either side (list_view of the kernels).
int bwd_grid(int P, uint32_t H, int block, int grid, const uint32_t *cnt, const uint32_t *cleared, int *light, int *heavy) {
  BatchState S;
  std::memset(&S, 0, sizeof(S));
  S.P = P;
  S.H = H;
  Launch L;
  L.block = block;
  L.grid = grid;
  const int g = bwd_level_grid(S, L, cnt, cleared), nwg = g / P;
  *heavy = H == 0 ? 0 : (nwg < 6 ? 1 : nwg / 3);
  *light = nwg - *heavy;
  return g;
}

// The autotuner's candidates around base, at most `cap`; returns their number.
int tune_candidates(const bcd_config *base, int weighted, bcd_config *out, int cap) {
  const std::vector<bcd_config> v = tune_around(*base, weighted != 0);
  for (int i = 0; i < (int)v.size() && i < cap; ++i) out[i] = v[(size_t)i];
  return (int)v.size();
}

// Algorithmic and schedule-aware bytes (forward, backward) recorded for a run of
// the batched unweighted engine whose path counts are stored in `count_bytes`.
void profile_bytes(int count_bytes, const uint64_t *ctr, double *alg, double *sched) {
  Graph g;
  ProfAcc p, other;
  p.count_bytes = count_bytes;
  p.merge(other);
  record_profile(&g, p, ctr);
  for (int k = 0; k < 2; ++k) {
    alg[k] = g.prof[k].alg_bytes;
    sched[k] = g.prof[k].sched_bytes;
  }
}

uint64_t workspace_bytes(int64_t n, int64_t m, uint32_t heavy, int weighted, int groups) {
  Graph g;
  g.n = n;
  g.m = m;
  g.heavy = heavy;
  g.weighted = weighted != 0;
  return batch_workspace_bytes(&g, groups);
}

int short_rows(int64_t longest) {
  Graph g;
  g.longest_row = longest;
  return lds_short_rows(&g);
}

}  // extern "C"

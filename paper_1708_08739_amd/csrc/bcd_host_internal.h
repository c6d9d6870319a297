// Host-side objects of libbcd: the resident graph and per-call workspaces.
#pragma once

#include <algorithm>
#include <atomic>
#include <functional>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "../../include/bcd.h"
#include "bcd_internal.h"

// Error propagation inside the host layer.
#define HIPCHK(expr)                                  \
  do {                                                \
    hipError_t _e = (expr);                           \
    if (_e != hipSuccess) return hip_fail(_e, #expr); \
  } while (0)

#define STCHK(expr)              \
  do {                           \
    bcd_status _s = (expr);      \
    if (_s != BCD_OK) return _s; \
  } while (0)

// Body of every exported call: a C++ exception (an allocation failure in
// host code) becomes a status with its message; none crosses the C ABI.
#define BCD_GUARD_BEGIN try {
#define BCD_GUARD_END                                                   \
  }                                                                     \
  catch (const std::bad_alloc &) {                                      \
    return bcd::fail(BCD_ERR_OUT_OF_MEMORY, "host allocation failed"); \
  }                                                                     \
  catch (...) {                                                         \
    return bcd::fail(BCD_ERR_DEVICE, "unexpected host exception");     \
  }

namespace bcd {

constexpr int kCtrSlots = 8192;       // max workgroups of a traversal launch
constexpr int kLevelChunkMax = 64;    // level launches enqueued between host checks
constexpr int kDefaultItems = 2;      // frontier items per wavefront step, pushed levels
// Bottom-up threshold denominator of the unweighted forward (0: top-down
// only).  ms without / with bottom-up levels at 1/4, 1,000 sources: R-MAT 20 32.2 /
// 28.7, 19 15.7 / 14.0, 18 8.2 / 7.7, 17 5.9 / 4.9, 16 2.46 / 2.58 (exact 36.9 /
// 32.1), uniform graphs of 500,000 vertices 29.6 / 17.5, of 100,000 7.5 / 4.2, layers
// of 30,000 vertices (360,000 in all) 23.7 / 24.6.  The line lies where the
// kernels before these had it (R-MAT 16 then lost 4 %); it is part of the
// interface's default, so a smaller graph that gains sets bottom_up itself.
inline int default_bottom_up(int64_t n) { return n >= (int64_t(1) << 19) ? 4 : 0; }
// Top-down levels of the unweighted forward add path counts along DAG arcs
// (1) instead of pulling them over in-arcs (0).
constexpr int kDefaultPush = 0;
// Item-list partitions of a workspace of G groups: two where they split
// evenly (nearly so above 8), else one.  More partitions keep a group's masks
// in fewer L2s, but groups are unlike (a batch's neighbouring sources are
// alike, so one group's wide levels fall on others' empty ones), and the
// workgroups of a partition without work wait for the launch's end.  8 / 4 / 2 /
// 1 partitions, ms: R-MAT 20 with 1,000 sources 33.8 / 29.6 / 26.5 / 27.0, R-MAT
// 16 with 1,000 2.65 / 2.45 / 2.35 / 2.28, exact (96 groups a batch: one list's
// counters are contended) 35.6 / 35.2 / 35.5 / 37.2; R-MAT 20 serving in batches
// of 3 groups: 3 / 2 / 1 partitions 272 / 325 / 270.
constexpr int kMaxParts = 2;
inline int default_parts(int G) { return G % 2 == 0 || G > 8 ? kMaxParts : 1; }
constexpr int kCntStage = (kLevelChunkMax + 2) * kMaxLists;  // pinned slots for level counts
// Vertices with more arcs than this (in- and out-arcs together) are taken by
// a whole workgroup in the unweighted engine and by several wavefronts in the
// weighted one, at most one vertex in kHeavyShare, so that their item lists
// stay small.  The limit is flat from 128
// to 1,024 (R-MAT 16, 1,000 sources: 3.42 / 3.40 / 3.36 / 3.38 ms at 128 / 256 /
// 512 / 1,024) and too high at 2,048 (3.82); weighted R-MAT 18, 2,048 draws: 130.5 /
// 131.1 / 131.0 / 131.0 ms.
constexpr int64_t kHeavyArcs = 512;
constexpr int64_t kHeavyShare = 256;

bcd_status fail(bcd_status s, const std::string &msg);
bcd_status fail_static(bcd_status s, const char *msg);  // records the message without allocating
bcd_status hip_fail(hipError_t e, const char *what);
bcd_status device_check(int *cus, size_t *lds_block_bytes = nullptr);

inline int default_groups(int64_t n, bool weighted) {
  // keep the [G][n][64] path-count and psi arrays near 64 GiB (HBM is 288 GB),
  // at least one group, at most 96 (128 weighted).  R-MAT 16 runs a query of
  // 33,358 sources in 6 batches of 96 groups 4 % faster than in 9 of 64;
  // wider batches gain nothing more there.  The weighted engine's longer
  // tails favour wider batches: R-MAT 18 weighted 44.6 -> 46.2 GTEPS at 128
  // (46.3 at 192, 41.7 at 256)
  int64_t g = (1ll << 36) / (2 * 8 * 64 * std::max<int64_t>(n, 1));
  if (g < 1) g = 1;
  const int64_t cap = weighted ? 128 : 96;
  if (g > cap) g = cap;
  while (g > 1 && (uint64_t)g * (uint64_t)n >= (1ull << 32)) --g;
  // an even width splits evenly over the partitions (default_parts), here a
  // multiple of 8
  if (g > 8) g -= g % 8;
  return (int)g;
}

// Sizes of a batch workspace of G column groups on an n-vertex graph with H
// heavy vertices: list and queue capacities as the workspace lays them out, and
// the device bytes of all its arrays.
struct BatchSizes {
  uint64_t GN, n;
  int G, P;
  uint64_t capP, capH, hbase, items;     // item lists (BatchState)
  uint64_t capQ, capQH, qhbase, qsize;   // relaxation queues, weighted graphs
  uint64_t levels;                       // (level, list) rows
  BatchSizes(int64_t n_, int G_, uint32_t H) {
    G = G_;
    n = (uint64_t)n_;
    GN = (uint64_t)G * n;
    P = default_parts(G);
    const uint64_t parts = (uint64_t)P, per = ((uint64_t)G + parts - 1) / parts;  // groups of a partition
    capP = (GN * 16 + parts - 1) / parts;
    // a (group, vertex) is an item at most once per level and on at most 64
    // levels, so the heavy lists cannot overflow
    capH = per * H * kLanes;
    hbase = capP * parts;
    items = hbase + capH * parts;
    capQ = per * n;
    capQH = per * H;
    qhbase = capQ * parts;
    qsize = qhbase + capQH * parts;
    levels = (n + kLevelChunkMax + 4) * kMaxLists;
  }
  uint64_t bytes(bool weighted, int64_t m) const {
    const uint64_t g = (uint64_t)G;
    uint64_t b = GN * kLanes * 16 + items * 12 + levels * 12 + n * 4;          // counts, psi, items, rows, targets
    b += g * kLanes * 28 + g * 16 + (uint64_t)kCtrSlots * C_COUNT * 8 + 4096;  // results, staging, counters
    if (!weighted) return b + GN * M_COUNT * 8;
    return b + GN * (kLanes * 8 + 64) + qsize * 16 + g * (uint64_t)m * 8 + 4096;  // distances, masks, queues
  }
};

struct Graph;

struct Workspace {
  Graph *graph = nullptr;
  int64_t n = 0;
  bool weighted_graph = false;
  hipStream_t stream = nullptr;
  // batched engine
  bool batch_ready = false;
  int G = 0;
  BatchState S{};
  size_t res_cap = 0;
  // every path count of S.sig is zero (after creation, a dense reset or a
  // batch whose counts were pushed and then cleared); a batch that pulls its
  // counts leaves them behind, and a pushing batch needs them zero
  bool sig_zero = false;
  uint32_t *d_items0 = nullptr;
  unsigned long long *d_masks0 = nullptr;
  uint32_t *d_dest0 = nullptr;
  int32_t *d_lane_slot = nullptr;
  uint32_t *h_items0 = nullptr;
  unsigned long long *h_masks0 = nullptr;
  uint32_t *h_dest0 = nullptr;
  uint32_t h_cnt0[kMaxLists] = {0};  // level-0 items per list of the staged batch
  double *h_res = nullptr;
  int last_depth = 8;
  // plain engine
  bool plain_ready = false;
  PlainState P{};
  // reachability
  bool reach_ready = false;
  uint32_t *rqn = nullptr;  // frontier counters (ReachCtr), a line per level mod 4; then the arrays below
  uint32_t *bitmap = nullptr;
  int32_t *rq[2] = {nullptr, nullptr};
  int32_t *d_roots = nullptr;  // several roots of one traversal
  size_t roots_cap = 0;
  uint32_t *h_reach = nullptr;  // the counters, then the bitmap
  uint32_t *h_bitmap = nullptr;
  // host staging
  uint32_t *h_cnt = nullptr;
  uint64_t *h_misc = nullptr;
  uint64_t *h_ctr = nullptr;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> events;
  // server batches: target list and result routes, grown on demand and kept
  // (a free in the batch loop would wait for every stream of the device)
  int32_t *d_tgt_list = nullptr;
  size_t tgt_list_cap = 0;
  ResultRoute *d_routes = nullptr;
  size_t routes_cap = 0;
  bcd_status ensure_server_lists(size_t ntgt, size_t nroutes);
  // LDS engine scratch (bcd_lds.hip), grown on demand
  void *lds_dev = nullptr;
  size_t lds_dev_bytes = 0;
  void *lds_host = nullptr;
  size_t lds_host_bytes = 0;

  ~Workspace();
  void release();
  bcd_status init_common(Graph *g);
  bcd_status ensure_reach();
  bcd_status ensure_batch(int G);
  bcd_status ensure_res(size_t need);
  bcd_status ensure_dout();
  bcd_status grow_items();
  bcd_status reset_batch_dense();
  bcd_status ensure_plain();
  // Stage a batch: lane i of the batch (column group i / 64, lane i % 64)
  // runs source vertex src[i]; vertices must be distinct within a group.
  void stage_sources(const int32_t *src, int k);
  static int lists(int P) { return 2 * P; }  // item lists of a batch on P partitions: light, heavy
  // Partitions a batch of k staged sources uses: its groups are 0..ceil(k/64)-1
  // and group g belongs to partition g % P, so a batch of fewer groups than
  // S.P uses one partition per group and no workgroup is left without work.
  int batch_parts(int k) const { return std::max(1, std::min(S.P, (k + kLanes - 1) / kLanes)); }
  int staged = 0;
  bool weighted_ready = false;
  int weighted_G = 0;
  bcd_status ensure_weighted();
  void release_weighted();
  std::pair<hipEvent_t, hipEvent_t> event_pair(size_t i);
};

struct Graph {
  int64_t n = 0, m = 0;
  bool weighted = false;
  uint32_t max_w = 1;
  int cus = 1;
  size_t lds_block_bytes = 0;  // LDS one workgroup may allocate
  std::vector<int64_t> h_rp;
  // compression (computed on the first compressed call): gate[v] = the vertex
  // every path from v leaves through when v lies on no cycle and all its
  // out-neighbours funnel into that one vertex, else -1
  std::mutex gate_mu;
  bool gates_ready = false;
  std::vector<int32_t> gate;
  unsigned char *d_arrays = nullptr;  // the one allocation that holds the arrays below
  int64_t *d_rp = nullptr;
  int32_t *d_col = nullptr;
  int64_t *d_irp = nullptr;
  int32_t *d_icol = nullptr;
  // the same graph in internal ids (DevGraph): rank[v] = internal id of v
  std::vector<int32_t> rank;
  uint32_t heavy = 0;          // internal ids below are heavy
  int64_t longest_row = 0;     // arcs of the vertex with the most out-arcs
  int64_t *d_prp = nullptr;
  int32_t *d_pcol = nullptr;
  int64_t *d_pirp = nullptr;
  int32_t *d_picol = nullptr;  // unweighted
  int32_t *d_orig = nullptr;
  uint32_t *d_lrp = nullptr;   // the CSR in 32- and 16-bit words, where lds_fits
  uint16_t *d_lcol = nullptr;
  uint2 *d_arcw = nullptr;     // weighted, internal ids: {head, length} per CSR arc
  uint2 *d_iarc = nullptr;     // weighted: {tail, length} per transpose arc
  uint32_t *d_iopos = nullptr; // weighted: CSR position per transpose arc
  mutable std::mutex cfg_mu;
  bcd_config cfg{};
  std::mutex pool_mu;
  std::vector<std::unique_ptr<Workspace>> pool;
  std::atomic<bool> profiling{false};
  // levels of the last traversal that took a launch per level (a hint: it
  // decides how a traversal runs, not what it finds)
  mutable std::atomic<int64_t> reach_depth{6};
  // a batch met a path count above 2^32 - 1: batches store 64-bit counts from then on
  std::atomic<bool> wide_counts{false};
  std::mutex lm_mu;                // landmark distance signatures (source ordering)
  bool lm_ready = false;
  std::vector<uint8_t> lm_sig;     // [n][16] BFS distance to each hub, 255 = unreachable
  mutable std::mutex prof_mu;
  bcd_kernel_profile prof[2]{};
  hipEvent_t prof_ref = nullptr;                      // origin of the launch intervals below
  std::vector<std::pair<double, double>> prof_iv[2];  // launch [start, end], ms after prof_ref
  double prof_solo_ms[2] = {0, 0};                    // launches timed without an interval
  bcd_status mark_profile_origin();

  ~Graph();
  DevGraph dev() const;           // caller's vertex ids
  DevGraph dev_internal() const;  // internal ids (batched and weighted engines)
  Launch launch() const;
  Launch launch_parts(int P, int groups) const;  // grid a multiple of P
  bcd_config config() const;
  // A pooled workspace, else a new one: the widest (a call's own), or, for the
  // second of a run, the narrowest of lo .. hi groups, else the widest below lo,
  // else the narrowest above hi (to be rebuilt).
  std::unique_ptr<Workspace> acquire(int lo = 0, int hi = INT32_MAX);
  void release(std::unique_ptr<Workspace> w);
  void trim_pool();  // free the device memory of idle pooled workspaces
  void add_profile(int kind, int64_t launches, double ms, const uint64_t *c3, double alg_bytes,
                   uint64_t items = 0, const std::vector<std::pair<double, double>> *intervals = nullptr,
                   uint64_t item_arcs = 0, double sched_bytes = -1.0);
  int64_t outdeg(int64_t v) const { return h_rp[(size_t)v + 1] - h_rp[(size_t)v]; }
};

// Scoped workspace lease.
struct Lease {
  Graph *g;
  std::unique_ptr<Workspace> w;
  explicit Lease(Graph *g_) : g(g_), w(g_->acquire()) {}
  Lease(Graph *g_, int lo, int hi) : g(g_), w(g_->acquire(lo, hi)) {}
  ~Lease() { g->release(std::move(w)); }
  Workspace *operator->() { return w.get(); }
  bool ok() const { return (bool)w; }
};

// Per-source results of one run over a source list.
struct SourceRun {
  std::vector<double> dep;          // [ns][ntgt]
  std::vector<uint64_t> counters;   // [ns][3] when requested
  uint64_t te = 0, reached = 0, dag = 0;
  int32_t width = 0;
  // sources of the run that this one is a timing sample of (0: none): its second
  // workspace is then as wide as that run's, so that it is had where that run has it
  size_t sample_of = 0;
};

struct TargetMap {
  Workspace *ws;
  std::vector<int32_t> ids;  // internal ids, kept until the copy has been read
  int32_t *d_verts = nullptr;
  int k = 0;
  bool set = false;
  ~TargetMap() {
    if (set) {
      (void)launch_scatter_targets(ws->S.tgt_of, d_verts, k, 0, ws->stream);
      (void)hipStreamSynchronize(ws->stream);
    }
    if (d_verts) (void)hipFree(d_verts);
  }
  bcd_status install(Workspace *w, const std::vector<int32_t> &tgt) {
    ws = w;
    k = (int)tgt.size();
    if (k == 0) return BCD_OK;
    if (hipMalloc((void **)&d_verts, (size_t)k * sizeof(int32_t)) != hipSuccess) {
      (void)hipGetLastError();
      d_verts = nullptr;
      return fail(BCD_ERR_OUT_OF_MEMORY, "target list allocation failed");
    }
    ids = tgt;
    for (int32_t &v : ids) v = ws->graph->rank[(size_t)v];
    HIPCHK(hipMemcpyAsync(d_verts, ids.data(), (size_t)k * sizeof(int32_t), hipMemcpyHostToDevice, ws->stream));
    HIPCHK(launch_scatter_targets(ws->S.tgt_of, d_verts, k, 1, ws->stream));
    set = true;
    return BCD_OK;
  }
};

// Launch timings of one run, per kind (0 forward, 1 backward), gathered while
// the graph's profiling is on.
struct ProfAcc {
  int64_t launches[2] = {0, 0};
  double ms[2] = {0, 0};
  uint64_t items[2] = {0, 0};
  std::vector<std::pair<double, double>> iv[2];  // launch intervals after the graph's profile origin
  int count_bytes = 0;  // widest stored path count of the batched unweighted engine's batches
  void merge(const ProfAcc &o) {
    count_bytes = std::max(count_bytes, o.count_bytes);
    for (int k = 0; k < 2; ++k) {
      launches[k] += o.launches[k];
      ms[k] += o.ms[k];
      items[k] += o.items[k];
      iv[k].insert(iv[k].end(), o.iv[k].begin(), o.iv[k].end());
    }
  }
  // one launch bracketed by the event pair (a, b)
  void add(const Graph *g, int kind, hipEvent_t a, hipEvent_t b);
};

// Batches b = first, first + stride, ... of one run on workspace `ws`
// (ws's own stream; results to their own positions).
using StripeFn = std::function<bcd_status(Workspace *ws, size_t first, size_t stride, ProfAcc &prof, bool &ovf)>;
// Readies a workspace for batches of `groups` column groups.
using PrepareFn = std::function<bcd_status(Workspace *ws, int groups)>;
size_t pipelined_batch(const Graph *g, size_t ns, size_t width);
// Column groups of the second workspace of a run of ns sources, a sample of a run
// of `sample_of` (0: none), batches at most `width` sources wide; 0: one batch.
int second_groups(const Graph *g, size_t ns, size_t sample_of, size_t width);
// Runs `stripe` over the batches of `per` sources each; when the run has more
// than one and a second workspace of `share` groups (second_groups) can be had
// (`prepare` readies it), every other batch goes to that workspace on a helper thread,
// else whole batches run on ws.  The second workspace's counters are added to
// `tot`; *width receives the sources per batch that ran.
bcd_status run_pipelined(Graph *g, Workspace *ws, size_t per, int share, const PrepareFn &prepare,
                         const StripeFn &stripe, ProfAcc &prof, bool &ovf, uint64_t *tot, int32_t *width);

// Configurations the autotuner times around `base` (bcd_tune.hip).
std::vector<bcd_config> tune_around(const bcd_config &base, bool weighted);
// Query layer (bcd_query.hip).
bcd_status reach_set(Graph *g, Workspace *ws, int32_t root, bool reverse, std::vector<uint32_t> &bits,
                     int64_t *count, uint8_t *d_lev);
// D of the set form: the union of RV(r) over the targets (ascending, distinct)
// with out-arcs, as a bitmap.
bcd_status reach_union(Graph *g, Workspace *ws, const std::vector<int32_t> &targets, std::vector<uint32_t> &uni);
// Whether the host check behind `level` levels, the last `chunk` of them just
// launched, brings the whole bitmap.
inline bool reach_copies_bitmap(int64_t level, int chunk, size_t bytes) {
  return level == chunk && bytes <= (size_t(1) << 20);
}
// Frontier arcs from which a reachability level goes bottom-up.
inline uint64_t reach_bu_arcs(const Graph *g) { return (uint64_t)std::max<int64_t>(64, g->m / 64); }
bcd_status run_weighted(Graph *g, Workspace *ws, const std::vector<int32_t> &src,
                        const std::vector<int32_t> &tgt, bool want_counters, SourceRun &out);
bcd_status multi_source_pass_weighted(Graph *g, const int32_t *sources, int64_t k, uint64_t *dist,
                                      uint64_t *sigma, double *delta);
// Device bytes of one batch workspace of `groups` column groups (bcd_server.hip).
uint64_t batch_workspace_bytes(const Graph *g, int groups);
// LDS engine (bcd_lds.hip): one workgroup per source at a time, state in LDS.
size_t lds_bytes_for(int64_t n);
bool lds_fits(const Graph *g);
// Whether the LDS engine takes a row's arcs one at a time.
bool lds_short_rows(const Graph *g);
// Whether a traversal of at least `levels` levels goes to one workgroup (n < 2^16,
// visited bits and queue in LDS) instead of a launch per level.
bool reach_one_workgroup(const Graph *g, int64_t levels);
hipError_t launch_lds_reach(const Graph *g, const int64_t *rp, const int32_t *col, int32_t root,
                            const int32_t *roots, int k, uint32_t *bitmap, hipStream_t st);
bcd_status run_lds(Graph *g, Workspace *ws, const std::vector<int32_t> &src, const std::vector<int32_t> &tgt,
                   bool want_counters, SourceRun &out);
bcd_status multi_source_pass_lds(Graph *g, Workspace *ws, const int32_t *sources, int64_t k, uint64_t *dist,
                                 uint64_t *sigma, double *delta);
// One batch of `k` sources already staged in ws->h_items0 / h_masks0 with
// ntgt targets installed in ws->S.tgt_of; per-lane target dependencies stay
// in ws->S.res on the device; per-group overflow lanes go to ovl_out[G].
// Launch timings go to *prof when the graph's profiling is on (may be NULL).
bcd_status run_staged_batch(Graph *g, Workspace *ws, int k, int ntgt, unsigned long long *ovl_out, bool *ovf,
                            ProfAcc *prof);
bcd_status run_staged_wbatch(Graph *g, Workspace *ws, int k, int ntgt, unsigned long long *ovl_out, bool *ovf,
                             ProfAcc *prof);
// Add one run's launch timings and its device counters to the graph's profile.
void record_profile(Graph *g, const ProfAcc &p, const uint64_t *ctr);
void record_wprofile(Graph *g, const ProfAcc &p, const uint64_t *ctr);
double compensated_sum(const double *x, size_t k, size_t stride);
// Positions of src in the order batches should take them (sources with
// similar hub-distance signatures together); results never depend on it.
bcd_status source_order(Graph *g, Workspace *ws, const std::vector<int32_t> &src, std::vector<uint32_t> &ord);
bcd_status collect_counters(Workspace *ws, uint64_t *ctr, uint64_t *dev_acc);
uint64_t splitmix_at(uint64_t seed, uint64_t t);
uint64_t index_below(uint64_t x, uint64_t k);
void bits_to_list(const std::vector<uint32_t> &bits, int64_t n, int32_t skip, std::vector<int32_t> &out);
bcd_status run_sources(Graph *g, Workspace *ws, const std::vector<int32_t> &src,
                       const std::vector<int32_t> &tgt, bool want_counters, SourceRun &out);

}  // namespace bcd

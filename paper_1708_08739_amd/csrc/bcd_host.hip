// libbcd host layer: the C ABI of include/bcd.h.
//
// Graph: the out-CSR and its transpose (the reverse graph of Def.2) are
// uploaded once and stay resident.  Queries: RV(r) by a device BFS on the
// transpose (Def.3, Prop.2), then batches of sources through the batched
// forward / backward kernels, then a compensated sum on the host in a fixed
// order (ascending source for Alg.1, draw order for Alg.2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/bcd.h"
#include "bcd_internal.h"
#include "bcd_host_internal.h"

namespace bcd {

// Message of the calling thread's last failing call, in a fixed buffer so
// that recording it never allocates.
static thread_local char t_last_error[512];

static void set_last_error(const char *msg, size_t len) {
  if (len >= sizeof(t_last_error)) len = sizeof(t_last_error) - 1;
  std::memcpy(t_last_error, msg, len);
  t_last_error[len] = '\0';
}

bcd_status fail(bcd_status s, const std::string &msg) {
  set_last_error(msg.data(), msg.size());
  return s;
}

bcd_status fail_static(bcd_status s, const char *msg) {
  set_last_error(msg, std::strlen(msg));
  return s;
}

bcd_status hip_fail(hipError_t e, const char *what) {
  return fail(BCD_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}


static double now_s() {
  return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

// ------------------------------------------------------------ device

bcd_status device_check(int *cus, size_t *lds_block_bytes) {
  int ndev = 0;
  hipError_t e = hipGetDeviceCount(&ndev);
  if (e != hipSuccess || ndev <= 0) return fail(BCD_ERR_DEVICE, "no HIP device available");
  int dev = 0;
  HIPCHK(hipGetDevice(&dev));
  hipDeviceProp_t prop;
  HIPCHK(hipGetDeviceProperties(&prop, dev));
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return fail(BCD_ERR_DEVICE, std::string("libbcd is built for gfx950; device is ") + prop.gcnArchName);
  if (cus) *cus = prop.multiProcessorCount;
  if (lds_block_bytes) *lds_block_bytes = prop.sharedMemPerBlock;
  return BCD_OK;
}

template <class T>
static bcd_status dalloc(T **p, size_t count) {
  *p = nullptr;
  if (count == 0) count = 1;
  hipError_t e = hipMalloc((void **)p, count * sizeof(T));
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    return fail(BCD_ERR_OUT_OF_MEMORY, std::string("device allocation of ") +
                                           std::to_string(count * sizeof(T)) + " bytes failed");
  }
  return BCD_OK;
}

template <class T>
static bcd_status halloc(T **p, size_t count) {
  *p = nullptr;
  if (count == 0) count = 1;
  hipError_t e = hipHostMalloc((void **)p, count * sizeof(T), hipHostMallocDefault);
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    return fail(BCD_ERR_OUT_OF_MEMORY, "pinned host allocation failed");
  }
  return BCD_OK;
}

template <class T>
static void dfree(T *&p) {
  if (p) (void)hipFree((void *)p);
  p = nullptr;
}

template <class T>
static void hfree(T *&p) {
  if (p) (void)hipHostFree((void *)p);
  p = nullptr;
}

// ---------------------------------------------------------- workspace

Workspace::~Workspace() { release(); }

void Workspace::release() {
  release_weighted();
  dfree(d_tgt_list);
  dfree(d_routes);
  tgt_list_cap = routes_cap = 0;
  if (lds_dev) (void)hipFree(lds_dev);
  if (lds_host) (void)hipHostFree(lds_host);
  lds_dev = lds_host = nullptr;
  lds_dev_bytes = lds_host_bytes = 0;
  dfree(S.sig);
  dfree(S.psi);
  dfree(S.dout);
  dfree(S.vis);
  dfree(S.fr);
  dfree(S.msk);
  dfree(S.items);
  dfree(S.imask);
  dfree(S.cnt);
  dfree(S.off);
  dfree(S.tail);
  dfree(S.tmin);
  dfree(S.tgt_of);
  dfree(S.res);
  dfree(S.ctr);
  dfree(S.acc);
  dfree(S.flags);
  dfree(S.ovl);
  dfree(d_items0);
  dfree(d_masks0);
  dfree(d_dest0);
  hfree(h_dest0);
  dfree(d_lane_slot);
  dfree(P.d);
  dfree(P.sig);
  dfree(P.psi);
  dfree(P.dout);
  dfree(P.queue);
  dfree(P.cnt);
  dfree(P.off);
  dfree(P.ctr);
  dfree(P.acc);
  dfree(P.flags);
  dfree(bitmap);
  dfree(rq[0]);
  dfree(rq[1]);
  dfree(rqn);
  dfree(d_roots);
  roots_cap = 0;
  hfree(h_items0);
  hfree(h_masks0);
  hfree(h_cnt);
  hfree(h_misc);
  hfree(h_res);
  hfree(h_ctr);
  hfree(h_bitmap);
  for (auto &ev : events) {
    (void)hipEventDestroy(ev.first);
    (void)hipEventDestroy(ev.second);
  }
  events.clear();
  if (stream) (void)hipStreamDestroy(stream);
  stream = nullptr;
  batch_ready = plain_ready = reach_ready = false;
}

bcd_status Workspace::init_common(Graph *g) {
  graph = g;
  n = g->n;
  weighted_graph = g->weighted;
  if (!stream) HIPCHK(hipStreamCreateWithFlags(&stream, hipStreamNonBlocking));
  return BCD_OK;
}

bcd_status Workspace::ensure_reach() {
  if (reach_ready) return BCD_OK;
  // what an earlier call that failed part way left allocated
  dfree(bitmap); dfree(rq[0]); dfree(rq[1]); dfree(rqn); hfree(h_bitmap);
  const size_t words = (size_t)(n + 31) / 32;
  STCHK(dalloc(&bitmap, words));
  STCHK(dalloc(&rq[0], (size_t)n));
  STCHK(dalloc(&rq[1], (size_t)n));
  STCHK(dalloc(&rqn, 4 * kTailStride));
  STCHK(halloc(&h_bitmap, words));
  if (!h_misc) STCHK(halloc(&h_misc, 64));  // shared with the plain engine
  reach_ready = true;
  return BCD_OK;
}

bcd_status Workspace::ensure_batch(int G_) {
  if (batch_ready && G == G_) return BCD_OK;
  // the previous width's arrays, or what an earlier call that failed part
  // way left allocated (every free is a no-op on a null pointer)
  release_weighted();
  dfree(S.sig); dfree(S.psi); dfree(S.dout); dfree(S.vis); dfree(S.fr); dfree(S.msk);
  dfree(S.items); dfree(S.imask); dfree(S.cnt); dfree(S.off); dfree(S.tail); dfree(S.tmin);
  dfree(S.tgt_of); dfree(S.res); dfree(S.ctr); dfree(S.acc); dfree(S.flags); dfree(S.ovl);
  dfree(d_items0); dfree(d_masks0); dfree(d_dest0); dfree(d_lane_slot); hfree(h_items0); hfree(h_masks0);
  hfree(h_dest0); hfree(h_res);
  res_cap = 0;
  batch_ready = false;
  if ((uint64_t)G_ * (uint64_t)n >= (1ull << 32))
    return fail(BCD_ERR_UNSUPPORTED, "groups * n must stay below 2^32");
  G = G_;
  const size_t GN = (size_t)G * (size_t)n;
  std::memset(&S, 0, sizeof(S));
  S.n = n;
  S.G = G;
  STCHK(dalloc(&S.sig, GN * kLanes));
  STCHK(dalloc(&S.psi, GN * kLanes));
  if (weighted_graph) {
    STCHK(dalloc(&S.vis, GN));
    STCHK(dalloc(&S.fr, 3 * GN));
  } else {
    STCHK(dalloc(&S.msk, M_COUNT * GN));
  }
  S.P = default_parts(G);
  S.NL = lists(S.P);
  S.H = graph->heavy;
  S.capP = ((uint64_t)GN * 16 + (uint64_t)S.P - 1) / (uint64_t)S.P;
  // a (group, vertex) is an item at most once per level and on at most 64
  // levels, so the heavy lists cannot overflow
  S.capH = (uint64_t)((G + S.P - 1) / S.P) * S.H * kLanes;
  S.hbase = S.capP * (uint64_t)S.P;
  STCHK(dalloc(&S.items, S.hbase + S.capH * S.P));
  STCHK(dalloc(&S.imask, S.hbase + S.capH * S.P));
  const size_t levels = ((size_t)n + kLevelChunkMax + 4) * kMaxLists;
  STCHK(dalloc(&S.cnt, levels));
  STCHK(dalloc(&S.off, levels));
  STCHK(dalloc(&S.tail, (size_t)4 * kMaxLists * kTailStride));
  STCHK(dalloc(&S.tmin, 4));
  STCHK(dalloc(&S.tgt_of, (size_t)n));
  STCHK(dalloc(&S.flags, 4));
  STCHK(dalloc(&S.ovl, 2 * (size_t)G));
  S.ctr_slots = kCtrSlots;
  STCHK(dalloc(&S.ctr, (size_t)kCtrSlots * C_COUNT));
  STCHK(dalloc(&S.acc, (size_t)C_COUNT));
  HIPCHK(hipMemsetAsync(S.acc, 0, (size_t)C_COUNT * sizeof(uint64_t), stream));
  res_cap = (size_t)G * kLanes;
  STCHK(dalloc(&S.res, res_cap));
  STCHK(dalloc(&d_items0, (size_t)G * kLanes));
  STCHK(dalloc(&d_masks0, (size_t)G * kLanes));
  STCHK(dalloc(&d_dest0, (size_t)G * kLanes));
  STCHK(halloc(&h_dest0, (size_t)G * kLanes));
  STCHK(dalloc(&d_lane_slot, (size_t)G * kLanes));
  STCHK(halloc(&h_items0, (size_t)G * kLanes));
  STCHK(halloc(&h_masks0, (size_t)G * kLanes));
  STCHK(halloc(&h_res, res_cap));
  if (!h_cnt) STCHK(halloc(&h_cnt, kCntStage + 16));
  if (!h_misc) STCHK(halloc(&h_misc, 64));
  if (!h_ctr) STCHK(halloc(&h_ctr, (size_t)kCtrSlots * C_COUNT));
  HIPCHK(hipMemsetAsync(S.sig, 0, GN * kLanes * sizeof(uint64_t), stream));
  if (S.vis) HIPCHK(hipMemsetAsync(S.vis, 0, GN * sizeof(uint64_t), stream));
  if (S.fr) HIPCHK(hipMemsetAsync(S.fr, 0, 3 * GN * sizeof(uint64_t), stream));
  if (S.msk) HIPCHK(hipMemsetAsync(S.msk, 0, M_COUNT * GN * sizeof(uint64_t), stream));
  HIPCHK(hipMemsetAsync(S.cnt, 0, levels * sizeof(uint32_t), stream));
  HIPCHK(hipMemsetAsync(S.off, 0, levels * sizeof(uint64_t), stream));
  HIPCHK(hipMemsetAsync(S.tgt_of, 0xFF, (size_t)n * sizeof(int32_t), stream));
  HIPCHK(hipMemsetAsync(S.flags, 0, 4 * sizeof(uint32_t), stream));
  HIPCHK(hipMemsetAsync(S.ctr, 0, (size_t)kCtrSlots * C_COUNT * sizeof(uint64_t), stream));
  HIPCHK(hipStreamSynchronize(stream));
  sig_zero = true;
  batch_ready = true;
  return BCD_OK;
}


void Workspace::stage_sources(const int32_t *src, int k) {
  for (int i = 0; i < k; ++i) {
    h_items0[i] = (uint32_t)((uint64_t)(i / kLanes) * (uint64_t)n + (uint64_t)graph->rank[(size_t)src[i]]);
    h_masks0[i] = 1ull << (i % kLanes);
  }
  staged = k;
  // the place of every staged item in its list (level0_slot)
  uint32_t fill[kMaxLists] = {0};
  BatchState T = S;
  T.P = batch_parts(k);
  T.NL = lists(T.P);
  for (int i = 0; i < k; ++i) {
    const uint32_t g = (uint32_t)(i / kLanes);
    h_dest0[i] = fill[list_of(T, g, h_items0[i] - g * (uint32_t)n)]++;
  }
  for (int l = 0; l < kMaxLists; ++l) h_cnt0[l] = fill[l];
}

bcd_status Workspace::ensure_res(size_t need) {
  if (need <= res_cap) return BCD_OK;
  dfree(S.res);
  hfree(h_res);
  res_cap = 0;  // recorded only once both buffers exist
  STCHK(dalloc(&S.res, need));
  STCHK(halloc(&h_res, need));
  res_cap = need;
  return BCD_OK;
}

bcd_status Workspace::ensure_server_lists(size_t ntgt, size_t nroutes) {
  ntgt = std::max<size_t>(ntgt, 1);
  nroutes = std::max<size_t>(nroutes, 1);
  if (ntgt > tgt_list_cap) {
    const size_t cap = std::max<size_t>(ntgt, 2 * tgt_list_cap + 64);
    dfree(d_tgt_list);
    tgt_list_cap = 0;
    STCHK(dalloc(&d_tgt_list, cap));
    tgt_list_cap = cap;
  }
  if (nroutes > routes_cap) {
    const size_t cap = std::max<size_t>(nroutes, 2 * routes_cap + 1024);
    dfree(d_routes);
    routes_cap = 0;
    STCHK(dalloc(&d_routes, cap));
    routes_cap = cap;
  }
  return BCD_OK;
}

bcd_status Workspace::ensure_dout() {
  if (S.dout) return BCD_OK;
  return dalloc(&S.dout, (size_t)G * (size_t)n * kLanes);
}

bcd_status Workspace::grow_items() {
  const uint64_t GN = (uint64_t)G * (uint64_t)n;
  const uint64_t ncapP = std::min<uint64_t>(S.capP * 2, (GN * kLanes) / (uint64_t)S.P + (uint64_t)kLanes * G);
  dfree(S.items);
  dfree(S.imask);
  S.capP = ncapP;
  S.hbase = S.capP * (uint64_t)S.P;
  // if an allocation fails the workspace must not be reused as it stands:
  // the next ensure_batch rebuilds every array
  batch_ready = false;
  STCHK(dalloc(&S.items, S.hbase + S.capH * S.P));
  STCHK(dalloc(&S.imask, S.hbase + S.capH * S.P));
  batch_ready = true;
  return BCD_OK;
}

// Full reset after an aborted batch (item list overflow, or a host exception
// in a server worker): the sparse cleanup cannot see items that were never
// stored.
bcd_status Workspace::reset_batch_dense() {
  const size_t GN = (size_t)G * (size_t)n;
  HIPCHK(hipMemsetAsync(S.sig, 0, GN * kLanes * sizeof(uint64_t), stream));
  sig_zero = true;
  if (S.vis) HIPCHK(hipMemsetAsync(S.vis, 0, GN * sizeof(uint64_t), stream));
  if (S.fr) HIPCHK(hipMemsetAsync(S.fr, 0, 3 * GN * sizeof(uint64_t), stream));
  if (S.msk) HIPCHK(hipMemsetAsync(S.msk, 0, M_COUNT * GN * sizeof(uint64_t), stream));
  HIPCHK(hipMemsetAsync(S.cnt, 0, ((size_t)n + kLevelChunkMax + 4) * kMaxLists * sizeof(uint32_t), stream));
  HIPCHK(hipMemsetAsync(S.flags, 0, 4 * sizeof(uint32_t), stream));
  HIPCHK(hipMemsetAsync(S.ctr, 0, (size_t)kCtrSlots * C_COUNT * sizeof(uint64_t), stream));
  if (weighted_ready) {
    HIPCHK(hipMemsetAsync(S.wd, 0xFF, GN * kLanes * sizeof(uint32_t), stream));
    HIPCHK(hipMemsetAsync(S.wc, 0, GN * kLanes * sizeof(uint32_t), stream));
    HIPCHK(hipMemsetAsync(S.chg, 0, 3 * GN * sizeof(unsigned long long), stream));
    HIPCHK(hipMemsetAsync(S.rtail, 0, (size_t)kMaxLists * kTailStride * sizeof(uint32_t), stream));
    HIPCHK(hipMemsetAsync(S.wdn, 0, GN * sizeof(unsigned long long), stream));
  }
  HIPCHK(hipStreamSynchronize(stream));
  return BCD_OK;
}

bcd_status Workspace::ensure_plain() {
  if (plain_ready) return BCD_OK;
  // what an earlier call that failed part way left allocated
  dfree(P.d); dfree(P.sig); dfree(P.psi); dfree(P.dout); dfree(P.queue);
  dfree(P.cnt); dfree(P.off); dfree(P.flags); dfree(P.ctr); dfree(P.acc);
  std::memset(&P, 0, sizeof(P));
  P.n = n;
  STCHK(dalloc(&P.d, (size_t)n));
  STCHK(dalloc(&P.sig, (size_t)n));
  STCHK(dalloc(&P.psi, (size_t)n));
  STCHK(dalloc(&P.dout, (size_t)n));
  STCHK(dalloc(&P.queue, (size_t)n));
  const size_t levels = (size_t)n + kLevelChunkMax + 4;
  STCHK(dalloc(&P.cnt, levels));
  STCHK(dalloc(&P.off, levels));
  STCHK(dalloc(&P.flags, 4));
  P.ctr_slots = kCtrSlots;
  STCHK(dalloc(&P.ctr, (size_t)kCtrSlots * C_COUNT));
  STCHK(dalloc(&P.acc, (size_t)C_COUNT));
  HIPCHK(hipMemsetAsync(P.acc, 0, (size_t)C_COUNT * sizeof(uint64_t), stream));
  if (!h_cnt) STCHK(halloc(&h_cnt, kCntStage + 16));
  if (!h_misc) STCHK(halloc(&h_misc, 64));
  if (!h_ctr) STCHK(halloc(&h_ctr, (size_t)kCtrSlots * C_COUNT));
  HIPCHK(hipMemsetAsync(P.d, 0xFF, (size_t)n * sizeof(int32_t), stream));
  HIPCHK(hipMemsetAsync(P.sig, 0, (size_t)n * sizeof(uint64_t), stream));
  HIPCHK(hipMemsetAsync(P.cnt, 0, levels * sizeof(uint32_t), stream));
  HIPCHK(hipMemsetAsync(P.off, 0, levels * sizeof(uint64_t), stream));
  HIPCHK(hipMemsetAsync(P.flags, 0, 4 * sizeof(uint32_t), stream));
  HIPCHK(hipMemsetAsync(P.ctr, 0, (size_t)kCtrSlots * C_COUNT * sizeof(uint64_t), stream));
  HIPCHK(hipStreamSynchronize(stream));
  plain_ready = true;
  return BCD_OK;
}

std::pair<hipEvent_t, hipEvent_t> Workspace::event_pair(size_t i) {
  while (events.size() <= i) {
    hipEvent_t a = nullptr, b = nullptr;
    (void)hipEventCreate(&a);
    (void)hipEventCreate(&b);
    events.emplace_back(a, b);
  }
  return events[i];
}

// ------------------------------------------------------------- graph

Graph::~Graph() {
  pool.clear();
  if (prof_ref) (void)hipEventDestroy(prof_ref);
  dfree(d_rp);
  dfree(d_col);
  dfree(d_irp);
  dfree(d_icol);
  dfree(d_prp);
  dfree(d_pcol);
  dfree(d_pirp);
  dfree(d_picol);
  dfree(d_orig);
  dfree(d_lrp);
  dfree(d_lcol);
  dfree(d_arcw);
  dfree(d_iarc);
  dfree(d_iopos);
}

DevGraph Graph::dev() const {
  DevGraph G;
  G.n = n;
  G.m = m;
  G.rp = d_rp;
  G.col = d_col;
  G.irp = d_irp;
  G.icol = d_icol;
  G.arcw = G.iarc = nullptr;
  G.iopos = nullptr;
  G.orig = nullptr;
  return G;
}

DevGraph Graph::dev_internal() const {
  DevGraph G;
  G.n = n;
  G.m = m;
  G.rp = d_prp;
  G.col = d_pcol;
  G.irp = d_pirp;
  G.icol = d_picol;
  G.arcw = d_arcw;
  G.iarc = d_iarc;
  G.iopos = d_iopos;
  G.orig = d_orig;
  return G;
}

// Launch of a batch of `groups` column groups on P partitions: a wavefront per
// (group, vertex) is as many as any level can use.
Launch Graph::launch_parts(int P, int groups) const {
  Launch L = launch();
  const uint64_t waves = (uint64_t)groups * (uint64_t)n, per = (uint64_t)(L.block / 64);
  L.grid = (int)std::min<uint64_t>((uint64_t)L.grid, (waves + per - 1) / per);
  L.grid = std::max(2 * P, L.grid - L.grid % P);  // two workgroups a partition at least (ListView)
  return L;
}

Launch Graph::launch() const {
  Launch L;
  std::lock_guard<std::mutex> lk(cfg_mu);
  L.block = cfg.block;
  L.grid = std::max(1, std::min(kCtrSlots, cus * cfg.grid_mult));
  L.items = cfg.items;
  return L;
}

bcd_config Graph::config() const {
  std::lock_guard<std::mutex> lk(cfg_mu);
  return cfg;
}

void Graph::trim_pool() {
  std::vector<std::unique_ptr<Workspace>> idle;
  {
    std::lock_guard<std::mutex> lk(pool_mu);
    idle.swap(pool);
  }
  // destroyed here, outside the lock
}

std::unique_ptr<Workspace> Graph::acquire(int lo, int hi) {
  {
    std::lock_guard<std::mutex> lk(pool_mu);
    auto groups = [](const std::unique_ptr<Workspace> &w) { return w->batch_ready ? w->G : 0; };
    auto better = [&](int a, int b) {
      if (lo == 0) return a > b;
      const int ra = a > hi ? 0 : a >= lo ? 2 : 1, rb = b > hi ? 0 : b >= lo ? 2 : 1;
      return ra != rb ? ra > rb : ra == 1 ? a > b : a < b;
    };
    if (!pool.empty()) {
      size_t best = pool.size() - 1;
      for (size_t i = best; i-- > 0;)
        if (better(groups(pool[i]), groups(pool[best]))) best = i;
      std::unique_ptr<Workspace> w = std::move(pool[best]);
      pool.erase(pool.begin() + (std::ptrdiff_t)best);
      return w;
    }
  }
  std::unique_ptr<Workspace> w(new (std::nothrow) Workspace());
  return w;
}

void Graph::release(std::unique_ptr<Workspace> w) {
  if (!w) return;
  std::lock_guard<std::mutex> lk(pool_mu);
  pool.push_back(std::move(w));
}

bcd_status Graph::mark_profile_origin() {
  if (!prof_ref) HIPCHK(hipEventCreate(&prof_ref));
  HIPCHK(hipEventRecord(prof_ref, nullptr));
  HIPCHK(hipEventSynchronize(prof_ref));
  return BCD_OK;
}

void Graph::add_profile(int kind, int64_t launches, double ms, const uint64_t *c3, double alg_bytes,
                        uint64_t items, const std::vector<std::pair<double, double>> *intervals,
                        uint64_t item_arcs, double sched_bytes) {
  std::lock_guard<std::mutex> lk(prof_mu);
  bcd_kernel_profile &p = prof[kind];
  p.launches += launches;
  p.total_ms += ms;
  p.alg_bytes += alg_bytes;
  p.item_arcs += item_arcs;
  p.sched_bytes += sched_bytes < 0 ? alg_bytes : sched_bytes;
  p.vertex_pairs += c3[0];
  p.arc_pairs += c3[1];
  p.dag_pairs += c3[2];
  p.items += items;
  if (intervals && !intervals->empty())
    prof_iv[kind].insert(prof_iv[kind].end(), intervals->begin(), intervals->end());
  else
    prof_solo_ms[kind] += ms;
}

}  // namespace bcd

using namespace bcd;

// ----------------------------------------------------------------- ABI

extern "C" {

const char *bcd_status_string(bcd_status s) {
  switch (s) {
    case BCD_OK: return "ok";
    case BCD_ERR_INVALID_ARG: return "invalid argument";
    case BCD_ERR_BAD_GRAPH: return "malformed graph";
    case BCD_ERR_SIGMA_OVERFLOW: return "shortest-path count overflows uint64";
    case BCD_ERR_OUT_OF_MEMORY: return "out of memory";
    case BCD_ERR_DEVICE: return "device error";
    case BCD_ERR_BUFFER_TOO_SMALL: return "buffer too small";
    case BCD_ERR_UNSUPPORTED: return "unsupported";
    case BCD_ERR_AGAIN: return "try again";
    case BCD_ERR_CANCELLED: return "cancelled";
  }
  return "unknown status";
}

const char *bcd_last_error(void) { return t_last_error; }

bcd_status bcd_sample_count(double eps_abs, double delta, double K, int64_t rv_size, int64_t *T) {
  BCD_GUARD_BEGIN
  if (!T) return fail(BCD_ERR_INVALID_ARG, "T is NULL");
  if (!(eps_abs > 0.0) || !std::isfinite(eps_abs)) return fail(BCD_ERR_INVALID_ARG, "eps must be > 0");
  if (!(delta > 0.0 && delta < 1.0)) return fail(BCD_ERR_INVALID_ARG, "delta must be in (0,1)");
  if (!(K >= 0.0) || !std::isfinite(K)) return fail(BCD_ERR_INVALID_ARG, "K must be >= 0");
  if (rv_size < 0) return fail(BCD_ERR_INVALID_ARG, "rv_size must be >= 0");
  // Eq.(8), evaluated in extended precision so that ceil is exact for the
  // integer-valued cases; at least one draw.
  const long double x = std::log(2.0L / (long double)delta) * (long double)K * (long double)K *
                        (long double)rv_size * (long double)rv_size /
                        (2.0L * (long double)eps_abs * (long double)eps_abs);
  long double c = std::ceil(x);
  if (!(c >= 1.0L)) c = 1.0L;
  *T = (c >= 9.2e18L) ? INT64_MAX : (int64_t)c;
  return BCD_OK;
  BCD_GUARD_END
}

bcd_status bcd_graph_load_csr(int64_t n, int64_t m, const int64_t *row_ptr, const int32_t *col,
                              const uint32_t *weight, bcd_graph **out) {
  BCD_GUARD_BEGIN
  if (!out) return fail(BCD_ERR_INVALID_ARG, "out is NULL");
  if (n <= 0 || n >= (1ll << 31)) return fail(BCD_ERR_INVALID_ARG, "n must be in [1, 2^31)");
  if (m < 0 || m >= (1ll << 32)) return fail(BCD_ERR_INVALID_ARG, "m must be in [0, 2^32)");
  if (!row_ptr || (m > 0 && !col)) return fail(BCD_ERR_INVALID_ARG, "row_ptr/col is NULL");
  // Section 2 graph model: validate fully on the host before touching the GPU.
  if (row_ptr[0] != 0) return fail(BCD_ERR_BAD_GRAPH, "row_ptr[0] != 0");
  if (row_ptr[n] != m) return fail(BCD_ERR_BAD_GRAPH, "row_ptr[n] != m");
  uint64_t max_w = 1;
  for (int64_t v = 0; v < n; ++v) {
    const int64_t a = row_ptr[v], b = row_ptr[v + 1];
    if (b < a) return fail(BCD_ERR_BAD_GRAPH, "row_ptr decreases at vertex " + std::to_string(v));
    if (a < 0 || b > m) return fail(BCD_ERR_BAD_GRAPH, "row_ptr out of [0, m]");
    for (int64_t e = a; e < b; ++e) {
      const int32_t w = col[e];
      if (w < 0 || w >= n) return fail(BCD_ERR_BAD_GRAPH, "column out of range at arc " + std::to_string(e));
      if (w == v) return fail(BCD_ERR_BAD_GRAPH, "self-loop at vertex " + std::to_string(v));
      if (e > a && w <= col[e - 1])
        return fail(BCD_ERR_BAD_GRAPH, "row " + std::to_string(v) + " not strictly increasing (repeated arc?)");
      if (weight) {
        if (weight[e] == 0) return fail(BCD_ERR_BAD_GRAPH, "zero weight at arc " + std::to_string(e));
        max_w = std::max<uint64_t>(max_w, weight[e]);
      }
    }
  }
  int cus = 0;
  size_t lds_block = 0;
  STCHK(device_check(&cus, &lds_block));
  std::unique_ptr<Graph> g(new (std::nothrow) Graph());
  if (!g) return fail(BCD_ERR_OUT_OF_MEMORY, "host allocation failed");
  g->n = n;
  g->m = m;
  g->weighted = weight != nullptr;
  g->max_w = (uint32_t)max_w;
  g->cus = cus;
  g->lds_block_bytes = lds_block;
  g->h_rp.assign(row_ptr, row_ptr + n + 1);
  // transpose by counting sort: rows of R(G) come out sorted
  std::vector<int64_t> irp((size_t)n + 1, 0);
  for (int64_t e = 0; e < m; ++e) irp[(size_t)col[e] + 1]++;
  for (int64_t v = 0; v < n; ++v) irp[(size_t)v + 1] += irp[(size_t)v];
  std::vector<int32_t> icol((size_t)std::max<int64_t>(m, 1));
  std::vector<uint32_t> iw(weight ? (size_t)std::max<int64_t>(m, 1) : 0);
  std::vector<uint32_t> ipos(weight ? (size_t)std::max<int64_t>(m, 1) : 0);
  {
    std::vector<int64_t> fill(irp.begin(), irp.end() - 1);
    for (int64_t u = 0; u < n; ++u)
      for (int64_t e = row_ptr[u]; e < row_ptr[u + 1]; ++e) {
        const int64_t p = fill[(size_t)col[e]]++;
        icol[(size_t)p] = (int32_t)u;
        if (weight) {
          iw[(size_t)p] = weight[e];
          ipos[(size_t)e] = (uint32_t)p;
        }
      }
  }
  STCHK(dalloc(&g->d_rp, (size_t)n + 1));
  STCHK(dalloc(&g->d_col, (size_t)m));
  STCHK(dalloc(&g->d_irp, (size_t)n + 1));
  STCHK(dalloc(&g->d_icol, (size_t)m));
  HIPCHK(hipMemcpy(g->d_rp, row_ptr, ((size_t)n + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
  HIPCHK(hipMemcpy(g->d_irp, irp.data(), ((size_t)n + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
  if (m > 0) {
    HIPCHK(hipMemcpy(g->d_col, col, (size_t)m * sizeof(int32_t), hipMemcpyHostToDevice));
    HIPCHK(hipMemcpy(g->d_icol, icol.data(), (size_t)m * sizeof(int32_t), hipMemcpyHostToDevice));
  }
  if (lds_fits(g.get())) {
    std::vector<uint32_t> lrp(row_ptr, row_ptr + n + 1);
    std::vector<uint16_t> lcol(col, col + m);
    STCHK(dalloc(&g->d_lrp, (size_t)n + 1));
    STCHK(dalloc(&g->d_lcol, (size_t)std::max<int64_t>(m, 1)));
    HIPCHK(hipMemcpy(g->d_lrp, lrp.data(), ((size_t)n + 1) * sizeof(uint32_t), hipMemcpyHostToDevice));
    if (m > 0) HIPCHK(hipMemcpy(g->d_lcol, lcol.data(), (size_t)m * sizeof(uint16_t), hipMemcpyHostToDevice));
  }
  // internal ids: vertices by falling total degree (a counting sort, ties by
  // the caller's id), and both CSRs renamed to them, rows kept in arc order
  std::vector<int32_t> orig((size_t)n);
  g->rank.resize((size_t)n);
  {
    auto deg = [&](int64_t v) {
      return row_ptr[v + 1] - row_ptr[v] + irp[(size_t)v + 1] - irp[(size_t)v];
    };
    int64_t top = 0;
    for (int64_t v = 0; v < n; ++v) top = std::max(top, deg(v));
    std::vector<int64_t> at((size_t)top + 2, 0);  // at[d]: vertices of degree > d so far placed before d
    for (int64_t v = 0; v < n; ++v) at[(size_t)deg(v)]++;
    int64_t before = 0;
    for (int64_t d = top; d >= 0; --d) {
      const int64_t c = at[(size_t)d];
      at[(size_t)d] = before;
      before += c;
    }
    for (int64_t v = 0; v < n; ++v) {
      const int64_t i = at[(size_t)deg(v)]++;
      orig[(size_t)i] = (int32_t)v;
      g->rank[(size_t)v] = (int32_t)i;
    }
    while (g->heavy < (uint64_t)(n / kHeavyShare) && deg(orig[g->heavy]) > kHeavyArcs) ++g->heavy;
  }
  std::vector<int64_t> prp((size_t)n + 1, 0), pirp((size_t)n + 1, 0);
  for (int64_t i = 0; i < n; ++i) {
    const size_t v = (size_t)orig[(size_t)i];
    prp[(size_t)i + 1] = prp[(size_t)i] + row_ptr[v + 1] - row_ptr[v];
    pirp[(size_t)i + 1] = pirp[(size_t)i] + irp[v + 1] - irp[v];
  }
  STCHK(dalloc(&g->d_prp, (size_t)n + 1));
  STCHK(dalloc(&g->d_pirp, (size_t)n + 1));
  STCHK(dalloc(&g->d_orig, (size_t)n));
  HIPCHK(hipMemcpy(g->d_prp, prp.data(), ((size_t)n + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
  HIPCHK(hipMemcpy(g->d_pirp, pirp.data(), ((size_t)n + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
  HIPCHK(hipMemcpy(g->d_orig, orig.data(), (size_t)n * sizeof(int32_t), hipMemcpyHostToDevice));
  if (weight) {
    STCHK(dalloc(&g->d_arcw, (size_t)m));
    STCHK(dalloc(&g->d_iarc, (size_t)m));
    STCHK(dalloc(&g->d_iopos, (size_t)m));
    if (m > 0) {
      std::vector<uint2> arcw((size_t)m), iarc((size_t)m);
      std::vector<uint32_t> iopos((size_t)m);
      for (int64_t i = 0; i < n; ++i) {
        const size_t v = (size_t)orig[(size_t)i];
        size_t p = (size_t)prp[(size_t)i];
        for (int64_t e = row_ptr[v]; e < row_ptr[v + 1]; ++e, ++p) {
          const size_t w = (size_t)col[e], j = (size_t)g->rank[w];
          arcw[p] = make_uint2((uint32_t)j, weight[e]);
          // an in-arc keeps its place in its row of the transpose
          iopos[(size_t)(pirp[j] + ((int64_t)ipos[(size_t)e] - irp[w]))] = (uint32_t)p;
        }
        p = (size_t)pirp[(size_t)i];
        for (int64_t e = irp[v]; e < irp[v + 1]; ++e, ++p)
          iarc[p] = make_uint2((uint32_t)g->rank[(size_t)icol[(size_t)e]], iw[(size_t)e]);
      }
      HIPCHK(hipMemcpy(g->d_arcw, arcw.data(), (size_t)m * sizeof(uint2), hipMemcpyHostToDevice));
      HIPCHK(hipMemcpy(g->d_iarc, iarc.data(), (size_t)m * sizeof(uint2), hipMemcpyHostToDevice));
      HIPCHK(hipMemcpy(g->d_iopos, iopos.data(), (size_t)m * sizeof(uint32_t), hipMemcpyHostToDevice));
    }
  }
  {
    STCHK(dalloc(&g->d_pcol, (size_t)m));
    if (!weight) STCHK(dalloc(&g->d_picol, (size_t)m));
    int32_t *d_rank = nullptr;
    STCHK(dalloc(&d_rank, (size_t)n));
    hipError_t e = hipMemcpy(d_rank, g->rank.data(), (size_t)n * sizeof(int32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess)
      e = launch_permute_rows(n, g->d_rp, g->d_col, g->d_prp, g->d_orig, d_rank, g->d_pcol, nullptr);
    if (e == hipSuccess && !weight)
      e = launch_permute_rows(n, g->d_irp, g->d_icol, g->d_pirp, g->d_orig, d_rank, g->d_picol, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    dfree(d_rank);
    if (e != hipSuccess) return hip_fail(e, "internal vertex order");
  }
  g->cfg.engine = BCD_ENGINE_BATCHED;
  g->cfg.groups = default_groups(n, weight != nullptr);
  // weighted kernels: one-wavefront workgroups, one resident grid (8 waves
  // per SIMD) -- 12 % faster than 256-thread blocks at R-MAT 18
  g->cfg.block = weight ? 64 : 256;
  g->cfg.grid_mult = 32;
  g->cfg.items = kDefaultItems;
  g->cfg.bottom_up = default_bottom_up(n);
  g->cfg.push = kDefaultPush;
  *out = reinterpret_cast<bcd_graph *>(g.release());
  return BCD_OK;
  BCD_GUARD_END
}

bcd_status bcd_graph_free(bcd_graph *g) {
  BCD_GUARD_BEGIN
  if (!g) return BCD_OK;
  delete reinterpret_cast<Graph *>(g);
  return BCD_OK;
  BCD_GUARD_END
}

bcd_status bcd_graph_info(const bcd_graph *gh, int64_t *n, int64_t *m, int32_t *weighted) {
  BCD_GUARD_BEGIN
  if (!gh) return fail(BCD_ERR_INVALID_ARG, "graph is NULL");
  const Graph *g = reinterpret_cast<const Graph *>(gh);
  if (n) *n = g->n;
  if (m) *m = g->m;
  if (weighted) *weighted = g->weighted ? 1 : 0;
  return BCD_OK;
  BCD_GUARD_END
}

bcd_status bcd_set_config(bcd_graph *gh, const bcd_config *cfg) {
  BCD_GUARD_BEGIN
  if (!gh || !cfg) return fail(BCD_ERR_INVALID_ARG, "NULL argument");
  Graph *g = reinterpret_cast<Graph *>(gh);
  if (cfg->engine != BCD_ENGINE_BATCHED && cfg->engine != BCD_ENGINE_PLAIN && cfg->engine != BCD_ENGINE_LDS)
    return fail(BCD_ERR_INVALID_ARG, "unknown engine");
  if (cfg->groups < 1 || (uint64_t)cfg->groups * (uint64_t)g->n >= (1ull << 32))
    return fail(BCD_ERR_INVALID_ARG, "groups must be >= 1 with groups * n < 2^32");
  if (cfg->block != 64 && cfg->block != 128 && cfg->block != 256 && cfg->block != 512)
    return fail(BCD_ERR_INVALID_ARG, "block must be 64, 128, 256 or 512");
  if (cfg->grid_mult < 1 || cfg->grid_mult > 32) return fail(BCD_ERR_INVALID_ARG, "grid_mult must be in [1, 32]");
  if (cfg->items != 0 && cfg->items != 1 && cfg->items != 2 && cfg->items != 4)
    return fail(BCD_ERR_INVALID_ARG, "items must be 1, 2 or 4 (0 = default)");
  if (cfg->bottom_up < -1 || cfg->bottom_up > 4096)
    return fail(BCD_ERR_INVALID_ARG, "bottom_up must be in [-1, 4096]");
  if (cfg->compress != 0 && cfg->compress != 1) return fail(BCD_ERR_INVALID_ARG, "compress must be 0 or 1");
  if (cfg->push < -1 || cfg->push > 1) return fail(BCD_ERR_INVALID_ARG, "push must be -1, 0 or 1");
  std::lock_guard<std::mutex> lk(g->cfg_mu);
  g->cfg = *cfg;
  if (g->cfg.items == 0) g->cfg.items = kDefaultItems;
  if (g->cfg.bottom_up < 0) g->cfg.bottom_up = default_bottom_up(g->n);
  if (g->cfg.push < 0) g->cfg.push = kDefaultPush;
  return BCD_OK;
  BCD_GUARD_END
}

bcd_status bcd_get_config(const bcd_graph *gh, bcd_config *cfg) {
  BCD_GUARD_BEGIN
  if (!gh || !cfg) return fail(BCD_ERR_INVALID_ARG, "NULL argument");
  *cfg = reinterpret_cast<const Graph *>(gh)->config();
  return BCD_OK;
  BCD_GUARD_END
}

bcd_status bcd_profile_enable(bcd_graph *gh, int32_t on) {
  BCD_GUARD_BEGIN
  if (!gh) return fail(BCD_ERR_INVALID_ARG, "graph is NULL");
  Graph *g = reinterpret_cast<Graph *>(gh);
  if (on) {
    std::lock_guard<std::mutex> lk(g->prof_mu);
    STCHK(g->mark_profile_origin());
  }
  g->profiling.store(on != 0);
  return BCD_OK;
  BCD_GUARD_END
}

bcd_status bcd_profile_get(const bcd_graph *gh, int32_t kind, bcd_kernel_profile *out) {
  BCD_GUARD_BEGIN
  if (!gh || !out || kind < 0 || kind > 1) return fail(BCD_ERR_INVALID_ARG, "bad argument");
  const Graph *g = reinterpret_cast<const Graph *>(gh);
  std::lock_guard<std::mutex> lk(g->prof_mu);
  *out = g->prof[kind];
  // measure of the union of the launch intervals (sweep over sorted starts)
  std::vector<std::pair<double, double>> iv = g->prof_iv[kind];
  std::sort(iv.begin(), iv.end());
  double u = 0.0, a = 0.0, b = -1.0;
  bool open = false;
  for (const auto &x : iv) {
    if (!open || x.first > b) {
      if (open) u += b - a;
      a = x.first;
      b = x.second;
      open = true;
    } else {
      b = std::max(b, x.second);
    }
  }
  if (open) u += b - a;
  // the union is at most the sum; the interval ends are single-precision
  // times after the origin, whose rounding can put it above where launches
  // hardly overlap
  out->union_ms = std::min(u + g->prof_solo_ms[kind], out->total_ms);
  return BCD_OK;
  BCD_GUARD_END
}

bcd_status bcd_profile_reset(bcd_graph *gh) {
  BCD_GUARD_BEGIN
  if (!gh) return fail(BCD_ERR_INVALID_ARG, "graph is NULL");
  Graph *g = reinterpret_cast<Graph *>(gh);
  std::lock_guard<std::mutex> lk(g->prof_mu);
  std::memset(g->prof, 0, sizeof(g->prof));
  for (int k = 0; k < 2; ++k) {
    g->prof_iv[k].clear();
    g->prof_solo_ms[k] = 0.0;
  }
  if (g->profiling.load()) STCHK(g->mark_profile_origin());
  return BCD_OK;
  BCD_GUARD_END
}

// Best-of-reps bandwidth of a copy (read = false: `bytes` read and `bytes`
// written per launch) or a read (`bytes` read per launch) over 16-byte words,
// 64 workgroups of 256 threads per compute unit, after one untimed launch.
static bcd_status stream_probe(int64_t bytes, int32_t reps, bool read, double *gbps) {
  if (bytes < 1024 || reps < 1 || !gbps) return fail(BCD_ERR_INVALID_ARG, "bad argument");
  int cus = 0;
  STCHK(device_check(&cus));
  const int64_t n16 = bytes / 16;
  const int grid = std::max(1, cus) * 64;
  uint8_t *a = nullptr, *b = nullptr;
  unsigned *sink = nullptr;
  STCHK(dalloc(&a, (size_t)n16 * 16));
  bcd_status rc = read ? dalloc(&sink, 4) : dalloc(&b, (size_t)n16 * 16);
  if (rc != BCD_OK) {
    dfree(a);
    return rc;
  }
  hipStream_t st;
  hipEvent_t e0, e1;
  if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) {
    dfree(a);
    dfree(b);
    dfree(sink);
    return fail(BCD_ERR_DEVICE, "stream create failed");
  }
  (void)hipEventCreate(&e0);
  (void)hipEventCreate(&e1);
  (void)hipMemsetAsync(a, 1, (size_t)n16 * 16, st);
  double best = 0;
  const double moved = (read ? 1.0 : 2.0) * (double)n16 * 16;
  for (int i = 0; i < reps + 1 && rc == BCD_OK; ++i) {
    (void)hipEventRecord(e0, st);
    const hipError_t e = read ? launch_read_probe(a, n16, sink, grid, st) : launch_copy_probe(a, b, n16, grid, st);
    if (e != hipSuccess) rc = fail(BCD_ERR_DEVICE, "probe launch failed");
    (void)hipEventRecord(e1, st);
    if (hipEventSynchronize(e1) != hipSuccess) rc = fail(BCD_ERR_DEVICE, "probe failed");
    float ms = 0;
    (void)hipEventElapsedTime(&ms, e0, e1);
    if (i > 0 && ms > 0) best = std::max(best, moved / (ms * 1e-3) / 1e9);
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipStreamDestroy(st);
  dfree(a);
  dfree(b);
  dfree(sink);
  if (rc == BCD_OK) *gbps = best;
  return rc;
}

bcd_status bcd_bandwidth_probe(int64_t bytes, int32_t reps, double *gbps) {
  BCD_GUARD_BEGIN
  return stream_probe(bytes, reps, false, gbps);
  BCD_GUARD_END
}

bcd_status bcd_read_bandwidth_probe(int64_t bytes, int32_t reps, double *gbps) {
  BCD_GUARD_BEGIN
  return stream_probe(bytes, reps, true, gbps);
  BCD_GUARD_END
}

}  // extern "C"

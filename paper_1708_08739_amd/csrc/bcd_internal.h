// Internal declarations shared by the host layer and the HIP kernels of
// libbcd.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bcd {

constexpr int kLanes = 64;  // sources per column group = wavefront width on gfx950

// Lane masks of the unweighted engine: one 64-bit word per (group, vertex) in
// each of these arrays, which follow each other in BatchState::msk.  A word
// array keeps 16 vertices to a 128-byte line, and as internal ids run by falling
// degree, the words of the vertices most arcs lead to are neighbours.
enum MaskArray {
  M_SEEN = 0,  // lanes settled, or flagged for the level being discovered
  M_FR = 1,    // 1..4: lanes of a level, by level mod 4 (current, next, previous, retiring)
  M_DN = 5,    // lanes on whose shortest-path DAG the vertex is a target or lies below one
  M_BW = 6,    // 6..8: lanes of a level the backward computed, by level mod 3
  M_COUNT = 9
};

// Counters accumulated per workgroup slot (no atomics), reduced on the host.
enum Ctr {
  C_FWD_VPAIRS = 0,  // (source, vertex) pairs expanded by the forward kernel
  C_FWD_APAIRS = 1,  // (source, arc) pairs scanned by the forward kernel  (= sum m_s)
  C_FWD_DPAIRS = 2,  // (source, DAG arc) pairs the forward kernel pushed sigma along (= sum a_s)
  C_BWD_VPAIRS = 3,  // (source, vertex) pairs whose psi the backward kernel produced
  C_BWD_APAIRS = 4,  // (source, arc) pairs the backward kernel scanned
  C_BWD_DPAIRS = 5,  // (source, DAG arc) pairs the backward kernel accumulated
  C_RLX_APAIRS = 6,  // (source, arc) relaxations of the weighted distance rounds (6..8)
  C_SCRATCH = 9,     // unused slots for kernels that only report overflow (9..11)
  C_FWD_ITEMS = 12,  // work items (64-source group, vertex, level) of the forward
  C_FWD_IARCS = 13,  // sum over those items of the vertex's out-degree
  C_BWD_ITEMS = 14,  // work items the backward computed psi for
  C_BWD_IARCS = 15,  // sum over those items of the vertex's out-degree
  C_COUNT = 16
};

// Device state of one batch of G column groups (64 sources each) over an
// n-vertex graph.  All [G][n][64] arrays are vertex-major inside a group, so
// the 64 sources of one vertex are one contiguous row a wavefront reads or
// writes with one coalesced access.
struct BatchState {
  int64_t n;
  int G;
  unsigned long long *sig;   // [G][n][64] path counts (rows of 64 uint32 when narrow)
  double *psi;               // [G][n][64] (1 + delta) / sigma
  double *dout;              // [G][n][64] delta, verification hook only (may be null)
  unsigned long long *msk;   // [M_COUNT][G][n] lane masks (unweighted engine, see MaskArray)
  unsigned long long *vis;   // [G][n] reached lanes (weighted engine)
  unsigned long long *fr;    // [3][G][n] rotating round masks (weighted engine)
  // Item lists are split into P partitions (group g belongs to partition
  // g % P); workgroup b serves partition b % P, so with P = 2 (workgroups
  // are dealt to the 8 XCDs round-robin) four XCDs walk each half of the
  // groups.  There are two lists per
  // partition and level: list p holds the vertices a wavefront takes alone,
  // list P + p the heavy ones (internal id < H), which a workgroup takes
  // together (unweighted engine) or several wavefronts in parts (weighted).
  uint32_t *items;           // [P * capP + P * capH] g * n + v, grouped by list, then level
  unsigned long long *imask; // the same shape: lanes of the item on its level
  uint64_t hbase;            // first item of the heavy lists (P * capP of the widest batch)
  uint64_t capP;             // items of list p: [p * capP, (p + 1) * capP)
  uint64_t capH;             // items of list P + p: [hbase + p * capH, hbase + (p + 1) * capH)
  int P;
  int NL;                    // lists: 2 P
  uint32_t H;                // heavy vertices: internal ids 0 .. H-1
  uint32_t *cnt;             // [(n + 2) * kMaxLists] items per (level, list): index level * NL + l
  uint32_t *tail;            // [4][kMaxLists] lengths of the lists being filled, by level mod 4, each in a
                             // 128-byte line of its own (see tail_at)
  uint64_t *off;             // [(n + 2) * kMaxLists] first item of each (level, list)
  uint32_t *tmin;            // [1] smallest over all lanes
  int32_t *tgt_of;           // [n] target index of a vertex, -1 if none
  double *res;               // [ntgt][G][64] delta of lane on target
  uint64_t *ctr;             // [grid][C_COUNT] per-workgroup counters
  uint64_t *acc;             // [C_COUNT] counters of completed batches
  uint32_t *flags;           // [4]: 0 sigma overflow, 1 item capacity exceeded, 2 a count too wide for a narrow row
  unsigned long long *ovl;   // [G] lanes whose sigma overflowed, then [G] lanes whose source is a target
  int ctr_slots;
  // per batch (unweighted engine)
  int gused;                     // column groups holding sources: 0 .. gused-1
  unsigned long long last_lanes; // lanes of group gused-1 that hold a source
  int bu_den;                    // bottom-up levels: see level_bottom_up (0 = never)
  int top;                       // deepest level of the batch (set before the backward)
  int keep_all;                  // 1: the backward runs on every lane (exports), else only below a target
  int push;                      // 1: top-down levels push path counts along DAG arcs (k_fwd_push), 0: pull
  int narrow;                // 1: path counts stored in 32 bits (pulled counts only)
  // weighted graphs only
  uint32_t *wd;              // [G][n][64] distances, 0xFFFFFFFF unreached
  uint32_t *wc;              // [G][n][64] shortest-path-DAG in-arcs not yet pushed
  unsigned long long *chg;   // [3][G][n] lanes whose distance dropped, by relaxation round mod 3
  uint32_t *bq;              // [3][queue] items changed in a round, by round mod 3 (lists as of `items`)
  uint32_t *rl;              // [queue] items reached by any lane
  uint32_t *qtail;           // [4][kMaxLists] lengths of a round's queue lists, by round mod 4, a line each (qtail_at)
  uint32_t *rtail;           // [kMaxLists] lengths of the reached lists, a line each (rtail_at)
  uint64_t capQ, capQH;      // a queue's list p: [p * capQ, (p + 1) * capQ), list P + p:
  uint64_t qhbase, qsize;    //   [qhbase + p * capQH, ...); its size
  unsigned long long *wdn;   // [G][n] lanes on whose DAG the vertex is a target or lies below one
  unsigned long long *dagm;  // [G][m] lanes on whose shortest-path DAG the arc lies, in CSR order
};

// Plain engine state (one source).
struct PlainState {
  int64_t n;
  int32_t *d;                // [n] level, -1 unreached
  unsigned long long *sig;   // [n]
  double *psi;               // [n]
  double *dout;              // [n] delta, verification only
  int32_t *queue;            // [n] vertices by level
  uint32_t *cnt;             // [n + 2]
  uint64_t *off;             // [n + 2]
  uint64_t *ctr;             // [grid][C_COUNT]
  uint64_t *acc;             // [C_COUNT]
  uint32_t *flags;           // [4]
  int ctr_slots;
};

// The graph as kernels see it, in the caller's vertex ids (reachability, the
// plain and LDS engines) or in internal ids (batched and weighted engines).
// Internal ids number the vertices by falling total degree, so that heavy
// vertices are told by an id comparison; every row keeps its arcs in the
// caller's order, so sums over a row run in the same order either way.
struct DevGraph {
  int64_t n, m;
  const int64_t *rp;    // [n+1]
  const int32_t *col;   // [m]
  const int64_t *irp;   // transpose
  const int32_t *icol;
  // weighted graphs: arc fields in pairs, so that one 8-byte load brings what
  // a kernel reads of an arc (separate 4-byte arrays and one 16-byte record
  // of all fields both measured slower)
  const uint2 *arcw;    // [m] CSR order: {head, length} (relaxation)
  const uint2 *iarc;    // [m] transpose order: {tail, length} (DAG in-degrees)
  const uint32_t *iopos;  // [m] transpose order: position of the arc in the CSR
  const int32_t *orig;  // [n] caller's id of an internal id (exports)
};

// Whether BFS level `level` (>= 2) of a batch is found bottom-up, from the
// item count of level-1 (complete before any kernel of `level` starts):
// when level-1 holds at least 1 / bu_den of the batch's (group, vertex)
// pairs, scanning the in-arcs of the unsettled pairs is cheaper than the
// out-arcs of the frontier.  Host and device evaluate the same integer rule.
__host__ __device__ inline bool bottom_up_rule(int bu_den, int level, uint64_t prev_count, int gused, int64_t n) {
  return bu_den > 0 && level >= 2 && prev_count * (uint64_t)bu_den >= (uint64_t)gused * (uint64_t)n;
}

struct Launch {
  int block;      // threads per workgroup
  int grid;       // workgroups
  int items = 1;  // items per wavefront step (pushed levels)
};

// ---- launchers (bcd_kernels.hip) ----
constexpr int kMaxLists = 4;  // two per partition (kMaxParts)
struct PartTotals {
  uint64_t t[kMaxLists];  // items per list over all levels of a batch
};
// Length of list l of a level while the level is being filled and read.  Every
// workgroup reads these words at the start of a launch and appends to the next
// level's through atomics from its own XCD, so neighbours in one line cost
// both sides: with a level's counters packed beside the next level's, a
// 601-vertex graph's levels took up to 156 us, with a line each up to 28.
constexpr int kTailStride = 32;
__host__ __device__ inline uint32_t *tail_at(const BatchState &S, int level, int l) {
  return S.tail + ((level & 3) * kMaxLists + l) * kTailStride;
}
__host__ __device__ inline uint32_t *qtail_at(const BatchState &S, int round, int l) {
  return S.qtail + ((round & 3) * kMaxLists + l) * kTailStride;
}
__host__ __device__ inline uint32_t *rtail_at(const BatchState &S, int l) { return S.rtail + l * kTailStride; }
// First item of list l in a relaxation queue (and in the reached list).
__host__ __device__ inline uint64_t queue_begin(const BatchState &S, int l) {
  return l < S.P ? (uint64_t)l * S.capQ : S.qhbase + (uint64_t)(l - S.P) * S.capQH;
}
__host__ __device__ inline uint64_t queue_end(const BatchState &S, int l) {
  return queue_begin(S, l) + (l < S.P ? S.capQ : S.capQH);
}
// First item of list l's region.
__host__ __device__ inline uint64_t list_begin(const BatchState &S, int l) {
  return l < S.P ? (uint64_t)l * S.capP : S.hbase + (uint64_t)(l - S.P) * S.capH;
}
__host__ __device__ inline uint64_t list_end(const BatchState &S, int l) {
  return list_begin(S, l) + (l < S.P ? S.capP : S.capH);
}
// List of vertex v (internal id) of group g, and the level-0 slot of a staged
// item that is the at-th of its list.  The slot is 64-bit: a heavy list begins
// behind all light ones, which grow to 64 items a (group, vertex), past 2^32.
__host__ __device__ inline int list_of(const BatchState &S, uint32_t g, uint32_t v) {
  return (int)(g % (uint32_t)S.P) + (v < S.H ? S.P : 0);
}
__host__ __device__ inline uint64_t level0_slot(const BatchState &S, uint32_t item, uint32_t at) {
  const uint32_t g = item / (uint32_t)S.n;
  return list_begin(S, list_of(S, g, item - g * (uint32_t)S.n)) + at;
}
hipError_t launch_batch_init(const BatchState &S, const uint32_t *items0, const unsigned long long *masks0,
                             const uint32_t *dest0, int k, hipStream_t st);
hipError_t launch_fwd_level(const DevGraph &G, const BatchState &S, int level, Launch L, hipStream_t st);
// cnt row of a level that is filled but whose launch has not run yet
hipError_t launch_publish_counts(const BatchState &S, int level, hipStream_t st);
hipError_t launch_bu_level(const DevGraph &G, const BatchState &S, int level, Launch L, hipStream_t st);
// Workgroups of a backward level of cnt[l] items on list l that also clears the
// masks of cleared[l] items (null: none): a wavefront per light item and per
// eighth of a heavy one (ListView deals a third of a partition's workgroups to
// those), a thread per mask, at most L's.  Deep graphs have thousands of levels
// of few items, and a workgroup without work still takes its LDS and adds its
// counters: a cycle of 1,500 vertices, every source (1,500 items a level), 15.6 us
// a level on 8,192 workgroups, 5.5 as here.
inline int bwd_level_grid(const BatchState &S, const Launch &L, const uint32_t *cnt, const uint32_t *cleared) {
  const uint64_t nw = (uint64_t)(L.block / 64);
  uint64_t nwg = 2;
  for (int p = 0; p < S.P; ++p) {
    const uint64_t light = (cnt[p] + nw - 1) / nw, heavy = ((uint64_t)cnt[S.P + p] * 8 + nw - 1) / nw;
    const uint64_t masks = cleared ? ((uint64_t)cleared[p] + cleared[S.P + p]) / (uint64_t)L.block + 1 : 0;
    nwg = nwg > masks ? nwg : masks;
    const uint64_t items = S.H == 0 ? light : light + light / 2 + 2;
    nwg = nwg > items ? nwg : items;
    nwg = heavy == 0 || nwg > 3 * heavy + 3 ? nwg : 3 * heavy + 3;
  }
  return nwg * (uint64_t)S.P < (uint64_t)L.grid ? (int)(nwg * (uint64_t)S.P) : L.grid;
}
hipError_t launch_bwd_level(const DevGraph &G, const BatchState &S, int level, int ntgt, Launch L, hipStream_t st);
hipError_t launch_batch_cleanup(const BatchState &S, const PartTotals &tot, Launch L, hipStream_t st);
hipError_t launch_batch_export(const DevGraph &G, const BatchState &S, int level, uint64_t begin, uint64_t count,
                               const int32_t *lane_slot, uint64_t *dist, unsigned long long *sigma,
                               double *delta, int64_t k, hipStream_t st);

hipError_t launch_plain_init(const PlainState &P, int32_t s, hipStream_t st);
hipError_t launch_plain_fwd(const DevGraph &G, const PlainState &P, int level, Launch L, hipStream_t st);
hipError_t launch_plain_bwd(const DevGraph &G, const PlainState &P, int level, int32_t target, int full,
                            Launch L, hipStream_t st);
hipError_t launch_plain_cleanup(const PlainState &P, uint64_t total, hipStream_t st);
hipError_t launch_plain_export(const PlainState &P, uint64_t total, uint64_t *dist,
                               unsigned long long *sigma, double *delta, hipStream_t st);

// Reachability BFS over one CSR (reverse graph for RV, forward for FR).
// Counters of the frontiers, by level mod 4: the queue's length and the arcs
// its vertices have in the traversed CSR, `stride` words apart; word 1 holds the
// deepest level that had vertices.
struct ReachCtr {
  uint32_t *c;
  int stride;
  __host__ __device__ uint32_t *len(int level) const { return c + (level & 3) * stride; }
  __host__ __device__ uint64_t *arcs(int level) const {
    return reinterpret_cast<uint64_t *>(c + (level & 3) * stride + 2);
  }
};
// Clears the bitmap and the counters, then enters the roots (root, or
// roots[0 .. k-1] on the device when roots is not null).
hipError_t launch_reach_init(uint32_t *bitmap, int64_t words, int32_t *q, ReachCtr ctr, int32_t root,
                             const int32_t *roots, int k, hipStream_t st);
// Launch of a reachability level: workgroups of 256 threads for as many
// wavefronts as the configured shape L has, at most 1,024 workgroups.
constexpr int kReachLevelBlock = 256;
inline int reach_level_grid(const Launch &L) {
  const int64_t wg = (int64_t)L.grid * L.block / kReachLevelBlock;
  return (int)(wg < 1 ? 1 : wg > 1024 ? 1024 : wg);
}
// One level: rp / col is the CSR traversed, rpo / colo the other direction; a
// level whose frontier has at least bu_arcs arcs goes bottom-up.
hipError_t launch_reach_level(const int64_t *rp, const int32_t *col, const int64_t *rpo, const int32_t *colo,
                              uint32_t *bitmap, int32_t *q0, int32_t *q1, ReachCtr ctr, uint8_t *lev, int level,
                              int64_t n, uint64_t bu_arcs, Launch L, hipStream_t st);
hipError_t launch_scatter_targets(int32_t *tgt_of, const int32_t *verts, int k, int set, hipStream_t st);
hipError_t launch_plain_gather(const PlainState &P, const int32_t *verts, int k, int32_t *d_out,
                               double *delta_out, hipStream_t st);
// What the load derives on the device.
struct LoadArgs {
  int64_t n, m;
  const int32_t *rank;     // [n] internal id of a caller's id
  // weighted graphs: the transpose as {tail, CSR position} and the lengths in CSR
  // order (inputs), the arrays of DevGraph made of them and the transpose's tails
  const uint2 *pairs;
  const uint32_t *weight;
  int32_t *icol;
  uint32_t *iopos;
  uint2 *arcw, *iarc;
  uint32_t *lrp;           // LDS engine's rows, or null
  uint16_t *lcol;
};
// Rows of both CSRs in internal order: row i of a new one holds the arcs of row
// orig[i] in the same order, their ends renamed by rank (weighted: with the
// arcs' lengths and positions).
hipError_t launch_internal_rows(const DevGraph &from, const DevGraph &to, int32_t *pcol, int32_t *picol,
                                const LoadArgs &A, hipStream_t st);
// weighted engine (bcd_weighted.hip)
hipError_t launch_w_init(const BatchState &S, const uint32_t *items0, const unsigned long long *masks0,
                         const uint32_t *dest0, int k, hipStream_t st);
hipError_t launch_w_relax(const DevGraph &G, const BatchState &S, int round, Launch L, hipStream_t st);
hipError_t launch_w_count(const DevGraph &G, const BatchState &S, Launch L, hipStream_t st);
hipError_t launch_w_sigma(const DevGraph &G, const BatchState &S, int round, Launch L, hipStream_t st);
hipError_t launch_w_bwd(const DevGraph &G, const BatchState &S, int round, int ntgt, int full, Launch L,
                        hipStream_t st);
hipError_t launch_w_cleanup(const BatchState &S, Launch L, hipStream_t st);
hipError_t launch_w_export(const DevGraph &G, const BatchState &S, const int32_t *lane_slot, uint64_t *dist,
                           unsigned long long *sigma, double *delta, int64_t k, Launch L, hipStream_t st);
struct ResultRoute {
  double *dst;      // device address in a query's result buffer
  uint32_t src;     // index into res ([ntgt][G][64])
  uint32_t pad;
};
hipError_t launch_route_results(const double *res, const ResultRoute *routes, int k, hipStream_t st);
// Add the per-workgroup counter slots into acc[C_COUNT] and zero them (one
// launch after every completed batch; an aborted batch just zeroes them).
hipError_t launch_ctr_fold(uint64_t *ctr, int slots, uint64_t *acc, hipStream_t st);
hipError_t launch_copy_probe(const void *src, void *dst, int64_t n16, int grid, hipStream_t st);
hipError_t launch_read_probe(const void *src, int64_t n16, unsigned *sink, int grid, hipStream_t st);

}  // namespace bcd

// Weighted graphs (positive integer arc lengths, Section 2): the per-source
// pass for 64 sources per wavefront lane group.
//
//   1. distances: rounds of label-correcting relaxation; lane b lowers
//      dist_b(w) with atomicMin and flags (g, w) for the next round;
//   2. shortest-path-DAG in-degrees: for every reached (g, w), count the
//      in-arcs (u, w) with dist_b(u) + len(u, w) = dist_b(w) (a pull over the
//      reverse graph), and store each in-arc's lanes of that test as one
//      64-bit mask per (group, arc), so that steps 3 and 4 find the DAG lanes
//      of an arc in one word instead of a distance per lane.  The masks lie in
//      CSR order: written once per arc at scattered places, and read by lanes
//      over consecutive arcs in every round that holds the tail;
//   3. path counts in topological rounds: a lane of a vertex is ready when
//      all its DAG in-arcs have pushed; it then pushes sigma along its DAG
//      out-arcs and counts them down (Kahn's order on each source's SPD);
//   4. backward: Eq.(4) over the rounds of step 3 in reverse -- every DAG
//      successor of v became ready in a later round, so its psi is final.
// Step 3's round of a vertex plays the role of the BFS level of the
// unweighted engine; the backward computes psi only on lanes where the
// vertex is a target or lies below one (marks OR'd along the sigma pushes).
//
// Work lists are kept per partition and split in light and heavy items
// as in the unweighted engine; a heavy item is taken in kParts parts of its
// arcs by as many wavefronts (nothing but atomics joins them, except in the
// backward, whose sums run in arc order and stay with one wavefront).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "../../include/bcd.h"
#include "bcd_device.h"
#include "bcd_host_internal.h"

namespace bcd {

constexpr uint32_t kInf = 0xFFFFFFFFu;

// Parts a heavy item's arcs are dealt in (R-MAT 18, 2,048 draws, on one box: 8
// parts 130.5 ms, 16 131.0, 32 135.5; 8,191-vertex exact 19.27 / 19.17 / 19.5).
constexpr uint32_t kParts = 16;
// Light items a wavefront takes at a time, at most.  Rows are uneven, and on a
// small graph a round waits for the block with the longest: weighted R-MAT 13
// exact / R-MAT 18 with 2,048 draws, ms, at 4 / 8 / 16 / 32 items: 13.3 / 13.6 / 14.5 /
// 16.1 and 101.3 / 98.6 / 98.0 / 98.5.
constexpr int kWBlockItems = 8;

// The lists of the relaxation queue being filled, and the reached lists.
struct QueueLists {
  const BatchState &S;
  int round;  // the round the queue is for
  __device__ __forceinline__ uint32_t *tail(int l) const { return qtail_at(S, round, l); }
  __device__ __forceinline__ uint64_t base(int l) const { return queue_begin(S, l); }
  __device__ __forceinline__ uint64_t end(int l) const { return queue_end(S, l); }
  __device__ __forceinline__ uint32_t *dst() const { return S.bq + (uint64_t)(round % 3) * S.qsize; }
};
struct ReachLists {
  const BatchState &S;
  __device__ __forceinline__ uint32_t *tail(int l) const { return rtail_at(S, l); }
  __device__ __forceinline__ uint64_t base(int l) const { return queue_begin(S, l); }
  __device__ __forceinline__ uint64_t end(int l) const { return queue_end(S, l); }
  __device__ __forceinline__ uint32_t *dst() const { return S.rl; }
};

__global__ void k_w_init(BatchState S, const uint32_t *items0, const ull *masks0, const uint32_t *dest0, int k) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < k; i += gridDim.x * blockDim.x) {
    const uint32_t it = items0[i];
    const ull m = masks0[i];
    const uint32_t g = it / (uint32_t)S.n, v = it - g * (uint32_t)S.n;
    const uint64_t q = queue_begin(S, list_of(S, g, v)) + dest0[i];
    S.fr[it] = m;       // topological round 0
    S.items[level0_slot(S, it, dest0[i])] = it;
    S.chg[it] = m;      // relaxation round 0: the sources changed
    S.bq[q] = it;
    S.rl[q] = it;
    S.vis[it] = m;      // reached lanes
    for (int b = 0; b < kLanes; ++b)
      if ((m >> b) & 1ull) {
        S.sig[(size_t)it * kLanes + b] = 1ull;
        S.wd[(size_t)it * kLanes + b] = 0u;
      }
  }
  if (blockIdx.x == 0 && threadIdx.x < (unsigned)S.NL) {
    const int l = (int)threadIdx.x;
    const uint32_t c = S.cnt[l];
    S.off[l] = list_begin(S, l);
    *tail_at(S, 0, l) = c;
    *tail_at(S, 1, l) = 0u;
    *tail_at(S, 2, l) = 0u;
    *qtail_at(S, 0, l) = c;
    *qtail_at(S, 1, l) = 0u;
    *qtail_at(S, 2, l) = 0u;
    *rtail_at(S, l) = c;
  }
}

// Part `part` of a heavy item's `deg` arcs: first arc and number.
static __device__ __forceinline__ void part_of(uint32_t deg, uint32_t part, uint32_t &first, uint32_t &num) {
  first = (uint32_t)((uint64_t)deg * part / kParts);
  num = (uint32_t)((uint64_t)deg * (part + 1) / kParts) - first;
}

// Lane compaction for one work item: the A lanes of `em` are renumbered
// 0..A-1 in lane order; lane L of the wavefront then serves source lane
// `src` (the one of number L mod A) on arc slot L / A of `slots` = 64 / A
// (slot >= slots: idle).  With few lanes per item the wavefront thus covers
// `slots` arcs of every source at once instead of one.  Wave-uniform `em`.
struct Compact {
  int A, slots, j, slot, src;
};
// Arcs per slot per step of the relaxation: four, so that each lane has four
// distance reads in flight before it waits (R-MAT 18, 2,048 draws: 131 ms; with
// two 135).
constexpr int kWU = 4;

// Orders this wavefront's LDS accesses before and after the call (lanes of
// one wavefront exchanging values through LDS).
static __device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// 64-bit lane shuffle (any source lane, every lane taking part).
static __device__ __forceinline__ ull shfl64_w(ull x, int src) {
  const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)x, src);
  const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(x >> 32), src);
  return ((ull)hi << 32) | lo;
}

static __device__ __forceinline__ Compact compact_lanes(ull em, bool mine) {
  Compact c;
  const int lane = lane_id();
  c.A = __popcll(em);
  c.slots = kLanes / c.A;
  // lane of number r learns its lane id (push: a bijection of all 64 lanes)
  const int rk = mine ? lanes_below(em) : c.A + lanes_below(~em);
  const int id = __builtin_amdgcn_ds_permute(rk * 4, lane);
  c.j = lane % c.A;
  c.slot = lane / c.A;
  c.src = __shfl(id, c.j);
  return c;
}

// One relaxation round.  Input: the queue of `round` with changed-lane masks
// chg[round % 3]; output: the queue and masks of round + 1; the masks of
// round - 1 are retired (their word is the one round + 2 collects).  A
// wavefront takes a block of light items (their masks and row bounds loaded
// with a lane per item) or one part of a heavy item; lanes are compacted per
// item (compact_lanes), the next arcs are loaded while the heads' distances of
// the current ones are compared.
// Bound by the latency of random accesses.  With one queue for all groups and
// XCDs, its counters in one cache line and every item walked by one wavefront
// the rounds of R-MAT 18 with 2,048 sources took 138 ms, as here 60; sigma
// rounds 85 and 49, in-degrees 21 and 14, the backward 18 and 8.  Held to 5 waves
// per SIMD or more the compiler takes 79 registers, left alone 89 (131 against
// 135 ms for the query; 8 waves 136).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(5, 8))) void k_w_relax(DevGraph G, BatchState S, int round) {
  constexpr int NW = BLOCK / 64;
  const uint32_t n = (uint32_t)S.n;
  const uint64_t GN = (uint64_t)S.G * n;
  const int P = S.P;
  const PartView pv = part_view<BLOCK>(P);
  const uint32_t nl = *qtail_at(S, round, pv.p), nh = *qtail_at(S, round, P + pv.p);
  if (pv.thread == 0) {
    *qtail_at(S, round + 2, pv.p) = 0u;
    *qtail_at(S, round + 2, P + pv.p) = 0u;
  }
  if ((nl | nh) == 0u) return;  // this partition has converged
  if (round > 0) {
    ull *old = S.chg + (uint64_t)((round + 2) % 3) * GN;
    const uint32_t *qold = S.bq + (uint64_t)((round + 2) % 3) * S.qsize;
    for (int l = pv.p; l < S.NL; l += P) {
      const uint64_t qb = queue_begin(S, l), qc = *qtail_at(S, round - 1, l);
      for (uint64_t i = pv.thread; i < qc; i += pv.nthreads) old[qold[qb + i]] = 0ull;
    }
  }
  const ull *ccur = S.chg + (uint64_t)(round % 3) * GN;
  ull *cnxt = S.chg + (uint64_t)((round + 1) % 3) * GN;
  const int lane = lane_id();
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  uint64_t c_r = 0;
  __shared__ uint32_t qst_all[NW * kStage], qht_all[NW * kStageHeavy];
  __shared__ uint32_t rst_all[NW * kStage], rht_all[NW * kStageHeavy];
  Stage qs = {qst_all + wv * kStage, qht_all + wv * kStageHeavy, 0, 0};
  Stage rs = {rst_all + wv * kStage, rht_all + wv * kStageHeavy, 0, 0};
  const QueueLists qlists{S, round + 1};
  const ReachLists rlists{S};
  // per slot: the lanes that improved the slot's head in this step, and those
  // that reached it first, combined so that the head's flags take one atomic
  // per step, not one per source
  __shared__ ull cm_all[BLOCK], cr_all[BLOCK];
  ull *cm = cm_all + wv * 64;
  ull *cr = cr_all + wv * 64;
  cm[lane] = 0ull;
  cr[lane] = 0ull;
  wave_lds_sync();
  const ListView lv = list_view(S);
  const uint32_t *qin = S.bq + (uint64_t)(round % 3) * S.qsize + queue_begin(S, (lv.heavy ? P : 0) + pv.p);
  const uint64_t count = lv.heavy ? (uint64_t)nh * kParts : nl;
  const uint64_t nwv = lv.nwg * NW;
  const uint32_t B = lv.heavy ? 1u : (uint32_t)min((uint64_t)kWBlockItems, (count + nwv - 1) / nwv);
  for (uint64_t b0 = (lv.wg * NW + (uint64_t)wv) * B; b0 < count; b0 += nwv * B) {
    const int nb = (int)min((uint64_t)B, count - b0);
    uint32_t it = 0, gb = 0, e0 = 0, ed = 0;
    ull mk = 0ull;
    if (lane < nb) {
      it = qin[lv.heavy ? b0 / kParts : b0 + lane];
      const uint32_t v = it % n;
      gb = it - v;
      mk = ccur[it];
      const int64_t r0 = G.rp[v];
      e0 = (uint32_t)r0;
      ed = (uint32_t)(G.rp[v + 1] - r0);
      if (lv.heavy) {
        uint32_t f;
        part_of(ed, (uint32_t)(b0 % kParts), f, ed);
        e0 += f;
      }
    }
    c_r += wave_sum((uint64_t)__popcll(mk) * ed);
    // distances of the first item's sources; the next item's are loaded while
    // one is relaxed
    uint32_t dnext = S.wd[(uint64_t)read_lane(it, 0) * kLanes + lane];
    for (int j = 0; j < nb; ++j) {
      const uint32_t drow = dnext;
      if (j + 1 < nb) dnext = S.wd[(uint64_t)read_lane(it, j + 1) * kLanes + lane];
      const ull mask = read_lane64(mk, j);
      const uint32_t dj = read_lane(ed, j), gj = read_lane(gb, j);
      if (mask == 0ull || dj == 0u) continue;
      const uint2 *arcs = G.arcw + read_lane(e0, j);
      const Compact cp = compact_lanes(mask, (mask >> lane) & 1ull);
      const bool on = cp.slot < cp.slots;
      const uint32_t dv = (uint32_t)__shfl((int)drow, cp.src);
      const bool live = on && dv != kInf;
      const ull bit = 1ull << cp.src;
      const uint32_t stepw = (uint32_t)cp.slots * kWU;
      uint2 a[kWU];
#pragma unroll
      for (int u = 0; u < kWU; ++u) {
        const uint32_t k = (uint32_t)(u * cp.slots + cp.slot);
        a[u] = arcs[k < dj ? k : 0u];
      }
      for (uint32_t k0 = 0; k0 < dj; k0 += stepw) {
        uint32_t wq[kWU], nd[kWU], dw[kWU];
#pragma unroll
        for (int u = 0; u < kWU; ++u) {
          wq[u] = a[u].x;
          nd[u] = (live && k0 + (uint32_t)(u * cp.slots + cp.slot) < dj) ? dv + a[u].y : kInf;
        }
#pragma unroll
        for (int u = 0; u < kWU; ++u)
          dw[u] = nd[u] != kInf ? S.wd[(uint64_t)(gj + wq[u]) * kLanes + (uint32_t)cp.src] : 0u;
#pragma unroll
        for (int u = 0; u < kWU; ++u) {
          const uint64_t k = (uint64_t)k0 + stepw + (uint32_t)(u * cp.slots + cp.slot);
          a[u] = arcs[k < dj ? k : 0u];
        }
        // a lower tentative distance: lower it (the minimum wins whatever the
        // order) and flag the vertex for the next round; a flag raised by a
        // value another wavefront has already beaten only costs a re-scan
        bool imp[kWU];
#pragma unroll
        for (int u = 0; u < kWU; ++u) {
          imp[u] = nd[u] != kInf && nd[u] < dw[u];
          if (imp[u])
            __hip_atomic_fetch_min(&S.wd[(uint64_t)(gj + wq[u]) * kLanes + (uint32_t)cp.src], nd[u], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        // all flags are issued before the result of any is used
        ull oldq[kWU], oldr[kWU];
#pragma unroll
        for (int u = 0; u < kWU; ++u) {
          oldq[u] = ~0ull;
          oldr[u] = ~0ull;
          if (__ballot(imp[u]) == 0ull) continue;  // nothing improved on this arc slot (wave-uniform)
          // a lane that read the head unreached: the wavefront whose lowering
          // of a lane lands first read it unreached, so the pair's first reach
          // is among these and the reached list needs no atomic for the others
          const bool fst = imp[u] && dw[u] == kInf;
          if (imp[u]) __hip_atomic_fetch_or(&cm[cp.slot], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
          if (fst) __hip_atomic_fetch_or(&cr[cp.slot], bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
          wave_lds_sync();
          ull m = 0ull, mr = 0ull;
          if (cp.j == 0 && on) {
            m = cm[cp.slot];
            mr = cr[cp.slot];
            cm[cp.slot] = 0ull;
            cr[cp.slot] = 0ull;
          }
          wave_lds_sync();
          if (m != 0ull) oldq[u] = atomicOr(&cnxt[gj + wq[u]], m);
          if (mr != 0ull) oldr[u] = atomicOr(&S.vis[gj + wq[u]], mr);
        }
#pragma unroll
        for (int u = 0; u < kWU; ++u) {
          append_chunk(S, qlists, pv.p, qs, gj, wq[u], oldq[u] == 0ull);
          append_chunk(S, rlists, pv.p, rs, gj, wq[u], oldr[u] == 0ull);
        }
      }
    }
  }
  flush_stage(S, qlists, pv.p, qs);
  flush_stage(S, rlists, pv.p, rs);
  const int ck[1] = {C_RLX_APAIRS};
  const uint64_t cv[1] = {c_r};
  flush_wave_counters<BLOCK, 1>(S.ctr, S.ctr_slots, ck, cv, false, S.flags);
}

// DAG in-degree of every reached (g, w) on each lane, pulled over in-arcs, and
// the DAG lanes of every in-arc.  A wavefront reads 64 in-arcs at a time with
// a lane each, then the tails' distance rows eight at a time; lane q keeps the
// DAG lanes of arc q, and the 64 masks go out as one store.  The parts of a
// heavy vertex add their counts.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_w_count(DevGraph G, BatchState S) {
  constexpr int NW = BLOCK / 64;
  const uint32_t n = (uint32_t)S.n;
  const int P = S.P;
  const PartView pv = part_view<BLOCK>(P);
  const int lane = lane_id();
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  uint64_t c_v = 0, c_a = 0, c_d = 0;
  const ListView lv = list_view(S);
  const int l = (lv.heavy ? P : 0) + pv.p;
  const uint32_t *rl = S.rl + queue_begin(S, l);
  const uint64_t len = *rtail_at(S, l), count = lv.heavy ? len * kParts : len;
  const uint64_t nwv = lv.nwg * NW;
  const uint32_t B = lv.heavy ? 1u : (uint32_t)min((uint64_t)kWBlockItems, (count + nwv - 1) / nwv);
  for (uint64_t b0 = (lv.wg * NW + (uint64_t)wv) * B; b0 < count; b0 += nwv * B) {
    const int nb = (int)min((uint64_t)B, count - b0);
    uint32_t it = 0, gb = 0, f0 = 0, fd = 0, od = 0;
    if (lane < nb) {
      it = rl[lv.heavy ? b0 / kParts : b0 + lane];
      const uint32_t v = it % n;
      gb = it - v;
      const int64_t r0 = G.irp[v];
      f0 = (uint32_t)r0;
      fd = (uint32_t)(G.irp[v + 1] - r0);
      od = (uint32_t)(G.rp[v + 1] - G.rp[v]);
      if (lv.heavy) {
        uint32_t f;
        part_of(fd, (uint32_t)(b0 % kParts), f, fd);
        f0 += f;
      }
    }
    const bool first_part = !lv.heavy || b0 % kParts == 0;
    for (int j = 0; j < nb; ++j) {
      const uint32_t ij = read_lane(it, j), gj = read_lane(gb, j), dj = read_lane(fd, j);
      const uint32_t dw = S.wd[(uint64_t)ij * kLanes + lane];
      const bool fin = dw != kInf;
      const uint2 *arcs = G.iarc + read_lane(f0, j);
      const uint32_t *opos = G.iopos + read_lane(f0, j);
      ull *dm = S.dagm + (uint64_t)(gj / n) * (uint64_t)G.m;
      uint32_t c = 0;
      for (uint32_t k = 0; k < dj; k += kLanes) {
        const uint32_t at = k + (uint32_t)lane < dj ? k + (uint32_t)lane : 0u;
        const uint2 a = arcs[at];
        const uint32_t op = opos[at];
        const int cc = (int)min(dj - k, (uint32_t)kLanes);
        ull mine = 0ull;
        for (int q0 = 0; q0 < cc; q0 += 8) {
          uint32_t du[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            du[q] = kInf;
            if (q0 + q < cc && fin) du[q] = S.wd[(uint64_t)(gj + read_lane(a.x, q0 + q)) * kLanes + lane];
          }
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const bool dag = du[q] != kInf && du[q] + read_lane(a.y, (q0 + q) & 63) == dw;
            if (dag) ++c;
            const ull bq = __ballot(dag);
            if (lane == q0 + q) mine = bq;
          }
        }
        if (lane < cc) dm[op] = mine;
      }
      if (!lv.heavy) S.wc[(uint64_t)ij * kLanes + lane] = c;
      else if (c != 0u) atomicAdd(&S.wc[(uint64_t)ij * kLanes + lane], c);
      c_d += c;
      const ull fm = __ballot(fin);
      if (lane == 0 && first_part) {
        c_v += (uint64_t)__popcll(fm);
        c_a += (uint64_t)__popcll(fm) * read_lane(od, j);
      }
    }
  }
  flush_counters<BLOCK>(S.ctr, S.ctr_slots, C_FWD_VPAIRS, c_v, c_a, c_d, false, S.flags);
}

// One topological round: items whose lanes became ready push sigma along
// their DAG out-arcs; a lane of w whose last DAG in-arc pushed is ready next
// round.  Level lists, rotation of the mask arrays and target bookkeeping
// mirror the unweighted forward kernel.  A wavefront lane takes one out-arc
// of the item and its DAG mask word (consecutive words), so the DAG test costs
// one coalesced load for 64 arcs and all 64 sources; pushes happen only on the
// (source, arc) pairs of the DAG, two sources of an arc at a time, and a
// head's ready and below-target lanes take one atomic each.  The next step's
// arcs and words and the next item's counts are loaded ahead.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_w_sigma(DevGraph G, BatchState S, int level) {
  constexpr int NW = BLOCK / 64;
  const uint32_t n = (uint32_t)S.n;
  const uint64_t GN = (uint64_t)S.G * n;
  const int P = S.P, NL = S.NL;
  const PartView pv = part_view<BLOCK>(P);
  const uint64_t lrow = (uint64_t)level * NL;
  const uint32_t nl = *tail_at(S, level, pv.p), nh = *tail_at(S, level, P + pv.p);
  {
    const uint64_t nb = S.off[lrow + pv.p] + nl, nhb = S.off[lrow + P + pv.p] + nh;
    if (pv.thread == 0) open_level(S, level, pv.p, nl, nh, nb, nhb);
    if ((nl | nh) == 0u) return;  // no lanes left in this partition's groups
    // capacity exceeded (workgroup-uniform test): the batch is redone
    if (nb > list_end(S, pv.p) || nhb > list_end(S, P + pv.p)) return;
  }
  const int lane = lane_id();
  const ull *cur = S.fr + (uint64_t)(level % 3) * GN;
  ull *nxt = S.fr + (uint64_t)((level + 1) % 3) * GN;
  if (level > 0) {
    ull *old = S.fr + (uint64_t)((level + 2) % 3) * GN;
    for (int l = pv.p; l < NL; l += P) {
      const uint64_t pb = S.off[lrow - NL + l], pc = S.cnt[lrow - NL + l];
      for (uint64_t i = pv.thread; i < pc; i += pv.nthreads) old[S.items[pb + i]] = 0ull;
    }
  }
  bool ovf = false;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  __shared__ uint32_t stage_all[NW * kStage], hstage_all[NW * kStageHeavy];
  Stage sg = {stage_all + wv * kStage, hstage_all + wv * kStageHeavy, 0, 0};
  const LevelLists<false> lists{S, level};
  const ListView lv = list_view(S);
  const uint64_t base = S.off[lrow + (lv.heavy ? P : 0) + pv.p];
  const uint64_t count = lv.heavy ? (uint64_t)nh * kParts : nl;
  const uint64_t nwv = lv.nwg * NW;
  const uint32_t B = lv.heavy ? 1u : (uint32_t)min((uint64_t)kWBlockItems, (count + nwv - 1) / nwv);
  for (uint64_t b0 = (lv.wg * NW + (uint64_t)wv) * B; b0 < count; b0 += nwv * B) {
    const int nb = (int)min((uint64_t)B, count - b0);
    uint32_t it = 0, gb = 0, e0 = 0, ed = 0;
    ull mk = 0ull, dnv = 0ull;
    if (lane < nb) {
      const uint64_t pos = base + (lv.heavy ? b0 / kParts : b0 + lane);
      const bool owner = !lv.heavy || b0 % kParts == 0;
      it = S.items[pos];
      const uint32_t v = it % n;
      gb = it - v;
      mk = cur[it];
      // lanes on which v is a target or lies below one: final now (every DAG
      // in-arc of a ready lane has pushed); the backward reads only these
      // (an atomic: waves pushing to v's other, not yet ready lanes may add
      // their bits in this round)
      dnv = S.wdn[it];
      const int64_t r0 = G.rp[v];
      e0 = (uint32_t)r0;
      ed = (uint32_t)(G.rp[v + 1] - r0);
      if (lv.heavy) {
        uint32_t f;
        part_of(ed, (uint32_t)(b0 % kParts), f, ed);
        e0 += f;
      }
      if (S.tgt_of[v] >= 0) {
        dnv |= mk;
        if (owner) {
          atomicOr(&S.wdn[it], mk);
          atomicMin(S.tmin, (uint32_t)level);
        }
      }
      if (owner) S.imask[pos] = mk;
    }
    // steps of 64 out-arcs, item after item
    auto advance = [&](int &j, uint32_t &c) {
      if (j >= nb) return;
      c += kLanes;
      if (c >= read_lane(ed, j)) {
        c = 0;
        ++j;
      }
    };
    auto load = [&](int j, uint32_t c, uint32_t &x, ull &d) {
      const int jj = j < nb ? j : 0;
      const bool has = j < nb && c + (uint32_t)lane < read_lane(ed, jj);
      const uint64_t e = has ? (uint64_t)read_lane(e0, jj) + c + (uint32_t)lane : 0u;
      const uint64_t row = (uint64_t)(read_lane(gb, jj) / n) * (uint64_t)G.m;
      x = (uint32_t)G.col[e];
      d = S.dagm[row + e];
      if (!has) d = 0ull;
    };
    int j0 = 0, j1;
    uint32_t c0 = 0, c1, x0, x1;
    ull d0, d1;
    load(j0, c0, x0, d0);
    ull srow = S.sig[(uint64_t)read_lane(it, 0) * kLanes + lane];
    while (j0 < nb) {
      const ull mask = read_lane64(mk, j0), dn = read_lane64(dnv, j0);
      const uint32_t gj = read_lane(gb, j0);
      j1 = j0;
      c1 = c0;
      advance(j1, c1);
      load(j1, c1, x1, d1);
      // lane b holds sigma_b(v) (a per-pair read of the row instead measured
      // 5 % slower on a full-width R-MAT 18 batch)
      const ull svl = srow;
      if (j1 != j0 && j1 < nb) srow = S.sig[(uint64_t)read_lane(it, j1) * kLanes + lane];
      ull d = d0 & mask;
      const uint64_t xrow = (uint64_t)(gj + x0) * kLanes;
      ull rdy = 0ull, mdn = d & dn;
      // the sources of each arc, lowest first, two per pass
      while (__ballot(d != 0ull) != 0ull) {
        const bool p0 = d != 0ull;
        const int q0 = p0 ? __builtin_ctzll(d) : 0;
        d &= d - 1ull;
        const bool p1 = p0 && d != 0ull;
        const int q1 = p1 ? __builtin_ctzll(d) : 0;
        if (p1) d &= d - 1ull;
        if (!p0) d = 0ull;
        const ull s0 = shfl64_w(svl, q0), s1 = shfl64_w(svl, q1);  // every lane takes part in the shuffles
        ull o0 = 0ull, o1 = 0ull;
        uint32_t k0 = 0u, k1 = 0u;
        if (p0) {
          o0 = atomicAdd(&S.sig[xrow + (uint32_t)q0], s0);
          k0 = atomicSub(&S.wc[xrow + (uint32_t)q0], 1u);
        }
        if (p1) {
          o1 = atomicAdd(&S.sig[xrow + (uint32_t)q1], s1);
          k1 = atomicSub(&S.wc[xrow + (uint32_t)q1], 1u);
        }
        // the push that completes the head's DAG in-arcs makes the lane ready
        if (k0 == 1u) rdy |= 1ull << q0;
        if (k1 == 1u) rdy |= 1ull << q1;
        const bool w0 = p0 && o0 + s0 < o0, w1 = p1 && o1 + s1 < o1;
        if (w0 || w1) {
          ovf = true;
          atomicOr(&S.ovl[gj / n], (w0 ? 1ull << q0 : 0ull) | (w1 ? 1ull << q1 : 0ull));
        }
      }
      if (mdn != 0ull) atomicOr(&S.wdn[gj + x0], mdn);
      bool first = false;
      if (rdy != 0ull) first = atomicOr(&nxt[gj + x0], rdy) == 0ull;
      // the first mark of the head appends it to the next round
      append_chunk(S, lists, pv.p, sg, gj, x0, first);
      j0 = j1;
      c0 = c1;
      x0 = x1;
      d0 = d1;
    }
  }
  flush_stage(S, lists, pv.p, sg);
  flush_counters<BLOCK>(S.ctr, S.ctr_slots, C_SCRATCH, 0, 0, 0, ovf, S.flags);
}

// Backward over topological round `level`: psi(v) = 1/sigma(v) + sum of
// psi(w) over DAG out-arcs (v, w) of the lane; lanes pruned as in the
// unweighted kernel (blocks of items, a lane each; items without lanes are
// passed over).  A wavefront lane takes one out-arc and its DAG mask word, psi
// is read only on the DAG (source, arc) pairs, and every source's sum runs in
// arc order, so the result does not depend on the item's lanes.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_w_bwd(DevGraph G, BatchState S, int level, int ntgt, int full) {
  constexpr int NW = BLOCK / 64;
  const uint32_t n = (uint32_t)S.n;
  const int P = S.P, NL = S.NL;
  const PartView pv = part_view<BLOCK>(P);
  const uint64_t lrow = (uint64_t)level * NL;
  const int lane = lane_id();
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  uint64_t c_v = 0, c_a = 0, c_d = 0;  // wave-uniform
  const ListView lv = list_view(S);
  const int l = (lv.heavy ? P : 0) + pv.p;
  const uint64_t base = S.off[lrow + l], count = S.cnt[lrow + l];
  const uint64_t nwv = lv.nwg * NW;
  const uint32_t B = lv.heavy ? 1u : (uint32_t)min((uint64_t)kWBlockItems, (count + nwv - 1) / nwv);
  for (uint64_t b0 = (lv.wg * NW + (uint64_t)wv) * B; b0 < count; b0 += nwv * B) {
    const int nb = (int)min((uint64_t)B, count - b0);
    uint32_t it = 0, gb = 0, e0 = 0, ed = 0;
    int32_t tg = -1;
    ull mk = 0ull;
    if (lane < nb) {
      it = S.items[base + b0 + lane];
      mk = S.imask[base + b0 + lane];
      const uint32_t v = it % n;
      gb = it - v;
      tg = S.tgt_of[v];
      // a target's dependency reads psi only on lanes where v is a target or
      // lies below one
      if (!full && tg < 0) mk &= S.wdn[it];
      const int64_t r0 = G.rp[v];
      e0 = (uint32_t)r0;
      ed = (uint32_t)(G.rp[v + 1] - r0);
    }
    ull todo = __ballot(mk != 0ull);
    c_v += wave_sum((uint64_t)__popcll(mk));
    c_a += wave_sum((uint64_t)__popcll(mk) * ed);
    for (; todo != 0ull; todo &= todo - 1ull) {
      const int j = __builtin_ctzll(todo);
      const ull em = read_lane64(mk, j);
      const uint32_t ij = read_lane(it, j), gj = read_lane(gb, j), dj = read_lane(ed, j);
      const uint64_t row = (uint64_t)ij * kLanes + (uint32_t)lane;
      const ull sv = ((em >> lane) & 1ull) ? S.sig[row] : 1ull;
      const uint32_t a0 = read_lane(e0, j);
      const int32_t *dst = G.col + a0;
      const ull *dm = S.dagm + (uint64_t)(gj / n) * (uint64_t)G.m + a0;
      double acc = 0.0;  // lane b: the sum of source b, over its DAG arcs in arc order
      for (uint32_t k = 0; k < dj; k += kLanes) {
        // lane q takes arc k + q and its DAG lanes among the needed ones
        const bool has = k + (uint32_t)lane < dj;
        const uint32_t x = (uint32_t)dst[has ? k + (uint32_t)lane : 0u];
        const ull d = has ? dm[k + (uint32_t)lane] & em : 0ull;
        const uint64_t xrow = (uint64_t)(gj + x) * kLanes;
        // eight sources at a time: the lanes of each source's DAG arcs load its
        // psi (all eight loads in flight together), then the source's sum takes
        // them in arc order, so every sum runs in the same order whatever the
        // lanes and batch
        ull rem = em;
        while (rem != 0ull) {
          int bq[8];
          ull aq[8];
          double y[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const bool live = rem != 0ull;
            bq[q] = live ? __builtin_ctzll(rem) : 0;
            aq[q] = __ballot(live && ((d >> bq[q]) & 1ull));
            if (live) rem &= rem - 1ull;
            y[q] = ((aq[q] >> lane) & 1ull) ? S.psi[xrow + (uint32_t)bq[q]] : 0.0;
          }
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            ull t = aq[q];
            if (t == 0ull) continue;
            c_d += (uint64_t)__popcll(t);
            double a = __longlong_as_double((long long)read_lane64((ull)__double_as_longlong(acc), bq[q]));
            while (t != 0ull) {
              const int z = __builtin_ctzll(t);
              t &= t - 1ull;
              a += __longlong_as_double((long long)read_lane64((ull)__double_as_longlong(y[q]), z));
            }
            if (lane == bq[q]) acc = a;
          }
        }
      }
      if ((em >> lane) & 1ull) {
        const double s = (double)sv;
        const double dl = s * acc;
        const int32_t t = (int32_t)read_lane((uint32_t)tg, j);
        S.psi[row] = acc + 1.0 / s;
        if (S.dout) S.dout[row] = dl;
        if (t >= 0 && t < ntgt) S.res[((uint64_t)t * S.G + gj / n) * kLanes + (uint32_t)lane] = (level > 0) ? dl : 0.0;
      }
    }
  }
  const int ck[3] = {C_BWD_VPAIRS, C_BWD_APAIRS, C_BWD_DPAIRS};
  const uint64_t cv[3] = {c_v, c_a, c_d};
  flush_wave_counters<BLOCK, 3>(S.ctr, S.ctr_slots, ck, cv, false, S.flags);
}

__global__ void k_w_cleanup(BatchState S) {
  const uint64_t GN = (uint64_t)S.G * (uint64_t)S.n;
  const int lane = lane_id();
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
  for (int l = 0; l < S.NL; ++l) {
    const uint32_t *rl = S.rl + queue_begin(S, l);
    for (uint64_t i = wave; i < *rtail_at(S, l); i += nwaves) {
      const uint32_t it = rl[i];
      const uint64_t row = (uint64_t)it * kLanes + lane;
      S.wd[row] = kInf;
      S.wc[row] = 0u;
      S.sig[row] = 0ull;
      if (lane == 0) S.vis[it] = 0ull;
      if (lane == 1) S.wdn[it] = 0ull;
      if (lane >= 2 && lane < 5) S.fr[(uint64_t)(lane - 2) * GN + it] = 0ull;
      if (lane >= 5 && lane < 8) S.chg[(uint64_t)(lane - 5) * GN + it] = 0ull;
    }
  }
}

__global__ void k_w_export(DevGraph G, BatchState S, const int32_t *lane_slot, uint64_t *dist, ull *sigma,
                           double *delta, int64_t k) {
  const uint64_t n = (uint64_t)S.n;
  const int lane = lane_id();
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
  for (int l = 0; l < S.NL; ++l) {
    const uint32_t *rl = S.rl + queue_begin(S, l);
    for (uint64_t i = wave; i < *rtail_at(S, l); i += nwaves) {
      const uint32_t it = rl[i];
      const uint32_t g = (uint32_t)(it / n);
      const uint32_t v = (uint32_t)(it - (uint64_t)g * n);
      const uint64_t row = (uint64_t)it * kLanes + lane;
      const uint32_t d = S.wd[row];
      if (d == kInf) continue;
      const int32_t slot = lane_slot[g * kLanes + lane];
      if (slot < 0 || slot >= k) continue;
      const uint64_t o = (uint64_t)slot * n + (uint32_t)G.orig[v];
      dist[o] = d;
      sigma[o] = S.sig[row];
      if (delta && S.dout) delta[o] = S.dout[row];
    }
  }
}

#define DISPATCH_BLOCK(L, KERNEL, ...)                                                                  \
  do {                                                                                                  \
    switch ((L).block) {                                                                                \
      case 64: hipLaunchKernelGGL(KERNEL<64>, dim3((L).grid), dim3(64), 0, st, __VA_ARGS__); break;    \
      case 128: hipLaunchKernelGGL(KERNEL<128>, dim3((L).grid), dim3(128), 0, st, __VA_ARGS__); break; \
      case 512: hipLaunchKernelGGL(KERNEL<512>, dim3((L).grid), dim3(512), 0, st, __VA_ARGS__); break; \
      default: hipLaunchKernelGGL(KERNEL<256>, dim3((L).grid), dim3(256), 0, st, __VA_ARGS__); break;  \
    }                                                                                                   \
  } while (0)

hipError_t launch_w_init(const BatchState &S, const uint32_t *items0, const ull *masks0, const uint32_t *dest0, int k,
                         hipStream_t st) {
  const int grid = std::max(1, (k + 255) / 256);
  hipLaunchKernelGGL(k_w_init, dim3(grid), dim3(256), 0, st, S, items0, masks0, dest0, k);
  return hipGetLastError();
}

hipError_t launch_w_relax(const DevGraph &G, const BatchState &S, int round, Launch L, hipStream_t st) {
  DISPATCH_BLOCK(L, k_w_relax, G, S, round);
  return hipGetLastError();
}

hipError_t launch_w_count(const DevGraph &G, const BatchState &S, Launch L, hipStream_t st) {
  DISPATCH_BLOCK(L, k_w_count, G, S);
  return hipGetLastError();
}

hipError_t launch_w_sigma(const DevGraph &G, const BatchState &S, int round, Launch L, hipStream_t st) {
  DISPATCH_BLOCK(L, k_w_sigma, G, S, round);
  return hipGetLastError();
}

hipError_t launch_w_bwd(const DevGraph &G, const BatchState &S, int round, int ntgt, int full, Launch L,
                        hipStream_t st) {
  DISPATCH_BLOCK(L, k_w_bwd, G, S, round, ntgt, full);
  return hipGetLastError();
}

hipError_t launch_w_cleanup(const BatchState &S, Launch L, hipStream_t st) {
  hipLaunchKernelGGL(k_w_cleanup, dim3(L.grid), dim3(256), 0, st, S);
  return hipGetLastError();
}

hipError_t launch_w_export(const DevGraph &G, const BatchState &S, const int32_t *lane_slot, uint64_t *dist, ull *sigma,
                           double *delta, int64_t k, Launch L, hipStream_t st) {
  hipLaunchKernelGGL(k_w_export, dim3(L.grid), dim3(256), 0, st, G, S, lane_slot, dist, sigma, delta, k);
  return hipGetLastError();
}

}  // namespace bcd

// ================================================================= host

namespace bcd {


template <class T>
static bcd_status walloc(T **p, size_t count) {
  *p = nullptr;
  if (hipMalloc((void **)p, std::max<size_t>(count, 1) * sizeof(T)) != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    return fail(BCD_ERR_OUT_OF_MEMORY, "device allocation for the weighted engine failed");
  }
  return BCD_OK;
}

bcd_status Workspace::ensure_weighted() {
  if (weighted_ready && weighted_G == G) return BCD_OK;
  release_weighted();
  const size_t GN = (size_t)G * (size_t)n;
  const BatchSizes B(n, G, S.H);
  S.capQ = B.capQ;
  S.capQH = B.capQH;
  S.qhbase = B.qhbase;
  S.qsize = B.qsize;
  STCHK(walloc(&S.wd, GN * kLanes));
  STCHK(walloc(&S.wc, GN * kLanes));
  STCHK(walloc(&S.chg, 3 * GN));
  STCHK(walloc(&S.bq, 3 * S.qsize));
  STCHK(walloc(&S.rl, S.qsize));
  STCHK(walloc(&S.qtail, (size_t)4 * kMaxLists * kTailStride));
  STCHK(walloc(&S.rtail, (size_t)kMaxLists * kTailStride));
  STCHK(walloc(&S.wdn, GN));
  STCHK(walloc(&S.dagm, (size_t)G * (size_t)graph->m));
  HIPCHK(hipMemsetAsync(S.wd, 0xFF, GN * kLanes * sizeof(uint32_t), stream));
  HIPCHK(hipMemsetAsync(S.wdn, 0, GN * sizeof(unsigned long long), stream));
  HIPCHK(hipMemsetAsync(S.wc, 0, GN * kLanes * sizeof(uint32_t), stream));
  HIPCHK(hipMemsetAsync(S.chg, 0, 3 * GN * sizeof(unsigned long long), stream));
  HIPCHK(hipMemsetAsync(S.rtail, 0, (size_t)kMaxLists * kTailStride * sizeof(uint32_t), stream));
  HIPCHK(hipStreamSynchronize(stream));
  weighted_ready = true;
  weighted_G = G;
  return BCD_OK;
}

void Workspace::release_weighted() {
  auto f = [](auto *&p) {
    if (p) (void)hipFree((void *)p);
    p = nullptr;
  };
  f(S.wd);
  f(S.wc);
  f(S.chg);
  f(S.bq);
  f(S.rl);
  f(S.qtail);
  f(S.rtail);
  f(S.wdn);
  f(S.dagm);
  weighted_ready = false;
}

struct WExport {
  uint64_t *dist = nullptr;
  unsigned long long *sigma = nullptr;
  double *delta = nullptr;
  int64_t k = 0;
};

// One batch of the weighted engine; `k` sources staged in h_items0/h_masks0.
static bcd_status run_one_wbatch(Graph *g, Workspace *ws, int k, int ntgt, bool full, WExport *ex, ProfAcc *prof,
                                 bool *sigma_overflow,
                                 bool copy_res = true, unsigned long long *ovl_out = nullptr) {
  hipStream_t st = ws->stream;
  const DevGraph D = g->dev_internal();
  const bool profiling = g->profiling.load();
  const size_t G64 = (size_t)ws->G * kLanes;
  HIPCHK(hipMemcpyAsync(ws->d_items0, ws->h_items0, (size_t)k * sizeof(uint32_t), hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(ws->d_masks0, ws->h_masks0, (size_t)k * sizeof(unsigned long long), hipMemcpyHostToDevice,
                        st));
  HIPCHK(hipMemcpyAsync(ws->d_dest0, ws->h_dest0, (size_t)k * sizeof(uint32_t), hipMemcpyHostToDevice, st));
  for (int attempt = 0;; ++attempt) {
    BatchState S = ws->S;
    if (!ex) S.dout = nullptr;
    S.P = ws->batch_parts(k);  // partitions that hold this batch's groups
    S.NL = ws->lists(S.P);
    const int NL = S.NL;
    const Launch L = g->launch_parts(S.P, (k + kLanes - 1) / kLanes);
    uint32_t *hc = ws->h_cnt;
    uint32_t *hc0 = hc + kCntStage;
    uint32_t *hm = reinterpret_cast<uint32_t *>(ws->h_misc);
    for (int l = 0; l < NL; ++l) hc0[l] = ws->h_cnt0[l];
    HIPCHK(hipMemcpyAsync(&S.cnt[0], hc0, (size_t)NL * sizeof(uint32_t), hipMemcpyHostToDevice, st));
    if (ntgt > 0) HIPCHK(hipMemsetAsync(S.res, 0, (size_t)ntgt * G64 * sizeof(double), st));
    HIPCHK(hipMemsetAsync(S.tmin, 0xFF, sizeof(uint32_t), st));
    HIPCHK(hipMemsetAsync(S.flags, 0, 4 * sizeof(uint32_t), st));
    HIPCHK(hipMemsetAsync(S.ovl, 0, 2 * (size_t)ws->G * sizeof(unsigned long long), st));
    HIPCHK(launch_w_init(S, ws->d_items0, ws->d_masks0, ws->d_dest0, k, st));
    size_t ev = 0;
    auto rec0 = [&]() -> hipError_t {
      return profiling ? hipEventRecord(ws->event_pair(ev).first, st) : hipSuccess;
    };
    auto rec1 = [&]() -> hipError_t {
      if (!profiling) return hipSuccess;
      hipError_t e = hipEventRecord(ws->event_pair(ev).second, st);
      ++ev;
      return e;
    };
    // 1. distances
    int round = 0;
    for (;;) {
      const int chunk = 8;
      for (int i = 0; i < chunk; ++i, ++round) {
        HIPCHK(rec0());
        HIPCHK(launch_w_relax(D, S, round, L, st));
        HIPCHK(rec1());
      }
      HIPCHK(hipMemcpyAsync(hc, qtail_at(S, round, 0), (size_t)kMaxLists * kTailStride * sizeof(uint32_t),
                            hipMemcpyDeviceToHost, st));
      HIPCHK(hipStreamSynchronize(st));
      uint64_t left = 0;
      for (int l = 0; l < NL; ++l) left += hc[l * kTailStride];
      if (left == 0) break;
      if (round > g->n + 16) return fail(BCD_ERR_DEVICE, "relaxation rounds did not converge");
    }
    // 2. DAG in-degrees
    HIPCHK(rec0());
    HIPCHK(launch_w_count(D, S, L, st));
    HIPCHK(rec1());
    // 3. path counts in topological rounds
    std::vector<uint32_t> cntp(hc0, hc0 + NL);
    int lmax = -1, level = 0;
    int chunk = std::min(kLevelChunkMax, std::max(4, ws->last_depth + 2));
    uint32_t flags_h[2] = {0, 0}, tmin_h = 0xFFFFFFFFu;
    while (lmax < 0) {
      const int first = level;
      int launched = 0;
      for (; launched < chunk && level <= g->n; ++launched, ++level) {
        HIPCHK(rec0());
        HIPCHK(launch_w_sigma(D, S, level, L, st));
        HIPCHK(rec1());
      }
      HIPCHK(launch_publish_counts(S, level, st));
      HIPCHK(hipMemcpyAsync(hc, &S.cnt[(size_t)(first + 1) * NL], (size_t)launched * NL * sizeof(uint32_t),
                            hipMemcpyDeviceToHost, st));
      HIPCHK(hipMemcpyAsync(hm, S.flags, 2 * sizeof(uint32_t), hipMemcpyDeviceToHost, st));
      HIPCHK(hipMemcpyAsync(hm + 2, S.tmin, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
      HIPCHK(hipStreamSynchronize(st));
      flags_h[0] = hm[0];
      flags_h[1] = hm[1];
      tmin_h = hm[2];
      if (flags_h[1]) break;
      for (int i = 0; i < launched; ++i) {
        uint64_t tot = 0;
        for (int l = 0; l < NL; ++l) tot += hc[(size_t)i * NL + l];
        if (tot == 0) {
          lmax = first + i;
          break;
        }
        cntp.insert(cntp.end(), hc + (size_t)i * NL, hc + (size_t)(i + 1) * NL);
      }
      if (lmax < 0 && level > g->n) return fail(BCD_ERR_DEVICE, "topological rounds did not terminate");
      chunk = kLevelChunkMax;
    }
    if (flags_h[1]) {
      HIPCHK(launch_w_cleanup(S, L, st));
      STCHK(ws->reset_batch_dense());
      STCHK(ws->grow_items());
      if (attempt > 8) return fail(BCD_ERR_OUT_OF_MEMORY, "frontier item list cannot grow further");
      continue;
    }
    ws->last_depth = lmax;
    if (flags_h[0]) *sigma_overflow = true;
    const size_t fwd_events = ev;
    // 4. backward
    int stop = -1;
    if (full) stop = 0;
    else if (ntgt > 0 && tmin_h != 0xFFFFFFFFu) stop = (int)tmin_h;
    if (stop >= 0)
      for (int lv = lmax; lv >= stop; --lv) {
        HIPCHK(rec0());
        HIPCHK(launch_w_bwd(D, S, lv, ntgt, full ? 1 : 0, L, st));
        HIPCHK(rec1());
      }
    if (ex) HIPCHK(launch_w_export(D, S, ws->d_lane_slot, ex->dist, ex->sigma, ex->delta, ex->k, L, st));
    if (ntgt > 0 && copy_res)
      HIPCHK(hipMemcpyAsync(ws->h_res, S.res, (size_t)ntgt * G64 * sizeof(double), hipMemcpyDeviceToHost, st));
    if (ovl_out)
      HIPCHK(hipMemcpyAsync(ovl_out, S.ovl, (size_t)ws->G * sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    HIPCHK(launch_w_cleanup(S, L, st));
    HIPCHK(launch_ctr_fold(S.ctr, kCtrSlots, S.acc, st));
    HIPCHK(hipStreamSynchronize(st));
    if (profiling && prof) {
      for (size_t i = 0; i < ev; ++i) prof->add(g, i < fwd_events ? 0 : 1, ws->events[i].first, ws->events[i].second);
      // work items: one per (group, vertex, topological round) with ready lanes
      for (size_t lv = 0; lv * NL < cntp.size(); ++lv)
        for (int l = 0; l < NL; ++l) {
          prof->items[0] += cntp[lv * NL + l];
          if (stop >= 0 && (int)lv >= stop) prof->items[1] += cntp[lv * NL + l];
        }
    }
    return BCD_OK;
  }
}

static bcd_status wcounters(Workspace *ws, uint64_t *c) { return collect_counters(ws, c, ws->S.acc); }

// Algorithmic bytes per (source, element) pair: 32 per vertex, 12 per arc
// (head index, arc length, head distance), 8 per DAG arc, in each pass.
void record_wprofile(Graph *g, const ProfAcc &p, const uint64_t *c) {
  const double fb = 32.0 * c[C_FWD_VPAIRS] + 12.0 * c[C_FWD_APAIRS] + 8.0 * c[C_FWD_DPAIRS];
  const double bb = 32.0 * c[C_BWD_VPAIRS] + 12.0 * c[C_BWD_APAIRS] + 8.0 * c[C_BWD_DPAIRS];
  g->add_profile(0, p.launches[0], p.ms[0], c + C_FWD_VPAIRS, fb, p.items[0], &p.iv[0], 0, 0.0);
  g->add_profile(1, p.launches[1], p.ms[1], c + C_BWD_VPAIRS, bb, p.items[1], &p.iv[1], 0, 0.0);
}

bcd_status run_staged_wbatch(Graph *g, Workspace *ws, int k, int ntgt, unsigned long long *ovl_out, bool *ovf,
                             ProfAcc *prof) {
  if ((uint64_t)g->n * (uint64_t)g->max_w >= 0xFFFFFFFFull)
    return fail(BCD_ERR_UNSUPPORTED, "n * max weight must stay below 2^32 - 1 for 32-bit distances");
  STCHK(ws->ensure_weighted());
  return run_one_wbatch(g, ws, k, ntgt, false, nullptr, prof, ovf, false, ovl_out);
}

bcd_status run_weighted(Graph *g, Workspace *ws, const std::vector<int32_t> &src, const std::vector<int32_t> &tgt,
                        bool want_counters, SourceRun &out) {
  const bcd_config cfg = g->config();
  if ((uint64_t)g->n * (uint64_t)g->max_w >= 0xFFFFFFFFull)
    return fail(BCD_ERR_UNSUPPORTED, "n * max weight must stay below 2^32 - 1 for 32-bit distances");
  STCHK(ws->ensure_batch(cfg.groups));
  STCHK(ws->ensure_weighted());
  const int ntgt = (int)tgt.size();
  const size_t G64 = (size_t)ws->G * kLanes;
  STCHK(ws->ensure_res((size_t)std::max(ntgt, 1) * G64));
  const size_t ns = src.size();
  out.dep.assign(ns * (size_t)ntgt, 0.0);
  if (want_counters) out.counters.assign(ns * 3, 0);
  // the plain engine on a weighted graph runs one source per batch
  const bool one = want_counters || cfg.engine == BCD_ENGINE_PLAIN;
  const size_t two = one ? 1 : pipelined_batch(g, ns, G64);
  out.width = 1;
  std::vector<uint32_t> ord;
  STCHK(source_order(g, ws, src, ord));
  ProfAcc prof;
  bool ovf = false;
  uint64_t tot[C_COUNT] = {0};
  // batches b = first, first + stride, ... on workspace w; each source's
  // dependencies go to its own position
  auto stripe = [&](Workspace *w, size_t first, size_t stride, ProfAcc &p, bool &o) -> bcd_status {
    TargetMap tm;
    STCHK(tm.install(w, tgt));
    const size_t w64 = (size_t)w->G * kLanes;
    const size_t per = one ? 1 : (stride == 1 ? w64 : two);  // alone: whole batches
    std::vector<int32_t> bsrc(per);
    for (size_t b0 = first * per; b0 < ns; b0 += stride * per) {
      const int k = (int)std::min(per, ns - b0);
      for (int i = 0; i < k; ++i) bsrc[(size_t)i] = src[ord[b0 + i]];
      w->stage_sources(bsrc.data(), k);
      STCHK(run_one_wbatch(g, w, k, ntgt, false, nullptr, &p, &o));
      for (int i = 0; i < k; ++i)
        for (int t = 0; t < ntgt; ++t) out.dep[(size_t)ord[b0 + i] * ntgt + t] = w->h_res[(size_t)t * w64 + i];
      if (want_counters) {
        uint64_t c[C_COUNT];
        STCHK(wcounters(w, c));
        out.counters[(size_t)ord[b0] * 3 + 0] = c[C_FWD_VPAIRS];
        out.counters[(size_t)ord[b0] * 3 + 1] = c[C_FWD_APAIRS];
        out.counters[(size_t)ord[b0] * 3 + 2] = c[C_FWD_DPAIRS];
        for (int j = 0; j < C_COUNT; ++j) tot[j] += c[j];
      }
    }
    return BCD_OK;
  };
  if (one) {
    STCHK(stripe(ws, 0, 1, prof, ovf));
  } else {
    auto prepare = [&](Workspace *w, int groups) -> bcd_status {
      STCHK(w->ensure_batch(groups));
      STCHK(w->ensure_weighted());
      return w->ensure_res((size_t)std::max(ntgt, 1) * (size_t)groups * kLanes);
    };
    STCHK(run_pipelined(g, ws, two, second_groups(g, ns, out.sample_of, G64), prepare, stripe, prof, ovf, tot, &out.width));
    uint64_t t1[C_COUNT];
    STCHK(wcounters(ws, t1));
    for (int j = 0; j < C_COUNT; ++j) tot[j] += t1[j];
  }
  out.te = tot[C_FWD_APAIRS];
  out.reached = tot[C_FWD_VPAIRS];
  out.dag = tot[C_FWD_DPAIRS];
  if (g->profiling.load()) record_wprofile(g, prof, tot);
  if (ovf) return fail(BCD_ERR_SIGMA_OVERFLOW, "a shortest-path count exceeded 2^64 - 1");
  return BCD_OK;
}

bcd_status multi_source_pass_weighted(Graph *g, const int32_t *sources, int64_t k, uint64_t *dist, uint64_t *sigma,
                                      double *delta) {
  const bcd_config cfg = g->config();
  if (k > (int64_t)cfg.groups * kLanes) return fail(BCD_ERR_INVALID_ARG, "k exceeds the batch width");
  if ((uint64_t)g->n * (uint64_t)g->max_w >= 0xFFFFFFFFull)
    return fail(BCD_ERR_UNSUPPORTED, "n * max weight must stay below 2^32 - 1 for 32-bit distances");
  for (int64_t i = 0; i < k; ++i) {
    if (sources[i] < 0 || sources[i] >= g->n) return fail(BCD_ERR_INVALID_ARG, "source out of range");
    for (int64_t j = 0; j < i; ++j)
      if (sources[j] == sources[i] && i / kLanes == j / kLanes) return fail(BCD_ERR_INVALID_ARG, "repeated source");
  }
  Lease ls(g);
  if (!ls.ok()) return fail(BCD_ERR_OUT_OF_MEMORY, "workspace allocation failed");
  STCHK(ls->init_common(g));
  Workspace *ws = ls.w.get();
  STCHK(ws->ensure_batch(cfg.groups));
  STCHK(ws->ensure_weighted());
  STCHK(ws->ensure_dout());
  const size_t G64 = (size_t)ws->G * kLanes;
  const size_t kn = (size_t)k * (size_t)g->n;
  WExport ex;
  ex.k = k;
  STCHK(walloc(&ex.dist, kn));
  bcd_status rc = walloc(&ex.sigma, kn);
  if (rc == BCD_OK) rc = walloc(&ex.delta, kn);
  hipStream_t st = ws->stream;
  std::vector<int32_t> slot(G64, -1);
  for (int64_t i = 0; i < k; ++i) slot[(size_t)i] = (int32_t)i;
  hipError_t e = hipSuccess;
  if (rc == BCD_OK) {
    e = hipMemcpyAsync(ws->d_lane_slot, slot.data(), G64 * sizeof(int32_t), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipMemsetAsync(ex.dist, 0xFF, kn * 8, st);
    if (e == hipSuccess) e = hipMemsetAsync(ex.sigma, 0, kn * 8, st);
    if (e == hipSuccess) e = hipMemsetAsync(ex.delta, 0, kn * 8, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) rc = hip_fail(e, "export setup");
  }
  bool ovf = false;
  if (rc == BCD_OK) {
    ws->stage_sources(sources, (int)k);
    rc = run_one_wbatch(g, ws, (int)k, 0, true, &ex, nullptr, &ovf);
  }
  if (rc == BCD_OK) {
    e = hipSuccess;
    if (dist) e = hipMemcpy(dist, ex.dist, kn * 8, hipMemcpyDeviceToHost);
    if (e == hipSuccess && sigma) e = hipMemcpy(sigma, ex.sigma, kn * 8, hipMemcpyDeviceToHost);
    if (e == hipSuccess && delta) e = hipMemcpy(delta, ex.delta, kn * 8, hipMemcpyDeviceToHost);
    if (e != hipSuccess) rc = hip_fail(e, "export copy");
  }
  if (ex.dist) (void)hipFree(ex.dist);
  if (ex.sigma) (void)hipFree(ex.sigma);
  if (ex.delta) (void)hipFree(ex.delta);
  uint64_t cc[C_COUNT];
  if (rc == BCD_OK) rc = wcounters(ws, cc);
  if (rc == BCD_OK && ovf) rc = fail(BCD_ERR_SIGMA_OVERFLOW, "a shortest-path count exceeded 2^64 - 1");
  return rc;
}

}  // namespace bcd

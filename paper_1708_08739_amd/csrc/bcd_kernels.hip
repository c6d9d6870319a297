// HIP kernels for gfx950 (CDNA4, wave64): the per-source shortest-path pass
// of the paper's Alg.1 / Alg.2 (forward path counting, then the Eq.(4)
// dependency accumulation), the RV(r) reachability traversal of Def.3, and
// a copy probe.
//
// Batched engine layout: a column group is 64 sources, one per wavefront
// lane.  A frontier item is (group g, vertex v) with a 64-bit mask of the
// lanes for which v sits on the current BFS level; lane b works for source b,
// so the 64 path counts of v are one coalesced row of 256 bytes (512 where a
// count does not fit 32 bits), and testing "has
// source b already settled w" for all 64 sources reads one 64-bit word per
// arc.
#include <algorithm>

#include "bcd_device.h"

namespace bcd {

// ------------------------------------------------------------ batched

// The path counts as rows of 64 T, T = uint32_t when S.narrow.  Sums are
// 64-bit either way; a sum that does not fit the stored type raises flags[2]
// and the batch is redone with 64-bit rows, so a narrow count is exact too.  The
// rows are what the large forward levels fetch, and half of a row is half of
// its cache lines (R-MAT 16 exact 40.7 -> 36.0 ms, R-MAT 20 with 1,000 sources
// 44.2 -> 39.6).
template <class T>
static __device__ __forceinline__ T *counts(const BatchState &S) {
  return reinterpret_cast<T *>(S.sig);
}

// Stores this lane's count, wide = a count that T cannot hold was met.
template <class T>
static __device__ __forceinline__ void store_count(T *row, ull c, bool &wide) {
  if (sizeof(T) == 4) wide |= (c >> 32) != 0ull;
  *row = (T)c;
}

// Level 0: each item is (g, source vertex) with the lanes it is the source
// of; sigma = 1 on those lanes.
__global__ void k_batch_init(BatchState S, const uint32_t *items0, const ull *masks0, const uint32_t *dest0, int k) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < k; i += gridDim.x * blockDim.x) {
    const uint32_t it = items0[i];
    const ull m = masks0[i];
    const uint64_t GN = (uint64_t)S.G * (uint64_t)S.n;
    S.msk[M_FR * GN + it] = m;  // level-0 masks
    S.msk[M_SEEN * GN + it] = m;
    const uint32_t g = it / (uint32_t)S.n;
    if (S.tgt_of[it - g * (uint32_t)S.n] >= 0) atomicOr(&S.ovl[S.G + g], m);
    S.items[level0_slot(S, it, dest0[i])] = it;
    for (int b = 0; b < kLanes; ++b)
      if ((m >> b) & 1ull) {
        if (S.narrow) counts<uint32_t>(S)[(size_t)it * kLanes + b] = 1u;
        else S.sig[(size_t)it * kLanes + b] = 1ull;
      }
  }
  // level-0 base of every item list of this batch
  if (blockIdx.x == 0 && threadIdx.x < (unsigned)S.NL) {
    const int l = (int)threadIdx.x;
    S.off[l] = list_begin(S, l);
    *tail_at(S, 0, l) = S.cnt[l];
    *tail_at(S, 1, l) = 0u;
    *tail_at(S, 2, l) = 0u;
  }
}

// Predecessor rows of a chunk of arc lanes, up to eight at a time: arc lane j
// holds the tail u and the lanes pm for which that arc is a DAG arc (bits:
// the arc lanes not taken yet), gb is the first item of the wavefront's
// group.  issue() starts the loads of the next eight rows; add() adds them
// into acc (this lane's source).  The sums are exact: eight counts below 2^60
// on top of a sum below 2^60 cannot pass 2^64, and where one is larger every
// add is checked for a carry (the true sum then exceeds 2^64 - 1), its lanes
// going to ov.  got collects the lanes that received a count.  bits, pm, u
// and gb are wave-uniform or read by lane number, so all address work is
// scalar.
template <class T>
struct Rows {
  T x[8];
  __device__ __forceinline__ void issue(const T *sig, uint32_t gb, uint32_t u, ull pm, ull &bits, ull &got,
                                        uint64_t &dag_pairs) {
    const int lane = lane_id();
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (bits != 0ull) {
        const int j = __builtin_ctzll(bits);
        bits &= bits - 1ull;
        const ull dq = read_lane64(pm, j);
        const T *row = sig + (uint64_t)(gb + read_lane(u, j)) * kLanes;
        dag_pairs += (uint64_t)__popcll(dq);
        got |= dq;
        if (__builtin_amdgcn_inverse_ballot_w64(dq)) x[q] = row[lane];
      }
    }
  }
  __device__ __forceinline__ void add(ull &acc, ull &ov) {
    if (sizeof(T) == 4) {  // fewer than 2^32 arcs: no carry
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        // keeps the widening out of issue()'s branches, where every load
        // would be waited for on its own
        asm volatile("" : "+v"(x[q]));
        acc += x[q];
      }
      return;
    }
    uint32_t hi = (uint32_t)(acc >> 32);
#pragma unroll
    for (int q = 0; q < 8; ++q) hi |= (uint32_t)((ull)x[q] >> 32);
    if (__ballot(hi >> 28 != 0u) == 0ull) {
#pragma unroll
      for (int q = 0; q < 8; ++q) acc += x[q];
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const ull sum = acc + x[q];
        ov |= __ballot(sum < acc);
        acc = sum;
      }
    }
  }
};

template <class T>
static __device__ __forceinline__ void pull_rows(const T *sig, uint32_t gb, uint32_t u, ull pm, ull &acc, ull &ov,
                                                 ull &got, uint64_t &dag_pairs) {
  ull bits = __ballot(pm != 0ull);
  while (bits != 0ull) {
    Rows<T> r;
    r.issue(sig, gb, u, pm, bits, got, dag_pairs);
    r.add(acc, ov);
  }
}

// OR of x over the wavefront (wave-uniform result).
static __device__ __forceinline__ ull wave_or(ull x) {
  ull out = 0ull, b = __ballot(x != 0ull);
  while (b != 0ull) {
    const int j = __builtin_ctzll(b);
    const ull v = read_lane64(x, j);
    out |= v;
    b &= b - 1ull;
    // arcs that add nothing new are skipped
    b &= __ballot((x & ~out) != 0ull);
  }
  return out;
}

__global__ void k_publish_counts(BatchState S, int level) {
  const int l = (int)threadIdx.x;
  if (l < S.NL) S.cnt[(uint64_t)level * S.NL + l] = *tail_at(S, level, l);
}

// One BFS level of the batched forward pass (unweighted graphs).  For every
// item (g, v, mask) on `level`:
//   1. sigma pull: sigma_b(v) = sum of sigma_b(u) over in-arcs (u, v) with u
//      on level-1 for lane b (the shortest-path-DAG predecessors of v), an
//      exact uint64 sum; no atomics;
//   2. discovery: for every out-arc (v, w), lanes b in mask not yet seen at w
//      are DAG arcs; they are marked seen and flagged for level+1, lanes over
//      arcs, and the first flagger appends (g, w) to the next level's list.
// Level masks rotate over four words of (g, v): cur (level), nxt (level+1,
// being built), prv (level-1, read by the pull) and old (level-2, retired
// here).  With bottom-up levels enabled, step 1 is skipped when the level was
// found by k_bu_level (which pulled the counts), and step 2 when level+1 will
// be; the item masks are recorded for the backward either way.
//
// Light items: a wavefront takes a block of up to kBlockItems, loads their masks
// and row bounds with a lane per item, then takes them one after the other in
// steps of 32 in-arcs (lower half of the wavefront) and 32 out-arcs (upper
// half), one gather bringing the words of all of them.  The arc ends of the
// step after next and the words of the next one are loaded while the current
// step's rows are added, so a step costs the latency of its rows and flags,
// not of the whole chain item -> bounds -> arc ends -> words -> rows.
// Heavy vertices (more than kHeavyArcs arcs, internal id < H) are on a list
// of their own, whose items a workgroup takes one at a time: its wavefronts
// share the item's steps and add their partial path counts in LDS.  A
// wavefront alone walks a hub's thousands of arcs as one serial chain of
// dependent loads, and every level waits for its largest hub.
// Every random 8-byte read asks memory for 128 bytes.  Wide batches are bound by
// that traffic (over the time any forward launch runs: R-MAT 16 exact 5.1 TB/s,
// R-MAT 20 in batches of 4,096 sources 6.6, the streaming read probe 5.7), narrow
// ones by the latency of their accesses (R-MAT 16, 1,000 sources: 56 % of the
// cycles of resident waves wait for memory, 2 TB/s).  A level with two items a step, 64-byte mask records and no
// heavy list took, summed over the levels of R-MAT 16 / 20 with 1,000 sources,
// 3.0 / 36 ms; as here 1.9 / 24.
// Narrow rows at 8 waves per SIMD (64 VGPRs, 60 bytes of scratch a lane): left
// alone the compiler takes 88 registers for 5 (R-MAT 16 exact, 5 / 6 / 7 / 8 waves:
// 38.7 / 36.6 / 35.9 / 35.4 ms; four or six rows at a time instead of eight 35.5 /
// 35.9).  64-bit rows at 6 (80 VGPRs, no scratch): on a graph with counts above
// 2^32, R-MAT 16 exact at 4 / 5 / 6 / 7 / 8 waves 49.7 / 49.8 / 48.6 / 48.5 / 51.2 ms,
// layers of 30,000 vertices with 1,000 sources 23.8 / 24.0 / 23.6 / 24.3 / 25.2.
template <int BLOCK, class T>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 8 : 6, 8))) void k_fwd_level(DevGraph G, BatchState S, int level) {
  constexpr int NW = BLOCK / 64;
  const uint32_t n = (uint32_t)S.n;
  const uint64_t GN = (uint64_t)S.G * n;
  const int P = S.P, NL = S.NL;
  const PartView pv = part_view<BLOCK>(P);
  const uint64_t lrow = (uint64_t)level * NL;
  __shared__ uint32_t stage_all[NW * kStage], hstage_all[NW * kStageHeavy];
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  Stage sg = {stage_all + wv * kStage, hstage_all + wv * kStageHeavy, 0, 0};
  const LevelLists<false> lists{S, level};
  {
    const uint32_t nl = *tail_at(S, level, pv.p), nh = *tail_at(S, level, P + pv.p);
    const uint64_t nb = S.off[lrow + pv.p] + nl, nhb = S.off[lrow + P + pv.p] + nh;
    if (pv.thread == 0) open_level(S, level, pv.p, nl, nh, nb, nhb);
    if ((nl | nh) == 0u) return;  // no lanes left in this partition's groups
    // capacity exceeded (the batch is redone); the test is the same for every
    // thread of the workgroup, so no wave leaves before the counter barrier
    if (nb > list_end(S, pv.p) || nhb > list_end(S, P + pv.p)) return;
  }
  const int lane = lane_id();
  ull *seen = S.msk + M_SEEN * GN;
  const ull *cur = S.msk + (M_FR + (level & 3)) * GN;
  ull *nxt = S.msk + (M_FR + ((level + 1) & 3)) * GN;
  const ull *prv = S.msk + (M_FR + ((level + 3) & 3)) * GN;

  // retire the masks of level-2 so that word can collect level+2
  if (level >= 2) {
    ull *old = S.msk + (M_FR + ((level + 2) & 3)) * GN;
    for (int l = pv.p; l < NL; l += P) {
      const uint64_t pb = S.off[lrow - 2 * NL + l], pc = S.cnt[lrow - 2 * NL + l];
      for (uint64_t i = pv.thread; i < pc; i += pv.nthreads) old[S.items[pb + i]] = 0ull;
    }
  }
  // This launch pulls sigma for the level's items unless the bottom-up kernel
  // already found them with their counts, and discovers level+1 unless that
  // level will be found bottom-up.  Both tests read complete counts, so every
  // workgroup decides alike.
  bool pull = true, disc = true;
  if (S.bu_den > 0) {
    uint64_t prev = 0, here = 0;
    if (level >= 1)
      for (int l = 0; l < NL; ++l) prev += S.cnt[lrow - NL + l];
    for (int l = 0; l < NL; ++l) here += *tail_at(S, level, l);
    pull = !bottom_up_rule(S.bu_den, level, prev, S.gused, S.n);
    disc = !bottom_up_rule(S.bu_den, level + 1, here, S.gused, S.n);
  }
  // Level 1 needs no pull: lane b's only level-0 vertex is its source and no
  // arc is repeated, so each lane of an item has the one predecessor: sigma is
  // 1, and v lies below a target iff the source is one (S.ovl[G + g]).  Level 1
  // holds the hubs, whose thousands of in-arcs would be read for one tail each
  // (R-MAT 20, 1,000 sources: the level takes 2.5 ms with the pull, 2.2 without).
  const bool rows = level > 1 && pull;

  // counters, all wave-uniform: (source, vertex), (source, arc) and
  // (source, DAG arc) pairs; items and the out-degree sum over items
  uint64_t c_v = 0, c_a = 0, c_d = 0, c_it = 0, c_ia = 0;
  bool ovf = false, wide = false;
  T *sig = counts<T>(S);
  const ListView lv = list_view(S);
  const uint64_t base = S.off[lrow + (lv.heavy ? P : 0) + pv.p];
  const uint64_t count = *tail_at(S, level, (lv.heavy ? P : 0) + pv.p);
  // light: a block holds as many items as give every wavefront one block, at
  // most kBlockItems, and its wavefront takes every step; heavy: a workgroup
  // per item, wavefront wv takes every NW-th step
  const uint64_t nwv = lv.heavy ? lv.nwg : lv.nwg * NW;
  const uint32_t B = lv.heavy ? 1u : (uint32_t)min((uint64_t)kBlockItems, (count + nwv - 1) / nwv);
  // a workgroup without items has no appends and counts to flush (a grid of
  // 3 x 5,000 vertices, 768 items a level: 19.8 us a level with them, 16 without)
  if (lv.wg * (lv.heavy ? 1u : NW * B) >= count) return;
  const uint32_t cstart = lv.heavy ? 32u * wv : 0u, cstep = lv.heavy ? 32u * NW : 32u;
  const bool upper = lane >= 32;
  const uint32_t k32 = (uint32_t)lane & 31u;
  __shared__ ull red_acc[NW][kLanes], red_ov[NW], red_dn[NW];
  for (uint64_t b0 = (lv.heavy ? lv.wg : lv.wg * NW + (uint64_t)wv) * B; b0 < count; b0 += nwv * B) {
    const int nb = (int)min((uint64_t)B, count - b0);
    // a lane per item: its lanes, where its rows start and how long they
    // are, and whether it is a target
    uint32_t it = 0, gb = 0, e0 = 0, ed = 0, f0 = 0, fd = 0;
    ull mk = 0ull, dnr = 0ull;
    bool tgt = false;
    if (lane < nb) {
      it = S.items[base + b0 + lane];
      const uint32_t g = it / n, v = it - g * n;
      gb = it - v;
      mk = cur[it];
      e0 = (uint32_t)G.rp[v];
      ed = (uint32_t)(G.rp[v + 1] - G.rp[v]);
      if (rows) {
        f0 = (uint32_t)G.irp[v];
        fd = (uint32_t)(G.irp[v + 1] - G.irp[v]);
      }
      if (pull) {
        tgt = S.tgt_of[v] >= 0;
        dnr = tgt ? mk : (level == 1 ? mk & S.ovl[S.G + g] : 0ull);
      } else {
        dnr = S.msk[M_DN * GN + it] & mk;
      }
    }
    if (!lv.heavy || wv == 0) {
      const uint64_t pc = (uint64_t)__popcll(mk);
      c_it += (uint64_t)nb;
      c_ia += wave_sum(ed);
      if (pull) {  // a level found bottom-up was counted there
        const uint64_t pairs = wave_sum(pc);
        c_v += pairs;
        c_a += wave_sum(pc * ed);
        if (level == 1) c_d += pairs;
        if (__ballot(tgt) != 0ull && lane == 0) atomicMin(S.tmin, (uint32_t)level);
      }
    }
    if (!disc) ed = 0;
    // the block's steps: 32 in-arcs (lower half of the wavefront) and 32
    // out-arcs (upper half) of an item, item after item
    const uint32_t longest = max(ed, fd);
    auto advance = [&](int &j, uint32_t &c) {
      if (j >= nb) return;
      c += cstep;
      if (c >= read_lane(longest, j)) {
        c = cstart;
        ++j;
      }
    };
    // loads without branches (a lane without an arc reads element 0), so
    // that they stay in flight across the step
    auto ends = [&](int j, uint32_t c, bool &has) -> uint32_t {
      const int jj = j < nb ? j : 0;
      const uint32_t at = c + k32;
      has = j < nb && at < (upper ? read_lane(ed, jj) : read_lane(fd, jj));
      const uint64_t i = (uint64_t)(upper ? read_lane(e0, jj) : read_lane(f0, jj)) + at;
      return (uint32_t)(upper ? G.col : G.icol)[has ? i : 0];
    };
    auto words = [&](int j, uint32_t x, bool has) -> ull {
      const uint32_t gj = read_lane(gb, j < nb ? j : 0);
      return (upper ? seen : prv)[has ? gj + x : 0u];
    };
    int j0 = 0, j1 = 0, j2;
    uint32_t c0 = cstart, c1 = cstart, c2;
    bool h0, h1, h2;
    uint32_t x0 = ends(j0, c0, h0);
    advance(j1, c1);
    uint32_t x1 = ends(j1, c1, h1);
    ull m0 = words(j0, x0, h0);
    ull acc = 0ull, ov = 0ull, got = 0ull, pdn = 0ull;
    while ((rows || disc) && j0 < nb) {
      const ull mj = read_lane64(mk, j0);
      const uint32_t gj = read_lane(gb, j0);
      // flags of the out-arcs; their results are used after the rows
      const ull dag = (upper && h0) ? mj & ~m0 : 0ull;
      const ull pm = (!upper && h0) ? mj & m0 : 0ull;
      ull was = ~0ull;
      if (dag != 0ull) was = atomicOr(&seen[gj + x0], dag);
      const ull pd = S.msk[M_DN * GN + (pm != 0ull ? gj + x0 : 0u)];
      ull bits = __ballot(pm != 0ull);
      Rows<T> r;
      r.issue(sig, gj, x0, pm, bits, got, c_d);
      // the next step's words and the arc ends of the one after
      j2 = j1;
      c2 = c1;
      advance(j2, c2);
      const ull m1 = words(j1, x1, h1);
      const uint32_t x2 = ends(j2, c2, h2);
      const ull fresh = dag & ~was;
      ull first = ~0ull;
      if (fresh != 0ull) first = atomicOr(&nxt[gj + x0], fresh);
      r.add(acc, ov);
      while (bits != 0ull) {
        r.issue(sig, gj, x0, pm, bits, got, c_d);
        r.add(acc, ov);
      }
      pdn |= pd & pm;
      if (j1 != j0 && !lv.heavy) {  // the item's last step
        if (rows) {
          const uint32_t ij = read_lane(it, j0);
          if (__builtin_amdgcn_inverse_ballot_w64(mj)) store_count(&sig[(uint64_t)ij * kLanes + lane], acc, wide);
          if (ov != 0ull) {
            ovf = true;
            if (lane == 0) atomicOr(&S.ovl[gj / n], ov);
          }
          const ull dn = wave_or(pdn);
          if (lane == j0) dnr |= dn;
        }
        acc = ov = pdn = 0ull;
      }
      append_chunk(S, lists, pv.p, sg, gj, x0, first == 0ull);
      j0 = j1;
      c0 = c1;
      j1 = j2;
      c1 = c2;
      x0 = x1;
      x1 = x2;
      h0 = h1;
      h1 = h2;
      m0 = m1;
    }
    if (level == 1)  // every lane's one path
      for (int j = 0; j < nb; ++j)
        if ((!lv.heavy || wv == 0) && __builtin_amdgcn_inverse_ballot_w64(read_lane64(mk, j)))
          sig[(uint64_t)read_lane(it, j) * kLanes + lane] = 1;
    if (lv.heavy) {
      if (rows) {  // the same for the whole workgroup
        const ull dn = wave_or(pdn);
        red_acc[wv][lane] = acc;
        if (lane == 0) {
          red_ov[wv] = ov;
          red_dn[wv] = dn;
        }
        __syncthreads();
        if (wv == 0) {
          ull dnt = dn;
          for (int q = 1; q < NW; ++q) {
            const ull sum = acc + red_acc[q][lane];
            ov |= red_ov[q] | __ballot(sum < acc);
            dnt |= red_dn[q];
            acc = sum;
          }
          if (__builtin_amdgcn_inverse_ballot_w64(read_lane64(mk, 0)))
            store_count(&sig[(uint64_t)read_lane(it, 0) * kLanes + lane], acc, wide);
          if (ov != 0ull) {
            ovf = true;
            if (lane == 0) atomicOr(&S.ovl[read_lane(gb, 0) / n], ov);
          }
          if (lane == 0) dnr |= dnt;
        }
        __syncthreads();  // the next item overwrites the partial sums
      }
      if (wv != 0) continue;
    }
    // the items' lanes for the backward: all of them for exports, else
    // those where v is a target or lies below one (a target's dependency
    // reads psi nowhere else)
    if (lane < nb) {
      if (pull && dnr != 0ull) S.msk[M_DN * GN + it] |= dnr;
      S.imask[base + b0 + lane] = S.keep_all ? mk : dnr;
    }
  }
  if (sizeof(T) == 4 && __ballot(wide) != 0ull && lane == 0) atomicOr(&S.flags[2], 1u);
  flush_stage_wg<BLOCK / 64>(S, lists, pv.p, sg);
  const int ck[5] = {C_FWD_VPAIRS, C_FWD_APAIRS, C_FWD_DPAIRS, C_FWD_ITEMS, C_FWD_IARCS};
  const uint64_t cv[5] = {c_v, c_a, c_d, c_it, c_ia};
  flush_wave_counters<BLOCK, 5>(S.ctr, S.ctr_slots, ck, cv, ovf, S.flags);
}

// Push form of the path counts: sigma_b(w) += sigma_b(v) for every DAG arc
// (v, w) of lane b, one 64-bit atomic add per (lane, DAG arc).  The chunk
// holds the out-arcs of up to K items (slot t = arc lane / (64 / K));
// `push` on an arc lane holds the lanes for which that arc is a DAG arc, sv[t]
// is this lane's path count at item t and dn[t] (wave-uniform) the item's
// lanes that are a target or lie below one, which follow the count to the
// head.  Adds of up to eight arcs are issued before their results are
// checked; an add whose result wraps means the exact count exceeds 2^64 - 1
// (every addend is nonnegative, so the running sum crosses 2^64 once).
template <int K>
static __device__ __forceinline__ void push_slots(const BatchState &S, uint64_t gbase, uint32_t w, ull push,
                                                  int lane, const ull (&sv)[K], const ull (&dn)[K], bool &ovf,
                                                  uint64_t &dag_pairs) {
  constexpr int SUB = kLanes / K;
  ull bits = __ballot(push != 0ull);
  while (bits != 0ull) {
    int j[8];
    int c = 0;
    for (; c < 8 && bits != 0ull; ++c) {
      j[c] = __ffsll((long long)bits) - 1;
      bits &= bits - 1ull;
    }
    ull old[8], add[8];
    uint64_t gq8[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      old[q] = 0ull;
      add[q] = 0ull;
      gq8[q] = 0;
      if (q < c) {
        const uint32_t wq = read_lane(w, j[q]);
        const ull dq = read_lane64(push, j[q]);
        const uint64_t gq = read_lane64(gbase, j[q]);
        const int slot = j[q] / SUB;
        ull x = sv[0], dnq = dn[0];
#pragma unroll
        for (int t = 1; t < K; ++t)
          if (slot == t) {
            x = sv[t];
            dnq = dn[t];
          }
        dag_pairs += (uint64_t)__popcll(dq);  // wave-uniform
        gq8[q] = gq + wq;
        if ((dq >> lane) & 1ull) {
          add[q] = x;
          old[q] = atomicAdd(&S.sig[(gq + wq) * kLanes + lane], x);
        }
        // the head's lanes below a target on this arc (one atomic per arc)
        const ull dd = dnq & dq;
        if (dd != 0ull && lane == 0) atomicOr(&S.msk[(uint64_t)M_DN * S.G * S.n + gq + wq], dd);
      }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (q < c && old[q] + add[q] < old[q]) {
        ovf = true;
        atomicOr(&S.ovl[(uint32_t)(gq8[q] / (uint64_t)S.n)], 1ull << lane);
      }
  }
}

// One BFS level of the batched forward pass with pushed path counts (the
// alternative to k_fwd_level's pull; same results bit for bit, since the
// counts are exact integer sums).  For every item (g, v, mask) on `level`:
// sigma_b(v) is final (pushed by the level before, or pulled by k_bu_level
// when this level was found bottom-up); every out-arc (v, w) whose head is
// not settled on a level <= `level` for lane b of mask is a DAG arc of lane
// b: w is flagged for level+1 (one atomicOr per arc, the first flagger
// appends it) and sigma_b(v) is added into sigma_b(w).  No in-arc is read.
// Here seen lags by a level (the owner of (g, v) ORs its lanes in during this
// launch, and a reader sees seen | cur, the same union either way), since a
// lane already flagged for level+1 still takes this arc's count.
// Path-count rows must start at zero on every lane (k_batch_cleanup resets
// the lanes a batch settled).
template <int BLOCK, int K>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_fwd_push(DevGraph G,
                                                                                                BatchState S,
                                                                                                int level) {
  constexpr int SUB = kLanes / K;
  const uint64_t n = (uint64_t)S.n;
  const int P = S.P, NL = S.NL;
  const PartView pv = part_view<BLOCK>(P);
  const uint64_t lrow = (uint64_t)level * NL;
  __shared__ uint32_t stage_all[(BLOCK / 64) * kStage], hstage_all[(BLOCK / 64) * kStageHeavy];
  const int wv = threadIdx.x >> 6;
  Stage sg = {stage_all + wv * kStage, hstage_all + wv * kStageHeavy, 0, 0};
  const LevelLists<false> lists{S, level};
  const uint32_t nl = *tail_at(S, level, pv.p), nh = *tail_at(S, level, P + pv.p);
  const uint64_t nb = S.off[lrow + pv.p] + nl, nhb = S.off[lrow + P + pv.p] + nh;
  if (pv.thread == 0) open_level(S, level, pv.p, nl, nh, nb, nhb);
  if ((nl | nh) == 0u) return;  // no lanes left in this partition's groups
  // capacity exceeded (workgroup-uniform test): the batch is redone
  if (nb > list_end(S, pv.p) || nhb > list_end(S, P + pv.p)) return;
  const int lane = lane_id();
  const int sl = lane % SUB;
  const uint64_t GN = (uint64_t)S.G * n;
  ull *seen = S.msk + M_SEEN * GN, *dnm = S.msk + M_DN * GN;
  const ull *cur = S.msk + (M_FR + (level & 3)) * GN;
  ull *nxt = S.msk + (M_FR + ((level + 1) & 3)) * GN, *old = S.msk + (M_FR + ((level + 2) & 3)) * GN;
  if (level >= 2)  // retire the masks of level-2
    for (int l = pv.p; l < NL; l += P) {
      const uint64_t pb = S.off[lrow - 2 * NL + l], pc = S.cnt[lrow - 2 * NL + l];
      for (uint64_t i = pv.thread; i < pc; i += pv.nthreads) old[S.items[pb + i]] = 0ull;
    }
  uint64_t prev = 0, here = 0;
  if (level >= 1)
    for (int l = 0; l < NL; ++l) prev += S.cnt[lrow - NL + l];
  for (int l = 0; l < NL; ++l) here += *tail_at(S, level, l);
  const bool own = !bottom_up_rule(S.bu_den, level, prev, S.gused, S.n);  // found top-down
  const bool disc = !bottom_up_rule(S.bu_den, level + 1, here, S.gused, S.n);

  uint64_t c_v = 0, c_a = 0, c_d = 0, c_it = 0, c_ia = 0;  // wave-uniform counters
  bool ovf = false;
  const ListView lv = list_view(S);
  const int l = lv.heavy ? P + pv.p : pv.p;
  const uint64_t base = S.off[lrow + l], count = *tail_at(S, level, l);
  const uint64_t step = lv.nwg * (uint64_t)(BLOCK / 64 * K);
  const uint64_t first = (lv.wg * (BLOCK / 64) + (uint64_t)wv) * (uint64_t)K;
  uint64_t ii = first + (uint64_t)(lane / SUB);  // this lane's item
  uint32_t it_next = ii < count ? S.items[base + ii] : 0u;
  for (uint64_t i0 = first; i0 < count; i0 += step, ii += step) {
    const bool has = ii < count;
    const uint32_t it = it_next;
    if (ii + step < count) it_next = S.items[base + ii + step];
    const uint32_t g = (uint32_t)(it / n);
    const uint32_t v = (uint32_t)(it - (uint64_t)g * n);
    const uint64_t gbase = (uint64_t)g * n;
    ull mask = 0ull, dnr = 0ull;
    int64_t e0 = 0, e1 = 0;
    int32_t tg = -1;
    if (has) {
      mask = cur[it];
      dnr = dnm[it];
      e0 = G.rp[v];
      e1 = G.rp[v + 1];
      if (own) tg = S.tgt_of[v];
    }
    const int64_t d1 = disc ? e1 : e0;  // end of the out-arcs to scan
    if (has && sl == 0 && own) seen[it] = seen[it] | mask;
    // per slot: the item's lanes, their marks, and this lane's path count
    ull mt[K], dn[K], sv[K];
#pragma unroll
    for (int t = 0; t < K; ++t) {
      const int ld = t * SUB;
      mt[t] = read_lane64(mask, ld);
      const bool is_tgt = (int32_t)read_lane((uint32_t)tg, ld) >= 0;
      dn[t] = (read_lane64(dnr, ld) | (is_tgt ? mt[t] : 0ull)) & mt[t];
      sv[t] = ((mt[t] >> lane) & 1ull) ? S.sig[(uint64_t)read_lane(it, ld) * kLanes + lane] : 0ull;
    }
    // first chunk of every slot's out-arcs: heads, their masks, the flags
    const int64_t mo = e0 + sl;
    uint32_t w = 0;
    ull push = 0ull;
    bool enq = false;
    if (mo < d1) {
      w = (uint32_t)G.col[mo];
      push = mask & ~(seen[gbase + w] | cur[gbase + w]);  // the DAG lanes of this arc
      const ull dag = push & ~nxt[gbase + w];  // lanes already flagged by another wavefront need no atomic
      if (dag != 0ull) enq = (atomicOr(&nxt[gbase + w], dag) == 0ull);
    }
    push_slots<K>(S, gbase, w, push, lane, sv, dn, ovf, c_d);
    append_chunk(S, lists, pv.p, sg, gbase, w, enq);
#pragma unroll
    for (int t = 0; t < K; ++t) {
      const int ld = t * SUB;
      const ull m = mt[t];
      if (m == 0ull) {  // slot past the end of the list (or an empty item)
        if (lane == 0 && i0 + (uint64_t)t < count) S.imask[base + i0 + t] = 0ull;
        continue;
      }
      const uint32_t itt = read_lane(it, ld);
      const uint64_t gbt = read_lane64(gbase, ld);
      const int64_t E0 = (int64_t)read_lane64((ull)e0, ld), E1 = (int64_t)read_lane64((ull)d1, ld);
      const uint64_t deg = (uint64_t)((int64_t)read_lane64((ull)e1, ld) - E0);
      c_it += 1;
      c_ia += deg;
      if (own) {  // a level found bottom-up was counted and marked there
        c_v += (uint64_t)__popcll(m);
        c_a += (uint64_t)__popcll(m) * deg;
        const bool is_tgt = (int32_t)read_lane((uint32_t)tg, ld) >= 0;
        if (is_tgt && lane == 0) {
          atomicMin(S.tmin, (uint32_t)level);
          dnm[itt] |= m;
        }
      }
      if (lane == 0) S.imask[base + i0 + t] = S.keep_all ? m : dn[t];
      ull s1[1] = {sv[t]}, d1m[1] = {dn[t]};
      for (int64_t e = E0 + SUB; e < E1; e += kLanes) {
        const int64_t my = e + lane;
        uint32_t ww = 0;
        ull pp = 0ull;
        bool eq = false;
        if (my < E1) {
          ww = (uint32_t)G.col[my];
          pp = m & ~(seen[gbt + ww] | cur[gbt + ww]);
          const ull dd = pp & ~nxt[gbt + ww];
          if (dd != 0ull) eq = (atomicOr(&nxt[gbt + ww], dd) == 0ull);
        }
        push_slots<1>(S, gbt, ww, pp, lane, s1, d1m, ovf, c_d);
        append_chunk(S, lists, pv.p, sg, gbt, ww, eq);
      }
    }
  }
  flush_stage_wg<BLOCK / 64>(S, lists, pv.p, sg);
  const int ck[5] = {C_FWD_VPAIRS, C_FWD_APAIRS, C_FWD_DPAIRS, C_FWD_ITEMS, C_FWD_IARCS};
  const uint64_t cv[5] = {c_v, c_a, c_d, c_it, c_ia};
  flush_wave_counters<BLOCK, 5>(S.ctr, S.ctr_slots, ck, cv, ovf, S.flags);
}

// One BFS level found bottom-up (direction-optimizing BFS, here over 64
// sources at once): every (g, w) of the batch with in-arcs and with lanes
// not yet settled scans its in-arcs (u, w); lanes b of u's previous-level
// mask that are unsettled at w are DAG arcs of w on this level, so one scan
// both finds the level's lanes of w and pulls their path counts (a lane is
// on the level iff some in-arc delivered a count to it).  No atomics on the
// masks; (g, w) is appended to the level's list if it gained any lane.
// Runs before the top-down kernel of the same level, and only when
// bottom_up_rule holds for the level.  The unsettled pairs of a 64-vertex
// block are taken two at a time in steps of 32 in-arcs each; a heavy vertex is
// taken by a workgroup, as in k_fwd_level.  Bound as that kernel is (R-MAT 20,
// 1,000 sources: 19 ms of two levels with one chain of loads per pair, 12.6
// with rows of words and a chunk at a time, 8.8 as here: 6.4 + 2.4; 5, 6 or 7
// waves per SIMD alike).
template <int BLOCK, class T>
__global__ __launch_bounds__(BLOCK) void k_bu_level(DevGraph G, BatchState S, int level) {
  constexpr int NW = BLOCK / 64;
  const uint64_t n = (uint64_t)S.n;
  const int P = S.P, NL = S.NL;
  const uint64_t lrow = (uint64_t)level * NL;
  uint64_t prev = 0;
  for (int l = 0; l < NL; ++l) prev += S.cnt[lrow - NL + l];
  if (!bottom_up_rule(S.bu_den, level, prev, S.gused, S.n)) return;
  const PartView pv = part_view<BLOCK>(P);
  __shared__ uint32_t stage_all[NW * kStage], hstage_all[NW * kStageHeavy];
  const int wv = threadIdx.x >> 6;
  Stage sg = {stage_all + wv * kStage, hstage_all + wv * kStageHeavy, 0, 0};
  const LevelLists<true> lists{S, level};
  // capacity exceeded earlier (workgroup-uniform test): the batch is redone
  if (S.off[lrow + pv.p] > list_end(S, pv.p) || S.off[lrow + P + pv.p] > list_end(S, P + pv.p)) return;
  const int lane = lane_id();
  const uint64_t GN = (uint64_t)S.G * n;
  ull *seen = S.msk + M_SEEN * GN, *dnm = S.msk + M_DN * GN, *cur = S.msk + (M_FR + (level & 3)) * GN;
  const ull *prv = S.msk + (M_FR + ((level + 3) & 3)) * GN;
  uint64_t c_v = 0, c_a = 0, c_d = 0;
  bool ovf = false, wide = false;
  T *sig = counts<T>(S);
  // groups p, p + P, ... below gused belong to this partition
  const uint64_t ngp = S.gused > pv.p ? (uint64_t)(S.gused - pv.p + P - 1) / (uint64_t)P : 0;
  // heavy vertices: a workgroup each, its wavefronts share the in-arcs
  const ListView lv = list_view(S);
  __shared__ ull red_acc[NW][kLanes], red_hit[NW], red_ov[NW], red_dn[NW];
  if (lv.heavy) for (uint64_t i = lv.wg; i < ngp * S.H; i += lv.nwg) {
    const uint64_t gl = i / S.H;
    const uint32_t g = (uint32_t)(pv.p + gl * (uint64_t)P);
    const uint32_t w = (uint32_t)(i - gl * S.H);
    const uint64_t gbase = (uint64_t)g * n;
    const ull un = ((g + 1 == (uint32_t)S.gused) ? S.last_lanes : ~0ull) & ~seen[gbase + w];
    const int64_t f1 = G.irp[w + 1];
    ull acc = 0ull, dnt = 0ull, ovm = 0ull, nm = 0ull;
    if (un != 0ull)
      for (int64_t e = G.irp[w] + 64 * wv; e < f1; e += BLOCK) {
        const int64_t my = e + lane;
        uint32_t u = 0;
        ull pm = 0ull, pd = 0ull;
        if (my < f1) {
          u = (uint32_t)G.icol[my];
          pm = prv[gbase + u] & un;
          if (pm != 0ull) pd = dnm[gbase + u] & pm;
        }
        pull_rows(sig, (uint32_t)gbase, u, pm, acc, ovm, nm, c_d);
        dnt |= wave_or(pd);
      }
    red_acc[wv][lane] = acc;
    if (lane == 0) {
      red_ov[wv] = ovm;
      red_hit[wv] = nm;
      red_dn[wv] = dnt;
    }
    __syncthreads();
    if (wv == 0) {
      for (int q = 1; q < NW; ++q) {
        const ull sum = acc + red_acc[q][lane];
        ovm |= red_ov[q] | __ballot(sum < acc);
        dnt |= red_dn[q];
        nm |= red_hit[q];
        acc = sum;
      }
      if (nm != 0ull) {
        const uint32_t it = (uint32_t)(gbase + w);
        const uint64_t deg = (uint64_t)(G.rp[w + 1] - G.rp[w]);
        const bool is_tgt = S.tgt_of[w] >= 0;
        if ((nm >> lane) & 1ull) store_count(&sig[(uint64_t)it * kLanes + lane], acc, wide);
        if (ovm != 0ull) {
          ovf = true;
          if (lane == 0) atomicOr(&S.ovl[g], ovm);
        }
        if (is_tgt) dnt |= nm;
        if (lane == 0) {
          cur[it] = nm;
          seen[it] |= nm;
          if (dnt != 0ull) dnm[it] |= dnt;
          if (is_tgt) atomicMin(S.tmin, (uint32_t)level);
        }
        c_v += (uint64_t)__popcll(nm);
        c_a += (uint64_t)__popcll(nm) * deg;
        append_chunk(S, lists, pv.p, sg, gbase, w, lane == 0);
      }
    }
    __syncthreads();  // the next vertex overwrites the partial results
  }
  // light vertices H .. n-1, 64 to a block; the ids run by falling degree, so
  // a block takes eight runs of eight (a line of words each) spread evenly
  // over them, and all blocks hold about the same arcs
  const uint64_t nlt = n - S.H, nvb = (nlt + 63) / 64;
  const uint64_t first = lv.heavy ? ngp * nvb : lv.wg * NW + (uint64_t)wv;
  const bool upper = lane >= 32;
  const uint32_t k32 = (uint32_t)lane & 31u;
  for (uint64_t b = first; b < ngp * nvb; b += lv.nwg * NW) {
    const uint64_t gl = b / nvb;
    const uint32_t g = (uint32_t)(pv.p + gl * (uint64_t)P);
    const uint32_t gb = g * (uint32_t)n;
    const uint64_t wl = S.H + (b - gl * nvb) * 8 + (uint64_t)(lane >> 3) * nvb * 8 + (uint64_t)(lane & 7);
    const ull act_lanes = (g + 1 == (uint32_t)S.gused) ? S.last_lanes : ~0ull;
    uint32_t w = 0, f0 = 0, fd = 0;
    ull un = 0ull;
    if (wl < n) {
      w = (uint32_t)wl;
      const int64_t r0 = G.irp[w];
      f0 = (uint32_t)r0;
      fd = (uint32_t)(G.irp[w + 1] - r0);
      if (fd != 0u) un = act_lanes & ~seen[gb + w];
      if (un == 0ull) fd = 0u;
    }
    const ull cm = __ballot(un != 0ull);
    const int nc = __popcll(cm);
    if (nc == 0) continue;
    // the candidates move to lanes 0 .. nc-1 (every lane takes part)
    {
      const int to = 4 * (un != 0ull ? lanes_below(cm) : nc + lanes_below(~cm));
      w = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)w);
      f0 = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)f0);
      fd = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)fd);
      const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(uint32_t)un);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(uint32_t)(un >> 32));
      un = ((ull)hi << 32) | lo;
    }
    // steps of 32 in-arcs of candidate j (lower half of the wavefront) and 32
    // of j + 1 (upper half), loaded ahead as in the forward
    const uint32_t longest = max(fd, (uint32_t)__shfl_xor((int)fd, 1));
    auto advance = [&](int &j, uint32_t &c) {
      if (j >= nc) return;
      c += 32;
      if (c >= read_lane(longest, j)) {
        c = 0;
        j += 2;
      }
    };
    auto ends = [&](int j, uint32_t c, bool &has) -> uint32_t {
      const int jj = j < nc ? j : 0;
      const uint32_t at = c + k32;
      has = j < nc && at < (upper ? read_lane(fd, jj + 1) : read_lane(fd, jj));
      const uint64_t i = (uint64_t)(upper ? read_lane(f0, jj + 1) : read_lane(f0, jj)) + at;
      return (uint32_t)G.icol[has ? i : 0];
    };
    auto words = [&](uint32_t x, bool has) -> ull { return prv[has ? gb + x : 0u]; };
    int j0 = 0, j1 = 0, j2;
    uint32_t c0 = 0, c1 = 0, c2;
    bool h0, h1, h2;
    uint32_t x0 = ends(j0, c0, h0);
    advance(j1, c1);
    uint32_t x1 = ends(j1, c1, h1);
    ull m0 = words(x0, h0);
    ull acc[2] = {0ull, 0ull}, ov[2] = {0ull, 0ull}, got[2] = {0ull, 0ull}, pdn = 0ull;
    ull nm = 0ull, dnr = 0ull;  // lane j: candidate j's lanes on this level, and those below a target
    while (j0 < nc) {
      const ull u0 = read_lane64(un, j0), u1 = read_lane64(un, j0 + 1);
      const ull pm = h0 ? m0 & (upper ? u1 : u0) : 0ull;
      const ull pd = dnm[pm != 0ull ? gb + x0 : 0u];
      const ull all = __ballot(pm != 0ull);
      ull bits = all & 0xFFFFFFFFull;
      Rows<T> r;
      r.issue(sig, gb, x0, pm, bits, got[0], c_d);
      j2 = j1;
      c2 = c1;
      advance(j2, c2);
      const ull m1 = words(x1, h1);
      const uint32_t x2 = ends(j2, c2, h2);
      r.add(acc[0], ov[0]);
      while (bits != 0ull) {
        r.issue(sig, gb, x0, pm, bits, got[0], c_d);
        r.add(acc[0], ov[0]);
      }
      bits = all & ~0xFFFFFFFFull;
      while (bits != 0ull) {
        r.issue(sig, gb, x0, pm, bits, got[1], c_d);
        r.add(acc[1], ov[1]);
      }
      pdn |= pd & pm;
      if (j1 != j0) {  // the pair's last step
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          if (got[t] != 0ull) {
            const uint64_t it = (uint64_t)(gb + read_lane(w, j0 + t));
            if (__builtin_amdgcn_inverse_ballot_w64(got[t])) store_count(&sig[it * kLanes + lane], acc[t], wide);
            if (ov[t] != 0ull) {
              ovf = true;
              if (lane == 0) atomicOr(&S.ovl[g], ov[t]);
            }
            const ull dn = wave_or((t == 1) == upper ? pdn : 0ull);
            if (lane == j0 + t) {
              nm = got[t];
              dnr = dn;
            }
          }
          acc[t] = ov[t] = got[t] = 0ull;
        }
        pdn = 0ull;
      }
      j0 = j1;
      c0 = c1;
      j1 = j2;
      c1 = c2;
      x0 = x1;
      x1 = x2;
      h0 = h1;
      h1 = h2;
      m0 = m1;
    }
    // a lane per candidate: its masks, marks and counters
    if (__ballot(nm != 0ull) == 0ull) continue;
    uint64_t pairs = 0, arcs = 0;
    if (nm != 0ull) {
      const uint32_t it = gb + w;
      const bool is_tgt = S.tgt_of[w] >= 0;
      if (is_tgt) {
        dnr |= nm;
        atomicMin(S.tmin, (uint32_t)level);
      }
      cur[it] = nm;
      seen[it] |= nm;
      if (dnr != 0ull) dnm[it] |= dnr;
      pairs = (uint64_t)__popcll(nm);
      arcs = pairs * (uint64_t)(G.rp[w + 1] - G.rp[w]);
    }
    c_v += wave_sum(pairs);
    c_a += wave_sum(arcs);
    append_chunk(S, lists, pv.p, sg, gb, w, nm != 0ull);
  }
  if (sizeof(T) == 4 && __ballot(wide) != 0ull && lane == 0) atomicOr(&S.flags[2], 1u);
  flush_stage_wg<BLOCK / 64>(S, lists, pv.p, sg);
  const int ck[3] = {C_FWD_VPAIRS, C_FWD_APAIRS, C_FWD_DPAIRS};
  const uint64_t cv[3] = {c_v, c_a, c_d};  // wave-uniform
  flush_wave_counters<BLOCK, 3>(S.ctr, S.ctr_slots, ck, cv, ovf, S.flags);
}

// Successor rows of a chunk of arc lanes, up to eight at a time, as Rows: arc
// lane j holds the head w and the lanes d for which it is a shortest-path-DAG
// successor.  add() adds psi_b(w) to acc (this lane's source) in arc lane
// order, which is arc order; adding 0.0 for a lane off the DAG leaves its sum
// unchanged.
struct PsiRows {
  double x[8];
  __device__ __forceinline__ void issue(const double *psi, uint32_t gb, uint32_t w, ull d, ull &bits,
                                        uint64_t &dag_pairs) {
    const int lane = lane_id();
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (bits != 0ull) {
        const int j = __builtin_ctzll(bits);
        bits &= bits - 1ull;
        const ull dq = read_lane64(d, j);
        const double *row = psi + (uint64_t)(gb + read_lane(w, j)) * kLanes;
        dag_pairs += (uint64_t)__popcll(dq);
        if (__builtin_amdgcn_inverse_ballot_w64(dq)) x[q] = row[lane];
      }
    }
  }
  __device__ __forceinline__ void add(double &acc) {
#pragma unroll
    for (int q = 0; q < 8; ++q) acc += x[q];
  }
};

// One level of the backward pass, Eq.(4) read as
//   delta(v) = sigma(v) * sum_{w: v in P(w)} psi(w),  psi(w) = (1 + delta(w)) / sigma(w),
// so psi(v) = 1/sigma(v) + sum psi(w).  Successor w of v is on the DAG for
// lane b iff w sits on level+1 for b, read from the masks the previous
// (deeper) launch wrote.  Only the lanes the forward kept in the item's mask
// are computed -- those where v is a target or lies below one (no target's
// dependency reads psi anywhere else) -- and target vertices report delta on
// their lanes.  No atomics: every sum runs in arc order, so results are
// bit-reproducible.  The masks rotate over three words: written (level), read
// (level+1) and cleared (level+2).
// Light items are taken in blocks as in the forward (a lane per
// item loads what is needed of it; items without lanes are passed over), each
// with the whole wavefront over its out-arcs, the next item's arc ends loaded
// ahead.  Heavy items are dealt to wavefronts by eight sources, lanes over
// eight of the part's DAG arcs by its eight sources, 64 arcs in flight: a hub
// summed by one wavefront a few rows at a time kept the level waiting with 2
// to 30 % of the wavefront slots used (R-MAT 20, 1,000 sources: the two
// shallowest levels 4.0 + 1.4 ms, as here 1.8 + 0.65; R-MAT 16 2.99 -> 2.60 ms a
// call).
template <int BLOCK, class T>
__global__ __launch_bounds__(BLOCK) void k_bwd_level(DevGraph G, BatchState S, int level, int ntgt) {
  constexpr int NW = BLOCK / 64;
  const uint32_t n = (uint32_t)S.n;
  const uint64_t GN = (uint64_t)S.G * n;
  const int P = S.P, NL = S.NL;
  const PartView pv = part_view<BLOCK>(P);
  const uint64_t lrow = (uint64_t)level * NL;
  if (S.off[lrow + pv.p] + S.cnt[lrow + pv.p] > list_end(S, pv.p) ||
      S.off[lrow + P + pv.p] + S.cnt[lrow + P + pv.p] > list_end(S, P + pv.p))
    return;
  const int lane = lane_id();
  const ull *bw_in = S.msk + (M_BW + (level + 1) % 3) * GN;
  ull *bw_out = S.msk + (M_BW + level % 3) * GN;
  // level+2's masks make room for level-1 (its lists exist: the forward ran
  // at least one level past the deepest one)
  if (level + 2 <= S.top) {
    ull *bw_old = S.msk + (M_BW + (level + 2) % 3) * GN;
    for (int l = pv.p; l < NL; l += P) {
      const uint64_t pb = S.off[lrow + 2 * NL + l], pc = S.cnt[lrow + 2 * NL + l];
      for (uint64_t i = pv.thread; i < pc; i += pv.nthreads)
        if (S.imask[pb + i] != 0ull) bw_old[S.items[pb + i]] = 0ull;
    }
  }
  uint64_t c_v = 0, c_a = 0, c_d = 0, c_it = 0, c_ia = 0;  // wave-uniform counters
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const ListView lv = list_view(S);
  __shared__ uint32_t part_w[NW][128], part_d[NW][128];
  __shared__ double part_x[NW][64 * 8];
  if (lv.heavy) {
    // a wavefront per (item, eight sources): psi's 64 bytes of those sources
    // are one access, so the parts share no line of it
    const uint64_t base = S.off[lrow + P + pv.p], count = S.cnt[lrow + P + pv.p];
    uint32_t *qw = part_w[wv], *qd = part_d[wv];  // arcs of the part's DAG lanes, a ring of 128
    double *xs = part_x[wv];
    const uint32_t a8 = (uint32_t)lane >> 3, b8 = (uint32_t)lane & 7u;
    uint32_t dl_pairs = 0;  // this lane's
    for (uint64_t t = lv.wg * NW + (uint64_t)wv; t < count * 8; t += lv.nwg * NW) {
      const uint32_t p = (uint32_t)(t & 7u);
      const ull em = first_lane64(S.imask[base + (t >> 3)]);
      if (em == 0ull) continue;
      const uint32_t eb = (uint32_t)(em >> (8 * p)) & 0xFFu;
      if (eb == 0u && p != 0u) continue;
      const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.items[base + (t >> 3)]);
      const uint32_t g = it / n, v = it - g * n, gb = g * n;
      const uint64_t e0 = (uint64_t)G.rp[v];
      const uint32_t ed = (uint32_t)((uint64_t)G.rp[v + 1] - e0);
      if (p == 0u) {
        if (lane == 0) bw_out[it] = em;
        c_v += (uint64_t)__popcll(em);
        c_a += (uint64_t)__popcll(em) * (uint64_t)ed;
        c_it += 1;
        c_ia += (uint64_t)ed;
        if (eb == 0u) continue;
      }
      const uint8_t *bytes = reinterpret_cast<const uint8_t *>(bw_in + gb) + p;
      const double *psi = S.psi + (uint64_t)gb * kLanes + 8 * p + b8;
      auto ends = [&](uint32_t c) -> uint32_t {
        const uint32_t at = c + (uint32_t)lane;
        return (uint32_t)G.col[at < ed ? e0 + at : 0];
      };
      auto byte_of = [&](uint32_t c, uint32_t x) -> uint32_t { return bytes[c + (uint32_t)lane < ed ? (uint64_t)x * 8 : 0]; };
      uint32_t c = 0, head = 0, queued = 0, flying = 0;
      uint32_t x0 = ends(0), x1 = ends(64), m0 = byte_of(0, x0);
      double acc = 0.0, x[8];  // acc: the sum of source 8 p + b8, the same in all eight lanes
      for (;;) {
        // the next 64 DAG arcs, in arc order; the words of the next step and
        // the arc ends of the one after are loaded ahead
        while (queued < 64u && c < ed) {
          const uint32_t d = c + (uint32_t)lane < ed ? m0 & eb : 0u;
          const uint32_t m1 = byte_of(c + 64, x1), x2 = ends(c + 128);
          const ull on = __ballot(d != 0u);
          if (d != 0u) {
            const uint32_t at = (head + queued + (uint32_t)lanes_below(on)) & 127u;
            qw[at] = x0;
            qd[at] = d;
          }
          dl_pairs += (uint32_t)__popc(d);
          queued += (uint32_t)__popcll(on);
          c += 64;
          x0 = x1;
          x1 = x2;
          m0 = m1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // the arcs in flight are added in their order
        if (flying != 0u) {
#pragma unroll
          for (int q = 0; q < 8; ++q) xs[q * 64 + lane] = x[q];
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          for (uint32_t r = 0; r < flying; r += 8)
#pragma unroll
            for (int q = 0; q < 8; ++q) acc += xs[(r + q) * 8 + b8];
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        flying = min(queued, 64u);
        if (flying == 0u) break;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const uint32_t k = 8u * q + a8, at = (head + k) & 127u;
          x[q] = 0.0;
          if (k < flying && ((qd[at] >> b8) & 1u)) x[q] = psi[(uint64_t)qw[at] * kLanes];
        }
        head += flying;
        queued -= flying;
      }
      if (lane < 8 && ((eb >> b8) & 1u)) {
        const int32_t tgt = S.tgt_of[v];
        const uint64_t o = (uint64_t)it * kLanes + 8 * p + b8;
        const double s = (double)counts<T>(S)[o];
        const double dl = s * acc;
        S.psi[o] = acc + 1.0 / s;
        if (S.dout) S.dout[o] = dl;
        if (tgt >= 0 && tgt < ntgt) S.res[((uint64_t)tgt * S.G + g) * kLanes + 8 * p + b8] = (level > 0) ? dl : 0.0;
      }
    }
    c_d += wave_sum(dl_pairs);
  } else {
    const uint64_t base = S.off[lrow + pv.p], count = S.cnt[lrow + pv.p];
    const uint64_t nwv = lv.nwg * NW;
    const uint32_t B = (uint32_t)min((uint64_t)kBlockItems, (count + nwv - 1) / nwv);
    for (uint64_t b0 = (lv.wg * NW + (uint64_t)wv) * B; b0 < count; b0 += nwv * B) {
      const int nb = (int)min((uint64_t)B, count - b0);
      uint32_t it = 0, gb = 0, e0 = 0, ed = 0;
      int32_t tg = -1;
      ull mk = 0ull;
      if (lane < nb) mk = S.imask[base + b0 + lane];
      ull todo = __ballot(mk != 0ull);
      if (todo == 0ull) continue;
      if (mk != 0ull) {
        it = S.items[base + b0 + lane];
        const uint32_t v = it % n;
        gb = it - v;
        e0 = (uint32_t)G.rp[v];
        ed = (uint32_t)(G.rp[v + 1] - G.rp[v]);
        tg = S.tgt_of[v];
        bw_out[it] = mk;
      }
      {
        const uint64_t pc = (uint64_t)__popcll(mk);
        c_it += (uint64_t)__popcll(todo);
        c_ia += wave_sum(ed);
        c_v += wave_sum(pc);
        c_a += wave_sum(pc * ed);
      }
      // the block's steps: 64 out-arcs of an item with lanes, item after item;
      // words of the next step and arc ends of the one after are loaded ahead
      auto advance = [&](ull &t, uint32_t &c) {
        c += kLanes;
        if (c >= read_lane(ed, __builtin_ctzll(t))) {
          c = 0;
          t &= t - 1ull;
        }
      };
      auto ends = [&](ull t, uint32_t c, bool &has) -> uint32_t {
        const int j = t != 0ull ? __builtin_ctzll(t) : 0;
        const uint32_t at = c + (uint32_t)lane;
        has = t != 0ull && at < read_lane(ed, j);
        return (uint32_t)G.col[has ? (uint64_t)read_lane(e0, j) + at : 0];
      };
      auto words = [&](ull t, uint32_t x, bool has) -> ull {
        const uint32_t gj = read_lane(gb, t != 0ull ? __builtin_ctzll(t) : 0);
        return bw_in[has ? gj + x : 0u];
      };
      ull t0 = todo, t1 = todo, t2;
      uint32_t c0 = 0, c1 = 0, c2;
      bool h0, h1, h2;
      uint32_t x0 = ends(t0, c0, h0);
      advance(t1, c1);
      uint32_t x1 = t1 != 0ull ? ends(t1, c1, h1) : (h1 = false, 0u);
      ull m0 = words(t0, x0, h0), sg = 1;
      double acc = 0.0;
      while (t0 != 0ull) {
        const int j = __builtin_ctzll(t0);
        const ull em = read_lane64(mk, j);
        const uint32_t gj = read_lane(gb, j), ij = read_lane(it, j);
        const bool mine = __builtin_amdgcn_inverse_ballot_w64(em);
        const ull d = h0 ? em & m0 : 0ull;
        if (c0 == 0 && mine) sg = counts<T>(S)[(uint64_t)ij * kLanes + lane];
        t2 = t1;
        c2 = c1;
        h2 = false;
        uint32_t x2 = 0;
        ull bits = __ballot(d != 0ull);
        PsiRows r;
        r.issue(S.psi, gj, x0, d, bits, c_d);
        const ull m1 = words(t1, x1, h1);
        if (t2 != 0ull) {
          advance(t2, c2);
          x2 = ends(t2, c2, h2);
        }
        r.add(acc);
        while (bits != 0ull) {
          r.issue(S.psi, gj, x0, d, bits, c_d);
          r.add(acc);
        }
        if (t1 != t0) {  // the item's last step
          const int32_t tgt = (int32_t)read_lane((uint32_t)tg, j);
          if (mine) {
            const double s = (double)sg;
            const double dl = s * acc;
            S.psi[(uint64_t)ij * kLanes + lane] = acc + 1.0 / s;
            if (S.dout) S.dout[(uint64_t)ij * kLanes + lane] = dl;
            if (tgt >= 0 && tgt < ntgt) S.res[((uint64_t)tgt * S.G + gj / n) * kLanes + lane] = (level > 0) ? dl : 0.0;
          }
          acc = 0.0;
        }
        t0 = t1;
        c0 = c1;
        t1 = t2;
        c1 = c2;
        x0 = x1;
        x1 = x2;
        h0 = h1;
        h1 = h2;
        m0 = m1;
      }
    }
  }
  const int ck[5] = {C_BWD_VPAIRS, C_BWD_APAIRS, C_BWD_DPAIRS, C_BWD_ITEMS, C_BWD_IARCS};
  const uint64_t cv[5] = {c_v, c_a, c_d, c_it, c_ia};
  flush_wave_counters<BLOCK, 5>(S.ctr, S.ctr_slots, ck, cv, false, S.flags);
}

// Reset what the batch touched: the masks of every item and, when the path
// counts were pushed (added into), the counts of every lane the batch
// settled, so the next batch's adds start from zero.  (Pulled counts need no
// reset: every lane's count is written before anything reads it, and only
// lanes named by a mask are ever read.)  A wavefront per item, lanes over
// the 64 counts of its row; an item repeated on several levels clears the
// row again or finds the masks already cleared, and either way every
// settled lane is zeroed by the first wavefront that read the masks.
__global__ void k_batch_cleanup(BatchState S, PartTotals tot) {
  const int lane = lane_id();
  const uint64_t GN = (uint64_t)S.G * (uint64_t)S.n;
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
  for (int l = 0; l < S.NL; ++l) {
    uint64_t total = tot.t[l];
    const uint64_t cap = list_end(S, l) - list_begin(S, l);
    if (total > cap) total = cap;
    const uint32_t *items = S.items + list_begin(S, l);
    for (uint64_t i = wave; i < total; i += nwaves) {
      const uint32_t it = items[i];
      if (S.push) {
        const ull vis = S.msk[M_SEEN * GN + it];
        if ((vis >> lane) & 1ull) S.sig[(uint64_t)it * kLanes + lane] = 0ull;
      }
      if (lane < M_COUNT) S.msk[lane * GN + it] = 0ull;
    }
  }
}

// The same for a batch that touched a good part of its groups' vertices: every
// mask word of the groups it used (pulled counts only), in whole lines.
__global__ void k_batch_clear(BatchState S) {
  const uint64_t GN = (uint64_t)S.G * (uint64_t)S.n, used = (uint64_t)S.gused * (uint64_t)S.n;
  for (int a = 0; a < M_COUNT; ++a)
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < used; i += (uint64_t)gridDim.x * blockDim.x)
      S.msk[a * GN + i] = 0ull;
}

// Verification export of one level: per lane with a slot, distance = level,
// sigma and delta from the state rows.
__global__ void k_batch_export(DevGraph G, BatchState S, int level, uint64_t begin, uint64_t count,
                               const int32_t *lane_slot, uint64_t *dist, ull *sigma, double *delta,
                               int64_t k) {
  const uint64_t n = (uint64_t)S.n;
  const int lane = lane_id();
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
  if (begin + count > list_end(S, S.NL - 1)) return;
  for (uint64_t i = wave; i < count; i += nwaves) {
    const uint32_t it = S.items[begin + i];  // begin: absolute position (partition region + level offset)
    const uint32_t g = (uint32_t)(it / n);
    const uint32_t v = (uint32_t)(it - (uint64_t)g * n);
    const ull mask = S.imask[begin + i];
    if (!((mask >> lane) & 1ull)) continue;
    const int32_t slot = lane_slot[g * kLanes + lane];
    if (slot < 0 || slot >= k) continue;
    const uint64_t o = (uint64_t)slot * n + (uint32_t)G.orig[v];
    dist[o] = (uint64_t)level;
    sigma[o] = S.narrow ? counts<uint32_t>(S)[(uint64_t)it * kLanes + lane] : S.sig[(uint64_t)it * kLanes + lane];
    if (delta && S.dout) delta[o] = S.dout[(uint64_t)it * kLanes + lane];
  }
}

// --------------------------------------------------------------- plain

__global__ void k_plain_init(PlainState P, int32_t s) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    P.d[s] = 0;
    P.sig[s] = 1ull;
    P.queue[0] = s;
    P.cnt[0] = 1u;
    P.off[0] = 0ull;
  }
}

// One BFS level from a single source: a wavefront per frontier vertex,
// lanes over its out-arcs; the first lane to claim a vertex appends it
// (ballot + mbcnt compaction, one queue atomic per wavefront).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_plain_fwd(DevGraph G, PlainState P, int level) {
  const uint64_t base = P.off[level];
  const uint64_t count = P.cnt[level];
  const uint64_t nbase = base + count;
  if (blockIdx.x == 0 && threadIdx.x == 0) P.off[level + 1] = nbase;
  if (nbase > (uint64_t)P.n) return;
  const int lane = lane_id();
  uint64_t c_v = 0, c_a = 0, c_d = 0;
  bool ovf = false;
  const uint64_t wave = ((uint64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6;
  const uint64_t nwaves = ((uint64_t)gridDim.x * BLOCK) >> 6;
  for (uint64_t i = wave; i < count; i += nwaves) {
    const int32_t v = P.queue[base + i];
    const ull sv = P.sig[v];
    const int64_t e0 = G.rp[v], e1 = G.rp[v + 1];
    if (lane == 0) {
      c_v += 1;
      c_a += (uint64_t)(e1 - e0);
    }
    for (int64_t e = e0; e < e1; e += 64) {
      const int64_t my = e + lane;
      bool enq = false, dag = false;
      int32_t w = 0;
      if (my < e1) {
        w = G.col[my];
        int32_t dw = P.d[w];
        if (dw < 0) {
          const int32_t o = atomicCAS(&P.d[w], -1, level + 1);
          if (o == -1) {
            enq = true;
            dw = level + 1;
          } else {
            dw = o;
          }
        }
        dag = (dw == level + 1);
        if (dag) {
          const ull o = atomicAdd(&P.sig[w], sv);
          if (o + sv < o) ovf = true;
        }
      }
      c_d += dag ? 1 : 0;
      const ull eb = __ballot(enq);
      if (eb != 0ull) {
        uint32_t p0 = 0;
        if (lane == 0) p0 = atomicAdd(&P.cnt[level + 1], (uint32_t)__popcll(eb));
        p0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)p0);
        if (enq) {
          const uint64_t p = nbase + p0 + (uint64_t)lanes_below(eb);
          if (p < (uint64_t)P.n) P.queue[p] = w;
        }
      }
    }
  }
  flush_counters<BLOCK>(P.ctr, P.ctr_slots, C_FWD_VPAIRS, c_v, c_a, c_d, ovf, P.flags);
}

// One backward level from a single source: lanes over out-arcs gather psi
// of successors on level+1; the wavefront sum is a fixed shuffle tree.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_plain_bwd(DevGraph G, PlainState P, int level, int32_t target,
                                                     int only_target) {
  const uint64_t base = P.off[level];
  const uint64_t count = P.cnt[level];
  if (base + count > (uint64_t)P.n) return;
  const int lane = lane_id();
  uint64_t c_v = 0, c_a = 0, c_d = 0;
  const uint64_t wave = ((uint64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6;
  const uint64_t nwaves = ((uint64_t)gridDim.x * BLOCK) >> 6;
  for (uint64_t i = wave; i < count; i += nwaves) {
    const int32_t v = P.queue[base + i];
    if (only_target && v != target) continue;
    const int64_t e0 = G.rp[v], e1 = G.rp[v + 1];
    double acc = 0.0;
    for (int64_t e = e0; e < e1; e += 64) {
      const int64_t my = e + lane;
      if (my < e1) {
        const int32_t w = G.col[my];
        if (P.d[w] == level + 1) {
          acc += P.psi[w];
          c_d += 1;
        }
      }
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) {
      const double s = (double)P.sig[v];
      P.psi[v] = acc + 1.0 / s;
      P.dout[v] = s * acc;
      c_v += 1;
      c_a += (uint64_t)(e1 - e0);
    }
  }
  flush_counters<BLOCK>(P.ctr, P.ctr_slots, C_BWD_VPAIRS, c_v, c_a, c_d, false, P.flags);
}

__global__ void k_plain_cleanup(PlainState P, uint64_t total) {
  if (total > (uint64_t)P.n) total = (uint64_t)P.n;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const int32_t v = P.queue[i];
    P.d[v] = -1;
    P.sig[v] = 0ull;
  }
}

__global__ void k_plain_export(PlainState P, uint64_t *dist, ull *sigma, double *delta) {
  for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < (uint64_t)P.n;
       v += (uint64_t)gridDim.x * blockDim.x) {
    const int32_t d = P.d[v];
    if (dist) dist[v] = d < 0 ? ~0ull : (uint64_t)d;
    if (sigma) sigma[v] = d < 0 ? 0ull : P.sig[v];
    if (delta) delta[v] = d < 0 ? 0.0 : P.dout[v];
  }
}

// --------------------------------------------------------- reachability

__global__ void k_reach_clear(uint32_t *bitmap, int64_t words, ReachCtr ctr) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (int64_t)gridDim.x * blockDim.x)
    bitmap[i] = 0u;
  if (blockIdx.x == 0 && threadIdx.x < 4) {
    *ctr.len((int)threadIdx.x) = 0u;
    *ctr.arcs((int)threadIdx.x) = 0u;
    if (threadIdx.x == 0) ctr.c[1] = 0u;
  }
}

__global__ void k_reach_init(uint32_t *bitmap, int32_t *q, ReachCtr ctr, int32_t root, const int32_t *roots, int k) {
  for (int i = threadIdx.x; i < k; i += blockDim.x) {
    const int32_t r = roots ? roots[i] : root;
    atomicOr(&bitmap[r >> 5], 1u << (r & 31));
    q[i] = r;
  }
  if (threadIdx.x == 0) *ctr.len(0) = (uint32_t)k;
}

// Append the vertices u of the lanes where `enq` holds to the queue.
static __device__ __forceinline__ void queue_append(uint32_t *stg, int &nst, uint32_t *tail, int32_t *q, int32_t u,
                                                    bool enq) {
  const ull eb = __ballot(enq);
  if (eb == 0ull) return;
  const int c = __popcll(eb);
  // every vertex is claimed once, so the queue (length n) cannot overflow
  if (nst + c > kStage) stage_flush(stg, nst, tail, (uint32_t *)q, 0, ~0ull, nullptr);
  if (enq) stg[nst + lanes_below(eb)] = (uint32_t)u;
  nst += c;
}

// One BFS level on a CSR, weights ignored.  Every append adds the vertex's arc
// count (its row in this CSR) to the next level's arcs, which decide its
// direction.
// Top-down: lanes over a frontier vertex's arcs, first setter of a bit appends
// the vertex.  A frontier smaller than the launch is dealt in parts: a row to
// several wavefronts (the first level is one vertex, for a query on a hub one
// with tens of thousands of arcs, which one wavefront walked in 370 us at
// R-MAT 20).
// Bottom-up (bu_arcs or more arcs to scan top-down, set only): every vertex
// not yet reached scans its arcs in the opposite direction and joins as soon
// as one of them leads to a reached vertex.  A vertex reached earlier in the
// same launch may be the one found, which can put a vertex in this level that
// the top-down order would put in a later one; the set is the same.  A thread
// per vertex looks at its first kReachAlone arcs, four at a time; the rest of a
// longer row is scanned by the whole wavefront, since a vertex that does not
// join reads its whole row.
// Bound by the latency of the row -> bitmap chain.  What cost most before were
// the ends of the launch: 32,768 wavefronts adding to the same two counters
// (about 10 ns each) made 390 and 320 us of the two large levels of R-MAT 20;
// with 1,024 workgroups adding once each they take 61 and 55.
constexpr int kReachAlone = 16;
__global__ __launch_bounds__(kReachLevelBlock) void k_reach_level(const int64_t *rp, const int32_t *col,
                                                                  const int64_t *rpo, const int32_t *colo,
                                                                  uint32_t *bitmap, int32_t *q0, int32_t *q1,
                                                                  ReachCtr ctr, uint8_t *lev, int level, int64_t n,
                                                                  uint64_t bu_arcs) {
  constexpr int BLOCK = kReachLevelBlock;
  const uint64_t tid = (uint64_t)blockIdx.x * BLOCK + threadIdx.x;
  const uint32_t count = *ctr.len(level);
  if (tid == 0) {
    *ctr.len(level + 2) = 0u;
    *ctr.arcs(level + 2) = 0u;
    if (count != 0u) ctr.c[1] = (uint32_t)level;
  }
  if (count == 0u) return;
  const bool bottom_up = *ctr.arcs(level) >= bu_arcs;
  const int32_t *qin = (level & 1) ? q1 : q0;
  int32_t *qout = (level & 1) ? q0 : q1;
  uint32_t *tail = ctr.len(level + 1);
  const int lane = lane_id();
  __shared__ uint32_t st_all[(BLOCK / 64) * kStage];
  uint32_t *stg = st_all + (threadIdx.x >> 6) * kStage;
  int nst = 0;
  uint64_t arcs = 0;
  const uint64_t nwaves = ((uint64_t)gridDim.x * BLOCK) >> 6;
  if (!bottom_up) {
    const uint64_t parts = count < nwaves ? min((uint64_t)64, nwaves / count) : 1;
    for (uint64_t i = tid >> 6; i < count * parts; i += nwaves) {
      const int32_t v = qin[i / parts];
      const int64_t r0 = rp[v], deg = rp[v + 1] - r0, part = (int64_t)(i % parts);
      const int64_t e1 = r0 + deg * (part + 1) / (int64_t)parts;
      for (int64_t e = r0 + deg * part / (int64_t)parts; e < e1; e += 64) {
        const int64_t my = e + lane;
        bool enq = false;
        int32_t u = 0;
        if (my < e1) {
          u = col[my];
          const uint32_t bit = 1u << (u & 31);
          if (!(bitmap[u >> 5] & bit)) enq = !(atomicOr(&bitmap[u >> 5], bit) & bit);
          if (enq && lev) lev[u] = (uint8_t)(level + 1 < 254 ? level + 1 : 254);
          if (enq) arcs += (uint64_t)(rp[u + 1] - rp[u]);
        }
        queue_append(stg, nst, tail, qout, u, enq);
      }
    }
  } else {
    // the loop bound is the same for every lane of a wavefront (whole
    // wavefronts stride together), so the ballots below see every lane
    const uint64_t span = (((uint64_t)n + 63) / 64) * 64, nth = (uint64_t)gridDim.x * BLOCK;
    auto reached = [&](uint32_t w) { return (bitmap[w >> 5] >> (w & 31)) & 1u; };
    for (uint64_t u = tid; u < span; u += nth) {
      bool join = false;
      int64_t e = 0, e1 = 0;
      const uint32_t mine = u < (uint64_t)n ? bitmap[u >> 5] : ~0u;
      if (!((mine >> (u & 31)) & 1u)) {
        e = rpo[u];
        e1 = rpo[u + 1];
        for (int k = 0; k < kReachAlone && e < e1 && !join; k += 4, e += 4) {
          uint32_t w[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) w[q] = (uint32_t)colo[e + q < e1 ? e + q : e];
#pragma unroll
          for (int q = 0; q < 4; ++q) join = join || reached(w[q]);
        }
      }
      for (ull rest = __ballot(!join && e < e1); rest != 0ull; rest &= rest - 1ull) {
        const int j = __builtin_ctzll(rest);
        const int64_t b1 = (int64_t)read_lane64((ull)e1, j);
        bool hit = false;
        for (int64_t b = (int64_t)read_lane64((ull)e, j); b < b1 && !hit; b += 64)
          hit = __ballot(b + lane < b1 && reached((uint32_t)colo[b + lane])) != 0ull;
        if (hit && lane == j) join = true;
      }
      // the wavefront owns its 64 vertices' two words in this launch: a plain
      // store each, no atomic per vertex (which bounced the bitmap's lines
      // between the XCDs)
      const ull jb = __ballot(join);
      if ((lane & 31) == 0 && (uint32_t)(jb >> lane) != 0u) bitmap[u >> 5] = mine | (uint32_t)(jb >> lane);
      if (join) arcs += (uint64_t)(rp[u + 1] - rp[u]);
      queue_append(stg, nst, tail, qout, (int32_t)u, join);
    }
  }
  // one atomic per workgroup for the queue and one for its arcs
  __shared__ uint32_t num[BLOCK / 64], at;
  __shared__ uint64_t wg_arcs[BLOCK / 64];
  const int wv = (int)(threadIdx.x >> 6);
  const uint64_t wsum = wave_sum(arcs);
  if (lane == 0) {
    num[wv] = (uint32_t)nst;
    wg_arcs[wv] = wsum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t c = 0;
    uint64_t a = 0;
    for (int w = 0; w < BLOCK / 64; ++w) {
      c += num[w];
      a += wg_arcs[w];
    }
    at = c != 0u ? atomicAdd(tail, c) : 0u;
    if (a != 0) atomicAdd((unsigned long long *)ctr.arcs(level + 1), (unsigned long long)a);
  }
  __syncthreads();
  uint32_t p0 = at;
  for (int w = 0; w < wv; ++w) p0 += num[w];
  for (int j = lane; j < nst; j += 64) qout[p0 + (uint32_t)j] = (int32_t)stg[j];
}

// At load: a wavefront per new row of either CSR, then the narrow copies.
// On weighted graphs arc e = pairs[q].y of the CSR is arc q of the transpose,
// and lies at the same place of its row in internal order.
__global__ void k_internal_rows(DevGraph F, DevGraph T, int32_t *pcol, int32_t *picol, LoadArgs A) {
  const int lane = lane_id();
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, nth = (int64_t)gridDim.x * blockDim.x;
  for (int64_t r = tid >> 6; r < 2 * A.n; r += nth >> 6) {
    const bool in = r >= A.n;
    const int64_t i = in ? r - A.n : r, *nrp = in ? T.irp : T.rp;
    const int64_t a = (in ? F.irp : F.rp)[T.orig[i]], b = nrp[i], k = nrp[i + 1] - b;
    for (int64_t j = lane; j < k; j += 64) {
      if (!in) {
        const int32_t w = A.rank[F.col[a + j]];
        pcol[b + j] = w;
        if (A.weight) A.arcw[b + j] = make_uint2((uint32_t)w, A.weight[a + j]);
      } else if (!A.weight) {
        picol[b + j] = A.rank[F.icol[a + j]];
      } else {
        const uint2 p = A.pairs[a + j];
        const int32_t u = A.rank[p.x];
        A.icol[a + j] = (int32_t)p.x;
        A.iarc[b + j] = make_uint2((uint32_t)u, A.weight[p.y]);
        A.iopos[b + j] = (uint32_t)(T.rp[u] + ((int64_t)p.y - F.rp[p.x]));
      }
    }
  }
  if (A.lrp) {
    for (int64_t i = tid; i <= A.n; i += nth) A.lrp[i] = (uint32_t)F.rp[i];
    for (int64_t e = tid; e < A.m; e += nth) A.lcol[e] = (uint16_t)F.col[e];
  }
}

hipError_t launch_internal_rows(const DevGraph &from, const DevGraph &to, int32_t *pcol, int32_t *picol,
                                const LoadArgs &A, hipStream_t st) {
  const int grid = (int)std::min<int64_t>(8192, (A.n + 1) / 2);
  hipLaunchKernelGGL(k_internal_rows, dim3(grid), dim3(256), 0, st, from, to, pcol, picol, A);
  return hipGetLastError();
}

// Streaming probes over n16 16-byte words: every thread keeps four 16-byte
// loads in flight (one per grid stride) before it uses them, so the probe is
// bound by HBM and not by the latency of one load at a time.  Copy: loads and
// stores marked non-temporal (streamed past the caches).  Read: the words are
// folded into one value that is stored only if it matches a sentinel, so the
// loads cannot be dropped.
typedef unsigned v4u __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_copy(const v4u *__restrict__ src, v4u *__restrict__ dst, int64_t n16) {
  const int64_t nth = (int64_t)gridDim.x * blockDim.x;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + 3 * nth < n16; i += 4 * nth) {
    v4u v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(&src[i + u * nth]);
#pragma unroll
    for (int u = 0; u < 4; ++u) __builtin_nontemporal_store(v[u], &dst[i + u * nth]);
  }
  for (; i < n16; i += nth) dst[i] = src[i];
}

__global__ __launch_bounds__(256) void k_read(const v4u *__restrict__ src, int64_t n16, unsigned *sink) {
  const int64_t nth = (int64_t)gridDim.x * blockDim.x;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  unsigned acc = 0;
  for (; i + 3 * nth < n16; i += 4 * nth) {
    v4u v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = src[i + u * nth];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  for (; i < n16; i += nth) acc ^= src[i].x;
  if (acc == 0x9E3779B9u) sink[0] = acc;
}

// ------------------------------------------------------------ launchers

#define DISPATCH_BLOCK(L, KERNEL, ...)                                                     \
  do {                                                                                     \
    switch ((L).block) {                                                                   \
      case 64: hipLaunchKernelGGL(KERNEL<64>, dim3((L).grid), dim3(64), 0, st, __VA_ARGS__); break;    \
      case 128: hipLaunchKernelGGL(KERNEL<128>, dim3((L).grid), dim3(128), 0, st, __VA_ARGS__); break; \
      case 512: hipLaunchKernelGGL(KERNEL<512>, dim3((L).grid), dim3(512), 0, st, __VA_ARGS__); break; \
      default: hipLaunchKernelGGL(KERNEL<256>, dim3((L).grid), dim3(256), 0, st, __VA_ARGS__); break;  \
    }                                                                                      \
  } while (0)

// the same for the kernels that read or write the path counts
#define DISPATCH_COUNTS(T, L, KERNEL, ...)                                                 \
  do {                                                                                     \
    switch ((L).block) {                                                                   \
      case 64: KERNEL<64, T><<<dim3((L).grid), dim3(64), 0, st>>>(__VA_ARGS__); break;     \
      case 128: KERNEL<128, T><<<dim3((L).grid), dim3(128), 0, st>>>(__VA_ARGS__); break;  \
      case 512: KERNEL<512, T><<<dim3((L).grid), dim3(512), 0, st>>>(__VA_ARGS__); break;  \
      default: KERNEL<256, T><<<dim3((L).grid), dim3(256), 0, st>>>(__VA_ARGS__); break;   \
    }                                                                                      \
  } while (0)

hipError_t launch_batch_init(const BatchState &S, const uint32_t *items0, const ull *masks0, const uint32_t *dest0,
                             int k, hipStream_t st) {
  if (k <= 0) return hipSuccess;
  const int grid = (k + 255) / 256;
  hipLaunchKernelGGL(k_batch_init, dim3(grid), dim3(256), 0, st, S, items0, masks0, dest0, k);
  return hipGetLastError();
}

template <int K>
static void launch_push_k(const DevGraph &G, const BatchState &S, int level, const Launch &L, hipStream_t st) {
  switch (L.block) {
    case 64: k_fwd_push<64, K><<<dim3(L.grid), dim3(64), 0, st>>>(G, S, level); break;
    case 128: k_fwd_push<128, K><<<dim3(L.grid), dim3(128), 0, st>>>(G, S, level); break;
    case 512: k_fwd_push<512, K><<<dim3(L.grid), dim3(512), 0, st>>>(G, S, level); break;
    default: k_fwd_push<256, K><<<dim3(L.grid), dim3(256), 0, st>>>(G, S, level); break;
  }
}

hipError_t launch_bu_level(const DevGraph &G, const BatchState &S, int level, Launch L, hipStream_t st) {
  if (S.narrow) DISPATCH_COUNTS(uint32_t, L, k_bu_level, G, S, level);
  else DISPATCH_COUNTS(ull, L, k_bu_level, G, S, level);
  return hipGetLastError();
}

hipError_t launch_fwd_level(const DevGraph &G, const BatchState &S, int level, Launch L, hipStream_t st) {
  if (S.push) {
    switch (L.items) {
      case 2: launch_push_k<2>(G, S, level, L, st); break;
      case 4: launch_push_k<4>(G, S, level, L, st); break;
      default: launch_push_k<1>(G, S, level, L, st); break;
    }
  } else {
    if (S.narrow) DISPATCH_COUNTS(uint32_t, L, k_fwd_level, G, S, level);
    else DISPATCH_COUNTS(ull, L, k_fwd_level, G, S, level);
  }
  return hipGetLastError();
}

hipError_t launch_publish_counts(const BatchState &S, int level, hipStream_t st) {
  hipLaunchKernelGGL(k_publish_counts, dim3(1), dim3(64), 0, st, S, level);
  return hipGetLastError();
}

hipError_t launch_bwd_level(const DevGraph &G, const BatchState &S, int level, int ntgt, Launch L, hipStream_t st) {
  if (S.narrow) DISPATCH_COUNTS(uint32_t, L, k_bwd_level, G, S, level, ntgt);
  else DISPATCH_COUNTS(ull, L, k_bwd_level, G, S, level, ntgt);
  return hipGetLastError();
}

hipError_t launch_batch_cleanup(const BatchState &S, const PartTotals &tot, Launch L, hipStream_t st) {
  // clearing every word costs M_COUNT words per (group, vertex) in whole
  // lines, the sparse form M_COUNT lines per item
  uint64_t items = 0;
  for (int l = 0; l < S.NL; ++l) items += tot.t[l];
  if (!S.push && items * 8 >= (uint64_t)S.gused * (uint64_t)S.n)
    hipLaunchKernelGGL(k_batch_clear, dim3(L.grid), dim3(256), 0, st, S);
  else
    hipLaunchKernelGGL(k_batch_cleanup, dim3(L.grid), dim3(256), 0, st, S, tot);
  return hipGetLastError();
}

hipError_t launch_batch_export(const DevGraph &G, const BatchState &S, int level, uint64_t begin, uint64_t count,
                               const int32_t *lane_slot, uint64_t *dist, ull *sigma, double *delta, int64_t k,
                               hipStream_t st) {
  if (count == 0) return hipSuccess;
  uint64_t waves = count < 65536 ? count : 65536;
  const int grid = (int)((waves * 64 + 255) / 256);
  hipLaunchKernelGGL(k_batch_export, dim3(grid), dim3(256), 0, st, G, S, level, begin, count, lane_slot, dist,
                     sigma, delta, k);
  return hipGetLastError();
}

hipError_t launch_plain_init(const PlainState &P, int32_t s, hipStream_t st) {
  hipLaunchKernelGGL(k_plain_init, dim3(1), dim3(64), 0, st, P, s);
  return hipGetLastError();
}

hipError_t launch_plain_fwd(const DevGraph &G, const PlainState &P, int level, Launch L, hipStream_t st) {
  DISPATCH_BLOCK(L, k_plain_fwd, G, P, level);
  return hipGetLastError();
}

hipError_t launch_plain_bwd(const DevGraph &G, const PlainState &P, int level, int32_t target, int only_target,
                            Launch L, hipStream_t st) {
  DISPATCH_BLOCK(L, k_plain_bwd, G, P, level, target, only_target);
  return hipGetLastError();
}

hipError_t launch_plain_cleanup(const PlainState &P, uint64_t total, hipStream_t st) {
  if (total == 0) return hipSuccess;
  uint64_t g = (total + 255) / 256;
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(k_plain_cleanup, dim3((int)g), dim3(256), 0, st, P, total);
  return hipGetLastError();
}

hipError_t launch_plain_export(const PlainState &P, uint64_t *dist, ull *sigma, double *delta,
                               hipStream_t st) {
  uint64_t g = ((uint64_t)P.n + 255) / 256;
  if (g > 4096) g = 4096;
  hipLaunchKernelGGL(k_plain_export, dim3((int)g), dim3(256), 0, st, P, dist, sigma, delta);
  return hipGetLastError();
}

hipError_t launch_plain_export(const PlainState &P, uint64_t total, uint64_t *dist, ull *sigma, double *delta,
                               hipStream_t st) {
  (void)total;
  return launch_plain_export(P, dist, sigma, delta, st);
}

hipError_t launch_reach_init(uint32_t *bitmap, int64_t words, int32_t *q, ReachCtr ctr, int32_t root,
                             const int32_t *roots, int k, hipStream_t st) {
  const int grid = (int)std::min<int64_t>(1024, (words + 255) / 256);
  hipLaunchKernelGGL(k_reach_clear, dim3(grid), dim3(256), 0, st, bitmap, words, ctr);
  hipLaunchKernelGGL(k_reach_init, dim3(1), dim3(256), 0, st, bitmap, q, ctr, root, roots, k);
  return hipGetLastError();
}

hipError_t launch_reach_level(const int64_t *rp, const int32_t *col, const int64_t *rpo, const int32_t *colo,
                              uint32_t *bitmap, int32_t *q0, int32_t *q1, ReachCtr ctr, uint8_t *lev, int level,
                              int64_t n, uint64_t bu_arcs, Launch L, hipStream_t st) {
  // a part of the resident workgroups: each adds to the same two counters at
  // its end, one after the other (RV(r) of R-MAT 20, whole call: 512 workgroups
  // 0.76 ms, 1,024 0.74, 2,048 0.78, 4,096 0.87).  Not the configured workgroup:
  // 1,024 of 64 threads (the weighted default) are a wavefront per SIMD
  // (R-MAT 20, edge factor 8, 64-thread workgroups configured: 0.51 ms, 0.43 as here)
  hipLaunchKernelGGL(k_reach_level, dim3(reach_level_grid(L)), dim3(kReachLevelBlock), 0, st, rp, col, rpo, colo, bitmap,
                     q0, q1, ctr, lev, level, n, bu_arcs);
  return hipGetLastError();
}

hipError_t launch_copy_probe(const void *src, void *dst, int64_t n16, int grid, hipStream_t st) {
  hipLaunchKernelGGL(k_copy, dim3(grid), dim3(256), 0, st, static_cast<const v4u *>(src), static_cast<v4u *>(dst),
                     n16);
  return hipGetLastError();
}

hipError_t launch_read_probe(const void *src, int64_t n16, unsigned *sink, int grid, hipStream_t st) {
  hipLaunchKernelGGL(k_read, dim3(grid), dim3(256), 0, st, static_cast<const v4u *>(src), n16, sink);
  return hipGetLastError();
}

// ------------------------------------------------------------- targets

__global__ void k_scatter_targets(int32_t *tgt_of, const int32_t *verts, int k, int set) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < k; i += gridDim.x * blockDim.x)
    tgt_of[verts[i]] = set ? i : -1;
}

// Plain engine: distance and delta of each listed vertex.
__global__ void k_plain_gather(PlainState P, const int32_t *verts, int k, int32_t *d_out, double *delta_out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < k; i += gridDim.x * blockDim.x) {
    const int32_t v = verts[i];
    if (d_out) d_out[i] = P.d[v];
    if (delta_out) delta_out[i] = P.d[v] < 0 ? 0.0 : P.dout[v];
  }
}

// Adds the per-workgroup counter slots into acc and clears them: a thread
// per slot row (rows are contiguous, so the reads coalesce), a wavefront
// sum per counter, one atomic per counter and wavefront.  Integer sums:
// the order does not matter.
constexpr int kFoldBlock = 256;
__global__ __launch_bounds__(kFoldBlock) void k_ctr_fold(uint64_t *ctr, int slots, uint64_t *acc) {
  uint64_t s[C_COUNT];
#pragma unroll
  for (int k = 0; k < C_COUNT; ++k) s[k] = 0;
  for (int i = blockIdx.x * kFoldBlock + threadIdx.x; i < slots; i += gridDim.x * kFoldBlock) {
    uint64_t *row = ctr + (size_t)i * C_COUNT;
#pragma unroll
    for (int k = 0; k < C_COUNT; ++k) {
      s[k] += row[k];
      row[k] = 0;
    }
  }
#pragma unroll
  for (int k = 0; k < C_COUNT; ++k) {
    uint64_t v = s[k];
    for (int off = 32; off > 0; off >>= 1) v += (uint64_t)__shfl_xor((unsigned long long)v, off);
    if (lane_id() == 0 && v != 0) atomicAdd((unsigned long long *)&acc[k], (unsigned long long)v);
  }
}

hipError_t launch_ctr_fold(uint64_t *ctr, int slots, uint64_t *acc, hipStream_t st) {
  const int grid = std::max(1, std::min(32, (slots + kFoldBlock - 1) / kFoldBlock));
  hipLaunchKernelGGL(k_ctr_fold, dim3(grid), dim3(kFoldBlock), 0, st, ctr, slots, acc);
  return hipGetLastError();
}

__global__ void k_route_results(const double *res, const ResultRoute *routes, int k) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < k; i += gridDim.x * blockDim.x)
    *routes[i].dst = res[routes[i].src];
}

hipError_t launch_route_results(const double *res, const ResultRoute *routes, int k, hipStream_t st) {
  if (k <= 0) return hipSuccess;
  const int grid = std::min(4096, (k + 255) / 256);
  hipLaunchKernelGGL(k_route_results, dim3(grid), dim3(256), 0, st, res, routes, k);
  return hipGetLastError();
}

hipError_t launch_scatter_targets(int32_t *tgt_of, const int32_t *verts, int k, int set, hipStream_t st) {
  if (k <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter_targets, dim3((k + 255) / 256), dim3(256), 0, st, tgt_of, verts, k, set);
  return hipGetLastError();
}

hipError_t launch_plain_gather(const PlainState &P, const int32_t *verts, int k, int32_t *d_out,
                               double *delta_out, hipStream_t st) {
  if (k <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_plain_gather, dim3((k + 255) / 256), dim3(256), 0, st, P, verts, k, d_out, delta_out);
  return hipGetLastError();
}

}  // namespace bcd

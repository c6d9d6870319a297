// Device helpers shared by the kernel files of libbcd (wave64 primitives
// and per-workgroup counter flushing).
#pragma once

#include "bcd_internal.h"

namespace bcd {

typedef unsigned long long ull;

static __device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

static __device__ __forceinline__ int lanes_below(ull m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

static __device__ __forceinline__ uint32_t read_lane(uint32_t x, int j) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, j);
}

static __device__ __forceinline__ ull read_lane64(ull x, int j) {
  uint32_t lo = read_lane((uint32_t)x, j);
  uint32_t hi = read_lane((uint32_t)(x >> 32), j);
  return ((ull)hi << 32) | lo;
}

static __device__ __forceinline__ uint64_t first_lane64(uint64_t x) {
  uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// Sum three per-thread counters over the workgroup and add them into this
// workgroup's private counter slot (one writer per slot per launch).
template <int BLOCK>
__device__ __forceinline__ void flush_counters(uint64_t *ctr, int slots, int k0, uint64_t a, uint64_t b,
                                               uint64_t c, bool ovf, uint32_t *flags) {
  __shared__ uint64_t red[3][BLOCK / 64];
  __shared__ int any_ovf;
  if (threadIdx.x == 0) any_ovf = 0;
  __syncthreads();
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_down(a, off);
    b += __shfl_down(b, off);
    c += __shfl_down(c, off);
  }
  if (ovf) any_ovf = 1;
  const int w = threadIdx.x >> 6;
  if (lane_id() == 0) {
    red[0][w] = a;
    red[1][w] = b;
    red[2][w] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t s0 = 0, s1 = 0, s2 = 0;
    for (int i = 0; i < BLOCK / 64; ++i) {
      s0 += red[0][i];
      s1 += red[1][i];
      s2 += red[2][i];
    }
    if ((int)blockIdx.x < slots) {
      uint64_t *p = ctr + (size_t)blockIdx.x * C_COUNT + k0;
      p[0] += s0;
      p[1] += s1;
      p[2] += s2;
    }
    if (any_ovf) atomicOr(&flags[0], 1u);
  }
}

// Add wave-uniform counters (the same value on every lane of a wavefront)
// into this workgroup's slot: counter slot k[i] receives the sum over the
// workgroup's wavefronts of v[i]; an overflow on any lane raises flags[0].
// Every thread of the workgroup must call it (once per launch).
template <int BLOCK, int NV>
__device__ __forceinline__ void flush_wave_counters(uint64_t *ctr, int slots, const int (&k)[NV],
                                                    const uint64_t (&v)[NV], bool ovf, uint32_t *flags) {
  __shared__ uint64_t red[NV][BLOCK / 64];
  __shared__ int any_ovf;
  if (threadIdx.x == 0) any_ovf = 0;
  __syncthreads();
  if (ovf) any_ovf = 1;
  const int w = threadIdx.x >> 6;
  if (lane_id() == 0)
    for (int i = 0; i < NV; ++i) red[i][w] = v[i];
  __syncthreads();
  if (threadIdx.x == 0) {
    if ((int)blockIdx.x < slots) {
      uint64_t *p = ctr + (size_t)blockIdx.x * C_COUNT;
      for (int i = 0; i < NV; ++i) {
        uint64_t s = 0;
        for (int j = 0; j < BLOCK / 64; ++j) s += red[i][j];
        p[k[i]] += s;
      }
    }
    if (any_ovf) atomicOr(&flags[0], 1u);
  }
}

// Sum over the wavefront (wave-uniform result).
static __device__ __forceinline__ uint64_t wave_sum(uint64_t x) {
  for (int off = 32; off > 0; off >>= 1) x += (uint64_t)__shfl_xor((ull)x, off);
  return first_lane64(x);
}

// Per-wavefront LDS staging of list appends: values are collected in an LDS
// buffer and copied out with one tail atomic per block, so a list's shared
// tail counter is not hit once per appended element.
static __device__ __forceinline__ void stage_flush(uint32_t *buf, int &nbuf, uint32_t *tail, uint32_t *dst,
                                                   uint64_t dst_base, uint64_t dst_end, uint32_t *overflow_flag) {
  if (nbuf == 0) return;
  uint32_t p0 = 0;
  if ((threadIdx.x & 63) == 0) p0 = atomicAdd(tail, (uint32_t)nbuf);
  p0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)p0);
  for (int j = (int)(threadIdx.x & 63); j < nbuf; j += 64) {
    const uint64_t p = dst_base + p0 + (uint64_t)j;
    if (p < dst_end) dst[p] = buf[j];
    else if (overflow_flag) atomicOr(overflow_flag, 1u);
  }
  nbuf = 0;
}

// Appended items are staged in per-wavefront LDS buffers, one for the light
// and one for the heavy list of the partition, and copied to the lists in
// blocks: one counter atomic per block instead of one per chunk of arcs, which
// keeps the lists' tail counters cold.
constexpr int kStage = 256;
constexpr int kStageHeavy = 64;
// Most items a wavefront takes as one block (level launches).
constexpr int kBlockItems = 32;

struct Stage {
  uint32_t *buf, *hbuf;  // this wavefront's LDS buffers
  int n, nh;             // entries staged
};

// The item lists of the level being built: they start behind `level`'s items
// (BU: the lists of `level` itself, which the bottom-up kernel fills).  The
// positions are read again at every flush, which is rare, so that no
// registers hold them in between.
template <bool BU>
struct LevelLists {
  const BatchState &S;
  int level;
  __device__ __forceinline__ uint32_t *tail(int l) const { return tail_at(S, level + (BU ? 0 : 1), l); }
  __device__ __forceinline__ uint64_t base(int l) const {
    return S.off[(uint64_t)level * S.NL + l] + (BU ? 0u : *tail_at(S, level, l));
  }
  __device__ __forceinline__ uint64_t end(int l) const { return list_end(S, l); }
  __device__ __forceinline__ uint32_t *dst() const { return S.items; }
};

template <class Lists>
static __device__ __forceinline__ void flush_list(const BatchState &S, const Lists &L, int l, const uint32_t *buf,
                                                  int &n) {
  if (n == 0) return;
  const uint64_t base = L.base(l), end = L.end(l);
  uint32_t p0 = 0;
  if (lane_id() == 0) p0 = atomicAdd(L.tail(l), (uint32_t)n);
  p0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)p0);
  for (int j = lane_id(); j < n; j += 64) {
    const uint64_t p = base + p0 + (uint64_t)j;
    if (p < end) L.dst()[p] = buf[j];
    else atomicOr(&S.flags[1], 1u);
  }
  n = 0;
}

template <class Lists>
static __device__ __forceinline__ void flush_stage(const BatchState &S, const Lists &L, int p, Stage &g) {
  flush_list(S, L, p, g.buf, g.n);
  flush_list(S, L, S.P + p, g.hbuf, g.nh);
}

// The same at the end of a launch, for the whole workgroup at once (every
// thread calls it): one atomic per list and workgroup instead of one per
// wavefront.  Tens of thousands of wavefronts adding to one word take about 10
// ns each, one after the other.
template <int NW, class Lists>
static __device__ __forceinline__ void flush_stage_wg(const BatchState &S, const Lists &L, int p, Stage &g) {
  __shared__ uint32_t num[2][NW], at[2];
  const int wv = (int)(threadIdx.x >> 6);
  __syncthreads();
  if (lane_id() == 0) {
    num[0][wv] = (uint32_t)g.n;
    num[1][wv] = (uint32_t)g.nh;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    uint32_t c = 0;
    for (int w = 0; w < NW; ++w) c += num[threadIdx.x][w];
    at[threadIdx.x] = c != 0u ? atomicAdd(L.tail(threadIdx.x == 0 ? p : S.P + p), c) : 0u;
  }
  __syncthreads();
  for (int h = 0; h < 2; ++h) {
    const int n = h == 0 ? g.n : g.nh;
    if (n == 0) continue;
    const uint32_t *buf = h == 0 ? g.buf : g.hbuf;
    const int l = h == 0 ? p : S.P + p;
    uint64_t base = L.base(l) + at[h];
    const uint64_t end = L.end(l);
    for (int w = 0; w < wv; ++w) base += num[h][w];
    for (int j = lane_id(); j < n; j += 64) {
      if (base + (uint64_t)j < end) L.dst()[base + (uint64_t)j] = buf[j];
      else atomicOr(&S.flags[1], 1u);
    }
  }
  g.n = g.nh = 0;
}

// Append the vertices w of the lanes where `enq` holds (items gbase + w) to
// partition p's lists.
template <class Lists>
static __device__ __forceinline__ void append_chunk(const BatchState &S, const Lists &L, int p, Stage &g,
                                                    uint64_t gbase, uint32_t w, bool enq) {
  ull eb = __ballot(enq);
  if (eb == 0ull) return;
  const ull hb = __ballot(enq && w < S.H);
  if (hb != 0ull) {
    const int c = __popcll(hb);
    if (g.nh + c > kStageHeavy) flush_list(S, L, S.P + p, g.hbuf, g.nh);
    if (enq && w < S.H) g.hbuf[g.nh + lanes_below(hb)] = (uint32_t)(gbase + w);
    g.nh += c;
    eb &= ~hb;
    if (eb == 0ull) return;
  }
  const int c = __popcll(eb);
  if (g.n + c > kStage) flush_list(S, L, p, g.buf, g.n);
  if (enq && w >= S.H) g.buf[g.n + lanes_below(eb)] = (uint32_t)(gbase + w);
  g.n += c;
}

// First thing of a level's top-down launch (one thread per partition): the
// level's counts go to its cnt row, the next level's lists start behind it and
// the tails of the level after that are cleared.
static __device__ __forceinline__ void open_level(const BatchState &S, int level, int p, uint32_t nl, uint32_t nh,
                                                  uint64_t nb, uint64_t nhb) {
  const uint64_t row = (uint64_t)level * S.NL + p, next = row + S.NL;
  S.cnt[row] = nl;
  S.cnt[row + S.P] = nh;
  S.off[next] = nb;
  S.off[next + S.P] = nhb;
  *tail_at(S, level + 2, p) = 0u;
  *tail_at(S, level + 2, S.P + p) = 0u;
}

// This workgroup's share of a partitioned item list (see BatchState).
struct PartView {
  int p;              // partition served
  uint64_t wave;      // this wavefront's index within the partition
  uint64_t nwaves;    // wavefronts serving the partition
  uint64_t thread;    // this thread's index within the partition
  uint64_t nthreads;
};

template <int BLOCK>
static __device__ __forceinline__ PartView part_view(int P) {
  PartView r;
  r.p = (int)(blockIdx.x % (unsigned)P);
  const uint64_t lb = blockIdx.x / (unsigned)P, nwg = gridDim.x / (unsigned)P;
  r.wave = (lb * BLOCK + threadIdx.x) >> 6;
  r.nwaves = (nwg * BLOCK) >> 6;
  r.thread = lb * BLOCK + threadIdx.x;
  r.nthreads = nwg * BLOCK;
  return r;
}

// How a partition's workgroups are dealt between its two lists: the first
// third takes heavy items (at least one workgroup, when the graph has any; a
// partition has at least two then), the others light ones, each side striding
// over its list.  A workgroup is on one side only, so that a barrier of a heavy
// item is met by all its wavefronts; the registers are the kernel's, those of
// both sides.  With a third of the workgroups the heavy items, which take
// longest, start first and end with the light ones (R-MAT 20, 1,000 sources: an
// eighth 54.1 ms, half 50.0, a third 48.3).
struct ListView {
  bool heavy;            // this workgroup's side
  uint64_t wg, nwg;      // its index among that side's workgroups, and their number
};
static __device__ __forceinline__ ListView list_view(const BatchState &S) {
  const uint64_t lb = blockIdx.x / (unsigned)S.P, nwg = gridDim.x / (unsigned)S.P;
  const uint64_t hw = S.H == 0 ? 0 : (nwg < 6 ? 1 : nwg / 3);
  ListView r;
  r.heavy = lb < hw;
  r.wg = r.heavy ? lb : lb - hw;
  r.nwg = r.heavy ? hw : nwg - hw;
  return r;
}

}  // namespace bcd

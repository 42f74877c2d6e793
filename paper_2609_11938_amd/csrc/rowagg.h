// Device code of the aggregation by operator row shared by the fused path's
// kernels and the compact path's: partial results, the reduction of a block of
// launches ordered by row, the table in LDS, and the rows of the table.
#pragma once
#include "accum.h"
#include "common.h"
#include "impl.h"

namespace opa {

constexpr int kFFields = 25;                   // kc, tns, mc, mns, 20 counters, NaN bits
constexpr int kBuckets = 256;                  // buckets of operator rows
// A block's bucket entries: the partials (<< 16) and launch records kept before
// each bucket, before the unattributed row (NOPS), which is on its own (it has
// a partial in almost every block, which would make its bucket's combine waves
// the last to finish by far), and in all.
constexpr int kBktStride = kBuckets + 2;
constexpr int kRThreads = 256;

// LDS of the row-ordered reduction: the row histogram, later the crossing rows'
// slots. Only stretches of longrow launches and more cross lanes into a slot, so
// a wave of per launches a lane has at most 64 per / longrow of them.
__host__ __device__ inline uint32_t r_hist_words(uint32_t G) { return (G + 1) / 2; }
__host__ __device__ inline int r_slots(int per, int longrow) {
  const int n = OPA_WAVE * per / longrow;
  return n < OPA_WAVE ? n : OPA_WAVE;
}
inline size_t r_agg_lds(uint32_t G, int per, int longrow) {
  const size_t h = (size_t)r_hist_words(G) * 4;
  const size_t sl = (size_t)(kRThreads / OPA_WAVE) * r_slots(per, longrow) * kFFields * 8;
  return h > sl ? h : sl;
}

// vector of kN 32-bit elements (at most 16 bytes)
template <int kN> struct VecOf { using type = uint4; };
template <> struct VecOf<2> { using type = uint2; };
template <> struct VecOf<1> { using type = uint32_t; };

// kN consecutive 32-bit elements from p[i..), vector loads when aligned
template <int kN, typename T>
__device__ __forceinline__ void load_n(const T *p, int64_t i, int nv, T (&o)[kN]) {
  static_assert(sizeof(T) == 4 && (kN <= 2 || kN % 4 == 0), "32-bit elements, whole vectors");
  using V = typename VecOf<kN>::type;
  constexpr int kB = (int)sizeof(V);
  if (nv == kN && (reinterpret_cast<uintptr_t>(p + i) & (kB - 1)) == 0) {
    const V *v = reinterpret_cast<const V *>(p + i);
#pragma unroll
    for (int q = 0; q < kN * 4 / kB; ++q) {
      const V t = v[q];
      memcpy(reinterpret_cast<char *>(o) + kB * q, &t, kB);
    }
  } else {
#pragma unroll
    for (int k = 0; k < kN; ++k) o[k] = k < nv ? p[i + k] : T(0);
  }
}

template <int kN, typename T>
__device__ __forceinline__ void store_n(T *p, int64_t i, int nv, const T (&o)[kN]) {
  using V = typename VecOf<kN>::type;
  constexpr int kB = (int)sizeof(V);
  if (nv == kN && (reinterpret_cast<uintptr_t>(p + i) & (kB - 1)) == 0) {
    V *v = reinterpret_cast<V *>(p + i);
#pragma unroll
    for (int q = 0; q < kN * 4 / kB; ++q) {
      V t;
      memcpy(&t, reinterpret_cast<const char *>(o) + kB * q, kB);
      v[q] = t;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kN; ++k)
      if (k < nv) p[i + k] = o[k];
  }
}

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a += partial result of some launches of row g, one lane at a time
// (device-scope atomics; only for what a block cannot keep)
__device__ __forceinline__ void acc_to_table(PartRow *acc, uint32_t g, const Acc &a,
                                             uint32_t mx) {
  PartRow *r = acc + g;
  atomicAdd(&r->kc, a.kc);
  atomicAdd(&r->tns, a.tns);
  if (a.mc == 0) return;  // no counter row reached: every counter field is still zero
  atomicAdd(&r->mc, a.mc);
  atomicAdd(&r->mns, a.mns);
#pragma unroll
  for (int c = 0; c < OPATTR_NUM_COUNTERS; ++c) {
    if ((mx >> c) & 1u) atomicMax(&r->v[c], a.v[c]);
    else unsafeAtomicAdd(reinterpret_cast<double *>(&r->v[c]), bits2d(a.v[c]));
  }
  if (a.nan) atomicOr(&r->nan, a.nan);
}

// one lane's partial result to parts[x] (row g)
__device__ __forceinline__ void part_store(PartRow *parts, size_t x, uint32_t g, const Acc &a) {
  unsigned long long *d = reinterpret_cast<unsigned long long *>(parts + x);
  d[0] = a.kc;
  d[1] = a.tns;
  d[2] = a.mc;
  d[3] = a.mns;
#pragma unroll
  for (int c = 0; c < OPATTR_NUM_COUNTERS; ++c) d[4 + c] = a.v[c];
  d[24] = (unsigned long long)a.nan | ((unsigned long long)g << 32);
}

// a lane's partial result added into an LDS slot
__device__ __forceinline__ void slot_add(unsigned long long *q, const Acc &a, uint32_t mx) {
  atomicAdd(&q[0], a.kc);
  atomicAdd(&q[1], a.tns);
  if (a.mc == 0) return;  // no counter row reached
  atomicAdd(&q[2], a.mc);
  atomicAdd(&q[3], a.mns);
#pragma unroll
  for (int c = 0; c < OPATTR_NUM_COUNTERS; ++c) {
    if ((mx >> c) & 1u) atomicMax(&q[4 + c], a.v[c]);
    else unsafeAtomicAdd(reinterpret_cast<double *>(&q[4 + c]), bits2d(a.v[c]));
  }
  if (a.nan) atomicOr(reinterpret_cast<unsigned int *>(&q[24]), a.nan);
}

// What a block of an aggregation writes to: partials and records by bucket, in
// a region of fixed size, so that what a block keeps does not depend on the
// others.
struct RowOut {
  uint32_t NOPS, rb;  // rb: operator rows per bucket
  PartRow *acc;       // [G] row accumulators of the run reduction (zeroed)
  PartRow *parts;     // [blocks][pcap] kept partials, by bucket (row in pad)
  uint4 *rec;         // [blocks][rcap] launch records: row, match, duration, 0
  uint32_t *bkt;      // [blocks][kBktStride]
  uint32_t pcap, rcap;
  int longrow;        // launches of one row in a wave from which they are added up
};
// The row-ordered reduction adds up a stretch of one row inside a wave if it
// has longrow launches or more; those of a shorter one are kept as records, and
// the combine reads their counters. So a block of n launches never has more
// than n / longrow partials, however many rows it holds, and its region holds
// whatever comes: 200 / longrow + 16 bytes a launch. (A common room for all
// blocks' partials fills in another order on each run, and what finds none left
// has to be added by atomics.)
template <int kPer>
struct RowLds {
  uint2 md[kRThreads * kPer];     // match and duration, in row order
  uint16_t sg[kRThreads * kPer];  // row, in row order
  uint32_t hx[kRThreads];         // partials << 16 | records before each thread's positions
  uint8_t lms[kRThreads];         // bit k: a long stretch starts at the thread's position k
  uint8_t rms[kRThreads];         // bit k: the launch there is a record
  uint8_t ord[kRThreads / OPA_WAVE][OPA_WAVE];
  uint32_t sh[4], turn;
};
constexpr int kMidLanes = 6;  // lanes inside one row above which they are added up first

// The waves of a block that add to one LDS array do so in turns, so that the
// order does not depend on scheduling. A wave that waits for its turn waits for
// waves of its own block only, which run and end their turns without waiting
// for later ones. The adds are atomic in any order; a wave's LDS instructions
// execute in order, so the next wave's come after them without a wait for
// their completion.
__device__ __forceinline__ void turn_begin(uint32_t *turn, uint32_t mine) {
  while (__hip_atomic_load(turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != mine) {
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void turn_end(uint32_t *turn, uint32_t mine) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  if (lane_id() == 0)
    __hip_atomic_store(turn, mine + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The reduction of one block of launches (the thread's kPer consecutive ones:
// match mt, duration du, row g, nv of them exist; nb in the block), by a
// whole block of kRThreads. raw: r_agg_lds bytes, its first r_hist_words
// words zeroed.
template <bool DEF, int kPer>
__device__ __forceinline__ void row_order_block(const RowOut &o, const AggIn &in, int64_t blk,
                                                int nb, int nv, const int32_t (&mt)[kPer],
                                                const uint32_t (&du)[kPer],
                                                const uint32_t (&g)[kPer], unsigned char *raw,
                                                RowLds<kPer> &lds) {
  uint32_t *hist = reinterpret_cast<uint32_t *>(raw);  // two rows a word
  unsigned long long *slots = reinterpret_cast<unsigned long long *>(raw);
  auto &md = lds.md;
  auto &sg = lds.sg;
  auto &hx = lds.hx;
  auto &sh = lds.sh;
  const int tid = threadIdx.x, ln = lane_id(), w = wave_id();
  const uint32_t mx = DEF ? kDefMaxMask : in.maxmask, dw = DEF ? kDefDwMask : in.dwmask;
  const uint32_t words = r_hist_words(o.NOPS + 1u);
  uint32_t rk[kPer];
  if (tid == 0) lds.turn = 0;
  __syncthreads();
  // rank of every launch in its row: one atomic per run of the thread, the
  // waves in turns (in whatever order they come, the last bits of a row's sums
  // differ from run to run)
  turn_begin(&lds.turn, (uint32_t)w);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (k >= nv) continue;
    if (k > 0 && g[k] == g[k - 1]) {
      rk[k] = rk[k - 1] + 1u;
      continue;
    }
    uint32_t len = 1;
#pragma unroll
    for (int j = 1; j < kPer; ++j)
      if (k + j < nv && len == (uint32_t)j && g[k + j < kPer ? k + j : 0] == g[k]) ++len;
    const int s16 = (int)(g[k] & 1u) * 16;
    rk[k] = (atomicAdd(&hist[g[k] >> 1], len << s16) >> s16) & 0xFFFFu;
  }
  turn_end(&lds.turn, (uint32_t)w);
  __syncthreads();
  // first position of every row: each thread scans a stretch of the words
  // (an odd count of them, so that the stretches start in different banks)
  const uint32_t ch = ((words + kRThreads - 1) / kRThreads) | 1u;
  const uint32_t wlo = tid * ch, whi = wlo + ch < words ? wlo + ch : words;
  uint32_t mine = 0;
  for (uint32_t x = wlo; x < whi; ++x) mine += (hist[x] & 0xFFFFu) + (hist[x] >> 16);
  uint32_t run = block_excl_scan_add<uint32_t>(mine, sh, nullptr);
  for (uint32_t x = wlo; x < whi; ++x) {
    const uint32_t v = hist[x];
    hist[x] = run | ((run + (v & 0xFFFFu)) << 16);
    run += (v & 0xFFFFu) + (v >> 16);
  }
  __syncthreads();
  auto row_pos = [&](uint32_t r) -> uint32_t {  // first position of row r (r <= NOPS)
    return (hist[r >> 1] >> ((r & 1u) * 16)) & 0xFFFFu;
  };
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    if (k < nv) {
      const uint32_t p = row_pos(g[k]) + rk[k];
      md[p] = make_uint2((uint32_t)mt[k], du[k]);
      sg[p] = (uint16_t)g[k];
    }
  // position at which this thread's bucket starts (kBuckets threads), and the
  // unattributed row's first
  static_assert(kBuckets == kRThreads, "a bucket per thread");
  const uint32_t bl = (uint32_t)tid * o.rb;
  const uint32_t p_lo = row_pos(bl < o.NOPS ? bl : o.NOPS);
  const uint32_t p_un = row_pos(o.NOPS);
  __syncthreads();  // the histogram's space becomes the slots
  // row starts among the thread's positions (a wave's first position is one),
  // and those of long stretches: their row goes on longrow - 1 positions
  // later, in the same wave
  const int p0 = tid * kPer;
  const int we = (w + 1) * OPA_WAVE * kPer < nb ? (w + 1) * OPA_WAVE * kPer : nb;
  const int np = nb - p0 < 0 ? 0 : (nb - p0 < kPer ? nb - p0 : kPer);
  uint32_t hm = 0, lm = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int p = p0 + k, pl = p + o.longrow - 1;
    if (p < nb && ((ln == 0 && k == 0) || sg[p] != sg[p - 1])) {
      hm |= 1u << k;
      if (pl < we && sg[pl] == sg[p]) lm |= 1u << k;
    }
  }
  // is the stretch that goes on at the thread's first position a long one? (it
  // started at the last row start of the nearest lane below that has one)
  const unsigned long long hl = __ballot(hm != 0);
  const unsigned long long ll = __ballot(hm != 0 && lm > (hm >> 1));
  const unsigned long long below = hl & lanemask_lt();
  const int from = below ? 63 - __clzll((long long)below) : 0;
  const bool cont = (ll >> from) & 1ull;
  uint32_t rm = 0;  // the launches of short stretches
  {
    bool lg = cont;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if ((hm >> k) & 1u) lg = (lm >> k) & 1u;
      if (k < np && !lg) rm |= 1u << k;
    }
  }
  uint32_t all;  // partials << 16 | records
  const uint32_t h0 = block_excl_scan_add<uint32_t>(
      ((uint32_t)__popc(lm) << 16) | (uint32_t)__popc(rm), sh, &all);
  hx[tid] = h0;
  lds.lms[tid] = (uint8_t)lm;
  lds.rms[tid] = (uint8_t)rm;
  // the next lane goes on with this lane's last row; if that is a long stretch
  // started here, this lane has a slot for it
  const uint32_t np_n = __shfl_down((uint32_t)np, 1, OPA_WAVE), hm_n = __shfl_down(hm, 1, OPA_WAVE);
  const bool out = ln < OPA_WAVE - 1 && np_n > 0 && (hm_n & 1u) == 0;
  const bool mine_out = out && hm != 0 && lm > (hm >> 1);
  const unsigned long long live = __ballot(mine_out);
  const int nl = __popcll(live);
  unsigned long long *wslot = slots + (size_t)w * r_slots(kPer, o.longrow) * kFFields;
  for (int x = ln; x < nl * kFFields; x += OPA_WAVE) wslot[x] = 0;
  __syncthreads();
  auto kept_before = [&](uint32_t p) -> uint32_t {  // partials << 16 | records of positions below p
    const uint32_t t = p / kPer;
    if (t >= (uint32_t)kRThreads) return all;
    const uint32_t m = (1u << (p % kPer)) - 1u;
    return hx[t] + ((uint32_t)__popc(lds.lms[t] & m) << 16) + (uint32_t)__popc(lds.rms[t] & m);
  };
  {
    uint32_t *e = o.bkt + blk * kBktStride;
    e[tid] = kept_before(p_lo);
    if (tid == 0) {
      e[kBuckets] = kept_before(p_un);
      e[kBuckets + 1] = all;
    }
  }
  PartRow *parts = o.parts + blk * o.pcap;
  uint4 *rec = o.rec + blk * o.rcap + (h0 & 0xFFFFu);
  unsigned long long *mine_slot = wslot + __popcll(live & lanemask_lt()) * kFFields;
  unsigned long long *from_slot = wslot + __popcll(live & ((1ull << from) - 1ull)) * kFFields;
  Acc acc;  // of the long stretch the lane is in, else zero
  acc_zero(acc);
  bool here = false;       // the stretch started in this lane
  bool lg = cont;          // it is a long one
  uint32_t hi = h0 >> 16;  // partials before it
  uint32_t gc = 0;
  auto flush_inside = [&]() {  // a long stretch that ends in this lane
    if (!here) slot_add(from_slot, acc, mx);
    else part_store(parts, hi, gc, acc);
  };
#pragma unroll 1
  for (int k = 0; k < kPer; ++k) {
    if (k >= np) break;
    if ((hm >> k) & 1u) {
      if (k > 0 && lg) {
        flush_inside();
        acc_zero(acc);
        if (here) ++hi;
      }
      here = true;
      lg = (lm >> k) & 1u;
      gc = sg[p0 + k];
    }
    const uint2 e = md[p0 + k];
    if (lg) acc_launch(acc, in, (int32_t)e.x, e.y, mx, dw);
    else *rec++ = make_uint4(sg[p0 + k], e.x, e.y, 0u);
  }
  // lanes inside one row: where they are many, they are added up across the
  // lanes first (LDS atomics on one address go one after the other), and the
  // last one adds their total to the slot of the lane the row starts in
  const bool mid = np > 0 && hm == 0 && lg;
  if (__popcll(__ballot(mid)) >= kMidLanes) {
    acc_seg_scan(acc, hm != 0 ? ln : from, mx);
    const bool last = ln == OPA_WAVE - 1 || np_n == 0 || hm_n != 0;
    if (np > 0 && lg && last) {
      if (mid) slot_add(from_slot, acc, mx);
      else if (mine_out) slot_add(mine_slot, acc, mx);
      else flush_inside();
    }
  } else if (np > 0 && lg) {
    if (mine_out) slot_add(mine_slot, acc, mx);
    else flush_inside();
  }
  uint8_t *ord = lds.ord[w];  // the live lanes in order
  if (mine_out) ord[__popcll(live & lanemask_lt())] = (uint8_t)ln;
  wave_sync_lds();
  // the crossing rows, coalesced: consecutive lanes take consecutive fields
  for (int x = ln; x < nl * kFFields; x += OPA_WAVE) {
    const int r = x / kFFields, f = x - r * kFFields, s = ord[r];
    const int st = w * OPA_WAVE + s;  // its thread: the slot's row is the thread's last start
    const uint32_t ls = lds.lms[st];
    const uint32_t sk = 31u - (uint32_t)__clz((int)ls);
    const uint32_t row = sg[st * kPer + (int)sk];
    const uint32_t idx = (hx[st] >> 16) + (uint32_t)__popc(ls) - 1u;
    const unsigned long long v = wslot[x];
    reinterpret_cast<unsigned long long *>(parts + idx)[f] =
        f < 24 ? v : ((v & 0xFFFFFFFFull) | ((unsigned long long)row << 32));
  }
}

constexpr int kTThreads = 1024;
constexpr int kTHot = 12;   // lanes of one row above which they are reduced first
constexpr int kTSegs = 40;  // stretches of lanes of one row up to which they are scanned

// A wave's adds to the table: its lanes with want set add acc to row g, and lane
// 0 adds hot to row gh if with_hot is set. The fields go in kTurns groups with a
// turn each, so that the next wave adds a group's fields while this one adds the
// following group's: 300k launches over 700 rows 93 us the call by one turn for
// all fields, 85 by four, 85 without an order.
constexpr int kTurns = 4;  // a count and five counters each
__device__ __forceinline__ void tab_turns(unsigned long long *tab, uint32_t *turn, uint32_t mine,
                                          bool want, uint32_t g, const Acc &acc, bool with_hot,
                                          uint32_t gh, const Acc &hot, uint32_t mx) {
  constexpr int kEach = OPATTR_NUM_COUNTERS / kTurns;
  static_assert(kTurns == 4 && kEach * kTurns == OPATTR_NUM_COUNTERS, "groups of fields");
#pragma unroll
  for (int t = 0; t < kTurns; ++t) {
    auto add = [&](unsigned long long *q, const Acc &a) {
      const unsigned long long n = t == 0 ? a.kc : t == 1 ? a.tns : t == 2 ? a.mc : a.mns;
      if (t < 2 || a.mc) atomicAdd(&q[t], n);
      if (a.mc == 0) return;  // no counter row reached
#pragma unroll
      for (int c = t * kEach; c < (t + 1) * kEach; ++c) {
        if ((mx >> c) & 1u) atomicMax(&q[4 + c], a.v[c]);
        else unsafeAtomicAdd(reinterpret_cast<double *>(&q[4 + c]), bits2d(a.v[c]));
      }
      if (t == kTurns - 1 && a.nan) atomicOr(reinterpret_cast<unsigned int *>(&q[24]), a.nan);
    };
    turn_begin(turn + t, mine);
    if (with_hot && lane_id() == 0) add(tab + (size_t)gh * kFFields, hot);
    if (want) add(tab + (size_t)g * kFFields, acc);
    turn_end(turn + t, mine);
  }
}

// The thread's kPer consecutive launches (nv of them exist) added to the
// block's table in LDS, in turns, so that a row's sums are added up in one
// order: turn r * waves + w is wave w's r-th. Called by the whole block, kPer
// turns a wave from turn t0 * waves on.
template <bool DEF, int kPer>
__device__ __forceinline__ void tab_add(unsigned long long *tab, uint32_t *turn, uint32_t t0,
                                        const AggIn &in, int nv, int32_t (&mt)[kPer],
                                        uint32_t (&du)[kPer], uint32_t (&g)[kPer]) {
  constexpr uint32_t kWaves = kTThreads / OPA_WAVE;
  const uint32_t mx = DEF ? kDefMaxMask : in.maxmask, dw = DEF ? kDefDwMask : in.dwmask;
  const int ln = lane_id();
  uint32_t my = t0 * kWaves + (uint32_t)wave_id();
  Acc acc;
  acc_zero(acc);
  const uint32_t g0 = g[0];
  uint32_t gc = g0;
  bool changed = false;
  // launch k is always at position 0 of the arrays (see k_f_agg)
#pragma unroll 1
  for (int k = 0; k < kPer; ++k) {
    if (k > 0) {
      const bool flush = k < nv && g[0] != gc;
      tab_turns(tab, turn, my, flush, gc, acc, false, 0, acc, mx);
      my += kWaves;
      if (flush) {
        acc_zero(acc);
        gc = g[0];
        changed = true;
      }
    }
    if (k < nv) acc_launch(acc, in, mt[0], du[0], mx, dw);
#pragma unroll
    for (int j = 0; j + 1 < kPer; ++j) {
      mt[j] = mt[j + 1];
      du[j] = du[j + 1];
      g[j] = g[j + 1];
    }
  }
  // Each lane's last piece. Neighbouring lanes of one row are added up across
  // the lanes first (a lane belongs to the one before it when it holds only
  // that lane's last row): with LDS atomics alone, lanes of one row go one
  // after the other, 24 fields each. Launches in an order of their own have
  // few neighbours; a row that many lanes hold is then reduced on its own.
  const uint32_t gp = __shfl_up(gc, 1, OPA_WAVE);
  const bool start = ln == 0 || changed || nv == 0 || g0 != gp;
  const unsigned long long sm = __ballot(start);
  const unsigned long long act = __ballot(nv > 0);
  bool add = nv > 0;
  Acc hot;
  bool with_hot = false;
  uint32_t gm = 0;
  if (__popcll(sm & act) <= kTSegs) {
    const unsigned long long upto = ln == OPA_WAVE - 1 ? sm : sm & ((2ull << ln) - 1);
    acc_seg_scan(acc, 63 - __clzll((long long)upto), mx);
    const bool last = ln == OPA_WAVE - 1 || ((sm >> (ln + 1)) & 1ull);
    add = add && last;
  } else {
    gm = (uint32_t)__builtin_amdgcn_readlane((int)gc, 31);
    const bool in_hot = nv > 0 && gc == gm;
    with_hot = __popcll(__ballot(in_hot)) >= kTHot;
    if (with_hot) {
      hot = acc;
      if (!in_hot) acc_zero(hot);
      acc_wave_reduce(hot, mx);
      add = add && !in_hot;
    }
  }
  tab_turns(tab, turn, my, add, gc, acc, with_hot, gm, hot, mx);
}

__device__ __forceinline__ unsigned long long merge_field(int f, unsigned long long x,
                                                          unsigned long long y, uint32_t mx) {
  if (f < 4) return x + y;
  if (f < 24) return ((mx >> (f - 4)) & 1u) ? (x > y ? x : y) : d2bits(bits2d(x) + bits2d(y));
  return x | y;
}

// field f of kN (a power of two) partial results added up in pairs, so that a
// sum takes log2(kN) roundings and not one after the other
template <int kN>
__device__ __forceinline__ unsigned long long merge_tree(int f, unsigned long long (&v)[kN],
                                                         uint32_t mx) {
  static_assert((kN & (kN - 1)) == 0, "pairs");
  const bool count = f < 4, most = f >= 4 && f < 24 && ((mx >> (f - 4)) & 1u), sum = !most && f < 24;
  if (count) {
#pragma unroll
    for (int k = 1; k < kN; ++k) v[0] += v[k];
  } else if (most) {
#pragma unroll
    for (int k = 1; k < kN; ++k) v[0] = v[k] > v[0] ? v[k] : v[0];
  } else if (sum) {
#pragma unroll
    for (int o = kN / 2; o > 0; o >>= 1)
#pragma unroll
      for (int k = 0; k < o; ++k) v[k] = d2bits(bits2d(v[k]) + bits2d(v[k + o]));
  } else {
#pragma unroll
    for (int k = 1; k < kN; ++k) v[0] |= v[k];
  }
  return v[0];
}

// output field o (four counts, then the counters) of a row from its 25
// accumulated fields p
__device__ __forceinline__ unsigned long long row_field(const unsigned long long *p, int o,
                                                        uint32_t absent, uint32_t mx, uint32_t dw) {
  if (o < 4) return p[o];
  const int c = o - 4;
  const unsigned long long qnan = 0x7FF8000000000000ull;
  if (((absent >> c) & 1u) || p[2] == 0) return qnan;
  if ((mx >> c) & 1u) return (((uint32_t)p[24] >> c) & 1u) ? qnan : d2bits((double)key2f((uint32_t)p[o]));
  if ((dw >> c) & 1u) return p[3] ? d2bits(bits2d(p[o]) / (double)p[3]) : qnan;
  return p[o];
}

// t (one field f of an LDS row) += the field's value x
__device__ __forceinline__ void field_add(unsigned long long *t, int f, unsigned long long x,
                                          uint32_t mx) {
  if (f < 4) {
    atomicAdd(t, x);
  } else if (f < 24) {
    if ((mx >> (f - 4)) & 1u) atomicMax(t, x);
    else unsafeAtomicAdd(reinterpret_cast<double *>(t), bits2d(x));
  } else if ((uint32_t)x) {
    atomicOr(reinterpret_cast<unsigned int *>(t), (uint32_t)x);
  }
}


struct CombParams {
  int64_t nblocks;
  uint32_t rb, G, NOPS;
  uint32_t mx, dw, absent;
  const PartRow *parts;
  const uint4 *rec;            // launch records, or NULL: there are none
  const uint32_t *bkt;
  uint32_t pcap, rcap;         // of a block (see RowOut)
  AggIn in;                    // the records' counters
  PartRow *split;              // [kBuckets][nsplit][rb]
  int nsplit;                  // shares of the blocks per bucket
  PartRow *hot;                // [kHot] the unattributed row's shares
  const PartRow *acc;          // [G] row accumulators (the run reduction's overflow)
  opattr_op_row *table;
  unsigned long long *part;    // [kBuckets][4] summary sums per bucket
  // the finalisation, by the last block of the per-row reduction to finish
  uint32_t *done;              // blocks finished (zero at launch)
  opattr_diag *diag;
  const uint8_t *sflag;        // [ns] per-stream crossing flags
  uint32_t ns;
  opattr_summary *sum;
};

constexpr int kList = 512;                     // entries a combine wave lists in LDS at once
constexpr int kBatch = 8;                      // loads per lane in flight

// Partials added into an LDS table of rb rows field by field: 25 lanes read the
// fields of one, two partials an instruction, so that a partial costs two cache
// lines of requests instead of 25. at(x) gives the place of entry x, or kNoEntry.
constexpr uint32_t kNoEntry = 0xFFFFFFFFu;
struct CombParts {
  static constexpr int kEach = 2;  // entries an instruction takes
  template <int kN, typename At>
  static __device__ __forceinline__ void add(unsigned long long *tab, uint32_t rb,
                                             const CombParams &a, At at, uint32_t mx, uint32_t) {
    const int ln = lane_id(), f = ln & 31;
    const unsigned long long *parts64 = reinterpret_cast<const unsigned long long *>(a.parts);
    unsigned long long v[kN];
    bool ok[kN];
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      const uint32_t x = at(2 * j + (ln >> 5));
      ok[j] = x != kNoEntry && f < kFFields;
      v[j] = ok[j] ? parts64[(size_t)x * (sizeof(PartRow) / 8) + f] : 0ull;
    }
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      const uint32_t g = (uint32_t)(__shfl(v[j], (ln & 32) + 24, OPA_WAVE) >> 32);
      if (ok[j]) field_add(tab + (size_t)(g % rb) * kFFields + f, f, v[j], mx);
    }
  }
};

// Launch records: five lanes each read four counters of the launch's row and add
// them, twelve records an instruction.
struct CombRecs {
  static constexpr int kEach = 12;
  template <int kN, typename At>
  static __device__ __forceinline__ void add(unsigned long long *tab, uint32_t rb,
                                             const CombParams &a, At at, uint32_t mx,
                                             uint32_t dw) {
    const int ln = lane_id(), sub = ln / 5, q = ln - sub * 5;
    uint4 r[kN];
    float4 v[kN];
    bool ok[kN], hit[kN];
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      const uint32_t x = sub < kEach ? at(kEach * j + sub) : kNoEntry;
      ok[j] = x != kNoEntry;
      r[j] = ok[j] ? a.rec[x] : make_uint4(0u, 0xFFFFFFFFu, 0u, 0u);
    }
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      const int32_t m = (int32_t)r[j].y;
      hit[j] = m >= 0 && (int64_t)m < a.in.P;
      v[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (!hit[j]) continue;
      const float *row = a.in.counters + (int64_t)m * a.in.rs;
      if (a.in.vec4) {
        v[j] = reinterpret_cast<const float4 *>(row)[q];
      } else {
        const int64_t c = 4 * q;
        v[j] = make_float4(row[c * a.in.cs], row[(c + 1) * a.in.cs], row[(c + 2) * a.in.cs],
                           row[(c + 3) * a.in.cs]);
      }
    }
#pragma unroll
    for (int j = 0; j < kN; ++j) {
      if (!ok[j]) continue;
      unsigned long long *t = tab + (size_t)(r[j].x % rb) * kFFields;
      if (q < 2 || (q < 4 && hit[j])) atomicAdd(t + q, (unsigned long long)((q & 1) ? r[j].z : 1u));
      if (!hit[j]) continue;
      const float w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
      const double d = (double)r[j].z;
#pragma unroll
      for (int k = 0; k < 4; ++k) {  // as acc_launch
        const int c = 4 * q + k;
        if ((mx >> c) & 1u) {
          atomicMax(t + 4 + c, (unsigned long long)f2key(w[k]));
          if (w[k] != w[k]) atomicOr(reinterpret_cast<unsigned int *>(t + 24), 1u << c);
        } else {
          const double x = (double)w[k];
          unsafeAtomicAdd(reinterpret_cast<double *>(t + 4 + c), ((dw >> c) & 1u) ? x * d : x);
        }
      }
    }
  }
};

// The entries of a wave's blocks in a bucket (per lane kPre blocks: ev entries
// from xv on, mine in all) added into an LDS table: listed in LDS, then some of
// them at a time.
template <typename Comb, int kN, int kPre>
__device__ __forceinline__ void comb_add(unsigned long long *tab, uint32_t rb, uint32_t *list,
                                         const CombParams &a, const uint32_t (&ev)[kPre],
                                         const uint32_t (&xv)[kPre], uint32_t mine, uint32_t mx,
                                         uint32_t dw) {
  const uint32_t incl = wave_incl_scan_add<uint32_t>(mine);
  const uint32_t n = __shfl(incl, OPA_WAVE - 1, OPA_WAVE);
  if (n == 0) return;
  if (n <= (uint32_t)kList) {
    uint32_t w = incl - mine;
#pragma unroll
    for (int k = 0; k < kPre; ++k) {
      for (uint32_t p = 0; p < ev[k]; ++p) list[w++] = xv[k] + p;
    }
    wave_sync_lds();
    for (uint32_t i = 0; i < n; i += Comb::kEach * kN)
      Comb::template add<kN>(tab, rb, a, [&](int x) -> uint32_t {
        return i + x < n ? list[i + x] : kNoEntry;
      }, mx, dw);
    wave_sync_lds();  // the list is free again
  } else {
    // more than the list holds: one lane's blocks at a time
#pragma unroll 1
    for (int k = 0; k < kPre; ++k) {
      uint32_t e = 0, xe = 0;
#pragma unroll
      for (int j = 0; j < kPre; ++j) {
        e = k == j ? ev[j] : e;
        xe = k == j ? xv[j] : xe;
      }
      for (uint64_t m = __ballot(e != 0); m; m &= m - 1) {
        const int src = __ffsll((unsigned long long)m) - 1;
        const uint32_t c = __shfl(e, src, OPA_WAVE);
        const uint32_t x0 = __shfl(xe, src, OPA_WAVE);
        for (uint32_t p = 0; p < c; p += Comb::kEach * 2)
          Comb::template add<2>(tab, rb, a, [&](int x) -> uint32_t {
            return p + x < c ? x0 + p + x : kNoEntry;
          }, mx, dw);
      }
    }
  }
}

// A wave adds the partials and records of bucket q in the blocks b0 + lane + 64 k.
template <int kPre>
__device__ __forceinline__ void comb_blocks(unsigned long long *tab, uint32_t rb, uint32_t *list,
                                            const CombParams &a, uint32_t q, int64_t b0,
                                            int64_t b_hi, uint32_t mx, uint32_t dw) {
  uint32_t e0[kPre], e1[kPre], ev[kPre], xv[kPre], mine = 0;
#pragma unroll
  for (int k = 0; k < kPre; ++k) {
    const int64_t b = b0 + lane_id() + (int64_t)OPA_WAVE * k;
    const uint32_t *e = a.bkt + b * kBktStride + q;
    e0[k] = b < b_hi ? e[0] : 0u;
    e1[k] = b < b_hi ? e[1] : 0u;
  }
#pragma unroll
  for (int k = 0; k < kPre; ++k) {
    const int64_t b = b0 + lane_id() + (int64_t)OPA_WAVE * k;
    ev[k] = (e1[k] >> 16) - (e0[k] >> 16);
    xv[k] = (uint32_t)b * a.pcap + (e0[k] >> 16);
    mine += ev[k];
  }
  comb_add<CombParts, kBatch>(tab, rb, list, a, ev, xv, mine, mx, dw);
  if (!a.rec) return;
  mine = 0;
#pragma unroll
  for (int k = 0; k < kPre; ++k) {
    const int64_t b = b0 + lane_id() + (int64_t)OPA_WAVE * k;
    ev[k] = (e1[k] & 0xFFFFu) - (e0[k] & 0xFFFFu);
    xv[k] = (uint32_t)b * a.rcap + (e0[k] & 0xFFFFu);
    mine += ev[k];
  }
  comb_add<CombRecs, kBatch / 2>(tab, rb, list, a, ev, xv, mine, mx, dw);
}

// The blocks' tables added up, kTRows rows a block (one element per thread
// and share of the tables), and the table rows. With kLast the blocks also
// leave their summary sums and the last one to finish writes the summary and
// the status; without, the launches' blocks left the sums (a.part) and the
// block after the rows' does that.
constexpr int kTRows = 4, kTShares = 10;
static_assert(kTRows * kFFields * kTShares <= 1024, "one block");

template <bool DEF, bool kLast>
__global__ void __launch_bounds__(1024) k_t_rows(CombParams a, const unsigned long long *tabs,
                                                 int ntabs) {
  constexpr int kEl = kTRows * kFFields;
  if (!kLast && blockIdx.x * kTRows >= a.G) {
    finish_block(a.diag, a.sflag, a.ns, a.part, ntabs, a.sum);
    return;
  }
  __shared__ unsigned long long part[kTShares][kEl];
  __shared__ unsigned long long red[4][kTRows];
  const uint32_t mx = DEF ? kDefMaxMask : a.mx, dw = DEF ? kDefDwMask : a.dw;
  const int tid = threadIdx.x, sh = tid / kEl, e = tid - sh * kEl, f = e % kFFields;
  const uint32_t g0 = blockIdx.x * kTRows, ne = a.G * kFFields;
  const uint32_t x = g0 * kFFields + e;
  if (sh < kTShares && x < ne) {
    unsigned long long v = 0;
    constexpr int kB = 16;
    for (int t0 = sh; t0 < ntabs; t0 += kTShares * kB) {
      unsigned long long y[kB];
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        const int t = t0 + j * kTShares;
        y[j] = t < ntabs ? tabs[(size_t)t * ne + x] : 0ull;
      }
      v = ntabs > kTShares ? merge_field(f, v, merge_tree(f, y, mx), mx) : y[0];
    }
    part[sh][e] = v;
  }
  __syncthreads();
  if (tid < kEl && x < ne) {
    unsigned long long y[16];
    static_assert(kTShares <= 16, "all shares");
#pragma unroll
    for (int s = 0; s < 16; ++s) y[s] = s < kTShares ? part[s][tid] : 0ull;
    part[0][tid] = merge_tree(f, y, mx);
  }
  __syncthreads();
  // 24 output fields a row
  if (tid < kTRows * 24) {
    const int r = tid / 24, o = tid - r * 24;
    const uint32_t g = g0 + r;
    if (g < a.G) {
      const unsigned long long *p = part[0] + r * kFFields;
      unsigned long long *row = reinterpret_cast<unsigned long long *>(a.table + g);
      row[o] = row_field(p, o, a.absent, mx, dw);
      if (o == 0) {
        red[0][r] = g < a.NOPS ? p[1] : 0ull;
        red[1][r] = g < a.NOPS ? 0ull : p[1];
        red[2][r] = p[1];
        red[3][r] = p[3];
      }
    } else if (o == 0) {
      red[0][r] = red[1][r] = red[2][r] = red[3][r] = 0;
    }
  }
  if (!kLast) return;
  __syncthreads();
  if (tid < 4) {
    unsigned long long v = 0;
    for (int r = 0; r < kTRows; ++r) v += red[tid][r];
    a.part[blockIdx.x * 4 + tid] = v;
  }
  __shared__ uint32_t last;
  if (tid < OPA_WAVE) {
    __threadfence();
    uint32_t l = 0;
    if (tid == 0) l = atomicAdd(a.done, 1u) == gridDim.x - 1 ? 1u : 0u;
    l = __shfl(l, 0);
    if (l) __threadfence();
    if (tid == 0) last = l;
  }
  __syncthreads();
  if (!last) return;
  finish_block(a.diag, a.sflag, a.ns, a.part, (int)gridDim.x, a.sum);
}

}  // namespace opa
